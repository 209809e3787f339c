"""The matrix-core kernel (frequencies over which the shape factor is one constant) at the edges of
its tiles -- 16-frequency rows, groups of 256, one to four groups per wave and more than one
frequency group, chunks of 64 and steps of 16 particles, odd numbers of directions -- against
the FP64 oracle.  Tolerances: the spectra's gate 1e-4, and 4e-6 of the largest intensity: each
factor of a term is a 22-bit number and its sign from a hardware sin (1.1e-7) of a phase rounded to 24 bits
(1.9e-7 rad), so |S| is off by at most about 1.1e-6 of the sum of the terms' sizes and I by
twice that where they add up, with FP32 sums of at most 1024 particles on top (4e-7)."""
import numpy as np
import pytest

import oracle
from workloads import SINGLE, TINY, flatten
from tests.helpers import assert_parity, step_slice, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rad():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1802_03972_amd as rad
    from paper_1802_03972_amd.build import ensure_built
    ensure_built()    # a built library is used as is
    rad._lib.lib()
    return rad


def check(rad, n, nx, ny, n_omega, shape="point", dtype="f32", steps=1, omega0=0.0, t0=0.0, shape_len=1e-7, omega_max=1e19,
          call="push_steps"):
    w = SINGLE.scaled(n_particles=n, n_steps=steps, nx_dir=nx, ny_dir=ny, n_omega=n_omega, seed=101, in_dtype=dtype,
                      t0=t0, omega_max=omega_max)
    st = w.steps()
    g = rad.Grid(w.directions(), omega0, w.domega, n_omega, shape=shape, shape_len=shape_len, dt=w.dt)
    dev = to_device(st, dtype)
    if call == "push_steps":
        g.push_steps(t0, steps, dev)
    else:
        for k, t in enumerate(w.times()):
            getattr(g, call)(float(t), step_slice(dev, k, n))
    om = omega0 + np.arange(n_omega) * w.domega
    ref = oracle.spectrum(flatten(st, w.times()), w.directions(), om, shape, shape_len, w.dt)
    I = g.spectrum()
    rep = assert_parity(I, ref, f"{n} x {steps}, {nx * ny} x {n_omega} {shape} {dtype}")
    assert rep["e_inf"] <= 4e-6, rep
    return g, I


@pytest.mark.parametrize("n_omega", [240, 255, 256, 257, 272, 511, 512, 640, 768, 1000, 1024, 1025, 1300, 2049])
def test_frequency_edges(rad, n_omega):
    check(rad, 100, 2, 3, n_omega)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 80, 129, 1000, 5000])
def test_particle_edges(rad, n):
    check(rad, n, 5, 1, 256)


@pytest.mark.parametrize("nx,ny", [(1, 1), (3, 1), (4, 1), (7, 1), (8, 2), (8, 16)])
def test_directions(rad, nx, ny):
    check(rad, 70, nx, ny, 300, dtype="f64")


# a Gaussian is zero from a frequency on: the general kernel takes the blocks below
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n_omega,omega_max", [(256, 1e19), (1000, 1e19), (1024, 1e18), (300, 2e17)])
def test_gauss_in_two_parts(rad, n_omega, omega_max, dtype):
    check(rad, 333, 3, 5, n_omega, shape="gauss", dtype=dtype, omega_max=omega_max)


# 1 to 4 first frequencies beside the constant are summed apart, with 5 the general kernel takes 16;
# exp(-(omega L / c)^2) is zero in FP32 from omega L / c = 10.2 on
@pytest.mark.parametrize("n_omega", [256, 600])
@pytest.mark.parametrize("first", [1, 2, 3, 4, 5, 17])
def test_gauss_heads(rad, first, n_omega):
    step = 10.2 * 299792458.0 / 1e-7 / (first - 0.5)
    check(rad, 150, 3, 1, n_omega, shape="gauss", omega_max=step * (n_omega - 1))


@pytest.mark.parametrize("shape", ["point", "gauss"])
def test_steps_offsets_and_first_frequency(rad, shape):
    check(rad, 123, 3, 3, 520, shape=shape, dtype="f64", steps=5, t0=1e-12)
    check(rad, 123, 3, 3, 520, shape=shape, dtype="f64", steps=3, omega0=3e18)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["identical", "spread", "small", "large", "still"])
def test_sizes_of_terms(rad, kind, dtype):
    """Terms that all add up (one particle 6000 times: the error of every value is that of one
    term and of the sum's roundings, so the 4e-6 hold at each point and not only at the peak),
    sizes spread over many decades within each 64 particles, and sizes far from 1."""
    w = SINGLE.scaled(n_particles=6000, n_steps=1, nx_dir=2, ny_dir=2, n_omega=256, seed=103, in_dtype=dtype, omega_max=1e15)
    st = w.steps()
    rates = ("dbx", "dby", "dbz")
    if kind == "identical":
        st = {k: np.repeat(v[:, :1], v.shape[1], axis=1) for k, v in st.items()}
    else:
        scale = {"spread": np.exp(4 * np.random.default_rng(5).standard_normal(6000)), "small": 1e-12, "large": 1e12,
                 "still": 0.0}[kind]
        held = np.float32 if dtype == "f32" else np.float64
        st = {k: (v * scale).astype(held).astype(np.float64) if k in rates else v for k, v in st.items()}
    g = rad.Grid(w.directions(), 0.0, w.domega, 256, shape="point", shape_len=1e-7, dt=w.dt)
    g.push_steps(0.0, 1, to_device(st, dtype))
    I = g.spectrum()
    ref = oracle.spectrum(flatten(st, w.times()), w.directions(), np.arange(256) * w.domega, "point", 1e-7, w.dt)
    bound = ref if kind == "identical" else ref.max()
    assert (np.abs(I - ref) <= 4e-6 * bound).all(), (np.abs(I - ref) / np.maximum(bound, 1e-300)).max()


def test_long_push_in_several_splits(rad):
    check(rad, 3000, 2, 2, 512, steps=4)


@pytest.mark.parametrize("shape", ["point", "gauss"])
def test_push_forms_agree(rad, shape):
    """push_step, push_step_noalloc and push_steps of one step share plan and kernel."""
    I = [check(rad, 900, 4, 4, 600, shape=shape, call=c)[1] for c in ("push_step", "push_step_noalloc", "push_steps")]
    assert np.array_equal(I[0], I[1]) and np.array_equal(I[0], I[2])


def test_bad_particle_sets_the_flag(rad):
    w = TINY.scaled(n_particles=100, n_steps=1, n_omega=256)
    st = w.steps()
    for field, value in (("w", -1.0), ("x", np.nan), ("bz", 1.5)):
        bad = {k: v.copy() for k, v in st.items()}
        bad[field][0, 77] = value
        g = rad.Grid(w.directions(), 0.0, w.domega, 256, shape="point", shape_len=1e-7, dt=w.dt)
        g.push_step(0.0, to_device(bad, "f64"))
        with pytest.raises(rad.RadError):
            g.spectrum()
        g.reset()
        g.push_step(0.0, to_device(st, "f64"))
        assert np.isfinite(g.spectrum()).all()


def test_profile_counts_both_parts(rad):
    w = SINGLE.scaled(n_particles=500, n_steps=1, nx_dir=4, ny_dir=4, n_omega=512, seed=102)
    dev = to_device(w.steps(), "f32")
    g = rad.Grid(w.directions(), 0.0, w.domega, 512, shape="gauss", shape_len=1e-7, dt=w.dt)
    g.profile(2)
    for _ in range(4):
        g.push_step(0.0, dev)
    st = g.profile_read()
    assert st["updates"] == 2 * 500 * 16 * 512 and st["accumulate_ms"] > 0 and st["fold_ms"] > 0
