"""Pushes too small to fill the chip: the wave groups that share a chunk's particles, the shorter
splits below them and the balanced splits above, at the sizes where the split changes, for every
number of waves a tile may have and every kernel variant, against the FP64 oracle (gate 1e-4)."""
import numpy as np
import pytest

import oracle
from workloads import SINGLE, block_log_omegas, flatten
from tests.helpers import assert_parity, to_device

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


def check(rad, n, nx, ny, n_omega, shape="cic", dtype="f32", omegas=None, tile=None, steps=1, seed=91):
    w = SINGLE.scaled(n_particles=n, n_steps=steps, nx_dir=nx, ny_dir=ny, n_omega=n_omega, seed=seed, in_dtype=dtype)
    st = w.steps()
    g = rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape=shape, shape_len=w.shape_len, dt=w.dt,
                 omegas=omegas)
    if tile:
        g.set_tile(**tile)
    g.push_steps(0.0, steps, to_device(st, dtype))
    ref = oracle.spectrum(flatten(st, w.times()), w.directions(), w.omegas() if omegas is None else omegas, shape,
                          w.shape_len, w.dt)
    assert_parity(g.spectrum(), ref, f"{n} x {steps}, {nx * ny} x {n_omega} {shape} {tile or ''}")


# 16 x 64 points, 1024 splits: 8 to 32 particles a split, one to eight groups
@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 33, 1023, 1024, 1025, 4097, 8193, 16385, 32768, 32769, 40000])
def test_split_edges(rad, n):
    check(rad, n, 4, 4, 64)


# one split per workgroup: 128 splits of 31, 32, 33 and 65 particles
@pytest.mark.parametrize("n", [3968, 4096, 4097, 8200])
def test_balanced_splits(rad, n):
    check(rad, n, 8, 16, 256)


@pytest.mark.parametrize("w,dpw,waves", [(16, 16, 1), (16, 16, 2), (16, 16, 3), (16, 16, 4), (16, 16, 5), (16, 32, 8),
                                         (16, 64, 1), (16, 64, 3), (32, 16, 1), (32, 32, 2), (32, 64, 4)])
@pytest.mark.parametrize("n", [5, 700])
def test_tiles(rad, n, w, dpw, waves):
    check(rad, n, 6, 6, 100, tile=dict(w_per_lane=w, dir_per_wave=dpw, waves=waves, wg_per_cu=8))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,kind", [("gauss", "uniform"), ("tsc3d", "uniform"), ("cic", "log"), ("cic", "blocks"),
                                        ("cic3d", "log"), ("cic3d", "blocks")])
def test_variants(rad, shape, kind, dtype):
    n_omega = 75
    om = {"uniform": None, "log": np.geomspace(1e15, 1e19, n_omega), "blocks": block_log_omegas(1e15, 1e19, n_omega)}
    check(rad, 150, 3, 5, n_omega, shape=shape, dtype=dtype, omegas=om[kind], steps=3)


# grids that fill their tiles badly: the default launch shape's choices of directions per wave,
# of waves (one to eight, odd numbers too) and of frequency tiles
@pytest.mark.parametrize("nx,ny,n_omega,shape,kind", [
    (37, 1, 100, "cic", "uniform"), (8, 5, 600, "cic", "uniform"), (8, 16, 100, "tsc", "uniform"),
    (8, 3, 200, "gauss", "uniform"), (8, 11, 137, "cic3d", "uniform"), (8, 11, 137, "cic", "log"),
    (1, 1, 1000, "cic", "uniform"), (8, 16, 17, "cic", "blocks"), (1, 1, 1, "cic", "uniform")])
def test_default_launch_shapes(rad, nx, ny, n_omega, shape, kind):
    om = {"uniform": None, "log": np.geomspace(1e15, 1e19, n_omega), "blocks": block_log_omegas(1e15, 1e19, n_omega)}
    check(rad, 1200, nx, ny, n_omega, shape=shape, omegas=om[kind])


# fewer than 16 directions: the flexible build's pairs, slots, groups and frequency tiles
@pytest.mark.parametrize("n", [1, 3, 37, 1000, 6000])
@pytest.mark.parametrize("nx,ny,n_omega", [(1, 1, 5), (1, 1, 64), (1, 1, 1000), (2, 1, 241), (3, 1, 17), (5, 1, 130),
                                           (7, 1, 300), (8, 1, 40), (3, 5, 100), (3, 5, 700)])
def test_few_directions(rad, n, nx, ny, n_omega):
    check(rad, n, nx, ny, n_omega)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,kind", [("cic3d", "uniform"), ("cic", "log"), ("tsc", "blocks"), ("cic3d", "log"),
                                        ("cic3d", "blocks"), ("gauss", "uniform")])
@pytest.mark.parametrize("nx,n_omega", [(1, 300), (2, 40), (3, 77), (13, 150)])
def test_few_directions_variants(rad, nx, n_omega, shape, kind, dtype):
    om = {"uniform": None, "log": np.geomspace(1e15, 1e19, n_omega), "blocks": block_log_omegas(1e15, 1e19, n_omega)}
    check(rad, 500, nx, 1, n_omega, shape=shape, dtype=dtype, omegas=om[kind], steps=3)


def test_few_directions_all_fp32(rad):
    """The FP32 study mode through the flexible build equals the fixed tiles' result."""
    w = SINGLE.scaled(n_particles=300, n_steps=1, nx_dir=3, ny_dir=1, n_omega=90, seed=92, omega_max=1e15)
    dev = to_device(w.steps(), "f32")
    out = []
    for tile in (None, dict(w_per_lane=16, dir_per_wave=16, waves=2, wg_per_cu=2)):
        g = rad.Grid(w.directions(), 0.0, w.domega, 90, shape="cic", shape_len=1e-7, dt=w.dt, precision=rad.ALL_F32,
                     tile=tile)
        g.push_step(0.0, dev)
        out.append(g.spectrum())
    assert np.allclose(out[0], out[1], rtol=1e-4, atol=1e-6 * out[1].max())
