"""Grids of fewer than 16 directions whose frequencies fill all eight waves of a workgroup once, where
the flexible build's chunks are of any length, odd ones too, against the FP64 oracle (gate 1e-4)."""
import numpy as np
import pytest

import oracle
from workloads import SINGLE, flatten
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


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,n_omega,kind,n", [(11, 529, "uniform", 13824), (11, 600, "uniform", 5003), (7, 1024, "uniform", 333),
                                               (11, 300, "log", 5003), (5, 800, "log", 2777), (15, 540, "uniform", 256)])
def test_odd_chunks(rad, nx, n_omega, kind, n, dtype):
    w = SINGLE.scaled(n_particles=n, n_steps=1, nx_dir=nx, ny_dir=1, n_omega=n_omega, seed=97, in_dtype=dtype)
    st = w.steps()
    om = np.geomspace(1e15, 1e19, n_omega) if kind == "log" else None
    g = rad.Grid(w.directions(), w.omega0, w.domega, n_omega, shape="cic", shape_len=w.shape_len, dt=w.dt, omegas=om)
    g.push_steps(0.0, 1, to_device(st, dtype))
    ref = oracle.spectrum(flatten(st, w.times()), w.directions(), w.omegas() if om is None else om, "cic", w.shape_len, w.dt)
    assert_parity(g.spectrum(), ref, f"{n} particles, {nx} x {n_omega} {kind} {dtype}")
