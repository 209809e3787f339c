"""Host and device read-outs of the same accumulator at the edges of the read-out kernels' 16 x 16
tiles and on both sides of the size up to which a host read-out goes through page-locked
memory (8 MB): bitwise the same intensity, the complex spectrum consistent with it, and no
output written when the data-error flag is set."""
import numpy as np
import pytest

from workloads import SINGLE
from tests.helpers import to_device

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


@pytest.mark.parametrize("nx,ny,n_omega", [(1, 1, 1), (1, 1, 17), (15, 1, 16), (17, 1, 33), (16, 1, 160), (3, 1, 1000),
                                           (16, 32, 400), (16, 32, 2047), (16, 32, 2049)])
def test_read_outs_agree(rad, nx, ny, n_omega):
    import torch
    w = SINGLE.scaled(n_particles=40, n_steps=1, nx_dir=nx, ny_dir=ny, n_omega=n_omega, seed=81)
    g = rad.Grid(w.directions(), w.omega0, w.domega, n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
    g.push_step(0.0, to_device(w.steps(), "f32"))
    out = torch.zeros(w.n_dir, n_omega, dtype=torch.float64, device="cuda")
    I, S = g.spectrum(), g.spectrum_complex()
    g.spectrum_device(out)
    assert np.array_equal(I, out.cpu().numpy())
    state = g.get_state().reshape(n_omega, w.n_dir, 4)
    amp = (state ** 2).sum(axis=2).T                          # |S1|^2 + |S2|^2
    assert I.max() > 0
    # a rotation of two components into three in FP64: a few roundings of each
    assert np.allclose((np.abs(S) ** 2).sum(axis=2), amp, rtol=1e-13, atol=1e-13 * amp.max())
    assert np.allclose(I / I.max(), amp / amp.max(), rtol=1e-13, atol=0)
    assert np.abs(np.einsum("dkc,dc->dk", S, w.directions())).max() <= 1e-12 * np.abs(S).max()


@pytest.mark.parametrize("n_omega", [64, 2049])
def test_bad_data_writes_nothing(rad, n_omega):
    import ctypes
    w = SINGLE.scaled(n_particles=40, n_steps=1, nx_dir=16, ny_dir=32, n_omega=n_omega, seed=82)
    dev = to_device(w.steps(), "f32")
    dev["w"][7] = -1.0
    g = rad.Grid(w.directions(), w.omega0, w.domega, n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
    g.push_step(0.0, dev)
    L = rad._lib.lib()
    out = np.full(w.n_dir * n_omega * 6, 7.0)
    p = out.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    for call in (L.rad_spectrum, L.rad_spectrum_complex):
        assert call(g.handle, p, None) == rad.RAD_ERR_BAD_DATA
        assert np.all(out == 7.0)
    g.reset()
    assert L.rad_spectrum(g.handle, p, None) == 0 and np.all(out[:w.n_dir * n_omega] == 0.0)
