"""Read-outs of grids with few directions or few frequencies, whose tiles have another shape, against the
same points of a grid of 40 directions x 300 frequencies: per point the arithmetic is the same, so the
values are equal bit for bit.  And one direction with as many frequencies as a grid may have."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DIRS, OMEGAS = 40, 300


@pytest.fixture(scope="module")
def rad():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1802_03972_amd as rad
    from paper_1802_03972_amd.build import ensure_built
    ensure_built()    # a built library is used as is
    rad._lib.lib()
    return rad


def directions(n):
    a = np.linspace(-0.02, 0.03, n)
    return np.stack([a, 0.5 * a, np.sqrt(1.0 - 1.25 * a * a)], axis=1)


@pytest.fixture(scope="module")
def wide(rad):
    """State [omega][dir][4], intensity and complex spectrum of the wide grid."""
    S = np.random.default_rng(11).standard_normal((OMEGAS, DIRS, 4))
    g = rad.Grid(directions(DIRS), 0.0, 1e15, OMEGAS, shape="cic", shape_len=1e-7, dt=5e-17)
    g.set_state(S.ravel())
    I = g.spectrum()
    scale = I / (S.transpose(1, 0, 2) ** 2).sum(axis=2)      # one prefactor everywhere
    assert np.allclose(scale, scale[0, 0], rtol=1e-13)
    return S, I, g.spectrum_complex()


@pytest.mark.parametrize("n_dir,n_omega", [
    (1, 1), (1, 2), (1, 15), (1, 16), (1, 17), (1, 255), (1, 256), (1, 257), (1, 300), (2, 128), (2, 129), (3, 64), (3, 65),
    (4, 300), (5, 32), (5, 33), (8, 300), (9, 16), (9, 17), (15, 300), (16, 16), (16, 300), (17, 17), (40, 1), (40, 2), (40, 3),
    (33, 5), (40, 8), (40, 9), (40, 15), (40, 16), (15, 15), (7, 1)])
def test_narrow_grids(rad, wide, n_dir, n_omega):
    import torch
    S, I, Z = wide
    d0, k0 = 40 - n_dir, (300 - n_omega) // 2
    g = rad.Grid(directions(DIRS)[d0:], k0 * 1e15, 1e15, n_omega, shape="cic", shape_len=1e-7, dt=5e-17)
    g.set_state(np.ascontiguousarray(S[k0:k0 + n_omega, d0:]).ravel())
    out = torch.full((n_dir, n_omega), -1.0, dtype=torch.float64, device="cuda")
    g.spectrum_device(out)
    assert np.array_equal(g.spectrum(), I[d0:, k0:k0 + n_omega])
    assert np.array_equal(out.cpu().numpy(), I[d0:, k0:k0 + n_omega])
    assert np.array_equal(g.spectrum_complex(), Z[d0:, k0:k0 + n_omega])


def test_one_direction_and_the_most_frequencies(rad):
    """2^28 points in one row: a launch may have 2^32 - 1 threads, which 16 x 16 tiles would exceed."""
    import torch
    n = 1 << 28
    g = rad.Grid(directions(1), 0.0, 1e10, n, shape="point", shape_len=1e-7, dt=5e-17)
    out = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    g.spectrum_device(out)
    assert int(torch.count_nonzero(out)) == 0
    g.close()
