"""A launch shape that is set runs the general kernel on all frequencies, also where the shape factor is
one constant; one that "auto" takes from the table of measured shapes leaves the matrix-core kernel in use."""
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


@pytest.mark.parametrize("shape", ["point", "gauss"])
@pytest.mark.parametrize("nx,ny,n_omega", [(4, 4, 64), (8, 8, 256), (8, 8, 1024)])   # sizes that the table has
def test_set_and_hinted_tiles(rad, nx, ny, n_omega, shape):
    w = SINGLE.scaled(n_particles=300, n_steps=1, nx_dir=nx, ny_dir=ny, n_omega=n_omega, seed=104)
    st = w.steps()
    dev = to_device(st, "f32")
    ref = oracle.spectrum(flatten(st, w.times()), w.directions(), w.omegas(), shape, w.shape_len, w.dt)
    I = {}
    for tile in (None, "auto", "set"):
        g = rad.Grid(w.directions(), w.omega0, w.domega, n_omega, shape=shape, shape_len=w.shape_len, dt=w.dt,
                     tile="auto" if tile else None)
        if tile == "set":
            g.set_tile()
            # the batched kernel with the same shape, which has no matrix-core route
            b = rad.Batcher(tile=g.get_tile())
            g2 = rad.Grid(w.directions(), w.omega0, w.domega, n_omega, shape=shape, shape_len=w.shape_len, dt=w.dt)
            b.push([(g2, 0.0, 1, dev)])
            I["batch"] = g2.spectrum()
        g.push_steps(0.0, 1, dev)
        I[tile] = g.spectrum()
        assert_parity(I[tile], ref, f"{nx * ny} x {n_omega} {shape}, tile {tile}")
    if n_omega > 64:
        assert np.array_equal(I["auto"], I[None])        # both on the matrix cores
        assert not np.array_equal(I["set"], I[None])
    # same terms from the same kernel; up to 300 of them summed in FP32 in another grouping
    assert np.abs(I["set"] - I["batch"]).max() <= 2e-6 * ref.max()
