"""The fixed-order FP64 folds at the edges of their groups: numbers of particle splits around
the groups of one block, numbers of points on both sides of each dispatch line, and the
tracked read-out's groups of particles, each against the FP64 oracle (gate 1e-4)."""
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


def workload(n, nx, ny, n_omega, seed):
    return SINGLE.scaled(n_particles=n, n_steps=1, nx_dir=nx, ny_dir=ny, n_omega=n_omega, seed=seed)


def reference(w, st):
    return oracle.spectrum(flatten(st, w.times()), w.directions(), w.omegas(), w.shape, w.shape_len, w.dt)


# 1 to 17 splits of 32 particles on 5 x 33 points (no multiple of a block's points); 8191,
# 8192, 32736 and 32768 points
@pytest.mark.parametrize("n,nx,ny,n_omega", [
    (32, 5, 1, 33), (96, 5, 1, 33), (97, 5, 1, 33), (480, 5, 1, 33), (481, 5, 1, 33), (513, 5, 1, 33),
    (300, 1, 1, 8191), (300, 8, 16, 64), (600, 8, 16, 64), (300, 11, 16, 186), (300, 16, 16, 128)])
def test_fold_groups(rad, n, nx, ny, n_omega):
    w = workload(n, nx, ny, n_omega, 51)
    st = w.steps()
    g = rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
    g.push_step(0.0, to_device(st, "f32"))
    assert_parity(g.spectrum(), reference(w, st), f"fold {n} particles, {nx * ny} x {n_omega}")


@pytest.mark.parametrize("n,nx,ny,n_omega", [
    (1, 3, 1, 37), (7, 3, 1, 37), (8, 3, 1, 37), (63, 3, 1, 37), (64, 3, 1, 37), (97, 3, 1, 37), (65, 16, 16, 128)])
def test_tracked_read_out_groups(rad, n, nx, ny, n_omega):
    w = workload(n, nx, ny, n_omega, 52)
    st = w.steps()
    tr = rad.Tracked(w.directions(), w.omega0, w.domega, w.n_omega, n, dt=w.dt)
    tr.push_step(0.0, to_device(st, "f32"))
    assert_parity(tr.spectrum(st["w"][0], w.shape, w.shape_len), reference(w, st), f"tracked {n} particles")


# one to forty segments of one tile, and bunches of very different sizes in one batch
@pytest.mark.parametrize("counts", [(20,), (300,), (1280, 33), (900, 1, 64)])
def test_batched_fold_groups(rad, counts):
    b = rad.Batcher(max_items=8)
    items, refs = [], []
    for k, n in enumerate(counts):
        w = workload(n, 5, 1, 40, 60 + k)
        st = w.steps()
        g = rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
        items.append((g, 0.0, 1, to_device(st, "f32")))
        refs.append(reference(w, st))
    b.push(items)
    for (g, *_), ref, n in zip(items, refs, counts):
        assert_parity(g.spectrum(), ref, f"batched fold, {n} of {counts}")
