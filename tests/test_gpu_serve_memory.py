"""The server's scratch and its sums: partial tiles in proportion to the workgroups of a launch, not
to its particles, and FP32 sums in registers of at most 512 particles, with and without graphs."""
import numpy as np
import pytest

import oracle
from workloads import FIELDS, SINGLE, flatten

pytestmark = pytest.mark.gpu

# 128 x 512 points, launch shape of the table: 1024 workgroups, tiles of 16 x 512 points, 16 B a point
TILE_BYTES, WORKGROUPS, BUNCHES = 16 * 512 * 16, 1024, 4


@pytest.fixture(scope="module")
def rad():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1802_03972_amd as rad
    from paper_1802_03972_amd.build import ensure_built
    ensure_built()    # a built library is used as is
    rad._lib.lib()
    return rad


def bunch(n):
    """One particle n times, on 128 x 512 points."""
    w = SINGLE.scaled(n_particles=1, n_steps=1, nx_dir=8, ny_dir=16, n_omega=512, seed=305, omega_max=1e17, in_dtype="f32")
    st = w.steps()
    return w, st, {k: np.full(n, st[k][0, 0], np.float32) for k in FIELDS}


@pytest.mark.parametrize("graph", [True, False])
def test_scratch_of_a_large_batch(rad, graph):
    """One batch of 4 x 60000 particles: a range for each workgroup, cut once more at the end of each
    of the 8 tiles of a grid, and a quarter on top (1.25 x (1024 + 16 x 64 items) tiles in graph mode)."""
    import torch
    w, _, chunk = bunch(60000)
    grids = [rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
             for _ in range(BUNCHES)]
    srv = rad.Server(hbm_budget=64 << 20, use_graph=graph)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    tickets = [srv.submit(g, 0.0, chunk) for g in grids]
    srv.drain()
    held = before - torch.cuda.mem_get_info()[0]
    batches = max(srv.wait(t)["batch_size"] for t in tickets)
    srv.close()
    print(f"graph {graph}: {held / 2**20:.0f} MiB held for batches of up to {batches}")
    assert held <= 1.25 * (WORKGROUPS + 16 * 64) * TILE_BYTES + (64 << 20)


@pytest.mark.parametrize("graph", [True, False])
def test_long_ranges_are_summed_in_short_sums(rad, graph):
    """2,000,000 equal terms.  512 of them in one FP32 sum are off by at most 256 x 2^-24 of it, where
    each addition rounds the same way; the 31 such sums of a workgroup's range, added in FP32, by 16 x
    2^-24 more; a term itself by 3e-6 (hardware sin and cos, walk): 2 x 1.93e-5 of the intensity
    together, at every point.  A range in one sum, 15625 terms, is allowed 9e-4.  The scratch is that
    of any large batch."""
    import torch
    n = 2_000_000
    w, st, chunk = bunch(n)
    g = rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape="cic", shape_len=w.shape_len, dt=w.dt)
    srv = rad.Server(hbm_budget=256 << 20, use_graph=graph)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    srv.wait(srv.submit(g, float(w.times()[0]), chunk))
    held = before - torch.cuda.mem_get_info()[0]
    srv.close()
    ref = oracle.spectrum(flatten(st, w.times()), w.directions(), w.omegas(), "cic", w.shape_len, w.dt) * float(n) ** 2
    err = np.abs(g.spectrum() / ref - 1.0).max()
    print(f"graph {graph}: worst {err:.2e}, {held / 2**20:.0f} MiB held")
    assert held <= 1.25 * (WORKGROUPS + 16 * 64) * TILE_BYTES + (64 << 20)
    assert err <= 4e-5
