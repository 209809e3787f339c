"""Ordering of one grid's calls issued on the null stream and on other streams in turn, with no
host synchronisation between them: the events that the library needs are recorded by a
launch, by the call, or (for work on the null stream) only when another stream asks, and every
order has to give the serial result.  Work queued first delays each stream in turn, so that a
missing wait shows."""
import numpy as np
import pytest

from workloads import SINGLE
from tests.helpers import step_slice, to_device

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


# 0: the null stream, 1..3: non-blocking streams; one entry per call
@pytest.mark.parametrize("profile", [False, True])
@pytest.mark.parametrize("order", ["000000", "010101", "101010", "001122", "123012", "110022", "000123", "321000"])
def test_calls_on_streams_in_turn(rad, order, profile):
    import torch
    w = SINGLE.scaled(n_particles=700, n_steps=3, nx_dir=4, ny_dir=4, n_omega=96, seed=71)
    st = w.steps()
    dev = to_device(st, "f32")
    heavy = torch.randn(2048, 2048, device="cuda")
    streams = [torch.cuda.default_stream()] + [torch.cuda.Stream() for _ in range(3)]

    def run(pick, delay):
        g = rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
        g.profile(1 if profile else 0)
        first = torch.empty(w.n_dir, w.n_omega, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        s = iter(pick)

        def at():
            stream = streams[next(s)]
            if delay:
                with torch.cuda.stream(stream):
                    for _ in range(12):
                        torch.mm(heavy, heavy)
            return stream
        for j in range(2):
            g.push_step(float(w.times()[j]), step_slice(dev, j, w.n_particles), at())
        g.spectrum_device(first, at())
        g.reset(at())
        g.push_step(float(w.times()[2]), step_slice(dev, 2, w.n_particles), at())
        last = g.spectrum(at())
        torch.cuda.synchronize()
        first = first.cpu().numpy()
        g.close()
        return first, last

    want = run([0] * 6, False)
    got = run([int(c) for c in order], True)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
