"""Stream capture: every call that keeps marks, plans or turns of a grid, or waits for its stream,
refuses a capturing stream and leaves both the capture and the grid as they were; rad_push_step_noalloc and
a tracked set's resets and pushes are recorded, and their replays do what the calls do."""
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


def test_calls_refuse_a_capturing_stream(rad):
    import torch
    w = SINGLE.scaled(n_particles=700, n_steps=1, nx_dir=4, ny_dir=8, n_omega=64, seed=76)
    part = step_slice(to_device(w.steps(), w.in_dtype), 0, w.n_particles)
    g = rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
    tr = rad.Tracked(w.directions(), w.omega0, w.domega, w.n_omega, w.n_particles, dt=w.dt)
    b = rad.Batcher(max_items=2)
    out = torch.empty((w.n_dir, w.n_omega), dtype=torch.float64, device="cuda")
    weights = np.ones(w.n_particles)
    g.push_step_noalloc(0.0, part)
    once = g.get_state()
    tr.push_step(0.0, part)
    tracked_once = tr.spectrum(weights)
    torch.cuda.synchronize()
    refused = [lambda: g.reset(), lambda: g.push_step(0.0, part), lambda: g.push_steps(0.0, 1, part),
               lambda: g.spectrum(), lambda: g.spectrum_device(out), lambda: g.spectrum_complex(), lambda: g.get_state(),
               lambda: g.set_state(once), lambda: b.push([(g, 0.0, 1, part)]), lambda: tr.spectrum(weights)]
    graph = torch.cuda.CUDAGraph()
    errors = []
    with torch.cuda.graph(graph):
        for call in refused:
            try:
                call()
                errors.append(None)
            except rad.RadError as e:
                errors.append(e.code)
        g.push_step_noalloc(0.0, part)
        tr.reset()
        tr.push_step(0.0, part)
    torch.cuda.synchronize()
    assert errors == [rad.RAD_ERR_INVALID_ARG] * len(refused)
    assert np.array_equal(g.get_state(), once)       # nothing ran
    other = torch.cuda.Stream()
    for rep in range(3):
        g.reset(other)
        tr.push_step(0.0, part)                      # what the replay's reset clears
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(g.get_state(), once), rep
        assert np.array_equal(tr.spectrum(weights), tracked_once), rep
    # the grid's calls on other streams are ordered as if there had been no capture
    g.reset(other)
    g.push_step(0.0, part)
    b.push([(g, 0.0, 1, part)], other)
    g.spectrum_device(out)
    torch.cuda.synchronize()
    assert np.allclose(out.cpu().numpy(), g.spectrum(other))


def test_another_thread_reads_during_a_capture(rad):
    """A host read-out's page-locked buffer may be allocated while another thread captures: that is
    no work on a stream, and must end neither the read-out nor the capture."""
    import threading
    import torch
    w = SINGLE.scaled(n_particles=300, n_steps=1, nx_dir=4, ny_dir=8, n_omega=2048, seed=77)
    part = step_slice(to_device(w.steps(), w.in_dtype), 0, w.n_particles)
    weights = np.ones(w.n_particles)
    g = rad.Grid(w.directions(), w.omega0, w.domega, w.n_omega, shape=w.shape, shape_len=w.shape_len, dt=w.dt)
    tr = rad.Tracked(w.directions(), w.omega0, w.domega, w.n_omega, w.n_particles, dt=w.dt)
    main = torch.cuda.default_stream()
    g.push_step(0.0, part, main)
    tr.push_step(0.0, part, main)
    torch.cuda.synchronize()
    got = {}

    def read():
        try:      # several sizes, so that buffers are allocated whatever the pool holds
            got["I"], got["Z"] = g.spectrum(main), g.spectrum_complex(main)
            got["tracked"] = tr.spectrum(weights, stream=main)
        except Exception as e:          # reported below, outside the capture
            got["error"] = e

    x = torch.zeros(1024, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x += 1
        t = threading.Thread(target=read)
        t.start()
        t.join()
        x += 1
    graph.replay()
    torch.cuda.synchronize()
    assert "error" not in got, got["error"]
    assert float(x[0]) == 2.0
    assert np.array_equal(got["I"], g.spectrum()) and np.array_equal(got["Z"], g.spectrum_complex())
    assert np.array_equal(got["tracked"], tr.spectrum(weights))
