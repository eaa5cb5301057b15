"""Time steps that a caller captures on its own stream (direct launches, an even number of steps), after
a call whose steps went as windows on pair lists: every replay against the same steps taken one
call at a time, on an MI355X.  The two differ by the order of sums, as in the window tests: 1e-10 of
the largest value."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def sheared(n=2500, fast=0.0):
    w = synth.bidisperse_box(n, 0.5, 31)
    rng = np.random.default_rng(5)
    u = 0.05 * rng.standard_normal(w.x.shape)
    u[:, 0] += w.x[:, 1]
    if fast:
        u[::40] += fast * rng.standard_normal((len(u[::40]), 3))
    return w, w.rad * 1.0005, u


def near_x(a, b, L):
    d = a - b
    d -= np.asarray(L) * np.round(d / np.asarray(L))
    return float(np.max(np.abs(d)))


# fast: particles that use up a window's margin, so that the call before the capture has stopped
@pytest.mark.parametrize("sync,fast", [(True, 0.0), (False, 0.0), (False, 40.0)])
def test_replays_after_a_window(sync, fast):
    import torch

    from paper_2108_01013_amd.dss import Simulation
    w, rad, u = sheared(fast=fast)
    stream = torch.cuda.Stream()
    a, b = Simulation(w.params, stream=stream.cuda_stream), Simulation(w.params)
    a.set_tuning(graph=False)
    for s in (a, b):
        s.set_particles(w.x, rad, u)
    print(f"case: captured steps after a window, sync={sync} fast={fast}", flush=True)
    a.step(20, sync=sync)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        a.step(2, sync=False)
    for _ in range(20):
        b.step(1)
    tol = 1e-8 if fast else 1e-10

    def same():
        torch.cuda.synchronize()
        sa, sb = a.state(), b.state()
        assert a.info()["step"] == b.info()["step"]
        for k in ("u", "w", "F", "T"):
            assert rel(sa[k], sb[k]) < tol, k
        assert near_x(sa["x"], sb["x"], w.params["L"]) < tol
        assert np.array_equal(a.history()[0], b.history()[0])

    for _ in range(4):
        with torch.cuda.stream(stream):
            g.replay()
        for _ in range(2):
            b.step(1)
        same()
    # the program's own steps between the replays
    a.step(12)
    for _ in range(12):
        b.step(1)
    same()
    for _ in range(3):
        with torch.cuda.stream(stream):
            g.replay()
        for _ in range(2):
            b.step(1)
    same()
    del g
    a.close()
    b.close()


def test_steps_after_replays():
    """Replays advance the device's clock without the host; a later call, and one on a handle that
    loads a snapshot taken then, with particles that would stop a window, goes on from there."""
    import torch

    from paper_2108_01013_amd.dss import Simulation
    w, rad, u = sheared(fast=40.0)
    stream = torch.cuda.Stream()
    a, b, c = Simulation(w.params, stream=stream.cuda_stream), Simulation(w.params), Simulation(w.params)
    a.set_tuning(graph=False)
    for s in (a, b, c):
        s.set_particles(w.x, rad, u)
    print("case: steps after replays of captured steps", flush=True)
    a.step(1)  # a replay begins, as it ends, with half-step velocities
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        a.step(2, sync=False)
    for _ in range(3):
        with torch.cuda.stream(stream):
            g.replay()
    torch.cuda.synchronize()
    c.load_state(a.save_state())
    a.step(30)
    c.step(30)
    for _ in range(37):
        b.step(1)
    want = b.state()
    for s in (a, c):
        got = s.state()
        assert s.info()["step"] == 37
        for k in ("u", "w", "F", "T"):
            assert rel(got[k], want[k]) < 1e-8, k
    del g
    for s in (a, b, c):
        s.close()
