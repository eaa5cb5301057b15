"""How long windows of time steps are after one has stopped, and that they come back, on an MI355X."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


def fast_start():
    """A few particles fast enough to use up the margin, slowed by the fluid within some 100 steps."""
    rng = np.random.default_rng(8)
    n, L = 1500, 45.0
    rad = synth.bidisperse_radii(n, seed=8)
    x = synth.relax_positions(rad, L, seed=8)
    u = rng.standard_normal((n, 3))
    u[:, 0] += x[:, 1]
    u[::40] += 40.0 * rng.standard_normal((len(u[::40]), 3))
    return synth.default_params([L] * 3, dt=5e-4), x, rad, u


@pytest.mark.parametrize("calls,steps,sync", [(1, 3000, True), (1, 3000, False), (30, 100, True), (30, 100, False)])
def test_windows_return_after_a_violent_start(calls, steps, sync):
    from paper_2108_01013_amd.dss import Simulation
    p, x, rad, u = fast_start()
    s = Simulation(p)
    s.set_particles(x, rad, u)
    assert s.windows() == {"taken": 0, "stopped": 0, "length": 64}
    print(f"case: windows after a violent start, {calls} calls of {steps}, sync={sync}", flush=True)
    for _ in range(calls):
        s.step(steps, sync=sync)
    w = s.windows()
    assert s.info()["step"] == calls * steps
    assert w["stopped"] > 0 and w["length"] == 64 and w["taken"] > 20, w
    s.step(640)
    assert s.windows()["taken"] == w["taken"] + 10 and s.windows()["stopped"] == w["stopped"]
    # new particles begin anew
    s.set_particles(x, rad)
    assert s.windows()["length"] == 64
    s.close()


def test_lists_that_do_not_fit_are_tried_again():
    """An overlapping cluster with more neighbours than a list holds: full steps, 64 and then twice as
    many after every trial."""
    from paper_2108_01013_amd.dss import Simulation
    rng = np.random.default_rng(3)
    x = rng.uniform(0.0, 1.0, (800, 3)) * [6.0, 6.0, 6.0]
    s = Simulation(synth.default_params([24.0] * 3, kn=1.0, kt=0.3, gamma_n=0.0, capacity=0), capacity=400)
    s.set_particles(x, np.ones(800))
    for steps, stopped in ((12, 1), (40, 1), (60, 2), (70, 2), (30, 3)):
        s.step(steps)
        assert s.windows() == {"taken": 0, "stopped": stopped, "length": 0}
    # another lattice may hold other lists
    s.set_tuning(cell_scale=1.25)
    s.step(1)
    assert s.windows()["length"] == 64
    s.close()


def test_snapshots_do_not_stop_windows():
    """A handle that goes back to a snapshot again and again takes windows every time."""
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(2500, 0.5, 31)
    s = Simulation(w.params)
    s.set_particles(w.x, w.rad)
    s.step(20)
    blob = s.save_state()
    for k in range(6):
        s.load_state(blob)
        s.step(40, stress_every=5)
        assert s.windows()["taken"] == 2 + k, s.windows()
    s.close()


def test_windows_lengthen_within_a_call():
    """One call of 20 000 steps that is waited for: its windows are short only around the violent start
    (20 000 steps are 313 windows of 64).  (A call that is not waited for lengthens them as far as the
    device has come when its steps are enqueued.)"""
    from paper_2108_01013_amd.dss import Simulation
    p, x, rad, u = fast_start()
    s = Simulation(p)
    s.set_particles(x, rad, u)
    print("case: one long call", flush=True)
    s.step(20000, stress_every=100)
    _, mean, ns = s.read_stress()
    w = s.windows()
    assert s.info()["step"] == 20000 and ns == 200 and np.all(np.isfinite(mean))
    assert w["stopped"] > 0 and w["length"] == 64
    assert w["taken"] < 800, w
    s.close()


@pytest.mark.parametrize("calls,sync", [(1, True), (1, False), (4, False)])
def test_stop_within_a_long_call(calls, sync):
    """A large particle hits a small one after about 1000 steps in a thin fluid, and drives it off faster than
    the margin allows for 64 steps: a window stops when later ones, and later calls, are enqueued.
    The state and the samples of the last call are those of steps taken one call at a time (three
    particles, one collision: 1e-9)."""
    from paper_2108_01013_amd.dss import Simulation
    p = synth.default_params([40.0, 16.0, 16.0], shear_rate=0.02, eta0=1e-3)
    x = np.array([[4.0, 6.0, 6.0], [7.6, 6.1, 6.0], [20.0, 2.0, 2.0]])
    rad = np.array([2.0, 1.0, 1.0])
    u = np.array([[6.0, 0.0, 0.0], [0.12, 0.0, 0.0], [0.04, 0.0, 0.0]])
    print(f"case: a stop within {calls} long calls, sync={sync}", flush=True)
    a, b = Simulation(p), Simulation(p)
    for s in (a, b):
        s.set_particles(x, rad, u)
    for c in range(calls):
        a.step(2400, stress_every=30, sync=sync and c == calls - 1)
    last, mean, ns = a.read_stress()
    samples = []
    for k in range(2400 * calls):
        b.step(1)
        if (k + 1) % 30 == 0 and k >= 2400 * (calls - 1):
            samples.append(b.read_stress()[0])
    assert ns == len(samples) and a.info()["step"] == b.info()["step"]
    for got, want in ((last, b.read_stress()[0]), (mean, np.mean(samples, axis=0))):
        assert np.max(np.abs(got - want)) <= 1e-9 * np.max(np.abs(want))
    sa, sb = a.state(), b.state()
    for k in ("u", "w", "F", "T"):
        assert np.max(np.abs(sa[k] - sb[k])) <= 1e-9 * np.max(np.abs(sb[k])), k
    assert a.windows()["stopped"] > 0
    a.close()
    b.close()
