"""The adjoint of a run that is recorded whole and of one that is checkpointed: the same J and
gradients however a run is cut, on an MI355X."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu

W = np.zeros((3, 3))
W[0, 1] = 1.0


def run(w, n_steps, every, ckpt):
    from paper_2108_01013_amd.dss import Simulation
    sim = Simulation(w.params)
    sim.set_particles(w.x, w.rad)
    r = sim.adjoint(n_steps, every, ckpt, W)
    s = sim.state()
    sim.close()
    return r, s


@pytest.mark.parametrize("n_steps,every", [(120, 10), (121, 50)])
def test_run_beyond_the_tape(n_steps, every):
    """20000 particles, more steps than are recorded at once (about 75): checkpoints every 20
    steps, every 59 and one for the whole run, and the forward run of dss_step.  The sums over
    pairs are taken in another order: the bounds of the checkpoint test of small boxes (1e-10 of J, 1e-8
    of the largest gradient entry)."""
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(20000, 0.5, seed=4)
    print(f"case: adjoint N=20000 steps={n_steps}", flush=True)
    sim = Simulation(w.params)
    sim.set_particles(w.x, w.rad)
    sim.step(n_steps, every)
    want = sim.state()["x"]
    sim.close()
    runs = [run(w, n_steps, every, c) for c in (20, 59, n_steps)]
    (r0, s0) = runs[0]
    assert np.max(np.abs(s0["x"] - want)) <= 1e-9 * np.max(np.abs(want))
    for r, s in runs[1:]:
        assert abs(r["J"] - r0["J"]) <= 1e-10 * abs(r0["J"])
        for k in ("dx", "du", "dw"):
            assert np.max(np.abs(r[k] - r0[k])) <= 1e-8 * np.max(np.abs(r0[k])), k
        assert np.max(np.abs(s["x"] - s0["x"])) <= 1e-9 * np.max(np.abs(s0["x"]))
