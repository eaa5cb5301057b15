"""The handle after an adjoint of a run that is recorded whole: it stands where dss_step of the same run
leaves it, on an MI355X."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


def test_listed_pairs():
    """The recorded pairs are those of the run's last evaluation (whole numbers: equal), on the row
    tiles and on the per-particle path."""
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(1200, 0.5, seed=3)
    u = 2.0 * np.random.default_rng(1).standard_normal(w.x.shape)
    for tiled in (True, False):
        out = []
        for adjoint in (True, False):
            s = Simulation(w.params, record_pairs=True)
            s.set_tuning(tiled=tiled)
            s.set_particles(w.x, w.rad, u)
            first = s.pairs()
            s.adjoint(20, 5, 7) if adjoint else s.step(20, 5)
            out.append(s.pairs())
            s.close()
        assert np.array_equal(*out) and not np.array_equal(out[0], first)


def test_after_set_step():
    """dss_set_step moves the Lees-Edwards offset under the forces, and a run without an evaluation in
    between starts with those forces: J is the mean of the step call's samples, and the state its
    state.  Sums of the same pairs in another order over 20 steps: 1e-10, as against the oracle."""
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(1200, 0.5, seed=3)
    out = []
    for adjoint in (True, False):
        s = Simulation(w.params)
        s.set_particles(w.x, w.rad)
        s.set_step(777)
        if adjoint:
            J = s.adjoint(20, 5, 7)["J"]
        else:
            s.step(20, 5)
            J = s.read_stress()[1][0, 1]
        out.append((J, s.state()))
        s.close()
    (a, x), (b, y) = out
    assert abs(a - b) <= 1e-10 * abs(b)
    for k in ("u", "w", "F", "T"):
        assert np.max(np.abs(x[k] - y[k])) <= 1e-10 * np.max(np.abs(y[k])), k
