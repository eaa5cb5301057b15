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
