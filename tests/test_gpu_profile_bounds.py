"""The phi(y) profile of a box from which particles have flown (velocities of many box lengths per step), on an
MI355X: the others' volume, each sphere once.  Sums of 2000 positive terms: 1e-12."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [1e20, 1e200])
@pytest.mark.parametrize("noalloc", [False, True])
def test_profile_without_lost_particles(bad, noalloc):
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(2000, 0.45, seed=18)
    u = np.zeros_like(w.x)
    u[:, 0] = w.x[:, 1]
    lost = np.array([3, 700, 1999])
    u[lost, 1] = bad
    print(f"case: profile, lost particles {bad} noalloc={noalloc}", flush=True)
    s = Simulation(w.params)
    s.set_particles(w.x, w.rad, u)
    s.step(1)
    y = s.state()["x"][:, 1]
    phi = (s.phi_profile_noalloc if noalloc else s.phi_profile)(16, 1.2)
    kept = np.abs(y) <= 1e5 * w.L
    assert not np.any(kept[lost]) and np.count_nonzero(~kept) < 200
    for g, pick in enumerate((w.rad <= 1.2, w.rad > 1.2)):
        want = 4.0 / 3.0 * np.pi * np.sum(w.rad[kept & pick] ** 3) / w.L ** 3
        assert abs(phi[g].mean() - want) <= 1e-12 * want
    s.close()
