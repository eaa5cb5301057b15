"""Short cell rows (boxes of a few hundred particles), whose occupancy varies most about its mean:
the row tiles against the per-particle path on an MI355X.  FP64 sums of the same pairs in another
order: 1e-10 of the largest entry, as against the oracle; pair sets and contacts equal."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,phi", [(300, 0.5), (500, 0.55), (855, 0.56), (1300, 0.4), (5000, 0.55)])
def test_short_rows(n, phi):
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(n, phi, seed=8)
    print(f"case: short rows N={n}", flush=True)
    out = []
    for tiled in (True, False):
        sim = Simulation(w.params)
        sim.set_tuning(tiled=tiled)
        sim.set_particles(w.x, w.rad)
        for _ in range(3):
            sim.step(1)
        last, _, _ = sim.read_stress()
        i = sim.info()
        out.append((sim.state(), last, (i["n_pairs"], i["n_contacts"])))
        sim.close()
    (a, sa, na), (b, sb, nb) = out
    assert na == nb and na[1] > 0
    for k in ("x", "u", "w", "F", "T"):
        assert np.max(np.abs(a[k] - b[k])) <= 1e-10 * np.max(np.abs(b[k])), k
    assert np.max(np.abs(sa - sb)) <= 1e-10 * np.max(np.abs(sb))
