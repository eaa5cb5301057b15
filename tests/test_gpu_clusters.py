"""Contact clusters over the shapes that the passes of the union-find treat differently: one long
chain under shuffled ids (deep trees), chains that end at the edges of workgroups, and a dense
box (one cluster of nearly everything), against the oracle on an MI355X.  Whole numbers: equal."""
import numpy as np
import pytest

import oracle
from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


def chains(lengths, seed):
    """Touching spheres in lines along x, one line per entry, ids shuffled."""
    p = dict(synth.bidisperse_box(400, 0.4, seed=1).params)
    side = 4.0
    p["L"] = [1.99 * max(lengths) + 14.0, 12.0, side * max(3, len(lengths))]
    x = np.concatenate([np.stack([3.0 + 1.99 * np.arange(n), np.full(n, 6.0), np.full(n, side * (k + 0.5))], 1)
                        for k, n in enumerate(lengths)])
    rng = np.random.default_rng(seed)
    return p, x[rng.permutation(len(x))], np.ones(len(x))


@pytest.mark.parametrize("lengths", [(3000,), (1, 2, 256, 257), (64, 63, 1, 1, 512)])
def test_chains(lengths):
    from paper_2108_01013_amd.dss import Simulation
    p, x, rad = chains(lengths, 5)
    print(f"case: contact clusters of chains {lengths}", flush=True)
    sim = Simulation(p)
    sim.set_particles(x, rad)
    sim.step(1)
    g = sim.contact_clusters(len(x))
    want = np.zeros(len(x), dtype=g.dtype)
    for n in lengths:
        want[n - 1] += 1
    assert np.array_equal(g, want), np.flatnonzero(g != want)[:10]
    sim.close()


def test_dense_box():
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(20000, 0.6, seed=3)
    print("case: contact clusters N=20000", flush=True)
    sim = Simulation(w.params)
    sim.set_particles(w.x, w.rad)
    sim.step(30)
    pairs, _ = sim.history()
    n = len(w.rad)
    assert np.array_equal(sim.contact_clusters(n), oracle.contact_clusters(n, pairs, n))
    sim.close()
