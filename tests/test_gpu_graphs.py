"""Calls of more shapes than the handle keeps graphs for, enqueued without a wait (the graphs that go out of use
are still under way), against steps taken one call at a time, on an MI355X.  1e-9 of the largest value: the
order of sums over some 1700 steps of a box at rest under shear."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiled", [True, False])
def test_more_shapes_than_graphs(tiled):
    """On windows (tiled) and in full steps; the tuning and the lattice change while steps are under way."""
    from paper_2108_01013_amd.dss import Simulation
    p = synth.default_params([22.0] * 3)
    rng = np.random.default_rng(4)
    g = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = (g + 0.5) * 22.0 / 6 + 0.2 * rng.uniform(-1, 1, (216, 3))
    print(f"case: many call shapes, tiled={tiled}", flush=True)
    sims = []
    for one in (False, True):
        s = Simulation(p)
        s.set_tuning(tiled=tiled)
        s.set_particles(x, np.ones(216))
        for n in range(2, 60):
            if n in (20, 40):
                s.set_tuning(queue_cap=n, cell_scale=1.0 + n / 400)
            if one:
                for _ in range(n):
                    s.step(1)
            else:
                s.step(n, stress_every=n % 7, sync=False)
        s.step(1)
        sims.append(s)
    a, b = sims
    sa, sb = a.state(), b.state()
    assert a.info()["step"] == b.info()["step"] == sum(range(2, 60)) + 1
    for k in ("u", "w", "F", "T"):
        assert np.max(np.abs(sa[k] - sb[k])) <= 1e-9 * np.max(np.abs(sb[k])), k
    assert (a.windows()["taken"] > 30) == tiled
    for s in sims:
        s.close()
