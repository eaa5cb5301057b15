"""Windows of time steps at the capacity of the history rows: which of a pair's particles holds its contact is
decided at the window's start, and by the step's own cells in a full step; a row that only overflows
with the former is no error.  Against the same steps taken one call at a time, on an MI355X."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth
from test_gpu_lists import rel, run_both

pytestmark = pytest.mark.gpu


def test_owner_changes_before_a_contact_begins():
    """Capacity 1.  Particle 0 holds its contact with 1; particle 2, a cell above 0 at first, sinks into the
    cell layer of 0 and then touches it, so that 2 holds that contact.  The window of the call ends with
    the step in which they touch."""
    from paper_2108_01013_amd.dss import DssError, Simulation
    p = synth.default_params([22.0] * 3, shear_rate=0.0, eta0=1e-3, kn=100.0, kt=30.0, gamma_n=0.0, F_ER=0.0)
    x = np.array([[10.0, 6.1, 6.1], [10.0, 8.09, 6.1], [8.4238, 6.1, 7.34]])
    u = np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 0.0], [0.0, 0.0, -2.0]])
    b = Simulation(p, capacity=1)
    b.set_particles(x, np.ones(3), u)
    n = 0
    while len(b.history()[0]) < 2:         # the step in which they touch
        b.step(1)
        n += 1
    assert 40 < n < 64
    for extra in range(2):                 # a window that ends with it, and one a step later
        a = Simulation(p, capacity=1)
        a.set_particles(x, np.ones(3), u)
        a.step(n + extra)
        w = a.windows()
        assert w["stopped"] > 0, w         # the row overflowed on the lists
        sa, sb = a.state(), b.state()
        for k in ("x", "u", "w", "F", "T"):
            assert rel(sa[k], sb[k]) < 1e-10, k
        assert np.array_equal(a.history()[0], b.history()[0]) and rel(a.history()[1], b.history()[1]) < 1e-9
        assert a.info()["error_flags"] == 0
        a.close()
        b.step(1)
    # a row that overflows in full steps too (particle 2 sinks onto 0, from above)
    y = x.copy()
    y[2] = [10.0, 6.1, 8.105]
    for steps in (40, 1):
        c = Simulation(p, capacity=1)
        c.set_particles(y, np.ones(3), u)
        with pytest.raises(DssError) as e:
            for _ in range(40 // steps):
                c.step(steps)
        assert e.value.status == 3
        c.close()
    b.close()


@pytest.mark.parametrize("rolling", [False, True])
def test_smallest_capacity(rolling):
    """Rows of the largest fill that the single steps reach."""
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(2500, 0.55, 31)
    rng = np.random.default_rng(5)
    u = 5.0 * rng.standard_normal(w.x.shape)
    u[:, 0] += w.x[:, 1]
    p = dict(w.params, **(dict(kr=0.05 * w.params["kn"], mu_r=0.1) if rolling else {}))
    s = Simulation(p)
    s.set_particles(w.x, w.rad * 1.0005, u)
    fill = 0
    for _ in range(60):
        s.step(1)
        fill = max(fill, s.info()["max_row_fill"])
    s.close()
    print(f"case: windows at history capacity {fill}", flush=True)

    def make():
        s = Simulation(p, capacity=fill)
        s.set_particles(w.x, w.rad * 1.0005, u)
        return s

    run_both(make, 20, 5, 1e-8, p["L"], calls=3)
