"""What a window of time steps may begin from: the state that a full step on the same Lees-Edwards
offset has left, on an MI355X."""
import numpy as np
import pytest

import oracle
from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


def gaps(p, x, rad, pairs, step):
    """Surface distances of the pairs (nearest image at time index step)."""
    L, delta = np.asarray(p["L"]), oracle.le_offset(p, step)
    r = x[pairs[:, 1]] - x[pairs[:, 0]]
    q = np.round(r[:, 1] / L[1])
    r[:, 1] -= q * L[1]
    r[:, 0] -= q * delta
    r[:, 0] -= L[0] * np.round(r[:, 0] / L[0])
    r[:, 2] -= L[2] * np.round(r[:, 2] / L[2])
    return np.sqrt(np.sum(r * r, axis=1)) - rad[pairs[:, 0]] - rad[pairs[:, 1]]


@pytest.mark.parametrize("prepare", [0, 4, 20])
def test_after_set_step(prepare):
    """A contact across the sheared faces that the new offset parts, and that the next step closes
    again, keeps its stretch (a search at the state of the call finds it parted, and drops it), also when
    the call's graphs were captured before.  Tolerance of test_gpu_lists over 20 steps."""
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(2500, 0.55, 31)
    rad = w.rad * 1.0005
    u = 10.0 * np.random.default_rng(5).standard_normal(w.x.shape)
    u[:, 0] += w.x[:, 1]
    print(f"case: window after set_step, prepare_steps({prepare})", flush=True)
    out = []
    for one in (False, True):
        s = Simulation(w.params)
        s.set_particles(w.x, rad, u)
        for _ in range(8):
            s.step(1)
        s.set_step(6)
        if one:
            pairs, before = s.history()[0], s.state()["x"]
            for k in range(20):
                s.step(1)
                if k == 0:
                    parted = gaps(w.params, before, rad, pairs, 6) > 0
                    assert np.any(parted & (gaps(w.params, s.state()["x"], rad, pairs, 7) < 0))
        else:
            if prepare:
                s.prepare_steps(prepare)
            s.step(20)
        out.append((s.state(), s.history()))
        s.close()
    (a, (pa, xa)), (b, (pb, xb)) = out
    assert np.array_equal(pa, pb)
    assert np.max(np.abs(xa - xb)) <= 1e-9 * np.max(np.abs(xb))
    for k in ("u", "w", "F", "T"):
        assert np.max(np.abs(a[k] - b[k])) <= 1e-10 * np.max(np.abs(b[k])), k


@pytest.mark.parametrize("path", ["plain", "sized", "far"])
@pytest.mark.parametrize("bad", [np.nan, np.inf, 1e7])
def test_particles_outside_the_box(path, bad):
    """Velocities that are no numbers, or that carry a particle out of the box in one step: no window
    begins where the search would take their cells for indices, the steps are full ones and the
    error is reported as it is for single steps."""
    from paper_2108_01013_amd.dss import DssError, Simulation
    ec = dict(ec_ranges=True, hamaker=1e-3) if path == "far" else {}
    w = synth.bidisperse_box(4500, 0.45, 23, **ec)
    u = np.zeros_like(w.x)
    u[:, 0] = w.x[:, 1]
    u[1::700] = bad
    u[2::700] = -bad
    print(f"case: particles outside the box, {path}, {bad}", flush=True)
    s = Simulation(w.params)
    if path == "sized":
        s.set_tuning(sized=True)
    if np.isfinite(bad):
        s.set_particles(w.x, w.rad, u)
    else:
        with pytest.raises(DssError):      # its forces are not finite; the particles are loaded
            s.set_particles(w.x, w.rad, u)

    def steps(n):
        try:
            s.step(n)
        except DssError as e:
            assert e.status == 5, e
            return True
        return False

    failed = steps(1)                  # a full step: its positions begin the windows of the next calls
    for n in (20, 80):
        failed = steps(n) or failed
    assert failed == (not np.isfinite(bad))
    if failed:
        with pytest.raises(DssError):
            s.read_stress()
    assert s.info()["step"] == 101 and s.windows()["taken"] == 0 and s.windows()["stopped"] > 0
    s.close()


@pytest.mark.parametrize("bad", [1e7, 1e200])
def test_far_forces_of_particles_outside_the_box(bad):
    """Full steps with the far pairs on a pass of their own: a particle whose position no cell number holds
    is searched around within the lattice, and all step on."""
    from paper_2108_01013_amd.dss import Simulation
    w = synth.bidisperse_box(4500, 0.45, 23, ec_ranges=True, hamaker=1e-3)
    u = np.zeros_like(w.x)
    u[:, 0] = w.x[:, 1]
    lone = np.array([7, 1234, 4000])
    u[lone] = [[bad, 0.0, 0.0], [-bad, 0.0, -bad], [0.0, bad, 0.0]]
    print(f"case: far forces, particles outside the box, {bad}", flush=True)
    s = Simulation(w.params)
    s.set_particles(w.x, w.rad, u)
    assert s.box_info(0)["ec_far_rows"][0] > 0
    for _ in range(3):
        s.step(1)
    f = s.state()["F"]
    assert s.info()["error_flags"] == 0 and np.all(np.isfinite(f))
    s.close()
