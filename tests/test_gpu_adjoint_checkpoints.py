"""The adjoint of checkpointed runs (no memory for a tape of the whole run) against that of runs
recorded whole, which the finite differences of test_gpu_adjoint check, on an MI355X: segments of 7, 7
and 6 steps, of 3 with a last one of 2, and of single steps."""
import numpy as np
import pytest

from paper_2108_01013_amd import synth

pytestmark = pytest.mark.gpu


def workload(kind):
    if kind == "far":
        w = synth.bidisperse_box(4000, 0.45, seed=23)
        return w, dict(w.params, ec_ranges=1, hamaker=2e-3)
    w = synth.bidisperse_box(400, 0.52, seed=21)
    return w, dict(w.params, mu=0.1, **(dict(kr=0.5 * w.params["kn"], mu_r=0.1) if kind == "rolling" else {}))


# the runs differ by the order of FP64 sums, as in the spacing test of test_gpu_adjoint: 1e-10 of J, 1e-8 of the
# largest gradient entry; a mixed forward run may round a pair to 32 bits the other way: the mixed
# tolerances of that file
@pytest.mark.parametrize("kind,tol_j,tol", [("plain", 1e-10, 1e-8), ("rolling", 1e-10, 1e-8), ("far", 1e-10, 1e-8),
                                            ("rows", 1e-10, 1e-8), ("mixed", 1e-5, 1e-4)])
def test_checkpointed_equals_recorded_whole(kind, tol_j, tol):
    from paper_2108_01013_amd.dss import DSS_FP64, DSS_MIXED, Simulation
    w, p = workload(kind)
    print(f"case: checkpointed adjoint, {kind}", flush=True)
    sim = Simulation(p, precision=DSS_MIXED if kind == "mixed" else DSS_FP64)
    if kind == "rows":
        sim.set_tuning(tiled=False)

    def run(tape, ckpt):
        sim.set_adjoint_tape(tape)
        sim.set_particles(w.x, w.rad)
        r = sim.adjoint(20, 5, ckpt)
        r.update({"end_" + k: v for k, v in sim.state().items()})
        assert sim.info()["step"] == 20
        return r

    want = run(2 << 30, 7)
    assert np.max(np.abs(want["dx"])) > 0 and abs(want["dmu"]) > 0 or kind == "far"
    for ckpt in (7, 3, 1):
        got = run(0, ckpt)
        assert abs(got["J"] - want["J"]) <= tol_j * abs(want["J"]), ckpt
        for k in ("dx", "du", "dw", "end_u", "end_w", "end_F", "end_T"):
            assert np.max(np.abs(got[k] - want[k])) <= tol * np.max(np.abs(want[k])), (ckpt, k)
        for k in ("dmu", "dF_ER"):
            assert abs(got[k] - want[k]) <= tol * abs(want[k]) + 1e-14 * abs(want["J"]), (ckpt, k)
    sim.close()


def test_tape_limit_bounds_memory():
    """N = 20 000, 60 steps: with no tape allowed, checkpoints of every 20 steps take less than half of what
    the whole tape does, and lowering the limit gives its memory back."""
    import torch

    from paper_2108_01013_amd.dss import DssError, Simulation
    w = synth.bidisperse_box(20000, 0.5, seed=4)
    sim = Simulation(w.params)
    sim.set_particles(w.x, w.rad)

    def used():
        torch.cuda.synchronize()
        free, total = torch.cuda.mem_get_info()
        return total - free

    base = used()
    out = []
    for tape in (2 << 30, 0, 2 << 30):
        sim.set_adjoint_tape(tape)
        if out and tape == 0:    # the longer tape is given back (a higher limit keeps what is there)
            assert used() - base < 64 << 20
        sim.compute_forces()
        sim.adjoint(60, 20, 20)
        out.append(used() - base)
    print("bytes of the adjoint's workspace:", out, flush=True)
    assert out[1] < 0.5 * out[0] and out[2] > 0.9 * out[0]
    with pytest.raises(DssError):
        sim.set_adjoint_tape(-1)
    sim.close()
