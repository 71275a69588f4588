"""Marches whose iteration counts rise past the prediction while the next window of
steps is in flight: the slots behind the step that missed run as no-ops and its
steps go out again.  The counts pass the first prediction of 8 in the first
window, and rise once more behind the damped quarter steps, whose dt theta is half
of the later steps'.

Against the oracle, whose march has no prediction (1e-10 of max(1, |V|), as for the
other marches); with kernel timing on and with checkpoints recorded bit for bit the
same grid (neither changes what the kernels compute), every working launch counted
once; and the gradient from states recorded by such a march against that from
recomputed segments, whose prediction is the counts themselves and never misses, and
against the oracle's dense adjoint (1e-8 of each quantity's scale, as for the other
reverse marches).
"""

import numpy as np
import pytest

import workloads
from oracle import adjoint as oadj
from oracle import integral, levy, scheme

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lp():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    import paper_2511_02700_amd as m
    return m


def _problem(w):
    m, h = w["model"], (w["y_hi"] - w["y_lo"]) / (w["n"] - 1)
    p = levy.nts_from_std(m["sigma1"], m["sigma2"], m["corr"], m["theta1"], m["theta2"], m["kappa"], m["alpha"])
    return scheme.Problem(w["n"], (w["y_lo"], w["y_lo"]), h, integral.discretize(p, h, w["r"]), payoff=w["payoff"],
                          K=w["K"], T=w["T"], N_t=w["N_t"], theta=w["theta"])


def _missed(plan):
    """Counts per step of the march from its prefixes: the first step above 8, and a rise behind it."""
    total = [0]
    for s in range(1, plan.info()["n_steps"] + 1):
        plan.solve_steps(s)
        total.append(plan.info()["total_iters"])
    counts = np.diff(total)
    print("[gpu-case] counts %s" % counts.tolist(), flush=True)
    return counts[0] > 8 and np.any(counts[4:] > counts[3])


@pytest.mark.parametrize("n,half,alpha,N_t,precision", [(33, 0.6, 0.5, 7, "fp64"), (64, 0.75, 0.7, 16, "fp64"),
                                                        (33, 0.6, 0.5, 7, "fp32conv")])
def test_march_that_misses(lp, n, half, alpha, N_t, precision):
    print("[gpu-case] recovery n=%d N_t=%d %s" % (n, N_t, precision), flush=True)
    w = workloads.workload("nig64", n=n, N_t=N_t, y_lo=-half, y_hi=half, alpha=alpha)
    plan = lp.plan_from_workload(w, precision=precision)
    assert _missed(plan)
    got = plan.solve().cpu().numpy()
    ref, _ = scheme.solve(_problem(w), tol=1e-14)
    assert np.max(np.abs(got - ref) / np.maximum(1.0, np.abs(ref))) < (1e-10 if precision == "fp64" else 1e-6)
    iters, steps = plan.info()["total_iters"], plan.info()["n_steps"]
    timed = ("line_rows", "line_cols", "cols", "sl_lin", "sl", "step_end")
    for every, classes in ((0, timed), (0, ()), (3, ()), (1 << 30, ())):
        plan.set_checkpoints(every)
        plan.set_timing(classes)
        v = plan.solve().cpu().numpy()
        assert np.array_equal(v, got), (every, classes)
        assert plan.info()["total_iters"] == iters
        if classes:                       # a march that records is not timed
            st = plan.kernel_stats()
            assert st["line_rows"][0] == st["line_cols"][0] == iters
            assert st["sl"][0] + st["sl_lin"][0] == steps
            assert all(st[c][1] > 0.0 for c in ("line_rows", "line_cols", "cols", "step_end"))


def test_recorded_states_of_a_march_that_misses(lp):
    import torch
    print("[gpu-case] recovery, recorded states", flush=True)
    w = workloads.workload("nig64", n=17, N_t=5, y_lo=-0.4, y_hi=0.4, corr=-0.4)
    plan = lp.plan_from_workload(w)
    assert _missed(plan)
    vbar = np.random.default_rng(17).standard_normal((17, 17))
    ref = oadj.adjoint(_problem(w), vbar)
    scale = np.maximum(np.abs(ref["native"]), 1e-3 * np.max(np.abs(ref["native"])))
    for every in (1, 3, 1 << 30):
        plan.set_checkpoints(every)
        plan.solve()
        _, native, _ = plan.adjoint(torch.from_numpy(vbar).cuda(), checkpoint_every=every)
        assert np.max(np.abs(native[:6] - ref["native"]) / scale) < 1e-8, every
        gw = native[6:].reshape(ref["omega"].shape)
        assert np.max(np.abs(gw - ref["omega"])) < 1e-8 * np.max(np.abs(ref["omega"])), every
