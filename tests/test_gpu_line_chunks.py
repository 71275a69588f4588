"""Marches at the edges of the line solves' chunk capacities: grids whose chunks just
fill, or just pass, the capacities whose factors stay in registers (4 and 8 rows per
thread), along both axes, and the row kernels' read-ahead forms (transform sides up to
1024 and above).

Small grids against the oracle's march, within 1e-10 of max(1, |V|) as for the other
marches.  Larger ones against the same march with 16 (or 8) elements per thread, whose line solves
take the other form: both stop at tol = 1e-12 with a contraction far below 1/2, so they
lie within 1e-10 of one another as well.
"""

import numpy as np
import pytest

import workloads
from oracle import integral, levy, scheme

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.max(np.abs(a - b) / np.maximum(1.0, np.abs(b))))


def _lp():
    import torch

    import paper_2511_02700_amd as lp
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    return lp


@pytest.mark.parametrize("n", [8, 15, 16, 17, 33, 63, 64, 65])
def test_march_matches_oracle(n):
    lp = _lp()
    print("[gpu-case] line chunks, oracle march n=%d" % n, flush=True)
    w = workloads.workload("nig64", n=n, N_t=3, y_lo=-1.5, y_hi=1.5)
    m, h = w["model"], 3.0 / (n - 1)
    p = levy.nts_from_std(m["sigma1"], m["sigma2"], m["corr"], m["theta1"], m["theta2"], m["kappa"], m["alpha"])
    prob = scheme.Problem(n, (-1.5, -1.5), h, integral.discretize(p, h, w["r"]), payoff=w["payoff"], K=w["K"], T=w["T"],
                          N_t=3, theta=w["theta"])
    ref, _ = scheme.solve(prob, tol=1e-14)
    got = lp.plan_from_workload(w).solve().cpu().numpy()
    assert _rel(got, ref) < 1e-10


@pytest.mark.parametrize("n,half,radix", [(127, 3.0, 8), (129, 3.0, 16), (256, 3.0, 16), (257, 3.0, 8), (511, 4.0, 16),
                                          (512, 4.0, 8), (513, 4.0, 16), (640, 4.0, 8), (1023, 4.0, 8)])
def test_march_matches_other_radix(n, half, radix):
    lp = _lp()
    print("[gpu-case] line chunks, n=%d against radix %d" % (n, radix), flush=True)
    w = workloads.workload("nig64", n=n, N_t=n // 4, y_lo=-half, y_hi=half)
    auto = lp.plan_from_workload(w)
    other = lp.plan_from_workload(w, fft_radix=radix, fft_size=1 << (auto.info()["L"] - 1).bit_length())
    v = [plan.solve_steps(8).cpu().numpy() for plan in (auto, other)]      # the damped steps and some of the others
    assert _rel(v[0], v[1]) < 1e-10
