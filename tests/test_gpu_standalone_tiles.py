"""The stand-alone correlation at every transform side and the Greeks around the
edges of their blocks, against the FP64 oracle.

B v: each side takes its own elements per thread and one of two forms of each
pass; odd and even n (a last row pair of one row or two) at sides forced to the
kernel's support.  Bar: 1e-12 of max |B v|, as for the automatic sides.  Greeks:
grids whose inner rows and columns end just before, at and just behind a block;
bar 1e-11 of each surface's largest value (at most 25 products of values that
the nodes' exponentials scale alike).
"""

import numpy as np
import pytest

import workloads
from oracle import integral, levy, output, scheme

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lp():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    import paper_2511_02700_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("L,n", [(256, 75), (512, 150), (512, 151), (768, 301), (1024, 302), (1024, 403), (1536, 605),
                                 (2048, 604), (2048, 807), (3072, 1001), (4096, 1202), (4096, 1203)])
def test_apply_B_by_side(lp, L, n):
    import torch
    print("[gpu-case] apply_B n=%d L=%d" % (n, L), flush=True)
    w = workloads.workload("nig64", n=n, y_lo=-3.0, y_hi=3.0)
    plan = lp.plan_from_workload(w, fft_size=L)
    assert plan.info()["L"] == L
    m = w["model"]
    p = levy.nts_from_std(m["sigma1"], m["sigma2"], m["corr"], m["theta1"], m["theta2"], m["kappa"], m["alpha"])
    d = integral.discretize(p, 6.0 / (n - 1), w["r"])
    v = workloads.random_grid(n, seed=n)
    got = plan.apply_B(torch.from_numpy(v).cuda()).cpu().numpy()
    ref = scheme.apply_B(v, d["W"], d["N_z"], 3, "fft")
    assert np.max(np.abs(got - ref)) < 1e-12 * np.max(np.abs(ref))


@pytest.mark.parametrize("n", [8, 9, 10, 11, 33, 129, 130, 131, 132, 259])
def test_greeks_around_blocks(lp, n):
    import torch
    print("[gpu-case] greeks n=%d" % n, flush=True)
    w = workloads.workload("nig64", n=n, y_lo=-1.0, y_hi=1.0)
    plan = lp.Plan(lp.make_grid(n, -1.0, 1.0), lp.levy_black_scholes(0.03, (0.04, 0.01, 0.06)),
                   lp.make_payoff("put_avg", w["K"], 1.0), M=4)
    V = workloads.random_grid(n, seed=n)
    got = plan.greeks(torch.from_numpy(V).cuda()).cpu().numpy()
    ref = output.greeks_on_grid(V, (-1.0, -1.0), 2.0 / (n - 1), w["K"])
    for q in range(5):
        assert np.max(np.abs(got[q] - ref[q])) < 1e-11 * np.max(np.abs(ref[q]))
