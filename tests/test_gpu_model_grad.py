"""The gradient with respect to the subordination parameters (lpide_adjoint with
std_params) against the native gradient times the oracle's central differences of the
model's quantities (same steps, 1e-4 max(|x|, 0.1)), for orders nu = 1 + alpha near 1, in
the middle and near 2, a cell quadrature of fewer and of more than 64 nodes.

Bar: 1e-7 of the sum of the absolute terms.  The oracle's covariance carries 1e-13, which
the smallest step (1e-5) turns into 1e-8 of it; the weights' rounding is below that.
"""

import numpy as np
import pytest

import workloads
from oracle import integral, levy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha,n,ng", [(0.02, 16, 8), (0.5, 19, 5), (0.9, 18, 10)])
def test_gradient_is_native_times_model_differences(alpha, n, ng):
    import torch

    import paper_2511_02700_amd as lp
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    print("[gpu-case] model gradient alpha=%g n=%d gl_nodes=%d" % (alpha, n, ng), flush=True)
    w = workloads.workload("nig64", n=n, N_t=4, y_lo=-2.0, y_hi=2.0, alpha=alpha, corr=-0.3)
    m, h = w["model"], 4.0 / (n - 1)
    x = [m["sigma1"], m["sigma2"], m["corr"], m["theta1"], m["theta2"], m["kappa"], m["alpha"], w["r"]]
    plan = lp.Plan(lp.make_grid(n, -2.0, 2.0, gl_nodes=ng), lp.levy_from_std(*x), lp.make_payoff("put_avg", w["K"], w["T"]),
                   M=4)
    vbar = np.random.default_rng(n).standard_normal((n, n))
    grad, native, _ = plan.adjoint(torch.from_numpy(vbar).cuda(), checkpoint_every=8, std_params=x)
    p0 = levy.nts_from_std(*x[:7])
    sz = integral.grid_sizes(p0, h)
    N = sz["N_z"]
    assert plan.info()["N_z"] == N
    gw = native[6:].reshape(2 * N, 2 * N)
    e = np.expm1((np.arange(-N, N) + 0.5) * h)
    full = gw + native[3] - native[4] * e[:, None] - native[5] * e[None, :]
    for q in range(7):
        hq = 1e-4 * max(abs(x[q]), 0.1)
        W, S = [], []
        for sgn in (1.0, -1.0):
            y = list(x)
            y[q] += sgn * hq
            p = levy.nts_from_std(*y[:7])
            W.append(integral.weights(p, h, N, sz["M1"], sz["M2"], ng))
            S.append(integral.small_jump_cov(p, h, sz["M1"]))
        dW, dS = (W[0] - W[1]) / (2 * hq), (S[0] - S[1]) / (2 * hq)
        terms = np.concatenate([(full * dW).ravel(), [native[0] * dS[0, 0], native[1] * dS[0, 1], native[2] * dS[1, 1]]])
        assert abs(grad[q] - np.sum(terms)) < 1e-7 * np.sum(np.abs(terms)), q
    assert grad[7] == pytest.approx(native[3] + native[4] + native[5], rel=1e-14)
