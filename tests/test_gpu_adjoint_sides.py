"""The native adjoint at every transform side against the oracle's dense discrete
adjoint: each side has its own instantiations of the reverse march's kernels (the
transposed stencil before the transform, the combined spectral term, the transposed
gather through LDS).  Odd and even grids (a last row pair of one row or two), one
checkpoint segment and several (the spectral term of a step's mu is added in the next
reverse step, across segments).  Bar: 1e-8 relative to each quantity's scale, as for
the automatic side.
"""

import numpy as np
import pytest

import workloads
from oracle import adjoint as oadj
from oracle import integral, levy, scheme

pytestmark = pytest.mark.gpu

_REF = {}


def _reference(n):
    if n not in _REF:
        w = workloads.workload("nig64", n=n, N_t=5, y_lo=-2.0, y_hi=2.0, corr=-0.4)
        m = w["model"]
        p = levy.nts_from_std(m["sigma1"], m["sigma2"], m["corr"], m["theta1"], m["theta2"], m["kappa"], m["alpha"])
        h = 4.0 / (n - 1)
        prob = scheme.Problem(n, (-2.0, -2.0), h, integral.discretize(p, h, w["r"]), payoff=w["payoff"], K=w["K"], T=w["T"],
                              N_t=w["N_t"], theta=w["theta"])
        vbar = np.random.default_rng(n).standard_normal((n, n))
        _REF[n] = w, vbar, prob.disc["N_z"], oadj.adjoint(prob, vbar)
    return _REF[n]


@pytest.mark.parametrize("L,n,C", [(64, 17, 3), (128, 18, 3), (256, 17, 32), (512, 18, 3), (768, 17, 3), (1024, 17, 1),
                                   (1536, 18, 3), (2048, 17, 32), (3072, 17, 3), (4096, 18, 3)])
def test_native_adjoint_by_side(L, n, C):
    import torch

    import paper_2511_02700_amd as lp
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    print("[gpu-case] adjoint n=%d L=%d C=%d" % (n, L, C), flush=True)
    w, vbar, Nz, ref = _reference(n)
    plan = lp.plan_from_workload(w, fft_size=L)
    assert plan.info()["L"] == L and plan.info()["N_z"] == Nz
    _, native, _ = plan.adjoint(torch.from_numpy(vbar).cuda(), checkpoint_every=C)
    scale = np.maximum(np.abs(ref["native"]), 1e-3 * np.max(np.abs(ref["native"])))
    assert np.max(np.abs(native[:6] - ref["native"]) / scale) < 1e-8
    gw = native[6:].reshape(2 * Nz, 2 * Nz)
    assert np.max(np.abs(gw - ref["omega"])) < 1e-8 * np.max(np.abs(ref["omega"]))
