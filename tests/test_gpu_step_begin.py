"""The step-begin kernel of the FP64 march (explicit part, SL gather, start value
and iteration 1's residual on a tile) at the edges of its tiles: grid sides
around one and two tile widths (252 columns at most) and with row remainders,
both SL orders, departure shifts of either sign (the sign of the skews turns
them), tiles of
2 rows (a plan alone) and of 8 (a batch that fills the chip).

Against the march that takes every product by the correlation, which never runs
that kernel: the bar that the two forms are held to elsewhere (1e-11 at tol 1e-12,
the stopping rule's residuals of about 20 steps).  The batch against the plan
alone: another tiling of the same sums, 5e-13.
"""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _plan(n, sl_order=3, skew=-0.1, **kw):
    import torch

    import paper_2511_02700_amd as lp
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    w = workloads.workload("nig64", n=n, N_t=16, theta1=skew, theta2=skew)
    return lp.plan_from_workload(w, sl_order=sl_order, **kw)


def _rel(a, b):
    return float(np.max(np.abs(a - b) / np.maximum(1.0, np.abs(b))))


@pytest.mark.parametrize("n,sl_order,skew", [(17, 3, -0.1), (63, 1, -0.1), (251, 3, -0.1), (252, 3, 0.1), (253, 3, -0.1),
                                             (254, 1, 0.1), (505, 3, -0.1)])
def test_tile_edges(n, sl_order, skew):
    one = _plan(n, sl_order, skew).solve().cpu().numpy()
    ref = _plan(n, sl_order, skew, all_correlations=True).solve().cpu().numpy()
    e = _rel(one, ref)
    print("[gpu-case] n=%d sl_order=%d skew=%g: %.2e" % (n, sl_order, skew, e), flush=True)
    assert np.isfinite(one).all()
    assert e < 1e-11


def test_eight_row_tiles():
    import paper_2511_02700_amd as lp
    sides = [253, 251, 185, 253, 250, 129] * 3
    plans = [_plan(n) for n in sides]
    outs = lp.Batch(plans).solve()
    for q in range(6):
        e = _rel(outs[q].cpu().numpy(), plans[q].solve().cpu().numpy())
        print("[gpu-case] batch member n=%d: %.2e" % (sides[q], e), flush=True)
        assert e < 5e-13
