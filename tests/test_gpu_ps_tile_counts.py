"""The price-space correlation by overlap-save tiles with the tile side and the
number of tiles per axis asserted, so that a rule that stops tiling cannot pass
as agreement of one form with itself: two tiles per axis (all of them first or
last ones) below and above #in = 8192, and three, four and six (interior tiles,
the block decode for more than two), against the same correlation as one
transform of the side forced; two of them against the oracle as well.

Bars: those of the operator against the oracle, 1e-12 of max |B v| off the x = 0
rows and, on them, that times the square of the absolute sum of T^out's
extrapolating row.
"""

import csv
import math
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GOLD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
GRID = {"NIG0": (600.0, 55.0673), "NIG1": (700.0, 45.0189)}     # x_max, c of Sec. 4


def _params(name):
    with open(os.path.join(GOLD, "table1_params.csv")) as f:
        return {r["name"]: r for r in csv.DictReader(line for line in f if not line.startswith("#"))}[name]


@pytest.fixture(scope="module")
def lp():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    import paper_2511_02700_amd as m
    return m


def _plan(lp, name, N_x, **opts):
    q = _params(name)
    lv = lp.levy_nts(float(q["alpha"]), float(q["delta"]), float(q["lambda"]), (float(q["eta1"]), float(q["eta2"])),
                     (float(q["rho11"]), float(q["rho12"]), float(q["rho22"])), float(q["r"]))
    x_max, c = GRID[name]
    return lp.PsPlan(lp.make_ps_grid(N_x, x_max, c=c), lv, lp.make_payoff("put_avg", 100.0, 0.5), N_t=4, **opts)


def _close(got, want, t0, tag):
    scale = np.max(np.abs(want))
    e_in = float(np.max(np.abs(got - want)[1:, 1:])) / scale
    e_all = float(np.max(np.abs(got - want))) / scale
    print("[gpu-case] %s: interior %.2e, all rows %.2e" % (tag, e_in, e_all), flush=True)
    assert e_in < 1e-12
    assert e_all < 1e-12 * t0 * t0


@pytest.mark.parametrize("name,N_x,side,tiles", [
    ("NIG0", 168, 3072, 2), ("NIG0", 200, 3584, 2), ("NIG1", 336, 4096, 2), ("NIG0", 360, 7168, 2),
    ("NIG0", 361, 8192, 2),
    ("NIG0", 244, 3584, 3), ("NIG0", 268, 4096, 3), ("NIG0", 328, 4096, 4), ("NIG0", 440, 4096, 6),
    ("NIG1", 800, 8192, 3)])
def test_tiles_match_one_transform(lp, name, N_x, side, tiles):
    import torch
    print("[gpu-case] %s N_x=%d: %d tiles of %d" % (name, N_x, tiles, side), flush=True)
    tiled = _plan(lp, name, N_x)
    info = tiled.info()
    assert (info["tile_L"], info["tiles"]) == (side, tiles)
    one = _plan(lp, name, N_x, fft_size=info["L"])
    o = one.info()
    assert (o["L"], o["tile_L"], o["tiles"]) == (info["L"], info["L"], 1)
    n = N_x + 1
    v = torch.from_numpy(np.random.default_rng(N_x).standard_normal((n, n)) * 10.0).to(tiled.device) + tiled.initial()
    e = math.exp(info["h_z"])
    _close(tiled.apply_B(v).cpu().numpy(), one.apply_B(v).cpu().numpy(), (e + 1.0) / (e - 1.0),
           "%s N_x=%d" % (name, N_x))


@pytest.mark.parametrize("N_x,tiles", [(168, 2), (244, 3)])
def test_tiles_match_oracle(lp, N_x, tiles):
    import torch
    from oracle import levy
    from oracle import price_space as ps
    print("[gpu-case] NIG0 N_x=%d against the oracle" % N_x, flush=True)
    plan = _plan(lp, "NIG0", N_x)
    assert plan.info()["tiles"] == tiles
    q = _params("NIG0")
    p = levy.nts_params(float(q["alpha"]), float(q["delta"]), float(q["lambda"]), (float(q["eta1"]), float(q["eta2"])),
                        ((float(q["rho11"]), float(q["rho12"])), (float(q["rho12"]), float(q["rho22"]))))
    x_max, c = GRID["NIG0"]
    prob = ps.PriceSpaceProblem(p, N_x, 100.0, x_max, 0.5, 4, float(q["r"]), c=c)
    v = np.random.default_rng(N_x).standard_normal((N_x + 1, N_x + 1)) * 10.0 + prob.V0()
    got = plan.apply_B(torch.from_numpy(v)).cpu().numpy()
    _close(got, prob.B(v), float(np.abs(prob.T_out[0].toarray()).sum()), "NIG0 N_x=%d" % N_x)
