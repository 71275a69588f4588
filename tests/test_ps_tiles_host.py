"""What the host-only discretization reports of the price-space correlation's
tiles (side and number per axis): one transform of the side where it is the
faster form, tiles below and above #in = 8192.  No device is touched."""

import csv
import os

import pytest

GOLD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
GRID = {"VG0": (5700.0, 21.6164), "VG1": (500.0, 67.1487), "NIG0": (600.0, 55.0673),
        "NIG1": (700.0, 45.0189)}     # x_max, c of Sec. 4


def _info(name, N_x, **kw):
    import paper_2511_02700_amd as lp
    with open(os.path.join(GOLD, "table1_params.csv")) as f:
        q = {r["name"]: r for r in csv.DictReader(line for line in f if not line.startswith("#"))}[name]
    lv = lp.levy_nts(float(q["alpha"]), float(q["delta"]), float(q["lambda"]), (float(q["eta1"]), float(q["eta2"])),
                     (float(q["rho11"]), float(q["rho12"]), float(q["rho22"])), float(q["r"]))
    x_max, c = GRID[name]
    return lp.ps_discretize_host(lp.make_ps_grid(N_x, x_max, c=c, **kw), lv, lp.make_payoff("put_avg", 100.0, 0.5))[0]


@pytest.mark.parametrize("name,N_x,L,side,tiles", [("VG1", 48, 512, 512, 1), ("NIG0", 128, 4096, 4096, 1),
                                                   ("NIG0", 168, 6144, 3072, 2), ("NIG0", 244, 12288, 3584, 3),
                                                   ("NIG0", 328, 12288, 4096, 4), ("NIG1", 336, 7168, 4096, 2)])
def test_reported_tiles(name, N_x, L, side, tiles):
    i = _info(name, N_x)
    assert (i["L"], i["tile_L"], i["tiles"]) == (L, side, tiles)
    if tiles > 1:      # the tiles' kept outputs, advancing by side - 2 N_z - 2, cover the #out - 3 stencil starts
        vs = side - 2 * i["N_z"] - 2
        assert (tiles - 1) * vs < i["n_out"] - 3 <= tiles * vs
    else:
        assert side >= i["n_in"]


def test_no_tiles_without_jumps():
    import paper_2511_02700_amd as lp
    i = lp.ps_discretize_host(lp.make_ps_grid(32, 500.0), lp.levy_black_scholes(0.0, (0.04, 0.0, 0.04)),
                              lp.make_payoff("put_avg", 100.0, 1.0))[0]
    assert (i["L"], i["tile_L"], i["tiles"]) == (0, 0, 0)


@pytest.mark.parametrize("name,N_x,nz,side,tiles", [
    ("NIG0", 448, 2, 7168, 3), ("NIG1", 600, 2, 8192, 2), ("NIG1", 656, 2, 7168, 3), ("NIG1", 760, 2, 8192, 3),
    ("NIG0", 264, 2, 4096, 3), ("VG1", 1096, 2, 12288, 1), ("VG0", 488, 6, 12288, 1)])
def test_faster_form_above_8192(name, N_x, nz, side, tiles):
    """Above #in = 8192 the rule takes the form that is measured to be the faster one: tiles against
    the two-level transform 2.32 ms : 3.57 (NIG0 448), 1.28 : 1.66 (NIG1 600), 2.37 : 2.90 (656), 2.73 : 3.64 (760),
    nine tiles of 4096 against four of 5120 0.52 : 0.59 (NIG0 264); and the transform where the weights leave a tile
    few outputs, 1.63 : 2.53 (VG1 1096), or its own are few, 1.07 : 1.20 (VG0 488 with N_z = 6 N_x)."""
    i = _info(name, N_x, nz_per_nx=nz)
    assert (i["tile_L"], i["tiles"]) == (side, tiles)
