"""The kernels that bench.py names for its timing classes are the ones the march
launches with its present schedules (FP64 and the mixed form have one each), the
launch that starts a steady FP64 step among them, and each is found in the
committed counter summaries by the name bench.py looks up."""
import json
import os

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# (workload, transform side, n): elements per thread of the columns, row c2r, line rows, SL
SCHEDULE = {("nig2048_m", 3072, 2048): {"fp64": (4, 4, 4, 4), "fp32conv": (4, 4, 16, 4)},
            ("fv512", 1024, 512): {"fp64": (4, 4, 4, 4), "fp32conv": (16, 4, 4, 4)}}
CASES = [(w, p) for w in SCHEDULE for p in ("fp64", "fp32conv")]


@pytest.mark.parametrize("workload, precision", CASES)
def test_names_are_profiled(workload, precision):
    name, L, n = workload
    with open(os.path.join(ROOT, "profiles", "pmc_%s.json" % name)) as fh:
        kernels = [k[5:] if k.startswith("void ") else k for k in json.load(fh)["kernels"]]
    mixed = precision == "fp32conv"
    for cls in ("line_rows", "cols", "rows_inv", "sl") + (() if mixed else ("sl_lin", "rows_lin")):
        sym = bench.kernel_symbol(cls, L, mixed, 3, SCHEDULE[workload][precision], n)
        assert [k for k in kernels if k.startswith(sym + "(")], (cls, sym)


def test_step_begin_rows_rule():
    # tiles of 8 rows where 1024 of them (four blocks on each of 256 CUs) cover the grid, else of 2
    assert bench.step_begin_rows(2048) == 8      # 256 x 9 tiles of 240 columns
    assert bench.step_begin_rows(1250) == 2      # 157 x 5
    assert bench.step_begin_rows(1280) == 2      # 160 x 6 = 960
    assert bench.step_begin_rows(1366) == 8      # 171 x 6 = 1026
    assert bench.step_begin_rows(512) == 2       # 64 x 3


@pytest.mark.gpu
@pytest.mark.parametrize("workload, precision", CASES)
def test_schedules_are_the_march_s(workload, precision):
    import paper_2511_02700_amd as lp
    import workloads
    name, L, n = workload
    print("[gpu-case] schedule of %s %s" % (name, precision), flush=True)
    info = lp.plan_from_workload(workloads.workload(name), precision=precision).info()
    assert (info["L"], info["n"]) == (L, n)
    assert tuple(info["radix"]) == SCHEDULE[workload][precision]
