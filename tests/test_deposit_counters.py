"""The VALU instruction counts of the deposit kernel under profiles/, that bench.py reports while they describe the committed sources:
between bounds per deposited grid point.  Not per (particle, sample, pixel) triple: arrival times are formed only where the
search for the window's grid points needs them, so that a step may take fewer than one wavefront instruction per 64
triples (the precision workload: 3.3e11 for 3.3e13 triples and 5.3e10 points)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("name, points", [("precision", 52661621409), ("bunch", 11087079962)])
def test_instructions_per_deposited_point(name, points):
    path = bench.SUMMARIES[name]["valu"]
    assert os.path.exists(os.path.join(bench.ROOT, path))
    valu = bench._summary_value(path, "sweep_valu_insts_per_step")
    if valu is None:
        pytest.skip("the counters predate the current deposit sources")
    # at least the fields at an interval's two ends and the interpolation, all as fused multiply-adds of 64 full lanes;
    # at most 1024 lane instructions a point
    assert (bench.HIT_F32_FLOPS + bench.POINT_F64_FLOPS) / 2 * points / 64 <= valu <= 1024 * points / 64
