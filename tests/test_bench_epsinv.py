"""The flops that bench.py counts for the Gauss-Jordan inverse, against a walk over the
steps and tiles that the kernels run for a Hermitian matrix."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402


@pytest.mark.parametrize("n", [1, 64, 65, 128, 200, 1000])
def test_executed_flops(n):
    nt = -(-n // 64)
    flops = 0
    for s in range(nt if nt > 1 else 0):
        k = min(64, n - 64 * s)
        flops += 6 * k * k * n  # row panel: Dinv times the block row
        for ti in range(nt):
            for tj in range(ti + 1):
                if ti != s:  # the block row is rewritten by the next step
                    flops += 6 * k * 64 * 64
    assert bench.epsinv_flops(n) == flops


def test_rate_is_of_executed_flops():
    r = bench.epsinv_roofline({"gj_update": (63, 6.0)}, {"neps": 4000, "omega": [0.0]})
    assert r["achieved"] == pytest.approx(bench.epsinv_flops(4000) / 6e-3 / 1e12)
    assert r["algorithmic_TFLOP_per_s"] == pytest.approx(8 * 4000.0 ** 3 / 6e-3 / 1e12)
    # six flops for eight, half of the blocks
    assert 0.36 < r["achieved"] / r["algorithmic_TFLOP_per_s"] < 0.41
