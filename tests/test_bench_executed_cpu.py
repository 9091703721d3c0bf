"""The headline's roofline states the rate of what the kernel executes: a far
field forms a fraction of the direct sum's pairs, whose rate passed the FP32
vector peak (1.17 of it) and measured nothing."""
import pytest

import bench


def _record(valu):
    return {"achieved": 184.0, "frac": 184.0 / 157.3, "peak": 157.3, "kernel_ms_mean": 0.125, "valu": valu}


def test_executed_flops_are_the_rate():
    r = bench.executed_roofline(_record({"executed_flops_per_launch": 2.5e9, "wait_frac": 0.5}))
    assert r["achieved"] == pytest.approx(20.0) and r["frac"] == pytest.approx(20.0 / 157.3)
    assert r["valu"]["executed_tflops"] == r["achieved"] and r["valu"]["executed_frac"] == r["frac"]
    assert r["valu"]["wait_frac"] == 0.5 and r["direct_sum_tflops"] == 184.0


@pytest.mark.parametrize("valu", [None, {"wait_frac": 0.5}])
def test_without_counters_there_is_no_rate(valu):
    r = bench.executed_roofline(_record(valu))
    assert r["achieved"] is None and r["frac"] is None and r["direct_sum_tflops"] == 184.0
