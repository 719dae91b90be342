"""bench.py's rooflines of the FP64 products: each route against its own peak."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def _info(**k):
    return {"gemm_kernel_ms": 100.0, "gemm_flops": 8e12, "gemm_launches": 1000, **k}


def test_routes_have_their_own_peaks():
    infos = [_info(residue_ms=60.0, residue_flops=6e12, residue_launches=100)] * 2 + \
            [{"gemm_kernel_ms": 0.0, "gemm_flops": 0.0, "gemm_launches": 0}]  # carried no events
    r = bench._roofline_gemm(infos)
    # 6e12 flops are 4.8e13 INT8 operations in 60 ms
    assert r["unit"] == "TOP/s" and abs(r["achieved"] - 800.0) < 1e-9
    assert abs(r["frac"] - 800.0 / bench.PEAK_TFLOPS["i8"]) < 1e-12
    assert r["kernel_ms_per_step"] == 60.0 and r["family_ms_per_step"] == 100.0
    o = r["other_route"]
    assert o["unit"] == "TFLOP/s" and abs(o["achieved"] - 50.0) < 1e-9 and o["launches"] == 1800
    assert abs(o["executed_frac"] - 0.75 * 50.0 / 78.6) < 1e-12


def test_without_residue_products():
    r = bench._roofline_gemm([_info()])
    assert r["unit"] == "TFLOP/s" and abs(r["frac"] - 80.0 / 78.6) < 1e-12 and "other_route" not in r
