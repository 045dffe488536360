"""The benchmark's signature roofline describes the kernel that runs: no unit's
share of its measured peak exceeds one at the recorded time (2.05e7
ROI-directions of 1006 atoms in 8.8 ms), and the work per unit is that of the
matrix-core form."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

PEAKS = {"fp32_fma_flop_per_s": 70.6e12, "bf16_mfma_flop_per_s": 2.02e15, "lds_atomics_per_s": 8.9e12,
         "lds_bytes_per_s": 117e12}


def test_work_per_unit():
    w = bench.signature_work(1000.0, 1024)
    assert w["fp32_flops"] == 7000 + 8 * 32 * 16 + 128
    assert w["fp16_mfma_flops"] == 2 * 2 * 16 * 32 * 32 * 2
    assert w["lds_bytes"] == 3000 + 4096 + 256 and w["lds_atomics"] == 1000
    assert w["paper_flops"] == 7000 + 25600


def test_no_unit_past_its_peak():
    r = bench.signature_roofline(1006.0, 1024, 2000 * 10242.0, 8.8e-3, PEAKS)
    assert r["kernel"].startswith("k_signatures_persistent_mm<10>")
    assert 0.2 < r["frac"] < 1.0 and max(r["frac_by_unit"].values()) == r["frac"]
