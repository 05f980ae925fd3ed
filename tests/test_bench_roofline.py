"""The bench line's roofline is a share of what the units that do the work can reach."""
import pytest

import bench


def test_fp32_scoring_counts_the_bf16_products(monkeypatch):
    monkeypatch.setattr(bench, "_traffic", lambda wl, k: None)
    monkeypatch.setattr(bench, "_valu_issue", lambda ms, wl, k: None)
    flops = 2.0 * 16384 * 1024 * 7552
    feat = bench._kernel_entry(0.8, "hbm", 1.6e9, "ragged", "features")
    score = bench._kernel_entry(1.25, "mfma", flops, "ragged", "score")
    roof = bench._roofline({"features": feat, "score_fp32": score})
    assert roof["kernel"] == "score_fp32"
    assert roof["achieved"] == pytest.approx(6 * flops / 1.25e-3 / 1e12)
    assert roof["peak"] == 2500.0 and roof["unit"] == "BF16 TFLOP/s"
    assert roof["frac"] == pytest.approx(roof["achieved"] / roof["peak"]) and roof["frac"] < 1
    roof = bench._roofline({"features": bench._kernel_entry(2.0, "hbm", 1.6e9, "r", "features"),
                            "score_fp32": score})
    assert roof["kernel"] == "features" and roof["frac"] == pytest.approx(0.1)


def test_precision_shares_count_what_is_executed():
    assert bench.EXEC_FACTOR["fp32"] == 6 and bench.PEAKS_TFLOPS["fp32"] == 2500.0
