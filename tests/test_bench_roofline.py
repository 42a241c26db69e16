"""The benchmark's roofline leads with bytes that were moved: a rate above the
device's peak can only be the streaming model's, and says so."""
import pytest

import bench


def test_measured_bytes_lead():
    r = bench.roofline(1.32e12, 2.31e12, 275.0, "k", (256, 1024, 1, 0))
    assert r["achieved"] == pytest.approx(1.32e12 / 0.275 / 1e9, abs=0.1)
    assert r["frac"] == pytest.approx(r["achieved"] / r["peak"], abs=1e-4) and r["frac"] < 1.0
    assert r["achieved_from"].startswith("measured")
    assert r["algorithmic_rate_GBs"] == pytest.approx(2.31e12 / 0.275 / 1e9, abs=0.1)
    assert r["traffic_over_algorithmic"] == pytest.approx(1.32 / 2.31, abs=1e-3)


def test_the_model_is_named_where_nothing_was_measured():
    r = bench.roofline(None, 2.31e12, 275.0, "k", (0, 0, 0, 0))
    assert r["achieved"] == r["algorithmic_rate_GBs"] and r["traffic"] is None
    assert r["achieved_from"] == "streaming model, no measured bytes"
    assert bench.roofline(None, 1.0, 0.0, "k", ())["achieved"] == 0.0
