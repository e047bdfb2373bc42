"""The bench line's roofline of the selection counts bytes that were read."""
import json

import pytest

import bench


@pytest.mark.parametrize("kernel", ["select_split_kernel", "select_hold_kernel", "select_stream_kernel"])
def test_selection_bandwidth_is_the_measured_traffic(kernel):
    # a call that reads 0.8 of 6.2 GB of algorithmic bytes in 1.2 ms
    r = bench.roofline_of("select", "hbm", 6.2e9, 1.2e-3, "bf16", 0.8e9, kernel, 1e8)
    assert r["achieved"] == pytest.approx(0.8e9 / 1.2e-3 / 1e9) and r["frac"] == pytest.approx(r["achieved"] / r["peak"])
    assert r["algorithmic_gbs"] == pytest.approx(6.2e9 / 1.2e-3 / 1e9)
    assert r["achieved_counts"] == "measured traffic"
    assert "cache-resident" not in r["regime"] and "client row" in r["regime"]


def test_selection_without_counters_counts_the_client_matrix_once():
    r = bench.roofline_of("select", "hbm", 6.2e9, 1.2e-3, "bf16", None, None, 1e8)
    assert r["achieved"] == pytest.approx(1e8 / 1.2e-3 / 1e9) and "regime" not in r


def test_other_stages_count_their_algorithmic_bytes():
    r = bench.roofline_of("gains", "hbm", 7e8, 1e-4, "bf16", 7.5e8, "gains_kernel", 1e8)
    assert r["achieved"] == pytest.approx(7000.0) and r["regime"].startswith("bandwidth")


def test_stored_kernels_have_a_regime():
    with open(bench.TRAFFIC_FILE) as f:
        stored = json.load(f)["workloads"]
    for name, ent in stored.items():
        r = bench.roofline_of(ent["stage"], "hbm", 1e9, 1e-3, "bf16", 5e8, ent["kernel"], 1e8)
        assert not r["regime"].endswith(": "), name
