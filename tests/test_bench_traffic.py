"""The HBM traffic that bench.py reports for the FP64 J v element pass: its counters where
they were taken for the source at hand, null for another source or workload."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_counters_of_the_source_at_hand(monkeypatch):
    monkeypatch.setattr(bench, "ELEM_TRAFFIC_SRC_SHA256", bench.elem_source_sha256())
    for config, n_el, n_nodes in ((2, 64 ** 3, 65 ** 3), (3, 160 * 160 * 320, 161 * 161 * 321)):
        read, written = bench.ELEM64_COUNTERS_KIB[config]
        got = bench.reported_traffic(config)
        assert got == pytest.approx(1024 * (read * bench.FETCH_SCALE + written * bench.WRITE_SCALE))
        # at least x, v, gamma and s read once and J v written once; tiles' rims at most double it
        least = bench.jv_bytes(n_nodes, n_el)
        assert 0.99 * least <= got <= 2.5 * least
    assert bench.reported_traffic(4) is None


def test_another_source_reports_no_traffic(monkeypatch):
    monkeypatch.setattr(bench, "ELEM_TRAFFIC_SRC_SHA256", "0" * 64)
    assert bench.reported_traffic(2) is None and bench.reported_traffic(3) is None
