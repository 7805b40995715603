"""The benchmark's roofline of a walk in cells, from its committed counter record, without a GPU."""
from __future__ import annotations

import json

import pytest

import bench


@pytest.fixture()
def record(monkeypatch):
    with open(bench.CELLS_RECORD) as fh:
        rec = json.load(fh)
    monkeypatch.setattr(bench, "source_sha256", lambda: rec["source_sha256"])
    return rec


def test_cells_roofline_reproduces_the_record(record):
    ms = sum(k["ms"] for k in record["kernel_ms_per_run"].values())
    roof = bench.cells_roofline(record["photons"], record["photon_steps"], ms)
    assert (roof["bound"], roof["kernel"], roof["unit"]) == ("valu", "k_cells_walk", "photon-steps/s")
    assert roof["achieved"] == pytest.approx(record["photon_steps"] / ms * 1e3)
    # the VALU of k_cells_walk busy for so much of the run's time
    share = record["kernel_ms_per_run"]["k_cells_walk"]["ms"] / ms
    assert roof["frac"] == pytest.approx(roof["achieved"] / roof["peak"])
    assert roof["frac"] == pytest.approx(record["k_cells_walk"]["valu_busy"] * share, rel=0.08)
    assert roof["traffic"] == pytest.approx(record["traffic_bytes_per_run"])
    assert 1.5e9 < record["clock_hz"] < 3.0e9


def test_cells_roofline_scales_with_the_run(record):
    full = bench.cells_roofline(record["photons"], record["photon_steps"], 500.0)
    half = bench.cells_roofline(record["photons"] // 2, record["photon_steps"] // 2, 250.0)
    assert half["frac"] == pytest.approx(full["frac"]) and half["traffic"] == pytest.approx(full["traffic"] / 2)


def test_cells_roofline_without_a_matching_record(monkeypatch):
    monkeypatch.setattr(bench, "source_sha256", lambda: "0" * 64)
    roof = bench.cells_roofline(10 ** 8, 10 ** 11, 500.0)
    assert roof["peak"] is None and roof["frac"] is None and roof["traffic"] is None
    assert roof["achieved"] == pytest.approx(2e11)


def test_form_roofline_names_the_kernel():
    cells = bench.form_roofline("batched", True, 10 ** 11, 900.0)
    assert (cells["kernel"], cells["bound"], cells["achieved"]) == ("k_cells_walk", "valu", pytest.approx(1e11 / 0.9))
    assert bench.form_roofline("differentiated", False, 10 ** 11, 900.0)["kernel"] == "k_walk"
