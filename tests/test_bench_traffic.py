"""The counted traffic the benchmark prints beside a timed sweep is of a launch of the same shape:
counts of two-step sweeps with other units, or of another unit rule, are not used.  CPU only."""
import json

import _host_plan as H
import bench


def test_counts_of_another_shape_are_not_used(tmp_path, monkeypatch):
    good = dict(kernel="k", cells=100, kernel_source_sha256_16=bench.kernel_source_hash(), steps_per_launch=2,
                rows_per_unit=bench.ROWS_PER_UNIT, hbm_bytes_per_launch=7)
    f = tmp_path / "t.json"
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(f))
    monkeypatch.setattr(bench, "TRAFFIC_FILE_BEYOND", str(f))
    for change, used in (({}, True), ({"rows_per_unit": 8}, False), ({"rows_per_unit": None}, False),
                         ({"steps_per_launch": 1, "rows_per_unit": None}, True), ({"cells": 99}, False)):
        e = {**good, **change}
        f.write_text(json.dumps(e))
        assert (bench.measured_traffic(100)["traffic"] == 7) == used
        f.write_text(json.dumps({**good, "entries": [{**e, "storage": "fp32"}]}))
        assert (bench.measured_traffic_beyond("fp32", 100)["traffic"] == 7) == used


def test_rows_of_the_timed_sweeps():
    for nx, ny in ((4096, 1024), (8192, 4096)):
        assert H.lattice(nx, ny, "fp32")["rows_particle"] == bench.ROWS_PER_UNIT


def test_the_unit_rule_counts(tmp_path, monkeypatch):
    was = bench.kernel_source_hash()
    text = open(bench.os.path.join(bench.CSRC, "lbib_host.cpp")).read()
    (tmp_path / "lbib_host.cpp").write_text(text.replace("? 16 :", "? 12 :"))
    assert text.count("? 16 :") == 1
    monkeypatch.setattr(bench, "CSRC", str(tmp_path))
    assert bench.kernel_source_hash() != was
