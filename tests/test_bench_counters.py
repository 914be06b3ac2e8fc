"""The roofline of bench.py: figures from the committed counters, for the sources
that they were taken on only."""
import hashlib
import json

import bench


def _record(root, sources, **over):
    h = hashlib.sha256()
    for f in sources:
        h.update(open(root / f, "rb").read())
    rec = dict(sources_sha256_16=h.hexdigest()[:16], fetch_kib=[1000], write_kib=[500], fetch_factor=2.0,
               write_factor=1.0, valu_busy=0.99, valu_lanes=0.44, l1_data_busy=0.88)
    rec.update(over)
    (root / "profiles" / "k_trace_pmc_soup1M.md").write_text("text\n\ntraffic-record: " + json.dumps(rec) + "\n")


def test_counters_of_these_sources_only(tmp_path, monkeypatch):
    (tmp_path / "profiles").mkdir()
    for f in ("a.h", "b.hip"):
        (tmp_path / f).write_text(f)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "TRACE_SOURCES", ["a.h", "b.hip"])
    assert bench.measured_counters() is None  # no record
    _record(tmp_path, ["a.h", "b.hip"])
    c = bench.measured_counters()
    assert c == dict(bytes=1024.0 * 2500, valu_busy=0.99, valu_lanes=0.44, l1_data_busy=0.88)
    (tmp_path / "b.hip").write_text("changed")
    assert bench.measured_counters() is None  # nothing is put in its place


def test_sources_exist_and_order_the_nodes():
    assert any(f.endswith("sppm_scan.h") for f in bench.TRACE_SOURCES)  # its scan numbers the four-child nodes
    for f in bench.TRACE_SOURCES:
        open(f"{bench.ROOT}/{f}").close()
