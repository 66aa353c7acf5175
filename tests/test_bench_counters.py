"""The counter figures in the benchmark's line belong to the scan kernel they were taken of: none where its sources have changed."""
import os
import shutil
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench


def test_counters_follow_the_sources(tmp_path, monkeypatch):
    name, entry = next(iter(bench.COUNTERS.items()))
    monkeypatch.setattr(bench, "scan_sources_digest", lambda: bench.COUNTERS_SOURCES)
    assert bench.counters_of(name, entry["chunk"]) == entry
    assert bench.counters_of(name, entry["chunk"] + 1) == {} and bench.counters_of(name + "x", entry["chunk"]) == {}
    monkeypatch.setattr(bench, "scan_sources_digest", lambda: "0" * 16)
    assert bench.counters_of(name, entry["chunk"]) == {}


def test_digest_sees_code_and_not_comments(tmp_path):
    csrc = tmp_path / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_2511_10909_amd", "csrc"), csrc)
    before = bench.scan_sources_digest(str(csrc))
    assert before == bench.scan_sources_digest()
    path = csrc / "emulate_scan.hip"
    text = path.read_text()
    path.write_text(text + "\n\n// a comment\n")
    assert bench.scan_sources_digest(str(csrc)) == before
    path.write_text(text + "\nstatic int added;\n")
    assert bench.scan_sources_digest(str(csrc)) != before
