"""The committed HBM counter records belong to the kernels' present code: bench.py
reports `traffic` from them only then."""
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench
from paper_1210_7774_amd import profile_summary as P


@pytest.mark.parametrize("record", sorted(P.RECORDS))
def test_record_is_of_the_present_code(record):
    with open(os.path.join(ROOT, "profiles", record)) as fh:
        rec = json.load(fh)
    assert rec["source_hash"] == P.code_hash(P.RECORDS[record]), \
        "the kernels changed: take the counters again (profiles/, FETCH_SIZE and WRITE_SIZE)"


@pytest.mark.parametrize("kernel", ["pre n=4095", "post n=4095", "w2pre_rr n=511", "w2post_norm n=511"])
def test_bench_reports_the_dominant_kernels(kernel):
    assert bench.traffic_of(kernel) > 0


def test_comments_do_not_count(tmp_path, monkeypatch):
    monkeypatch.setattr(P, "CSRC", str(tmp_path))
    (tmp_path / "a.hip").write_text("int x;  // one\n/* two\n lines */ int y;\n")
    one = P.code_hash(["a.hip"])
    (tmp_path / "a.hip").write_text("int x;\n\nint y;  // other words\n")
    assert P.code_hash(["a.hip"]) == one
    (tmp_path / "a.hip").write_text("int x;\nint z;\n")
    assert P.code_hash(["a.hip"]) != one
