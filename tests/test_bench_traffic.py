"""bench.py's traffic record (no GPU): no kernel of the launch may be missing from it."""
import json
import os

import pytest

import bench
from test_bench_host import _counters


@pytest.fixture
def record(tmp_path, monkeypatch):
    """record(f, w): the record of two counter files, each edited by a function of its text"""
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles").mkdir()
    for s in bench.TRAFFIC_SOURCES:
        os.makedirs(os.path.dirname(tmp_path / s), exist_ok=True)
        (tmp_path / s).write_text("")

    def make(edit_fetch=lambda t: t, edit_write=lambda t: t):
        f, w = tmp_path / "f.csv", tmp_path / "w.csv"
        for path, counter, edit in ((f, "FETCH_SIZE", edit_fetch), (w, "WRITE_SIZE", edit_write)):
            _counters(path, counter, [100.0, 102.0], 262144.0)
            path.write_text(edit(path.read_text()))
        bench.write_traffic(str(f), str(w), "divrem_2p16_b4096")
        return json.load(open(tmp_path / "profiles" / "k_divrem_2p16_b4096_traffic.json"))
    return make


def test_every_division_kernel_counts(record):
    one = lambda t: "\n".join(x for x in t.splitlines() if "k_head" not in x) + "\n"  # noqa: E731
    r = record(one, one)
    assert len(r["kernels"]) == 1 and abs(r["traffic_bytes_per_dispatch"] - 1024 * 202.0) < 1e-6
    r = record()
    assert len(r["kernels"]) == 2 and abs(r["traffic_bytes_per_dispatch"] - 1024 * 204.0) < 1e-6
    r = record(*[lambda t: t.replace("k_head_divrem", "k_other_divrem")] * 2)        # a kernel of another name
    assert abs(r["traffic_bytes_per_dispatch"] - 1024 * 204.0) < 1e-6


def test_a_missing_kernel_is_an_error(record):
    lost = lambda t: "\n".join(x for x in t.splitlines() if "k_divrem<" not in x) + "\n"  # noqa: E731
    other = lambda t: "\n".join(x for x in t.splitlines() if "k_head" not in x) + "\n"  # noqa: E731
    for edits in ((lost, lost), (lost,), (other,)):
        with pytest.raises(AssertionError):
            record(*edits)
