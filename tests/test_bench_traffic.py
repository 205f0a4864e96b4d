"""The measured HBM traffic that bench.py reports belongs to the kernel sources it was taken on: a change of the kernel's file or of
any header it includes makes the figure void.  CPU only."""
import os
import shutil

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2501_08090_amd", "csrc")


@pytest.mark.parametrize("src,changed,void", [("attention.hip", "attention.hip", True), ("attention.hip", "attn_plan.h", True),
                                              ("attention.hip", "device_util.h", True), ("attention.hip", "linear.hip", False),
                                              ("linear.hip", "chiron_internal.h", True), ("linear.hip", "attn_plan.h", False)])
def test_a_changed_source_or_header_voids_the_figure(tmp_path, src, changed, void):
    csrc = str(tmp_path / "csrc")
    shutil.copytree(CSRC, csrc)
    before = bench.source_hash(src, csrc)
    assert before == bench.source_hash(src)
    with open(os.path.join(csrc, changed), "a") as f:
        f.write("// changed\n")
    assert (bench.source_hash(src, csrc) != before) == void


def test_figures_are_reported_for_their_own_sources_only(monkeypatch):
    key = ("llama8b-b64-lognormal800", "attn")
    src, _, fetch, write = bench.TRAFFIC[key]
    monkeypatch.setitem(bench.TRAFFIC, key, (src, bench.source_hash(src), fetch, write))
    assert bench.measured_traffic(*key) == dict(fetch_bytes=fetch, write_bytes=write, total_bytes=fetch + write)
    monkeypatch.setitem(bench.TRAFFIC, key, (src, "0" * 64, fetch, write))
    assert bench.measured_traffic(*key) is None
    assert bench.source_hash("missing.hip") is None
