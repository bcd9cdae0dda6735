"""bench.py: the fabric traffic it carries belongs to the sources that the counters were taken on."""
import os
import shutil
from types import SimpleNamespace

import pytest

import bench
from paper_2511_19835_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "paper_2511_19835_amd", "csrc")


@pytest.mark.parametrize("changed", [None, "attn_kernels.hip", "attn_side_kernels.hip", "attn_sched.hpp"])
def test_traffic_goes_with_its_sources(tmp_path, monkeypatch, changed):
    """A change to the kernel, to the kernels that order and deal its rows or to the rules of the schedule: null."""
    csrc = tmp_path / "paper_2511_19835_amd" / "csrc"
    shutil.copytree(CSRC, csrc)
    monkeypatch.setattr(bench, "__file__", str(tmp_path / "bench.py"))
    monkeypatch.setattr(bench, "MEASURED_TRAFFIC_SHA", bench.traffic_sources_sha(CSRC))
    if changed:
        with open(csrc / changed, "a") as f:
            f.write("\n")
    got = bench.measured_traffic(synth.CONFIGS["hunyuan"], 0.9, SimpleNamespace(mask_rule="topk", seed=0))
    assert (got is None) == (changed is not None)
