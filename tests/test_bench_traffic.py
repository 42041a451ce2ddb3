"""bench.py reports a committed profile's HBM traffic only while every source
that the profiled kernel is built from is the one the profile was taken from."""
import os
import shutil

import pytest

import bench

CSRC = os.path.dirname(bench.FFN_SOURCE)


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """A copy of the sources, and a profile taken from them."""
    csrc = tmp_path / "csrc"
    shutil.copytree(CSRC, csrc)
    source = str(csrc / "expert_ffn.hip")
    monkeypatch.setattr(bench, "FFN_SOURCE", source)
    monkeypatch.setattr(bench, "ffn_source_key", lambda key=bench.ffn_source_key: key(source))
    profile = tmp_path / "profile.md"
    profile.write_text("traffic_bytes_per_launch (ffn up, read + write): 12345\n"
                       f"ffn_sources_sha256_16: {bench.ffn_source_key()}\n")
    monkeypatch.setattr(bench, "PROFILE", str(profile))
    assert bench.measured_traffic() == 12345
    return csrc


def _edit(path):
    path.write_text(path.read_text() + "\n// changed\n")


@pytest.mark.parametrize("name", ["expert_ffn.hip", "ffn_common.hpp", "common.hpp", "ffn_slim.hpp", "ffn_wide.hpp"])
def test_a_changed_source_drops_the_figure(tree, name):
    _edit(tree / name)
    assert bench.measured_traffic() is None


@pytest.mark.parametrize("name", ["bucket.hip", "combine.hip", "signature.hip", "route.cpp"])
def test_other_sources_keep_it(tree, name):
    _edit(tree / name)
    assert bench.measured_traffic() == 12345


def test_a_profile_without_the_key_is_not_used(tree):
    with open(bench.PROFILE, "w") as f:
        f.write("traffic_bytes_per_launch (ffn up, read + write): 12345\n")
    assert bench.measured_traffic() is None
