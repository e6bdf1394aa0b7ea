"""bench.py reports counters only for the source and the launch shapes that they were taken at."""
import hashlib

import pytest

import bench


@pytest.fixture
def profile(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles").mkdir()
    csrc = tmp_path / "paper_1412_5989_amd" / "csrc"
    csrc.mkdir(parents=True)
    (csrc / "k.hip").write_text("source")

    def write(shape):
        digest = hashlib.sha256((csrc / "k.hip").read_bytes()).hexdigest()
        (tmp_path / "profiles" / "p.md").write_text(
            "# kernel\n\ntraffic_bytes_per_launch: 7\nkernel_source_files: k.hip\nkernel_source_sha256: %s\n%s" % (digest, shape))
        return csrc / "k.hip"

    return write


SHAPE = {"adj_rows": 64, "adj_tile_n": 8}


def test_same_shape(profile):
    profile("launch_shape: adj_wide=1,adj_rows=64,adj_tile_n=8\n")
    assert bench.measured_counters("p.md", SHAPE) == {"traffic_bytes_per_launch": 7}
    assert bench.measured_counters("p.md") == {"traffic_bytes_per_launch": 7}


@pytest.mark.parametrize("shape", ["", "launch_shape: adj_rows=64\n", "launch_shape: adj_rows=64,adj_tile_n=16\n"])
def test_other_or_no_shape(profile, shape):
    profile(shape)
    assert bench.measured_counters("p.md", SHAPE) is None


def test_other_source(profile):
    profile("launch_shape: adj_rows=64,adj_tile_n=8\n").write_text("other")
    assert bench.measured_counters("p.md", SHAPE) is None


def test_leg_finds_the_summary_of_its_shape(profile, tmp_path):
    profile("launch_shape: adj_rows=64,adj_tile_n=8\n")
    other = (tmp_path / "profiles" / "p.md").read_text().replace("launch: 7", "launch: 9").replace("=64", "=96")
    (tmp_path / "profiles" / "p_96x8.md").write_text(other)
    for rows, traffic, name in ((64, 7, "p.md"), (96, 9, "p_96x8.md"), (32, None, None)):
        r = bench.leg(1.0, 1, 8, "p.md", {"adj_rows": rows, "adj_tile_n": 8})["roofline"]
        assert (r["traffic"], r["profile"]) == (traffic, name)
