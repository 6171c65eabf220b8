"""Host-side checks of bench.py: which memory counters its line may quote."""
import json
import os

import pytest

import bench

SHAPE = dict(variant=2, sib_blocks=1, tile_z=16, tile_y=16)
OTHER = dict(SHAPE, variant=6)


@pytest.fixture
def profiles(tmp_path, monkeypatch):
    """An empty profiles/ beside the sources; write(lines) fills one summary."""
    os.mkdir(tmp_path / "profiles")
    monkeypatch.setattr(bench, "kernel_source_hash", lambda: "0123")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))

    def write(*entries):
        with open(tmp_path / "profiles" / "counters_w.md", "w") as f:
            f.write("# counters\n\ntext\n")
            for e in entries:
                f.write("traffic-json: %s\n" % json.dumps(e))
    return write


def _entry(shape, read, **kw):
    e = dict(source_hash="0123", fetch_scale=2.0, write_scale=1.0,
             kernels={"block": {"fetch_kib": read, "write_kib": 1.0}})
    if shape is not None:
        e["shape"] = shape
    e.update(kw)
    return e


def test_traffic_of_the_installed_shape(profiles):
    """The counters of the launch shape that the solves ran, no other's."""
    profiles(_entry(OTHER, 100.0), _entry(SHAPE, 10.0))
    assert bench.measured_traffic("block", "w", SHAPE) == (2 * 10 + 1) * 1024
    assert bench.measured_traffic("block", "w", OTHER) == (2 * 100 + 1) * 1024
    assert bench.measured_traffic("block", "w", dict(SHAPE, variant=1)) is None
    assert bench.measured_traffic("block", "w", dict(SHAPE, tile_y=8)) is None
    assert bench.measured_traffic("gs_dot", "w", SHAPE) is None   # not counted
    assert bench.measured_traffic("block", "v", SHAPE) is None    # no summary


def test_no_traffic_of_an_unnamed_shape_or_other_sources(profiles):
    profiles(_entry(None, 10.0))
    assert bench.measured_traffic("block", "w", SHAPE) is None
    profiles(_entry(SHAPE, 10.0, source_hash="4567"))
    assert bench.measured_traffic("block", "w", SHAPE) is None
