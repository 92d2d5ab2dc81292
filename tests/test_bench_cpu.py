"""The benchmark's stored counters are reported only for the kernel that they were
taken from: a change to any source that is compiled into it withdraws them."""
import json
import os
import shutil

import pytest

import bench

CSRC = os.path.join("paper_2305_01867_amd", "csrc")


@pytest.fixture
def root(tmp_path, monkeypatch):
    os.makedirs(tmp_path / CSRC)
    os.makedirs(tmp_path / "profiles")
    for name in os.listdir(os.path.join(bench.ROOT, CSRC)):
        if name.endswith((".h", ".hip")):
            shutil.copy(os.path.join(bench.ROOT, CSRC, name), tmp_path / CSRC / name)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    rec = {"build": "restructured", "sources_sha256": bench.traversal_hash(), "fetch_bytes_per_launch": 3,
           "write_bytes_per_launch": 4, "counters": {"x": 1}}
    (tmp_path / "profiles" / "traffic.json").write_text(json.dumps({"boolean_certified": rec}))
    return tmp_path


def test_stored_counters_of_the_same_sources(root):
    assert bench.measured_traffic("boolean", "certified", "restructured") == (7, {"x": 1})
    assert bench.measured_traffic("boolean", "certified", "radix_tree") == (None, None)


@pytest.mark.parametrize("name", ["traverse.hip", "segment.h", "pool.h", "rsi_internal.h"])
def test_stored_counters_of_other_sources_are_withdrawn(root, name):
    with open(root / CSRC / name, "a") as fh:
        fh.write("// one more line\n")
    assert bench.measured_traffic("boolean", "certified", "restructured") == (None, None)


def test_every_header_of_the_traversal_is_hashed(root):
    """The sources follow each other by their quoted includes."""
    todo, seen = ["traverse.hip"], set()
    while todo:
        name = todo.pop()
        if name in seen or not os.path.exists(root / CSRC / name):
            continue
        seen.add(name)
        todo += [line.split('"')[1] for line in (root / CSRC / name).read_text().splitlines()
                 if line.startswith('#include "')]
    assert seen == set(bench.TRAVERSAL_SOURCES)
