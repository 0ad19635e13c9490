"""The key under which the benchmark keeps hardware counters: every file of the library's kernels."""
import os
import re
import shutil

import bench

CSRC = os.path.join("paper_1710_11246_amd", "csrc")


def test_a_change_of_any_kernel_file_changes_the_key(tmp_path, monkeypatch):
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    names, todo = set(), ["slabhash.hip"]
    while todo:  # the file and what it includes from its own folder
        f = todo.pop()
        if f in names or not (tmp_path / CSRC / f).exists():
            continue
        names.add(f)
        todo += re.findall(r'#include "([^"]+)"', (tmp_path / CSRC / f).read_text())
    assert {"slabhash.hip", "bulk.hpp", "bulk_plan.hpp"} <= names
    for f in sorted(names):
        before = bench.source_sha()
        with open(tmp_path / CSRC / f, "a") as out:
            out.write("// another line\n")
        assert bench.source_sha() != before, f
    before = bench.source_sha()
    with open(tmp_path / CSRC / "roofs.hip", "a") as out:  # of another library
        out.write("// another line\n")
    assert bench.source_sha() == before
