"""The hash that says which solver source the committed launch shapes and
counter summaries were made for covers everything the solver's kernels are
compiled from."""
import os
import re
import shutil

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_1709_09763_amd", "csrc")


def _included(name, seen):
    """what the compiler would read of this folder for `name`"""
    if name not in seen:
        seen.add(name)
        for line in open(os.path.join(CSRC, name)):
            m = re.match(r'#include "(\w+\.h)"', line)
            if m:
                _included(m.group(1), seen)
    return seen


NAMES = sorted(_included("solver.hip", set()))


def test_the_kernels_headers_are_among_them():
    assert {"solver.hip", "common.h", "walks.h", "lanes.h", "strips.h", "strips7.h"} <= set(NAMES)
    assert [os.path.basename(f) for f in bench.solver_sources()] == NAMES


@pytest.mark.parametrize("name", NAMES)
def test_an_edit_of_any_of_them_changes_the_stamp(name, tmp_path, monkeypatch):
    before = bench.solver_sha()
    copy = tmp_path / "paper_1709_09763_amd" / "csrc"
    shutil.copytree(CSRC, copy)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.solver_sha() == before
    with open(copy / name, "a") as f:
        f.write("// edited\n")
    assert bench.solver_sha() != before
