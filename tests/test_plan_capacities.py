"""Capacities that a captured run is planned for (csrc/plan.hpp), on the CPU:
headroom over what the eager call met, and never more nodes than an entry of a
node list can name (csrc/runs.hpp holds a node above 6 bits of a 32-bit word)."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "plan.hpp"
extern "C" int64_t grids(int64_t n, int64_t g, int levels) { return gd::planned_grids(n, g, levels != 0); }
extern "C" int64_t nodes(int64_t ncell, int64_t m) { return gd::planned_nodes(ncell, m); }
"""
MOST = (2**32 >> 6) - 1  # nodes 0 .. MOST fit an entry


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    so = str(tmp_path_factory.mktemp("plan") / "plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-x", "c++", "-",
                    "-I", os.path.join(ROOT, "paper_2210_07580_amd", "csrc"), "-o", so],
                   input=SOURCE, text=True, check=True)
    lib = ctypes.CDLL(so)
    for f in (lib.grids, lib.nodes):
        f.restype = ctypes.c_int64
    lib.grids.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    lib.nodes.argtypes = [ctypes.c_int64, ctypes.c_int64]
    return lib


@pytest.mark.parametrize("grids", [1, 1000, 60_000_000, 63_200_000, MOST - 5000, MOST])
def test_levels_never_plan_for_nodes_an_entry_cannot_name(plan, grids):
    n = 2**31 - 1
    most = plan.grids(n, grids, 1)
    assert grids <= most <= MOST
    assert grids <= plan.nodes(most, grids) <= most
    assert most == min(grids + grids // 16 + 1024, MOST)


def test_lists_per_grid_keep_their_headroom(plan):
    for grids in (MOST, 2**28):
        assert plan.grids(2**31 - 1, grids, 0) == grids + grids // 16 + 1024
        assert plan.grids(grids + 3, grids, 0) == grids + 3
