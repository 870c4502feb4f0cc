"""How a batched launch's waves share its items (csrc/rlx_share.hpp, compiled
for the host): whatever the plan's capacity, no more waves have work than the
limit unless every item has one, the grid holds them, and the parts of an item
cover it once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_shares(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "share")
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2106_02504_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "host_arith", "share.cpp")], check=True)
    rows = [(items, grid, cost, lgs) for items in (4, 100, 1000, 2048, 2052, 3660, 4096, 4100, 8192, 87380)
            for grid in (100, 8192, 8292, 87480, 1 << 26) if grid >= items
            for cost in (1, 2, 63, 64, 65, 683, 8191, 8192, 1 << 26) for lgs in (0, 4, 5, 6)]
    out = subprocess.run([exe], input="".join("%d %d %d %d\n" % r for r in rows), text=True, check=True,
                         capture_output=True).stdout.split("\n")
    for (items, grid, cost, lgs), line in zip(rows, out):
        share, live, once = (int(v) for v in line.split())
        assert once == 1, (items, grid, cost, lgs)
        assert 1 <= share <= 64 and items * share <= max(grid, items)
        assert live <= max(8192, items), (items, grid, cost, lgs, live)
    # a server's plan with room for 87 381 segments: as with one that holds
    # just these items in the least grid
    at = {r: line for r, line in zip(rows, out)}
    for items in (100, 1000, 3660):
        assert at[items, 87480, 8192, 6] == at[items, 8192, 8192, 6]
