"""The tile arithmetic of the GEMM launches (csrc/tiling.h), compiled for the CPU."""

from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WRAPPERS = """
#include "tiling.h"
extern "C" int share(int total, int workgroups) { return xcd_share(total, workgroups); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiling")
    src, out = d / "tiling.cpp", d / "libtiling.so"
    src.write_text(WRAPPERS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2608_02625_amd", "csrc"), str(src), "-o", str(out)], check=True)
    return ctypes.CDLL(str(out))


def test_shares_cover_every_tile_in_the_fewest_rounds(lib):
    """The walk of the kernels: workgroup i of XCD x takes tiles x * share + i,
    + workgroups, ... below the share's end."""
    for workgroups in (1, 2, 5, 6, 32, 38, 64, 96):
        for total in list(range(1, 120)) + [255, 256, 257, 511, 1000, 2049, 5000]:
            share = lib.share(total, workgroups)
            rounds, seen = 0, []
            for x in range(8):
                mine = range(min(x * share, total), min(x * share + share, total))
                seen += mine
                rounds = max(rounds, -(-len(mine) // workgroups))
            assert seen == list(range(total)), (total, workgroups)
            assert rounds == -(-total // (8 * workgroups)), (total, workgroups, share)
