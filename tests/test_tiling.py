"""The tile arithmetic of the GEMM launches (csrc/tiling.h), compiled for the CPU."""

from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WRAPPERS = """
#include "tiling.h"
extern "C" int qkv(long long M, long long N, long long K) { const GemmTile t = qkv_tile(M, N, K); return t.bm * 1000 + t.bn; }
extern "C" int resid(long long M, long long N, long long K) { const GemmTile t = resid_tile(M, N, K); return t.bm * 1000 + t.bn; }
extern "C" int gate_up(long long M, long long N, long long K) { const GemmTile t = gate_up_tile(M, N, K); return t.bm * 1000 + t.bn; }
extern "C" int expert(long long groups, long long ffn, double rows) {
    const GemmTile t = expert_tile(groups, ffn, rows);
    return t.bm * 1000 + t.bn;
}
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


# (M, N, K, us on 256x256 tiles, us on the best of the small ones), measured on an MI355X
QKV = [
    (3072, 4096, 2048, 58.6, 58.8), (3072, 6144, 2048, 105.3, 88.8), (3072, 10240, 2048, 121.5, 150.9),
    (6144, 1024, 4096, 82.8, 68.5), (6144, 2048, 4096, 96.2, 112.7), (2560, 5120, 1536, 48.4, 58.3),
    (2560, 8192, 1536, 87.7, 75.6), (2560, 32768, 1536, 242.0, 313.3), (1920, 6144, 1152, 40.2, 36.9),
    (1920, 16384, 1152, 83.3, 94.7), (3072, 2048, 1024, 33.2, 22.9), (3072, 4200, 1024, 38.7, 43.3),
    (3072, 8192, 1024, 68.8, 64.2), (3072, 10240, 1024, 74.6, 83.2), (3072, 32768, 1024, 214.7, 251.8),
    (2304, 6144, 768, 34.6, 36.6), (2304, 16384, 768, 87.0, 77.3), (2304, 65536, 768, 263.4, 321.3),
    (1536, 16384, 512, 48.8, 41.6), (1536, 32768, 512, 76.1, 79.8), (768, 32768, 256, 39.6, 32.1),
    (768, 65536, 256, 56.0, 58.1), (1152, 65536, 384, 102.4, 99.8), (512, 65536, 128, 41.0, 36.8),
]
RESID = [
    (6144, 2048, 2048, 59.3, 59.6), (8192, 2048, 2048, 73.1, 78.5), (10240, 2048, 2048, 112.3, 94.2),
    (16384, 2048, 2048, 144.7, 173.7), (8100, 2048, 2048, 96.7, 79.8), (12200, 2048, 2048, 133.5, 121.9),
    (16300, 2048, 2048, 163.1, 168.2), (32768, 2176, 2176, 349.1, 375.2), (6144, 2176, 2176, 92.7, 77.5),
    (32768, 1152, 1152, 153.7, 127.1), (24576, 1152, 4608, 264.3, 292.9), (4096, 4096, 4096, 124.5, 147.9),
    (4000, 4096, 4096, 137.6, 147.7), (6100, 4096, 4096, 243.0, 228.4), (8192, 1536, 4096, 99.1, 112.7),
    (16384, 1024, 4096, 121.7, 141.4), (16300, 1024, 4096, 144.3, 145.3), (8192, 1536, 1536, 49.8, 51.0),
    (32768, 1536, 1536, 171.9, 207.5), (8100, 1536, 1536, 71.5, 52.2), (16384, 1024, 1024, 51.6, 47.0),
    (32768, 1024, 1024, 95.1, 111.7), (32700, 1024, 1024, 117.1, 107.0), (40960, 768, 768, 82.8, 86.9),
    (20480, 768, 768, 45.5, 40.0), (32768, 512, 512, 40.9, 34.0), (65536, 512, 512, 72.0, 76.0),
    (65536, 384, 384, 110.2, 53.5), (65536, 384, 1536, 152.6, 113.3), (65536, 256, 256, 36.5, 29.1),
]
GATE_UP = [
    (512, 22016, 4096, 80.9, 102.4), (128, 22016, 4096, 73.7, 51.8), (1024, 8704, 2176, 45.8, 51.6),
    (2048, 8704, 2176, 91.7, 83.3), (4096, 8704, 2176, 145.1, 155.2), (512, 11264, 2048, 39.3, 32.6),
    (1024, 11264, 2048, 46.0, 51.1), (2048, 11264, 2048, 86.6, 100.0), (2048, 10240, 1280, 58.0, 57.0),
    (1024, 8192, 1024, 24.6, 22.8), (2048, 8192, 1024, 33.4, 38.9), (4200, 8192, 1024, 74.1, 76.4),
    (2111, 8192, 1024, 49.2, 43.5), (32768, 8192, 1024, 435.2, 551.5), (2048, 4096, 512, 17.5, 15.2),
    (4096, 4096, 512, 21.9, 23.6), (5120, 4096, 512, 30.3, 27.5), (6144, 4096, 512, 30.8, 32.6),
    (6144, 2048, 256, 14.6, 14.0), (20480, 2048, 256, 30.4, 32.2), (32768, 2048, 256, 40.9, 47.0),
    (24576, 1024, 128, 20.1, 19.1), (65536, 2048, 128, 63.1, 70.0),
]
# gate/up on (64x128, 128x128)
GATE_UP_SMALL = [
    (256, 8192, 1024, 10.9, 13.6), (320, 8192, 1024, 15.9, 13.9), (512, 4096, 512, 8.8, 10.8),
    (640, 4096, 512, 10.5, 10.2), (128, 11264, 2048, 15.3, 20.8), (256, 11264, 2048, 22.7, 21.9),
    (64, 22016, 4096, 44.0, 46.6), (128, 22016, 4096, 65.1, 51.8),
]


@pytest.mark.parametrize("rule,points", [("qkv", QKV), ("resid", RESID), ("gate_up", GATE_UP)])
def test_rules_take_the_faster_tile(lib, rule, points):
    """At every measured point the rule's side is the faster one, or within 4 %
    of it (runs differ by 2 % a side)."""
    f = getattr(lib, rule)
    f.argtypes = [ctypes.c_longlong] * 3
    for M, N, K, big, small in points:
        mine = big if f(M, N, K) == 256256 else small
        assert mine <= 1.04 * min(big, small), (rule, M, N, K, mine, big, small)


def test_small_gate_up_tiles(lib):
    lib.gate_up.argtypes = [ctypes.c_longlong] * 3
    for M, N, K, narrow, wide in GATE_UP_SMALL:
        mine = {64128: narrow, 128128: wide}[lib.gate_up(M, N, K)]
        assert mine <= 1.04 * min(narrow, wide), (M, N, K, mine, narrow, wide)


# (groups, ffn, rows per expert, us of gate/up + down on 64x128, 128x128 and 256x256 tiles), d 2048, 8 experts per
# token (65 and 161 groups: one of them shared)
EXPERTS = [
    (65, 1024, 16, 170.4, 191.7, 202.0), (65, 1024, 48, 179.9, 195.7, 212.9), (65, 1024, 64, 201.0, 198.3, 217.5),
    (65, 1024, 96, 200.7, 199.3, 218.9), (65, 1024, 192, 341.3, 265.5, 253.3), (65, 1024, 512, 723.1, 558.6, 428.5),
    (40, 1536, 64, 176.8, 179.5, 190.0), (40, 1536, 102, 212.2, 193.3, 204.4), (40, 1536, 205, 315.6, 249.6, 229.9),
    (96, 768, 32, 182.2, 194.3, 205.6), (96, 768, 64, 186.6, 196.3, 209.7), (96, 768, 85, 235.6, 217.9, 225.3),
    (96, 768, 107, 233.3, 217.7, 223.9), (96, 768, 128, 285.7, 253.6, 237.2), (128, 768, 24, 228.3, 227.0, 228.7),
    (128, 768, 48, 224.5, 230.4, 230.9), (128, 768, 64, 277.2, 255.3, 251.4), (128, 768, 80, 278.6, 251.3, 248.6),
    (128, 768, 96, 316.9, 273.7, 261.1), (161, 1024, 38, 372.3, 382.3, 400.9), (161, 1024, 77, 496.1, 435.2, 437.6),
    (161, 1024, 102, 561.1, 492.3, 458.7),
]


def test_expert_tiles(lib):
    lib.expert.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_double]
    for groups, ffn, rows, *us in EXPERTS:
        mine = us[[64128, 128128, 256256].index(lib.expert(groups, ffn, rows))]
        assert mine <= 1.04 * min(us), (groups, ffn, rows, mine, us)
