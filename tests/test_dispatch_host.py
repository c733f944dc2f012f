"""The dispatch rules of csrc/dispatch.h, compiled for the host and checked over the range of sizes the calls accept: no
GPU is needed."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NONE, D32, D64, D64H = range(4)
WRAPPER = r"""
#include "%s"
extern "C" {
int few_tiles(long long M, long long N, int ncu) { return sb::few_tiles(M, N, ncu); }
long long plan_product(long long M, long long N, long long K, int ncu, int *split) {
    const sb::ProductPlan p = sb::plan_product(M, N, K, ncu);
    *split = p.split;
    return p.tile_rows;
}
int persistent_grid(long long tiles, int slots) { return sb::persistent_grid(tiles, slots); }
// Every plan of M = lo..hi (step) must cover each row once: returns the first M whose plan does not, or 0.
long long bad_plan(long long lo, long long hi, long long step, long long N, long long K, int ncu) {
    for (long long M = lo; M <= hi; M += step) {
        const sb::ProductPlan p = sb::plan_product(M, N, K, ncu);
        const bool direct = p.split != sb::DIRECT_NONE;
        if (p.split < 0 || p.split > sb::DIRECT_64H || p.tile_rows < 0 || p.tile_rows > M) return M;
        if (direct != (p.tile_rows < M)) return M;                       // rows past the tiles need a split, and only they
        if (p.tile_rows == 0 && !sb::few_tiles(M, N, ncu)) return M;     // many tiles: never all rows off the tiles
        if (direct && p.tile_rows %% 256) return M;                      // the tiles that stay are whole
        if (p.tile_rows > 0 && sb::persistent_grid((p.tile_rows + 255) / 256 * ((N + 255) / 256), ncu) < 8) return M;
    }
    return 0;
}
}
"""


@pytest.fixture(scope="session")
def rules(tmp_path_factory):
    folder = tmp_path_factory.mktemp("dispatch")
    src, lib = str(folder / "rules.cpp"), str(folder / "rules.so")
    with open(src, "w") as fh:
        fh.write(WRAPPER % os.path.join(ROOT, "paper_2304_13013_amd", "csrc", "dispatch.h"))
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", lib, src])
    rules = ctypes.CDLL(lib)
    rules.few_tiles.argtypes = [ctypes.c_longlong] * 2 + [ctypes.c_int]
    rules.plan_product.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    rules.plan_product.restype = ctypes.c_longlong
    rules.persistent_grid.argtypes = [ctypes.c_longlong, ctypes.c_int]
    rules.bad_plan.argtypes = [ctypes.c_longlong] * 5 + [ctypes.c_int]
    rules.bad_plan.restype = ctypes.c_longlong
    return rules


# Few tokens into a very wide output: one partial row of more than ncu / 2 tiles, none of it full.
@pytest.mark.parametrize("ncu", [256, 304, 64, 8])
def test_every_plan_covers_each_row_once(rules, ncu):
    widths = [64, 768, 2880, 8192, 16384, 32768, 32832, 36864, 43008, 50304, 65536, 131072]
    for N in widths:
        for K in (64, 192, 1088, 1664, 2048, 2688, 5120, 8192, 131072):
            for lo, hi, step in ((1, 1100, 1), (1101, 70000, 251)):
                assert rules.bad_plan(lo, hi, step, N, K, ncu) == 0, (N, K, ncu)


@pytest.mark.parametrize("slots", [8, 64, 256, 512, 608])
def test_persistent_grid(rules, slots):
    for tiles in list(range(0, 4 * slots + 20)) + [10 ** 6, 2 ** 31]:
        grid = rules.persistent_grid(tiles, slots)
        assert grid % 8 == 0 and 8 <= grid <= slots
        rounds = -(-tiles // slots)
        assert -(-tiles // grid) <= max(rounds, 1)          # a shrunk grid makes no more rounds
