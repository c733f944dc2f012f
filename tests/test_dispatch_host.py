"""The size rules of csrc/dispatch.h and csrc/adamw_rules.h, compiled for the host and checked over the range of sizes
the calls accept: no GPU is needed."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NONE, D32, D64, D64H = range(4)
PLAIN, LONG_EPILOGUE, F8 = range(3)
FORMS = [(PLAIN, 2), (PLAIN, 4), (LONG_EPILOGUE, 2), (LONG_EPILOGUE, 4)]  # of the int8 product: epilogue, bytes of an output
WRAPPER = r"""
#include "dispatch.h"
#include "adamw_rules.h"
extern "C" {
int few_tiles(long long M, long long N, int ncu) { return sb::few_tiles(M, N, ncu); }
long long plan_product(long long M, long long N, long long K, int kind, int out_bytes, int ncu, int *split) {
    const sb::ProductPlan p = sb::plan_product(M, N, K, (sb::ProductKind)kind, out_bytes, ncu);
    *split = p.split;
    return p.tile_rows;
}
// Rows [0, result) on 256x256 tiles, the others on `rest` ones.
long long plan_tiles(long long M, long long N, long long K, int kind, int out_bytes, int ncu, int *rest) {
    const sb::ProductPlan p = sb::plan_product(M, N, K, (sb::ProductKind)kind, out_bytes, ncu);
    *rest = p.rest;
    return p.first_rows;
}
int plan_weight_gradient(long long b, long long n, long long m, int ncu, int *out) {
    const sb::WeightGradPlan p = sb::plan_weight_gradient(b, n, m, ncu);
    out[0] = p.splits, out[1] = p.stages_per_split, out[2] = p.pieces, out[3] = p.stages_per_piece;
    out[4] = sb::least_pieces(b, n, m, ncu);
    return p.small;
}
int one_stage(long long M, long long N, long long K, int ncu) { return sb::one_stage(M, N, K, ncu); }
int persistent_grid(long long tiles, int slots) { return sb::persistent_grid(tiles, slots); }
int adamw_blocks(long long count) { return sb::adamw_blocks(count); }
long long adamw_elements_at_least(long long blocks, long long n) { return sb::adamw_elements_at_least(blocks, n); }
int adamw_streams(long long elements, int grad_bf16) { return sb::adamw_streams(elements, grad_bf16); }
// Every plan of M = lo..hi (step) must cover each row once: returns the first M whose plan does not, or 0.
long long bad_plan(long long lo, long long hi, long long step, long long N, long long K, int kind, int out_bytes,
                   int ncu) {
    for (long long M = lo; M <= hi; M += step) {
        const sb::ProductPlan p = sb::plan_product(M, N, K, (sb::ProductKind)kind, out_bytes, ncu);
        const bool direct = p.split != sb::DIRECT_NONE;
        if (p.split < 0 || p.split > sb::DIRECT_64H || p.tile_rows < 0 || p.tile_rows > M) return M;
        if (direct != (p.tile_rows < M)) return M;                       // rows past the tiles need a split, and only they
        if (p.tile_rows == 0 && !sb::few_tiles(M, N, ncu)) return M;     // many tiles: never all rows off the tiles
        if (direct && p.tile_rows % 256) return M;                      // the tiles that stay are whole
        if (p.first_rows < 0 || p.first_rows > p.tile_rows || p.first_rows % 256) return M;
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
        fh.write(WRAPPER)
    csrc = os.path.join(ROOT, "paper_2304_13013_amd", "csrc")
    subprocess.check_call(["g++", "-I", csrc, "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", lib, src])
    rules = ctypes.CDLL(lib)
    rules.few_tiles.argtypes = [ctypes.c_longlong] * 2 + [ctypes.c_int]
    rules.plan_product.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_int)]
    rules.plan_product.restype = ctypes.c_longlong
    rules.plan_tiles.argtypes = rules.plan_product.argtypes
    rules.plan_tiles.restype = ctypes.c_longlong
    rules.one_stage.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int]
    rules.persistent_grid.argtypes = [ctypes.c_longlong, ctypes.c_int]
    rules.adamw_blocks.argtypes = [ctypes.c_longlong]
    rules.adamw_elements_at_least.argtypes = [ctypes.c_longlong] * 2
    rules.adamw_elements_at_least.restype = ctypes.c_longlong
    rules.adamw_streams.argtypes = [ctypes.c_longlong, ctypes.c_int]
    rules.bad_plan.argtypes = [ctypes.c_longlong] * 5 + [ctypes.c_int] * 3
    rules.bad_plan.restype = ctypes.c_longlong
    return rules


# Few tokens into a very wide output: one partial row of more than ncu / 2 tiles, none of it full.
@pytest.mark.parametrize("ncu", [256, 304, 64, 8])
def test_every_plan_covers_each_row_once(rules, ncu):
    widths = [64, 768, 2880, 8192, 16384, 32768, 32832, 36864, 43008, 50304, 65536, 131072]
    for N in widths:
        for K in (64, 192, 1088, 1664, 2048, 2688, 5120, 8192, 131072):
            for lo, hi, step in ((1, 1100, 1), (1101, 70000, 251)):
                for kind, out_bytes in ((PLAIN, 2), (PLAIN, 4), (LONG_EPILOGUE, 2), (F8, 2)):
                    assert rules.bad_plan(lo, hi, step, N, K, kind, out_bytes, ncu) == 0, (N, K, kind, out_bytes, ncu)


def route(rules, M, N, K, out_bytes=2, kind=PLAIN):
    """(rows on the tiles, split of the rest) on an MI355X."""
    split = ctypes.c_int(-1)
    rows = rules.plan_product(M, N, K, kind, out_bytes, 256, ctypes.byref(split))
    return rows, split.value


# Products near the lines that were slower on the other route (up to 27 %): 64x64 blocks just past two per compute unit
# stay on the 128x128 tiles, and last rows that cost more than the round they save stay on the 256x256 ones.
@pytest.mark.parametrize("M,N,K,out_bytes", [(1137, 1856, 128, 2), (1358, 1600, 128, 2), (7233, 320, 1920, 2),
                                             (12045, 192, 896, 2), (9108, 256, 4864, 4), (338, 5760, 7552, 2),
                                             (4337, 8192, 1600, 2), (6837, 7232, 1024, 2),
                                             (19692, 2496, 768, 2), (19484, 2496, 384, 2),
                                             (35816, 2752, 1280, 4), (52260, 1088, 2624, 4), (32956, 1024, 768, 4)])
def test_products_that_stay_on_the_tiles(rules, M, N, K, out_bytes):
    assert route(rules, M, N, K, out_bytes) == (M, NONE)


@pytest.mark.parametrize("M,N,K", [(64, 1024, 4096), (197, 3072, 768), (2000, 768, 3072), (1121, 1792, 128)])
def test_products_that_leave_the_tiles(rules, M, N, K):
    rows, split = route(rules, M, N, K)
    assert rows == 0 and split != NONE


@pytest.mark.parametrize("M,N,K", [(16448, 1024, 4096), (16448, 4096, 1024), (32896, 5120, 1280), (8200, 2048, 512)])
def test_last_rows_that_leave_the_tiles(rules, M, N, K):
    rows, split = route(rules, M, N, K)
    assert rows == M // 256 * 256 and split != NONE


def stages_per_wave(K, split):
    return -(-K // 128) // (2 if split == D64H else 4)


# The sizes of the GPU tests reach every split of the small-product kernel and every instance of the tiled one: a retuned
# rule that empties their coverage fails here.
def test_sizes_of_the_gpu_tests_reach_every_path(rules):
    import test_dispatch_gpu as sizes
    plans = [(K, route(rules, M, N, K)) for M, N, K in sizes.SMALL]
    assert all(rows == 0 for _, (rows, _) in plans)
    assert {(split, K % 128) for K, (_, split) in plans} == {(s, h) for s in (D32, D64, D64H) for h in (0, 64)}
    assert {split for K, (_, split) in plans if stages_per_wave(K, split) > 2} == {D32, D64, D64H}
    plans = [(K, route(rules, M, N, K, 4, F8)) for M, N, K in sizes.SMALL_F8]
    assert all(rows == 0 for _, (rows, _) in plans)
    assert {split for K, (_, split) in plans if stages_per_wave(K, split) > 2} == {D32, D64, D64H}
    for kind, out_bytes in FORMS:  # last rows split off, with whole and half last stages
        plans = [(K, *route(rules, M, N, K, out_bytes, kind)) for M, N, K in sizes.SPLIT]
        assert all(rows > 0 for _, rows, _ in plans)
        assert {K % 128 for K, _, split in plans if split != NONE} == {0, 64}, (kind, out_bytes, plans)
    for out_bytes in (2, 4):
        plans = [(M, *route(rules, M, N, K, out_bytes, F8)) for M, N, K in sizes.TILES_F8]
        assert all(rows > 0 for _, rows, _ in plans) and {rows < M for M, rows, _ in plans} == {True, False}


def test_sizes_of_the_float8_error_test_take_both_routes(rules):
    import test_dispatch_gpu as sizes
    for K in sizes.CHAIN_K:
        assert route(rules, sizes.CHAIN_ROWS, sizes.CHAIN_COLS, K, 4, F8) == (sizes.CHAIN_ROWS, NONE)
        assert route(rules, sizes.CHAIN_LAST, sizes.CHAIN_COLS, K, 4, F8)[0] == 0


TILES_128, TILES_256X128, TILES_256 = range(3)


def tiles(rules, M, N, K, kind, out_bytes):
    """(rows on the first tiles, TILES_256 or None, kind of the others or None) on an MI355X."""
    rest = ctypes.c_int(-1)
    rows = rules.plan_tiles(M, N, K, kind, out_bytes, 256, ctypes.byref(rest))
    return rows, TILES_256 if rows else None, rest.value if rows < route(rules, M, N, K, out_bytes, kind)[0] else None


def only(rules, tile, M, N, K, kind, out_bytes):
    """Whether the whole product runs on this one kind of tiles."""
    return tiles(rules, M, N, K, kind, out_bytes) == (0, None, tile) and route(rules, M, N, K, out_bytes, kind) == (M, NONE)


def test_sizes_of_the_gpu_tests_reach_every_tile(rules):
    import test_dispatch_gpu as sizes
    for form in FORMS:  # each listed size runs what its list is named for, whichever the output and scale
        assert all(only(rules, TILES_256, *s, *form) and not rules.one_stage(*s, 256) for s in sizes.LARGE), form
        assert all(only(rules, TILES_256, *s, *form) and rules.one_stage(*s, 256) for s in sizes.ONE_STAGE), form
        assert all(only(rules, TILES_128, *s, *form) for s in sizes.SMALL_TILES), form
    for out_bytes in (2, 4):
        for name, tile in (("256", TILES_256), ("one stage", TILES_256), ("256x128", TILES_256X128), ("128", TILES_128)):
            assert all(only(rules, tile, *s, F8, out_bytes) for s in sizes.FORMATS_F8[name]), (name, out_bytes)
    assert all(rules.one_stage(*s, 256) == (name == "one stage") for name in ("256", "one stage") for s in sizes.FORMATS_F8[name])
    stages = lambda listed: {(-(-K // 128), K % 128) for _, _, K in listed}
    assert stages(sizes.LARGE) >= {(s, h) for s in (1, 2, 3) for h in (0, 64)}
    assert stages(sizes.SMALL_TILES) >= {(s, h) for s in (1, 2, 5) for h in (0, 64)}
    assert {-(-M // 256) * -(-N // 256) // 256 for M, N, _ in sizes.LARGE} == {1, 2}  # whole rounds before the last one
    assert any(-(-M // 128) * -(-N // 128) > 512 for M, N, _ in sizes.SMALL_TILES)
    assert all(M % 256 and N % 256 for M, N, _ in sizes.LARGE)
    assert all(-(-M // 256) * -(-N // 256) > 256 for M, N, _ in sizes.FORMATS_F8["256"])
    for kind, out_bytes in FORMS:
        plans = [(M, N, K, *tiles(rules, M, N, K, kind, out_bytes)) for M, N, K in sizes.NARROW]
        narrow = {("half" if K % 128 else "whole", -(-M // 256) * -(-N // 128) > 256)
                  for M, N, K, rows, _, second in plans if rows == 0 and second == TILES_256X128}
        assert {("half", True), ("whole", True)} <= narrow, (kind, out_bytes, plans)
        if (kind, out_bytes) == (LONG_EPILOGUE, 2):
            assert {K for _, _, K, _, _, second in plans if second == TILES_256X128} >= {64, 128}
        if out_bytes == 2:
            assert any(rows and second is not None for *_, rows, _, second in plans), plans
    assert {second for M, N, K in sizes.NARROW_F8 for second in tiles(rules, M, N, K, F8, 2)[1:]} >= {
        TILES_256X128, TILES_256}
    assert any(rows and second is not None for rows, _, second in (tiles(rules, M, N, K, F8, 2) for M, N, K in sizes.NARROW_F8))


# Four-byte outputs just past one round of 128x128 tiles, where a compute unit gets four of them, and just up to it.
@pytest.mark.parametrize("M,N,K,kind,tile", [(34752, 192, 384, PLAIN, TILES_256), (4455, 2048, 64, PLAIN, TILES_256),
                                             (35776, 192, 640, PLAIN, TILES_256), (5014, 2048, 256, F8, TILES_256),
                                             (6890, 1280, 384, F8, TILES_256), (25074, 192, 128, PLAIN, TILES_128),
                                             (16000, 320, 128, F8, TILES_128)])
def test_tiles_of_four_byte_outputs(rules, M, N, K, kind, tile):
    assert only(rules, tile, M, N, K, kind, 4)


def weight_gradient(rules, b, n, m, ncu=256):
    out = (ctypes.c_int * 5)()
    small = rules.plan_weight_gradient(ctypes.c_longlong(b), ctypes.c_longlong(n), ctypes.c_longlong(m), ncu, out)
    return (bool(small), *out)


# Every token is in one split and one piece, no split is empty, and no chain is longer than the fewest pieces allowed make it.
@pytest.mark.parametrize("ncu", [256, 64, 8])
def test_weight_gradient_plans_cover_every_token_once(rules, ncu):
    widths = [64, 192, 320, 768, 1088, 2880, 5120, 16384, 131072]
    for b in list(range(0, 700, 13)) + [1024, 4097, 6304, 16448, 28030, 32896, 1048319]:
        stages = -(-b // 64)
        for n in widths:
            for m in widths:
                small, splits, per_split, pieces, per_piece, least = weight_gradient(rules, b, n, m, ncu)
                assert 1 <= splits <= 64 and 1 <= least <= 16 and (splits == 1 or pieces == 1)
                assert splits * per_split >= stages and (splits == 1 or (splits - 1) * per_split < stages), (b, n, m)
                assert pieces == 1 or (small and splits == 1 and pieces * per_piece >= stages), (b, n, m)
                assert min(per_split, per_piece) <= -(-stages // least), (b, n, m)
                assert small or stages > 0, "an empty range has no item on the large tiles"


def test_sizes_of_the_gpu_tests_reach_both_weight_gradients(rules):
    import test_dispatch_gpu as sizes
    assert all(weight_gradient(rules, *s)[:2] == (False, 1) for s in sizes.LARGE_DW)
    assert any(-(-n // 256) * -(-m // 256) > 256 for _, n, m in sizes.LARGE_DW)
    assert all(weight_gradient(rules, *s)[0] for s in sizes.SMALL_DW)
    assert max(weight_gradient(rules, *s)[1] for s in sizes.SMALL_DW) > 16
    assert weight_gradient(rules, 8637, 1920, 1984)[:2] == (False, 4)
    plans = [(-(-n // 128) * -(-m // 128), *weight_gradient(rules, b, n, m)) for b, n, m in sizes.MANY_SMALL_DW]
    assert all(items > 512 and small and splits == 1 for items, small, splits, *_ in plans)
    assert {pieces for _, _, _, _, pieces, *_ in plans} == {1, 7}


# The instances of one stage are for launches in which no workgroup has a second tile, on any XCD.
@pytest.mark.parametrize("ncu", [256, 304, 60, 8])
def test_one_stage_is_one_tile_per_workgroup(rules, ncu):
    for M in list(range(1, 9000, 83)) + [32768, 65536, 70000]:
        for N in (64, 256, 320, 2048, 8192, 65536):
            tiles = -(-M // 256) * -(-N // 256)
            one = rules.one_stage(M, N, 128, ncu)
            assert not rules.one_stage(M, N, 192, ncu)
            assert not one or -(-tiles // 8) <= rules.persistent_grid(tiles, ncu) // 8
            assert bool(one) == (tiles <= ncu // 8 * 8)


@pytest.mark.parametrize("slots", [8, 64, 256, 512, 608])
def test_persistent_grid(rules, slots):
    for tiles in list(range(0, 4 * slots + 20)) + [10 ** 6, 2 ** 31]:
        grid = rules.persistent_grid(tiles, slots)
        assert grid % 8 == 0 and 8 <= grid <= slots
        rounds = -(-tiles // slots)
        assert -(-tiles // grid) <= max(rounds, 1)          # a shrunk grid makes no more rounds


def block_of(n):
    return [3 * n * n, n * n, 4 * n * n, 4 * n * n, 3 * n, n, 4 * n, n, n, n]


# Batched optimizer steps: sets of many small tensors that fit the last-level cache, transformer blocks on both sides of
# the line, and the bound for tensors of more than 2048 workgroups, which counts them as 8.4 million elements.
@pytest.mark.parametrize("counts,streams", [([256] * 5000, False), ([1024] * 5000, False), ([4097] * 4500, False),
                                            (block_of(768), False), (block_of(1280), True), (block_of(512) * 12, True),
                                            ([67_108_864], False), ([67_108_864] * 3, True)])
def test_batched_optimizer_step_streams(rules, counts, streams):
    at_least = rules.adamw_elements_at_least(sum(rules.adamw_blocks(c) for c in counts), len(counts))
    assert at_least <= sum(counts)
    assert rules.adamw_streams(at_least, 1) == streams
