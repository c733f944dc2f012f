"""GPU parity at the sizes where a dispatch rule or a kernel variant can go wrong: tile edges, remainders, the smallest
and largest sizes of a variant's range.  Bars as in test_parity_gpu.py: codes, states and int32 accumulators bit-exact,
dequantized values within one binary32 ulp of the oracle."""
import numpy as np
import pytest
import torch

from paper_2304_13013_amd import inputs as I
from paper_2304_13013_amd import switchback as sb
from test_parity_gpu import assert_f8_outputs, layer_like_codes

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def to_dev(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(DEV).view(torch.bfloat16)


def host(t):
    return t.detach().cpu().numpy()


def ulp(ref):
    return np.spacing(np.abs(ref).astype(np.float32))


def rand_bf16(rng, shape, scale=1.0):
    return I.f32_to_bf16_bits((rng.standard_normal(shape) * scale).astype(np.float32))


def test_stream_handle_is_the_current_streams():
    side = torch.cuda.Stream()
    assert sb._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert sb._stream() == side.cuda_stream == torch.cuda.current_stream().cuda_stream


# The rows of W follow those of X in one launch: one wavefront per row (n <= 2048, the boundary inside a workgroup),
# one workgroup per row, and the two-pass rows (n > 16384); no rows of X at all.
@pytest.mark.parametrize("b,n,m", [(5, 64, 128), (3, 2048, 64), (2, 2112, 64), (1, 16448, 64), (0, 256, 128)])
def test_rows_of_w_follow_rows_of_x_in_one_launch(oracle, b, n, m):
    rng = np.random.default_rng(b + n + m)
    x, w = rand_bf16(rng, (b, n)), rand_bf16(rng, (m, n), n ** -0.5)
    _, bufs = sb.forward_q(to_dev(x), to_dev(w))
    torch.cuda.synchronize()
    wq, sw = oracle.quantize_rowwise(w)
    np.testing.assert_array_equal(host(bufs.wq), wq)
    np.testing.assert_array_equal(host(bufs.state_w_row).view(np.uint32), sw.view(np.uint32))
    if b:
        xq, sx = oracle.quantize_rowwise(x)
        np.testing.assert_array_equal(host(bufs.xq), xq)
        np.testing.assert_array_equal(host(bufs.state_x).view(np.uint32), sx.view(np.uint32))


# Row runs of the column-wise quantizer's first pass: a run of fewer rows than its eight row lanes, ragged runs, the
# bound of 64 runs, and the last chunk block partly outside the matrix.
@pytest.mark.parametrize("rows,cols", [(16, 272), (80, 256), (1040, 528), (4096, 16), (4112, 48)])
def test_colwise_quantizer_row_runs(oracle, rows, cols):
    rng = np.random.default_rng(rows + cols)
    w = rand_bf16(rng, (rows, cols))
    q_t, s = sb.quantize_colwise_transpose(to_dev(w))
    torch.cuda.synchronize()
    qo, so = oracle.quantize_colwise_transpose(w)
    np.testing.assert_array_equal(host(s).view(np.uint32), so.view(np.uint32))
    np.testing.assert_array_equal(host(q_t), qo)


# The small-product kernel, all three of its splits, each with whole and half last stages (K = 64 mod 128) and with more
# stages per wave than the ring holds: one row, rows and columns past a block's edge, a contraction shorter than one stage,
# one that leaves waves idle, and every output and scale.  (A host test checks which split each size takes.)
SMALL = [(1, 64, 64), (33, 64, 192), (197, 192, 4096), (64, 1024, 576), (300, 1024, 8192), (197, 3072, 768),
         (512, 2048, 320), (2000, 768, 768), (1990, 768, 3008), (197, 3072, 832), (1000, 1024, 4032), (513, 1984, 2048)]


@pytest.mark.parametrize("M,N,K", SMALL)
def test_small_int8_products(oracle, M, N, K):
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-127, 128, size=(M, K)).astype(np.int8)
    b = rng.integers(-127, 128, size=(N, K)).astype(np.int8)
    sr = (np.abs(rng.standard_normal(M)) + 0.01).astype(np.float32)
    sc = (np.abs(rng.standard_normal(N)) + 0.01).astype(np.float32)
    bias, gamma = rng.standard_normal((2, N)).astype(np.float32)
    dev = [torch.from_numpy(v).to(DEV) for v in (a, sr, b, sc)]
    st = torch.full((1,), 0.37, device=DEV)
    acc = oracle.matmul_int8(a, b)
    np.testing.assert_array_equal(host(sb.matmul_int8_dequant(dev[0], None, dev[2], None, out_dtype=torch.int32)), acc)
    ref = oracle.dequantize(acc, sr, np.float32(0.37))
    y32 = host(sb.matmul_int8_dequant(dev[0], dev[1], dev[2], st, out_dtype=torch.float32))
    np.testing.assert_array_equal(y32, ref)
    ybf = sb.matmul_int8_dequant(dev[0], dev[1], dev[2], st).view(torch.int16)
    np.testing.assert_array_equal(host(ybf).view(np.uint16), oracle.round_to_bf16(ref))
    post = sb.matmul_int8_dequant_bias_layerscale(dev[0], dev[1], dev[2], st, torch.from_numpy(bias).to(DEV),
                                                  torch.from_numpy(gamma).to(DEV), out_dtype=torch.float32)
    np.testing.assert_array_equal(host(post), oracle.bias_layerscale(ref, bias, gamma))
    rc = host(sb.matmul_int8_dequant_rc(*dev, out_dtype=torch.float32))
    np.testing.assert_array_equal(rc, oracle.dequantize_rowcol(acc, sr, sc))


# Codes 0, +-1/4, +-1/2, +-1: no product is truncated and binary32 holds every partial sum, so the float8 sum is exact.
SMALL_F8 = [(1, 64, 128), (197, 192, 4096), (300, 1024, 640), (1990, 768, 768), (197, 3072, 768), (1000, 1024, 4096),
            (2001, 704, 3072)]


@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", SMALL_F8)
def test_small_float8_products(M, N, K, fa, fb):
    check_exact_float8_product(M, N, K, fa, fb)


def check_exact_float8_product(M, N, K, fa, fb):
    rng = np.random.default_rng(M + N + K)
    vals = np.array([0.0, 0.25, -0.25, 0.5, -0.5, 1.0, -1.0], np.float32)
    a, b = (torch.from_numpy(vals[rng.integers(0, 7, size=(r, K))]).to(DEV) for r in (M, N))
    types = (torch.float8_e4m3fn, torch.float8_e5m2)
    sr = torch.rand(M, device=DEV) + 0.5
    st = torch.full((1,), 0.37, device=DEV)
    args = a.to(types[fa]).view(torch.uint8), fa, sr, b.to(types[fb]).view(torch.uint8), fb, st
    want = (a.double() @ b.double().t()).float() * (sr * st)[:, None]
    assert torch.equal(sb.matmul_f8_dequant(*args, out_dtype=torch.float32), want)
    assert torch.equal(sb.matmul_f8_dequant(*args), want.bfloat16())


# The tiled kernels with a last stage of half zeros (K = 64 mod 128; K = 64, where it is the only one), and products whose
# last rows leave the tiles because they would start another round of the grid: 1 row, a tile row less one, a width that is
# no multiple of the tile; every output type and scale.
SPLIT = [(11237, 2880, 192), (5000, 1088, 320), (16385, 1024, 1024), (16639, 1024, 1536), (16448, 960, 1216),
         (32896, 2048, 1088), (9000, 1088, 64), (16000, 4224, 192)]


@pytest.mark.parametrize("M,N,K", SPLIT)
def test_half_stages_and_last_rows(oracle, M, N, K):
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-127, 128, size=(M, K)).astype(np.int8)
    b = rng.integers(-127, 128, size=(N, K)).astype(np.int8)
    sr = (np.abs(rng.standard_normal(M)) + 0.01).astype(np.float32)
    sc = (np.abs(rng.standard_normal(N)) + 0.01).astype(np.float32)
    bias, gamma = rng.standard_normal((2, N)).astype(np.float32)
    dev = [torch.from_numpy(v).to(DEV) for v in (a, sr, b, sc)]
    st = torch.full((1,), 0.37, device=DEV)
    acc = host(sb.matmul_int8_dequant(dev[0], None, dev[2], None, out_dtype=torch.int32))
    # |acc| <= 127^2 K < 2^53: the binary64 product is the whole number itself.
    np.testing.assert_array_equal(acc, host(dev[0].double() @ dev[2].double().t()).astype(np.int32))
    ref = oracle.dequantize(acc, sr, np.float32(0.37))
    ybf = sb.matmul_int8_dequant(dev[0], dev[1], dev[2], st).view(torch.int16)
    np.testing.assert_array_equal(host(ybf).view(np.uint16), oracle.round_to_bf16(ref))
    np.testing.assert_array_equal(host(sb.matmul_int8_dequant(dev[0], dev[1], dev[2], st, out_dtype=torch.float32)), ref)
    vecs = [torch.from_numpy(v).to(DEV) for v in (bias, gamma)]
    ref_post, ref_rc = oracle.bias_layerscale(ref, bias, gamma), oracle.dequantize_rowcol(acc, sr, sc)
    post = sb.matmul_int8_dequant_bias_layerscale(dev[0], dev[1], dev[2], st, *vecs, out_dtype=torch.float32)
    np.testing.assert_array_equal(host(post), ref_post)
    np.testing.assert_array_equal(host(sb.matmul_int8_dequant_rc(*dev, out_dtype=torch.float32)), ref_rc)
    post = sb.matmul_int8_dequant_bias_layerscale(dev[0], dev[1], dev[2], st, *vecs).view(torch.int16)
    np.testing.assert_array_equal(host(post).view(np.uint16), oracle.round_to_bf16(ref_post))
    rc = sb.matmul_int8_dequant_rc(*dev).view(torch.int16)
    np.testing.assert_array_equal(host(rc).view(np.uint16), oracle.round_to_bf16(ref_rc))


# 256x256 tiles, with every output and scale: one, two and three stages a tile, the last one whole or half, two and three tiles
# per workgroup, partial in both directions.  At these lengths the epilogue of a tile stands in the first half stage of the
# next one, right before its hand-over.
LARGE = [(16385, 1472, 64), (8449, 2880, 128), (20011, 2240, 192), (14000, 3264, 256), (12345, 2240, 320), (12345, 2240, 384)]
# One stage and at most one tile per workgroup (instances of their own): half a stage and a whole one, partial both ways.
ONE_STAGE = [(25615, 320, 64), (25615, 320, 128), (2501, 4032, 128)]
# 128x128 tiles: the same for a single stage, two and five; one tile per workgroup and more than fit the GPU at once.
SMALL_TILES = [(3000, 704, 64), (33000, 320, 128), (3000, 704, 192), (3000, 704, 256), (3000, 704, 576), (3000, 704, 640)]


# The other sizes: a single column of partial tiles (128x128), and short contractions on whichever tile the output takes.
@pytest.mark.parametrize("M,N,K", LARGE + ONE_STAGE + SMALL_TILES + [(33000, 64, 64), (33000, 2304, 64), (8449, 1088, 128), (17000, 2240, 192),
                                                         (16700, 2112, 320)])
def test_large_tiles(oracle, M, N, K):
    test_half_stages_and_last_rows(oracle, M, N, K)


# 256x128 tiles: a contraction shorter than the two stages they make of it (with the longer epilogues), half a last stage,
# one tile and several per workgroup, partial in both directions; and the same rows on two kinds of tiles, split after whole
# rounds of the grid.  (A host test checks which tiles each size takes.)
NARROW = [(34462, 384, 64), (34462, 384, 128), (4048, 1984, 192), (6304, 832, 1088), (11237, 2880, 192),
          (12345, 3328, 384), (22069, 2240, 2048)]


@pytest.mark.parametrize("M,N,K", NARROW)
def test_narrow_tiles_and_whole_rounds(oracle, M, N, K):
    test_half_stages_and_last_rows(oracle, M, N, K)


# Exact sums, as for the small float8 products: last rows, the small tile with ragged edges, 256x128 tiles, whole rounds.
TILES_F8 = [(16448, 1024, 1024), (16385, 960, 1152), (6304, 832, 1152), (1999, 2112, 384)]
NARROW_F8 = [(6304, 768, 3072), (5431, 960, 4096), (22069, 1472, 384)]


# Every pair of formats on each tile: 256x256 with one stage a tile and with two, one stage in one round, 256x128, 128x128 with one stage, also with more
# tiles than fit the GPU at once; partial in both directions.
FORMATS_F8 = {"256": [(8449, 2880, 128), (14000, 3264, 256)], "one stage": [(25615, 320, 128)], "256x128": [(5431, 960, 4096)],
              "128": [(3000, 704, 128), (33000, 320, 128)]}


@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", sum(FORMATS_F8.values(), []))
def test_formats_on_every_tile_of_a_float8_product(M, N, K, fa, fb):
    check_exact_float8_product(M, N, K, fa, fb)


@pytest.mark.parametrize("fa,fb", [(1, 0), (0, 0)])
@pytest.mark.parametrize("M,N,K", TILES_F8 + NARROW_F8)
def test_tiles_of_a_float8_product(M, N, K, fa, fb):
    check_exact_float8_product(M, N, K, fa, fb)


# The small-product kernel adds a float8 contraction in up to four pieces, the tiles in one: the last rows of a product,
# split off, may differ in the last bits from the same token rows among the first ones.  Both lie within the bound of the
# matrix instruction, and the pieces are no further from the exact sum (root mean square) than the one chain.
@pytest.mark.parametrize("fa", [0, 1])
def test_float8_rows_on_both_sides_of_a_split(oracle, fa, M=16448, N=1024, K=1024, last=64):
    rng = np.random.default_rng(fa)
    a, b = layer_like_codes(rng, (M, K), fa), layer_like_codes(rng, (N, K), 0)
    a[-last:] = a[:last]
    sr = rng.uniform(0.5, 4.0, M).astype(np.float32)
    sr[-last:] = sr[:last]
    sw = np.float32(0.37)
    acc, abs_acc = oracle.matmul_f8(a[:last], fa, b, 0, want_abs=True)
    y = host(sb.matmul_f8_dequant(torch.from_numpy(a).to(DEV), fa, torch.from_numpy(sr).to(DEV),
                                  torch.from_numpy(b).to(DEV), 0, torch.tensor([sw], device=DEV), out_dtype=torch.float32))
    err = []
    for rows in (y[:last], y[-last:]):
        assert_f8_outputs(rows, None, acc, abs_acc, sr[:last], sw, K, oracle)
        _, exact = oracle.dequantize_f8(acc, sr[:last], sw, want_f64=True)
        err.append(np.sqrt(np.mean((rows - exact) ** 2)))
    # 65536 outputs: the ratio of the two errors scatters by about 1 / sqrt(65536) = 0.4 %.
    assert err[1] <= 1.02 * err[0], err


# The same for contractions of three to 256 stages, on codes of layer data: neither the pieces nor the one chain is further from
# binary64 than the other (the products inside an instruction lose far more than the additions between them).
CHAIN_ROWS, CHAIN_LAST, CHAIN_COLS, CHAIN_K = 16384, 256, 1024, [384, 1024, 4096, 8192, 32768]


@pytest.mark.parametrize("fa", [0, 1])
@pytest.mark.parametrize("K", CHAIN_K)
def test_float8_sums_in_one_chain_and_in_pieces(K, fa):
    gen = torch.Generator(device=DEV).manual_seed(K + fa)
    x = torch.randn(CHAIN_ROWS, K, generator=gen, device=DEV).bfloat16()
    w = (torch.randn(CHAIN_COLS, K, generator=gen, device=DEV) / K ** 0.5).bfloat16()
    a, sr = sb.quantize_rowwise_f8(x, fa)
    b, _, st = sb.quantize_tensorwise_f8(w, 0)
    some = slice(0, CHAIN_LAST)
    chain = sb.matmul_f8_dequant(a, fa, sr, b, 0, st, out_dtype=torch.float32)[some]
    pieces = sb.matmul_f8_dequant(a[some].contiguous(), fa, sr[some].contiguous(), b, 0, st, out_dtype=torch.float32)
    values = a[some].view((torch.float8_e4m3fn, torch.float8_e5m2)[fa]).double()
    exact = values @ b.view(torch.float8_e4m3fn).double().t().contiguous() * sr[some].double()[:, None] * st.double()
    err = [(y.double() - exact).norm() for y in (chain, pieces)]
    assert abs(err[0] - err[1]) <= 0.02 * err[1], err  # 262144 outputs: the ratio scatters by about 0.2 %


# A few tokens into a very wide output: 129 tiles in the only, partial row of tiles, so that nothing is left for the tiles
# if the "last rows" leave them.  Every form of the product.
@pytest.mark.parametrize("M", [1, 32, 64])
def test_few_rows_of_a_very_wide_output(oracle, M, N=32832, K=2048):
    rng = np.random.default_rng(M)
    a = rng.integers(-127, 128, size=(M, K)).astype(np.int8)
    b = rng.integers(-127, 128, size=(N, K)).astype(np.int8)
    sr = (np.abs(rng.standard_normal(M)) + 0.01).astype(np.float32)
    sc = (np.abs(rng.standard_normal(N)) + 0.01).astype(np.float32)
    bias, gamma = rng.standard_normal((2, N)).astype(np.float32)
    dev = [torch.from_numpy(v).to(DEV) for v in (a, sr, b, sc)]
    st = torch.full((1,), 0.37, device=DEV)
    acc = host(sb.matmul_int8_dequant(dev[0], None, dev[2], None, out_dtype=torch.int32))
    np.testing.assert_array_equal(acc, host(dev[0].double() @ dev[2].double().t()).astype(np.int32))
    ref = oracle.dequantize(acc, sr, np.float32(0.37))
    ybf = sb.matmul_int8_dequant(dev[0], dev[1], dev[2], st).view(torch.int16)
    np.testing.assert_array_equal(host(ybf).view(np.uint16), oracle.round_to_bf16(ref))
    post = sb.matmul_int8_dequant_bias_layerscale(dev[0], dev[1], dev[2], st, torch.from_numpy(bias).to(DEV),
                                                  torch.from_numpy(gamma).to(DEV), out_dtype=torch.float32)
    np.testing.assert_array_equal(host(post), oracle.bias_layerscale(ref, bias, gamma))
    rc = host(sb.matmul_int8_dequant_rc(*dev, out_dtype=torch.float32))
    np.testing.assert_array_equal(rc, oracle.dequantize_rowcol(acc, sr, sc))
    vals = np.array([0.0, 0.25, -0.25, 0.5, -0.5, 1.0, -1.0], np.float32)  # exact float8 sums, as above
    a8, b8 = (torch.from_numpy(vals[rng.integers(0, 7, size=(r, K))]).to(DEV) for r in (M, N))
    got = sb.matmul_f8_dequant(a8.to(torch.float8_e4m3fn).view(torch.uint8), 0, dev[1],
                               b8.to(torch.float8_e4m3fn).view(torch.uint8), 0, st, out_dtype=torch.float32)
    assert torch.equal(got, (a8.double() @ b8.double().t()).float() * (dev[1] * st)[:, None])


# Small weight gradients whose reduction launch is not worth its cost still sum the tokens in the pieces of the split they
# replace, in two or three (the last one ragged): the bits of the gradients over those token ranges, added in order.
@pytest.mark.parametrize("b,n,m,piece", [(512, 256, 1024, 256), (758, 3264, 256, 384), (641, 384, 2048, 384),
                                         (1016, 896, 1024, 384)])
def test_small_weight_gradient_sums_its_pieces(b, n, m, piece):
    rng = np.random.default_rng(b + n + m)
    x, dy = to_dev(rand_bf16(rng, (b, n))), to_dev(rand_bf16(rng, (b, m), 0.1))
    want = torch.zeros(m, n, device=DEV)
    for lo in range(0, b, piece):
        want += sb.backward_weight(dy[lo:lo + piece], x[lo:lo + piece], dw_dtype=torch.float32)
    assert torch.equal(sb.backward_weight(dy, x, dw_dtype=torch.float32), want)
    assert torch.equal(sb.backward_weight(dy, x), want.bfloat16())


# Weight gradients on 256x256 tiles without a split: one token past a pair of 32-token stages, one short of a stage and one
# past it, whole ones, a second item per workgroup (342 tiles), tiles that are partial in both directions; on 128x128 tiles:
# one token, more splits than a reduction step adds at once (40 pieces of 11 stages, the last one ragged).  Every element; a
# binary32 result is at most the additions of a chain from the exact sum, in units of the sum of magnitudes (the matrix
# instruction adds 16 products or more at a time).
LARGE_DW = [(65, 1344, 5952), (95, 1344, 5952), (97, 1344, 5952), (64, 1600, 5056), (64, 4544, 4736)]
SMALL_DW = [(1, 64, 64), (200, 64, 576), (28030, 320, 192)]


@pytest.mark.parametrize("b,n,m", LARGE_DW + SMALL_DW)
def test_weight_gradient_tiles(oracle, b, n, m):
    rng = np.random.default_rng(b + n + m)
    dyb, xb = rand_bf16(rng, (b, m), 0.1), rand_bf16(rng, (b, n))
    dw32 = sb.backward_weight(to_dev(dyb), to_dev(xb), dw_dtype=torch.float32)
    dwbf = sb.backward_weight(to_dev(dyb), to_dev(xb))
    magnitude = oracle.weight_grad(dyb & 0x7fff, xb & 0x7fff)
    assert np.all(np.abs(host(dw32) - oracle.weight_grad(dyb, xb)) <= (b / 16 + 16) * 2.0 ** -23 * magnitude)
    assert torch.equal(dwbf, dw32.bfloat16())


# A second item per workgroup on the 128x128 tiles (969 to 1008 tiles on 512 places): without a split, and with the tokens of a
# tile summed in seven pieces, which start over with the next item.  Bound as above.
MANY_SMALL_DW = [(70, 2624, 6080), (303, 2368, 6464), (14434, 3136, 4928)]


@pytest.mark.parametrize("b,n,m", MANY_SMALL_DW)
def test_weight_gradient_small_tiles_with_a_second_item(b, n, m):
    rng = np.random.default_rng(b + n + m)
    dy, x = to_dev(rand_bf16(rng, (b, m), 0.1)), to_dev(rand_bf16(rng, (b, n)))
    dw32, dwbf = sb.backward_weight(dy, x, dw_dtype=torch.float32), sb.backward_weight(dy, x)
    dy_t, x = dy.double().t().contiguous(), x.double()
    bound = (b / 16 + 16) * 2.0 ** -23 * (dy_t.abs() @ x.abs())
    assert bool(((dw32 - dy_t @ x).abs() <= bound).all())
    assert torch.equal(dwbf, dw32.bfloat16())


# A step whose arrays exceed the last-level cache (24 million elements in four tensors, 20 million in one: 280 to 390 MB;
# the second pass runs backwards and non-temporally) computes what each tensor's own step does, bit for bit, and the single-tensor form of the same rule
# agrees with the binary64 evaluation; ragged counts, so that the last workgroups are partial.
@pytest.mark.parametrize("grad_dtype", [torch.bfloat16, torch.float32])
def test_adamw_step_larger_than_the_last_level_cache(grad_dtype):
    gen = torch.Generator(device=DEV).manual_seed(5)
    rand = lambda c: torch.randn(c, generator=gen, device=DEV)
    counts = [9_000_001, 7_000_003, 5, 8_388_608 + 4099]
    sets = [(rand(c) * 0.02, rand(c) * 3e-4, rand(c).square() * 1e-6, (rand(c) * 1e-3).to(grad_dtype)) for c in counts]
    single = [tuple(t.clone() for t in s) for s in sets]
    args = (1e-3, 0.9, 0.98, 1e-6, 0.2, 7)
    rms = sb.stable_adamw_step_multi(sb.AdamwPlan(sets), *args)
    for i, (a, s) in enumerate(zip(sets, single)):
        assert torch.equal(rms[i:i + 1], sb.stable_adamw_step(*s, *args)), counts[i]
        for x, y in zip(a[:3], s[:3]):
            assert torch.equal(x, y), counts[i]
    c = 20_000_007
    big = (rand(c) * 0.02, rand(c) * 3e-4, rand(c).square() * 1e-6, (rand(c) * 1e-3).to(grad_dtype))
    th, v, u, g = (t.double() for t in big)
    alpha, b1, b2, eps, lam = (float(np.float32(x)) for x in args[:5])
    b1, b2 = (b * (1 - b ** 6) / (1 - b ** 7) for b in (b1, b2))
    v, u = b1 * v + (1 - b1) * g, b2 * u + (1 - b2) * g * g
    want_rms = (g * g / u.clamp(min=eps * eps)).mean().sqrt()
    eta = alpha / want_rms.clamp(min=1.0)
    want = (th - eta * lam * th - eta * v / (u.sqrt() + eps), v, u)
    rms = sb.stable_adamw_step(*big, *args)
    assert abs(rms.item() - want_rms.item()) <= 2e-6 * want_rms.item()
    for got, ref in zip(big[:3], want):  # a handful of binary32 roundings (2^-24 each) of the tensor's values
        assert (got.double() - ref).norm() <= 4 * 2.0 ** -24 * ref.norm()


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("case", ["plain", "view", "parameter", "subclass", "transposed", "wrong dtype", "host", "rank",
                                  "function mode", "empty", "lazy negation"])
def test_builtin_tensor_checks_agree_with_the_general_ones(case):
    """The built-in forms of the two checks answer and refuse as the Python ones that they stand for."""
    base = torch.arange(64 * 64, device=DEV, dtype=torch.float32).view(64, 64)
    t = {"view": base[8:], "parameter": torch.nn.Parameter(base), "subclass": base.as_subclass(_Sub), "transposed": base.t(),
         "wrong dtype": base.bfloat16(), "host": base.cpu(), "rank": base.view(-1), "empty": base[:0],
         "lazy negation": torch._neg_view(base)}.get(case, base)
    sb._entries()

    def answer(f, *args):
        try:
            return f(*args)
        except sb.SwitchBackError as e:
            return str(e)

    mode = torch.overrides.BaseTorchFunctionMode() if case == "function mode" else torch.no_grad()
    with mode:
        assert answer(sb._dev, t, torch.float32, 2) == answer(sb._dev_general, t, torch.float32, 2)
        assert answer(sb._dev, t, torch.float32) == answer(sb._dev_general, t, torch.float32)
        assert answer(sb._dev, t, torch.float32, 2 ** 70) == answer(sb._dev_general, t, torch.float32, 2 ** 70)
        a, g = (answer(f, t, (64, 64), torch.float32, t.device, "y") for f in (sb._out, sb._out_general))
        assert a is g or a == g
        fresh, want = (f(None, (3, 5), t.dtype, t.device, "y") for f in (sb._out, sb._out_general))
    assert (fresh.shape, fresh.dtype, fresh.device, fresh.stride(), type(fresh), fresh.requires_grad) == (
        want.shape, want.dtype, want.device, want.stride(), type(want), want.requires_grad)


def test_ctypes_path_computes_the_same(monkeypatch, b=100, n=192, m=128):
    """The calls through ctypes, which another torch than the binding's takes: every entry point with an sb_saved, and one without."""
    rng = np.random.default_rng(5)
    x, w, dy = to_dev(rand_bf16(rng, (b, n))), to_dev(rand_bf16(rng, (m, n), n ** -0.5)), to_dev(rand_bf16(rng, (b, m), 0.1))

    def everything():
        y, bufs = sb.forward(x, w)
        out = [y, sb.backward_input(dy, bufs), *sb.backward_weight_m(dy, bufs), sb.backward_weight(dy, x, bufs),
               sb.forward_static(x, w, bufs)[0], sb.forward_bias_layerscale(x, w, bufs=bufs)[0], *sb.quantize_rowwise(x)]
        x8, w8 = x[:, :128].contiguous(), w[:, :128].contiguous()
        y8, bufs8 = sb.forward_f8(x8, w8)
        return out + [y8, sb.backward_input_f8(dy, bufs8)]

    built_in = everything()
    assert sb._dev is not sb._dev_general
    for name in ("_native", "_bound_to", "_dev", "_out"):
        monkeypatch.setattr(sb, name, getattr(sb, name))
    monkeypatch.setattr(sb, "_load_binding", lambda: None)
    sb._bind()
    assert sb._dev is sb._dev_general
    assert all(torch.equal(a, c) for a, c in zip(built_in, everything(), strict=True))
