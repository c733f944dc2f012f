// Which kernels a product or a weight gradient of a given size runs: host arithmetic alone (no HIP in this file), so that the
// rules can be compiled and checked over their whole range without a GPU.
#pragma once
#include <stdint.h>

namespace sb {

// The small-product kernel's splits of the work (gemm_i8_direct.hip).
enum { DIRECT_NONE = 0, DIRECT_32, DIRECT_64, DIRECT_64H };

// Fewer than half as many 256x256 tiles as compute units.
inline bool few_tiles(int64_t M, int64_t N, int ncu) {
    const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256);
    return tiles * 2 <= ncu;
}

// Estimated time (us) of the small-product kernel's best split for a product, and that split.  Fitted to 1300 products
// (1..33000 rows, 64..8192 columns, K = 64..8192; int8 with every scale and output type, float8) on an MI355X: the ratio to
// the measured time has a standard deviation of 10 % per split, and the split picked is 0.3 % slower than the best one in
// the mean.  k is in stages of 128 bytes.  The 32x32 split is for outputs whose 64x64 blocks leave compute units idle;
// beyond one block per compute unit it fetches too much (734 x 1600, K = 8064: 45 us, the 64x64 splits 29.5).
inline double direct_product_time(int64_t M, int64_t N, int64_t K, int ncu, int *split) {
    const double k = (double)((K + 127) / 128);
    const int64_t blocks32 = ((M + 31) / 32) * (N / 32), blocks64 = ((M + 63) / 64) * (N / 64);
    const int64_t rounds32 = (blocks32 + ncu - 1) / ncu, rounds64 = (blocks64 + ncu - 1) / ncu;
    const int64_t rounds64h = (blocks64 + 2 * ncu - 1) / (2 * ncu);
    const double t32 = 1.6 + (double)rounds32 * (0.5 + 0.079 * k);
    const double t64 = rounds64 <= 1 ? 2.75 + 0.19 * k : (double)rounds64 * (2.45 + 0.24 * k);
    const double t64h = rounds64 <= 1 ? 2.65 + 0.275 * k : (double)rounds64h * (3.35 + 0.45 * k);
    *split = rounds64 <= 1 && t32 <= t64 && t32 <= t64h ? DIRECT_32 : t64 <= t64h ? DIRECT_64 : DIRECT_64H;
    return *split == DIRECT_32 ? t32 : *split == DIRECT_64 ? t64 : t64h;
}

// Workgroups of the tiled kernel's persistent grid: a multiple of the XCD count, at most `slots` (what the GPU holds at
// once).  When the tiles make only a few rounds of the full grid and do not fill the last one, the grid is shrunk so that
// every workgroup gets the same number of tiles (645 tiles: 216 workgroups x 3 instead of 256 x 2.5): the number of
// rounds is the same, and the kernel being power-bound, fewer active compute units run at a higher clock, which measures
// 4-10 % faster than a last round that leaves half the GPU idle.  With many rounds the tail is a small share and the full
// grid measures better.
inline int persistent_grid(int64_t tiles, int slots) {
    int full = slots & ~7;
    if (full < 8) full = 8;
    const int64_t rounds = (tiles + full - 1) / full;
    if (rounds < 1) return 8;
    if (rounds > 4) return full;
    const int64_t per_round = (tiles + rounds - 1) / rounds;
    const int grid = (int)((per_round + 7) & ~7LL);
    return grid > full ? full : grid < 8 ? 8 : grid;
}

// What a product does besides the contraction: int8 with one weight scale; int8 with column scales or with bias and
// layer-scale; float8.
enum ProductKind { PRODUCT_PLAIN = 0, PRODUCT_LONG_EPILOGUE, PRODUCT_F8 };

// The tiled kernels: 128x128 (gemm_i8_kernel.h, two workgroups per compute unit), 256x128 and 256x256
// (gemm_i8_wide_kernel.h).
enum TileKind { TILES_128 = 0, TILES_256X128, TILES_256, TILE_KINDS };

// 256x256 tiles of a single stage, one per workgroup at most: they have instances of their own (gemm_i8_wide_kernel.h).
inline bool one_stage(int64_t M, int64_t N, int64_t K, int ncu) {
    return K <= 128 && ((M + 255) / 256) * ((N + 255) / 256) <= (ncu & ~7);
}

// Estimated time (us) of a product on tiles.  With r rounds of the persistent grid (of the XCD with most tiles), u tiles on
// the compute unit that gets most (2 r where two workgroups share one), k stages of 128 bytes and enough tiles for f rounds of
// a full grid:
//   launch + r * boundary + u * boundary_u + k * (r * stage + f * stage_f + u * stage_u) + store * megabytes of output
// Two-byte outputs fitted to 1200 products (100..40000 rows, 64..8192 columns, K = 128..8192; every output and scale) on an
// MI355X: the ratio to the measured time has a standard deviation of 4 to 6 %, the tile picked is 0.3 to 0.7 % slower than the
// best one in the mean.  Four-byte ones, whose stores weigh as much as the product of a short contraction, to 7000 and (float8)
// 6000 products within 30 % of the best tile: picked / best 1.003 (1.016 without u: 34752 x 192, K = 384 makes 532 tiles of
// 128x128, two on a few compute units' both workgroups, 17.6 us, 14.0 on 256x256 ones).
inline double tiled_product_time(TileKind tile, int64_t M, int64_t N, int64_t K, ProductKind kind, int out_bytes,
                                 int ncu) {
    struct Fit {
        double launch, boundary, stage, stage_f, store, boundary_u, stage_u;
    };
    static const Fit fits[5][TILE_KINDS] = {
        // 128x128, 256x128, 256x256: int8; int8 with the longer epilogues; float8; four-byte outputs, int8 and float8
        {{2.29, 1.36, 0.541, 0.502, 0.055, 0, 0}, {2.79, 1.56, 0.548, 0.274, 0.013, 0, 0}, {2.84, 2.72, 0.971, 0.484, 0.034, 0, 0}},
        {{2.02, 2.28, 0.534, 0.496, 0.089, 0, 0}, {2.82, 2.18, 0.536, 0.267, 0.011, 0, 0}, {2.39, 4.41, 0.954, 0.500, 0.008, 0, 0}},
        {{1.74, 1.60, 0.537, 0.368, 0.056, 0, 0}, {2.07, 2.18, 0.473, 0.242, 0.072, 0, 0}, {1.54, 3.66, 0.851, 0.444, 0.034, 0, 0}},
        {{3.80, 0, 0.339, 0.489, 0.036, 1.90, 0.119}, {4.60, 3.60, 0.426, 0.465, 0.012, 0, 0}, {5.15, 6.61, 0.780, 0.807, 0.016, 0, 0}},
        {{3.47, 0, 0.399, 0.432, 0.028, 2.12, 0.056}, {4.54, 3.65, 0.367, 0.459, 0.015, 0, 0}, {4.88, 6.79, 0.641, 0.844, 0.018, 0, 0}}};
    const Fit &fit = fits[out_bytes == 2 ? (int)kind : kind == PRODUCT_F8 ? 4 : 3][tile];
    const int bm = tile == TILES_128 ? 128 : 256, bn = tile == TILES_256 ? 256 : 128;
    const int slots = tile == TILES_128 ? 2 * ncu : ncu;
    const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn), per_xcd = persistent_grid(tiles, slots) / 8;
    const double rounds = (double)(((tiles + 7) / 8 + per_xcd - 1) / per_xcd), unit = per_xcd * 8 > ncu ? 2 * rounds : rounds;
    const double k = (double)((K + 127) / 128 > 1 || tile != TILES_256X128 ? (K + 127) / 128 : 2);
    return fit.launch + rounds * fit.boundary + unit * fit.boundary_u +
           k * (rounds * fit.stage + (double)tiles / slots * fit.stage_f + unit * fit.stage_u) +
           fit.store * 1e-6 * (double)M * (double)N * out_bytes;
}

// The tile with the smallest estimate; the 128x128 ones on equal terms, up to 3 % with two-byte outputs (the wider ones lose 7
// % on a narrow miss at worst, where they win 4 % in the mean).  Not for a single stage, where a narrow miss goes the other way
// (6251 x 1408, K = 128: 8.1 us on 128x128 tiles, 7.3 on 256x256 ones; 24576 x 320: 8.0 and 7.1).
inline double best_tiles(int64_t M, int64_t N, int64_t K, ProductKind kind, int out_bytes, int ncu, TileKind *tile) {
    double best = (K > 128 && out_bytes == 2 ? 0.97 : 1.0) * tiled_product_time(TILES_128, M, N, K, kind, out_bytes, ncu);
    *tile = TILES_128;
    for (int i = TILES_128 + 1; i < TILE_KINDS; ++i) {
        const double t = tiled_product_time((TileKind)i, M, N, K, kind, out_bytes, ncu);
        if (t < best) {
            best = t;
            *tile = (TileKind)i;
        }
    }
    return best;
}

// A product's rows [0, first_rows) go to 256x256 tiles, [first_rows, tile_rows) to `rest` ones, the others to the small-product
// kernel with `split`.  Any of the three parts may be empty; split is DIRECT_NONE exactly if the last one is.
struct ProductPlan {
    int64_t first_rows, tile_rows;
    TileKind rest;
    int split;
};

// The whole product on the small-product kernel: while its 64x64 blocks fit the GPU at once, two per compute unit, and few
// 256x256 tiles; 0.15 to 1.04 of the 128x128 tiles' time up to there and 0.9 to 2.3 of it past it.  64 x 1024, K = 4096:
// 4.4 us against 22.7; 197 x 3072, K = 768: 4.3 / 7.3; 2000 x 768, K = 3072: 11.9 / 18.3; on the other side of the line
// 1137 x 1856, K = 128: 5.6 / 4.4; 7233 x 320, K = 1920: 16.7 / 13.5; 338 x 5760, K = 7552 with bias and layer-scale: 52.7 /
// 41.6.  Long contractions of nearly that many blocks are bound by their operands' way from L2 (12.5 TB/s assumed, 11.4
// measured with float8 at K = 6784) and run on tiles if those save a tenth by the estimates.  Those are cautious: it takes
// float8, two-byte outputs and K above 8192.  Below, the blocks are slower by up to a fifth (us, blocks / 256x128 tiles: 5431 x
// 384, K = 6784, float8 39.0 / 31.8; 190 x 8128, K = 8128 52.9 / 42.2).
//
// Otherwise the fastest of the tiles by the estimates, or 256x256 tiles for the whole rows of them that fill whole rounds of
// the grid and another kernel for the rows that would start the next round:
//   LAST ROWS.  The last, partial row of tiles starts another round, which keeps a few workgroups busy with tiles that are
//   mostly past the end; the small-product kernel may do those rows in less time.  16448 x 1024, K = 4096 (64 rows split off)
//   80.6 / 62.6 us; 16448 x 4096, K = 1024 91.3 / 80.3 (eight-wave tiles).  What the round takes, by 900 products: 7 us per
//   1024 of K and 1 us more if it is the second one; if more come before it, workgroups that finish early start it, and it
//   takes 5.5 us per 1024 of K; 7 with the longer epilogues (K >= 1024); 4 where the stores of full rounds get into each
//   other's way (the plain int8 product at K < 1024, and four-byte outputs).  Four-byte outputs in several rounds are bound by
//   their stores if there are many or K is small, and gain nothing reliable.  Where the number of rounds stays nothing is
//   split off, and neither where the partial row is the only one (fewer than 256 rows of a very wide output).
//   WHOLE ROUNDS.  More than a partial row is left: other tiles do those rows.  It has to save 5 % by the estimates.
// us on 128x128, 256x128 and 256x256 tiles alone / so: 6304 x 768, K = 3072 24.1, 19.9, 31.3 / 20.1; 8000 x 1024, K = 4096 37.5,
// 29.9, 43.1 / 29.7; 11237 x 2880, K = 1088 49.8, 39.2, 46.4 / 39.4; 30000 x 1280, K = 4096 169, 130, 134 / 124 (whole rounds);
// 16448 x 1024, K = 4096 87.5, 68.8, 78.9 / 54.0 (last rows).
inline ProductPlan plan_product(int64_t M, int64_t N, int64_t K, ProductKind kind, int out_bytes, int ncu) {
    ProductPlan plan{0, M, TILES_256, DIRECT_NONE};
    int split = DIRECT_NONE;
    double best = best_tiles(M, N, K, kind, out_bytes, ncu, &plan.rest);
    if (few_tiles(M, N, ncu)) {
        const int64_t blocks = ((M + 63) / 64) * (N / 64);
        if (blocks > 2 * (int64_t)ncu) return plan;
        const double latency = direct_product_time(M, N, K, ncu, &split), traffic = (double)(blocks * 128 * K) / 12.5e6;
        if (best < 0.9 * (latency > traffic ? latency : traffic)) return plan;
        plan.tile_rows = 0;
        plan.split = split;
        return plan;
    }
    const int64_t full = M / 256, tiles_n = (N + 255) / 256, rounds = (full * tiles_n + ncu - 1) / ncu;
    // LAST ROWS
    if (full > 0 && M % 256 != 0 && ((full + 1) * tiles_n + ncu - 1) / ncu != rounds &&
        (out_bytes == 2 || rounds == 1 || (rounds <= 3 && K >= 1024))) {
        const double k1024 = (double)K / 1024.0;
        const double later = out_bytes > 2 || (kind == PRODUCT_PLAIN && K < 1024) ? 4.0
                             : kind == PRODUCT_LONG_EPILOGUE && K >= 1024 ? 7.0 : 5.5;
        const double rest = direct_product_time(M - full * 256, N, K, ncu, &split);
        const double t = tiled_product_time(TILES_256, full * 256, N, K, kind, out_bytes, ncu) + rest;
        if (rest < (rounds == 1 ? 1.0 + 7.0 * k1024 : later * k1024) && t < 1.05 * best) {
            best = t < best ? t : best;
            plan = ProductPlan{full * 256, full * 256, TILES_256, split};
        }
    }
    // WHOLE ROUNDS
    const int64_t whole = full * tiles_n / ncu * ncu / tiles_n;  // rows of tiles in whole rounds
    if (whole > 0 && whole < full) {
        TileKind rest;
        const double t = tiled_product_time(TILES_256, whole * 256, N, K, kind, out_bytes, ncu) +
                         best_tiles(M - whole * 256, N, K, kind, out_bytes, ncu, &rest);
        if (t < 0.95 * best) plan = ProductPlan{whole * 256, M, rest, DIRECT_NONE};
    }
    return plan;
}

// ---- Weight gradient of b tokens, dW [m, n]: 256x256 tiles (gemm_bf16_tn_wide_kernel.h) or 128x128 ones, two workgroups
// per compute unit (gemm_bf16_tn_kernel.h), and into how many items the token range of a tile is split.

enum { DW_STAGE = 64 };  // tokens; every token range but the last is whole stages

// Pieces that the tokens of a tile are summed in, at least: long chains of binary32 additions lose precision (512 tokens,
// 256 -> 1024: relative error 0.90e-7 in two pieces, 1.25e-7 in one; 16448 tokens, 1024 -> 3072, 3.5e-7 in five pieces, twice
// that in one).  As many as once were the fastest splits, of 256x256 tiles where they leave 32 stages each (whole rounds of
// the GPU with as few as that takes), else of 128x128 ones (in units of a stage, 1.1 us: the stages of an item, at 0.64 of
// the unit while a compute unit has one workgroup; the partial sums at 2.9 TB/s and 2.7 for the launch that adds them, which
// does not count where it is what keeps the range whole).
inline int least_pieces(int64_t b, int64_t n, int64_t m, int ncu) {
    const int64_t stages = (b + DW_STAGE - 1) / DW_STAGE;
    const int64_t tiles = ((m + 255) / 256) * ((n + 255) / 256), small_tiles = ((m + 127) / 128) * ((n + 127) / 128);
    int best = 1;
    double best_score = -1.0;
    for (int s = 1; s <= 16 && (s == 1 || (int64_t)s * DW_STAGE * 4 <= b); ++s) {
        const int64_t items = tiles * s, rounds = (items + ncu - 1) / ncu;
        const double score = (double)items / (double)(rounds * ncu) - 0.015 * s;
        if (score > best_score) {
            best_score = score;
            best = s;
        }
    }
    if (best == 1 || stages / best >= 32) return best;
    const double pass = (double)m * (double)n * 4.0 / (2.9e12 * 1.1e-6);
    for (double launch = 2.7; launch >= 0.0; launch -= 2.7) {
        double best_cost = 0.0;
        for (int s = 1; s <= 16 && (s == 1 || (int64_t)s * DW_STAGE * 4 <= b); ++s) {
            double cost = s > 1 ? (s + 0.5) * pass + launch : 0.0;
            for (int64_t left = small_tiles * s; left > 0; left -= 2 * ncu) {
                const int64_t k = left < 2 * ncu ? left : 2 * ncu;
                cost += (double)((stages + s - 1) / s) * (k <= ncu ? 0.64 : 0.64 + 0.36 * (double)(k - ncu) / ncu);
            }
            if (s == 1 || cost < best_cost) {
                best_cost = cost;
                best = s;
            }
        }
        if (best > 1) break;
    }
    return best;
}

// splits > 1: partial sums and a launch that adds them.  pieces > 1 (128x128 tiles, one item per tile): the pieces are summed
// in registers, to the bits of the split product.  No split of the 256x256 tiles is empty.
struct WeightGradPlan {
    bool small;
    int splits, stages_per_split, pieces, stages_per_piece;
};

// Estimated time (us).  r rounds of the grid, enough items for f full grids, k stages per item, w the compute units' second
// workgroups over all rounds (small tiles), MB megabytes of binary32 result:
//   256x256: 1.3 + 4.45 r + k (0.995 r + 0.341 f);  128x128: 2.8 + k (0.465 r + 0.072 w + 0.434 f);  both 0.09 to 0.17 MB
//   split: 6.6 + 0.02 s + 0.23 s MB;  3.7 + 0.07 s + 0.31 s MB
// fitted to 5900 launches of 1000 weight gradients (100..34000 tokens, widths 128..8192, 1 to 96 splits): the ratio to the
// measured time has a standard deviation of 5 and 9 %.
// Int: 32 bits where the sizes allow it (all that the calls take): a plan divides whole numbers up to 78 times over, on the host
// and in every call (with the stop below 1.4 -> 0.2 us at 16448 tokens, 1024 -> 3072, 1.7 -> 0.8 at 28030, 320 -> 192).
template <class Int>
struct WeightGradTime {
    Int side, slots, ncu, stages, tiles;
    double mb;
    WeightGradTime(bool small, int64_t b, int64_t n, int64_t m, int ncu)
        : side(small ? 128 : 256), slots(small ? 2 * ncu : ncu), ncu(ncu), stages((Int)((b + DW_STAGE - 1) / DW_STAGE)),
          tiles((Int)((m + side - 1) / side) * (Int)((n + side - 1) / side)), mb((double)m * (double)n * 4e-6) {}
    double of(Int s) const {
        const Int items = tiles * s, rounds = (items + slots - 1) / slots;
        const double k = (double)((stages + s - 1) / s), full = (double)items / slots;
        if (side == 256)
            return 1.32 + 4.45 * rounds + k * (0.995 * rounds + 0.341 * full) + 0.087 * mb +
                   (s > 1 ? 6.62 + (0.017 + 0.232 * mb) * s : 0.0);
        const Int last = items - (rounds - 1) * slots;
        const double second = (double)(rounds - 1) + (last > ncu ? (double)(last - ncu) / ncu : 0.0);
        return 2.84 + k * (0.465 * rounds + 0.072 * second + 0.434 * full) + 0.17 * mb +
               (s > 1 ? 3.71 + (0.07 + 0.314 * mb) * s : 0.0);
    }
    // No larger than of(s) or any of(s' > s): the work of a full GPU and the cost of the partial sums.
    double at_least(int s) const {
        const double work = (double)stages * tiles / slots;
        return side == 256 ? (0.995 + 0.341) * work + (0.017 + 0.232 * mb) * s : (0.465 + 0.434) * work + (0.07 + 0.314 * mb) * s;
    }
};

// The fastest by the estimates that sums in least_pieces or more; the split that the pieces are of, unless another saves 6 %
// (what looks 3 % better loses 5 to 13 % in one of ten: 23446 tokens, 576 -> 1792 66.6 against 75.6 us).  Measured against that
// split always (us): 28030 tokens, 320 -> 192 405 / 25; 5214 tokens, 256 -> 448 81 / 14; 197 tokens, 768 -> 3072 9.8 / 5.6; 0.72
// of the time in the mean over 5541 weight gradients (eight-wave kernel before), 32 of them 5 to 11 % slower.
template <class Int>
inline WeightGradPlan plan_weight_gradient_in(int64_t b, int64_t n, int64_t m, int ncu) {
    const int64_t stages = (b + DW_STAGE - 1) / DW_STAGE;
    const int least = least_pieces(b, n, m, ncu);
    const bool long_items = least == 1 || stages / least >= 32;
    WeightGradPlan plan{true, 1, (int)stages, least, (int)((stages + least - 1) / least)};
    double best = WeightGradTime<Int>(true, b, n, m, ncu).of(1) + (least > 1 ? 0.3 : 0.0);
    for (int i = 0; i < 2 && stages > 0; ++i) {
        const bool small = i == 0;
        const int most = small ? 64 : 16, shortest = small ? 4 : 6;  // splits; stages of one, if there are more than `least`
        const WeightGradTime<Int> time(small, b, n, m, ncu);
        for (int s = least; s <= most && (s == least || stages >= s * shortest); ++s) {
            if (small && s == 1) continue;
            if (s > least && time.at_least(s) > best) break;
            const double t = time.of(s) * (s == least && small != long_items ? 0.94 : 1.0);
            if (t >= best) continue;
            const int64_t per_split = (stages + s - 1) / s;
            best = t;
            plan = WeightGradPlan{small, (int)((stages + per_split - 1) / per_split), (int)per_split, 1, (int)per_split};
        }
    }
    return plan;
}
inline WeightGradPlan plan_weight_gradient(int64_t b, int64_t n, int64_t m, int ncu) {
    const bool narrow = b <= (int64_t)1 << 30 && n <= (int64_t)1 << 18 && m <= (int64_t)1 << 18;  // 64 splits of 2^22 tiles
    return narrow ? plan_weight_gradient_in<int32_t>(b, n, m, ncu) : plan_weight_gradient_in<int64_t>(b, n, m, ncu);
}

}  // namespace sb
