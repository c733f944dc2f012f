// Which kernels an int8 or float8 product of a given size runs: host arithmetic alone (no HIP in this file), so that the
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

// The split that beats the 128x128-tile instance, or DIRECT_NONE.  The line is where the 64x64 blocks no longer fit the
// GPU at once, two per compute unit: over the same products the best split takes 0.15 to 1.04 of the tiles' time up to
// there (median 0.4) and 0.9 to 2.3 of it past it (median 1.4).  Tiles against blocks: 64 x 1024, K = 4096: 22.7 / 4.4 us;
// 197 x 3072, K = 768: 7.3 / 4.3; 2000 x 768, K = 3072: 18.3 / 11.9; and on the other side of the line 1137 x 1856,
// K = 128: 4.4 / 5.6; 7233 x 320, K = 1920: 13.5 / 16.7; 338 x 5760, K = 7552 with bias and layer-scale: 41.6 / 52.7.
inline int direct_split_for(int64_t M, int64_t N, int64_t K, int ncu) {
    int split = DIRECT_NONE;
    if (((M + 63) / 64) * (N / 64) <= 2 * (int64_t)ncu) direct_product_time(M, N, K, ncu, &split);
    return split;
}

// What a product does besides the contraction: int8 with one weight scale; int8 with column scales or with bias and
// layer-scale; float8.
enum ProductKind { PRODUCT_PLAIN = 0, PRODUCT_LONG_EPILOGUE, PRODUCT_F8 };

// A product's rows [0, tile_rows) go to the tiled kernel (128x128 tiles if they make few 256x256 ones), the rest to the
// small-product kernel with `split`; either part may be empty, and split is DIRECT_NONE exactly if the second one is.
struct ProductPlan {
    int64_t tile_rows;
    int split;
};

// When the last, partial row of tiles starts another round of the persistent grid, that round keeps a few workgroups
// busy with tiles that are mostly past the end, and the small-product kernel may do those rows in less time.  Measured,
// one launch against two: 16448 x 1024, K = 4096 (260 tiles, 64 rows split off) 87.4 / 62.1 us, K = 3072 72.0 / 51.7,
// K = 1024 28.4 / 23.7; 16448 x 4096, K = 1024 91.3 / 80.3; 32896 x 5120, K = 1280 (128 rows) 248.5 / 205.0;
// 8200 x 2048, K = 512 18.8 / 17.1.  What the round takes, by 900 products: 7 us per 1024 of K and 1 us more if it is
// the second one; if more come before it, workgroups that finish early start it, and it takes 5.5 us per 1024 of K; 7
// with the longer epilogues (K >= 1024); 4 where the stores of full rounds get into each other's way (the plain int8
// product, whose waves share the rows 3 : 5, at K < 1024; and four-byte outputs).  One line at 6 us per 1024 of K made
// 4337 x 8192, K = 1600 67.2 / 72.9 and 19692 x 2496, K = 768 50.8 / 56.2.  Four-byte outputs in several rounds are
// bound by their stores if there are many or K is small, and gain nothing reliable (52260 x 1088, K = 2624 216 / 231;
// 32956 x 1024, K = 768 53.2 / 59.8).  Where the number of rounds stays (21000 x 800, K = 1536: 41.0 / 45.8) nothing is
// split off, and neither where the partial row is the only one (fewer than 256 rows of a very wide output): the tiles
// keep at least one whole row of tiles.
inline ProductPlan plan_product(int64_t M, int64_t N, int64_t K, ProductKind kind, int out_bytes, int ncu) {
    int split = DIRECT_NONE;
    if (few_tiles(M, N, ncu)) {
        split = direct_split_for(M, N, K, ncu);
        return ProductPlan{split == DIRECT_NONE ? M : 0, split};
    }
    const int64_t full = M / 256 * 256, tiles_n = (N + 255) / 256, tiles = full / 256 * tiles_n;
    const int64_t rounds = (tiles + ncu - 1) / ncu;
    if (full == 0 || full == M || (tiles + tiles_n + ncu - 1) / ncu == rounds) return ProductPlan{M, DIRECT_NONE};
    if (out_bytes > 2 && rounds > 1 && (rounds > 3 || K < 1024)) return ProductPlan{M, DIRECT_NONE};
    const double k1024 = (double)K / 1024.0;
    const double later = out_bytes > 2 || (kind == PRODUCT_PLAIN && K < 1024) ? 4.0
                         : kind == PRODUCT_LONG_EPILOGUE && K >= 1024 ? 7.0 : 5.5;
    const double round = rounds == 1 ? 1.0 + 7.0 * k1024 : later * k1024;
    if (direct_product_time(M - full, N, K, ncu, &split) < round) return ProductPlan{full, split};
    return ProductPlan{M, DIRECT_NONE};
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

}  // namespace sb
