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

// Estimated time (us) of the small-product kernel's best split for a product, and that split.  Fitted to a sweep of 30
// products (64..6304 rows, 128..8192 columns, K = 128..8192) on an MI355X; within 15 % on most of them.  k is in stages
// of 128 bytes.
inline double direct_product_time(int64_t M, int64_t N, int64_t K, int ncu, int *split) {
    const double k = (double)((K + 127) / 128);
    const int64_t blocks32 = ((M + 31) / 32) * (N / 32), blocks64 = ((M + 63) / 64) * (N / 64);
    const double t32 = 2.0 + (double)((blocks32 + ncu - 1) / ncu) * (0.35 + 0.091 * k);
    const double t64 = 2.8 + (double)((blocks64 + ncu - 1) / ncu) * (0.3 + 0.2 * k);
    const double fill = (double)blocks64 / ncu;  // two small workgroups share a compute unit's throughput
    const double t64h = 2.6 + (0.15 + 0.27 * k) * (fill > 1.0 ? fill : 1.0);
    *split = t32 <= t64 && t32 <= t64h ? DIRECT_32 : t64 <= t64h ? DIRECT_64 : DIRECT_64H;
    return *split == DIRECT_32 ? t32 : *split == DIRECT_64 ? t64 : t64h;
}

// The split that beats the 128x128-tile instance, or DIRECT_NONE.  That instance's workgroups take 0.61 us per k-tile
// while they are alone on their compute unit (a chain of LDS stages) and up to a third more when two share it.  Measured,
// tiles against blocks: 64 x 1024, K = 4096: 22.7 / 4.4 us; 512 x 256, K = 1024: 8.3 / 2.8; 197 x 3072, K = 768: 7.3 /
// 4.3; 2000 x 768, K = 3072: 18.3 / 11.9; and on the other side of the line 2000 x 3072, K = 768: 9.5 / 15.0; 1000 x 4096,
// K = 1024: 9.4 / 12.3.
inline int direct_split_for(int64_t M, int64_t N, int64_t K, int ncu) {
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
    const double over = tiles > ncu ? (double)(tiles - ncu) / ncu : 0.0;
    const double tiled = 2.9 + 0.61 * (double)((K + 127) / 128) * (1.0 + 0.35 * over);
    int split;
    return direct_product_time(M, N, K, ncu, &split) < tiled ? split : DIRECT_NONE;
}

// A product's rows [0, tile_rows) go to the tiled kernel (128x128 tiles if they make few 256x256 ones), the rest to the
// small-product kernel with `split`; either part may be empty, and split is DIRECT_NONE exactly if the second one is.
struct ProductPlan {
    int64_t tile_rows;
    int split;
};

// When the last, partial row of tiles starts another round of the persistent grid, that round keeps a few workgroups
// busy with tiles that are mostly past the end: the small-product kernel does those rows in less time than the round
// takes, if it is estimated below 6 us per 1024 of K.  Measured, one launch against two: 16448 x 1024, K = 4096 (260
// tiles, 64 rows split off) 87.4 / 62.1 us, K = 3072 72.0 / 51.7, K = 1024 28.4 / 23.7; 16448 x 4096, K = 1024 91.3 /
// 80.3; 32896 x 5120, K = 1280 (128 rows) 248.5 / 205.0; 8200 x 2048, K = 512 18.8 / 17.1.  Where the number of rounds
// stays (21000 x 800, K = 1536: 41.0 / 45.8) nothing is split off, and neither where the partial row is the only one (fewer
// than 256 rows of a very wide output): the tiles keep at least one whole row of tiles.
inline ProductPlan plan_product(int64_t M, int64_t N, int64_t K, int ncu) {
    int split = DIRECT_NONE;
    if (few_tiles(M, N, ncu)) {
        split = direct_split_for(M, N, K, ncu);
        return ProductPlan{split == DIRECT_NONE ? M : 0, split};
    }
    const int64_t full = M / 256 * 256, tiles_n = (N + 255) / 256, tiles = full / 256 * tiles_n;
    const bool same_rounds = (tiles + ncu - 1) / ncu == (tiles + tiles_n + ncu - 1) / ncu;
    if (full == 0 || full == M || same_rounds) return ProductPlan{M, DIRECT_NONE};
    if (direct_product_time(M - full, N, K, ncu, &split) < 6.0 / 1024.0 * (double)K) return ProductPlan{full, split};
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
