// The product of gemm_i8_kernel.h for few output elements: the same arithmetic, another split of the work, hand-written
// for gfx950.  int8 results are the same bits; a float8 sum is formed in up to four pieces instead of one chain.
//
// A product with few output tiles is bound by latency, not by matrix instructions: on 128x128 tiles a 197 x 3072
// output is 48 workgroups for 256 compute units, and each of them walks the contraction as a serial chain of k-tiles
// whose operands arrive one LDS stage ahead.  Here a workgroup owns a small output block (ROWS x COLS) and its waves
// split the CONTRACTION: every wave has its own ring of LDS stages, which it alone fills and reads, so nothing waits
// for another wave until the partial sums meet in LDS at the end.  Integer partial sums are exact, so the bits do not
// depend on the split.  The float8 sums are added in wave order, so the bits of a row may depend on whether its product
// (or its place among the last rows of a large one) takes this kernel; the group sums of the matrix instruction lie on a
// coarse grid and binary32 mostly holds their sums exactly: over 18 products (64..4000 rows, K = 128..8192, both data
// families) the error against binary64 is that of the tiled kernel to four digits (5.9e-5 of the result with uniform
// codes, 8.8e-6 with normal data).
//
// The operands go through LDS although no two waves share them: a load straight into the registers of a matrix
// fragment has neighbouring lanes in different rows, which the address path serves at 17-20 bytes per clock and compute
// unit whatever the fragment (a 64 x 1024 product with K = 4096 took 9.0 us so on the 32-row and on the 16-row
// instruction); eight lanes per 128-byte row segment are what it is made for (4.4 us).
//
// Operand bytes per multiply-add are 1/ROWS + 1/COLS, four to eight times those of the 256x256 tile: the line up to
// which this pays is in the dispatch.
#pragma once
#include "gemm_i8_kernel.h"

namespace sb {

template <int ROWS_, int COLS_, int WAVES_>
struct DirectCfg {
    static constexpr int ROWS = ROWS_, COLS = COLS_, WAVES = WAVES_;
    static constexpr int STAGES = 2;  // of a wave's ring
    static constexpr int RB = ROWS / 32, CB = COLS / 32, THREADS = 64 * WAVES;
    static constexpr int BK = 128;                          // bytes of k per stage: one cache line per operand row
    static constexpr int STAGE_BYTES = (ROWS + COLS) * BK;  // token rows, then weight rows
    static constexpr int REQ = STAGE_BYTES / 1024;          // 1 KiB requests per stage, eight rows each
    static constexpr int PITCH = COLS + 4;  // dwords per row of a partial-sum block in LDS (16-byte aligned, rows 4 banks apart)
    static constexpr int WAVE_BYTES = STAGES * STAGE_BYTES;  // a wave's ring; its partial sums follow in the same place
    static constexpr int LDS_BYTES = WAVES * WAVE_BYTES;
    static constexpr int QUADS = ROWS * COLS >= 8 * THREADS ? 2 : 1;  // column quads a lane finishes and stores at once
    static_assert(ROWS % 32 == 0 && (COLS == 32 || COLS == 64), "configuration");
    static_assert(LDS_BYTES <= 160 * 1024 && ROWS * PITCH * 4 <= WAVE_BYTES, "LDS");
    static_assert(REQ * (STAGES - 1) < 64, "vmcnt range");
};

// K is a multiple of 64 (int8; the last stage of an odd multiple is half zeros) or of 128 (float8); N of 64.
template <class C, int OUT, bool COLSCALE, int MATH, bool POST>
__device__ __forceinline__ void gemm_i8_direct_body(const GemmI8Args &p) {
    constexpr bool F8 = MATH >= MATH_F8;
    constexpr int FMT_X = MATH & 1, FMT_W = (MATH >> 1) & 1;
    constexpr int RPF = F8 ? 2 : 1;  // 16-byte LDS reads per operand fragment
    constexpr int KKG = 4 / RPF;     // matrix instructions per stage and block
    typedef typename std::conditional<F8, v16f, v16i>::type AccT;
    typedef typename std::conditional<F8, v8i, v4i>::type FragT;
    typedef typename std::conditional<F8, v4f, v4i>::type QuadT;
    typedef typename std::conditional<F8, float, int>::type ElemT;
    typedef __attribute__((address_space(3))) void lds_void;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int frow = lane & 31, fhalf = lane >> 5;
    // Blocks are numbered row block fastest: consecutive workgroups share the weight rows, the larger operand.
    const int m0 = ((int)blockIdx.x % p.tiles_m) * C::ROWS, n0 = ((int)blockIdx.x / p.tiles_m) * C::COLS;
    const int steps = (p.K + C::BK - 1) / C::BK;
    const int s0 = (int)((long long)wave * steps / C::WAVES), s1 = (int)((long long)(wave + 1) * steps / C::WAVES);
    const int n = s1 - s0;

    // Requests.  LDS slot (row, q) of a stage holds 16-byte chunk q ^ (row/2 % 8) of that row (no bank conflicts in the
    // fragment reads); the swizzle is applied to the address a lane fetches.  Request i covers rows 8i .. 8i+7, so the
    // swizzle takes two values.  Rows past M and, in a last stage that is half a stage, chunks past K read as zero
    // through the bounds check of the buffer resource.
    const __amdgpu_buffer_rsrc_t rsrc_a =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.a, 0, (unsigned)((size_t)p.M * (size_t)p.K), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_b =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.b, 0, (unsigned)((size_t)p.N * (size_t)p.K), 0x00020000);
    unsigned voff[2], voff_last[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int row = 8 * v + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
        voff[v] = (unsigned)(lane >> 3) * (unsigned)p.K + (unsigned)chunk * 16;
        voff_last[v] = (steps - 1) * C::BK + chunk * 16 < p.K ? voff[v] : 0xfffffff0u;
    }
    unsigned char *ring = smem + wave * C::WAVE_BYTES;
    const unsigned req_step = 8u * (unsigned)p.K;
    auto issue = [&](int i) {  // stage i of this wave's n
        unsigned char *dst = ring + (i % C::STAGES) * C::STAGE_BYTES;
        const unsigned k0 = (unsigned)(s0 + i) * C::BK;
        const bool last = s0 + i + 1 == steps;
        const unsigned v0 = last ? voff_last[0] : voff[0], v1 = last ? voff_last[1] : voff[1];
#pragma unroll
        for (int r = 0; r < C::ROWS / 8; ++r)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lds_void *)(dst + r * 1024), 16, r & 1 ? v1 : v0,
                                                     (unsigned)m0 * (unsigned)p.K + (unsigned)r * req_step + k0, 0, 0);
#pragma unroll
        for (int r = 0; r < C::COLS / 8; ++r)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lds_void *)(dst + C::ROWS * C::BK + r * 1024), 16,
                                                     r & 1 ? v1 : v0,
                                                     (unsigned)n0 * (unsigned)p.K + (unsigned)r * req_step + k0, 0, 0);
    };

    AccT acc[C::RB][C::CB];
#pragma unroll
    for (int r = 0; r < C::RB; ++r)
#pragma unroll
        for (int c = 0; c < C::CB; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[r][c][e] = 0;

    // What the epilogue needs besides the sums, requested before the operands so that it is there when they are summed
    // (fetched in the epilogue, one element at a time, bias and layer-scale took a 197 x 3072 product from 5.1 to 7.6 us).  A
    // lane finishes V consecutive columns, the same ones in all of its rows.
    constexpr int V = 4 * C::QUADS, ROW_LANES = C::THREADS / (C::COLS / V), ITEMS = C::ROWS / ROW_LANES;
    static_assert(C::THREADS % (C::COLS / V) == 0 && C::ROWS % ROW_LANES == 0, "rows and columns of a lane");
    const int col = ((int)threadIdx.x % (C::COLS / V)) * V, row0 = (int)threadIdx.x / (C::COLS / V);
    const bool has_bias = POST && p.bias != nullptr, has_gamma = POST && p.gamma != nullptr;
    float srow[ITEMS], tensor_scale = 0.0f;
    v4f scol[C::QUADS], bias[C::QUADS], gamma[C::QUADS];
    if (OUT != OUT_I32) {
        if (!COLSCALE) tensor_scale = p.state_tensor[0];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) srow[i] = p.state_row[min(m0 + row0 + i * ROW_LANES, p.M - 1)];
#pragma unroll
        for (int h = 0; h < C::QUADS; ++h) {
            const int j = n0 + col + 4 * h;
            if (COLSCALE) scol[h] = *reinterpret_cast<const v4f *>(p.state_col + j);
            if (has_bias) bias[h] = *reinterpret_cast<const v4f *>(p.bias + j);
            if (has_gamma) gamma[h] = *reinterpret_cast<const v4f *>(p.gamma + j);
        }
    }
    asm volatile("" ::: "memory");  // not sunk to their uses

    // Fragment reads: inline asm with counted waits, because the compiler would put a wait for every outstanding
    // request in front of each LDS read.
    const unsigned ring_at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring;
    int frag_off[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) frag_off[kk] = frow * C::BK + (((kk * 2 + fhalf) ^ ((frow >> 1) & 7)) << 4);
    FragT xf[2][C::RB], wf[2][C::CB];
    auto read_group = [&](int buf, int slot, int g) {
        const unsigned at = ring_at + slot * C::STAGE_BYTES + frag_off[g * RPF];
        const unsigned at2 = ring_at + slot * C::STAGE_BYTES + frag_off[g * RPF + RPF - 1];  // second half (float8)
        auto read = [&](auto off) -> FragT {
            constexpr int OFF = decltype(off)::value;
            if constexpr (F8) {
                const v4i lo = lds_read_b128<OFF>(at);
                const v4i hi = lds_read_b128<OFF>(at2);
                return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            } else {
                return lds_read_b128<OFF>(at);
            }
        };
        xf[buf][0] = read(std::integral_constant<int, 0>());
        if constexpr (C::RB == 2) xf[buf][1] = read(std::integral_constant<int, 32 * C::BK>());
        wf[buf][0] = read(std::integral_constant<int, C::ROWS * C::BK>());
        if constexpr (C::CB == 2) wf[buf][1] = read(std::integral_constant<int, (C::ROWS + 32) * C::BK>());
    };
    constexpr int GROUP_READS = (C::RB + C::CB) * RPF;
    static_assert(C::RB <= 2 && 2 * GROUP_READS <= 16, "fragment reads");

#pragma unroll
    for (int i = 0; i < C::STAGES; ++i)
        if (i < n) issue(i);
    for (int i = 0; i < n; ++i) {
        const int slot = i % C::STAGES;
        wait_stage<C::REQ>(min(C::STAGES - 1, n - 1 - i));  // the requests of a wave retire in order
        __builtin_amdgcn_sched_barrier(0);
        read_group(0, slot, 0);
#pragma unroll
        for (int g = 0; g < KKG; ++g) {
            const int cur = g & 1;
            if (g + 1 < KKG) {
                read_group(cur ^ 1, slot, g + 1);
                wait_lgkmcnt<(GROUP_READS < 16 ? GROUP_READS : 15)>();
            } else {
                wait_lgkmcnt<0>();
            }
#pragma unroll
            for (int r = 0; r < C::RB; ++r) asm volatile("" : "+v"(xf[cur][r]));
#pragma unroll
            for (int c = 0; c < C::CB; ++c) asm volatile("" : "+v"(wf[cur][c]));
#pragma unroll
            for (int r = 0; r < C::RB; ++r)
#pragma unroll
                for (int c = 0; c < C::CB; ++c) {
                    if constexpr (F8)
                        acc[r][c] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wf[cur][c], xf[cur][r], acc[r][c], FMT_W,
                                                                                    FMT_X, 0, 0, 0, 0);
                    else
                        acc[r][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[cur][c], xf[cur][r], acc[r][c], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (i + C::STAGES < n) issue(i + C::STAGES);  // every read of the slot has returned
        __builtin_amdgcn_sched_barrier(0);
    }

    // Partial sums -> the wave's own LDS, row-major (its requests have landed and its reads have returned).  A lane holds
    // row frow of a 32-row block and, per quad q, columns 8q + 4*fhalf .. +3.
    constexpr int PART_DWORDS = C::WAVE_BYTES / 4;
    ElemT *part = reinterpret_cast<ElemT *>(smem) + wave * PART_DWORDS;
#pragma unroll
    for (int r = 0; r < C::RB; ++r)
#pragma unroll
        for (int c = 0; c < C::CB; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                QuadT v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[r][c][4 * q + e];
                *reinterpret_cast<QuadT *>(part + (32 * r + frow) * C::PITCH + 32 * c + 8 * q + 4 * fhalf) = v;
            }
    __syncthreads();

    if (!F8) tensor_scale = tensor_scale / 16129.0f;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int row = row0 + i * ROW_LANES;
        const ElemT *src = reinterpret_cast<const ElemT *>(smem) + row * C::PITCH + col;
        ElemT sum[V];
#pragma unroll
        for (int h = 0; h < C::QUADS; ++h) {
            QuadT t = *reinterpret_cast<const QuadT *>(src + 4 * h);
#pragma unroll
            for (int w = 1; w < C::WAVES; ++w) t += *reinterpret_cast<const QuadT *>(src + w * PART_DWORDS + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[4 * h + e] = t[e];
        }
        const int gr = m0 + row, gc = n0 + col;
        if (gr >= p.M) continue;
        if (OUT == OUT_I32) {
            v4i *out = reinterpret_cast<v4i *>(static_cast<int *>(p.out) + (int64_t)gr * p.N + gc);
#pragma unroll
            for (int h = 0; h < C::QUADS; ++h)
                out[h] = v4i{(int)sum[4 * h], (int)sum[4 * h + 1], (int)sum[4 * h + 2], (int)sum[4 * h + 3]};
            continue;
        }
        const float rscale = COLSCALE ? srow[i] : srow[i] * tensor_scale;
        v4f y[C::QUADS];
#pragma unroll
        for (int h = 0; h < C::QUADS; ++h) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = (float)sum[4 * h + e] * (COLSCALE ? rscale * (scol[h][e] / 16129.0f) : rscale);
                if (has_bias) v = v + bias[h][e];  // skipped, not added, when absent: -0 + 0 would lose the sign
                if (has_gamma) v = gamma[h][e] * v;
                y[h][e] = v;
            }
        }
        if (OUT == OUT_BF16) {
            unsigned short *out = static_cast<unsigned short *>(p.out) + (int64_t)gr * p.N + gc;
            v2u bits[C::QUADS];
#pragma unroll
            for (int h = 0; h < C::QUADS; ++h) bits[h] = __builtin_bit_cast(v2u, __builtin_convertvector(y[h], v4bf));
            if constexpr (C::QUADS == 2)
                *reinterpret_cast<v4u *>(out) = v4u{bits[0].x, bits[0].y, bits[1].x, bits[1].y};
            else
                *reinterpret_cast<v2u *>(out) = bits[0];
        } else {
            v4f *out = reinterpret_cast<v4f *>(static_cast<float *>(p.out) + (int64_t)gr * p.N + gc);
#pragma unroll
            for (int h = 0; h < C::QUADS; ++h) out[h] = y[h];
        }
    }
}

// Launchers (gemm_i8_direct.hip).  split: which of the kernel's splits of the work (dispatch.h); they take 0 < M, and
// operand sizes the tiled kernel accepts too.
// The product's rows [first, end) (out_bytes: size of an output element).
GemmI8Args rows_of(const GemmI8Args &a, int64_t first, int64_t end, size_t out_bytes);
// out_dtype SB_I32_RAW ignores the states; a.state_col != nullptr: row-and-column scales; post: a.bias / a.gamma follow.
hipError_t launch_gemm_i8_direct(int split, const GemmI8Args &a, bool post, sb_dtype out_dtype, hipStream_t stream);
hipError_t launch_gemm_f8_direct(int split, const GemmI8Args &a, int fmt_a, int fmt_b, sb_dtype out_dtype,
                                 hipStream_t stream);

}  // namespace sb
