// Weight-gradient GEMM dW[j,k] = sum_i dY[i,j] * X[i,k] on 256x256 tiles: four waves of 128x128, one per SIMD.
//
// The same contraction as gemm_bf16_tn_kernel.h (which describes the layout: both operands lie in LDS as in memory,
// [token][column], and ds_read_b64_tr_b16 transposes), for weight gradients with long token ranges.
//
// What bounds it: the power the chip may draw (1.9 GHz instead of 2.4 on real values) and, with that out of the way
// (all-zero operands), the reads and requests that stand between the matrix instructions.  So the kernel moves as little
// as possible per multiply-add and lets nothing stand in their way:
//   * Wave tiles of 128x128 (256 accumulators a lane, in the AGPRs) read 128 KiB of LDS per 64 tokens where eight waves of
//     128x64 read 192, and v_mfma_f32_16x16x32_bf16 draws less power than 32x32x16 (1.99 against 1.80 PFLOP/s from
//     registers).
//   * One wave per SIMD has nobody to cover for it, so everything is issued in the shadow of a matrix instruction (16
//     cycles, of which it takes 4 to issue): a period is one 32-token stage, 64 matrix instructions, 32 transposing reads
//     of the next stage's fragments (three after every four instructions, from the ninth on) and eight 1 KiB requests
//     (one per eight instructions).  All requests in a row after the barrier would stop the wave for 1200 cycles.
//   * Four stages of 32 KiB: a request has at least two periods (2048 matrix cycles) to land.
// The loop keeps a constant number of requests in flight, so its one wait per period is a constant: past the last stage
// of a workgroup the requests go on with an empty buffer resource (zeros from the bounds check, no memory traffic).
// The matrix instructions are inline asm: their accumulators have to stay in AGPRs, and no fragment may be moved while
// its asm read is in flight (an instance that spills must never run, and the build refuses one).
//
// 32896 tokens, 1280 -> 5120: 395 -> 351 us with the reduction of its five splits (eight waves of 128x64 before; 1.09 ->
// 1.23 PFLOP/s); 16384 tokens, 4096 -> 16384: 1630 -> 1515 us (1.45 PFLOP/s; all-zero operands 1420 -> 1185); 16448
// tokens, 1024 -> 3072: 101 -> 92.
#pragma once
#include "gemm_bf16_tn_kernel.h"

namespace sb {

struct WideCfg {
    static constexpr int BM = 256, BN = 256, BKT = 32, STAGES = 4, THREADS = 256;
    static constexpr int UNIT = 2 * BKT;               // token ranges are whole pairs of stages: fragments alternate buffers
    static constexpr int WT = 128, NB = WT / 16;       // wave tile, in blocks of 16x16
    static constexpr int PITCH = 512;                  // bytes of one token row of an operand tile in LDS
    static constexpr int OP_BYTES = BKT * PITCH, STAGE_BYTES = 2 * OP_BYTES;  // dY tile, then X tile
    static constexpr int LPW = STAGE_BYTES / 1024 / 4; // 1 KiB requests per wave and stage
    static constexpr int NREADS = 4 * NB;              // transposing reads per wave and stage (two per fragment)
    static constexpr int EPI_WAVE_BYTES = 16 * WT * 2; // 16 rows of bf16
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES + 4 * EPI_WAVE_BYTES;
    static_assert((STAGES & (STAGES - 1)) == 0 && LDS_BYTES <= 160 * 1024, "configuration");
};

// No item may be empty (every token range holds a token): the caller sees to it.
__device__ __forceinline__ void gemm_bf16_tn_wide_body(const GemmBf16Args &p) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    typedef __attribute__((address_space(3))) void lds_void;
    typedef WideCfg C;
    constexpr int S = C::STAGES, NB = C::NB;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: what derives from it is scalar
    const int lane = threadIdx.x & 63;
    const int wm0 = (wave >> 1) * C::WT, wn0 = (wave & 1) * C::WT;

    // Requests.  Waves 0 and 1 load dY, 2 and 3 X; request i of a wave fills the token rows tok0 + 2i and tok0 + 2i + 1.
    // LDS slot (token, p) holds 16-byte column chunk p ^ (key << 1), key = bits 0, 1 and 3 of the token: the eight token
    // rows that half a transposing read touches (32 bytes each) then fall into eight different 32-byte bank windows.
    // Tokens past b read as zero through the bounds check; columns past the operand's width read the next token row or,
    // at the very end, zeros, and only feed results that are never stored.
    const bool loads_dy = wave < 2;
    const unsigned ld = loads_dy ? p.m : p.n;
    void *const operand = (void *)(loads_dy ? p.dy : p.x);
    const int l_tok = lane >> 5, l_pos = lane & 31;
    const int tok0 = (wave & 1) * (C::BKT / 2);
    unsigned voff[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) voff[v] = (unsigned)l_tok * ld * 2 + ((l_pos ^ ((l_tok | v << 1) << 1)) << 4);
    const unsigned req_step = 4 * ld, stage_step = (unsigned)C::BKT * 2 * ld;

    // Work items (GemmBf16Args): this workgroup's item `round` counts if it is below `total`.
    const int tiles = p.tiles_m * p.tiles_n, total = tiles * p.splits;
    const int first = (blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    struct Item {
        int tm, tn, split, stages;  // stages: even
        bool have;
    };
    auto item_of = [&](int round) -> Item {
        const int id = round * (int)gridDim.x + first;
        Item it;
        it.have = id < total;
        it.split = id / tiles;
        const int tile = id % tiles, minor = p.tiles_m < p.tiles_n ? p.tiles_m : p.tiles_n;
        const int i = tile % minor, j = tile / minor;
        it.tm = p.tiles_m < p.tiles_n ? i : j;
        it.tn = p.tiles_m < p.tiles_n ? j : i;
        it.stages = (min(p.b - it.split * p.k_per_split, p.k_per_split) + C::UNIT - 1) / C::UNIT * 2;
        return it;
    };

    // Load cursor: four stages ahead of the matrix instructions, across items.
    int l_round = 0, l_left = 0;
    unsigned l_soff = 0, l_bytes = 0;  // offset of the next stage; size of the operand, 0 past the last item
    auto next_item_sources = [&]() {
        const Item it = item_of(l_round++);
        l_left = it.have ? it.stages : 1 << 30;
        l_bytes = it.have ? (unsigned)p.b * ld * 2 : 0;
        l_soff = ((unsigned)(it.split * p.k_per_split + tok0) * ld + (unsigned)(loads_dy ? it.tm * C::BM : it.tn * C::BN)) * 2;
    };
    auto issue_req = [&](int slot, int i) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            __builtin_amdgcn_make_buffer_rsrc(operand, 0, l_bytes, 0x00020000),
            (lds_void *)(smem + slot * C::STAGE_BYTES + (wave * C::LPW + i) * 1024), 16, voff[(i & 1) | (i >> 2) << 1],
            l_soff + (unsigned)i * req_step, 0, 0);
    };
    auto advance = [&]() {
        l_soff += stage_step;
        if (--l_left == 0) next_item_sources();
    };
    next_item_sources();
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int i = 0; i < C::LPW; ++i) issue_req(s, i);
        advance();
    }

    // Fragments: lane l holds column l % 16 of a 16-column block at tokens 8 * (l / 16) .. + 7, fetched by two transposing
    // reads of four tokens each; within a 16-lane group lane r addresses token r / 4 and columns 4 * (r % 4) ...
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const int f_r = lane & 15, f_g = lane >> 4;
    const int f_tok = f_g * 8 + (f_r >> 2);
    const int f_key = (f_tok & 3) | (f_g & 1) << 2;  // the same for f_tok + 4
    const unsigned f_lane = lds_base + f_tok * C::PITCH + (f_r & 3) * 8;
    unsigned goff[NB], xoff[NB];
#pragma unroll
    for (int f = 0; f < NB; ++f) {
        goff[f] = f_lane + wm0 * 2 + ((f ^ f_key) << 5);
        xoff[f] = f_lane + C::OP_BYTES + wn0 * 2 + ((f ^ f_key) << 5);
    }
    v2u gf[2][NB][2], xf[2][NB][2];
    auto issue_read = [&](int i, int buf, int slot) {  // i-th read of the stage in `slot`, into register buffer buf
        const int f = i >> 2;
        const unsigned x_at = xoff[f] + slot * C::STAGE_BYTES, g_at = goff[f] + slot * C::STAGE_BYTES;
        switch (i & 3) {
            case 0: asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(xf[buf][f][0]) : "v"(x_at)); break;
            case 1: asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(xf[buf][f][1]) : "v"(x_at), "n"(4 * C::PITCH)); break;
            case 2: asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(gf[buf][f][0]) : "v"(g_at)); break;
            default: asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(gf[buf][f][1]) : "v"(g_at), "n"(4 * C::PITCH)); break;
        }
    };
    auto pin_frags = [&](int buf) {  // ties the registers to the wait before this call
#pragma unroll
        for (int f = 0; f < NB; ++f)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                asm volatile("" : "+v"(xf[buf][f][h]));
                asm volatile("" : "+v"(gf[buf][f][h]));
            }
    };
    auto frag = [&](const v2u (&q)[2]) -> v8bf {
        return __builtin_bit_cast(v8bf, __builtin_shufflevector(q[0], q[1], 0, 1, 2, 3));
    };

    wait_vmcnt<(S - 1) * C::LPW>();
    block_barrier();
#pragma unroll
    for (int i = 0; i < C::NREADS; ++i) issue_read(i, 0, 0);

    int g = 0;      // stages done; stage g lies in slot g % S
    int slack = 0;  // periods whose wait may leave an epilogue's stores outstanding
    Item it = item_of(0);
    for (int round = 1; it.have; ++round) {
        v4f acc[NB][NB];
        // One stage: its fragments are in registers (or on their way), the next one's are read, the one after the last
        // requested takes the slot that this one has left.  The barrier says that every wave has its fragments of this
        // stage and that its share of the next one has landed.
        auto period = [&](auto cur_c, auto first_c) __attribute__((always_inline)) {
            constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1;
            constexpr bool first = decltype(first_c)::value;  // of the item: the accumulators start at zero
            const int slot = g & (S - 1), next_slot = (g + 1) & (S - 1);
            // The requests of the next stage are older than those of the two after it and, for three periods after an
            // epilogue, than its stores (at least 32).
            if (slack == 0) {
                wait_vmcnt<2 * C::LPW>();
            } else {
                --slack;
                wait_vmcnt<2 * C::LPW + 32>();
            }
            wait_lds_reads();
            block_barrier();
            pin_frags(cur);
#pragma unroll
            for (int idx = 0; idx < NB * NB; ++idx) {
                const int a = idx / NB, b = a & 1 ? NB - 1 - idx % NB : idx % NB;
                if (first)
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[a][b]) : "v"(frag(xf[cur][b])), "v"(frag(gf[cur][a])));
                else
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[a][b]) : "v"(frag(xf[cur][b])), "v"(frag(gf[cur][a])));
                if (idx >= 8) {
#pragma unroll
                    for (int i = (idx - 8) * 3 / 4; i < (idx - 7) * 3 / 4; ++i)
                        if (i < C::NREADS) issue_read(i, nxt, next_slot);
                }
                if (idx % 8 == 4) issue_req(slot, idx / 8);
                __builtin_amdgcn_sched_barrier(0);
            }
            advance();
            ++g;
        };
        period(std::integral_constant<int, 0>(), std::true_type());
        period(std::integral_constant<int, 1>(), std::false_type());
        for (int kt = 2; kt < it.stages; kt += 2) {
            period(std::integral_constant<int, 0>(), std::false_type());
            period(std::integral_constant<int, 1>(), std::false_type());
        }
        // Nobody knows of the matrix instructions in the asm: their last results need up to 18 wait states.
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");

        // A lane owns row l % 16 of dW and four consecutive columns of every block.  Rows past the end lie beyond the
        // buffer resource of the wave tile, columns past the end are sent there: the number of stores is always the same.
        const int m_base = it.tm * C::BM + wm0, n_base = it.tn * C::BN + wn0;
        const unsigned rows_in = __builtin_amdgcn_readfirstlane(min(max(p.m - m_base, 0), C::WT));
        const int cols_in = p.n - n_base;
        // The addresses are formed from opaque copies, so that none is kept through the main loop.
        int lane_e = lane, n = p.n;
        asm volatile("" : "+v"(lane_e));
        asm volatile("" : "+s"(n));
        const int e_r = lane_e & 15, e_g = lane_e >> 4;
        constexpr unsigned NOWHERE = 0x80000000u;
        if (p.splits == 1 && p.out_bf16) {
            // Final bf16 result: transposed through the wave-private patch, 256-byte row segments.
            const __amdgpu_buffer_rsrc_t rsrc_out = __builtin_amdgcn_make_buffer_rsrc(
                static_cast<unsigned short *>(p.out) + (int64_t)m_base * n + n_base, 0, rows_in * n * 2, 0x00020000);
            unsigned char *epi = smem + S * C::STAGE_BYTES + wave * C::EPI_WAVE_BYTES;
            const unsigned o_voff = e_r * 8 < cols_in ? (unsigned)(e_g * n + e_r * 8) * 2 : NOWHERE;
#pragma unroll
            for (int a = 0; a < NB; ++a) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    v4f v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {  // asm: the compiler would read all 256 of them first, and spill
                        float x;
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[a][b][e]));
                        v[e] = x;
                    }
                    *reinterpret_cast<v4bf *>(epi + e_r * 256 + (((b * 2 + (e_g >> 1)) ^ e_r) << 4) + (e_g & 1) * 8) =
                        __builtin_convertvector(v, v4bf);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int prow = j * 4 + e_g;
                    const v4u val = *reinterpret_cast<const v4u *>(epi + prow * 256 + ((e_r ^ prow) << 4));
                    __builtin_amdgcn_raw_buffer_store_b128(val, rsrc_out, o_voff, (unsigned)(a * 16 + j * 4) * n * 2, 0);
                }
            }
        } else {
            // binary32: final result (one split) or this split's partial sums, straight from the accumulators.
            float *out = p.splits > 1 ? p.partial + (int64_t)it.split * p.m * n : static_cast<float *>(p.out);
            const __amdgpu_buffer_rsrc_t rsrc_out = __builtin_amdgcn_make_buffer_rsrc(out + (int64_t)m_base * n + n_base, 0,
                                                                                      rows_in * n * 4, 0x00020000);
            const unsigned o_voff = (unsigned)(e_r * n + 4 * e_g) * 4;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const unsigned at = b * 16 < cols_in ? o_voff : NOWHERE;
#pragma unroll
                for (int a = 0; a < NB; ++a)
                    asm volatile("buffer_store_dwordx4 %0, %1, %2, %3 offen" ::"a"(acc[a][b]), "v"(at), "s"(rsrc_out),
                                 "s"((unsigned)(a * 16 * n + b * 16) * 4)
                                 : "memory");
            }
        }
        slack = 3;
        it = item_of(round);
    }
    wait_vmcnt<0>();  // the requests past the end write LDS
    wait_lds_reads();
}

}  // namespace sb
