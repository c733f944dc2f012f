// The 8-bit product on 256x256 tiles: four waves of 128x128, one per SIMD.
//
//   out[i,j] = scale * sum_k aq[i,k] * bq[j,k]      aq [M,K], bq [N,K], K contiguous; scales, outputs and arguments as in
//                                                   gemm_i8_kernel.h, which serves products with few tiles
//
// What bounds it: power (1.9 to 2.0 GHz instead of 2.4 on real codes) and, next to the matrix instructions, the way of the
// operands from L2 into LDS.  So it moves little per multiply-add and issues everything in the shadow of the matrix
// instructions; there is no second wave on the SIMD to cover for a wave that waits.
//   * Wave tiles of 128x128: 256 accumulators a lane (all AGPRs), 128 KiB of LDS read per 128 bytes of k where eight waves
//     of 128x64 read 192.  int8 runs v_mfma_i32_16x16x64_i8, which draws less power than 32x32x32 (3.95 against 3.43
//     POP/s from registers); float8 v_mfma_f32_32x32x64_f8f6f4 (the 16-row instruction takes 128 bytes of k, whose
//     fragments do not fit twice).  The weight-side tile is the first operand: a lane owns one output row and four
//     consecutive columns per accumulator quad.
//   * A stage is 128 bytes of k, whole cache lines: with stages of 64 bytes every request fetched its lines twice
//     (32896 x 5120, K = 1280: 201 us, 185 so; 8192^3: 392, 360).  It is worked off in two halves, whose fragments alternate
//     between two register buffers: while one half is multiplied the other's are read, one read per three instructions
//     from the fifth on.
//   * Two stages.  A stage's LDS is free when its second half's fragments are in registers, so one barrier per stage, at
//     the start of the second half, hands it over, and the 16 requests per wave of the stage after the next go out during that
//     half, one per four instructions (16 per 32 or 48 of them: 4 to 10 % slower; spread over both halves: the same).
//   * The epilogue of a tile is interleaved with the first half stage of the next one: a block's accumulators are read
//     just before the instruction that starts them again from zero, and converted in its shadow and the next ones'.  The last
//     tile's epilogue follows its own last instructions at a distance (3588 x 2560, K = 128: 7.8 -> 7.4 us; 7.1 on the
//     instances of one stage).
//     Results go through a wave-private LDS patch (padded rows) and leave as 16-byte non-temporal stores in row segments of
//     256 (float8: 128) bytes.
//   * Row states, column states, bias and layer-scale of a tile are requested into LDS with its first stage.
// 256x128 tiles (waves of 128x64, half the accumulators) are for products whose 256x256 tiles do not fill the GPU or fill its
// last round badly.  A stage is 48 KiB and three fit; its requests are spread over two half stages, and land a stage later.
// 128x128 tiles, two workgroups per compute unit / 256x256 tiles / these (us): 6304 x 768, K = 3072 24.1 / 31.3 / 19.9; 8000 x
// 1024, K = 4096 37.5 / 43.1 / 29.9; 6304 x 3072, K = 768 23.1 / 21.5 / 19.6; 11237 x 2880, K = 1088 49.8 / 46.4 / 39.2.
//
// All loops count on a constant number of vector-memory operations: past the last tile the requests go on with an empty
// buffer resource, rows past the end lie beyond the output's resource and columns past the end are sent there.
//
// Accumulators, fragment reads and matrix instructions are inline asm.  No fragment may be moved while its read is in
// flight: an instance that spills must never run, and the build refuses one, as it does a value of the compiler's in an AGPR.
//
// Measured against eight waves of 128x64 with two in-row bursts of requests per stage (us, codes of normal data):
//   32896 x 5120, K = 1280: 207 -> 185 (2.34 POP/s); 32896 x 1280, K = 5120: 183 -> 170; 16384 x 4096, K = 16384: 870 ->
//   787; 8192^3: 420 -> 360 (3.06); 11237 x 2880, K = 1088: 46.0 -> 43.0; with row and column scales 32896 x 1280,
//   K = 1280: 64.4 -> 56.6; bias and layer-scale 64.9 -> 56.0; binary32 output 76.2 -> 67.9; float8 32896 x 1280, K = 5120:
//   180 -> 165; all-zero codes, 8192^3: 296 -> 283.
#pragma once
#include "gemm_i8_kernel.h"

namespace sb {

// The 256 accumulators of a lane are the AGPRs, named in the asm text (as values of the compiler's they would be copied
// at the joins of the control flow, and spilled).  This keeps values of the compiler's out of them.
__device__ __forceinline__ void keep_out_of_agprs() {
    asm volatile("" ::
                     :
                 "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15",
                 "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31",
                 "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47",
                 "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63",
                 "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79",
                 "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95",
                 "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111",
                 "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127",
                 "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143",
                 "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159",
                 "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175",
                 "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191",
                 "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207",
                 "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223",
                 "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239",
                 "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255");
}

template <int MATH, bool COLSCALE, bool POST, int BN_ = 256>
struct WideI8Cfg {
    static constexpr bool F8 = MATH >= MATH_F8;
    static constexpr int BM = 256, BN = BN_, BK = 128, THREADS = 256;
    static constexpr int STAGES = BN == 256 ? 2 : 3;
    static constexpr int WTM = 128, WTN = BN / 2;        // wave tile
    static constexpr int A_BYTES = BM * BK, STAGE_BYTES = (BM + BN) * BK;  // token-side tile, then weight-side tile
    static constexpr int REQ_A = BM / 32, REQ_B = BN / 32, LPW = REQ_A + REQ_B;  // 1 KiB requests per wave and stage
    static constexpr int BLK = F8 ? 32 : 16, NBM = WTM / BLK, NBN = WTN / BLK;  // matrix instruction blocks of a wave tile
    static constexpr int QUADS = F8 ? 4 : 1;             // accumulator quads of a block, eight columns apart
    static constexpr int SLOTS = NBM * NBN;              // matrix instructions per half stage
    static constexpr int RPF = F8 ? 2 : 1;               // 16-byte reads per fragment
    static constexpr int NREADS = (NBM + NBN) * RPF;     // fragment reads per wave and half stage
    // Requests of a stage that go out during the second half of the stage STAGES before it; the others follow during the
    // next first half.
    static constexpr int REQ_2ND = BN == 256 ? LPW : LPW / 2;
    // Patch that transposes the bf16 results of one block row (part of one with 32-row blocks), padded rows.
    static constexpr int PATCH_COLS = F8 ? WTN / 2 : WTN, PATCH_PITCH = PATCH_COLS * 2 + 16;
    static constexpr int PATCH_BYTES = BLK * PATCH_PITCH, PATCH_SLOTS = PATCH_COLS / BLK;
    static constexpr int PPR = PATCH_COLS / 8, PATCH_READS = BLK * PPR / 64;  // 16-byte pieces per row; reads of a patch
    // Vectors of a tile in LDS (a float per row or column), and the tiles they are kept for.  A new tile's vectors are
    // requested up to STAGES + 1 stages ahead of its first epilogue, and what they overwrite must have been read before the
    // last barrier: with tiles of at least MIN_KT stages this many places do.
    static constexpr int MIN_KT = BN == 256 ? 1 : 2, RING = BN == 256 ? 4 : 3;
    static constexpr int VEC_AT = STAGES * STAGE_BYTES + 4 * PATCH_BYTES;
    static constexpr int VEC_BYTES = BM * 4 + (COLSCALE + 2 * POST) * BN * 4;
    static constexpr int LDS_BYTES = VEC_AT + RING * VEC_BYTES;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// ONE_STAGE: the contraction is one stage and no workgroup has a second tile.  Instances of their own, which make no requests
// past the stage and multiply both halves block by block, so that the epilogue starts at once (one round of 256x256 tiles, K =
// 128: 7.3 -> 7.0 us, K = 64: 7.6 -> 7.1; as a way through the other instances, those lost 0.4 %).
template <int OUT, bool COLSCALE, int MATH, bool POST, int BN = 256, bool ONE_STAGE = false>
__device__ __forceinline__ void gemm_i8_wide_body(const GemmI8Args &p) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    typedef __attribute__((address_space(3))) void lds_void;
    typedef WideI8Cfg<MATH, COLSCALE, POST, BN> C;
    constexpr int S = C::STAGES, NBM = C::NBM, NBN = C::NBN, RPF = C::RPF;
    constexpr bool F8 = C::F8;
    constexpr int FMT_X = MATH & 1, FMT_W = (MATH >> 1) & 1;
    typedef typename std::conditional<F8, float, int>::type AccE;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: what derives from it is scalar
    const int lane = threadIdx.x & 63;
    const int wm0 = (wave >> 1) * C::WTM, wn0 = (wave & 1) * C::WTN;
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    // Stages of a tile; K = 64 mod 128 ends in half a stage of zeros, and a stage of zeros follows if that makes too few.
    const int KT = max((p.K + C::BK - 1) / C::BK, C::MIN_KT);
    const int zero_stages = KT - (p.K + C::BK - 1) / C::BK;
    const bool half_last = !F8 && p.K % C::BK != 0;

    // ---- Requests.  Every wave loads a quarter of the token side's rows (a) and of the weight side's (b), eight rows a
    // request; LDS slot (row, p) holds 16-byte chunk p ^ f(row), f = the row's lowest three bits (16-row blocks) or the three
    // above the lowest (32-row blocks).  Rows past M (or N) read as zero through the bounds check.
    const int l_row = lane >> 3;
    unsigned voff[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int key = F8 ? (v * 8 + l_row) >> 1 : l_row;
        voff[v] = (unsigned)l_row * p.K + (((lane ^ key) & 7) << 4);
    }
    const unsigned voff_half = (voff[0] - (unsigned)l_row * p.K) & 64 ? 0xfffffff0u : voff[0];  // chunks past K: out of bounds
    const unsigned req_step = 8u * p.K;

    struct Tile {
        int tm, tn;
        bool have;
    };
    auto tile_of = [&](int round) -> Tile {
        Tile t;
        t.tm = t.tn = 0;
        t.have = gemm_tile_of(blockIdx.x, round, gridDim.x, p.tiles_m, p.tiles_n, p.group_m, &t.tm, &t.tn);
        return t;
    };
    // Load cursor: STAGES stages ahead of the matrix instructions, across tiles.
    int l_round = 0, l_left = 0, l_ring = C::RING - 1;
    unsigned l_a = 0, l_b = 0;              // offsets of the next stage in the operands
    unsigned l_a_bytes = 0, l_b_bytes = 0;  // sizes of the operands, 0 past the last tile
    auto request_vec = [&](const float *src, int at, int first, int count, int n) {  // n of src's floats from `first`
        if (wave * 64 < n)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, (unsigned)count * 4, 0x00020000),
                (lds_void *)(smem + C::VEC_AT + l_ring * C::VEC_BYTES + at + wave * 256), 4, lane * 4,
                (unsigned)(first + wave * 64) * 4, 0, 0);
    };
    auto next_tile_sources = [&]() {
        const Tile t = tile_of(l_round++);
        l_left = t.have ? KT : 1 << 30;
        l_a_bytes = t.have ? (unsigned)p.M * (unsigned)p.K : 0;
        l_b_bytes = t.have ? (unsigned)p.N * (unsigned)p.K : 0;
        l_a = (unsigned)(t.tm * C::BM + wave * (C::BM / 4)) * (unsigned)p.K;
        l_b = (unsigned)(t.tn * C::BN + wave * (C::BN / 4)) * (unsigned)p.K;
        l_ring = l_ring + 1 == C::RING ? 0 : l_ring + 1;
        if (t.have && OUT != OUT_I32) {
            request_vec(p.state_row, 0, t.tm * C::BM, p.M, C::BM);
            if (COLSCALE) request_vec(p.state_col, C::BM * 4, t.tn * C::BN, p.N, C::BN);
            if (POST && p.bias != nullptr) request_vec(p.bias, C::BM * 4, t.tn * C::BN, p.N, C::BN);
            if (POST && p.gamma != nullptr) request_vec(p.gamma, C::BM * 4 + C::BN * 4, t.tn * C::BN, p.N, C::BN);
        }
    };
    auto issue_req = [&](int slot, int i) {
        const bool is_a = i < C::REQ_A;
        const int r = is_a ? i : i - C::REQ_A;
        unsigned char *dst = smem + slot * C::STAGE_BYTES +
                             (is_a ? wave * C::REQ_A * 1024 : C::A_BYTES + wave * C::REQ_B * 1024) + r * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            __builtin_amdgcn_make_buffer_rsrc((void *)(is_a ? p.a : p.b), 0, is_a ? l_a_bytes : l_b_bytes, 0x00020000),
            (lds_void *)dst, 16, half_last && l_left == 1 + zero_stages ? voff_half : voff[F8 ? r & 1 : 0],
            (is_a ? l_a : l_b) + (unsigned)r * req_step, 0, 0);
    };
    auto advance = [&]() {
        l_a += C::BK;
        l_b += C::BK;
        if (--l_left == 0)
            next_tile_sources();
        else if (C::MIN_KT > 1 && l_left <= zero_stages)
            l_a_bytes = l_b_bytes = 0;
    };
    next_tile_sources();
#pragma unroll
    for (int s = 0; s < (ONE_STAGE ? 1 : S); ++s) {
#pragma unroll
        for (int i = 0; i < C::LPW; ++i) issue_req(s, i);
        if (!ONE_STAGE) advance();
    }

    // ---- Fragments: 16 (float8: 32) bytes of one row a lane.  Which bytes of k a lane holds does not matter as long as both
    // operands agree.
    typedef v4i Half;
    const int f_r = lane & (C::BLK - 1), f_g = lane / C::BLK;
    // Chunk h * 4 + f_g (int8) or h * 4 + 2 * f_g and the one after it (float8) of row f_r, for half h of the stage.
    const unsigned f_off = f_r * C::BK + (F8 ? ((f_g * 2) ^ ((f_r >> 1) & 7)) << 4 : (f_g ^ (f_r & 7)) << 4);
    const unsigned x_lane = lds_base + wm0 * C::BK + f_off, w_lane = lds_base + C::A_BYTES + wn0 * C::BK + f_off;
    Half xf[2][NBM][RPF], wf[2][NBN][RPF];
    auto issue_read = [&](int i, int buf, int slot) {  // of half `buf` of the stage in `slot`, into register buffer buf
        constexpr int STEP = C::BLK * C::BK;
        // Fragments in the order w0 x0 w1 x1 ..., then the token side's others.
        const int n = i / RPF, h = i % RPF;
        const bool is_x = n < 2 * NBN ? n & 1 : true;
        const int f = n < 2 * NBN ? n >> 1 : n - NBN;
        const unsigned at = ((is_x ? x_lane : w_lane) ^ (buf << 6 | h << 4)) + slot * C::STAGE_BYTES;
        Half &dst = is_x ? xf[buf][f][h] : wf[buf][f][h];
        switch (f) {
            case 0: dst = lds_read_b128<0>(at); break;
            case 1: dst = lds_read_b128<STEP>(at); break;
            case 2: dst = lds_read_b128<2 * STEP>(at); break;
            case 3: dst = lds_read_b128<3 * STEP>(at); break;
            case 4: dst = lds_read_b128<4 * STEP>(at); break;
            case 5: dst = lds_read_b128<5 * STEP>(at); break;
            case 6: dst = lds_read_b128<6 * STEP>(at); break;
            default: dst = lds_read_b128<7 * STEP>(at); break;
        }
    };
    auto pin_frags = [&](int buf) {
#pragma unroll
        for (int h = 0; h < RPF; ++h) {
#pragma unroll
            for (int f = 0; f < NBM; ++f) asm volatile("" : "+v"(xf[buf][f][h]));
#pragma unroll
            for (int f = 0; f < NBN; ++f) asm volatile("" : "+v"(wf[buf][f][h]));
        }
    };

    float tensor_scale = 0.0f;
    if (OUT != OUT_I32 && !COLSCALE) tensor_scale = F8 ? p.state_tensor[0] : p.state_tensor[0] / 16129.0f;
    asm volatile("" : "+v"(tensor_scale));

    wait_vmcnt<(ONE_STAGE ? 0 : (S - 1) * C::LPW)>();
    block_barrier();
#pragma unroll
    for (int i = 0; i < C::NREADS; ++i) issue_read(i, 0, 0);

    int slot = 0;   // of the stage in work
    int slack = 0;  // hand-overs whose wait may leave an epilogue's stores outstanding

    // ---- Epilogue of the tile that has just been finished.  Bias and layer-scale that are absent become -0 and 1, which
    // change no value.
    float rscale[NBM];
    v4f scol[COLSCALE || POST ? NBN : 1], sgam[POST ? NBN : 1];
    __amdgpu_buffer_rsrc_t rsrc_out;
    unsigned o_voff = 0;
    int cols_in = 0, n_out = p.N;
    constexpr unsigned NOWHERE = 0x80000000u;
    constexpr int OB = OUT == OUT_BF16 ? 2 : 4;
    const unsigned patch = lds_base + S * C::STAGE_BYTES + wave * C::PATCH_BYTES;
    const unsigned patch_w = patch + f_r * C::PATCH_PITCH + f_g * 8;
    constexpr int PPR = C::PPR;
    const unsigned patch_r = patch + (lane / PPR) * C::PATCH_PITCH + (lane % PPR) * 16;

    auto epi_begin = [&](const Tile &t, int ring) {
        const unsigned vec = lds_base + C::VEC_AT + ring * C::VEC_BYTES;
        if (OUT != OUT_I32) {
            const unsigned at = vec + (wm0 + f_r) * 4;
#pragma unroll
            for (int a = 0; a < NBM; ++a)
                asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(rscale[a]) : "v"(at), "n"(a * C::BLK * 4));
        }
        if (COLSCALE || POST) {
            const unsigned at = vec + C::BM * 4 + (wn0 + 4 * f_g) * 4;
#pragma unroll
            for (int b = 0; b < NBN; ++b)
                asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(scol[b]) : "v"(at), "n"(b * 64));
            if (POST)
#pragma unroll
                for (int b = 0; b < NBN; ++b)
                    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(sgam[b]) : "v"(at + C::BN * 4), "n"(b * 64));
        }
        wait_lds_reads();
        if (OUT != OUT_I32) {
#pragma unroll
            for (int a = 0; a < NBM; ++a) asm volatile("" : "+v"(rscale[a]));
#pragma unroll
            for (int a = 0; a < NBM; ++a) rscale[a] = COLSCALE ? rscale[a] : rscale[a] * tensor_scale;
        }
        if (COLSCALE || POST)
#pragma unroll
            for (int b = 0; b < NBN; ++b) {
                asm volatile("" : "+v"(scol[b]));
                if (POST) asm volatile("" : "+v"(sgam[b]));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (COLSCALE) scol[b][e] = scol[b][e] / 16129.0f;
                    if (POST) scol[b][e] = p.bias != nullptr ? scol[b][e] : -0.0f;
                    if (POST) sgam[b][e] = p.gamma != nullptr ? sgam[b][e] : 1.0f;
                }
            }
        const int m_base = t.tm * C::BM + wm0, n_base = t.tn * C::BN + wn0;
        const unsigned rows_in = __builtin_amdgcn_readfirstlane(min(max(p.M - m_base, 0), C::WTM));
        cols_in = p.N - n_base;
        n_out = p.N;
        asm volatile("" : "+s"(n_out));
        rsrc_out = __builtin_amdgcn_make_buffer_rsrc(static_cast<char *>(p.out) + ((int64_t)m_base * p.N + n_base) * OB, 0,
                                                     rows_in * (unsigned)p.N * OB, 0x00020000);
        int lane_e = lane;
        asm volatile("" : "+v"(lane_e));
        if (OUT == OUT_BF16)
            o_voff = (unsigned)((lane_e / PPR) * p.N + (lane_e % PPR) * 8) * 2;
        else if (F8)
            o_voff = (unsigned)((lane_e & 15) * p.N + (lane_e >> 4 & 1) * 8 + (lane_e >> 5) * 4) * 4;
        else
            o_voff = (unsigned)((lane_e & (C::BLK - 1)) * p.N + (lane_e / C::BLK) * 4) * 4;
    };
    v4u val[C::PATCH_READS];
    // Quad q of block (a, b), dequantized: x are the block's accumulators.
    auto epi_value = [&](int a, int b, int q, const AccE *x) -> v4f {
        v4f y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            y[e] = (float)x[4 * q + e] * (COLSCALE ? rscale[a] * scol[b][e] : rscale[a]);
            if (POST) y[e] = sgam[b][e] * (y[e] + scol[b][e]);
        }
        return y;
    };
    auto epi_quad = [&](int a, int b, int q, const AccE *x) {
        const unsigned at = b * C::BLK < cols_in ? o_voff : NOWHERE;
        if (OUT == OUT_I32) {
            v4u v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __builtin_bit_cast(unsigned, x[4 * q + e]);
            __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_out, at, (unsigned)(a * C::BLK * n_out + b * C::BLK + q * 8) * 4, 0);
        } else if (OUT == OUT_F32 && !F8) {
            const v4f y = epi_value(a, b, q, x);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, y), rsrc_out, at,
                                                   (unsigned)(a * C::BLK * n_out + b * C::BLK + q * 8) * 4, 0);
        } else if (OUT == OUT_F32) {
            // A quad is 32 bytes of each of 32 rows; two of them, exchanged between groups of 16 lanes, are 64 bytes of 16 rows
            // each, as the int8 blocks store them (rows a power of two apart lose most by 32-byte pieces: 8127 x 1024, K = 768 26.1
            // -> 16.4 us; 3584 x 8192, K = 256 51.8 -> 35.7).
            if (q & 1) return;
            v4f y0 = epi_value(a, b, q, x), y1 = epi_value(a, b, q + 1, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(y0[e]), __float_as_uint(y1[e]), false, false);
                y0[e] = __uint_as_float(s[0]);
                y1[e] = __uint_as_float(s[1]);
            }
            const unsigned soff = (unsigned)(a * C::BLK * n_out + b * C::BLK + q * 8) * 4;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, y0), rsrc_out, at, soff, 0);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, y1), rsrc_out, at, soff + 16u * n_out * 4, 0);
        } else {
            const v2u pk = __builtin_bit_cast(v2u, __builtin_convertvector(epi_value(a, b, q, x), v4bf));
            const int col = (b * C::BLK) % C::PATCH_COLS + q * 8;
            asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(patch_w), "v"(pk), "n"(col * 2));
        }
    };
    auto epi_read_patch = [&]() {
#pragma unroll
        for (int j = 0; j < C::PATCH_READS; ++j)
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(val[j]) : "v"(patch_r), "n"(j * (64 / PPR) * C::PATCH_PITCH));
    };
    auto epi_store_patch = [&](int a, int col0) {  // after a wait
        const unsigned at = (lane % PPR) * 8 + col0 < cols_in ? o_voff : NOWHERE;
#pragma unroll
        for (int j = 0; j < C::PATCH_READS; ++j) {
            asm volatile("" : "+v"(val[j]));
            __builtin_amdgcn_raw_buffer_store_b128(val[j], rsrc_out, at,
                                                   (unsigned)((a * C::BLK + j * (64 / PPR)) * n_out + col0) * 2, 2);
        }
    };
    constexpr int PATCH_SLOTS = C::PATCH_SLOTS;  // blocks of a patch
    // Stores of an epilogue, per lane, that follow its last request (four-byte int8 results are stored block by block, from the
    // first one on, which has its share of the requests).
    constexpr int STORES = (OUT == OUT_BF16 ? C::WTM * C::WTN / 512 : C::WTM * C::WTN / 256) -
                           (OUT != OUT_BF16 && !F8 ? C::LPW - C::REQ_2ND : 0);

    // The matrix instruction of a block, with its first accumulator and a fragment of either operand; fresh: from zero.
    auto multiply = [](auto fresh, int r0, const Half (&w)[RPF], const Half (&x)[RPF]) __attribute__((always_inline)) {
        if constexpr (F8) {
            const v8i w8 = __builtin_shufflevector(w[0], w[RPF - 1], 0, 1, 2, 3, 4, 5, 6, 7);
            const v8i x8 = __builtin_shufflevector(x[0], x[RPF - 1], 0, 1, 2, 3, 4, 5, 6, 7);
            if constexpr (decltype(fresh)::value)
                asm volatile("v_mfma_f32_32x32x64_f8f6f4 a[%0:%1], %2, %3, 0 cbsz:%4 blgp:%5" ::"n"(r0), "n"(r0 + 15), "v"(w8), "v"(x8), "n"(FMT_W), "n"(FMT_X));
            else
                asm volatile("v_mfma_f32_32x32x64_f8f6f4 a[%0:%1], %2, %3, a[%0:%1] cbsz:%4 blgp:%5" ::"n"(r0), "n"(r0 + 15), "v"(w8), "v"(x8), "n"(FMT_W), "n"(FMT_X));
        } else {
            if constexpr (decltype(fresh)::value)
                asm volatile("v_mfma_i32_16x16x64_i8 a[%0:%1], %2, %3, 0" ::"n"(r0), "n"(r0 + 3), "v"(w[0]), "v"(x[0]));
            else
                asm volatile("v_mfma_i32_16x16x64_i8 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(r0), "n"(r0 + 3), "v"(w[0]), "v"(x[0]));
        }
    };

    // Half a stage: NORMAL; the FIRST of a tile, which starts the accumulators from zero; the same with the epilogue of the
    // tile before; the LAST of the workgroup, with its tile's own epilogue; ONLY: both halves of the one stage of its one tile,
    // with the epilogue.  cur: which half, and its register buffer.
    enum { NORMAL, FIRST, FIRST_EPI, LAST, ONLY };
    auto period = [&](auto cur_c, auto kind_c) __attribute__((always_inline)) {
        constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1, kind = decltype(kind_c)::value;
        constexpr bool own_epi = kind == LAST || kind == ONLY, epi = kind == FIRST_EPI || own_epi;
        constexpr bool more = !own_epi;  // another half stage follows
        // The epilogue of a block in the LAST half stage comes this many instructions after its last one: a result is there
        // 11 (float8: 19) wait states after its instruction, and nobody but these distances sees to it.  With the ONLY stage a
        // block's second instruction comes as far behind its first one.
        constexpr int DIST = F8 ? 2 : 4, LAG = kind == LAST ? DIST : kind == ONLY ? 2 * DIST : 0;
        const int next_slot = !cur ? slot : slot + 1 == S ? 0 : slot + 1, prev_slot = slot == 0 ? S - 1 : slot - 1;
        keep_out_of_agprs();
        if (cur && more) {
            // The next stage has landed.  Behind it are the requests of the STAGES - 2 stages after it and the stores of an
            // epilogue in one of the STAGES - 1 first halves before.
            constexpr int later = (S - 2) * C::LPW, with_stores = later + STORES < 63 ? later + STORES : 63;
            if (slack == 0) {
                wait_vmcnt<later>();
            } else {
                --slack;
                wait_vmcnt<with_stores>();
            }
        }
        wait_lds_reads();
        if (cur && more) block_barrier();
        pin_frags(cur);
        if (kind == ONLY) pin_frags(nxt);
#pragma unroll
        for (int idx = 0; idx < C::SLOTS + LAG; ++idx) {
            constexpr int NACC = F8 ? 16 : 4;
            const int a = idx / NBN, b = !F8 && !epi && (a & 1) ? NBN - 1 - idx % NBN : idx % NBN;
            const int e = idx - LAG, ea = e / NBN, eb = e % NBN;  // block whose epilogue it is
            AccE x[NACC];
            auto read_block = [&]() {
#pragma unroll
                for (int i = 0; i < NACC; ++i) asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x[i]) : "n"(e * NACC + i));
            };
            auto store_patch_before = [&](int behind) {  // its reads have landed, at least `behind` operations are behind them
                if (behind == 3) wait_lgkmcnt<3>(); else if (behind == 2) wait_lgkmcnt<2>(); else wait_lgkmcnt<0>();
                const int last = e / PATCH_SLOTS * PATCH_SLOTS - 1;
                epi_store_patch(last / NBN, last % NBN / PATCH_SLOTS * C::PATCH_COLS);
            };
            if (kind == FIRST_EPI) read_block();
            if (idx < C::SLOTS)
                multiply(std::integral_constant<bool, kind == FIRST || kind == FIRST_EPI || kind == ONLY>(), (a * NBN + b) * NACC,
                         wf[cur][b], xf[cur][a]);
            if (kind == ONLY && idx >= DIST && idx - DIST < C::SLOTS)
                multiply(std::false_type(), (idx - DIST) * NACC, wf[nxt][(idx - DIST) % NBN], xf[nxt][(idx - DIST) / NBN]);
            if constexpr (more) {
                // Fragment reads: the first ones with the fifth int8 instruction, so that all land before the half stage ends.
                constexpr int RD = C::SLOTS / C::NREADS - (BN == 256 ? 1 : 0);
                if constexpr (F8) {
#pragma unroll
                    for (int i = 2 * idx; i < 2 * idx + 2; ++i)
                        if (i < C::NREADS) issue_read(i, nxt, next_slot);
                } else if (idx >= 4 && (idx - 4) % RD == 0 && (idx - 4) / RD < C::NREADS) {
                    issue_read((idx - 4) / RD, nxt, next_slot);
                }
                // Requests.
                constexpr int N2 = C::REQ_2ND, N1 = C::LPW - N2;
                if constexpr (cur == 1) {
                    constexpr int RQ = C::SLOTS / N2;
                    if (idx % RQ == RQ / 2 && idx / RQ < N2) issue_req(slot, idx / RQ);
                } else if constexpr (N1 > 0 && kind != FIRST) {
                    constexpr int RQ = epi ? 1 : C::SLOTS / N1, PER = epi && F8 ? N1 : 1;
#pragma unroll
                    for (int i = idx / RQ * PER; i < (idx / RQ + 1) * PER; ++i)
                        if (idx % RQ == RQ / 2 && i < N1) issue_req(prev_slot, N2 + i);
                }
            }
            if (epi && e >= 0) {
                // A patch is stored after its reads have travelled for a while: behind them are the writes of three int8 blocks,
                // or (float8, right after the matrix instruction) two fragment reads while there are any.
                const bool store = OUT == OUT_BF16 && e >= PATCH_SLOTS && e % PATCH_SLOTS == (F8 ? 0 : 3);
                if (store && F8) store_patch_before(more && 2 * idx + 2 <= C::NREADS ? 2 : 0);
                if (store && !F8) store_patch_before(3);
                if (own_epi) read_block();
#pragma unroll
                for (int q = 0; q < C::QUADS; ++q) epi_quad(ea, eb, q, x);
                if (OUT == OUT_BF16 && (e + 1) % PATCH_SLOTS == 0) epi_read_patch();
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (epi && OUT == OUT_BF16) {
            wait_lds_reads();
            epi_store_patch(NBM - 1, C::WTN - C::PATCH_COLS);
        }
        if (C::REQ_2ND == C::LPW ? cur == 1 && more : cur == 0 && (kind == NORMAL || kind == FIRST_EPI)) advance();
        if (cur) slot = next_slot;
        if (epi) slack = S - 1;
        keep_out_of_agprs();
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, NORMAL> KNormal;
    typedef std::integral_constant<int, FIRST> KFirst;
    typedef std::integral_constant<int, FIRST_EPI> KFirstEpi;
    typedef std::integral_constant<int, LAST> KLast;
    typedef std::integral_constant<int, ONLY> KOnly;

    Tile t = tile_of(0);
    if (!t.have) {
        wait_vmcnt<0>();
        wait_lds_reads();
        return;
    }
    int ring = 0;
    if constexpr (ONE_STAGE) {
#pragma unroll
        for (int i = 0; i < C::NREADS; ++i) issue_read(i, 1, 0);
        epi_begin(t, ring);
        period(I0(), KOnly());
        return;
    }
    period(I0(), KFirst());
    for (int round = 1;; ++round) {
        for (int kt = 1; kt < KT; ++kt) {
            period(I1(), KNormal());
            period(I0(), KNormal());
        }
        const Tile next = tile_of(round);
        if (!next.have) break;
        period(I1(), KNormal());
        epi_begin(t, ring);
        ring = ring + 1 == C::RING ? 0 : ring + 1;
        t = next;
        period(I0(), KFirstEpi());
    }
    epi_begin(t, ring);
    period(I1(), KLast());
    wait_vmcnt<0>();  // the requests past the end write LDS
}

}  // namespace sb
