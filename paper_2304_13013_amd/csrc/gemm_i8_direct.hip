// Host-side dispatch of the small-product kernel (gemm_i8_direct_kernel.h): int8 and 8-bit float codes, every epilogue.
#include "gemm_i8_direct_kernel.h"

#include <atomic>

namespace sb {
namespace {

// The three splits of the work.  D32: 32x32 blocks, four waves, two workgroups per compute unit.  D64: 64x64 blocks, four
// waves, one workgroup per compute unit: half the operand bytes, for outputs of more than a few hundred 32x32 blocks.
// D64H: 64x64 blocks, two waves, two workgroups per compute unit: when there are more 64x64 blocks than compute units.
typedef DirectCfg<32, 32, 4> D32;
typedef DirectCfg<64, 64, 4> D64;
typedef DirectCfg<64, 64, 2> D64H;

template <class C>
hipError_t launch_direct(void (*kernel)(GemmI8Args), std::atomic<bool> *attr_set, GemmI8Args a, hipStream_t stream) {
    if (!attr_set->load(std::memory_order_acquire)) {  // setting it twice (two host threads racing) is harmless
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set->store(true, std::memory_order_release);
    }
    a.tiles_m = (a.M + C::ROWS - 1) / C::ROWS;
    a.tiles_n = a.N / C::COLS;
    kernel<<<a.tiles_m * a.tiles_n, C::THREADS, C::LDS_BYTES, stream>>>(a);
    return hipGetLastError();
}

#define SB_DIRECT_ENTRY(name, CFG, OUT, COLSCALE, MATH, POST)                \
    __global__ __launch_bounds__(CFG::THREADS) void name(GemmI8Args p) {     \
        gemm_i8_direct_body<CFG, OUT, COLSCALE, MATH, POST>(p);              \
    }
// One launcher per epilogue and arithmetic; it picks the split.
#define SB_DIRECT(name, OUT, COLSCALE, MATH, POST)                                                               \
    SB_DIRECT_ENTRY(name##_d32, D32, OUT, COLSCALE, MATH, POST)                                                  \
    SB_DIRECT_ENTRY(name##_d64, D64, OUT, COLSCALE, MATH, POST)                                                  \
    SB_DIRECT_ENTRY(name##_d64h, D64H, OUT, COLSCALE, MATH, POST)                                                \
    hipError_t name(int split, const GemmI8Args &a, hipStream_t stream) {                                        \
        static std::atomic<bool> attr_set[3];                                                                    \
        if (split == DIRECT_32) return launch_direct<D32>(name##_d32, &attr_set[0], a, stream);                  \
        if (split == DIRECT_64) return launch_direct<D64>(name##_d64, &attr_set[1], a, stream);                  \
        return launch_direct<D64H>(name##_d64h, &attr_set[2], a, stream);                                        \
    }
SB_DIRECT(gemm_i8d_bf16, OUT_BF16, false, MATH_I8, false)
SB_DIRECT(gemm_i8d_f32, OUT_F32, false, MATH_I8, false)
SB_DIRECT(gemm_i8d_i32, OUT_I32, false, MATH_I8, false)
SB_DIRECT(gemm_i8dq_bf16, OUT_BF16, true, MATH_I8, false)
SB_DIRECT(gemm_i8dq_f32, OUT_F32, true, MATH_I8, false)
SB_DIRECT(gemm_i8dp_bf16, OUT_BF16, false, MATH_I8, true)
SB_DIRECT(gemm_i8dp_f32, OUT_F32, false, MATH_I8, true)
// a: format of the token-side operand, b: of the weight-side operand (4 = E4M3, 5 = E5M2)
SB_DIRECT(gemm_f8d_a4b4_bf16, OUT_BF16, false, MATH_F8 + 0, false)
SB_DIRECT(gemm_f8d_a4b4_f32, OUT_F32, false, MATH_F8 + 0, false)
SB_DIRECT(gemm_f8d_a5b4_bf16, OUT_BF16, false, MATH_F8 + 1, false)
SB_DIRECT(gemm_f8d_a5b4_f32, OUT_F32, false, MATH_F8 + 1, false)
SB_DIRECT(gemm_f8d_a4b5_bf16, OUT_BF16, false, MATH_F8 + 2, false)
SB_DIRECT(gemm_f8d_a4b5_f32, OUT_F32, false, MATH_F8 + 2, false)
SB_DIRECT(gemm_f8d_a5b5_bf16, OUT_BF16, false, MATH_F8 + 3, false)
SB_DIRECT(gemm_f8d_a5b5_f32, OUT_F32, false, MATH_F8 + 3, false)
#undef SB_DIRECT
#undef SB_DIRECT_ENTRY

}  // namespace

hipError_t launch_gemm_i8_direct(int split, const GemmI8Args &a, bool post, sb_dtype out_dtype, hipStream_t stream) {
    const bool bf = out_dtype == SB_BF16;
    if (out_dtype == SB_I32_RAW) return gemm_i8d_i32(split, a, stream);
    if (a.state_col != nullptr) return bf ? gemm_i8dq_bf16(split, a, stream) : gemm_i8dq_f32(split, a, stream);
    if (post) return bf ? gemm_i8dp_bf16(split, a, stream) : gemm_i8dp_f32(split, a, stream);
    return bf ? gemm_i8d_bf16(split, a, stream) : gemm_i8d_f32(split, a, stream);
}

hipError_t launch_gemm_f8_direct(int split, const GemmI8Args &a, int fmt_a, int fmt_b, sb_dtype out_dtype,
                                 hipStream_t stream) {
    const bool bf = out_dtype == SB_BF16;
    if (fmt_b)
        return fmt_a ? (bf ? gemm_f8d_a5b5_bf16(split, a, stream) : gemm_f8d_a5b5_f32(split, a, stream))
                     : (bf ? gemm_f8d_a4b5_bf16(split, a, stream) : gemm_f8d_a4b5_f32(split, a, stream));
    return fmt_a ? (bf ? gemm_f8d_a5b4_bf16(split, a, stream) : gemm_f8d_a5b4_f32(split, a, stream))
                 : (bf ? gemm_f8d_a4b4_bf16(split, a, stream) : gemm_f8d_a4b4_f32(split, a, stream));
}

}  // namespace sb
