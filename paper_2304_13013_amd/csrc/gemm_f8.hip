// Host-side dispatch of the 8-bit float GEMM with dequantizing epilogue (the float8 variant of SwitchBack; kernels:
// gemm_i8_wide_kernel.h and gemm_i8_kernel.h with the float8 arithmetic selected).
#include "gemm_i8_direct_kernel.h"
#include "gemm_i8_wide_kernel.h"

#include <atomic>

namespace sb {
namespace {

typedef WideI8Cfg<MATH_F8, false, false> F8Cfg;
// Products with few large tiles, the same line as for the int8 product.
typedef GemmI8Cfg F8Small;

#define SB_GEMM_F8_ENTRY(name, OUT, FW, FX)                                                                \
    __global__ __launch_bounds__(F8Cfg::THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void name(     \
        GemmI8Args p) {                                                                                    \
        gemm_i8_wide_body<OUT, false, MATH_F8 + 2 * FW + FX, false>(p);                                    \
    }                                                                                                      \
    __global__ __launch_bounds__(F8Small::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void name##_s(  \
        GemmI8Args p) {                                                                                    \
        gemm_i8_dequant_body<OUT, false, MATH_F8 + 2 * FW + FX>(p);                                        \
    }
// name suffix: format of the token-side operand a, then of the weight-side operand b (4 = E4M3, 5 = E5M2)
SB_GEMM_F8_ENTRY(gemm_f8_a4b4_bf16, OUT_BF16, 0, 0)
SB_GEMM_F8_ENTRY(gemm_f8_a4b4_f32, OUT_F32, 0, 0)
SB_GEMM_F8_ENTRY(gemm_f8_a5b4_bf16, OUT_BF16, 0, 1)
SB_GEMM_F8_ENTRY(gemm_f8_a5b4_f32, OUT_F32, 0, 1)
SB_GEMM_F8_ENTRY(gemm_f8_a4b5_bf16, OUT_BF16, 1, 0)
SB_GEMM_F8_ENTRY(gemm_f8_a4b5_f32, OUT_F32, 1, 0)
SB_GEMM_F8_ENTRY(gemm_f8_a5b5_bf16, OUT_BF16, 1, 1)
SB_GEMM_F8_ENTRY(gemm_f8_a5b5_f32, OUT_F32, 1, 1)
#undef SB_GEMM_F8_ENTRY

}  // namespace

hipError_t launch_gemm_f8_dequant(const uint8_t *aq, int fmt_a, const float *state_row, const uint8_t *bq, int fmt_b,
                                  const float *state_tensor, int64_t M, int64_t N, int64_t K, void *out,
                                  sb_dtype out_dtype, hipStream_t stream) {
    if (M == 0 || N == 0) return hipSuccess;
    GemmI8Args args{reinterpret_cast<const int8_t *>(aq), reinterpret_cast<const int8_t *>(bq), state_row, state_tensor,
                    nullptr, out, (int)M, (int)N, (int)K, 0, 0, 8, nullptr, nullptr};
    // Tiles, a small product, or tiles and a small product for the last rows, by the rules of the int8 product.
    const int out_bytes = out_dtype == SB_BF16 ? 2 : 4;
    const ProductPlan plan = plan_product(M, N, K, PRODUCT_F8, out_bytes, num_compute_units());
    const GemmI8Args rest = rows_from(args, plan.tile_rows, out_bytes);
    if (plan.tile_rows == 0) return launch_gemm_f8_direct(plan.split, rest, fmt_a, fmt_b, out_dtype, stream);
    typedef void (*Kernel)(GemmI8Args);
    static const Kernel kernels[16] = {
        gemm_f8_a4b4_bf16, gemm_f8_a4b4_f32, gemm_f8_a5b4_bf16, gemm_f8_a5b4_f32, gemm_f8_a4b5_bf16, gemm_f8_a4b5_f32,
        gemm_f8_a5b5_bf16, gemm_f8_a5b5_f32, gemm_f8_a4b4_bf16_s, gemm_f8_a4b4_f32_s, gemm_f8_a5b4_bf16_s,
        gemm_f8_a5b4_f32_s, gemm_f8_a4b5_bf16_s, gemm_f8_a4b5_f32_s, gemm_f8_a5b5_bf16_s, gemm_f8_a5b5_f32_s};
    static std::atomic<bool> attr_set[16];  // zero-initialized; a racing second set is harmless
    const bool small = few_tiles(M, N, num_compute_units());
    const int which = (small ? 8 : 0) + (fmt_b ? 4 : 0) + (fmt_a ? 2 : 0) + (out_dtype == SB_BF16 ? 0 : 1);
    const int lds = small ? F8Small::LDS_BYTES : F8Cfg::LDS_BYTES;
    if (!attr_set[which].load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernels[which]),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set[which].store(true, std::memory_order_release);
    }
    int grid = 0;
    args.M = (int)plan.tile_rows;
    if (small) {
        gemm_i8_prepare<F8Small>(args, 2 * num_compute_units(), &grid);
        kernels[which]<<<grid, F8Small::THREADS, lds, stream>>>(args);
    } else {
        gemm_i8_prepare<F8Cfg>(args, num_compute_units(), &grid);
        kernels[which]<<<grid, F8Cfg::THREADS, lds, stream>>>(args);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || plan.split == DIRECT_NONE) return e;
    return launch_gemm_f8_direct(plan.split, rest, fmt_a, fmt_b, out_dtype, stream);
}

}  // namespace sb
