// Host-side dispatch of the 8-bit float GEMM with dequantizing epilogue (the float8 variant of SwitchBack; kernels:
// gemm_i8_wide_kernel.h, gemm_i8_kernel.h and gemm_i8_direct_kernel.h with the float8 arithmetic selected; dispatch.h picks).
#include "gemm_i8_direct_kernel.h"
#include "gemm_i8_wide_kernel.h"

#include <atomic>

namespace sb {
namespace {

typedef WideI8Cfg<MATH_F8, false, false> F8Cfg;
typedef WideI8Cfg<MATH_F8, false, false, 128> F8Narrow;
typedef GemmI8Cfg F8Small;

#define SB_GEMM_F8_ENTRY(name, OUT, FW, FX)                                                                \
    __global__ __launch_bounds__(F8Cfg::THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void name(     \
        GemmI8Args p) {                                                                                    \
        gemm_i8_wide_body<OUT, false, MATH_F8 + 2 * FW + FX, false>(p);                                    \
    }                                                                                                      \
    __global__ __launch_bounds__(F8Cfg::THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void name##_1( \
        GemmI8Args p) {                                                                                    \
        gemm_i8_wide_body<OUT, false, MATH_F8 + 2 * FW + FX, false, 256, true>(p);                         \
    }                                                                                                      \
    __global__ __launch_bounds__(F8Narrow::THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void name##_n( \
        GemmI8Args p) {                                                                                    \
        gemm_i8_wide_body<OUT, false, MATH_F8 + 2 * FW + FX, false, 128>(p);                               \
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

// The instance for a tile (256x256 ones: with or without further stages), a pair of formats and an output type (`which`, in the
// order of the entries above).
hipError_t launch_tiled(TileKind tile, int which, GemmI8Args args, hipStream_t stream) {
    typedef void (*Kernel)(GemmI8Args);
    static const Kernel kernels[TILE_KINDS + 1][8] = {
        {gemm_f8_a4b4_bf16_s, gemm_f8_a4b4_f32_s, gemm_f8_a5b4_bf16_s, gemm_f8_a5b4_f32_s, gemm_f8_a4b5_bf16_s,
         gemm_f8_a4b5_f32_s, gemm_f8_a5b5_bf16_s, gemm_f8_a5b5_f32_s},
        {gemm_f8_a4b4_bf16_n, gemm_f8_a4b4_f32_n, gemm_f8_a5b4_bf16_n, gemm_f8_a5b4_f32_n, gemm_f8_a4b5_bf16_n,
         gemm_f8_a4b5_f32_n, gemm_f8_a5b5_bf16_n, gemm_f8_a5b5_f32_n},
        {gemm_f8_a4b4_bf16, gemm_f8_a4b4_f32, gemm_f8_a5b4_bf16, gemm_f8_a5b4_f32, gemm_f8_a4b5_bf16, gemm_f8_a4b5_f32,
         gemm_f8_a5b5_bf16, gemm_f8_a5b5_f32},
        {gemm_f8_a4b4_bf16_1, gemm_f8_a4b4_f32_1, gemm_f8_a5b4_bf16_1, gemm_f8_a5b4_f32_1, gemm_f8_a4b5_bf16_1,
         gemm_f8_a4b5_f32_1, gemm_f8_a5b5_bf16_1, gemm_f8_a5b5_f32_1}};
    static std::atomic<bool> attr_set[TILE_KINDS + 1][8];  // zero-initialized; a racing second set is harmless
    const int row = tile == TILES_256 && one_stage(args.M, args.N, args.K, num_compute_units()) ? (int)TILE_KINDS : (int)tile;
    const Kernel kernel = kernels[row][which];
    int grid = 0, threads = 0, lds = 0;
    auto shape = [&](auto config, int per_cu) {
        typedef decltype(config) C;
        gemm_i8_prepare<C>(args, per_cu * num_compute_units(), &grid);
        threads = C::THREADS;
        lds = C::LDS_BYTES;
    };
    if (tile == TILES_128)
        shape(F8Small(), 2);
    else if (tile == TILES_256X128)
        shape(F8Narrow(), 1);
    else
        shape(F8Cfg(), 1);
    if (!attr_set[row][which].load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set[row][which].store(true, std::memory_order_release);
    }
    kernel<<<grid, threads, lds, stream>>>(args);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f8_dequant(const uint8_t *aq, int fmt_a, const float *state_row, const uint8_t *bq, int fmt_b,
                                  const float *state_tensor, int64_t M, int64_t N, int64_t K, void *out,
                                  sb_dtype out_dtype, hipStream_t stream) {
    if (M == 0 || N == 0) return hipSuccess;
    GemmI8Args args{reinterpret_cast<const int8_t *>(aq), reinterpret_cast<const int8_t *>(bq), state_row, state_tensor,
                    nullptr, out, (int)M, (int)N, (int)K, 0, 0, 8, nullptr, nullptr};
    const int out_bytes = out_dtype == SB_BF16 ? 2 : 4;
    const ProductPlan plan = plan_product(M, N, K, PRODUCT_F8, out_bytes, num_compute_units());
    const int which = (fmt_b ? 4 : 0) + (fmt_a ? 2 : 0) + (out_dtype == SB_BF16 ? 0 : 1);
    if (plan.first_rows > 0) {
        const hipError_t e = launch_tiled(TILES_256, which, rows_of(args, 0, plan.first_rows, out_bytes), stream);
        if (e != hipSuccess) return e;
    }
    if (plan.tile_rows > plan.first_rows) {
        const hipError_t e =
            launch_tiled(plan.rest, which, rows_of(args, plan.first_rows, plan.tile_rows, out_bytes), stream);
        if (e != hipSuccess) return e;
    }
    if (plan.split == DIRECT_NONE) return hipSuccess;
    return launch_gemm_f8_direct(plan.split, rows_of(args, plan.tile_rows, M, out_bytes), fmt_a, fmt_b, out_dtype, stream);
}

}  // namespace sb
