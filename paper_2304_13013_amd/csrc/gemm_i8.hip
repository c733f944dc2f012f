// Host-side dispatch of the int8 GEMM with dequantizing epilogue (kernels: gemm_i8_wide_kernel.h for 256x256 and 256x128 tiles,
// gemm_i8_kernel.h for 128x128 ones, gemm_i8_direct_kernel.h for small products and last rows; dispatch.h picks).
#include "gemm_i8_direct_kernel.h"
#include "gemm_i8_wide_kernel.h"

#include <atomic>

namespace sb {
namespace {

template <class C>
hipError_t launch(void (*kernel)(GemmI8Args), std::atomic<bool> *attr_set, GemmI8Args args, hipStream_t stream) {
    if (!attr_set->load(std::memory_order_acquire)) {  // setting it twice (two host threads racing) is harmless
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set->store(true, std::memory_order_release);
    }
    int grid = 0;
    // Workgroups that fit a compute unit at once: its 160 KiB of LDS decide (the 128x128 tile's registers allow two).
    constexpr int per_cu = C::LDS_BYTES * 2 <= 160 * 1024 ? 2 : 1;
    gemm_i8_prepare<C>(args, num_compute_units() * per_cu, &grid);
    kernel<<<grid, C::THREADS, C::LDS_BYTES, stream>>>(args);
    return hipGetLastError();
}

// The kernels of a form on 256x256 (_w; _w1: one stage and one tile per workgroup) and 256x128 tiles (_w128) and their launcher.
// One wave per SIMD: all 512 registers are a lane's.
#define SB_WIDE_KERNEL(name, OUT, COLSCALE, POST, BN, ONE_STAGE)                          \
    __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void name( \
        GemmI8Args p) {                                                                   \
        gemm_i8_wide_body<OUT, COLSCALE, MATH_I8, POST, BN, ONE_STAGE>(p);                \
    }
#define SB_WIDE(name, OUT, COLSCALE, POST)                                                \
    SB_WIDE_KERNEL(name##_w, OUT, COLSCALE, POST, 256, false)                             \
    SB_WIDE_KERNEL(name##_w1, OUT, COLSCALE, POST, 256, true)                             \
    SB_WIDE_KERNEL(name##_w128, OUT, COLSCALE, POST, 128, false)                          \
    hipError_t name(bool narrow, const GemmI8Args &args, hipStream_t stream) {            \
        typedef WideI8Cfg<MATH_I8, COLSCALE, POST, 256> C;                                \
        typedef WideI8Cfg<MATH_I8, COLSCALE, POST, 128> C128;                             \
        static std::atomic<bool> attr_set[3]; /* zero-initialized */                      \
        if (narrow) return launch<C128>(name##_w128, &attr_set[0], args, stream);         \
        if (one_stage(args.M, args.N, args.K, num_compute_units()))                       \
            return launch<C>(name##_w1, &attr_set[1], args, stream);                      \
        return launch<C>(name##_w, &attr_set[2], args, stream);                           \
    }
// A small-tile instance: K a multiple of 128 (_k) and K = 64 mod 128 (_h).  Two waves per SIMD (two workgroups per compute
// unit): at most 256 registers a lane.
#define SB_SMALL_KERNEL(name, OUT, COLSCALE, POST, HALF)                                  \
    __global__ __launch_bounds__(GemmI8Cfg::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void name( \
        GemmI8Args p) {                                                                   \
        gemm_i8_dequant_body<OUT, COLSCALE, MATH_I8, POST, HALF>(p);                      \
    }
#define SB_SMALL(name, OUT, COLSCALE, POST)                                               \
    SB_SMALL_KERNEL(name##_k, OUT, COLSCALE, POST, false)                                 \
    SB_SMALL_KERNEL(name##_h, OUT, COLSCALE, POST, true)                                  \
    hipError_t name(const GemmI8Args &args, hipStream_t stream) {                         \
        static std::atomic<bool> attr_set[2]; /* zero-initialized */                      \
        if (args.K % 128) return launch<GemmI8Cfg>(name##_h, &attr_set[0], args, stream); \
        return launch<GemmI8Cfg>(name##_k, &attr_set[1], args, stream);                   \
    }
SB_WIDE(gemm_i8_k128_bf16, OUT_BF16, false, false)
SB_WIDE(gemm_i8_k128_f32, OUT_F32, false, false)
SB_WIDE(gemm_i8_k128_i32, OUT_I32, false, false)
SB_WIDE(gemm_i8q_k128_bf16, OUT_BF16, true, false)
SB_WIDE(gemm_i8q_k128_f32, OUT_F32, true, false)
SB_WIDE(gemm_i8p_k128_bf16, OUT_BF16, false, true)
SB_WIDE(gemm_i8p_k128_f32, OUT_F32, false, true)
SB_SMALL(gemm_i8_k128s_bf16, OUT_BF16, false, false)
SB_SMALL(gemm_i8_k128s_f32, OUT_F32, false, false)
SB_SMALL(gemm_i8_k128s_i32, OUT_I32, false, false)
SB_SMALL(gemm_i8q_k128s_bf16, OUT_BF16, true, false)
SB_SMALL(gemm_i8q_k128s_f32, OUT_F32, true, false)
SB_SMALL(gemm_i8p_k128s_bf16, OUT_BF16, false, true)
SB_SMALL(gemm_i8p_k128s_f32, OUT_F32, false, true)
#undef SB_SMALL
#undef SB_SMALL_KERNEL
#undef SB_WIDE
#undef SB_WIDE_KERNEL

}  // namespace

// Compute units of the current device (queried once per process; the library serves one GPU).  Host threads may race
// to the first query: both store the same value.
int num_compute_units() {
    static std::atomic<int> cached{0};
    int n = cached.load(std::memory_order_relaxed);
    if (n == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            n = prop.multiProcessorCount;
        if (n <= 0) n = 256;  // no device visible (host-only callers sizing a workspace): an MI355X has 256
        cached.store(n, std::memory_order_relaxed);
    }
    return n;
}

GemmI8Args rows_of(const GemmI8Args &a, int64_t first, int64_t end, size_t out_bytes) {
    GemmI8Args r = a;
    r.a += (size_t)first * (size_t)a.K;
    if (r.state_row != nullptr) r.state_row += first;
    r.out = static_cast<char *>(a.out) + (size_t)first * (size_t)a.N * out_bytes;
    r.M = (int)(end - first);
    return r;
}

// The tiled kernels' instances.
static hipError_t launch_tiled(TileKind tile, const GemmI8Args &args, bool post, sb_dtype out_dtype, hipStream_t stream) {
    const bool small = tile == TILES_128, narrow = tile == TILES_256X128, bf = out_dtype == SB_BF16;
    if (post)
        return small ? (bf ? gemm_i8p_k128s_bf16(args, stream) : gemm_i8p_k128s_f32(args, stream))
                     : (bf ? gemm_i8p_k128_bf16(narrow, args, stream) : gemm_i8p_k128_f32(narrow, args, stream));
    if (args.state_col != nullptr && out_dtype != SB_I32_RAW)
        return small ? (bf ? gemm_i8q_k128s_bf16(args, stream) : gemm_i8q_k128s_f32(args, stream))
                     : (bf ? gemm_i8q_k128_bf16(narrow, args, stream) : gemm_i8q_k128_f32(narrow, args, stream));
    switch (out_dtype) {
        case SB_BF16: return small ? gemm_i8_k128s_bf16(args, stream) : gemm_i8_k128_bf16(narrow, args, stream);
        case SB_F32: return small ? gemm_i8_k128s_f32(args, stream) : gemm_i8_k128_f32(narrow, args, stream);
        default: return small ? gemm_i8_k128s_i32(args, stream) : gemm_i8_k128_i32(narrow, args, stream);
    }
}

static hipError_t launch_product(const GemmI8Args &args, bool post, sb_dtype out_dtype, hipStream_t stream) {
    const int out_bytes = out_dtype == SB_BF16 ? 2 : 4;
    const ProductKind kind = post || args.state_col != nullptr ? PRODUCT_LONG_EPILOGUE : PRODUCT_PLAIN;
    const ProductPlan plan = plan_product(args.M, args.N, args.K, kind, out_bytes, num_compute_units());
    if (plan.first_rows > 0) {
        const hipError_t e = launch_tiled(TILES_256, rows_of(args, 0, plan.first_rows, out_bytes), post, out_dtype, stream);
        if (e != hipSuccess) return e;
    }
    if (plan.tile_rows > plan.first_rows) {
        const hipError_t e = launch_tiled(plan.rest, rows_of(args, plan.first_rows, plan.tile_rows, out_bytes), post,
                                          out_dtype, stream);
        if (e != hipSuccess) return e;
    }
    if (plan.split == DIRECT_NONE) return hipSuccess;
    return launch_gemm_i8_direct(plan.split, rows_of(args, plan.tile_rows, args.M, out_bytes), post, out_dtype, stream);
}

hipError_t launch_gemm_i8_dequant_post(const int8_t *aq, const float *state_row, const int8_t *bq,
                                       const float *state_tensor, const float *bias, const float *gamma, int64_t M,
                                       int64_t N, int64_t K, void *out, sb_dtype out_dtype, hipStream_t stream) {
    if (M == 0 || N == 0) return hipSuccess;
    return launch_product(GemmI8Args{aq, bq, state_row, state_tensor, nullptr, out, (int)M, (int)N, (int)K, 0, 0, 8, bias,
                                     gamma}, true, out_dtype, stream);
}

hipError_t launch_gemm_i8_dequant(const int8_t *aq, const float *state_row, const int8_t *bq,
                                  const float *state_tensor, const float *state_col, int64_t M, int64_t N,
                                  int64_t K, void *out, sb_dtype out_dtype, hipStream_t stream) {
    if (M == 0 || N == 0) return hipSuccess;
    return launch_product(GemmI8Args{aq, bq, state_row, state_tensor, state_col, out, (int)M, (int)N, (int)K, 0, 0, 8,
                                     nullptr, nullptr}, false, out_dtype, stream);
}

}  // namespace sb
