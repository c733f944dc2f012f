// Host-side dispatch of the bf16 weight-gradient GEMM (kernel: gemm_bf16_tn_kernel.h) and its split-K reduction.
#include "gemm_bf16_tn_wide_kernel.h"

#include <atomic>

namespace sb {
namespace {

typedef WideCfg Big;       // 256 x 256 tiles, four waves of 128 x 128
typedef GemmBf16Cfg Small;  // 128 x 128 tiles, two workgroups per compute unit
static_assert(Big::UNIT == DW_STAGE && Small::BKT == DW_STAGE, "token ranges are whole stages of either");

// One wave per SIMD: all 512 registers are a lane's.
__global__ __launch_bounds__(Big::THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_tn_kernel(
    GemmBf16Args p) {
    gemm_bf16_tn_wide_body(p);
}
__global__ __launch_bounds__(Small::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void gemm_bf16_tn_small_kernel(
    GemmBf16Args p) {
    gemm_bf16_tn_body<false>(p);
}

// One item per tile, its token range summed in pieces (WeightGradPlan).
__global__ __launch_bounds__(Small::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void gemm_bf16_tn_small_fold_kernel(
    GemmBf16Args p) {
    gemm_bf16_tn_body<true>(p);
}

// out[e] = sum over splits (ascending) of partial[s][e]; four elements per thread, eight splits' loads in flight.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const v4f *__restrict__ partial, int64_t quads,
                                                            int splits, void *__restrict__ out, int out_bf16) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= quads) return;
    v4f s = partial[i];
    int k = 1;
    for (; k + 8 <= splits; k += 8) {
        v4f v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = partial[(int64_t)(k + j) * quads + i];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; k < splits; ++k) s += partial[(int64_t)k * quads + i];
    if (out_bf16)
        static_cast<v4bf *>(out)[i] = __builtin_convertvector(s, v4bf);
    else
        static_cast<v4f *>(out)[i] = s;
}

template <class C>
hipError_t set_lds_limit_once(void (*kernel)(GemmBf16Args), std::atomic<bool> &done) {
    if (done.load(std::memory_order_acquire)) return hipSuccess;  // a second set by a racing host thread is harmless
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if (e == hipSuccess) done.store(true, std::memory_order_release);
    return e;
}

}  // namespace

// The plan is a function of the shape alone, so the workspace query and the launch agree.
WeightGradPlan plan_gemm_bf16_tn(int64_t b, int64_t n, int64_t m) {
    return plan_weight_gradient(b, n, m, num_compute_units());
}

size_t gemm_bf16_tn_workspace_bytes(const WeightGradPlan &plan, int64_t n, int64_t m) {
    return plan.splits > 1 ? (size_t)plan.splits * (size_t)m * (size_t)n * sizeof(float) : 0;
}

hipError_t launch_gemm_bf16_tn(const WeightGradPlan &plan, const void *dy, const void *x, int64_t b, int64_t n, int64_t m, void *dw,
                               sb_dtype dw_dtype, void *ws, hipStream_t stream) {
    static std::atomic<bool> big_set{false}, small_set{false}, fold_set{false};
    hipError_t e = plan.pieces > 1 ? set_lds_limit_once<Small>(gemm_bf16_tn_small_fold_kernel, fold_set)
                   : plan.small    ? set_lds_limit_once<Small>(gemm_bf16_tn_small_kernel, small_set)
                                   : set_lds_limit_once<Big>(gemm_bf16_tn_kernel, big_set);
    if (e != hipSuccess) return e;
    GemmBf16Args a;
    a.dy = static_cast<const unsigned short *>(dy);
    a.x = static_cast<const unsigned short *>(x);
    a.b = (int)b;
    a.n = (int)n;
    a.m = (int)m;
    const int side = plan.small ? 128 : 256;
    a.tiles_m = (int)((m + side - 1) / side);
    a.tiles_n = (int)((n + side - 1) / side);
    a.splits = plan.splits;
    a.k_per_split = plan.stages_per_split * DW_STAGE;
    a.k_per_piece = plan.stages_per_piece * DW_STAGE;
    a.partial = static_cast<float *>(ws);
    a.out = dw;
    a.out_bf16 = dw_dtype == SB_BF16;
    // Persistent grid: at most as many workgroups as the GPU holds at once, the same number on every XCD.
    const int total = a.tiles_m * a.tiles_n * a.splits;
    const int per_xcd = (total + 7) / 8, cus_per_xcd = num_compute_units() / 8 > 0 ? num_compute_units() / 8 : 1;
    const int slots_per_xcd = cus_per_xcd * (plan.small ? 2 : 1);
    const int grid = 8 * (per_xcd < slots_per_xcd ? per_xcd : slots_per_xcd);
    if (plan.pieces > 1)
        gemm_bf16_tn_small_fold_kernel<<<grid, Small::THREADS, Small::LDS_BYTES, stream>>>(a);
    else if (plan.small)
        gemm_bf16_tn_small_kernel<<<grid, Small::THREADS, Small::LDS_BYTES, stream>>>(a);
    else
        gemm_bf16_tn_kernel<<<grid, Big::THREADS, Big::LDS_BYTES, stream>>>(a);
    e = hipGetLastError();
    if (e != hipSuccess || a.splits == 1) return e;
    const int64_t quads = m * n / 4;
    splitk_reduce_kernel<<<(unsigned int)((quads + 255) / 256), 256, 0, stream>>>(
        static_cast<const v4f *>(ws), quads, a.splits, dw, a.out_bf16);
    return hipGetLastError();
}

}  // namespace sb
