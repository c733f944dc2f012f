// Measured ceilings of the GPU the library runs on: what the matrix pipes and the memory system deliver to code that
// does nothing else, so that the fraction of the published peak a product kernel reaches can be read against what the
// chip sustains.  Measurement aids only (include/switchback_ceilings.h); no step of the layer runs through them.
//
//   * matrix-instruction loops: the instructions, the block walk and the register fragments of the four-wave product kernels
//     (gemm_i8_wide_kernel.h, gemm_bf16_tn_wide_kernel.h): one wave per SIMD with a 128x128 tile, both of its fragment
//     buffers, every (fragment, fragment) product of a buffer in the kernels' order, over and over.  No LDS, no memory traffic
//     inside the loop.  The fragments are read once from caller-supplied code buffers, so the same loop can run on all-zero
//     operands, on uniform random codes and on the codes the quantizers of this library produce from a workload: the matrix
//     pipes draw power according to how many operand bits toggle, and the clock the GPU holds depends on it.
//   * a plain copy: 16 bytes per lane, grid-stride, read once and written once.
#include "sb_common.h"

#include <type_traits>

namespace sb {
namespace {

enum { CEIL_I8 = 0, CEIL_BF16 = 1, CEIL_F8 = 2 };

constexpr int kBufs = 2, kWaves = 4;  // fragment buffers; waves of a workgroup, one per SIMD

// The instructions are asm, so that their accumulators stay where they are (as values of the builtins they are copied).
// FRAGS: fragments per buffer and operand, blocks of a side of the wave tile.  OPS: operations of an instruction.
template <int KIND>
struct CeilTraits;
template <>
struct CeilTraits<CEIL_I8> {
    typedef v4i Frag;
    typedef v4i Acc;
    static constexpr int FRAGS = 8, OPS = 2 * 16 * 16 * 64;
    static __device__ __forceinline__ void mma(Frag b, Frag a, Acc &c) {
        asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(c) : "v"(b), "v"(a));
    }
};
template <>
struct CeilTraits<CEIL_BF16> {
    typedef v8bf Frag;
    typedef v4f Acc;
    static constexpr int FRAGS = 8, OPS = 2 * 16 * 16 * 32;
    static __device__ __forceinline__ void mma(Frag b, Frag a, Acc &c) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(b), "v"(a));
    }
};
template <>
struct CeilTraits<CEIL_F8> {
    typedef v8i Frag;
    typedef v16f Acc;
    static constexpr int FRAGS = 4, OPS = 2 * 32 * 32 * 64;
    static __device__ __forceinline__ void mma(Frag b, Frag a, Acc &c) {  // E4M3 x E4M3
        asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, %0 cbsz:0 blgp:0" : "+a"(c) : "v"(b), "v"(a));
    }
};

// a, b: operand bytes; wave w of the grid takes its fragment f of either operand at byte (w * kBufs * FRAGS + f) * 64 *
// sizeof(Frag) modulo the buffer's length (a_bytes, b_bytes: multiples of 64 * sizeof(Frag)).  sink receives one value per
// lane so that the accumulators stay live.
template <int KIND>
__device__ __forceinline__ void mfma_loop_body(const unsigned char *a, size_t a_bytes, const unsigned char *b,
                                               size_t b_bytes, int iters, float *sink) {
    typedef CeilTraits<KIND> T;
    typedef typename T::Frag Frag;
    typedef typename T::Acc Acc;
    constexpr int FRAGS = T::FRAGS, REGS = sizeof(Acc) / 4;
    const int lane = threadIdx.x & 63;
    const size_t wave = (size_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr size_t kWaveFrag = 64 * sizeof(Frag);
    size_t at_a = wave * (kBufs * FRAGS * kWaveFrag) % a_bytes, at_b = wave * (kBufs * FRAGS * kWaveFrag) % b_bytes;
    Frag fa[kBufs][FRAGS], fb[kBufs][FRAGS];
#pragma unroll
    for (int u = 0; u < kBufs; ++u)
#pragma unroll
        for (int i = 0; i < FRAGS; ++i) {
            fa[u][i] = *reinterpret_cast<const Frag *>(a + at_a + lane * sizeof(Frag));
            fb[u][i] = *reinterpret_cast<const Frag *>(b + at_b + lane * sizeof(Frag));
            at_a = at_a + kWaveFrag == a_bytes ? 0 : at_a + kWaveFrag;
            at_b = at_b + kWaveFrag == b_bytes ? 0 : at_b + kWaveFrag;
        }
    Acc acc[FRAGS][FRAGS] = {};
    for (int it = 0; it < iters; ++it) {
        asm volatile("s_nop 3");  // the compiler knows of no matrix instruction in the asm, and wrote its operands just now
#pragma unroll
        for (int u = 0; u < kBufs; ++u)
#pragma unroll
            for (int i = 0; i < FRAGS; ++i)
#pragma unroll
                for (int k = 0; k < FRAGS; ++k) {
                    const int j = FRAGS == 8 && (i & 1) ? FRAGS - 1 - k : k;  // 16-row blocks: to and fro
                    T::mma(fb[u][j], fa[u][i], acc[i][j]);
                }
    }
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");  // nor of the last results, which need up to 18 wait states
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < FRAGS; ++i)
#pragma unroll
        for (int j = 0; j < FRAGS; ++j)
#pragma unroll
            for (int r = 0; r < REGS; ++r) {
                typename std::remove_reference<decltype(acc[0][0][0])>::type x;
                asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[i][j][r]));
                s += (float)x;
            }
    sink[wave * 64 + lane] = s;
}

#define SB_CEILING_KERNEL(name, KIND)                                                                                     \
    __global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(1, 1))) void name(                       \
        const unsigned char *a, size_t a_bytes, const unsigned char *b, size_t b_bytes, int iters, float *sink) {         \
        mfma_loop_body<KIND>(a, a_bytes, b, b_bytes, iters, sink);                                                        \
    }
SB_CEILING_KERNEL(ceiling_mfma_i8_kernel, CEIL_I8)
SB_CEILING_KERNEL(ceiling_mfma_bf16_kernel, CEIL_BF16)
SB_CEILING_KERNEL(ceiling_mfma_f8_kernel, CEIL_F8)
#undef SB_CEILING_KERNEL

__global__ __launch_bounds__(256) void ceiling_copy_kernel(const v4u *__restrict__ src, v4u *__restrict__ dst,
                                                           size_t chunks) {
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < chunks; i += stride)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace
}  // namespace sb

extern "C" {

int switchback_ceiling_mfma(int kind, const void *a_codes, size_t a_bytes, const void *b_codes, size_t b_bytes,
                            int workgroups, int waves_per_workgroup, int iters, float *sink, double *ops_out,
                            void *stream) {
    using namespace sb;
    if (kind < CEIL_I8 || kind > CEIL_F8 || workgroups <= 0 || iters <= 0) return SB_INVALID_ARG;
    if (waves_per_workgroup != 4 && waves_per_workgroup != 8) return SB_INVALID_ARG;
    const size_t frag = kind == CEIL_F8 ? 32 * 64 : 16 * 64;  // bytes one wave reads per fragment
    if (a_codes == nullptr || b_codes == nullptr || sink == nullptr || !aligned16(a_codes) || !aligned16(b_codes))
        return SB_INVALID_ARG;
    if (a_bytes < frag || b_bytes < frag || a_bytes % frag || b_bytes % frag) return SB_INVALID_ARG;
    const unsigned char *a = static_cast<const unsigned char *>(a_codes), *b = static_cast<const unsigned char *>(b_codes);
    // Waves come in workgroups of four, one per SIMD: a lane's fragments and accumulators leave no room for a second one.
    if ((int64_t)workgroups * waves_per_workgroup / kWaves > (int64_t)1 << 30) return SB_INVALID_ARG;
    const dim3 grid((unsigned)workgroups * (unsigned)waves_per_workgroup / kWaves), block(kWaves * 64);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (kind == CEIL_I8)
        ceiling_mfma_i8_kernel<<<grid, block, 0, s>>>(a, a_bytes, b, b_bytes, iters, sink);
    else if (kind == CEIL_BF16)
        ceiling_mfma_bf16_kernel<<<grid, block, 0, s>>>(a, a_bytes, b, b_bytes, iters, sink);
    else
        ceiling_mfma_f8_kernel<<<grid, block, 0, s>>>(a, a_bytes, b, b_bytes, iters, sink);
    if (ops_out) {
        auto per_wave = [](auto traits) { return (double)kBufs * traits.FRAGS * traits.FRAGS * traits.OPS; };
        *ops_out = (kind == CEIL_I8     ? per_wave(CeilTraits<CEIL_I8>())
                    : kind == CEIL_BF16 ? per_wave(CeilTraits<CEIL_BF16>())
                                        : per_wave(CeilTraits<CEIL_F8>())) *
                   iters * workgroups * waves_per_workgroup;
    }
    return hipGetLastError() == hipSuccess ? SB_OK : SB_HIP_ERROR;
}

int switchback_ceiling_copy(const void *src, void *dst, size_t bytes, void *stream) {
    if (src == nullptr || dst == nullptr || !sb::aligned16(src) || !sb::aligned16(dst) || bytes % 16) return SB_INVALID_ARG;
    if (bytes == 0) return SB_OK;
    const size_t chunks = bytes / 16;
    size_t blocks = (chunks + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    sb::ceiling_copy_kernel<<<(unsigned)blocks, 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<const sb::v4u *>(src), static_cast<sb::v4u *>(dst), chunks);
    return hipGetLastError() == hipSuccess ? SB_OK : SB_HIP_ERROR;
}

}  // extern "C"
