"""What the build refuses: kernels whose registers the compiler has spilled, whose named accumulators it uses itself, or that
touch a register before its LDS read has landed."""
import subprocess

import pytest

from paper_2304_13013_amd import build

HEAD = """
#include <hip/hip_runtime.h>
typedef int v4i __attribute__((ext_vector_type(4)));
"""
# 160 values live over a barrier; with 64 registers a lane most of them are spilled.
LIVE = HEAD + """
extern "C" __global__ __launch_bounds__(64) __attribute__((amdgpu_num_vgpr(%d))) void live(float *p) {
    float v[160];
    for (int i = 0; i < 160; ++i) v[i] = p[i * 64 + threadIdx.x];
    __syncthreads();
    for (int i = 0; i < 160; ++i) p[i * 64 + threadIdx.x] = v[i] * v[(i + 7) %% 160];
}
"""
# An accumulator by name, as in the four-wave kernels, and (second form) a value that is put into one by the compiler.
NAMED = HEAD + """
extern "C" __global__ __launch_bounds__(64) void named(v4i *p, int *q) {
    const v4i a = p[threadIdx.x];
    asm volatile("v_mfma_i32_16x16x64_i8 a[%%0:%%1], %%2, %%3, 0" ::"n"(0), "n"(3), "v"(a), "v"(a) : "a0", "a1", "a2", "a3");
    %s
    int r;
    asm volatile("v_accvgpr_read_b32 %%0, a[%%1]" : "=v"(r) : "n"(2));
    q[threadIdx.x] = r;
}
"""
# A fragment read that is waited for before its use, or (second form) used on one of two ways without a wait.
READ = HEAD + """
extern "C" __global__ __launch_bounds__(64) void read(int *p, int n) {
    __shared__ int s[64];
    s[threadIdx.x] = p[threadIdx.x];
    __syncthreads();
    int v;
    asm volatile("ds_read_b32 %%0, %%1" : "=v"(v) : "v"((unsigned)(threadIdx.x ^ 1) * 4));
    if (n > 0) __builtin_amdgcn_s_waitcnt(0xc07f);
    %s
    asm volatile("v_add_u32 %%0, %%0, %%0" : "+v"(v));
    p[threadIdx.x] = v;
}
"""


@pytest.mark.parametrize("source,fault", [(LIVE % 256, None), (LIVE % 64, "vgpr_spill_count"), (NAMED % "", None),
                                          (NAMED % 'asm volatile("; %0" ::"a"(q[threadIdx.x]));', " a"),
                                          (READ % "__builtin_amdgcn_s_waitcnt(0xc07f);", None), (READ % "", "landed")],
                         ids=["fits", "spills", "named", "used", "waited", "early"])
def test_build_refuses_kernels_that_must_not_run(tmp_path, source, fault):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(source.replace("%%", "%"))
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "-S", "--offload-device-only", str(src), "-o", str(asm)], check=True,
                   capture_output=True)
    faults = build.check_kernels(asm.read_text())
    assert (faults == []) if fault is None else any(fault in f for f in faults), faults
