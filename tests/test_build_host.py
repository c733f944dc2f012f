"""What the build refuses: kernels whose registers the compiler has spilled, or whose named accumulators it uses itself."""
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


@pytest.mark.parametrize("source,fault", [(LIVE % 256, None), (LIVE % 64, "vgpr_spill_count"), (NAMED % "", None),
                                          (NAMED % 'asm volatile("; %0" ::"a"(q[threadIdx.x]));', " a")],
                         ids=["fits", "spills", "named", "used"])
def test_build_refuses_spills_and_used_accumulators(tmp_path, source, fault):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(source.replace("%%", "%"))
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "-S", "--offload-device-only", str(src), "-o", str(asm)], check=True,
                   capture_output=True)
    faults = build.check_kernels(asm.read_text())
    assert (faults == []) if fault is None else any(fault in f for f in faults), faults
