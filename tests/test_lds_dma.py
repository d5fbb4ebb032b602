"""The load to LDS that the compiler does not see (csrc/lds_dma.h) beside one that it does see: both address LDS through m0, so the compiler
has to set m0 again behind the first.  Looks at the assembly of a small kernel with both in a loop."""
import os
import re
import subprocess

import pytest

from paper_1509_03371_amd import build

KERNEL = r"""
#include "lds_dma.h"
using global_ptr = const __attribute__((address_space(1))) void *;
using lds_ptr = __attribute__((address_space(3))) void *;
__global__ void both(const char *s, const char *t, float *o, int n, int m)
{
    extern __shared__ char lds[];
    for (int i = 0; i < n; ++i) {
        __builtin_amdgcn_global_load_lds((global_ptr)(s + i * 64), (lds_ptr)lds, 16, 0, 0);
        sk::lds_dma16(t + i * 64, lds + 4096);
        __builtin_amdgcn_global_load_lds((global_ptr)(s + i * 64 + m), (lds_ptr)lds, 16, 0, 0);
    }
    __syncthreads();
    o[threadIdx.x] = reinterpret_cast<float *>(lds)[threadIdx.x];
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc here")
def test_the_compiler_sets_its_lds_address_again(tmp_path):
    src, out = tmp_path / "both.hip", tmp_path / "both.s"
    src.write_text(KERNEL)
    subprocess.run([build.HIPCC] + build.FLAGS + ["-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True, capture_output=True)
    events = re.findall(r"s_mov_b32 m0|global_load_lds_dwordx4|s_cbranch", out.read_text())
    loads = [i for i, e in enumerate(events) if e.startswith("global_load_lds")]
    assert len(loads) == 3, events
    for i in loads:
        assert events[i - 1] == "s_mov_b32 m0", events
