// Global memory straight into LDS for kernels whose LDS reads are transposing ones.
//
// The compiler cannot tell which LDS addresses a transposing read (ds_read_b64_tr_b16) touches, and waits for EVERY
// __builtin_amdgcn_global_load_lds under way ahead of it: rows that are loaded steps ahead of their use were waited for at once.  This load is
// out of its sight, so the kernel waits for it alone: s_waitcnt vmcnt with the number of younger loads, then a barrier.
#pragma once
#include <hip/hip_runtime.h>

namespace sk {

// lane l's sixteen bytes at src to dst + 16 l (dst: the same in every lane; inactive lanes move nothing)
__device__ __forceinline__ void lds_dma16(const void *src, const void *dst)
{
    const unsigned at = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(const __attribute__((address_space(3))) void *)dst);
    // m0 holds the LDS address, one instruction ahead of its use.  The compiler keeps operands of its own there: it has to know that they are
    // lost, also where it warns that the register is not its to allocate
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(at) : "memory", "m0");
#pragma clang diagnostic pop
}

// meet the workgroup with this wave's LDS operations done (loads to LDS stay under way)
__device__ __forceinline__ void wide_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// wait until at most N of this wave's memory operations are outstanding
template <int N> __device__ __forceinline__ void wide_wait()
{
    static_assert(N >= 0 && N < 64, "vmcnt is six bits");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace sk
