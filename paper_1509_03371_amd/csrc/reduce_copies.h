// Sums of private copies in a fixed order (internal device code of the weight-gradient reductions).
#pragma once
#include <hip/hip_runtime.h>

namespace sk {

// Sum over `copies` copies, `stride` floats apart, of elements [first, first + 64) below `count`, by a workgroup of 256
// threads; thread t < 64 receives element first + t.  stride, first and count are multiples of 4 and src is 16-byte aligned.
// Latency-bound (a few waves per CU, every load new): 16 lanes take a float4 each and 16 thread groups share the copies
// out, so that 256 copies are two rounds of eight loads in flight.  One float per lane, four waves and four loads in
// flight took 16 rounds: the 256 copies of a 48 -> 48 gradient (38 MB) 17.6 -> 7.5 us, the head's
// (14 MB) 8.9 -> 6.7 us.
__device__ __forceinline__ float sum_copies64(const float *__restrict__ src, long stride, int first, int count, int copies, float (&sh)[16][64])
{
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    const int t = threadIdx.x, quad = t & 15, grp = t >> 4, e = first + 4 * quad;
    floatx4 s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (e < count) {
        const float *p = src + e;
        int c = grp;
        for (; c + 7 * 16 < copies; c += 8 * 16) {
            floatx4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const floatx4 *>(p + (long)(c + 16 * i) * stride);
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] += v[i] + v[i + 4];
        }
        for (; c + 3 * 16 < copies; c += 4 * 16) {
            floatx4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const floatx4 *>(p + (long)(c + 16 * i) * stride);
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] += v[i];
        }
        for (; c < copies; c += 16) s[0] += *reinterpret_cast<const floatx4 *>(p + (long)c * stride);
    }
    *reinterpret_cast<floatx4 *>(&sh[grp][4 * quad]) = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    float r = 0.f;
    if (t < 64) {
        float a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = (sh[4 * i][t] + sh[4 * i + 1][t]) + (sh[4 * i + 2][t] + sh[4 * i + 3][t]);
        r = (a[0] + a[1]) + (a[2] + a[3]);
    }
    return r;
}

}  // namespace sk
