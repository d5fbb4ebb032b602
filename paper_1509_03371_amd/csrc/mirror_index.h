// Source index of sample t of an image line of `len` samples continued by mirroring (Section 1.3).
#pragma once
#include <hip/hip_runtime.h>

namespace sk {

__device__ __forceinline__ int mirror_index(int t, int len, int mode)
{
    if (len == 1) return 0;
    if (mode == 0) {                       // reflect: ... 2 1 | 0 1 2 ... L-1 | L-2 L-3 ...
        const int period = 2 * (len - 1);
        t %= period;
        if (t < 0) t += period;
        return t < len ? t : period - t;
    }
    const int period = 2 * len;            // symmetric: ... 1 0 | 0 1 ... L-1 | L-1 L-2 ...
    t %= period;
    if (t < 0) t += period;
    return t < len ? t : period - 1 - t;
}

}  // namespace sk
