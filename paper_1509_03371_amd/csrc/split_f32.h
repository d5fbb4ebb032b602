// fp32 values as pairs of fp16 values, for products on the 16-bit matrix unit.
//
// A value times a power of two that takes the largest of its kind to 2^12 .. 2^15 (where fp16 ends, 2^16, values round up to infinity) is
// the sum of an fp16 value and the fp16-rounded rest:
// exactly or (a quarter of the values) to one bit of 24, as long as it is above 2^-17 of the largest, and to 2^-40 of the largest below.  A
// product takes three of the four partial products; the fourth is below 2^-22 of it, on average 2^-24 and of either sign.  The matrix unit
// adds 32 products to an fp32 sum at a time, where its fp32 form adds four, so long sums are rounded less often and come out closer to 64
// bits than with fp32 operands (conv_split_f32_packed).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace sk {

namespace {

typedef float split_floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 split_halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 split_halfx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

constexpr int SPLIT_WIDE = 1000;      // in the place of a weights' power of two: pairs cannot hold them
constexpr int SPLIT_MOST = 110;       // largest power of two that values are scaled by (values below 2^-98 lose bits)

__device__ __forceinline__ split_floatx4 split_mfma(uint4v a, uint4v b, split_floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(split_halfx8, a), __builtin_bit_cast(split_halfx8, b), c, 0, 0, 0);
}

// p[0][e] + p[1][e] = v[e] * scale
__device__ __forceinline__ void split2(const float (&v)[8], float scale, uint4v (&p)[2])
{
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const split_halfx2 h = {(_Float16)__builtin_fmaf(v[e], scale, 0.f), (_Float16)__builtin_fmaf(v[e + 1], scale, 0.f)};
        const split_halfx2 l = {(_Float16)__builtin_fmaf(v[e], scale, -(float)h[0]), (_Float16)__builtin_fmaf(v[e + 1], scale, -(float)h[1])};
        p[0][e / 2] = __builtin_bit_cast(unsigned, h);
        p[1][e / 2] = __builtin_bit_cast(unsigned, l);
    }
}

// Largest of non-negative values; their bits are in the values' order, and comparing those needs no quieting of NaNs
__device__ __forceinline__ float split_max(float a, float b)
{
    return __builtin_bit_cast(float, max(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b)));
}

// ... over the wave, in every lane
__device__ __forceinline__ float split_wave_max(float m)
{
    const auto step = [&](auto ctrl) {
        m = split_max(m, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, m), decltype(ctrl)::value, 0xf, 0xf, true)));
    };
    step(std::integral_constant<int, 0x111>{});      // row_shr 1, 2, 4, 8: lane 15 of a row has the row's
    step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{});
    step(std::integral_constant<int, 0x118>{});
    const int v = __builtin_bit_cast(int, m);
    const int a = max(__builtin_amdgcn_readlane(v, 15), __builtin_amdgcn_readlane(v, 31)), b = max(__builtin_amdgcn_readlane(v, 47), __builtin_amdgcn_readlane(v, 63));
    return __builtin_bit_cast(float, max(a, b));
}

// the power of two that takes m to 2^top .. 2^(top + 1)
__device__ __forceinline__ int split_exponent(float m, int top)
{
    const int e = (int)((__builtin_bit_cast(unsigned, m) >> 23) & 0xff) - 127;
    const int s = top - e;
    return s < SPLIT_MOST ? s : SPLIT_MOST;
}
__device__ __forceinline__ float split_pow2(int s) { return __builtin_bit_cast(float, (unsigned)(s + 127) << 23); }     // -126 <= s <= 127

__device__ __forceinline__ float split_finite(float v) { return (__builtin_bit_cast(unsigned, v) & 0x7f800000u) == 0x7f800000u ? 0.f : v; }

}  // namespace

}  // namespace sk
