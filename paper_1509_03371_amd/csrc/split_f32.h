// fp32 values as pairs of fp16 values, for products on the 16-bit matrix unit.
//
// A value times a power of two that takes the largest of its kind below 2^15 is an fp16 value h and the fp16-rounded rest times 2^12, l: v = h + l / 2^12
// exactly or (a quarter of the values) to one bit of 24 from 2^-13 on, and to 2^-36 below.  Where a value that is not zero lies below 2^SPLIT_LEAST = 2^-16,
// or one is infinite, products are made on the fp32 matrix unit.  A product takes three of the four partial products: h h' in one sum, h l' + l h' in
// another, which is worth 2^-12 of it; the fourth is below 2^-22 of the product, on average 2^-24 and of either sign.  The matrix unit adds 32
// products to an fp32 sum at a time, where its fp32 form adds four, so long sums are rounded less often and come out closer to 64 bits than with
// fp32 operands (conv_split_f32_packed), also sums of the least values alone, which are held to 2^-21.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace sk {

namespace {

typedef float split_floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 split_halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 split_halfx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

constexpr int SPLIT_MOST = 110;       // largest power of two that values are scaled by
constexpr int SPLIT_WIDE = 1000;      // in the place of a power of two: pairs do not hold the values
constexpr int SPLIT_LEAST = -16;      // power of two of the least scaled values that pairs hold

__device__ __forceinline__ split_floatx4 split_mfma(uint4v a, uint4v b, split_floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(split_halfx8, a), __builtin_bit_cast(split_halfx8, b), c, 0, 0, 0);
}

// p[0][e] + p[1][e] / 2^12 = v[e] * scale
__device__ __forceinline__ void split2(const float (&v)[8], float scale, uint4v (&p)[2])
{
    const float low = scale * 4096.f;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const split_halfx2 h = {(_Float16)__builtin_fmaf(v[e], scale, 0.f), (_Float16)__builtin_fmaf(v[e + 1], scale, 0.f)};
        const split_halfx2 l = {(_Float16)__builtin_fmaf((float)h[0], -4096.f, v[e] * low), (_Float16)__builtin_fmaf((float)h[1], -4096.f, v[e + 1] * low)};
        p[0][e / 2] = __builtin_bit_cast(unsigned, h);
        p[1][e / 2] = __builtin_bit_cast(unsigned, l);
    }
}
// the sum of both sums
__device__ __forceinline__ float split_sum(float high, float low) { return __builtin_fmaf(low, 0x1p-12f, high); }

// The range of magnitudes: the largest, as its bits, and 2^32 - 2 * (bits of the least that is not zero), 0 where there is none.  Bits of
// magnitudes are in the values' order; NaNs count in neither beside values that are not zero
struct SplitRange {
    unsigned most = 0, least = 0;
};
__device__ __forceinline__ SplitRange split_range(const float (&v)[8])
{
    float m = 0.f;
    unsigned l = 0xffffffffu;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        m = fmaxf(fmaxf(fabsf(v[e]), fabsf(v[e + 1])), m);
        l = min(min(2 * __builtin_bit_cast(unsigned, v[e]) - 1, 2 * __builtin_bit_cast(unsigned, v[e + 1]) - 1), l);
    }
    return {__builtin_bit_cast(unsigned, m), ~l};
}
__device__ __forceinline__ SplitRange split_range(SplitRange a, SplitRange b) { return {max(a.most, b.most), max(a.least, b.least)}; }
// Largest of a wave, in its last lane
__device__ __forceinline__ unsigned split_wave_max(unsigned m)
{
    const auto step = [&](auto ctrl) { m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, decltype(ctrl)::value, 0xf, 0xf, true)); };
    step(std::integral_constant<int, 0x111>{});      // row_shr 1, 2, 4, 8: lane 15 of a row has the row's
    step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{});
    step(std::integral_constant<int, 0x118>{});
    step(std::integral_constant<int, 0x142>{});      // row_bcast 15, 31: the rows before
    step(std::integral_constant<int, 0x143>{});
    return m;
}
__device__ __forceinline__ SplitRange split_wave_range(SplitRange r) { return {split_wave_max(r.most), split_wave_max(r.least)}; }
constexpr int SPLIT_LAST_LANE = 63;

// the power of two that takes a magnitude with these bits to 2^top .. 2^(top + 1)
__device__ __forceinline__ int split_exponent(unsigned bits, int top)
{
    const int s = top + 127 - (int)(bits >> 23);
    return s < SPLIT_MOST ? s : SPLIT_MOST;
}
__device__ __forceinline__ float split_pow2(int s) { return __builtin_bit_cast(float, (unsigned)(s + 127) << 23); }     // -126 <= s <= 127

constexpr unsigned SPLIT_INFINITE = 0x7f800000u;      // bits

// Does this range hold values that pairs do not hold with the power of two s?  (Integers alone: the scalar unit does it)
__device__ __forceinline__ bool split_wide(SplitRange r, int s)
{
    const int e = (int)((0u - r.least) >> 24) - 127 + s;       // of the least scaled value (a subnormal one counts as less)
    return r.most == SPLIT_INFINITE || (r.least != 0 && e < SPLIT_LEAST);
}

}  // namespace

}  // namespace sk
