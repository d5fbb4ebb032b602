#pragma once
// What the 16-bit convolutions for many maps share (kernels_conv_wide_h.hip, kernels_conv_wide_big_h.hip): tile geometry,
// direct global -> LDS loads, waits, and the epilogue.
#include "lds_dma.h"
#include "sk_kernels.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace sk {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

constexpr int WV_XQ = 8;        // input loads (64 units each) of a wave per chunk at most

struct WideGeom {
    int xtiles, ytiles, tiles_hi, tiles_lo, rem;      // 3x3: tiles of the output; 1x1: xtiles linear tiles, ytiles = 1
    int mgroups, pgroups;                             // map groups of a workgroup / packed groups of GT (four) map tiles
    int nchunks, split, tiles, total;                 // tiles: without the split; total: with it
    int pw, oct_units;                                // staged row pitch, staged units per octet (a multiple of 64)
    float *ws;                                        // split > 1: partial sums
};
struct WideArgs {
    ConvHArgs a;
    WideGeom w;
};

template <int DT> __device__ __forceinline__ floatx4 wide_mfma(uint4v a, uint4v b, floatx4 c)
{
    if constexpr (DT == 1) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
}
template <int DT> __device__ __forceinline__ unsigned wide_cvt(float f)
{
    if constexpr (DT == 1) return __builtin_bit_cast(unsigned short, static_cast<__bf16>(f));
    else return __builtin_bit_cast(unsigned short, static_cast<_Float16>(f));
}

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int N, class F> __device__ __forceinline__ void wide_for(F &&f)
{
    if constexpr (N > 0) {
        wide_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

__device__ __forceinline__ void wide_load_lds(const void *src, uint4v *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// zero the halves of an octet whose mask value is not positive
__device__ __forceinline__ unsigned wide_mask2(unsigned v, unsigned m)
{
    if ((m & 0x8000u) || !(m & 0x7fffu)) v &= 0xffff0000u;
    if ((m & 0x80000000u) || !(m & 0x7fff0000u)) v &= 0x0000ffffu;
    return v;
}

// MT: map tiles of a wave; GT: map tiles of a packed group (a workgroup takes MG groups)
template <int NWV, int KS, int MG, int R, int XW, int MT = 4, int GT = 4> struct WideTile {
    static constexpr int PWV = NWV / (MG * GT / MT);                  // pixel waves
    static constexpr int YW = KS == 1 ? 1 : PWV / XW, RT = R * YW;         // 3x3: wave rows, output rows of a tile
    static constexpr int TX = KS == 1 ? 16 * R * PWV : 16 * XW;            // output columns (1x1: linear pixels) of a tile
    static constexpr long FLOATS = (long)NWV * R * MT * 256;          // partial sums of a tile
    static_assert(GT % MT == 0 && NWV % (MG * GT / MT) == 0, "map waves share out the tiles of a group");
    static_assert(KS == 1 || PWV % XW == 0, "pixel waves form a grid");
    static_assert(R % 2 == 0, "rows are stored in pairs");
};

struct WidePos {
    int mg, b, py, ty, x0;
};

template <int KS, class T>
__device__ __forceinline__ WidePos wide_decode(const WideGeom &w, int n, int tile)
{
    WidePos p;
    const int xt = tile % w.xtiles;
    int rest = tile / w.xtiles;
    const int yt = rest % w.ytiles;
    rest /= w.ytiles;
    p.b = rest % n;
    p.mg = rest / n;
    p.py = p.ty = 0;
    if (KS != 1) {
        if (yt < w.rem * w.tiles_hi) {
            p.py = yt / w.tiles_hi;
            p.ty = yt - p.py * w.tiles_hi;
        } else {
            const int y2 = yt - w.rem * w.tiles_hi;
            p.py = w.rem + y2 / w.tiles_lo;
            p.ty = y2 % w.tiles_lo;
        }
    }
    p.x0 = xt * T::TX;
    return p;
}

// output row and column of this lane in row y (1x1: 16-pixel group y) of the tile; false outside the image
template <int KS, int R, int XW, class T>
__device__ __forceinline__ bool wide_pixel(const ConvHArgs &a, const WidePos &p, int pw, int y, int l16, int &oy, int &ox)
{
    if (KS == 1) {
        const int q = p.x0 + (pw * R + y) * 16 + l16;
        oy = q / a.Wo;
        ox = q - oy * a.Wo;
        return q < a.Ho * a.Wo;
    }
    oy = p.py + a.d * (p.ty * T::RT + (pw / XW) * R + y);
    ox = p.x0 + (pw % XW) * 16 + l16;
    return oy < a.Ho && ox < a.Wo;
}

constexpr int WV_OCT = 0, WV_OCT_MASK = 1, WV_F32 = 2;      // what a launch writes: octets, octets under a mask, fp32 planes

// Epilogue of rows y and y + 1 of the four map tiles from mt0 on (v0, v1: this lane's four maps of its pixel in either row):
// bias, ReLU, conversion, mask, store.  After one v_permlane16_swap per register the even lane groups own whole octets of row
// y and the odd ones of row y + 1, so every store is a 16-byte one.  `at`: this lane's address of octet mt0 * 2 in y (octet
// planes of plane_bytes, or fp32 planes in WV_F32, where both rows are stored by every lane: at[0], at[1]).
template <int OUT>
struct WideDst {
    char *at[2];
    bool ok[2];
};

template <int OUT, int KS, int R, int XW, class T>
__device__ __forceinline__ WideDst<OUT> wide_dst(const ConvHArgs &a, const WidePos &p, int pwv, int y, int l16, int g, int mt0)
{
    WideDst<OUT> r;
    const int unit = OUT == WV_F32 ? 4 : 16, row_bytes = a.OW * unit;
    const long plane_bytes = (long)a.OH * row_bytes;
    char *base = reinterpret_cast<char *>(a.y);
    if (OUT == WV_F32) base += ((long)p.b * a.c_out + mt0 * 16 + 4 * g) * plane_bytes;
    else base += ((long)p.b * a.c8_out_total + a.o8_off + mt0 * 2 + (g >> 1)) * plane_bytes;
#pragma unroll
    for (int s = 0; s < (OUT == WV_F32 ? 2 : 1); ++s) {
        int oy, ox;
        r.ok[s] = wide_pixel<KS, R, XW, T>(a, p, pwv, y + (OUT == WV_F32 ? s : (g & 1)), l16, oy, ox);
        r.at[s] = base + ((oy * a.oy_mul + a.oy_off) * (long)row_bytes + (long)((ox * a.ox_mul + a.ox_off) * unit));
    }
    return r;
}

// stacked up-convolution taps: bytes from octet mtile * 2 to where the tile's tap stores it (its own octet, its pixel of the 2x2 block)
__device__ __forceinline__ long wide_tap(const ConvHArgs &a, int mtile)
{
    if (a.tap_maps == 0) return 0;
    const int tap = mtile * 16 / a.tap_maps;
    return ((long)(tap >> 1) * a.OW + (tap & 1)) * 16 - (long)tap * (a.tap_maps / 8) * ((long)a.OH * a.OW * 16);
}

template <int DT, int OUT>
__device__ __forceinline__ void wide_store(const ConvHArgs &a, floatx4 v0, floatx4 v1, const float (&bia)[4], const WideDst<OUT> &dst, int mt0, int mt,
                                           int g, uint4v mask)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        v0[r] += bia[r];
        v1[r] += bia[r];
        if (a.relu) {
            v0[r] = fmaxf(v0[r], 0.f);
            v1[r] = fmaxf(v1[r], 0.f);
        }
    }
    if constexpr (OUT == WV_F32) {
        const long plane_bytes = (long)a.OH * a.OW * 4;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if ((mt0 + mt) * 16 + 4 * g + r < a.c_out) {
                if (dst.ok[0]) *reinterpret_cast<float *>(dst.at[0] + (mt * 16 + r) * plane_bytes) = v0[r];
                if (dst.ok[1]) *reinterpret_cast<float *>(dst.at[1] + (mt * 16 + r) * plane_bytes) = v1[r];
            }
    } else {
        const unsigned lo0 = wide_cvt<DT>(v0[0]) | (wide_cvt<DT>(v0[1]) << 16), hi0 = wide_cvt<DT>(v0[2]) | (wide_cvt<DT>(v0[3]) << 16);
        const unsigned lo1 = wide_cvt<DT>(v1[0]) | (wide_cvt<DT>(v1[1]) << 16), hi1 = wide_cvt<DT>(v1[2]) | (wide_cvt<DT>(v1[3]) << 16);
        const auto s0 = __builtin_amdgcn_permlane16_swap(lo0, lo1, false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(hi0, hi1, false, false);
        uint4v octet = uint4v{s0[0], s1[0], s0[1], s1[1]};
        if constexpr (OUT == WV_OCT_MASK) {
#pragma unroll
            for (int r = 0; r < 4; ++r) octet[r] = wide_mask2(octet[r], mask[r]);
        }
        if (dst.ok[0] && (mt0 + mt) * 2 + (g >> 1) < a.c8_out)
            *reinterpret_cast<uint4v *>(dst.at[0] + mt * 2 * ((long)a.OH * a.OW * 16) + wide_tap(a, mt0 + mt)) = octet;
    }
}

// The kernel's arguments, to be read where they are used: what only the epilogue or the next tile needs would otherwise hold
// scalar registers through the multiplication (a hundred of them spilled to lanes of vector registers).
__device__ __forceinline__ const WideArgs *wide_args()
{
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (const WideArgs *)p;
}

int wide_cus()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8)
            cus = 256;
    }
    return cus;
}

}  // namespace
}  // namespace sk
