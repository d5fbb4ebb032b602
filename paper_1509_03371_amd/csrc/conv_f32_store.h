// Stores of the fp32 convolutions' accumulators (kernels_conv_f32.hip, kernels_conv_split_f32.hip).
#pragma once
#include <type_traits>

#include "sk_kernels.h"

namespace sk {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Epilogue of the fp32 convolutions: bias, ReLU, optional ReLU-derivative mask, predicated store.
// acc[rw][xt][nt][r] belongs to output map o_first + 16*nt + r, row oy_first + rw*d, column
// ox_first + 16*xt.  The vector memory counter is one in-order queue for loads and stores, so a
// load awaited between stores makes that wait cover every store before it.  The bias is therefore
// fetched in one batch and awaited once; the store loop without a mask then contains no load at
// all, and the masked variant fetches the masks of a whole pixel tile before its first store.
template <int NT, int RW, int XN = 4, int XD = 4>
__device__ __forceinline__ void store_outputs(const ConvF32Args &a, floatx4 (&acc)[RW][XD][NT], int b, int o_first,
                                              int oy_first, int d, int ox_first)
{
    float bia[NT][4];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) bia[nt][r4] = 0.f;
    if (a.bias) {                                       // uniform branch; the vector holds n_pad entries
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int o = o_first + nt * 16 + r4;
                bia[nt][r4] = a.bias[o < a.n_pad ? o : a.n_pad - 1];
            }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): the bias is in registers from here on
    __builtin_amdgcn_sched_barrier(0);
    const long oplane = (long)a.OH * a.OW;
    // mode 0: plain store; 1: ReLU-derivative mask; 2: the value already in y is added before bias and ReLU
    auto store_tiles = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
#pragma unroll
        for (int rw = 0; rw < RW; ++rw) {
            const int oy = oy_first + rw * d;
            if (oy >= a.Ho) continue;
            const long rowbase = (((long)b * a.out_maps + a.o_off + o_first) * a.OH + (long)oy * a.oy_mul + a.oy_off) * a.OW + a.ox_off;
#pragma unroll
            for (int xt = 0; xt < XN; ++xt) {
                const int ox = ox_first + xt * 16;
                if (ox >= a.Wo) continue;
                const long pbase = rowbase + (long)ox * a.ox_mul;
                float mk[NT][4];
                if constexpr (MODE != 0) {
                    const float *side = MODE == 1 ? a.mask : a.y;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int r4 = 0; r4 < 4; ++r4) {
                            // maps beyond c_out are never stored; their mask address is clamped to
                            // map 0 of the same pixel so that the load stays inside the tensor
                            const int oo = nt * 16 + r4;
                            mk[nt][r4] = side[pbase + (o_first + oo < a.c_out ? oo : -o_first) * oplane];
                        }
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const int oo = nt * 16 + r4;
                        if (o_first + oo >= a.c_out) continue;
                        float v = acc[rw][xt][nt][r4] + bia[nt][r4];
                        if constexpr (MODE == 2) v += mk[nt][r4];
                        if (a.relu) v = v > 0.f ? v : 0.f;
                        if constexpr (MODE == 1)
                            if (!(mk[nt][r4] > 0.f)) v = 0.f;
                        a.y[pbase + oo * oplane] = v;
                    }
            }
        }
    };
    // the four taps of an up-convolution stacked as GEMM maps: each 16-map tile belongs to one tap, which
    // moves its maps back by tap*tap_maps and its pixels to the tap's place in the 2x2 block (no mask here)
    auto store_taps = [&]() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int o0 = o_first + nt * 16;
            const int tap = o0 / a.tap_maps, om = o0 - tap * a.tap_maps;
#pragma unroll
            for (int rw = 0; rw < RW; ++rw) {
                const int oy = oy_first + rw * d;
                if (oy >= a.Ho) continue;
                const long rowbase = (((long)b * a.out_maps + a.o_off + om) * a.OH + (long)oy * a.oy_mul + (tap >> 1)) * a.OW + (tap & 1);
#pragma unroll
                for (int xt = 0; xt < XN; ++xt) {
                    const int ox = ox_first + xt * 16;
                    if (ox >= a.Wo) continue;
                    const long pbase = rowbase + (long)ox * a.ox_mul;
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        if (o0 + r4 >= a.c_out) continue;
                        float v = acc[rw][xt][nt][r4] + bia[nt][r4];
                        if (a.relu) v = v > 0.f ? v : 0.f;
                        a.y[pbase + r4 * oplane] = v;
                    }
                }
            }
        }
    };
    if (a.tap_maps > 0) store_taps();
    else if (a.mask) store_tiles(std::integral_constant<int, 1>{});
    else if (a.accumulate) store_tiles(std::integral_constant<int, 2>{});
    else store_tiles(std::integral_constant<int, 0>{});
}

}  // namespace sk
