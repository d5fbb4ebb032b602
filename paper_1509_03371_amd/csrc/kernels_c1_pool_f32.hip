// First layer of an fp32 inference plan together with its mirror padding and its pool (gfx950):
//
//   Y[o,y,x] = max_{a,b < 2} act(bias[o] + sum_{i,j < k} W[o][0][i][j] * P[y+a+i, x+b+j]),  P = the padded image
//
// One input map leaves k*k multiplications an output sample, so three launches (padding, convolution, pool) moved the 48
// maps of a 512^2 image through memory three times for 0.4 GFLOP.  Here a thread owns R rows of four adjacent pooled
// samples: it keeps the (R + k) x (k + 4) window of the padded image that they need in registers -- read from the caller's
// image, mirrored where the window leaves it -- and walks over `per` output maps, two at a time: (R + 1) x 5
// accumulators each, weights and biases at wave-uniform addresses, i.e. scalar loads.  What is left to move is the pooled
// map, one float4 store a row.  The edge rows and columns are computed twice (1.56 times the multiplications
// at R = 4): with 64 operations a sample that stays below the time of the stores.  The sums and maxima are taken in the order of
// conv_c1_f32_kernel and maxpool2_chain_f32_kernel, so the results are theirs bit for bit.
// The padded image goes to memory on the way (sknet_get_activation hands it out), by the threads of the first map group, and so do
// the weights and biases of the pass, by a workgroup beside the others: the layer's output, which is not stored, is made from these three.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mirror_index.h"
#include "sk_kernels.h"

namespace sk {
namespace {

typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));      // sixteen bytes at any float

template <int KS, int R>
__global__ __launch_bounds__(64) void conv_c1_pool_f32_kernel(C1PoolF32Args a, int per)
{
    constexpr int WR = R + KS, WC = KS + 4;              // window: R + 1 rows and 5 columns of outputs
    const int H = a.h_pad, W = a.w_pad, Ho = H - KS, Wo = W - KS;
    const int w4 = (Wo + 3) / 4, rows = (Ho + R - 1) / R;
    if (blockIdx.x == 0) {               // ahead of the samples: behind them its loads and stores would be the launch's tail
        if (blockIdx.y == 0 && blockIdx.z == 0) {
            auto copy = [](const float *from, float *to, int floats) {        // (a multiple of sixteen, at sixteen bytes)
                for (int q = 4 * threadIdx.x; q < floats; q += 4 * 64) *reinterpret_cast<float4 *>(to + q) = *reinterpret_cast<const float4 *>(from + q);
            };
            copy(a.wp, a.used_w, KS * KS * a.n_pad);
            copy(a.bias, a.used_b, a.n_pad);
        }
        return;
    }
    const int idx = (blockIdx.x - 1) * 64 + threadIdx.x;
    if (idx >= rows * w4) return;
    const int rg = idx / w4;
    // the last group of a row or column is moved back inside the map: its samples are written twice, with the same values
    const int x0 = min(4 * (idx - rg * w4), Wo - 4), y0 = min(R * rg, Ho - R), b = blockIdx.z;
    const float *src = a.image + (long)b * a.h * a.w;
    const int sy = y0 - a.top, sx = x0 - a.left;
    float win[WR][WC];
    if (sy >= 0 && sy + WR <= a.h && sx >= 0 && sx + WC <= a.w) {
        const float *p = src + (long)sy * a.w + sx;
#pragma unroll
        for (int r = 0; r < WR; ++r) {
            const float4u v = *reinterpret_cast<const float4u *>(p + (long)r * a.w);
#pragma unroll
            for (int c = 0; c < 4; ++c) win[r][c] = v[c];
            if constexpr (WC == 8) {
                const float4u u = *reinterpret_cast<const float4u *>(p + (long)r * a.w + 4);
#pragma unroll
                for (int c = 0; c < 4; ++c) win[r][4 + c] = u[c];
            } else {
#pragma unroll
                for (int c = 4; c < WC; ++c) win[r][c] = p[(long)r * a.w + c];
            }
        }
    } else {
        int cx[WC];
#pragma unroll
        for (int c = 0; c < WC; ++c) cx[c] = mirror_index(sx + c, a.w, a.mode);
#pragma unroll
        for (int r = 0; r < WR; ++r) {
            const float *p = src + (long)mirror_index(sy + r, a.h, a.mode) * a.w;
#pragma unroll
            for (int c = 0; c < WC; ++c) win[r][c] = p[cx[c]];
        }
    }
    if (blockIdx.y == 0) {
        float *dst = a.padded + ((long)b * H + y0) * W + x0;
#pragma unroll
        for (int r = 0; r < WR; ++r)
#pragma unroll
            for (int c = 0; c < WC; c += 4) {
                // the last columns of a 3x3 window (seven wide) overlap the first ones
                const int c0 = c + 4 <= WC ? c : WC - 4;
                *reinterpret_cast<float4u *>(dst + (long)r * W + c0) = float4u{win[r][c0], win[r][c0 + 1], win[r][c0 + 2], win[r][c0 + 3]};
            }
    }
    const unsigned off = 4u * ((unsigned)y0 * (unsigned)Wo + (unsigned)x0);     // 4*Ho*Wo < 2^32 (checked by the launcher)
    const int o_end = min((int)(blockIdx.y + 1) * per, a.c_out);
#pragma unroll 1
    for (int o = blockIdx.y * per; o < o_end; o += 2) {          // n_pad is a multiple of 16: the second of a pair is readable
        float acc[2][R + 1][5];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int r = 0; r <= R; ++r)
#pragma unroll
                for (int c = 0; c < 5; ++c) acc[e][r][c] = a.bias[o + e];
#pragma unroll
        for (int i = 0; i < KS; ++i)
#pragma unroll
            for (int j = 0; j < KS; ++j)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float w = a.wp[(i * KS + j) * a.n_pad + o + e];
#pragma unroll
                    for (int r = 0; r <= R; ++r)
#pragma unroll
                        for (int c = 0; c < 5; ++c) acc[e][r][c] = fmaf(w, win[r + i][c + j], acc[e][r][c]);
                }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (o + e >= o_end) break;                           // uniform
            char *map = reinterpret_cast<char *>(a.y + ((long)b * a.c_out + o + e) * Ho * Wo);
            float4u h[R + 1];
#pragma unroll
            for (int r = 0; r <= R; ++r) {
                float v[5];
#pragma unroll
                for (int c = 0; c < 5; ++c) v[c] = a.relu ? fmaxf(acc[e][r][c], 0.f) : acc[e][r][c];
#pragma unroll
                for (int c = 0; c < 4; ++c) h[r][c] = v[c + 1] > v[c] ? v[c + 1] : v[c];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float4u best;
#pragma unroll
                for (int c = 0; c < 4; ++c) best[c] = h[r + 1][c] > h[r][c] ? h[r + 1][c] : h[r][c];
                *reinterpret_cast<float4u *>(map + off + 4u * (unsigned)(r * Wo)) = best;
            }
        }
    }
}

template <int KS, int R>
hipError_t launch_t(const C1PoolF32Args &a, long waves, hipStream_t stream)
{
    // maps a thread walks over: as many as still leave two waves a SIMD (every further group reads the windows again)
    int per = (a.c_out + 1) & ~1;
    while (per > 2 && waves * ((a.c_out + per - 1) / per) < 2048) per = std::max(2, per / 2 & ~1);
    hipLaunchKernelGGL((conv_c1_pool_f32_kernel<KS, R>), dim3((unsigned)waves + 1, (a.c_out + per - 1) / per, a.n), dim3(64), 0, stream, a, per);
    return hipGetLastError();
}

template <int KS>
hipError_t launch_k(const C1PoolF32Args &a, hipStream_t stream)
{
    const long Ho = a.h_pad - KS, w4 = (a.w_pad - KS + 3) / 4;
    const long waves4 = ((Ho + 3) / 4 * w4 + 63) / 64;
    // four rows a thread compute the fewest edge samples; a small image has too few of them for one wave a SIMD.  78 layers (k 3 and 4, 8 to 200
    // maps, 32 x 40 to 8 x 700^2): two rows 0.76 to 1.0 of four's time below the line up to 48 maps (200 maps: up to 1.14), 0.99 to 1.6
    // above it (200 maps at 200^2: 0.9); either at most 0.55 of padding, convolution and pool as launches
    if (Ho >= 4 && waves4 * a.n * ((a.c_out + 1) / 2) >= 1024) return launch_t<KS, 4>(a, waves4, stream);
    return launch_t<KS, 2>(a, ((Ho + 1) / 2 * w4 + 63) / 64, stream);
}

}  // namespace

bool conv_c1_pool_f32_supported(int k, int n, int h_pad, int w_pad)
{
    return (k == 3 || k == 4) && n <= 65535 && h_pad - k >= 2 && w_pad - k >= 4 && (long)h_pad * w_pad < (1L << 29);
}

hipError_t launch_conv_c1_pool_f32(const C1PoolF32Args &a, hipStream_t stream)
{
    if (!conv_c1_pool_f32_supported(a.k, a.n, a.h_pad, a.w_pad) || a.c_out < 1 || a.c_out > a.n_pad || a.n_pad % 16 != 0) return hipErrorInvalidValue;
    return a.k == 3 ? launch_k<3>(a, stream) : launch_k<4>(a, stream);
}

}  // namespace sk
