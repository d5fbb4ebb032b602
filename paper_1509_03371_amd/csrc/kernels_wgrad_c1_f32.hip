// Weight gradient of an fp32 layer with ONE input map (the first layer of a net): kernels of at most sixteen taps, at most 64 output maps.
//
// dW[o][tap] = sum over pixels of dY[o][pixel] X[pixel + tap] is 0.4 GFLOP for the 48 maps of a 512^2 image (three us of the fp32 matrix unit) behind 55 MB of
// dY, so it is bound by reading dY once.  Both operands come from global memory as they are: lane (g, l16) of a wave loads pixels 4 g .. 4 g + 3 of map l16
// of a tile, the operand of four K steps, and the same pixels of X moved by tap l16, which the caches hold.  Blocks of 32 pixels of a row, two such
// loads, so that a wave takes whole lines; the loads of the next block are on the way while this one is multiplied.  Eight waves, each with sums of its
// own, meet in LDS; a workgroup writes one private copy, which wgrad_reduce_kernel adds up, and its sums of dY, which come along in registers.
// 4x4, 1 -> 48 maps at 564^2 with the sums of dY, which were a launch of their own: 44.1 + 16.6 -> 20.2 us.
#include <algorithm>

#include "sk_kernels.h"

namespace sk {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));      // sixteen bytes at any float

constexpr int C1W_WAVES = 8, C1W_THREADS = 64 * C1W_WAVES, C1W_PX = 32;

struct WgradC1Args {
    const float *x, *dy;
    float *scratch, *bias_part;            // bias_part[map * gridDim.x + workgroup], or nullptr
    int c_out, H, W, Ho, Wo, k, d;
    int per_row, total;                    // blocks of a row, of all images
};

template <int MT>
__global__ __launch_bounds__(C1W_THREADS, 2) void wgrad_c1_f32_kernel(WgradC1Args a)
{
    __shared__ floatx4 red[C1W_WAVES][MT][64];
    __shared__ float bred[C1W_WAVES][MT * 16];
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int plane = a.Ho * a.Wo, tap = l16 < a.k * a.k ? l16 : 0, ti = tap / a.k, tj = tap - ti * a.k;
    const unsigned x_off = (unsigned)(ti * a.d * a.W + tj * a.d + 4 * g);
    unsigned y_off[MT];                    // (missing maps of the last tile read the last one)
#pragma unroll
    for (int t = 0; t < MT; ++t) y_off[t] = (unsigned)(min(16 * t + l16, a.c_out - 1) - min(16 * t, a.c_out - 1)) * (unsigned)plane + 4u * g;
    struct Block { floatx4 y[MT][2], x[2]; };
    auto load = [&](Block &v, int blk) {
        const int row = blk / a.per_row, px0 = (blk - row * a.per_row) * C1W_PX, b = row / a.Ho, y = row - b * a.Ho;
        const float *xs = a.x + ((long)b * a.H + y) * a.W + px0, *ys = a.dy + (long)b * a.c_out * plane + (long)y * a.Wo + px0;
        if (px0 + C1W_PX <= a.Wo) {                                          // uniform
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int t = 0; t < MT; ++t) v.y[t][h] = *reinterpret_cast<const float4u *>(ys + (long)min(16 * t, a.c_out - 1) * plane + 16 * h + y_off[t]);
                v.x[h] = *reinterpret_cast<const float4u *>(xs + 16 * h + x_off);
            }
            return;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool real = px0 + 16 * h + 4 * g + e < a.Wo;
#pragma unroll
                for (int t = 0; t < MT; ++t) v.y[t][h][e] = real ? ys[(long)min(16 * t, a.c_out - 1) * plane + 16 * h + y_off[t] + e] : 0.f;
                v.x[h][e] = real ? xs[16 * h + x_off + e] : 0.f;
            }
    };
    floatx4 acc[MT];
    float sum[MT] = {};
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    int blk = blockIdx.x * C1W_WAVES + wave;
    const int stride = gridDim.x * C1W_WAVES;
    if (blk < a.total) {
        Block v, next;
        load(v, blk);
        while (true) {
            const bool more = blk + stride < a.total;
            if (more) load(next, blk + stride);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < MT; ++t) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v.y[t][h][e], v.x[h][e], acc[t], 0, 0, 0);
                    sum[t] += (v.y[t][h][0] + v.y[t][h][1]) + (v.y[t][h][2] + v.y[t][h][3]);
                }
            if (!more) break;
            blk += stride;
            v = next;
        }
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        red[wave][t][lane] = acc[t];
        float s = sum[t];                  // of a tile's maps over the four lane groups
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (g == 0) bred[wave][16 * t + l16] = s;
    }
    __syncthreads();
    // wave t adds tile t: rows 4 g .. 4 g + 3 (maps), column l16 (tap)
    if (wave < MT) {
        floatx4 s = red[0][wave][lane];
#pragma unroll
        for (int w = 1; w < C1W_WAVES; ++w) s += red[w][wave][lane];
        float *const copy = a.scratch + (long)blockIdx.x * (MT * 256) + (16 * wave + 4 * g) * 16 + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r) copy[16 * r] = s[r];
    }
    if (a.bias_part && (int)threadIdx.x < a.c_out) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < C1W_WAVES; ++w) s += bred[w][threadIdx.x];
        a.bias_part[(long)threadIdx.x * gridDim.x + blockIdx.x] = s;
    }
}

}  // namespace

// 120 gradients of 2x2 to 4x4 to 3 to 64 maps, 24 x 30 to 3 x 700 x 500, d = 1 and 3, with their reductions: 0.23 to 0.81 of the time on wgrad_f32_kernel
bool wgrad_c1_f32_supported(int c_in, int c_out, int k, int n, int Ho, int Wo)
{
    const long plane = (long)Ho * Wo;
    return c_in == 1 && c_out >= 1 && c_out <= 64 && k >= 2 && k <= 4 && Ho >= 1 && Wo >= 1 && plane <= 0x3ffffffL &&     // (offsets inside a tile are 32 bits)
           n * (plane / C1W_PX + Ho) <= 0x3fffffffL;
}

hipError_t launch_wgrad_c1_f32(const float *x, const float *dy, float *scratch, float *bias_part, int n, int H, int W, int c_out, int k, int d,
                               int max_copies, int *copies, hipStream_t stream)
{
    WgradC1Args a;
    a.x = x; a.dy = dy; a.scratch = scratch; a.bias_part = bias_part;
    a.c_out = c_out; a.H = H; a.W = W; a.k = k; a.d = d;
    a.Ho = H - (k - 1) * d; a.Wo = W - (k - 1) * d;
    if (n < 1 || d < 1 || max_copies < 1 || !wgrad_c1_f32_supported(1, c_out, k, n, a.Ho, a.Wo)) return hipErrorInvalidValue;
    a.per_row = (a.Wo + C1W_PX - 1) / C1W_PX;
    a.total = n * a.Ho * a.per_row;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    *copies = std::max(1, std::min(std::min(max_copies, cus), (a.total + C1W_WAVES - 1) / C1W_WAVES));
    const dim3 grid(*copies), block(C1W_THREADS);
    switch ((c_out + 15) / 16) {
    case 1: hipLaunchKernelGGL(wgrad_c1_f32_kernel<1>, grid, block, 0, stream, a); break;
    case 2: hipLaunchKernelGGL(wgrad_c1_f32_kernel<2>, grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL(wgrad_c1_f32_kernel<3>, grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL(wgrad_c1_f32_kernel<4>, grid, block, 0, stream, a); break;
    }
    return hipGetLastError();
}

}  // namespace sk
