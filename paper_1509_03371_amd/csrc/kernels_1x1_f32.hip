// fp32 1x1 layers of few maps on one side (gfx950, MFMA 16x16x4 fp32): the convolution, its data gradient, its weight gradient, and the
// fused classification head of inference plans.
//
// All of them are bound by the maps they read and write (48 -> 200 maps: 992 bytes a pixel for 19 kFLOP), and what the kernels
// for any size spend beyond that goes into memory instructions of one float a lane, each of which holds a CU's memory pipeline for tens of
// cycles.  Here a lane owns four consecutive pixels everywhere: lane (g, l16) of a wave loads pixels 4 l16 .. 4 l16 + 3 of map 4 s + g with one
// 16-byte access, which is the B operand of K step s for FOUR products (one for each of its pixels), and these leave it with the same
// four pixels of output maps 4 g .. 4 g + 3, so results and ReLU masks move in 16-byte accesses too (256 bytes in a row per map).
// Planes of odd sizes put these accesses at any float, which global memory takes.
//
//   conv1x1_in_kernel    up to 48 input maps: a wave holds them for its 64 pixels and walks over the output maps (48 -> 200 at 512^2
//                        105 -> 61 us, 8 x 512^2 925 -> 455 = 4.6 TB/s; the masked data gradient 2 -> 200 148 -> 89);
//   conv1x1_out_kernel   up to 48 output maps: a wave holds the sums and streams the input maps (200 -> 48 61 -> 59, 8 x 512^2 526 -> 434);
//   head1x1_kernel       the first with the output maps (the hidden layer) folded into class sums and a softmax on the spot;
//   wgrad1x1_kernel      see there.
// The weights stand in LDS as A fragments.  Waves stride over groups of 64 pixels of an image; the last group of a plane moves back
// so that it lies inside (what overlaps is computed twice, with the same result).
#include <algorithm>

#include "sk_kernels.h"

namespace sk {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));      // sixteen bytes at any float

constexpr int P1_THREADS = 256, P1_WAVES = 4, P1_PX = 64;

__device__ __forceinline__ floatx4 load4(const float *p) { return *reinterpret_cast<const float4u *>(p); }
__device__ __forceinline__ void store4(float *p, floatx4 v) { *reinterpret_cast<float4u *>(p) = v; }
__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

struct Conv1Args {
    const float *x, *wp, *bias, *mask;     // wp: [c_pad][n_pad], as launch_conv_f32 takes it
    float *y;
    long x_bstride;
    int n, c_in, c_out, n_pad, plane, relu;
    int tiles, ksteps, per_image;          // 16-map tiles of the output, steps of four input maps, pixel groups of an image
    int tiles_per;                         // conv1x1_in_kernel: tiles of a workgroup (blockIdx.y the share)
};

// the pixel groups of a wave: image and first pixel
struct Groups {
    int next, stride, total, per_image, plane;
    __device__ __forceinline__ bool at(int grp, int &b, int &px) const
    {
        if (grp >= total) return false;
        b = grp / per_image;
        px = min((grp - b * per_image) * P1_PX, plane - P1_PX);
        return true;
    }
};

// Fragments f = 0 .. count - 1 (64 floats each) to LDS; from(f) gives this lane's float of fragment f (always some address that exists).  A
// wave takes every fourth, eight loads on the way together: one after the other, each waited for, the 150 of a 200 -> 48 layer took longer
// than the multiplication of a small map.
template <class From>
__device__ __forceinline__ void stage_fragments(float *dst, int count, From &&from)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int f0 = wave; f0 < count; f0 += 8 * P1_WAVES) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = from(min(f0 + u * P1_WAVES, count - 1));
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (f0 + u * P1_WAVES < count) dst[(f0 + u * P1_WAVES) * 64 + lane] = v[u];
    }
}

// A fragments [tile][step][lane] of tiles t0 .. t0 + tiles - 1 of the packed weights (zero rows beyond c_in exist up to a multiple of 16)
__device__ __forceinline__ void stage_weights(float *dst, const Conv1Args &a, int t0, int tiles, int ksteps)
{
    const int lane = threadIdx.x & 63;
    stage_fragments(dst, tiles * ksteps, [&](int f) {
        const int t = f / ksteps, c = 4 * (f - t * ksteps) + (lane >> 4);
        const float v = a.wp[(long)(c < a.c_in ? c : 0) * a.n_pad + (t0 + t) * 16 + (lane & 15)];
        return c < a.c_in ? v : 0.f;
    });
}

// rows 4 g + r of N tiles: bias as the sum's start
template <int N>
__device__ __forceinline__ void start_sums(floatx4 (&acc)[N][4], const float *bias, int t0, int g)
{
#pragma unroll
    for (int t = 0; t < N; ++t) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(bias + (t0 + t) * 16 + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][e] = b;
    }
}

template <int N, bool MASK>
__device__ __forceinline__ void store_sums(const floatx4 (&acc)[N][4], const floatx4 (&mk)[MASK ? N : 1][4], const Conv1Args &a, float *y, int t0, int g)
{
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = (t0 + t) * 16 + 4 * g + r;
            floatx4 v = floatx4{acc[t][0][r], acc[t][1][r], acc[t][2][r], acc[t][3][r]};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (a.relu) v[e] = fmaxf(v[e], 0.f);
                if (MASK) v[e] = mk[t][r][e] > 0.f ? v[e] : 0.f;
            }
            if (o < a.c_out) store4(y + (long)o * a.plane, v);
        }
}

template <int N, bool MASK>
__device__ __forceinline__ void load_masks(floatx4 (&mk)[MASK ? N : 1][4], const Conv1Args &a, const float *m, int t0, int g)
{
    if constexpr (MASK) {
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = (t0 + t) * 16 + 4 * g + r;
                mk[t][r] = load4(m + (long)(o < a.c_out ? o : 0) * a.plane);
            }
    }
}

template <int KS, bool MASK>
__global__ __launch_bounds__(P1_THREADS, 2) void conv1x1_in_kernel(Conv1Args a)
{
    extern __shared__ float smem[];
    const int tile0 = blockIdx.y * a.tiles_per, ntiles = min(a.tiles_per, a.tiles - tile0);
    float *const w = smem, *const bias = w + a.tiles_per * KS * 64;
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    stage_weights(w, a, tile0, ntiles, KS);
    for (int q = threadIdx.x; q < ntiles * 16; q += P1_THREADS) bias[q] = a.bias && tile0 * 16 + q < a.c_out ? a.bias[tile0 * 16 + q] : 0.f;
    __syncthreads();
    const Groups groups{0, 0, a.n * a.per_image, a.per_image, a.plane};
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), stride = gridDim.x * P1_WAVES;
    auto load = [&](floatx4 (&x)[KS], int b, int px) {
        const float *src = a.x + (long)b * a.x_bstride + px + 4 * l16;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int c = 4 * s + g;
            x[s] = load4(src + (long)(c < a.c_in ? c : 0) * a.plane);       // (beyond the last map: its weights are zero)
        }
        // (zero times a value that is not finite would not be)
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (4 * s + g >= a.c_in) x[s] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    int grp = blockIdx.x * P1_WAVES + wave, b, px;
    if (!groups.at(grp, b, px)) return;
    floatx4 x[KS], xn[KS];
    load(x, b, px);
    while (true) {
        int nb = 0, npx = 0;
        const bool more = groups.at(grp + stride, nb, npx);
        if (more) load(xn, nb, npx);                                         // in flight while this group is multiplied
        const long at = (long)b * a.c_out * a.plane + px + 4 * l16;
        auto tiles = [&](auto count, int t0) {
            constexpr int N = decltype(count)::value;
            floatx4 acc[N][4], mk[MASK ? N : 1][4];
            load_masks<N, MASK>(mk, a, a.mask + at, tile0 + t0, g);
            start_sums<N>(acc, bias, t0, g);
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int t = 0; t < N; ++t) {
                    const float av = w[((t0 + t) * KS + s) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[t][e] = mfma4(av, x[s][e], acc[t][e]);
                }
            store_sums<N, MASK>(acc, mk, a, a.y + at, tile0 + t0, g);
        };
        int t0 = 0;
        for (; t0 + 2 <= ntiles; t0 += 2) tiles(std::integral_constant<int, 2>{}, t0);
        if (t0 < ntiles) tiles(std::integral_constant<int, 1>{}, t0);
        if (!more) return;
        grp += stride;
        b = nb;
        px = npx;
#pragma unroll
        for (int s = 0; s < KS; ++s) x[s] = xn[s];
    }
}

// KB: input steps (of four maps) a wave loads together, one batch ahead of the multiplication
template <int MT, int KB, bool MASK>
__global__ __launch_bounds__(P1_THREADS, 2) void conv1x1_out_kernel(Conv1Args a)
{
    extern __shared__ float smem[];
    const int batches = (a.ksteps + KB - 1) / KB, ksteps = batches * KB;
    float *const w = smem, *const bias = w + MT * ksteps * 64;
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    stage_weights(w, a, 0, MT, ksteps);
    for (int q = threadIdx.x; q < MT * 16; q += P1_THREADS) bias[q] = a.bias && q < a.c_out ? a.bias[q] : 0.f;
    __syncthreads();
    const Groups groups{0, 0, a.n * a.per_image, a.per_image, a.plane};
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), stride = gridDim.x * P1_WAVES;
    auto load = [&](floatx4 (&x)[KB], int b, int px, int s0) {
        const float *src = a.x + (long)b * a.x_bstride + px + 4 * l16;
#pragma unroll
        for (int s = 0; s < KB; ++s) {
            const int c = 4 * (s0 + s) + g;
            x[s] = load4(src + (long)(c < a.c_in ? c : 0) * a.plane);
        }
    };
    int grp = blockIdx.x * P1_WAVES + wave, b, px;
    if (!groups.at(grp, b, px)) return;
    floatx4 x[KB], xn[KB];
    load(x, b, px, 0);
    while (true) {
        const long at = (long)b * a.c_out * a.plane + px + 4 * l16;
        floatx4 acc[MT][4], mk[MASK ? MT : 1][4];
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[t][e] = floatx4{0.f, 0.f, 0.f, 0.f};
        int nb = 0, npx = 0;
        const bool more = groups.at(grp + stride, nb, npx);
        for (int k = 0; k < batches; ++k) {
            if (k + 1 < batches) load(xn, b, px, (k + 1) * KB);
            else if (more) load(xn, nb, npx, 0);
#pragma unroll
            for (int s = 0; s < KB; ++s) {
                if (4 * (k * KB + s) + g >= a.c_in) x[s] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    const float av = w[(t * ksteps + k * KB + s) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[t][e] = mfma4(av, x[s][e], acc[t][e]);
                }
            }
#pragma unroll
            for (int s = 0; s < KB; ++s) x[s] = xn[s];
        }
        load_masks<MT, MASK>(mk, a, a.mask + at, 0, g);                      // (earlier they do not fit the registers)
#pragma unroll
        for (int t = 0; t < MT; ++t) {                                       // (the bias behind hundreds of products, where it rounds once)
            const floatx4 bb = *reinterpret_cast<const floatx4 *>(bias + t * 16 + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[t][e] += bb;
        }
        store_sums<MT, MASK>(acc, mk, a, a.y + at, 0, g);
        if (!more) return;
        grp += stride;
        b = nb;
        px = npx;
    }
}

// Fused head: h = ReLU(W1 x + b1), z = W2 h + b2, softmax.  A lane has hidden maps 4 g .. 4 g + 3 of every tile for its four pixels and adds
// their share of the class sums; the four lane groups' shares meet in two shuffles, and group g writes class g (and g + 4).
// 48 -> 200 -> 2 at 512^2: 73 -> 56 us; the matrix unit alone needs 35 and the staging of the weights five.
// POOL: the input is that of an SK pool of kernel 2 and stride a.pool in front of the head, whose maps are not stored.  The waves then
// walk the pixels with the pitch of the input rows, W + pool, so that the four samples of a window lie at fixed distances
// for any lane (pixels x >= W are computed and dropped: 1.5 % at 512^2); maxima in the order of the pool kernel.
// 48 maps at 512^2, d = 8: pool 22.7 + head 63.9 -> 79 us under the profiler, the forward pass 736 -> 726 us (the 96^2 net of 16 maps 22.6 -> 20.0,
// 4 x 900 x 1000 9.55 -> 8.44 ms with the first layer's pool).
template <int KS, int CL, bool POOL>
__global__ __launch_bounds__(P1_THREADS, 2) void head1x1_kernel(HeadArgs a, int per_image)
{
    extern __shared__ float smem[];
    const int tiles = (a.hidden + 15) / 16, plane = a.H * a.W;
    float *const w = smem, *const b1 = w + tiles * KS * 64, *const w2 = b1 + tiles * 16;      // w2: [CL][tiles * 16]
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    // (launch_pack_head_w1 packs [tile][step][lane] too, with a.ksteps steps)
    stage_fragments(w, tiles * KS, [&](int f) {
        const int t = f / KS, s = f - t * KS;
        const float v = static_cast<const float *>(a.w1p)[(t * a.ksteps + min(s, a.ksteps - 1)) * 64 + lane];
        return s < a.ksteps ? v : 0.f;
    });
    for (int q = threadIdx.x; q < tiles * 16; q += P1_THREADS) b1[q] = q < a.hidden ? a.b1[q] : 0.f;
    for (int q = threadIdx.x; q < CL * tiles * 16; q += P1_THREADS) {
        const int c = q / (tiles * 16), m = q - c * tiles * 16;
        w2[q] = c < a.classes && m < a.hidden ? a.w2[c * a.hidden + m] : 0.f;
    }
    __syncthreads();
    const int pitch = a.W + (POOL ? a.pool : 0), walk = POOL ? a.H * pitch - a.pool : plane;
    const long in_plane = POOL ? (long)(a.H + a.pool) * pitch : plane;
    const Groups groups{0, 0, a.n * per_image, per_image, walk};
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), stride = gridDim.x * P1_WAVES;
    auto load = [&](floatx4 (&x)[KS], int b, int px) {
        const float *src = static_cast<const float *>(a.x) + (long)b * a.c_in * in_plane + px + 4 * l16;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const float *p = src + (4 * s + g < a.c_in ? 4 * s + g : 0) * in_plane;
            x[s] = load4(p);
            if constexpr (POOL) {
                const floatx4 right = load4(p + a.pool), below = load4(p + (long)a.pool * pitch), corner = load4(p + (long)a.pool * pitch + a.pool);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float up = right[e] > x[s][e] ? right[e] : x[s][e], down = corner[e] > below[e] ? corner[e] : below[e];
                    x[s][e] = down > up ? down : up;
                }
            }
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
            if (4 * s + g >= a.c_in) x[s] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    int grp = blockIdx.x * P1_WAVES + wave, b, px;
    if (!groups.at(grp, b, px)) return;
    floatx4 x[KS], xn[KS];
    load(x, b, px);
    while (true) {
        int nb = 0, npx = 0;
        const bool more = groups.at(grp + stride, nb, npx);
        if (more) load(xn, nb, npx);
        float z[CL][4];
#pragma unroll
        for (int c = 0; c < CL; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) z[c][e] = 0.f;
        auto tile_group = [&](auto count, int t0) {
            constexpr int N = decltype(count)::value;
            floatx4 acc[N][4];
            start_sums<N>(acc, b1, t0, g);
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int t = 0; t < N; ++t) {
                    const float av = w[((t0 + t) * KS + s) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[t][e] = mfma4(av, x[s][e], acc[t][e]);
                }
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
                for (int c = 0; c < CL; ++c) {
                    const floatx4 ww = *reinterpret_cast<const floatx4 *>(w2 + (c * tiles + t0 + t) * 16 + 4 * g);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int r = 0; r < 4; ++r) z[c][e] += fmaxf(acc[t][e][r], 0.f) * ww[r];
                }
        };
        int t0 = 0;
        constexpr int GT = CL == 2 ? 4 : 2;                                  // (registers)
        for (; t0 + GT <= tiles; t0 += GT) tile_group(std::integral_constant<int, GT>{}, t0);
        if (GT > 2 && t0 + 2 <= tiles) {
            tile_group(std::integral_constant<int, 2>{}, t0);
            t0 += 2;
        }
        if (t0 < tiles) tile_group(std::integral_constant<int, 1>{}, t0);
        float m[4], sum[4];
#pragma unroll
        for (int c = 0; c < CL; ++c) {
            const float b2 = c < a.classes ? a.b2[c] : 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                z[c][e] += __shfl_xor(z[c][e], 16, 64);
                z[c][e] += __shfl_xor(z[c][e], 32, 64);
                z[c][e] += b2;
                m[e] = c == 0 ? z[c][e] : (c < a.classes ? fmaxf(m[e], z[c][e]) : m[e]);
            }
        }
#pragma unroll
        for (int c = 0; c < CL; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                z[c][e] = c < a.classes ? expf(z[c][e] - m[e]) : 0.f;
                sum[e] = c == 0 ? z[c][e] : sum[e] + z[c][e];
            }
        const int q = px + 4 * l16, row = POOL ? (int)((unsigned)q / (unsigned)pitch) : 0, col = POOL ? q - row * pitch : 0;
        float *dst = a.prob + (long)b * a.classes * plane + (POOL ? row * a.W + col : q);
#pragma unroll
        for (int c = 0; c < CL; ++c)
            if (c < a.classes && (c & 3) == g) {
                floatx4 p;
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = z[c][e] * (1.f / sum[e]);
                if (!POOL || col + 4 <= a.W) {
                    store4(dst + (long)c * plane, p);
                    continue;
                }
                // the end of a row: pixels up to W, then a gap of `pool`, then those of the next row (H*W of them in all)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (col + e < a.W) dst[(long)c * plane + e] = p[e];
                    else if (col + e >= pitch) dst[(long)c * plane + e - a.pool] = p[e];
                }
            }
        if (!more) return;
        grp += stride;
        b = nb;
        px = npx;
#pragma unroll
        for (int s = 0; s < KS; ++s) x[s] = xn[s];
    }
}

// Weight gradient of a 1x1 layer: D[r][s] = sum over pixels of R[r] S[s], where R is the side with more maps (RT tiles of 16) and S the other
// (at most three): of dY and X.  Both operands come from global memory as they are: lane (g, l16) loads pixels 4 g .. 4 g + 3 of map l16 of a
// tile, the operand of four K steps.  Eight waves, each with sums of its own, stride over blocks of 16 pixels and meet in LDS at the end; a
// workgroup writes one private copy, which wgrad_reduce_kernel adds up.  The sums of dY come along in registers.
// 48 -> 200 maps at 512^2, sums of dY and reduction included: 267 -> 142 us, 104 with a workgroup on every CU; 200 -> 2: 146 -> 45 (260 and 212 MB read; 8 x 512^2 2.2 ms -> 1.0,
// 1.04 -> 0.36).
constexpr int W1_WAVES = 8, W1_THREADS = 64 * W1_WAVES, W1_PX = 16, W1_ROUND = 4;

struct Wgrad1Args {
    const float *r, *s;
    float *scratch, *bias_part;            // bias_part[map * gridDim.x + workgroup] of dY, or nullptr
    int n, cr, cs, plane;
    int swap;                              // 0: R = dY (copy rows), S = X (copy columns); 1: the other way round
    int m_rows, ncols;                     // of a private copy [map of dY][map of X]
    int per_image, total;                  // blocks of pixels
};

// RT tiles of R a wave: 14 tiles at most as two halves (RG = 2), waves 4 .. 7 with the second one for the same pixels as waves 0 .. 3.  The
// tiles of the next block of pixels are loaded while this one's are multiplied, which 13 x 3 tiles of sums in one wave would leave no
// registers for (158 us instead of 142).
template <int RT, int CT, int RG>
__global__ __launch_bounds__(W1_THREADS, 2) void wgrad1x1_kernel(Wgrad1Args a)
{
    constexpr int GW = W1_WAVES / RG;                    // waves that share a half
    __shared__ floatx4 red[W1_WAVES][W1_ROUND][64];
    __shared__ float bred[W1_WAVES][(RT > CT ? RT : CT) * 16];
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = wave / GW, wi = wave % GW;
    floatx4 acc[RT][CT];
    float rsum[RT] = {}, ssum[CT] = {};
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // a tile's address is a uniform base and this lane's offset (bytes, checked by the launcher): one for whole tiles, one for the last
    // tile of either side, whose missing maps read the last one
    const int last_r = (a.cr - 1) / 16, last_s = (a.cs - 1) / 16;
    const unsigned whole = (unsigned)(l16 * a.plane + 4 * g) * 4u, end_r = (unsigned)(min(l16, a.cr - 1 - last_r * 16) * a.plane + 4 * g) * 4u,
                   end_s = (unsigned)(min(l16, a.cs - 1 - last_s * 16) * a.plane + 4 * g) * 4u;
    auto load = [&](floatx4 (&rv)[RT], floatx4 (&sv)[CT], int blk) {
        const int b = blk / a.per_image, px0 = (blk - b * a.per_image) * W1_PX;
        auto fetch = [&](const float *base, int maps, int last, unsigned end, int tile) {
            const int t = tile < last ? tile : last;
            const float *p = reinterpret_cast<const float *>(reinterpret_cast<const char *>(base + ((long)b * maps + t * 16) * a.plane + px0) +
                                                             (t == last ? end : whole));
            floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
            if (px0 + W1_PX <= a.plane) v = load4(p);                        // uniform
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (px0 + 4 * g + e < a.plane) v[e] = p[e];
            }
            return v;
        };
#pragma unroll
        for (int j = 0; j < CT; ++j) sv[j] = fetch(a.s, a.cs, last_s, end_s, j);
#pragma unroll
        for (int i = 0; i < RT; ++i) rv[i] = fetch(a.r, a.cr, last_r, end_r, half * RT + i);
    };
    int blk = blockIdx.x * GW + wi;
    const int stride = gridDim.x * GW;
    if (blk < a.total) {
        floatx4 rv[RT], sv[CT], rn[RT], sn[CT];
        load(rv, sv, blk);
        while (true) {
            const bool more = blk + stride < a.total;
            if (more) load(rn, sn, blk + stride);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < CT; ++j) acc[i][j] = mfma4(rv[i][e], sv[j][e], acc[i][j]);
                rsum[i] += (rv[i][0] + rv[i][1]) + (rv[i][2] + rv[i][3]);
            }
#pragma unroll
            for (int j = 0; j < CT; ++j) ssum[j] += (sv[j][0] + sv[j][1]) + (sv[j][2] + sv[j][3]);
            if (!more) break;
            blk += stride;
#pragma unroll
            for (int i = 0; i < RT; ++i) rv[i] = rn[i];
#pragma unroll
            for (int j = 0; j < CT; ++j) sv[j] = sn[j];
        }
    }
    // the sums of the waves of a half, W1_ROUND tiles a round; wave wi < W1_ROUND adds tile wi of the round and writes it
    float *const copy = a.scratch + (long)blockIdx.x * a.m_rows * a.ncols;
#pragma unroll
    for (int t0 = 0; t0 < RT * CT; t0 += W1_ROUND) {
        __syncthreads();
#pragma unroll
        for (int t = t0; t < t0 + W1_ROUND && t < RT * CT; ++t) red[wave][t - t0][lane] = acc[t / CT][t % CT];
        __syncthreads();
        const int t = t0 + wi;
        if (wi < W1_ROUND && t < RT * CT) {
            floatx4 v = red[half * GW][wi][lane];
#pragma unroll
            for (int w = 1; w < GW; ++w) v += red[half * GW + w][wi][lane];
            const int i = t / CT, j = t - i * CT, row = (half * RT + i) * 16 + 4 * g, col = j * 16 + l16;     // maps of R and of S
            if (a.swap) {
                if (col < a.m_rows && row < a.ncols) *reinterpret_cast<floatx4 *>(copy + (long)col * a.ncols + row) = v;
            } else if (col < a.ncols) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row + r < a.m_rows) copy[(long)(row + r) * a.ncols + col] = v[r];
            }
        }
    }
    if (!a.bias_part) return;
    auto sums = [&](float v, int tile) {                 // of a tile's 16 maps over the four lane groups
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (g == 0) bred[wave][tile * 16 + l16] = v;
    };
    if (a.swap) {
#pragma unroll
        for (int j = 0; j < CT; ++j) sums(ssum[j], j);
    } else {
#pragma unroll
        for (int i = 0; i < RT; ++i) sums(rsum[i], i);
    }
    __syncthreads();
    const int maps = a.swap ? a.cs : a.cr;               // (S is the same in both halves)
    for (int o = threadIdx.x; o < maps; o += W1_THREADS) {
        const int h = a.swap ? 0 : o / (RT * 16), at = o - h * (RT * 16);
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < GW; ++w) v += bred[h * GW + w][at];
        a.bias_part[(long)o * gridDim.x + blockIdx.x] = v;
    }
}

int device_cus()
{
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    return cus;
}

template <class K> hipError_t allow_lds(K kernel, bool &done)
{
    if (done) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    done = e == hipSuccess;
    return e;
}

// two workgroups of four waves a CU (one where the weights leave room for one), no more than there are pixel groups
int p1_blocks(int groups, size_t smem)
{
    const int per_cu = smem <= 80 * 1024 ? 2 : 1;
    return std::max(1, std::min((groups + P1_WAVES - 1) / P1_WAVES, per_cu * device_cus()));
}

template <int KS>
hipError_t launch_in(Conv1Args a, hipStream_t stream)
{
    // where the pixel groups are too few to give every SIMD two waves, the output maps are shared out as well
    const int groups = a.n * a.per_image, split = std::max(1, std::min(a.tiles, 8 * device_cus() / groups));
    a.tiles_per = (a.tiles + split - 1) / split;
    const size_t smem = sizeof(float) * ((size_t)a.tiles_per * KS * 64 + a.tiles_per * 16);
    static bool set[2];
    const dim3 blocks(p1_blocks(groups, smem), (a.tiles + a.tiles_per - 1) / a.tiles_per);
    hipError_t e = a.mask ? allow_lds(&conv1x1_in_kernel<KS, true>, set[1]) : allow_lds(&conv1x1_in_kernel<KS, false>, set[0]);
    if (e != hipSuccess) return e;
    if (a.mask) hipLaunchKernelGGL((conv1x1_in_kernel<KS, true>), blocks, dim3(P1_THREADS), smem, stream, a);
    else hipLaunchKernelGGL((conv1x1_in_kernel<KS, false>), blocks, dim3(P1_THREADS), smem, stream, a);
    return hipGetLastError();
}

constexpr int P1_KB = 5;

template <int MT>
hipError_t launch_out(const Conv1Args &a, hipStream_t stream)
{
    const int ksteps = (a.ksteps + P1_KB - 1) / P1_KB * P1_KB;
    const size_t smem = sizeof(float) * ((size_t)MT * ksteps * 64 + MT * 16);
    static bool set[2];
    const int blocks = p1_blocks(a.n * a.per_image, smem);
    hipError_t e = a.mask ? allow_lds(&conv1x1_out_kernel<MT, P1_KB, true>, set[1]) : allow_lds(&conv1x1_out_kernel<MT, P1_KB, false>, set[0]);
    if (e != hipSuccess) return e;
    if (a.mask) hipLaunchKernelGGL((conv1x1_out_kernel<MT, P1_KB, true>), dim3(blocks), dim3(P1_THREADS), smem, stream, a);
    else hipLaunchKernelGGL((conv1x1_out_kernel<MT, P1_KB, false>), dim3(blocks), dim3(P1_THREADS), smem, stream, a);
    return hipGetLastError();
}

template <int KS, int CL, bool POOL>
hipError_t launch_head_cl(const HeadArgs &a, hipStream_t stream)
{
    const int tiles = (a.hidden + 15) / 16, per_image = ((POOL ? a.H * (a.W + a.pool) - a.pool : a.H * a.W) + P1_PX - 1) / P1_PX;
    const size_t smem = sizeof(float) * ((size_t)tiles * KS * 64 + (size_t)tiles * 16 * (1 + CL));
    static bool set;
    const hipError_t e = allow_lds(&head1x1_kernel<KS, CL, POOL>, set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((head1x1_kernel<KS, CL, POOL>), dim3(p1_blocks(a.n * per_image, smem)), dim3(P1_THREADS), smem, stream, a, per_image);
    return hipGetLastError();
}

template <int KS>
hipError_t launch_head_ks(const HeadArgs &a, hipStream_t stream)
{
    if (a.pool) return a.classes <= 2 ? launch_head_cl<KS, 2, true>(a, stream) : launch_head_cl<KS, 4, true>(a, stream);
    if (a.classes <= 2) return launch_head_cl<KS, 2, false>(a, stream);
    if (a.classes <= 4) return launch_head_cl<KS, 4, false>(a, stream);
    return launch_head_cl<KS, 8, false>(a, stream);
}

template <int RT, int CT, int RG>
hipError_t launch_w1(const Wgrad1Args &a, int blocks, hipStream_t stream)
{
    hipLaunchKernelGGL((wgrad1x1_kernel<RT, CT, RG>), dim3(blocks), dim3(W1_THREADS), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

// plain 1x1 layers: whole planes in and out, at least 64 pixels, few maps on one side, the weights within the LDS
bool conv1x1_f32_supported(const ConvF32Args &a)
{
    if (a.k != 1 || a.in_off != 0 || a.tap_maps || a.accumulate || a.grp_maps || a.H != a.Ho || a.W != a.Wo || a.OH != a.Ho || a.OW != a.Wo ||
        a.o_off != 0 || a.out_maps != a.c_out || a.oy_mul != 1 || a.ox_mul != 1 || a.oy_off != 0 || a.ox_off != 0 || a.n < 1)
        return false;
    const long plane = (long)a.Ho * a.Wo;
    if (plane < P1_PX || plane > 0x3fffffffL || a.n * ((plane + P1_PX - 1) / P1_PX) > 0x3fffffffL) return false;
    const int tiles = (a.c_out + 15) / 16, ksteps = (a.c_in + 3) / 4;
    return (a.c_in <= 48 || tiles <= 3) && (long)tiles * (ksteps + P1_KB) * 256 + tiles * 64 <= 150 * 1024;
}

hipError_t launch_conv1x1_f32(const ConvF32Args &c, hipStream_t stream)
{
    if (!conv1x1_f32_supported(c)) return hipErrorInvalidValue;
    Conv1Args a;
    a.x = c.x; a.wp = c.wp; a.bias = c.bias; a.mask = c.mask; a.y = c.y;
    a.plane = c.Ho * c.Wo;
    a.x_bstride = c.x_bstride ? c.x_bstride : (long)c.c_in * a.plane;
    a.n = c.n; a.c_in = c.c_in; a.c_out = c.c_out; a.n_pad = c.n_pad; a.relu = c.relu;
    a.tiles = (c.c_out + 15) / 16;
    a.ksteps = (c.c_in + 3) / 4;
    a.per_image = (a.plane + P1_PX - 1) / P1_PX;
    // the side with fewer maps stays in registers
    if (a.tiles > 3 || (c.c_in <= 48 && c.c_in <= c.c_out)) {
        if (a.ksteps <= 1) return launch_in<1>(a, stream);
        if (a.ksteps <= 2) return launch_in<2>(a, stream);
        if (a.ksteps <= 4) return launch_in<4>(a, stream);
        if (a.ksteps <= 6) return launch_in<6>(a, stream);
        if (a.ksteps <= 8) return launch_in<8>(a, stream);
        return launch_in<12>(a, stream);
    }
    if (a.tiles == 1) return launch_out<1>(a, stream);
    if (a.tiles == 2) return launch_out<2>(a, stream);
    return launch_out<3>(a, stream);
}

// Here a wave takes 64 pixels through all hidden tiles, head_fused_kernel 16 or 32: with many hidden tiles it needs enough pixels, and with
// few input maps the class sums outweigh the product.  42 heads of 8 to 48 -> 16 to 200 -> 2 to 5 on 12 x 60 to 8 x 512^2, both in turn: up to
// four hidden tiles 1.01 to 1.97 times as fast here; 7 and 13 tiles 0.62 to 0.93 below 1024 groups of pixels (48 -> 200 -> 2 on 2 x 82 x 152:
// 15.2 us there, 17.2 here) but for three of 1.07 to 1.22, 0.76 at 8 input maps, 1.07 to 1.34 from there on.
bool head1x1_f32_supported(const HeadArgs &a)
{
    const long plane = (long)a.H * a.W, groups = a.n * ((plane + P1_PX - 1) / P1_PX);
    if (a.pool < 0 || (a.pool > 0 && (a.classes > 4 || a.W < 4 || (plane + (long)a.H * a.pool) * a.n > 0x3fffffffL))) return false;
    return a.dtype == 0 && a.hd == 0 && a.c_in <= 48 && a.classes <= 8 && plane >= P1_PX && a.hidden <= 256 &&
           (a.hidden <= 64 || (groups >= 4L * device_cus() && a.c_in > 8));
}

hipError_t launch_head1x1_f32(const HeadArgs &a, hipStream_t stream)
{
    if (!head1x1_f32_supported(a)) return hipErrorInvalidValue;
    if (a.ksteps <= 2) return launch_head_ks<2>(a, stream);
    if (a.ksteps <= 4) return launch_head_ks<4>(a, stream);
    if (a.ksteps <= 6) return launch_head_ks<6>(a, stream);
    if (a.ksteps <= 8) return launch_head_ks<8>(a, stream);
    return launch_head_ks<12>(a, stream);
}

// One side at most 48 maps, the other at most 208: 13 of the 14 tiles that two halves of seven hold; beyond, other kernels were not compared.
bool wgrad1x1_f32_supported(int c_in, int c_out, int n, long plane)
{
    const int hi = std::max(c_in, c_out), lo = std::min(c_in, c_out);
    return lo >= 1 && lo <= 48 && hi <= 208 && plane <= 0x3ffffffL &&       // (offsets inside a tile of 16 maps are 32 bits)
           n * ((plane + W1_PX - 1) / W1_PX) <= 0x3fffffffL;
}

hipError_t launch_wgrad1x1_f32(const float *x, const float *dy, float *scratch, float *bias_part, int n, int c_in, long plane, int c_out,
                               int max_copies, int *copies, hipStream_t stream)
{
    if (!wgrad1x1_f32_supported(c_in, c_out, n, plane) || n < 1 || plane < 1 || max_copies < 1) return hipErrorInvalidValue;
    Wgrad1Args a;
    a.swap = c_in > c_out;
    a.r = a.swap ? x : dy;
    a.s = a.swap ? dy : x;
    a.cr = a.swap ? c_in : c_out;
    a.cs = a.swap ? c_out : c_in;
    a.scratch = scratch; a.bias_part = bias_part; a.n = n; a.plane = (int)plane;
    a.m_rows = (c_out + 15) / 16 * 16;
    a.ncols = (c_in + 15) / 16 * 16;
    a.per_image = (int)((plane + W1_PX - 1) / W1_PX);
    a.total = n * a.per_image;
    const int rt = (a.cr + 15) / 16, ct = (a.cs + 15) / 16;
    // eight waves a CU (they have the next pixels on the way while they multiply; a second workgroup would double the copies)
    const int rg = rt > 7 ? 2 : 1;
    *copies = std::max(1, std::min(std::min(max_copies, device_cus()), (a.total + W1_WAVES / rg - 1) / (W1_WAVES / rg)));
#define SK_W1_CASE(R, C, G) if (ct == C) return launch_w1<R, C, G>(a, *copies, stream);
    if (rt <= 3) { SK_W1_CASE(3, 1, 1) SK_W1_CASE(3, 2, 1) SK_W1_CASE(3, 3, 1) }
    else if (rt <= 7) { SK_W1_CASE(7, 1, 1) SK_W1_CASE(7, 2, 1) SK_W1_CASE(7, 3, 1) }
    else { SK_W1_CASE(7, 1, 2) SK_W1_CASE(7, 2, 2) SK_W1_CASE(7, 3, 2) }
#undef SK_W1_CASE
    return hipErrorInvalidValue;
}

}  // namespace sk
