// SK (dilated) convolution for fp32 activations on the 16-bit matrix unit of gfx950: 3x3 and 4x4 layers and their data gradients.
//
// The 16-bit unit is sixteen times as fast as its fp32 form.  Samples and weights are pairs of fp16 values (split_f32.h), a product is three
// MFMAs, so the unit needs 3/16 of the time; memory holds fp32 as before.  A workgroup of four waves owns 16 WX columns of 4 R / WX rows
// that lie d apart (as in kernels_conv_f32.hip, their kernel rows fall on few input rows).  Per chunk of eight input maps it
//  - loads its samples into registers while it multiplies the chunk before,
//  - finds their largest and least magnitude (one LDS exchange).  The power of two that scales them follows from the largest; where it has to move
//    (there are three bits of room), the sums so far follow it.  Weights have one for each output map,
//  - writes the pairs to LDS as units of one pixel's eight maps: a B operand is 16 pixels x (4 kernel columns x 8 maps), one 16-byte read a
//    lane, as in the 16-bit convolution; the fourth column of a 3x3 kernel has zero weights,
//  - multiplies kernel rows in steps of G whose weights are in registers, so that a staged row is read once for G kernel rows.  Weight
//    fragments come straight into LDS, a step ahead.
// A tile that meets a sample or a weight that pairs would hold in fewer bits (infinite, or not zero and more than 2^28 to 2^31 below the chunk's or the
// output map's largest: one chunk in thirty thousand of normal samples) starts again on the fp32 matrix unit, unscaled.
// What bounds it: MFMAs take 0.42 of the time at 2.4 GHz (8 x 1024^2; such load lowers the clock); the rest are the two barriers a chunk, LDS reads and
// one other vector instruction an MFMA.  Two workgroups share a CU and fill each other's waits (three did with one sum instead of two, which held
// 2^-37 of the tile's largest: 59 us at 537^2).
// 48 -> 48 maps, 4x4, us (TFLOP/s) on the fp32 matrix unit and here: 537^2 d = 2 216 -> 69 (301), 8 x 1024^2 d = 8 4775 -> 1676 (352); 64 -> 64, 3x3,
// 566^2 234 -> 92.  With every tile sent to the fp32 unit 537^2 takes 242; seven such layers 0.95 to 1.25 of conv_f32_pf_kernel.
// Tried: three bf16 parts and six products (exact parts, no scale) 537^2 113 us, its sums rounded six times a step 1.2 times as far off as
// fp32 operands; the second sum added to the first by the vector unit after each step: 72 us; a wide chunk alone on the fp32 unit and the next as pairs
// again: the compiler keeps two copies of the sums, 15 % slower; both staged chunks in LDS: no gain; four pixels a load: a tenth slower (bank
// conflicts of the writes); 64-bit addresses in loads and stores, which were as many vector instructions as all others: a tenth slower.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lds_dma.h"
#include "sk_kernels.h"
#include "split_f32.h"

namespace sk {

typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace {

// KS x KS kernels; MT tiles of sixteen output maps; a wave owns R output rows of sixteen columns, WX waves lie side by side and 4 / WX one
// above the other; PITCH: staged columns
template <int KS, int MT, int R, int WX, int PITCH> struct SplitTile {
    static constexpr int TX = 16 * WX, RT = R * (4 / WX);    // output columns and rows of a tile
    static constexpr int RR = RT + KS - 1;                   // staged rows
    static constexpr int G = KS == 4 ? 2 : KS;               // kernel rows of a step, whose weights are in registers together
    static constexpr int STEPS = KS / G;
    static constexpr int PLANE = RR * PITCH;                 // 16-byte units of one staged part
    static constexpr int UPT = (PLANE + 255) / 256;          // units a thread stages
    static constexpr int WSTEP = G * MT * 2 * 1024;          // bytes of a step's weight fragments
    static constexpr size_t SMEM = (size_t)2 * PLANE * 16 + 2 * WSTEP + 64;       // (64: ranges)
    static_assert(KS % G == 0, "whole steps");
};

// base + a 32-bit offset of the lane + one of the wave: no vector arithmetic, where a pointer costs a 64-bit addition per access.  What lies at
// SPLIT_NOWHERE is not read or written
constexpr unsigned SPLIT_NOWHERE = 0xfffffff0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t split_rsrc(const void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, SPLIT_NOWHERE, 0x00027000);
}

// (acc + low / 2^12) * 2^-(se + the output map's power of two), bias, ReLU and stores of R rows d apart from oy on, lane column ox, maps o_first + 4 g ..  MODE 1: where the mask is positive;
// 2: added to what y holds.  Masks and old values are read ahead of the first store (one queue holds loads and stores).
template <int MT, int R, int MODE>
__device__ __forceinline__ void split_store(const ConvF32Args &a, const floatx4 (&acc)[R][MT], const floatx4 (&low)[R][MT], int se, const int *wexp,
                                            int b, int o_first, int oy, int ox, int g)
{
    const long oplane = (long)a.OH * a.OW;                         // below 2^26: offsets inside sixteen maps are 32-bit
    const long first = ((long)b * a.out_maps + a.o_off + o_first) * oplane;
    unsigned at[MT][4];
    float bia[MT][4];
    int down[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int o = o_first + 16 * m + 4 * g + r4;
            at[m][r4] = ox < a.Wo && o < a.c_out ? 4u * ((unsigned)(4 * g + r4) * (unsigned)oplane + (unsigned)(ox * a.ox_mul + a.ox_off)) : SPLIT_NOWHERE;
            bia[m][r4] = a.bias ? a.bias[min(o, a.n_pad - 1)] : 0.f;
            down[m][r4] = wexp ? -(se + wexp[min(o, a.n_pad - 1)]) : 0;          // (none: sums as they are)
        }
    const auto row = [&](int y) { return 4u * (unsigned)(((oy + y * a.d) * a.oy_mul + a.oy_off) * a.OW); };
    float old[R][MT][4];
    if constexpr (MODE != 0) {
#pragma unroll
        for (int y = 0; y < R; ++y) {
            if (oy + y * a.d >= a.Ho) break;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const auto r = split_rsrc((MODE == 1 ? a.mask : a.y) + first + (long)(16 * m) * oplane);
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) old[y][m][r4] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, at[m][r4], row(y), 0));
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int y = 0; y < R; ++y) {
        if (oy + y * a.d >= a.Ho) break;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const auto r = split_rsrc(a.y + first + (long)(16 * m) * oplane);
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                float v = __builtin_ldexpf(split_sum(acc[y][m][r4], low[y][m][r4]), down[m][r4]) + bia[m][r4];
                if constexpr (MODE == 2) v += old[y][m][r4];
                if (a.relu) v = fmaxf(v, 0.f);
                if constexpr (MODE == 1) v = old[y][m][r4] > 0.f ? v : 0.f;
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, at[m][r4], row(y), 0);
            }
        }
    }
}

template <int KS, int MT, int R, int WX, int PITCH, bool PADZ>
__global__ __launch_bounds__(256, 2) void conv_split_f32_kernel(ConvF32Args a, const unsigned char *wsp, const int *wexp, const int *wwide, int m_tiles,
                                                                int tiles_hi, int tiles_lo, int rem, int nblocks, int gx, int gy, int total, int per_xcd)
{
    using T = SplitTile<KS, MT, R, WX, PITCH>;
    constexpr int RR = T::RR, G = T::G, STEPS = T::STEPS, UPT = T::UPT, PLANE = T::PLANE;
    extern __shared__ unsigned char smem[];
    unsigned char *xs = smem, *ws = smem + 2 * PLANE * 16;
    unsigned *ranges = reinterpret_cast<unsigned *>(ws + 2 * T::WSTEP);      // [2][most, least][4]: of what each wave stages, by chunk
    const int d = a.d, pw = T::TX + (KS - 1) * d, units = RR * pw;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wx = wave % WX, wy = wave / WX;

    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= total) return;
    const int bx = tile % gx, byz = tile / gx;
    const int by = byz % gy, bz = byz / gy;
    int py, ty;
    if (by < rem * tiles_hi) {
        py = by / tiles_hi;
        ty = by - py * tiles_hi;
    } else {
        const int b2 = by - rem * tiles_hi;
        py = rem + b2 / tiles_lo;
        ty = b2 % tiles_lo;
    }
    const int b = bz / nblocks, nb = bz - b * nblocks;
    const int x0 = bx * T::TX, tile0 = nb * MT;

    floatx4 acc[R][MT], low[R][MT];                           // sums of h h' and of h l' + l h'
#pragma unroll
    for (int y = 0; y < R; ++y)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[y][m] = low[y][m] = floatx4{0.f, 0.f, 0.f, 0.f};

    const long plane = (long)a.H * a.W;
    const float *xb = a.x + (long)b * (a.x_bstride ? a.x_bstride : (long)a.c_in * plane);
    const int nchunks = (a.c_in + 7) / 8;

    // the units (pixel, eight maps) that this thread stages: byte offset inside a map, LDS address, whether the pixel lies in the image
    unsigned off[UPT];
    int dst[UPT];
    bool ok[UPT];
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
        const int u = min(tid + 256 * q, units - 1);
        const int t = u / pw, c = u - t * pw;
        int iy = py + d * (ty * T::RT + t) - a.in_off, ix = x0 + c - a.in_off;
        ok[q] = iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
        iy = min(max(iy, 0), a.H - 1);
        ix = min(max(ix, 0), a.W - 1);
        off[q] = 4u * (unsigned)(iy * a.W + ix);
        dst[q] = (t * PITCH + c) * 16;
    }
    const int grp_chunks = a.grp_maps > 0 ? a.grp_maps / 8 : 0x7fffffff;
    int pf_left = grp_chunks;
    long pf_skip = 0;
    float xr[UPT][8];
    auto prefetch = [&](int chunk) {
        // (the compiler does not see that these are the same in every lane)
        const unsigned long at = (unsigned long)(xb + pf_skip + (long)chunk * 8 * plane);
        const unsigned at_lo = __builtin_amdgcn_readfirstlane((unsigned)at), at_hi = __builtin_amdgcn_readfirstlane((unsigned)(at >> 32));
        const float *const maps = reinterpret_cast<const float *>((unsigned long)at_hi << 32 | at_lo);
        const int last = __builtin_amdgcn_readfirstlane(a.c_in - 1 - chunk * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const auto src = split_rsrc(maps + (long)min(e, last) * plane);
#pragma unroll
            for (int q = 0; q < UPT; ++q) xr[q][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(src, off[q], 0, 0));
        }
        if (--pf_left == 0) {
            pf_left = grp_chunks;
            pf_skip += a.grp_skip;
        }
    };
    // the scale of the samples: 2^se; it moves where they are larger or much smaller than those before.  `first` is the first one
    int se = SPLIT_MOST, first = 2 * SPLIT_MOST, wide_weights = 0;
    bool pairs = true;                                        // false from the first chunk on that pairs cannot hold
    const auto *const flags = reinterpret_cast<const __attribute__((address_space(4))) int *>(reinterpret_cast<size_t>(wwide));     // (scalar loads)
    auto measure = [&](int chunk) {
        wide_weights = 0;
#pragma unroll
        for (int m = 0; m < MT; ++m) wide_weights |= flags[chunk * m_tiles + min(tile0 + m, m_tiles - 1)];
        SplitRange r;
#pragma unroll
        for (int q = 0; q < UPT; ++q) r = split_range(r, split_range(xr[q]));
        r = split_wave_range(r);
        if (lane == SPLIT_LAST_LANE) {
            ranges[(chunk & 1) * 8 + wave] = r.most;
            ranges[(chunk & 1) * 8 + 4 + wave] = r.least;
        }
    };
    // The scale for a chunk's samples, or SPLIT_WIDE: pairs don't hold them, or the scaled sums would leave fp32's range
    auto scale_chunk = [&](int chunk) {
        const uint4v m4 = *reinterpret_cast<const uint4v *>(ranges + (chunk & 1) * 8), l4 = *reinterpret_cast<const uint4v *>(ranges + (chunk & 1) * 8 + 4);
        const SplitRange r{(unsigned)__builtin_amdgcn_readfirstlane((int)max(max(m4[0], m4[1]), max(m4[2], m4[3]))),
                           (unsigned)__builtin_amdgcn_readfirstlane((int)max(max(l4[0], l4[1]), max(l4[2], l4[3])))};
        const int need = split_exponent(r.most, 14), to = split_exponent(r.most, 13);      // a bit of room: neighbouring chunks don't ask again
        const bool move = r.most > 0 && (need < se || need > se + 2);
        const int next = move ? to : se;
        first = first > SPLIT_MOST && r.most > 0 ? next : first;
        const bool wide = wide_weights || split_wide(r, next) || (move && (to - first > 60 || first - to > 60));
        return __builtin_amdgcn_readfirstlane(wide ? SPLIT_WIDE : next);      // (the compiler does not see that it is uniform)
    };
    auto move_scale = [&](int to) {
        if (to != se) {
            const float f = to - se < -126 ? 0.f : split_pow2(to - se);      // (less: from the start, where sums are zero)
#pragma unroll
            for (int y = 0; y < R; ++y)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    acc[y][mt] *= f;
                    low[y][mt] *= f;
                }
        }
        se = to;
    };
    auto commit = [&]() {
        const float scale = split_pow2(se);
#pragma unroll
        for (int q = 0; q < UPT; ++q) {
            if (256 * q + 255 >= RR * (T::TX + KS - 1) && tid + 256 * q >= units) continue;
            uint4v p[2];
            split2(xr[q], scale, p);
            if constexpr (PADZ)
                if (!ok[q]) p[0] = p[1] = uint4v{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 2; ++s) *reinterpret_cast<uint4v *>(xs + s * PLANE * 16 + dst[q]) = p[s];
        }
    };
    // fragments [chunk][kernel row][map tile][part] of 1 KB; a step's stand in LDS as [kernel row][MT][part]
    auto load_weights = [&](int chunk, int step, int buf) {
        const unsigned char *src = wsp + (long)(chunk * KS + step * G) * m_tiles * 2048 + lane * 16;
#pragma unroll
        for (int f = 0; f < G * MT * 2; f += 4) {
            const int fw = f + wave;
            if (G * MT * 2 % 4 == 0 || fw < G * MT * 2) {
                const int i = fw / (MT * 2), m = min(tile0 + fw / 2 % MT, m_tiles - 1);
                lds_dma16(src + ((i * m_tiles + m) * 2 + (fw & 1)) * 1024, ws + buf * T::WSTEP + fw * 1024);
            }
        }
    };
    const bool idle = x0 + wx * 16 >= a.Wo;                   // this wave's columns lie right of the image
    const unsigned char *xp = xs + (wy * R * PITCH + wx * 16 + l16 + min(g, KS - 1) * d) * 16;     // the column behind a 3x3 kernel meets zero weights

    int chunk = 0;
    load_weights(0, 0, 0);
    prefetch(0);
    measure(0);
    for (; chunk < nchunks; ++chunk) {
        const bool more = chunk + 1 < nchunks;
        wide_barrier();                                       // every wave is done with the staged maps and has measured its share of the next
        const int scale = scale_chunk(chunk);
        pairs = scale != SPLIT_WIDE;
        if (!pairs) break;
        move_scale(scale);
        commit();
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            // the step's weights have arrived: behind them only the loads of the next chunk's maps may be under way
            if (s == 1 && more) wide_wait<8 * UPT>();
            else wide_wait<0>();
            wide_barrier();
            const int buf = (STEPS & 1) ? ((chunk + s) & 1) : (s & 1);
            if (s + 1 < STEPS) load_weights(chunk, s + 1, buf ^ 1);
            else if (more) load_weights(chunk + 1, 0, buf ^ 1);
            if (s == 0 && more) prefetch(chunk + 1);
            if (!idle) {
                const unsigned char *wb = ws + buf * T::WSTEP + lane * 16, *xq = xp + s * G * PITCH * 16;
                uint4v A[G][MT][2], B[2][2];
                auto fetch = [&](int r) {
#pragma unroll
                    for (int p = 0; p < 2; ++p) B[r & 1][p] = *reinterpret_cast<const uint4v *>(xq + (p * PLANE + r * PITCH) * 16);
                };
                fetch(0);
#pragma unroll
                for (int i = 0; i < G; ++i)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
#pragma unroll
                        for (int p = 0; p < 2; ++p) A[i][m][p] = *reinterpret_cast<const uint4v *>(wb + ((i * MT + m) * 2 + p) * 1024);
#pragma unroll
                for (int r = 0; r < R + G - 1; ++r) {             // staged row r is kernel row i of output row r - i
                    if (r + 1 < R + G - 1) fetch(r + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int PA[3] = {1, 0, 0}, PB[3] = {0, 0, 1};
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int i = 0; i < G; ++i) {
                            const int y = r - i;
                            if (y < 0 || y >= R) continue;
#pragma unroll
                            for (int m = 0; m < MT; ++m) {
                                floatx4 &sum = q == 1 ? acc[y][m] : low[y][m];
                                sum = split_mfma(A[i][m][PA[q]], B[r & 1][PB[q]], sum);
                            }
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (more) measure(chunk + 1);
    }
    if (!pairs) {
        // All of it on the fp32 matrix unit: the LDS of a unit's two parts holds its eight samples as they are, weights come from their fp32 form.  Only
        // taps and maps that exist are multiplied: 0 * inf is NaN
        wide_wait<0>();                                       // weights on their way to LDS
#pragma unroll
        for (int y = 0; y < R; ++y)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[y][m] = low[y][m] = floatx4{0.f, 0.f, 0.f, 0.f};
        pf_left = grp_chunks;
        pf_skip = 0;
        chunk = 0;
        prefetch(0);
        while (true) {
#pragma unroll
            for (int q = 0; q < UPT; ++q) {
                if (256 * q + 255 >= RR * (T::TX + KS - 1) && tid + 256 * q >= units) continue;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    floatx4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = chunk * 8 + 4 * h + e < a.c_in && (!PADZ || ok[q]) ? xr[q][4 * h + e] : 0.f;
                    *reinterpret_cast<floatx4 *>(xs + h * PLANE * 16 + dst[q]) = v;
                }
            }
            wide_barrier();
            if (chunk + 1 < nchunks) prefetch(chunk + 1);
            if (!idle) {
                const float *wf = a.wp + (long)(chunk * 8 + g) * (KS * KS) * a.n_pad + l16;
#pragma unroll 2
                for (int t = 0; t < 2 * KS; ++t) {
                    const int h = t >= KS, i = t - h * KS;
                    const float *xq = reinterpret_cast<const float *>(xs + (h * PLANE + (wy * R + i) * PITCH + wx * 16 + l16) * 16) + g;
                    float A[KS][MT];
#pragma unroll
                    for (int j = 0; j < KS; ++j)
#pragma unroll
                        for (int m = 0; m < MT; ++m) A[j][m] = wf[(long)((h * 4 * KS + i) * KS + j) * a.n_pad + min(tile0 + m, m_tiles - 1) * 16];
#pragma unroll
                    for (int j = 0; j < KS; ++j)
#pragma unroll
                        for (int y = 0; y < R; ++y) {
                            const float B = xq[(y * PITCH + j * d) * 4];
#pragma unroll
                            for (int m = 0; m < MT; ++m) acc[y][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[j][m], B, acc[y][m], 0, 0, 0);
                        }
                }
            }
            if (++chunk == nchunks) break;
            wide_barrier();                                   // every wave is done with the staged maps
        }
    }
    if (idle) return;
    const int o_first = tile0 * 16, oy = py + d * (ty * T::RT + wy * R), ox = x0 + wx * 16 + l16;
    const int *we = pairs ? wexp : nullptr;
    if (a.mask) split_store<MT, R, 1>(a, acc, low, se, we, b, o_first, oy, ox, g);
    else if (a.accumulate) split_store<MT, R, 2>(a, acc, low, se, we, b, o_first, oy, ox, g);
    else split_store<MT, R, 0>(a, acc, low, se, we, b, o_first, oy, ox, g);
}

template <int KS, int MT, int R, int WX, int PITCH, bool PADZ>
hipError_t launch_split_t(const ConvF32Args &a, hipStream_t stream)
{
    using T = SplitTile<KS, MT, R, WX, PITCH>;
    static_assert(T::SMEM <= 81920, "two workgroups share a CU");
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_split_f32_kernel<KS, MT, R, WX, PITCH, PADZ>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::SMEM);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int q = a.Ho / a.d, rem = a.Ho % a.d;
    const int tiles_hi = (q + 1 + T::RT - 1) / T::RT, tiles_lo = (q + T::RT - 1) / T::RT;
    const long gy = (long)rem * tiles_hi + (long)(a.d - rem) * tiles_lo;
    const int m_tiles = a.n_pad / 16, nblocks = (m_tiles + MT - 1) / MT, gx = (a.Wo + T::TX - 1) / T::TX;
    const long total = gx * gy * a.n * nblocks;
    if (total <= 0 || total > 0x7ffffff0L) return hipErrorInvalidValue;
    const int per_xcd = (int)((total + 7) / 8);
    const float *tail = a.wp + split_tail_at(KS, a.c_in, a.n_pad);
    hipLaunchKernelGGL((conv_split_f32_kernel<KS, MT, R, WX, PITCH, PADZ>), dim3(per_xcd * 8), dim3(256), T::SMEM, stream, a,
                       reinterpret_cast<const unsigned char *>(a.wp + split_weights_at(KS, a.c_in, a.n_pad)),
                       reinterpret_cast<const int *>(tail + SPLIT_PARTS * a.n_pad), reinterpret_cast<const int *>(tail + (SPLIT_PARTS + 1) * a.n_pad), m_tiles,
                       tiles_hi, tiles_lo > 0 ? tiles_lo : 1, rem, nblocks, gx, (int)gy, (int)total, per_xcd);
    return hipGetLastError();
}

template <int KS, int MT, int R, int WX, bool PADZ> hipError_t launch_split_d(const ConvF32Args &a, hipStream_t stream)
{
    constexpr int TX = 16 * WX;
    const int halo = (KS - 1) * a.d;
    if (halo <= 8) return launch_split_t<KS, MT, R, WX, TX + 8, PADZ>(a, stream);
    if (halo <= 16) return launch_split_t<KS, MT, R, WX, TX + 16, PADZ>(a, stream);
    return launch_split_t<KS, MT, R, WX, TX + 24, PADZ>(a, stream);
}

template <int KS, int MT, int R, int WX> hipError_t launch_split_p(const ConvF32Args &a, hipStream_t stream)
{
    if (a.in_off != 0) return launch_split_d<KS, MT, R, WX, true>(a, stream);
    return launch_split_d<KS, MT, R, WX, false>(a, stream);
}

// What a tile costs, in us: a launch takes about chunks * max(lat * rounds of resident workgroups, work * tiles per CU) + over * tiles per
// CU (+ 3).  Fitted to 211 layers of 24 to 512 -> 16 to 512 maps on 8 x 8 to 940 x 900, d = 1 to 8; with the tile it picks a pass of the layer and two
// 1x1 layers is on average 0.6 % and at most 6 % longer than with the fastest of the eight.
struct SplitCost {
    int mt, r, wx, slots;             // as SplitTile; workgroups that count as resident on a CU
    float lat, work, over;
};
constexpr int SPLIT_TILES = 8;
constexpr SplitCost SPLIT_COST3[SPLIT_TILES] = {{2, 8, 4, 2, 1.63f, 1.19f, 3.72f}, {2, 6, 4, 2, 1.51f, 0.97f, 2.95f}, {2, 4, 2, 4, 1.31f, 0.66f, 1.75f},
                                                {1, 4, 4, 4, 1.10f, 0.47f, 0.98f}, {1, 4, 2, 4, 1.09f, 0.47f, 0.93f}, {3, 5, 4, 2, 1.68f, 1.05f, 4.04f},
                                                {3, 4, 2, 2, 1.60f, 0.96f, 3.26f}, {1, 2, 2, 4, 0.95f, 0.34f, 0.72f}};
constexpr SplitCost SPLIT_COST4[SPLIT_TILES] = {{2, 8, 4, 3, 2.16f, 1.84f, 2.42f}, {2, 6, 4, 2, 1.70f, 1.41f, 2.08f}, {2, 4, 2, 3, 1.31f, 0.96f, 1.25f},
                                                {1, 4, 4, 2, 0.88f, 0.64f, 0.49f}, {1, 4, 2, 3, 0.88f, 0.65f, 0.45f}, {3, 5, 4, 3, 1.97f, 1.59f, 2.52f},
                                                {3, 4, 2, 3, 1.69f, 1.35f, 2.07f}, {1, 2, 2, 3, 0.63f, 0.44f, 0.43f}};

double split_cost(const ConvF32Args &a, const SplitCost &c)
{
    const long tx = 16 * c.wx, rt = c.r * (4 / c.wx), q = a.Ho / a.d, rem = a.Ho % a.d;
    const long gy = rem * ((q + rt) / rt) + (a.d - rem) * ((q + rt - 1) / rt);
    const double tiles = (double)((a.Wo + tx - 1) / tx) * gy * a.n * ((a.n_pad / 16 + c.mt - 1) / c.mt);
    const double per_cu = std::ceil(tiles / 256), rounds = std::ceil(tiles / (256 * c.slots));
    return (a.c_in + 7) / 8 * std::max(c.lat * rounds, c.work * per_cu) + c.over * per_cu;
}

int best_tile(const ConvF32Args &a, const SplitCost *cost)
{
    int best = 0;
    for (int t = 1; t < SPLIT_TILES; ++t)
        if (split_cost(a, cost[t]) < split_cost(a, cost[best])) best = t;
    return best;
}

template <int KS> hipError_t launch_ks(const ConvF32Args &a, hipStream_t stream)
{
    switch (best_tile(a, KS == 3 ? SPLIT_COST3 : SPLIT_COST4)) {
    case 0: return launch_split_p<KS, 2, 8, 4>(a, stream);
    case 1: return launch_split_p<KS, 2, 6, 4>(a, stream);
    case 2: return launch_split_p<KS, 2, 4, 2>(a, stream);
    case 3: return launch_split_p<KS, 1, 4, 4>(a, stream);
    case 4: return launch_split_p<KS, 1, 4, 2>(a, stream);
    case 5: return launch_split_p<KS, 3, 5, 4>(a, stream);
    case 6: return launch_split_p<KS, 3, 4, 2>(a, stream);
    default: return launch_split_p<KS, 1, 2, 2>(a, stream);
    }
}

}  // namespace

// 3x3 layers of so few pixels are no slower on the fp32 matrix unit (64 -> 64 on 20 x 24 13.5 us; on 40 x 36 17.8 against 13.2)
bool conv_split_f32_supported(const ConvF32Args &a)
{
    return conv_split_f32_packed(a.k, a.c_in) && (a.k - 1) * a.d <= 24 && (long)a.H * a.W < (1L << 29) && (long)a.OH * a.OW < (1L << 26) && a.tap_maps == 0 &&
           (a.k == 4 || (long)a.n * a.Ho * a.Wo >= 1000) &&
           (a.grp_maps == 0 || (a.grp_maps > 0 && a.grp_maps % 8 == 0 && a.c_in % a.grp_maps == 0 && a.grp_skip >= 0));
}

SplitPath conv_split_f32_path(const ConvF32Args &a)
{
    if (!conv_split_f32_supported(a)) return {0, 0, 0};
    const SplitCost &c = a.k == 3 ? SPLIT_COST3[best_tile(a, SPLIT_COST3)] : SPLIT_COST4[best_tile(a, SPLIT_COST4)];
    return {c.mt, c.r, c.wx};
}

hipError_t launch_conv_split_f32(const ConvF32Args &a, hipStream_t stream)
{
    return a.k == 3 ? launch_ks<3>(a, stream) : launch_ks<4>(a, stream);
}

}  // namespace sk
