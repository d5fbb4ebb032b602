// HBM-bound layers on the 16-bit octet layout ([n][ceil(C/8)][H][W][8] bf16 or fp16): conversion
// from / to fp32 NCHW (with the mirror padding of Section 1.3 fused into the conversion of the
// image), max pooling with kernel stride (forward with winner codes, gather-form backward) and the
// bias gradient.  One 16-byte unit (8 maps of one pixel) per thread, pixels fastest, so a wavefront
// moves 1 KB of consecutive addresses per access.  Comparisons are done on the exactly widened
// fp32 values, so pooling is bit-exact in both formats.
#include <type_traits>

#include "sk_kernels.h"

namespace sk {

typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));

static inline int grid_for(long total, int block = 256, int cap = 1 << 20)
{
    long b = (total + block - 1) / block;
    if (b < 1) b = 1;
    return (int)(b < cap ? b : cap);
}

template <int DT> __device__ __forceinline__ float up16(unsigned u);
template <> __device__ __forceinline__ float up16<1>(unsigned u) { return __uint_as_float(u << 16); }
template <> __device__ __forceinline__ float up16<2>(unsigned u) { return (float)__builtin_bit_cast(_Float16, (unsigned short)u); }
template <int DT> __device__ __forceinline__ unsigned down16(float f);
template <> __device__ __forceinline__ unsigned down16<1>(float f) { return __builtin_bit_cast(unsigned short, static_cast<__bf16>(f)); }
template <> __device__ __forceinline__ unsigned down16<2>(float f) { return __builtin_bit_cast(unsigned short, static_cast<_Float16>(f)); }

__device__ __forceinline__ unsigned elem16(const uint4v &u, int e) { return (u[e >> 1] >> ((e & 1) * 16)) & 0xffffu; }

__device__ __forceinline__ int mirror_index_h(int t, int len, int mode)
{
    if (len == 1) return 0;
    if (mode == 0) {
        const int period = 2 * (len - 1);
        t %= period;
        if (t < 0) t += period;
        return t < len ? t : period - t;
    }
    const int period = 2 * len;
    t %= period;
    if (t < 0) t += period;
    return t < len ? t : period - 1 - t;
}

// out[b][o][y][x][e] = in[b][8o+e][m(y-top)][m(x-left)] rounded to nearest even (0 for maps >= c)
template <int DT>
__global__ void pad_pack_h_kernel(const float *in, uint4v *out, int n, int c, int h, int w, int top, int left,
                                  int ho, int wo, int mode)
{
    const int c8 = (c + 7) / 8;
    const long total = (long)n * c8 * ho * wo;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const int x = (int)(q % wo);
        long t = q / wo;
        const int y = (int)(t % ho);
        t /= ho;
        const int o = (int)(t % c8);
        const long b = t / c8;
        const int sy = (top | left) ? mirror_index_h(y - top, h, mode) : y;
        const int sx = (top | left) ? mirror_index_h(x - left, w, mode) : x;
        unsigned hv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int ch = o * 8 + e;
            hv[e] = ch < c ? down16<DT>(in[((b * c + ch) * h + sy) * (long)w + sx]) : 0u;
        }
        out[q] = uint4v{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16), hv[4] | (hv[5] << 16), hv[6] | (hv[7] << 16)};
    }
}

hipError_t launch_pad_pack_h(const float *in, void *out, int dtype, int n, int c, int h, int w, int top, int left,
                             int ho, int wo, int mode, hipStream_t stream)
{
    const long total = (long)n * ((c + 7) / 8) * ho * wo;
    if (dtype == 1)
        hipLaunchKernelGGL(pad_pack_h_kernel<1>, dim3(grid_for(total)), dim3(256), 0, stream, in, static_cast<uint4v *>(out), n, c, h, w, top, left, ho, wo, mode);
    else
        hipLaunchKernelGGL(pad_pack_h_kernel<2>, dim3(grid_for(total)), dim3(256), 0, stream, in, static_cast<uint4v *>(out), n, c, h, w, top, left, ho, wo, mode);
    return hipGetLastError();
}

template <int DT>
__global__ void unpack_h_kernel(const uint4v *in, float *out, int n, int c, int h, int w)
{
    const int c8 = (c + 7) / 8;
    const long plane = (long)h * w, total = (long)n * c8 * plane;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const long pix = q % plane;
        const long t = q / plane;
        const int o = (int)(t % c8);
        const long b = t / c8;
        const uint4v u = in[q];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (o * 8 + e < c) out[(b * c + o * 8 + e) * plane + pix] = up16<DT>(elem16(u, e));
    }
}

hipError_t launch_unpack_h(const void *in, float *out, int dtype, int n, int c, int h, int w, hipStream_t stream)
{
    const long total = (long)n * ((c + 7) / 8) * h * w;
    if (dtype == 1)
        hipLaunchKernelGGL(unpack_h_kernel<1>, dim3(grid_for(total)), dim3(256), 0, stream, static_cast<const uint4v *>(in), out, n, c, h, w);
    else
        hipLaunchKernelGGL(unpack_h_kernel<2>, dim3(grid_for(total)), dim3(256), 0, stream, static_cast<const uint4v *>(in), out, n, c, h, w);
    return hipGetLastError();
}

// ---- max pooling with kernel stride d and layer stride s (Section 5.2.1) on octets --------------------
// winner code of element e of unit q (see maxpool_h_kernel)
__device__ __forceinline__ unsigned pool_code_h(const void *tap, long q, int e, bool bits)
{
    if (bits) {
        const unsigned w = static_cast<const unsigned *>(tap)[q];
        return ((w >> e) & 1u) | (((w >> (8 + e)) & 1u) << 1);
    }
    return (static_cast<const uint2v *>(tap)[q][e >> 2] >> ((e & 3) * 8)) & 0xffu;
}

// Winner codes: one byte i * k + j per element, laid out like y -- except for k = 2, s = 1 (pool_bits_h), the SK pools,
// whose codes are three bit planes of the octet in one 32-bit word per unit: bit e of byte 0 = j, of byte 1 = i of
// element e's winner, of byte 2 = its value is positive.  Half the bytes, and the backward pass has the ReLU mask of the
// layer below in them: that layer's output at the winner IS the window's maximum.
// grid: x = column blocks, y = output row, z = plane (image x octet); no index division
template <int DT>
__global__ void maxpool_h_kernel(const uint4v *x, uint4v *y, void *tap, int H, int W, int Ho, int Wo,
                                 int k, int d, int s)
{
    const int xx = blockIdx.x * blockDim.x + threadIdx.x, yy = blockIdx.y;
    if (xx >= Wo) return;
    const long p = blockIdx.z;
    const uint4v *src = x + (p * H + (long)s * yy) * W + (long)s * xx;
    const uint4v first = src[0];
    float best[8];
    unsigned bits[8], code[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bits[e] = elem16(first, e);
        best[e] = up16<DT>(bits[e]);
        code[e] = 0;
    }
    for (int i = 0; i < k; ++i)
        for (int j = 0; j < k; ++j) {
            const uint4v u = src[(long)i * d * W + j * d];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned b16 = elem16(u, e);
                const float v = up16<DT>(b16);
                if (v > best[e]) {          // strictly greater: the first maximum wins
                    best[e] = v;
                    bits[e] = b16;
                    code[e] = i * k + j;
                }
            }
        }
    const long q = (p * Ho + yy) * Wo + xx;
    y[q] = uint4v{bits[0] | (bits[1] << 16), bits[2] | (bits[3] << 16), bits[4] | (bits[5] << 16), bits[6] | (bits[7] << 16)};
    if (!tap) return;
    if (pool_bits_h(k, s)) {
        unsigned word = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) word |= ((code[e] & 1u) << e) | ((code[e] >> 1) << (8 + e)) | ((best[e] > 0.f ? 1u : 0u) << (16 + e));
        static_cast<unsigned *>(tap)[q] = word;
    } else {
        static_cast<uint2v *>(tap)[q] = uint2v{code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24),
                                               code[4] | (code[5] << 8) | (code[6] << 16) | (code[7] << 24)};
    }
}

// ... of a 3-D pool (see maxpool3d_h_kernel)
__device__ __forceinline__ unsigned pool3d_code_h(const void *tap, long q, int e, bool bits)
{
    if (bits) {
        const unsigned w = static_cast<const unsigned *>(tap)[q];
        return ((w >> e) & 1u) | (((w >> (8 + e)) & 1u) << 1) | (((w >> (16 + e)) & 1u) << 2);
    }
    return pool_code_h(tap, q, e, false);
}

// k = 2, s = 1 (every SK pool of the paper): window (y, x) is {h[y], h[y + d]} where h[r] is the
// first maximum of X[r][x], X[r][x + d].  A thread walks one column down the rows y0, y0 + d,
// y0 + 2d, ... of one residue class mod d, so each h is formed once and serves both windows it
// belongs to, and a block reads every input row it needs exactly once (no second workgroup, on
// another XCD with another L2, fetches the same rows again).  Grid and workgroup: see pool_cut; segments are M windows long,
// z = plane.  The winner follows the row-major scan: row y before row y + d, strictly-greater replaces.
// Sets of elements come in split form: element 2 w in bit 2 w, element 2 w + 1 in bit 16 + 2 w, as a word's two halves give them.
template <int DT>
__device__ __forceinline__ void row_first_max(const uint4v a, const uint4v b, uint4v &h, unsigned &hc)
{
    hc = 0u;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const unsigned lo = up16<DT>(b[w] & 0xffffu) > up16<DT>(a[w] & 0xffffu) ? 0x0000ffffu : 0u;
        const unsigned m = lo | (up16<DT>(b[w] >> 16) > up16<DT>(a[w] >> 16) ? 0xffff0000u : 0u);
        hc |= (m & 0x00010001u) << (2 * w);
        h[w] = (a[w] & ~m) | (b[w] & m);
    }
}

// the positive elements (not zero, no NaN).  Packed 16-bit integers: u - 1 of 1 .. infinity, and of nothing else, stays below the top bit
// when the rest of the range is added with saturation.
template <int DT>
__device__ __forceinline__ unsigned positive_h(const uint4v o)
{
    typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
    constexpr unsigned short REST = DT == 1 ? 0x8000 - 0x7f80 : 0x8000 - 0x7c00;
    unsigned not_pos = 0u;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const unsigned word = o[w];
        const ushort2v v = __builtin_elementwise_add_sat((ushort2v)(__builtin_bit_cast(ushort2v, word) - (unsigned short)1), ushort2v{REST, REST});
        not_pos |= (__builtin_bit_cast(unsigned, v) >> 15 & 0x00010001u) << (2 * w);
    }
    return not_pos ^ 0x00550055u;
}

// two sets in split form as two bit planes: bit e of byte 0, of byte 1
__device__ __forceinline__ unsigned bit_planes_h(unsigned a, unsigned b)
{
    const unsigned both = a | (b << 8);
    return (both | (both >> 15)) & 0xffffu;
}

// U: windows whose loads are in flight together; NT: see pool_stores_around
template <int DT, bool TAP, int U, bool NT>
__global__ void __launch_bounds__(256) maxpool2_chain_h_kernel(const uint4v *__restrict__ x, uint4v *__restrict__ y,
                                                               unsigned *__restrict__ tap, int H, int W, int Ho, int Wo,
                                                               int d, int M, int nseg, int pblocks)
{
    const int xx = blockIdx.x * blockDim.x + threadIdx.x;
    const int sblock = blockIdx.y / pblocks, phase = (blockIdx.y - sblock * pblocks) * blockDim.y + threadIdx.y, seg = sblock * blockDim.z + threadIdx.z;
    if (xx >= Wo || phase >= d || phase >= Ho || seg >= nseg) return;
    const int links = (Ho - phase + d - 1) / d;           // windows of this residue class
    const int m0 = seg * M, m1 = min(links, m0 + M);
    if (m0 >= m1) return;
    const long p = blockIdx.z;
    const long rstep = (long)d * W;
    const uint4v *src = x + (p * H + phase + (long)m0 * d) * W + xx;
    uint4v *dst = y + (p * Ho + phase + (long)m0 * d) * Wo + xx;
    unsigned *tdst = TAP ? tap + (p * Ho + phase + (long)m0 * d) * Wo + xx : nullptr;
    const long ostep = (long)d * Wo;
    uint4v a[U], b[U];
    auto load = [&](int m) {                              // the lower rows of windows m .. m + U - 1
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint4v *r = src + (m + u < m1 ? (long)(u + 1) * rstep : 0);
            a[u] = r[0];
            b[u] = r[d];
        }
    };
    const uint4v first = src[0], right = src[d];
    load(m0);                                             // in flight together with the first row
    uint4v h;
    unsigned hc;
    row_first_max<DT>(first, right, h, hc);
    for (int m = m0;;) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (m + u >= m1) break;
            uint4v h2;
            unsigned hc2;
            row_first_max<DT>(a[u], b[u], h2, hc2);
            uint4v o;
            unsigned lower;                               // whose winner lies in row y + d
            row_first_max<DT>(h, h2, o, lower);
            if constexpr (NT) __builtin_nontemporal_store(o, dst + (long)u * ostep);
            else dst[(long)u * ostep] = o;
            if constexpr (TAP) {
                const unsigned code = bit_planes_h((hc & ~lower) | (hc2 & lower), lower) | (bit_planes_h(positive_h<DT>(o), 0u) << 16);
                if constexpr (NT) __builtin_nontemporal_store(code, tdst + (long)u * ostep);
                else tdst[(long)u * ostep] = code;
            }
            h = h2;
            hc = hc2;
        }
        m += U;
        if (m >= m1) return;
        src += (long)U * rstep;
        dst += (long)U * ostep;
        if (TAP) tdst += (long)U * ostep;
        load(m);
    }
}

template <int DT, bool TAP>
static void launch_maxpool2_chain_h(const PoolCut &c, dim3 grid, hipStream_t stream, const void *x, void *y, void *tap, int H, int W, int Ho, int Wo, int d)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, c.block(), 0, stream, static_cast<const uint4v *>(x), static_cast<uint4v *>(y),
                           static_cast<unsigned *>(tap), H, W, Ho, Wo, d, c.len, c.nseg, c.pblocks);
    };
    const auto with = [&](auto around) {
        constexpr bool NT = decltype(around)::value;
        if (c.len >= 4) go(&maxpool2_chain_h_kernel<DT, TAP, 4, NT>);
        else if (c.len >= 2) go(&maxpool2_chain_h_kernel<DT, TAP, 2, NT>);
        else go(&maxpool2_chain_h_kernel<DT, TAP, 1, NT>);
    };
    if (TAP && pool_stores_around(16L * grid.z * Ho * Wo)) with(std::integral_constant<bool, TAP>{});
    else with(std::false_type{});
}

hipError_t launch_maxpool_h(const void *x, void *y, void *tap, int dtype, long planes8, int H, int W, int Ho, int Wo,
                            int k, int d, int s, hipStream_t stream)
{
    if (Ho > 65535 || planes8 > 65535) return hipErrorInvalidValue;
    if (k == 2 && s == 1 && Ho == H - d && Wo == W - d) {
        const PoolCut c = pool_cut(Ho, Wo, d, planes8, tap ? POOL_WAVES : POOL_WAVES / 4);
        if (c.gy <= 65535) {
            const dim3 grid = c.grid(Wo, planes8);
            if (dtype == 1 && tap) launch_maxpool2_chain_h<1, true>(c, grid, stream, x, y, tap, H, W, Ho, Wo, d);
            else if (dtype == 1) launch_maxpool2_chain_h<1, false>(c, grid, stream, x, y, tap, H, W, Ho, Wo, d);
            else if (tap) launch_maxpool2_chain_h<2, true>(c, grid, stream, x, y, tap, H, W, Ho, Wo, d);
            else launch_maxpool2_chain_h<2, false>(c, grid, stream, x, y, tap, H, W, Ho, Wo, d);
            return hipGetLastError();
        }
    }
    const dim3 grid((Wo + 255) / 256, Ho, (unsigned)planes8);
    if (dtype == 1)
        hipLaunchKernelGGL(maxpool_h_kernel<1>, grid, dim3(256), 0, stream, static_cast<const uint4v *>(x),
                           static_cast<uint4v *>(y), tap, H, W, Ho, Wo, k, d, s);
    else
        hipLaunchKernelGGL(maxpool_h_kernel<2>, grid, dim3(256), 0, stream, static_cast<const uint4v *>(x),
                           static_cast<uint4v *>(y), tap, H, W, Ho, Wo, k, d, s);
    return hipGetLastError();
}

// ---- 3-D max pooling on the slice-major octet layout [D][C8][H][W][8] (Section 5.2.2) -----------------------
// Y[z][o8][y][x] = max over the k^3 taps X[s z + a d][o8][s y + i d][s x + j d]; tap (optional, laid out like y, one
// byte per element): the winner's code (a k + i) k + j, the first maximum in that scan order.  k = 2, s = 1: four bit planes in a
// 32-bit word per unit instead, as in the 2-D pools: j, i, a and whether the maximum is positive.
// grid: x = column blocks, y = output row, z = (output slice, octet)
template <int DT>
__global__ void maxpool3d_h_kernel(const uint4v *x, uint4v *y, void *tap, int C8, int H, int W, int Ho, int Wo, int k, int d, int s)
{
    const int xx = blockIdx.x * blockDim.x + threadIdx.x, yy = blockIdx.y;
    if (xx >= Wo) return;
    const int zo = blockIdx.z / C8, o8 = blockIdx.z - zo * C8;
    const long plane = (long)H * W;
    const uint4v *src = x + ((long)s * zo * C8 + o8) * plane + (long)s * yy * W + (long)s * xx;
    const uint4v first = src[0];
    float best[8];
    unsigned bits[8], code[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bits[e] = elem16(first, e);
        best[e] = up16<DT>(bits[e]);
        code[e] = 0;
    }
    for (int a = 0; a < k; ++a)
        for (int i = 0; i < k; ++i)
            for (int j = 0; j < k; ++j) {
                const uint4v u = src[(long)a * d * C8 * plane + (long)i * d * W + j * d];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const unsigned b16 = elem16(u, e);
                    const float v = up16<DT>(b16);
                    if (v > best[e]) {          // strictly greater: the first maximum wins
                        best[e] = v;
                        bits[e] = b16;
                        code[e] = (a * k + i) * k + j;
                    }
                }
            }
    const long q = ((long)blockIdx.z * Ho + yy) * Wo + xx;
    y[q] = uint4v{bits[0] | (bits[1] << 16), bits[2] | (bits[3] << 16), bits[4] | (bits[5] << 16), bits[6] | (bits[7] << 16)};
    if (!tap) return;
    if (pool_bits_h(k, s)) {
        unsigned word = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            word |= ((code[e] & 1u) << e) | ((code[e] >> 1 & 1u) << (8 + e)) | ((code[e] >> 2) << (16 + e)) | ((best[e] > 0.f ? 1u : 0u) << (24 + e));
        static_cast<unsigned *>(tap)[q] = word;
    } else {
        static_cast<uint2v *>(tap)[q] = uint2v{code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24),
                                               code[4] | (code[5] << 8) | (code[6] << 16) | (code[7] << 24)};
    }
}

// k = 2, s = 1: a thread owns one position of an output octet plane and walks down the slices z0, z0 + d, ... of one residue class.
// The first maximum of the 2x2 samples of slice z serves the windows of slices z - d and z, so each is formed once: four loads a window
// instead of eight, three of which the neighbouring threads load too (the two pools of the 81x145x145 net, with codes: 160 -> 92 us).  grid: x = (residue class and chain segment, block of 256 positions), y = octet
template <int DT, bool TAP>
__global__ void __launch_bounds__(256) maxpool3d_k2_chain_h_kernel(const uint4v *__restrict__ x, uint4v *__restrict__ y, unsigned *__restrict__ tap,
                                                                   int C8, int H, int W, int Do, int Ho, int Wo, int d, int M, int nseg, int pblocks)
{
    const int chain = blockIdx.x / pblocks, pb = blockIdx.x - chain * pblocks, phase = chain / nseg, seg = chain - phase * nseg;
    const int pos = pb * 256 + threadIdx.x, o8 = blockIdx.y, m0 = seg * M;
    if (pos >= Ho * Wo || phase >= Do) return;
    const int m1 = min((Do - phase + d - 1) / d, m0 + M);
    if (m0 >= m1) return;
    const int yy = pos / Wo, xx = pos - yy * Wo;
    const long zstep = (long)d * C8 * H * W, ostep = (long)d * C8 * Ho * Wo, below = (long)d * W;
    const uint4v *src = x + (((long)(phase + m0 * d) * C8 + o8) * H + yy) * W + xx;
    const long o0 = ((long)(phase + m0 * d) * C8 + o8) * Ho * Wo + pos;
    uint4v *dst = y + o0;
    unsigned *tdst = TAP ? tap + o0 : nullptr;
    struct Quad {
        uint4v v;
        unsigned j, i;
    };
    auto quad = [](uint4v a, uint4v b, uint4v c, uint4v e) {
        uint4v top, low;
        unsigned jt, jl;
        Quad q;
        row_first_max<DT>(a, b, top, jt);
        row_first_max<DT>(c, e, low, jl);
        row_first_max<DT>(top, low, q.v, q.i);
        q.j = (jt & ~q.i) | (jl & q.i);
        return q;
    };
    Quad q = quad(src[0], src[d], src[below], src[below + d]);
    constexpr int U = 2;
    for (int m = m0; m < m1; m += U) {
        uint4v s[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {                     // all loads of the group first
            const uint4v *p = src + (m + u < m1 ? (u + 1) * zstep : 0);
            s[u][0] = p[0];
            s[u][1] = p[d];
            s[u][2] = p[below];
            s[u][3] = p[below + d];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (m + u >= m1) break;
            const Quad q2 = quad(s[u][0], s[u][1], s[u][2], s[u][3]);
            uint4v o;
            unsigned far;                                 // whose winner lies in slice z + d
            row_first_max<DT>(q.v, q2.v, o, far);
            dst[u * ostep] = o;
            if (TAP)
                tdst[u * ostep] = bit_planes_h((q.j & ~far) | (q2.j & far), (q.i & ~far) | (q2.i & far)) | (bit_planes_h(far, positive_h<DT>(o)) << 16);
            q = q2;
        }
        src += U * zstep;
        dst += U * ostep;
        if (TAP) tdst += U * ostep;
    }
}

// Chains of 16 slices, shorter where that leaves the GPU empty; false: a grid too large for this form
static bool pool3d_cut(int C8, int D, long plane, int d, int &len, int &nseg, unsigned &gx, int &pblocks)
{
    const int links = (D + d - 1) / d;
    const long pb = (plane + 255) / 256;
    for (len = 16;; len /= 2) {
        nseg = (links + len - 1) / len;
        if (len == 4 || pb * 4 * d * nseg * C8 >= POOL_WAVES) break;
    }
    if (plane > 0x3fffffffL || (long)d * nseg * pb > 0x7fffffffL || C8 > 65535) return false;
    gx = (unsigned)(d * nseg * pb);
    pblocks = (int)pb;
    return true;
}

// Gather form of the 3-D pool gradient (s = 1) on the slice-major octet layout: input unit (z, u, v) of octet o8 collects,
// per map, dY of the windows whose recorded winner it is; fp32 sums, rounded once; relu_src as in the 2-D kernel.
// grid: x = column blocks, y = input row, z = (input slice, octet)
template <int DT>
__global__ void maxpool3d_bwd_h_kernel(const uint4v *__restrict__ dy, const void *__restrict__ tap, const uint4v *__restrict__ relu_src,
                                       uint4v *__restrict__ dx, int C8, int H, int W, int Do, int Ho, int Wo, int k, int d)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x, u = blockIdx.y;
    if (v >= W) return;
    const int z = blockIdx.z / C8, o8 = blockIdx.z - z * C8;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    for (int a = 0; a < k; ++a) {
        const int zo = z - a * d;
        if (zo < 0 || zo >= Do) continue;
        for (int i = 0; i < k; ++i) {
            const int yo = u - i * d;
            if (yo < 0 || yo >= Ho) continue;
            for (int j = 0; j < k; ++j) {
                const int xo = v - j * d;
                if (xo < 0 || xo >= Wo) continue;
                const long o = (((long)zo * C8 + o8) * Ho + yo) * Wo + xo;
                const uint4v g = dy[o];
                const unsigned want = (unsigned)((a * k + i) * k + j);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (pool3d_code_h(tap, o, e, pool_bits_h(k, 1)) == want) acc[e] += up16<DT>(elem16(g, e));
            }
        }
    }
    const long q = ((long)blockIdx.z * H + u) * W + v;
    uint4v rs = uint4v{0u, 0u, 0u, 0u};
    if (relu_src) rs = relu_src[q];
    unsigned hv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float t = acc[e];
        if (relu_src && !(up16<DT>(elem16(rs, e)) > 0.f)) t = 0.f;
        hv[e] = down16<DT>(t);
    }
    dx[q] = uint4v{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16), hv[4] | (hv[5] << 16), hv[6] | (hv[7] << 16)};
}

// k = 2: a thread walks position (u, v) of dX down the slices z0, z0 + d, ... of one residue class, as the forward kernel walks its
// windows.  Slice z collects from the windows of slices z (a = 0) and z - d (a = 1), so the four windows of a slice are loaded once
// and what they give the next step is kept as a sum; MASKED takes the ReLU mask of the layer below from the codes.  (Eight windows with
// byte codes a thread and the layer's output: 208 bytes loaded a unit, 80 here; the same two pools 196 -> 87 us.)
template <int DT, bool MASKED>
__global__ void __launch_bounds__(256) maxpool3d_k2_bwd_chain_h_kernel(const uint4v *__restrict__ dy, const unsigned *__restrict__ tap,
                                                                       uint4v *__restrict__ dx, int C8, int H, int W, int D, int Do, int Ho, int Wo,
                                                                       int d, int M, int nseg, int pblocks)
{
    const int chain = blockIdx.x / pblocks, pb = blockIdx.x - chain * pblocks, phase = chain / nseg, seg = chain - phase * nseg;
    const int pos = pb * 256 + threadIdx.x, o8 = blockIdx.y, m0 = seg * M;
    if (pos >= H * W || phase >= D) return;
    const int m1 = min((D - phase + d - 1) / d, m0 + M);
    if (m0 >= m1) return;
    const int u = pos / W, v = pos - u * W;
    // the four windows (i, j) of a slice that can have chosen this position, clamped into the plane; `in`: all ones where they exist
    int at[4];
    unsigned in[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int yy = u - (t >> 1) * d, xx = v - (t & 1) * d;
        in[t] = yy >= 0 && yy < Ho && xx >= 0 && xx < Wo ? 0xffu : 0u;
        at[t] = in[t] ? yy * Wo + xx : 0;
    }
    struct Slice {
        uint4v g[4];
        unsigned c[4];
    };
    auto load = [&](int z) {                              // windows of slice z, clamped into the volume
        const long base = ((long)(z < 0 ? 0 : (z < Do ? z : Do - 1)) * C8 + o8) * Ho * Wo;
        Slice s;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            s.g[t] = dy[base + at[t]];
            s.c[t] = tap[base + at[t]];
        }
        return s;
    };
    auto pick = [](uint4v g, unsigned t, int e) {         // the element, or +0
        return __int_as_float(__float_as_int(up16<DT>(elem16(g, e))) & ((int)(t << (31 - e)) >> 31));
    };
    // what the windows of slice z give slice z (near) and slice z + d (far)
    auto split = [&](const Slice &s, int z, float (&near)[8], float (&far)[8]) {
        const unsigned row = z >= 0 && z < Do ? 0xffu : 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) near[e] = far[e] = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const unsigned c = s.c[t], j = t & 1 ? c : ~c, i = t & 2 ? c >> 8 : ~(c >> 8);
            const unsigned mine = (MASKED ? c >> 24 : 0xffu) & in[t] & row & j & i, nm = mine & ~(c >> 16), fm = mine & (c >> 16);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                near[e] += pick(s.g[t], nm, e);
                far[e] += pick(s.g[t], fm, e);
            }
        }
    };
    int z = phase + m0 * d;
    uint4v *dst = dx + ((long)z * C8 + o8) * H * W + pos;
    const long ostep = (long)d * C8 * H * W;
    float kept[8], near[8], far[8];
    split(load(z - d), z - d, near, kept);
    constexpr int U = 2;
    for (int m = m0; m < m1; m += U) {
        Slice s[U];
#pragma unroll
        for (int w = 0; w < U; ++w) s[w] = load(z + w * d);          // all loads of the group first
#pragma unroll
        for (int w = 0; w < U; ++w) {
            if (m + w >= m1) break;
            split(s[w], z + w * d, near, far);
            unsigned hv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                hv[e] = down16<DT>(near[e] + kept[e]);
                kept[e] = far[e];
            }
            dst[w * ostep] = uint4v{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16), hv[4] | (hv[5] << 16), hv[6] | (hv[7] << 16)};
        }
        z += U * d;
        dst += U * ostep;
    }
}

hipError_t launch_maxpool3d_bwd_h(const void *dy, const void *tap, const void *relu_src, void *dx, int dtype, int C, int D, int H, int W,
                                  int Do, int Ho, int Wo, int k, int d, hipStream_t stream)
{
    const int C8 = (C + 7) / 8;
    if (H > 65535 || (long)D * C8 > 65535 || (dtype != 1 && dtype != 2) || k < 1 || k > 6) return hipErrorInvalidValue;
    if (Do != D - (k - 1) * d || Ho != H - (k - 1) * d || Wo != W - (k - 1) * d || Do < 1 || Ho < 1 || Wo < 1) return hipErrorInvalidValue;
    const dim3 grid((W + 255) / 256, H, (unsigned)(D * C8));
    const uint4v *g = static_cast<const uint4v *>(dy), *rs = static_cast<const uint4v *>(relu_src);
    uint4v *out = static_cast<uint4v *>(dx);
    int len, nseg, pblocks;
    unsigned gx;
    if (k == 2 && pool3d_cut(C8, D, (long)H * W, d, len, nseg, gx, pblocks)) {
        const unsigned *tp = static_cast<const unsigned *>(tap);
        const dim3 cgrid(gx, C8);
        if (dtype == 1) {
            if (rs) hipLaunchKernelGGL((maxpool3d_k2_bwd_chain_h_kernel<1, true>), cgrid, dim3(256), 0, stream, g, tp, out, C8, H, W, D, Do, Ho, Wo, d, len, nseg, pblocks);
            else hipLaunchKernelGGL((maxpool3d_k2_bwd_chain_h_kernel<1, false>), cgrid, dim3(256), 0, stream, g, tp, out, C8, H, W, D, Do, Ho, Wo, d, len, nseg, pblocks);
        } else {
            if (rs) hipLaunchKernelGGL((maxpool3d_k2_bwd_chain_h_kernel<2, true>), cgrid, dim3(256), 0, stream, g, tp, out, C8, H, W, D, Do, Ho, Wo, d, len, nseg, pblocks);
            else hipLaunchKernelGGL((maxpool3d_k2_bwd_chain_h_kernel<2, false>), cgrid, dim3(256), 0, stream, g, tp, out, C8, H, W, D, Do, Ho, Wo, d, len, nseg, pblocks);
        }
        return hipGetLastError();
    }
    const void *tp = tap;
    if (dtype == 1) hipLaunchKernelGGL(maxpool3d_bwd_h_kernel<1>, grid, dim3(256), 0, stream, g, tp, rs, out, C8, H, W, Do, Ho, Wo, k, d);
    else hipLaunchKernelGGL(maxpool3d_bwd_h_kernel<2>, grid, dim3(256), 0, stream, g, tp, rs, out, C8, H, W, Do, Ho, Wo, k, d);
    return hipGetLastError();
}

// winner codes of a 3-D pool on the octet layout -> flat offsets ((z_in*H + y_in)*W + x_in) inside the map's input
// volume, int32 [Do][C][Ho][Wo] (for the parity accessor)
__global__ void tap3d_to_index_h_kernel(const void *tap, int32_t *idx, int C, int Do, int Ho, int Wo, int H, int W, int k, int d, int s,
                                        long total)
{
    const int C8 = (C + 7) / 8;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const int xo = (int)(q % Wo);
        long t = q / Wo;
        const int yo = (int)(t % Ho);
        t /= Ho;
        const int c = (int)(t % C), zo = (int)(t / C);
        const int code = (int)pool3d_code_h(tap, (((long)zo * C8 + (c >> 3)) * Ho + yo) * Wo + xo, c & 7, pool_bits_h(k, s));
        const int j = code % k, i = (code / k) % k, a = code / (k * k);
        idx[q] = (int32_t)((((long)s * zo + a * d) * H + s * yo + i * d) * W + s * xo + j * d);
    }
}

hipError_t launch_tap3d_to_index_h(const void *tap, int32_t *idx, int C, int Do, int Ho, int Wo, int H, int W, int k, int d, int s,
                                   hipStream_t stream)
{
    const long total = (long)C * Do * Ho * Wo;
    hipLaunchKernelGGL(tap3d_to_index_h_kernel, dim3(grid_for(total)), dim3(256), 0, stream, tap, idx, C, Do, Ho, Wo,
                       H, W, k, d, s, total);
    return hipGetLastError();
}

// A 3-D kernel [o][c][a][i][j] (fp32 master) as the OIHW master of the 2-D convolution that computes it on the slice-major
// octet layout.  Forward (bwd = 0): out[o][a * C8*8 + c][i][j] = w[o][c][a][i][j] (c_out x k*C8*8 maps; the maps an octet pads
// stay zero).  Data gradient (bwd = 1): out[a' * O8*8 + o][c][i][j] = w[o][c][k-1-a'][i][j] (k*O8*8 x c_in maps), which the
// 2-D data-gradient packing then flips in the plane and transposes.
struct ExpandJobs { ExpandTaps3d job[BATCH_MAX]; };

// blockIdx.y: job
__global__ void expand_taps3d_kernel(ExpandJobs jobs)
{
    const ExpandTaps3d &jb = jobs.job[blockIdx.y];
    const float *__restrict__ w = jb.w;
    const int c_out = jb.c_out, c_in = jb.c_in, k = jb.k, bwd = jb.bwd;
    const int kk = k * k, C8 = (c_in + 7) / 8 * 8, O8 = (c_out + 7) / 8 * 8;
    const long total = jb.floats();
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const int r = (int)(q % kk);
        long t = q / kk;
        float v = 0.f;
        if (!bwd) {
            const int m = (int)(t % (k * C8)), o = (int)(t / (k * C8));
            const int a = m / C8, c = m - a * C8;
            if (c < c_in) v = w[(((long)o * c_in + c) * k + a) * kk + r];
        } else {
            const int c = (int)(t % c_in), m = (int)(t / c_in);
            const int a = m / O8, o = m - a * O8;
            if (o < c_out) v = w[(((long)o * c_in + c) * k + (k - 1 - a)) * kk + r];
        }
        jb.out[q] = v;
    }
}

hipError_t launch_expand_taps3d(const ExpandTaps3d *jobs, int n, hipStream_t stream)
{
    if (n < 1 || n > BATCH_MAX) return hipErrorInvalidValue;
    ExpandJobs b{};
    long most = 0;
    for (int t = 0; t < n; ++t) {
        if (jobs[t].c_out < 1 || jobs[t].c_in < 1 || jobs[t].k < 1) return hipErrorInvalidValue;
        b.job[t] = jobs[t];
        most = std::max(most, jobs[t].floats());
    }
    hipLaunchKernelGGL(expand_taps3d_kernel, dim3(grid_for(most), n), dim3(256), 0, stream, b);
    return hipGetLastError();
}

hipError_t launch_maxpool3d_h(const void *x, void *y, void *tap, int dtype, int C, int D, int H, int W, int Do, int Ho, int Wo, int k, int d,
                              int s, hipStream_t stream)
{
    const int C8 = (C + 7) / 8;
    if (Ho > 65535 || (long)Do * C8 > 65535 || (dtype != 1 && dtype != 2) || D < 1) return hipErrorInvalidValue;
    const uint4v *in = static_cast<const uint4v *>(x);
    uint4v *out = static_cast<uint4v *>(y);
    int len, nseg, pblocks;
    unsigned gx;
    if (pool_bits_h(k, s) && Do == D - d && Ho == H - d && Wo == W - d && pool3d_cut(C8, Do, (long)Ho * Wo, d, len, nseg, gx, pblocks)) {
        unsigned *tp = static_cast<unsigned *>(tap);
        const dim3 cgrid(gx, C8);
        if (dtype == 1) {
            if (tap) hipLaunchKernelGGL((maxpool3d_k2_chain_h_kernel<1, true>), cgrid, dim3(256), 0, stream, in, out, tp, C8, H, W, Do, Ho, Wo, d, len, nseg, pblocks);
            else hipLaunchKernelGGL((maxpool3d_k2_chain_h_kernel<1, false>), cgrid, dim3(256), 0, stream, in, out, tp, C8, H, W, Do, Ho, Wo, d, len, nseg, pblocks);
        } else {
            if (tap) hipLaunchKernelGGL((maxpool3d_k2_chain_h_kernel<2, true>), cgrid, dim3(256), 0, stream, in, out, tp, C8, H, W, Do, Ho, Wo, d, len, nseg, pblocks);
            else hipLaunchKernelGGL((maxpool3d_k2_chain_h_kernel<2, false>), cgrid, dim3(256), 0, stream, in, out, tp, C8, H, W, Do, Ho, Wo, d, len, nseg, pblocks);
        }
        return hipGetLastError();
    }
    const dim3 grid((Wo + 255) / 256, Ho, (unsigned)(Do * C8));
    if (dtype == 1) hipLaunchKernelGGL(maxpool3d_h_kernel<1>, grid, dim3(256), 0, stream, in, out, tap, C8, H, W, Ho, Wo, k, d, s);
    else hipLaunchKernelGGL(maxpool3d_h_kernel<2>, grid, dim3(256), 0, stream, in, out, tap, C8, H, W, Ho, Wo, k, d, s);
    return hipGetLastError();
}

// MergeCrop's second operand on octets (Section 5.3.1): dst[b][o8_off + o][y][x] = src[b][o][y + cy][x + cx]
__global__ void crop_copy_h_kernel(const uint4v *__restrict__ src, uint4v *__restrict__ dst, int n, int c8, int Hs, int Ws,
                                   int c8_total, int o8_off, int H, int W, int cy, int cx)
{
    const long plane = (long)H * W, total = (long)n * c8 * plane;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const long pix = q % plane, t = q / plane;
        const int x = (int)(pix % W), y = (int)(pix / W);
        const int o = (int)(t % c8);
        const long b = t / c8;
        dst[((b * c8_total + o8_off + o) * H + y) * W + x] = src[((b * c8 + o) * Hs + y + cy) * Ws + x + cx];
    }
}

hipError_t launch_crop_copy_h(const void *src, void *dst, int n, int c8, int Hs, int Ws, int c8_total, int o8_off,
                              int H, int W, int cy, int cx, hipStream_t stream)
{
    if (cy < 0 || cx < 0 || cy + H > Hs || cx + W > Ws || o8_off < 0 || o8_off + c8 > c8_total) return hipErrorInvalidValue;
    const long total = (long)n * c8 * H * W;
    hipLaunchKernelGGL(crop_copy_h_kernel, dim3(grid_for(total)), dim3(256), 0, stream, static_cast<const uint4v *>(src),
                       static_cast<uint4v *>(dst), n, c8, Hs, Ws, c8_total, o8_off, H, W, cy, cx);
    return hipGetLastError();
}

// Gather form of the pool gradient (s = 1): input unit (u, v) collects, per map, dY of the windows
// whose recorded winner it is.  Sums are formed in fp32 and rounded once.  relu_src (optional,
// same shape as dx) zeroes the result where the layer below produced a non-positive value (for k = 2 the codes say so).
// Any k; k = 2 comes here only where the grid of the chain form below would be too large.
template <int DT>
__global__ void maxpool_bwd_h_kernel(const uint4v *__restrict__ dy, const void *__restrict__ tap, const uint4v *__restrict__ relu_src,
                                     uint4v *__restrict__ dx, int H, int W, int Ho, int Wo, int k, int d)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x, u = blockIdx.y;
    if (v >= W) return;
    const long p = blockIdx.z;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    for (int i = 0; i < k; ++i) {
        const int yy = u - i * d;
        if (yy < 0 || yy >= Ho) continue;
        for (int j = 0; j < k; ++j) {
            const int xx = v - j * d;
            if (xx < 0 || xx >= Wo) continue;
            const long o = (p * Ho + yy) * Wo + xx;
            const uint4v g = dy[o];
            const unsigned want = i * k + j;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (pool_code_h(tap, o, e, pool_bits_h(k, 1)) == want) acc[e] += up16<DT>(elem16(g, e));
        }
    }
    const long q = (p * H + u) * W + v;
    unsigned hv[8];
    uint4v rs = uint4v{0u, 0u, 0u, 0u};
    if (relu_src) rs = relu_src[q];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float a = acc[e];
        if (relu_src && !(up16<DT>(elem16(rs, e)) > 0.f)) a = 0.f;
        hv[e] = down16<DT>(a);
    }
    dx[q] = uint4v{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16), hv[4] | (hv[5] << 16), hv[6] | (hv[7] << 16)};
}

// k = 2: a thread walks column v of dX down the rows u = y0, y0 + d, ... of one residue class, as the forward kernel walks
// its windows.  Row u collects from the windows of rows u (codes 0 at column v, 1 at column v - d) and u - d (codes 2, 3),
// so every window row is loaded once per walk and kept for the next step: 36 bytes read and 16 written per unit against
// 112 and 16 when each input unit fetched its four windows and the layer's output for the ReLU mask (MASKED takes that from
// the codes).  Bound by HBM (6 B read, 2 written per element and direction would be the least without codes) and, close
// behind, by the vector instructions that pick among 32 (element, window) pairs: with bit planes the codes of a unit are
// eight bitwise operations and a pick is a sign-extended bit, an AND and the addition.  48 maps of 8 x 1066^2: 562 -> 410 us
// (4.8 TB/s), the forward pass 447 -> 409; at 527x527 20.7 -> 15.8.
template <int DT, bool MASKED, int U>
__global__ void __launch_bounds__(256) maxpool2_bwd_chain_h_kernel(const uint4v *__restrict__ dy, const unsigned *__restrict__ tap,
                                                                   uint4v *__restrict__ dx, int H, int W, int Ho, int Wo, int d, int M, int nseg,
                                                                   int pblocks)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    const int sblock = blockIdx.y / pblocks, phase = (blockIdx.y - sblock * pblocks) * blockDim.y + threadIdx.y, seg = sblock * blockDim.z + threadIdx.z;
    if (v >= W || phase >= d || phase >= H || seg >= nseg) return;
    const int links = (H - phase + d - 1) / d, windows = links - 1;      // rows of this residue class, and of windows
    const int m0 = seg * M, m1 = min(links, m0 + M);
    if (m0 >= m1) return;
    const long p = blockIdx.z;
    // windows at column v and at column v - d (clamped into the row; `in`: all ones where the window exists)
    const unsigned xa = (unsigned)min(v, Wo - 1), xb = (unsigned)max(v - d, 0);
    const unsigned ina = v < Wo ? 0xffu : 0u, inb = v >= d ? 0xffu : 0u;
    struct Row {
        uint4v ga, gb;
        unsigned ca, cb;
    };
    const int row0 = windows > 0 ? phase : 0;             // (a class without windows reads row 0)
    auto load = [&](int l) {                              // window row l of the class, clamped into the map
        const long base = (p * Ho + row0 + (long)max(0, min(l, windows - 1)) * d) * Wo;
        Row r;
        r.ga = dy[base + xa];
        r.gb = dy[base + xb];
        r.ca = tap[base + xa];
        r.cb = tap[base + xb];
        return r;
    };
    // bit e of t[c]: element e of that window chose code c (c = 0, 2 at column v; 1, 3 at column v - d)
    auto picks = [&](const Row &r, int l, unsigned (&t)[4]) {
        const unsigned row = l >= 0 && l < windows ? 0xffu : 0u;
        const unsigned pa = (MASKED ? r.ca >> 16 : 0xffu) & ina & row, pb = (MASKED ? r.cb >> 16 : 0xffu) & inb & row;
        const unsigned a0 = pa & ~r.ca, b1 = pb & r.cb, la = r.ca >> 8, lb = r.cb >> 8;
        t[0] = a0 & ~la;
        t[1] = b1 & ~lb;
        t[2] = a0 & la;
        t[3] = b1 & lb;
    };
    auto pick = [](uint4v g, unsigned t, int e) {         // the element, or +0
        return __int_as_float(__float_as_int(up16<DT>(elem16(g, e))) & ((int)(t << (31 - e)) >> 31));
    };
    uint4v *dst = dx + (p * H + phase + (long)m0 * d) * W + v;
    const long ostep = (long)d * W;
    Row above = load(m0 - 1), r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = load(m0 + u);      // all in flight together
    unsigned ta[4];
    picks(above, m0 - 1, ta);
    for (int m = m0;;) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (m + u >= m1) break;
            unsigned t[4];
            picks(r[u], m + u, t);
            unsigned hv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                hv[e] = down16<DT>(((pick(r[u].ga, t[0], e) + pick(r[u].gb, t[1], e)) + pick(above.ga, ta[2], e)) + pick(above.gb, ta[3], e));
            dst[(long)u * ostep] = uint4v{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16), hv[4] | (hv[5] << 16), hv[6] | (hv[7] << 16)};
            above = r[u];
            ta[2] = t[2];
            ta[3] = t[3];
        }
        m += U;
        if (m >= m1) return;
        dst += (long)U * ostep;
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = load(m + u);
    }
}

template <int DT, bool MASKED>
static void launch_maxpool2_bwd_chain_h(const PoolCut &c, dim3 grid, hipStream_t stream, const void *dy, const void *tap, void *dx, int H, int W, int Ho,
                                        int Wo, int d)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, c.block(), 0, stream, static_cast<const uint4v *>(dy), static_cast<const unsigned *>(tap),
                           static_cast<uint4v *>(dx), H, W, Ho, Wo, d, c.len, c.nseg, c.pblocks);
    };
    if (c.len >= 4) go(&maxpool2_bwd_chain_h_kernel<DT, MASKED, 4>);
    else if (c.len >= 2) go(&maxpool2_bwd_chain_h_kernel<DT, MASKED, 2>);
    else go(&maxpool2_bwd_chain_h_kernel<DT, MASKED, 1>);
}

hipError_t launch_maxpool_bwd_h(const void *dy, const void *tap, const void *relu_src, void *dx, int dtype,
                                long planes8, int H, int W, int Ho, int Wo, int k, int d, hipStream_t stream)
{
    if (H > 65535 || planes8 > 65535) return hipErrorInvalidValue;
    const uint4v *g = static_cast<const uint4v *>(dy), *rs = static_cast<const uint4v *>(relu_src);
    uint4v *out = static_cast<uint4v *>(dx);
    if (k == 2 && Ho == H - d && Wo == W - d && Ho >= 1 && Wo >= 1) {
        const PoolCut c = pool_cut(H, W, d, planes8, POOL_WAVES);
        if (c.gy <= 65535) {
            const dim3 grid = c.grid(W, planes8);
            if (dtype == 1 && rs) launch_maxpool2_bwd_chain_h<1, true>(c, grid, stream, dy, tap, dx, H, W, Ho, Wo, d);
            else if (dtype == 1) launch_maxpool2_bwd_chain_h<1, false>(c, grid, stream, dy, tap, dx, H, W, Ho, Wo, d);
            else if (rs) launch_maxpool2_bwd_chain_h<2, true>(c, grid, stream, dy, tap, dx, H, W, Ho, Wo, d);
            else launch_maxpool2_bwd_chain_h<2, false>(c, grid, stream, dy, tap, dx, H, W, Ho, Wo, d);
            return hipGetLastError();
        }
    }
    const dim3 grid((W + 255) / 256, H, (unsigned)planes8);
    if (dtype == 1) hipLaunchKernelGGL(maxpool_bwd_h_kernel<1>, grid, dim3(256), 0, stream, g, tap, rs, out, H, W, Ho, Wo, k, d);
    else hipLaunchKernelGGL(maxpool_bwd_h_kernel<2>, grid, dim3(256), 0, stream, g, tap, rs, out, H, W, Ho, Wo, k, d);
    return hipGetLastError();
}

// Gradient of a pool with layer stride s = k at d = 1 (the U-Net pools, Section 3.4): the windows do not overlap, input
// unit (u, v) belongs to window (u / k, v / k) and takes that window's dY where it is the recorded winner; units beyond
// the last window get zero.  acc != 0: added to what dx holds (another consumer of the same map wrote first).  relu_src
// as in the gather form above (applied to the sum).
template <int DT>
__global__ void maxpool_stride_bwd_h_kernel(const uint4v *__restrict__ dy, const uint2v *__restrict__ tap, const uint4v *__restrict__ relu_src,
                                            uint4v *__restrict__ dx, int H, int W, int Ho, int Wo, int k, int acc)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x, u = blockIdx.y;
    if (v >= W) return;
    const long p = blockIdx.z;
    const int yy = u / k, xx = v / k;
    const unsigned want = (unsigned)((u - yy * k) * k + (v - xx * k));
    const long q = (p * H + u) * W + v;
    float a[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = 0.f;
    if (yy < Ho && xx < Wo) {
        const long o = (p * Ho + yy) * Wo + xx;
        const uint2v c = tap[o];
        const uint4v g = dy[o];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned code = (c[e >> 2] >> ((e & 3) * 8)) & 0xffu;
            if (code == want) a[e] = up16<DT>(elem16(g, e));
        }
    }
    if (acc) {
        const uint4v old = dx[q];
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] += up16<DT>(elem16(old, e));
    }
    uint4v rs = uint4v{0u, 0u, 0u, 0u};
    if (relu_src) rs = relu_src[q];
    unsigned hv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float t = a[e];
        if (relu_src && !(up16<DT>(elem16(rs, e)) > 0.f)) t = 0.f;
        hv[e] = down16<DT>(t);
    }
    dx[q] = uint4v{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16), hv[4] | (hv[5] << 16), hv[6] | (hv[7] << 16)};
}

hipError_t launch_maxpool_stride_bwd_h(const void *dy, const void *tap, const void *relu_src, void *dx, int dtype, long planes8, int H, int W,
                                       int Ho, int Wo, int k, int acc, hipStream_t stream)
{
    if (H > 65535 || planes8 > 65535 || k < 1 || (dtype != 1 && dtype != 2) || Ho * k > H || Wo * k > W) return hipErrorInvalidValue;
    const dim3 grid((W + 255) / 256, H, (unsigned)planes8);
    const uint4v *g = static_cast<const uint4v *>(dy), *rs = static_cast<const uint4v *>(relu_src);
    const uint2v *tp = static_cast<const uint2v *>(tap);
    uint4v *out = static_cast<uint4v *>(dx);
    if (dtype == 1) hipLaunchKernelGGL(maxpool_stride_bwd_h_kernel<1>, grid, dim3(256), 0, stream, g, tp, rs, out, H, W, Ho, Wo, k, acc);
    else hipLaunchKernelGGL(maxpool_stride_bwd_h_kernel<2>, grid, dim3(256), 0, stream, g, tp, rs, out, H, W, Ho, Wo, k, acc);
    return hipGetLastError();
}

// Backward of the 2x2 stride-2 up-convolution (Section 3.4), first step: the gradient of the merged buffer's first c8
// octets (the up path; the buffer has c8_total octets of 2h x 2w) as four interleaved sub-images stacked along the maps:
// out[b][t * c8 + o][y][x] = in[b][o][2y + t/2][2x + t%2].  Bits are moved, nothing is rounded.
__global__ void space_to_depth2_h_kernel(const uint4v *__restrict__ in, uint4v *__restrict__ out, int n, int c8_total, int c8, int h, int w)
{
    const long plane = (long)h * w, total = (long)n * 4 * c8 * plane;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const long pix = q % plane, r = q / plane;
        const int x = (int)(pix % w), y = (int)(pix / w);
        const int o4 = (int)(r % (4 * c8)), t = o4 / c8, o = o4 - t * c8;
        const long b = r / (4 * c8);
        out[q] = in[((b * c8_total + o) * (2 * h) + 2 * y + (t >> 1)) * (2L * w) + 2 * x + (t & 1)];
    }
}

hipError_t launch_space_to_depth2_h(const void *in, void *out, int n, int c8_total, int c8, int h, int w, hipStream_t stream)
{
    if (n < 1 || c8 < 1 || c8 > c8_total || h < 1 || w < 1) return hipErrorInvalidValue;
    const long total = (long)n * 4 * c8 * h * w;
    hipLaunchKernelGGL(space_to_depth2_h_kernel, dim3(grid_for(total)), dim3(256), 0, stream, static_cast<const uint4v *>(in),
                       static_cast<uint4v *>(out), n, c8_total, c8, h, w);
    return hipGetLastError();
}

// MergeCrop's backward into the skip map (Section 5.3.1, when enabled): dst [n][c8][Hd][Wd] takes octets o8_off .. of
// src [n][c8_total][Hs][Ws] in its centre window (offset cy, cx) and zero elsewhere
__global__ void place_h_kernel(const uint4v *__restrict__ src, uint4v *__restrict__ dst, int n, int c8, int Hd, int Wd, int c8_total,
                               int o8_off, int Hs, int Ws, int cy, int cx)
{
    const long plane = (long)Hd * Wd, total = (long)n * c8 * plane;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const long pix = q % plane, r = q / plane;
        const int x = (int)(pix % Wd) - cx, y = (int)(pix / Wd) - cy;
        const int o = (int)(r % c8);
        const long b = r / c8;
        uint4v v = uint4v{0u, 0u, 0u, 0u};
        if (x >= 0 && x < Ws && y >= 0 && y < Hs) v = src[((b * c8_total + o8_off + o) * Hs + y) * Ws + x];
        dst[q] = v;
    }
}

hipError_t launch_place_h(const void *src, void *dst, int n, int c8, int Hd, int Wd, int c8_total, int o8_off, int Hs, int Ws, int cy,
                          int cx, hipStream_t stream)
{
    if (cy < 0 || cx < 0 || cy + Hs > Hd || cx + Ws > Wd || o8_off < 0 || o8_off + c8 > c8_total || n < 1) return hipErrorInvalidValue;
    const long total = (long)n * c8 * Hd * Wd;
    hipLaunchKernelGGL(place_h_kernel, dim3(grid_for(total)), dim3(256), 0, stream, static_cast<const uint4v *>(src), static_cast<uint4v *>(dst),
                       n, c8, Hd, Wd, c8_total, o8_off, Hs, Ws, cy, cx);
    return hipGetLastError();
}

// winner codes on the octet layout -> flat input offsets, int32 NCHW (for the parity accessor)
__global__ void tap_to_index_h_kernel(const void *tap, int32_t *idx, int n, int c, int Ho, int Wo, int W, int k, int d, int s)
{
    const int c8 = (c + 7) / 8;
    const long plane = (long)Ho * Wo, total = (long)n * c8 * plane;
    for (long q = blockIdx.x * (long)blockDim.x + threadIdx.x; q < total; q += (long)gridDim.x * blockDim.x) {
        const long pix = q % plane;
        const int xx = (int)(pix % Wo), yy = (int)(pix / Wo);
        const long t = q / plane;
        const int o = (int)(t % c8);
        const long b = t / c8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (o * 8 + e >= c) continue;
            const int code = (int)pool_code_h(tap, q, e, pool_bits_h(k, s)), i = code / k, j = code - i * k;
            idx[(b * c + o * 8 + e) * plane + pix] = (s * yy + i * d) * W + s * xx + j * d;
        }
    }
}

hipError_t launch_tap_to_index_h(const void *tap, int32_t *idx, int n, int c, int Ho, int Wo, int W, int k, int d, int s,
                                 hipStream_t stream)
{
    const long total = (long)n * ((c + 7) / 8) * Ho * Wo;
    hipLaunchKernelGGL(tap_to_index_h_kernel, dim3(grid_for(total)), dim3(256), 0, stream, tap, idx, n, c, Ho, Wo, W, k, d, s);
    return hipGetLastError();
}

// db[o] = sum over images and pixels of dY (octet layout), in two stages with a fixed summation
// order: workgroup (s, octet) sums slice s of the pixels of its octet over all images into
// part[(8*octet + e) * slices + s]; wgrad_reduce_kernel (kernels_wgrad_f32.hip) adds the slices.
template <int DT>
__global__ void __launch_bounds__(256) bias_grad_h_kernel(const uint4v *__restrict__ dy, float *__restrict__ part, int n, int c,
                                                          long plane, int slices)
{
    __shared__ float sh[4][8];
    const int c8 = (c + 7) / 8, o = blockIdx.y, sl = blockIdx.x;
    const long per = (plane + slices - 1) / slices, q0 = sl * per, q1 = q0 + per < plane ? q0 + per : plane;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.f;
    for (int b = 0; b < n; ++b) {
        const uint4v *src = dy + ((long)b * c8 + o) * plane;
        for (long q = q0 + threadIdx.x; q < q1; q += 256) {
            const uint4v u = src[q];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += up16<DT>(elem16(u, e));
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        for (int off = 32; off > 0; off >>= 1) v[e] += __shfl_down(v[e], off, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][e] = v[e];
    }
    __syncthreads();
    if (threadIdx.x < 8)
        part[(long)(o * 8 + threadIdx.x) * slices + sl] = sh[0][threadIdx.x] + sh[1][threadIdx.x] + sh[2][threadIdx.x] + sh[3][threadIdx.x];
}

hipError_t launch_bias_grad_h(const void *dy, float *part, int dtype, int n, int c, long plane, int slices, hipStream_t stream)
{
    const dim3 grid(slices, (c + 7) / 8);
    if (dtype == 1)
        hipLaunchKernelGGL(bias_grad_h_kernel<1>, grid, dim3(256), 0, stream, static_cast<const uint4v *>(dy), part, n, c, plane, slices);
    else
        hipLaunchKernelGGL(bias_grad_h_kernel<2>, grid, dim3(256), 0, stream, static_cast<const uint4v *>(dy), part, n, c, plane, slices);
    return hipGetLastError();
}

}  // namespace sk
