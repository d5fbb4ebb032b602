// 16-bit 1x1 layers of at most sixteen output maps whose sums are stored as fp32: the classes of a net that does not end in a fused head.
//
// Bound by the maps they read (64 maps: 128 bytes a pixel for two classes).  The octet layout is the MFMA's B operand as it stands: lane (g, l16)
// loads the eight maps of octet 4 chunk + g of pixel l16, so nothing but the weights goes through LDS and there is no tile to fill: a wave takes N
// runs of sixteen pixels of the flattened plane, and has the chunks of the next batch on the way while it multiplies this one's.  On the
// convolutions' tiles of 128 x 4 pixels a 128^2 map was 32 tiles, each a chain of 16 chunks.  Sums, order and bias are those of the
// convolutions, bit for bit.
// bf16, us before and here: 512 -> 2 at 128^2 24.9 -> 6.6, 64 -> 2 at 388^2 13.3 -> 7.1, at 508^2 15.2 -> 9.9, on 65 slices of 129^2 40.3 -> 26.0
// (5.7 TB/s).
#include "conv_wide.h"

namespace sk {

namespace {

constexpr int H1_THREADS = 256, H1_WAVES = 4, H1_MAX_CHUNKS = 64;        // 64 KB of weights

struct H1Args {
    const void *x, *wp;
    const float *bias;
    float *y;
    long x_image;                       // 16-byte units from one image to the next
    int c8_in, c_out, plane, relu, nchunks, frag_step, per_image, total;
};

// N runs of sixteen pixels a wave, U chunks of 32 input maps a batch
template <int DT, int N, int U>
__global__ __launch_bounds__(H1_THREADS, 2) void conv1x1_few_h_kernel(H1Args a)
{
    extern __shared__ uint4v wl[];
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int batches = (a.nchunks + U - 1) / U, stride = gridDim.x * H1_WAVES;
    const uint4v zero = uint4v{0u, 0u, 0u, 0u};
    int grp = blockIdx.x * H1_WAVES + wave;
    const bool any = grp < a.total;
    auto load = [&](uint4v (&x)[U][N], int group, int k) {
        const int b = group / a.per_image, px0 = (group - b * a.per_image) * 16 * N;
        const uint4v *img = static_cast<const uint4v *>(a.x) + (long)b * a.x_image;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int oct = 4 * (k * U + u) + g;
            const uint4v *p = img + (long)min(oct, a.c8_in - 1) * a.plane;
#pragma unroll
            for (int j = 0; j < N; ++j) x[u][j] = p[min(px0 + 16 * j + l16, a.plane - 1)];
        }
    };
    uint4v x[U][N], xn[U][N];
    if (any) load(x, grp, 0);
    for (int q = threadIdx.x; q < batches * U * 64; q += H1_THREADS)        // (the map tile's fragments only; zeros behind the last chunk)
        wl[q] = (q >> 6) < a.nchunks ? static_cast<const uint4v *>(a.wp)[(long)(q >> 6) * a.frag_step + (q & 63)] : zero;
    float bia[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) bia[r] = a.bias ? a.bias[4 * g + r] : 0.f;
    __syncthreads();
    if (!any) return;
    while (true) {
        floatx4 acc[N];
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
        const bool more = grp + stride < a.total;
        for (int k = 0; k < batches; ++k) {
            if (k + 1 < batches) load(xn, grp, k + 1);
            else if (more) load(xn, grp + stride, 0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint4v w = wl[(k * U + u) * 64 + lane];
                const bool real = 4 * (k * U + u) + g < a.c8_in;
#pragma unroll
                for (int j = 0; j < N; ++j) acc[j] = wide_mfma<DT>(w, real ? x[u][j] : zero, acc[j]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < N; ++j) x[u][j] = xn[u][j];
        }
        const int b = grp / a.per_image, px0 = (grp - b * a.per_image) * 16 * N;
        float *dst = a.y + ((long)b * a.c_out + 4 * g) * a.plane;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int px = px0 + 16 * j + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float v = acc[j][r] + bia[r];
                if (a.relu) v = fmaxf(v, 0.f);
                if (px < a.plane && 4 * g + r < a.c_out) dst[(long)r * a.plane + px] = v;
            }
        }
        if (!more) return;
        grp += stride;
    }
}

template <int DT, int N, int U> hipError_t launch_few(H1Args a, int n, hipStream_t stream)
{
    a.per_image = (a.plane + 16 * N - 1) / (16 * N);
    a.total = n * a.per_image;
    const size_t smem = (size_t)(a.nchunks + U - 1) / U * U * 1024;
    static bool set;
    if (smem > 48 * 1024 && !set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv1x1_few_h_kernel<DT, N, U>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (H1_MAX_CHUNKS + U) * 1024);
        if (e != hipSuccess) return e;
        set = true;
    }
    const int per_cu = smem <= 36 * 1024 ? 4 : 2, blocks = std::min((a.total + H1_WAVES - 1) / H1_WAVES, per_cu * wide_cus());
    hipLaunchKernelGGL((conv1x1_few_h_kernel<DT, N, U>), dim3(blocks), dim3(H1_THREADS), smem, stream, a);
    return hipGetLastError();
}

template <int DT> hipError_t launch_few_dt(const H1Args &a, int n, hipStream_t stream)
{
    // runs of a wave: as many as still give every SIMD two waves
    const long runs = (long)n * ((a.plane + 15) / 16), waves = 8L * wide_cus();
    if (runs >= 4 * waves) return launch_few<DT, 4, 2>(a, n, stream);
    if (runs >= 2 * waves) return launch_few<DT, 2, 4>(a, n, stream);
    return launch_few<DT, 1, 8>(a, n, stream);
}

}  // namespace

// Whole planes in and out, fp32 sums, one map tile; results below 2 GB an image, as on the convolutions' kernels.  90 layers of 8 to 1600 -> 1 to 16 maps,
// 20 x 30 to 1000 x 1010: 0.12 to 0.88 of their time, so there is no line between the two
bool conv1x1_few_h_applies(const ConvHArgs &a)
{
    return a.k == 1 && a.out_f32 && a.c_out <= 16 && !a.mask && a.in_off == 0 && !a.vpool && !a.hd && !a.grp8 && a.tap_maps == 0 && !a.img && a.H == a.Ho &&
           a.W == a.Wo && a.OH == a.Ho && a.OW == a.Wo && a.oy_mul == 1 && a.ox_mul == 1 && a.oy_off == 0 && a.ox_off == 0 &&
           (a.c8_in + 3) / 4 <= H1_MAX_CHUNKS && 4L * a.c_out * a.Ho * a.Wo < 0x7fffffffL && a.n * (((long)a.Ho * a.Wo + 15) / 16) <= 0x3fffffffL;
}

// mt: map tiles a group that the weights were packed for
hipError_t launch_conv1x1_few_h(const ConvHArgs &c, int mt, hipStream_t stream)
{
    if (!conv1x1_few_h_applies(c) || c.n < 1 || mt < 1) return hipErrorInvalidValue;
    H1Args a;
    a.x = c.x; a.wp = c.wp; a.bias = c.bias; a.y = static_cast<float *>(c.y);
    a.plane = c.Ho * c.Wo;
    a.x_image = (long)(c.xb8 ? c.xb8 : c.c8_in) * a.plane;
    a.c8_in = c.c8_in; a.c_out = c.c_out; a.relu = c.relu;
    a.nchunks = (c.c8_in + 3) / 4;
    a.frag_step = mt * 64;
    a.per_image = a.total = 0;
    if (c.dtype == 1) return launch_few_dt<1>(a, c.n, stream);
    if (c.dtype == 2) return launch_few_dt<2>(a, c.n, stream);
    return hipErrorInvalidValue;
}

}  // namespace sk
