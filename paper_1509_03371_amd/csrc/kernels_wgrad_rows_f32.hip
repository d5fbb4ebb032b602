// fp32 weight and bias gradient of 4x4 SK convolutions with 8 to 48 input and at most 48 output maps (gfx950, MFMA 16x16x4 fp32):
// input rows kept in LDS from one output row to the next.
//
//   dW[o][c][i][j] = sum_{b,y,x} dY[b,o,y,x] * X[b,c,y+i*d,x+j*d]        db[o] = sum dY[b,o,y,x]
//
// The multiplication takes 7.7 us for 64 output pixels x 48 -> 48 maps of a CU; wgrad_f32_kernel spends twice that again on
// staging, because it loads all four input rows of every output row (each input row four times) with one float a lane: some 600
// memory instructions a segment, each of which holds the CU's memory pipeline for tens of cycles.  Here a workgroup walks down a
// strip of 64 output columns along the rows y, y + d, y + 2d, ... of one residue class of the kernel stride, so that consecutive
// steps share three of their four input rows: the rows stand in a ring of five LDS slots per map, a step loads ONE new input row
// and one dY row, sixteen bytes a lane (about 30 instructions), into registers before its MFMAs and writes them to LDS behind them.
//
// A column tile of the product is the sixteen taps (i, j) of one input map; wave w of eight takes NBW maps and all MB map tiles of
// dY: MB + NBW four-byte LDS reads for MB * NBW MFMAs of 32 cycles.  Row and slot pitches spread the 64 addresses of a read over the
// banks (two a bank).  Steps are dealt out in equal contiguous ranges; a range writes one private copy, which wgrad_reduce_kernel
// sums in a fixed order.  The sums of dY come from the registers that its rows pass through.
//
// 48 -> 48 maps at 527^2 .. 557^2, without the 20 us of bias_grad_kernel that fell away too: 345 .. 424 -> 184 .. 211 us with the reduction
// (105 TFLOP/s); 8 x 1047^2 11.3 -> 5.5 ms.  A step is 10.1 us where its MFMAs are 7.7 at 2.4 GHz (8.2 at the 2.26 GHz fp32 MFMAs run at).
#include <algorithm>

#include "sk_kernels.h"

namespace sk {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));      // sixteen bytes at any float

constexpr int RF_WAVES = 8, RF_THREADS = 64 * RF_WAVES;
constexpr int RF_SEG = 64;               // output columns of a strip
constexpr int RF_DYP = RF_SEG + 4;       // LDS pitch of a dY row
constexpr int RF_SLOTS = 5;              // input rows of a map in LDS: four in use, one arriving
constexpr int RF_MAXB = 6, RF_MAXM = 3;  // input maps of a wave, 16-map tiles of dY

struct Args {
    const float *x, *dy;
    float *scratch, *bias_part;          // bias_part[map * gridDim.x + workgroup], or nullptr
    int n, c_in, c_out, H, W, d, Ho, Wo;
    int xsegs, total;                    // strips across; steps = output rows x strips x images
    int nq, pitch;                       // staged 16-byte units of an input row, LDS pitch (floats) of a slot
};

template <int MB, int NBW>
__global__ __launch_bounds__(RF_THREADS, 2) void wgrad_rows_f32_kernel(Args a)
{
    extern __shared__ float smem[];
    constexpr int XU = NBW >= 4 ? 3 : (NBW >= 2 ? 2 : 1), YU = (MB * 16 * 16 + RF_THREADS - 1) / RF_THREADS;   // 16-byte units a thread stages
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int map_pitch = RF_SLOTS * a.pitch;
    float *const xs = smem, *const dys = smem + a.c_in * map_pitch;          // [c_in][slot][pitch], two of [MB*16][RF_DYP]
    const long xplane = (long)a.H * a.W, yplane = (long)a.Ho * a.Wo;

    // this thread's units of an input row (map, four columns) and of a dY row
    int xc[XU], xq[XU];
#pragma unroll
    for (int u = 0; u < XU; ++u) {
        const int idx = tid + RF_THREADS * u;
        xc[u] = idx / a.nq;
        xq[u] = 4 * (idx - xc[u] * a.nq);
    }
    const int yq = 4 * (tid & 15), yo = tid >> 4;                            // maps yo, yo + 32
    // four columns of a row from column x on; zeros from column `width` on
    auto load4 = [](const float *row, int x, int width) {
        if (x + 3 < width) return floatx4(*reinterpret_cast<const float4u *>(row + x));
        floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
        if (x < width) v[0] = row[x];
        if (x + 1 < width) v[1] = row[x + 1];
        if (x + 2 < width) v[2] = row[x + 2];
        return v;
    };
    floatx4 px[XU], py[YU];
    float bsum[YU] = {};
    auto load_x = [&](int b, int y, int x0) {
#pragma unroll
        for (int u = 0; u < XU; ++u)
            if (xc[u] < a.c_in) px[u] = load4(a.x + ((long)b * a.c_in + xc[u]) * xplane + (long)y * a.W, x0 + xq[u], a.W);
    };
    auto store_x = [&](int slot) {
#pragma unroll
        for (int u = 0; u < XU; ++u)
            if (xc[u] < a.c_in) *reinterpret_cast<floatx4 *>(xs + xc[u] * map_pitch + slot * a.pitch + xq[u]) = px[u];
    };
    auto load_dy = [&](int b, int y, int x0) {
#pragma unroll
        for (int u = 0; u < YU; ++u) {
            py[u] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (yo + 32 * u < a.c_out) py[u] = load4(a.dy + ((long)b * a.c_out + yo + 32 * u) * yplane + (long)y * a.Wo, x0 + yq, a.Wo);
        }
    };
    auto store_dy = [&](int buf) {
#pragma unroll
        for (int u = 0; u < YU; ++u) {
            if (yo + 32 * u < MB * 16) *reinterpret_cast<floatx4 *>(dys + (buf * MB * 16 + yo + 32 * u) * RF_DYP + yq) = py[u];
            bsum[u] += (py[u][0] + py[u][1]) + (py[u][2] + py[u][3]);
        }
    };

    floatx4 acc[MB][NBW];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int q = 0; q < NBW; ++q) acc[m][q] = floatx4{0.f, 0.f, 0.f, 0.f};
    // B operand: tap (i, j) = (l16 / 4, l16 % 4) of map wave * NBW + q (beyond the last map: the last one, nobody reads the sums)
    const int ti = l16 >> 2, bcol = (l16 & 3) * a.d + g;
    const float *bmap[NBW];
#pragma unroll
    for (int q = 0; q < NBW; ++q) bmap[q] = xs + min(wave * NBW + q, a.c_in - 1) * map_pitch + bcol;
    const float *const arow = dys + l16 * RF_DYP + g;
    auto multiply = [&](int slot0, int buf, int p0) {        // half of the output row whose first input row stands in slot0
        const int s = slot0 + ti, off = (s >= RF_SLOTS ? s - RF_SLOTS : s) * a.pitch;
        const float *ar = arow + buf * MB * 16 * RF_DYP;
#pragma unroll 4
        for (int p = p0; p < p0 + RF_SEG / 2; p += 4) {
            float av[MB], bv[NBW];
#pragma unroll
            for (int m = 0; m < MB; ++m) av[m] = ar[m * 16 * RF_DYP + p];
#pragma unroll
            for (int q = 0; q < NBW; ++q) bv[q] = bmap[q][off + p];
#pragma unroll
            for (int q = 0; q < NBW; ++q)
#pragma unroll
                for (int m = 0; m < MB; ++m) acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[m], bv[q], acc[m][q], 0, 0, 0);
        }
    };

    // workgroup ids go round-robin over the 8 XCDs: XCD x takes the x-th eighth of the ranges, neighbours share rows in its L2
    const int blk = gridDim.x % 8 == 0 ? (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) : (int)blockIdx.x;
    int s = (int)((long)a.total * blk / gridDim.x);
    const int s_end = (int)((long)a.total * (blk + 1) / gridDim.x);
    const int q = a.Ho / a.d, rem = a.Ho % a.d;              // rows of a residue class: q + 1 in the first rem, q in the others
    while (s < s_end) {
        // the part of a strip's walk that starts at step s: image b, columns x0 .., `count` rows from y on
        const int t = s / a.Ho, yy = s - t * a.Ho, b = t / a.xsegs, x0 = (t - b * a.xsegs) * RF_SEG;
        int phase, m, rows;
        if (yy < rem * (q + 1)) {
            rows = q + 1;
            phase = yy / rows;
            m = yy - phase * rows;
        } else {
            rows = q;
            const int y2 = yy - rem * (q + 1);
            phase = y2 / rows;
            m = y2 - phase * rows;
            phase += rem;
        }
        const int count = min(rows - m, s_end - s), y0 = phase + m * a.d;
        s += count;
        __syncthreads();                                     // the previous walk's last row has been multiplied
        load_dy(b, y0, x0);
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            load_x(b, y0 + i * a.d, x0);
            store_x(i);
        }
        store_dy(0);
        __syncthreads();
        int slot = 0;
        for (int r = 0; r < count; ++r) {
            const bool more = r + 1 < count;
            if (more) {                                      // in flight while this row is multiplied
                load_x(b, y0 + (r + 4) * a.d, x0);
                load_dy(b, y0 + (r + 1) * a.d, x0);
            }
            multiply(slot, r & 1, 0);
            if (more) {                                      // (half a row on the loads have landed, and no wave waits for the writes)
                store_x(slot == 0 ? RF_SLOTS - 1 : slot - 1);      // the slot that fell free with the previous row
                store_dy((r + 1) & 1);
            }
            multiply(slot, r & 1, RF_SEG / 2);
            slot = slot + 1 == RF_SLOTS ? 0 : slot + 1;
            if (more) __syncthreads();
        }
    }

    // private copy [map tile * 16 + row][16 * c_in], as wgrad_reduce_kernel reads it
    const long ncols = 16L * a.c_in;
    float *dst = a.scratch + (long)blockIdx.x * (MB * 16) * ncols;
#pragma unroll
    for (int qq = 0; qq < NBW; ++qq) {
        const int c = wave * NBW + qq;
        if (c >= a.c_in) break;
#pragma unroll
        for (int mm = 0; mm < MB; ++mm)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) dst[(long)(mm * 16 + 4 * g + r4) * ncols + c * 16 + l16] = acc[mm][qq][r4];
    }
    if (a.bias_part) {
#pragma unroll
        for (int u = 0; u < YU; ++u) {
            float v = bsum[u];
#pragma unroll
            for (int sh = 8; sh > 0; sh >>= 1) v += __shfl_xor(v, sh, 16);
            if ((tid & 15) == 0 && yo + 32 * u < a.c_out) a.bias_part[(long)(yo + 32 * u) * gridDim.x + blockIdx.x] = v;
        }
    }
}

// LDS pitch of a slot: at kernel strides that are multiples of 8 the four columns of a read lie eight banks apart and slots go into
// the gaps; otherwise they fill less than half of the banks and slots alternate between the halves
int rf_pitch(int d)
{
    const int units = (RF_SEG + 3 * d + 3) / 4 * 4, want = d % 8 == 0 ? 4 : 16;
    return units + ((want - units) % 32 + 32) % 32;
}

size_t rf_smem(int c_in, int c_out, int d)
{
    return sizeof(float) * ((size_t)c_in * RF_SLOTS * rf_pitch(d) + 2 * (size_t)((c_out + 15) / 16 * 16) * RF_DYP);
}

template <int MB, int NBW>
hipError_t launch_t(const Args &a, size_t smem, int blocks, hipStream_t stream)
{
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad_rows_f32_kernel<MB, NBW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((wgrad_rows_f32_kernel<MB, NBW>), dim3(blocks), dim3(RF_THREADS), smem, stream, a);
    return hipGetLastError();
}

template <int MB>
hipError_t launch_m(const Args &a, size_t smem, int blocks, hipStream_t stream)
{
    switch ((a.c_in + RF_WAVES - 1) / RF_WAVES) {
    case 1: return launch_t<MB, 1>(a, smem, blocks, stream);
    case 2: return launch_t<MB, 2>(a, smem, blocks, stream);
    case 3: return launch_t<MB, 3>(a, smem, blocks, stream);
    case 4: return launch_t<MB, 4>(a, smem, blocks, stream);
    case 5: return launch_t<MB, 5>(a, smem, blocks, stream);
    case 6: return launch_t<MB, 6>(a, smem, blocks, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// a thread stages at most XU units of an input row: c_in rows of (64 + 3d) / 4 units among 512 threads
bool wgrad_rows_f32_supported(int c_in, int c_out, int k, int d)
{
    if (k != 4 || d < 1 || c_in < RF_WAVES || c_in > RF_WAVES * RF_MAXB || c_out < 1 || c_out > 16 * RF_MAXM) return false;
    const int nbw = (c_in + RF_WAVES - 1) / RF_WAVES, xu = nbw >= 4 ? 3 : (nbw >= 2 ? 2 : 1), nq = (RF_SEG + 3 * d + 3) / 4;
    return c_in * nq <= RF_THREADS * xu && rf_smem(c_in, c_out, d) <= 160 * 1024;
}

hipError_t launch_wgrad_rows_f32(const float *x, const float *dy, float *scratch, float *bias_part, int n, int c_in, int H, int W, int c_out, int d,
                                 int max_copies, int *copies, hipStream_t stream)
{
    Args a;
    a.x = x; a.dy = dy; a.scratch = scratch; a.bias_part = bias_part;
    a.n = n; a.c_in = c_in; a.c_out = c_out; a.H = H; a.W = W; a.d = d; a.Ho = H - 3 * d; a.Wo = W - 3 * d;
    if (!wgrad_rows_f32_supported(c_in, c_out, 4, d) || n < 1 || a.Ho < 1 || a.Wo < 1 || max_copies < 1) return hipErrorInvalidValue;
    a.xsegs = (a.Wo + RF_SEG - 1) / RF_SEG;
    const long total = (long)n * a.xsegs * a.Ho;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    a.total = (int)total;
    a.nq = (RF_SEG + 3 * d + 3) / 4;
    a.pitch = rf_pitch(d);
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    *copies = (int)std::min<long>(std::min(cus, max_copies), total);
    const size_t smem = rf_smem(c_in, c_out, d);
    switch ((c_out + 15) / 16) {
    case 1: return launch_m<1>(a, smem, *copies, stream);
    case 2: return launch_m<2>(a, smem, *copies, stream);
    default: return launch_m<3>(a, smem, *copies, stream);
    }
}

}  // namespace sk
