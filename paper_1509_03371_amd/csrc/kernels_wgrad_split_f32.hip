// fp32 weight and bias gradient of 4x4 SK convolutions of at most 48 maps on either side, on the 16-bit matrix unit of gfx950.
//
//   dW[o][c][i][j] = sum_{b,y,x} dY[b,o,y,x] * X[b,c,y+i*d,x+j*d]        db[o] = sum dY[b,o,y,x]
//
// The walks of kernels_wgrad_rows_h.hip (strips of 64 output columns, down the rows of one phase of the kernel stride; operands turned by
// the transposing LDS read; wave w takes tap column w % 4 and half w / 4 of the strip) on pairs of fp16 values (split_f32.h): a step loads
// one input row and one gradient row into registers, a unit (pixel, eight maps) at a time, while the rows before are multiplied, and writes
// the pairs to LDS.  Input rows alternate between two buffers; gradient rows stand in a ring of five, where a step reads the four that
// meet its input row.  A product is three MFMAs.  Every row has a scale of its own, from its largest magnitude; the products of a step are summed apart
// and added to the gradient by the vector unit, which undoes the scales of the two rows and rounds to nearest (sums left in the matrix unit over hundreds
// of steps came out 1.1 times as far off as fp32 operands', 4 x 676^2; so they are half as far).  Where a sample of either row is infinite or would be
// held in fewer bits as a pair (split_f32.h), the fp32 matrix unit multiplies the two rows, from memory.
//
// What bounds it: a step of 64 pixels is 108 MFMAs a wave, 3456 cycles a SIMD, 2300 cycles of LDS reads and 2600 of vector instructions, in
// two waves a SIMD that meet at a barrier a step: 7000 cycles, MFMAs in 0.45 of them.  48 -> 48 maps, on the fp32 matrix unit and here, with the
// reduction: 537^2 d = 2 217 -> 105 to 112 us, 4 x 676^2 d = 8 1139 -> 492; with every row on the fp32 unit 0.9 to 1.1 times the former.
// Tried: the loads of a row one step ahead instead of two (a quarter slower); half of the waves staging while the others multiply: no difference; the fp32
// unit's sums in the private copy, in memory (131 us for 97, spills); all input map tiles' sums of a step at once (116, spills drain the loads under way).
#include <algorithm>

#include "lds_dma.h"
#include "sk_kernels.h"
#include "split_f32.h"

namespace sk {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));      // sixteen bytes at any float
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));

constexpr int WS_TX = 64, WS_WAVES = 8, WS_RING = 5;
constexpr int WS_DP = 68;            // LDS pitch (units) between the octets of a row: octet o + 1 lands 16 banks further
constexpr unsigned WS_NOWHERE = 0xfffffff0u;
constexpr int WS_MOST = 63;           // rows' powers of two are in +-63, so that the sum of two is one of fp32's

struct Args {
    const float *x, *dy;
    float *scratch, *bias_part;
    int n, c_in, c_out, c8i, c8o, H, W, Ho, Wo, d;
    int pw, xp;                      // staged columns of an input row, LDS pitch between its octets
    int xgroups;                     // loads of 64 units of an input row
    int xstrips, total_rows, copy_floats;
};

struct Walk {
    int b, x0, py, r0, rows;         // rows: gradient rows of this walk (it has rows + 3 steps)
};

// one operand fragment: 16 maps x 32 pixels, this lane's 8 pixels of its map (two transposing reads, 4 pixels each)
__device__ __forceinline__ uint4v read_frag(const char *lds, unsigned off)
{
    typedef short4v __attribute__((address_space(3))) *lds_s4;
    const uint2v lo = __builtin_bit_cast(uint2v, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(lds + off)));
    const uint2v hi = __builtin_bit_cast(uint2v, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(lds + off + 64)));
    return uint4v{lo[0], lo[1], hi[0], hi[1]};
}

template <int MT, int NCT>
__global__ __launch_bounds__(64 * WS_WAVES) void wgrad_split_f32_kernel(Args a)
{
    extern __shared__ uint4v smem16[];
    char *lds = reinterpret_cast<char *>(smem16);
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, jl = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tapj = wave & 3, ip = wave >> 2, d = a.d;
    // [buffer][part][octet][xp] input rows, [slot][part][octet][WS_DP] gradient rows, then ranges [2][input, gradient][most, least][wave]
    const int x_part = a.c8i * a.xp * 16, x_buf = 2 * x_part, y_part = a.c8o * WS_DP * 16, y_slot = 2 * y_part, y_base = 2 * x_buf;
    unsigned *ranges = reinterpret_cast<unsigned *>(lds + y_base + WS_RING * y_slot);

    // this lane's read offsets inside a part (lane 4r + q of a 16-lane group names pixel r, map quad q)
    const int rr = jl >> 2, q = jl & 3, pix = 8 * g + rr;
    unsigned a_off[MT], b_off[NCT];
#pragma unroll
    for (int m = 0; m < MT; ++m) a_off[m] = (unsigned)((min(2 * m + (q >> 1), a.c8o - 1) * WS_DP + pix) * 16 + (q & 1) * 8);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) b_off[ct] = (unsigned)((min(2 * ct + (q >> 1), a.c8i - 1) * a.xp + pix + tapj * d) * 16 + (q & 1) * 8);

    // This workgroup's rows: an equal share of all (image, strip, phase, row in the phase), in walks that end with their phase or the share.
    const int row_begin = (int)((long)a.total_rows * blockIdx.x / gridDim.x), row_end = (int)((long)a.total_rows * (blockIdx.x + 1) / gridDim.x);
    const int short_rows = a.Ho / d, long_phases = a.Ho % d;     // rows of a phase: one more in the first ones
    auto decode = [&](int row) {                                 // the walk that starts at a row of the share
        Walk w{};
        if (row >= row_end) return w;
        const int strip = row / a.Ho, yy = row - strip * a.Ho;
        w.b = strip / a.xstrips;
        w.x0 = (strip - w.b * a.xstrips) * WS_TX;
        int rows = short_rows + 1;
        if (yy < long_phases * rows) {
            w.py = yy / rows;
            w.r0 = yy - w.py * rows;
        } else {
            const int y2 = yy - long_phases * rows;
            rows = short_rows;
            w.py = y2 / rows;
            w.r0 = y2 - w.py * rows;
            w.py += long_phases;
        }
        w.rows = min(rows - w.r0, row_end - row);
        return w;
    };

    // A wave stages two groups of 64 units (pixel, eight maps).  Groups 0 .. c8o - 1 (first groups only) are the gradient row's octets, the
    // others the input row's units, octet after octet
    const long xplane = (long)a.H * a.W, yplane = (long)a.Ho * a.Wo;
    const bool grad = wave < a.c8o;                              // is the first group the gradient's?
    bool mine[2];
    int col[2], dst[2];
    unsigned plane_off[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const bool y = u == 0 && grad;
        const int id = wave + WS_WAVES * u, L = (id - a.c8o) * 64 + lane, o8 = y ? id : L / a.pw;
        col[u] = y ? lane : L - o8 * a.pw;
        mine[u] = y || (id < a.c8o + a.xgroups && o8 < a.c8i);
        plane_off[u] = 4u * (unsigned)(o8 * 8) * (unsigned)(y ? yplane : xplane);
        dst[u] = (o8 * (y ? WS_DP : a.xp) + col[u]) * 16;
    }
    const unsigned plane0 = 4u * (unsigned)(grad ? yplane : xplane), plane1 = 4u * (unsigned)xplane;

    // the cursor of the loads: the row its walk starts at, the walk, the step inside it, the addresses of that step's rows and this lane's
    // offsets in them.  What lies beyond the images or behind the last gradient row reads as zero
    int lrow = row_begin, is = 0;
    Walk lw = decode(lrow);
    const float *xrow, *yrow;
    unsigned at[2];
    auto start_walk = [&]() {
        const int gy = lw.py + lw.r0 * d;
        xrow = a.x + (long)lw.b * a.c_in * xplane + (long)gy * a.W;
        yrow = a.dy + (long)lw.b * a.c_out * yplane + (long)gy * a.Wo;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int gx = lw.x0 + col[u];
            at[u] = mine[u] && gx < (u == 0 && grad ? a.Wo : a.W) ? plane_off[u] + 4u * (unsigned)gx : WS_NOWHERE;
        }
        is = 0;
    };
    start_walk();
    // two sets of rows on their way, by the parity of the step they are for.  No branch around the loads: the compiler could not count them
    // and waited for all
    float xr[2][2][8];
    auto load = [&](auto set) {
        constexpr int S = decltype(set)::value;
        // (the compiler does not see that these are the same in every lane)
        const auto rsrc = [](const float *row, bool there) {
            const unsigned long at = (unsigned long)row;
            const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)at), hi = __builtin_amdgcn_readfirstlane((unsigned)(at >> 32));
            return __builtin_amdgcn_make_buffer_rsrc((void *)((unsigned long)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(there ? WS_NOWHERE : 0u), 0x00027000);
        };
        const auto xs = rsrc(xrow, lw.rows > 0), first = rsrc(grad ? yrow : xrow, lw.rows > 0 && (!grad || is < lw.rows));
#pragma unroll
        for (int e = 0; e < 8; ++e) xr[S][0][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(first, at[0], e * plane0, 0));
#pragma unroll
        for (int e = 0; e < 8; ++e) xr[S][1][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xs, at[1], e * plane1, 0));
        xrow += (long)d * a.W;
        yrow += (long)d * a.Wo;
        ++is;
        if (lw.rows > 0 && is == lw.rows + 3) {
            lrow += lw.rows;
            lw = decode(lrow);
            start_walk();
        }
    };
    auto measure = [&](int step, auto set) {                     // the range of this wave's rows
        constexpr int S = decltype(set)::value;
        SplitRange y = split_range(xr[S][0]), x = split_range(xr[S][1]);
        if (!grad) {                                             // uniform
            x = split_range(x, y);
            y = SplitRange{};
        } else y = split_wave_range(y);
        x = split_wave_range(x);
        if (lane == SPLIT_LAST_LANE) {
            unsigned *to = ranges + (step & 1) * 32 + wave;
            to[0] = x.most;
            to[8] = x.least;
            to[16] = y.most;
            to[24] = y.least;
        }
    };
    // powers of two, or SPLIT_WIDE: of the input row that is multiplied and of the gradient rows that it meets; of the rows that follow
    int sx = 0, sy[4] = {}, nx = 0, ny = 0;
    auto scales = [&](int step) {
        const uint4v *r4 = reinterpret_cast<const uint4v *>(ranges + (step & 1) * 32);
        const auto most8 = [&](int at) {
            const uint4v v = r4[at], w = r4[at + 1];
            return (unsigned)__builtin_amdgcn_readfirstlane((int)max(max(max(v[0], v[1]), max(v[2], v[3])), max(max(w[0], w[1]), max(w[2], w[3]))));
        };
        const auto scale = [](SplitRange r) {
            const int s = min(split_exponent(r.most, 14), WS_MOST);
            return s < -WS_MOST || split_wide(r, s) ? SPLIT_WIDE : s;
        };
        nx = scale({most8(0), most8(2)});
        ny = scale({most8(4), most8(6)});
    };
    float bsum[8] = {};
    auto commit = [&](int step, int slot, auto set) {
        constexpr int S = decltype(set)::value;
        char *xb = lds + (step & 1) * x_buf;
        uint4v p[2];
        const float scale_x = nx == SPLIT_WIDE ? 1.f : split_pow2(nx), scale_y = ny == SPLIT_WIDE ? 1.f : split_pow2(ny);      // (wide: nobody reads the pairs)
        split2(xr[S][0], grad ? scale_y : scale_x, p);
        if (mine[0]) {
            char *to = (grad ? lds + y_base + slot * y_slot : xb) + dst[0];
            *reinterpret_cast<uint4v *>(to) = p[0];
            *reinterpret_cast<uint4v *>(to + (grad ? y_part : x_part)) = p[1];
        }
        split2(xr[S][1], scale_x, p);
        if (mine[1]) {
            *reinterpret_cast<uint4v *>(xb + dst[1]) = p[0];
            *reinterpret_cast<uint4v *>(xb + dst[1] + x_part) = p[1];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) bsum[e] += xr[S][0][e];      // (of the input's: nobody reads them)
    };

    floatx4 acc[NCT][2][MT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[ct][i][m] = floatx4{0.f, 0.f, 0.f, 0.f};

    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    Walk cw = lw;                                                // the walk that is multiplied: the loads are three steps on, less than a walk
    load(Even{});
    load(Odd{});
    measure(0, Even{});
    wide_barrier();
    scales(0);
    commit(0, 0, Even{});
    sx = nx;
    sy[0] = ny;
    load(Even{});
    measure(1, Odd{});
    wide_barrier();
    int s = 0, slot = 0;
    // The input row of step s and the gradient row of step s - i on the fp32 matrix unit, from memory: lane (g, jl) loads pixels 4 g .. 4 g + 3 of map jl of
    // a tile, the operand of four K steps.  (Maps that do not exist read the last one: nobody reads their sums)
    auto multiply_f32 = [&](int ii, int i) {
        const float *xs = a.x + (long)cw.b * a.c_in * xplane + (long)(cw.py + (cw.r0 + s) * d) * a.W + cw.x0 + tapj * d;
        const float *ys = a.dy + (long)cw.b * a.c_out * yplane + (long)(cw.py + (cw.r0 + s - i) * d) * a.Wo + cw.x0;
        const int last = a.Wo - 4 - cw.x0;                       // (rows have four gradient pixels at least)
        // sixteen bytes from pixel px of the strip on, zeros behind the row's end: from where they end at it, moved down
        const auto load4 = [&](const float *row, int px) {
            const int at = min(px, last), down = px - at;
            floatx4 v = *reinterpret_cast<const float4u *>(row + at);
            if (down & 1) v = floatx4{v[1], v[2], v[3], 0.f};
            if (down & 2) v = floatx4{v[2], v[3], 0.f, 0.f};
            return down & ~3 ? floatx4{0.f, 0.f, 0.f, 0.f} : v;
        };
#pragma unroll 1
        for (int p0 = 0; p0 < WS_TX && cw.x0 + p0 < a.Wo; p0 += 16) {
            floatx4 A[MT], B[NCT];
#pragma unroll
            for (int m = 0; m < MT; ++m) A[m] = load4(ys + (long)min(16 * m + jl, a.c_out - 1) * yplane, p0 + 4 * g);
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) B[ct] = load4(xs + (long)min(16 * ct + jl, a.c_in - 1) * xplane, p0 + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
                    for (int m = 0; m < MT; ++m) acc[ct][ii][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[m][e], B[ct][e], acc[ct][ii][m], 0, 0, 0);
        }
    };
    // Step `step` multiplies its rows, which stand in LDS, writes those of the next (scaled by what everybody measured before the last barrier),
    // sets out for those three steps on and measures those of the step after the next, which have had two steps to arrive
    auto body = [&](int step, auto even, auto odd) {
        scales(step + 1);
        const char *xrow = lds + (step & 1) * x_buf;
        uint4v bf[2][NCT][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
                for (int p = 0; p < 2; ++p) bf[h][ct][p] = read_frag(xrow, p * x_part + b_off[ct] + h * 512);
        commit(step + 1, slot == WS_RING - 1 ? 0 : slot + 1, odd);
        load(odd);
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
            const int i = 2 * ip + ii;
            if (s < i || s - i >= cw.rows) continue;             // uniform
            const int syi = ip ? sy[2 + ii] : sy[ii];
            if (sx == SPLIT_WIDE || syi == SPLIT_WIDE) {
                multiply_f32(ii, i);
                continue;
            }
            int sl = slot - i;
            sl = sl < 0 ? sl + WS_RING : sl;
            const char *yrow = lds + y_base + sl * y_slot;
            const float scale = split_pow2(-(sx + syi));
            auto multiply = [&](auto halves) {                   // of the strip that hold gradient pixels
                constexpr int HALVES = decltype(halves)::value;
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    uint4v af[HALVES][2];
#pragma unroll
                    for (int h = 0; h < HALVES; ++h)
#pragma unroll
                        for (int p = 0; p < 2; ++p) af[h][p] = read_frag(yrow, p * y_part + a_off[m] + h * 512);
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {           // (a tile at a time: registers)
                        floatx4 hi = {0.f, 0.f, 0.f, 0.f}, lo = hi;
#pragma unroll
                        for (int h = 0; h < HALVES; ++h) {
                            lo = split_mfma(af[h][1], bf[h][ct][0], lo);
                            hi = split_mfma(af[h][0], bf[h][ct][0], hi);
                            lo = split_mfma(af[h][0], bf[h][ct][1], lo);
                        }
#pragma unroll
                        for (int r4 = 0; r4 < 4; ++r4) acc[ct][ii][m][r4] = __builtin_fmaf(split_sum(hi[r4], lo[r4]), scale, acc[ct][ii][m][r4]);
                    }
                }
            };
            if (cw.x0 + 32 < a.Wo) multiply(std::integral_constant<int, 2>{});
            else multiply(std::integral_constant<int, 1>{});
        }
        measure(step + 2, even);
        wide_barrier();
        sx = nx;
        sy[3] = sy[2];
        sy[2] = sy[1];
        sy[1] = sy[0];
        sy[0] = ny;
        slot = slot == WS_RING - 1 ? 0 : slot + 1;
        if (++s == cw.rows + 3) {
            cw = lw;
            s = 0;
        }
    };
    for (int step = 0; cw.rows > 0; step += 2) {
        body(step, Even{}, Odd{});
        if (cw.rows == 0) break;
        body(step + 1, Odd{}, Even{});
    }

    // the private copy, in accumulator order: [tap column][ct][tap row][map tile][lane][4]
    float *copy = a.scratch + (long)blockIdx.x * a.copy_floats;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int m = 0; m < MT; ++m) *reinterpret_cast<floatx4 *>(copy + ((((tapj * NCT + ct) * 4 + 2 * ip + i) * MT + m) * 64 + lane) * 4) = acc[ct][i][m];
    if (a.bias_part != nullptr && grad) {                     // uniform: wave o8 < c8o has the sums of octet o8
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = bsum[e];
#pragma unroll
            for (int sh = 32; sh > 0; sh >>= 1) v += __shfl_xor(v, sh, 64);
            if (lane == 0) a.bias_part[(long)blockIdx.x * (MT * 16) + wave * 8 + e] = v;
        }
    }
}

// octet o + 1 lands 16 or 48 banks further
int ws_xp(int d) { return (WS_TX + 3 * d + 3) / 8 * 8 + 4; }

size_t ws_smem(int c8i, int c8o, int d) { return ((size_t)4 * c8i * ws_xp(d) + (size_t)2 * WS_RING * c8o * WS_DP) * 16 + 256; }

template <int MT, int NCT> hipError_t launch_t(const Args &a, size_t smem, int blocks, hipStream_t stream)
{
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad_split_f32_kernel<MT, NCT>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((wgrad_split_f32_kernel<MT, NCT>), dim3(blocks), dim3(64 * WS_WAVES), smem, stream, a);
    return hipGetLastError();
}

}  // namespace

// From these rows of strips on it is no slower and at least as close to 64 bits: 96 gradients of 16 to 48 -> 16 to 48 maps, 200 x 220 to 2 x 500^2, d = 1 to 4:
// above the lines 0 to 260 us less of 50 to 460 a backward pass, errors 0.65 to 1.0 of the fp32 unit's; below (200 rows) 1.0 to 1.7 of the time.  16 -> 16
// maps, whose tiles are too few for a step, take 5 us more of 106 at 2 x 500^2.
bool wgrad_split_f32_supported(int c_in, int c_out, int k, int d, int n, int H, int W)
{
    if (k != 4 || d < 1 || (c_in == 16 && c_out == 16) || c_in < 16 || c_in > 48 || c_in % 8 != 0 || c_out < 16 || c_out > 48 || c_out % 8 != 0 || (long)H * W >= 1L << 24) return false;
    if (W - 3 * d < 4 || (long)n * ((W - 3 * d + WS_TX - 1) / WS_TX) * (H - 3 * d) < (c_in >= 32 ? 700 : 3000)) return false;
    const int c8i = (c_in + 7) / 8, c8o = (c_out + 7) / 8, groups = c8o + (c8i * (WS_TX + 3 * d) + 63) / 64;
    return groups <= 2 * WS_WAVES && ws_smem(c8i, c8o, d) <= 160 * 1024;
}

size_t wgrad_split_f32_copy_floats(int c_in, int c_out)
{
    const size_t MT = (c_out + 15) / 16, NCT = (c_in + 15) / 16;
    return 16 * NCT * MT * 256 + MT * 16;
}

hipError_t launch_wgrad_split_f32(const float *x, const float *dy, float *dw, float *db, float *scratch, size_t scratch_floats, int n, int c_in, int H,
                                  int W, int c_out, int d, hipStream_t stream)
{
    if (!wgrad_split_f32_supported(c_in, c_out, 4, d, n, H, W)) return hipErrorInvalidValue;
    Args a;
    a.x = x; a.dy = dy; a.scratch = scratch;
    a.n = n; a.c_in = c_in; a.c_out = c_out; a.c8i = (c_in + 7) / 8; a.c8o = (c_out + 7) / 8;
    a.H = H; a.W = W; a.Ho = H - 3 * d; a.Wo = W - 3 * d; a.d = d;
    if (a.Ho < 1 || a.Wo < 1 || n < 1) return hipErrorInvalidValue;
    a.pw = WS_TX + 3 * d;
    a.xp = ws_xp(d);
    a.xgroups = (a.c8i * a.pw + 63) / 64;
    const int MT = (c_out + 15) / 16, NCT = (c_in + 15) / 16;
    a.copy_floats = 16 * NCT * MT * 256;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    long blocks = std::min<long>(cus, (long)(scratch_floats / wgrad_split_f32_copy_floats(c_in, c_out)));
    if (blocks < 1) return hipErrorInvalidValue;
    a.xstrips = (a.Wo + WS_TX - 1) / WS_TX;
    const long total_rows = (long)n * a.xstrips * a.Ho;
    if (total_rows > 0x7fffffffL) return hipErrorInvalidValue;
    a.total_rows = (int)total_rows;
    blocks = std::min(blocks, total_rows);
    a.bias_part = db ? scratch + (size_t)blocks * a.copy_floats : nullptr;
    const size_t smem = ws_smem(a.c8i, a.c8o, d);
    hipError_t e = hipErrorInvalidValue;
#define SK_WS_CASE(mt, nct) if (MT == mt && NCT == nct) e = launch_t<mt, nct>(a, smem, (int)blocks, stream);
    SK_WS_CASE(2, 1) SK_WS_CASE(3, 1)
    SK_WS_CASE(1, 2) SK_WS_CASE(2, 2) SK_WS_CASE(3, 2)
    SK_WS_CASE(1, 3) SK_WS_CASE(2, 3) SK_WS_CASE(3, 3)
#undef SK_WS_CASE
    if (e != hipSuccess) return e;
    return launch_wgrad_rows_reduce(scratch, dw, (int)blocks, a.copy_floats, c_out, c_in, MT, NCT, a.bias_part, db, stream);
}

}  // namespace sk
