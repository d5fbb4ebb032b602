// 16-bit convolution with many output maps and a large kernel (5x5, 6x6, 8x8, 10x10; 64 maps and more, forward and data
// gradient): the scheme of kernels_conv_wide_h.hip with the four lane groups of the MFMA on four kernel columns of one input octet.
//
// A chunk is one input octet; its kernel is walked in steps of four columns x KR rows (KR = 4 or 5; 3 for 6x6), and the one or two
// columns left behind the last four in one step more, whose fragments hold four or two kernel rows of them (as a column step of
// their own, padded with zero weights, they were a sixth of the MFMAs at 10x10, a quarter at 6x6 and three tenths at 5x5).  A step's
// weights (64 maps: 4 KR fragments of 1 KB) lie in a ring of three slots, two steps ahead; the input tile of the next octet loads meanwhile.
// What bounded conv_h_kernel here is LDS: 16 maps x 64 pixels a wave at 10x10 are 23 fragments read per 40 MFMAs, more than the
// 128 bytes a CU moves per cycle while the matrix unit keeps up.  A wave of this kernel multiplies 32 maps x 128 pixels: 22
// fragments per 80 MFMAs.
//
// The lane groups take the columns in the order 0, 2, 1, 3 (the packing does the same): ds_read_b128 serves lanes of groups 0
// and 1 (2 and 3) together, and columns two kernel strides apart fall on different banks at stride 8, one apart on the same.
//
// Measured (bf16, us, conv_h_kernel -> here with the columns left padded to four -> here): 10x10 d = 8 192 -> 1024 at 200^2 756 -> 457 -> 411
// (1.57 PFLOP/s, where the clock falls with the power), 64 -> 256 at 322^2 - -> 173 -> 151; 8x8 d = 8 128 -> 512 at 314^2 640 -> 490 (1.14:
// 1296 tiles are 5.06 rounds of 256); 6x6 64 -> 128 at 344^2 107 -> 81 -> 64, d = 8 128 -> 128 at 300^2 - -> 137 -> 105; 5x5 64 -> 128 at
// 2 x 300^2 - -> 95 -> 79.  4x4 layers stay on the ring kernel: a step would be 32 MFMAs a wave.
#include "conv_wide.h"

namespace sk {

namespace {

// rows of a step
template <int KS> constexpr int big_rows() { return KS == 10 ? 5 : KS == 8 ? 4 : KS == 6 ? 3 : KS; }

template <int DT, int KS, int XW, int NX, bool PAD, int OUT>
__global__ __launch_bounds__(512, 2) void conv_wide_big_h_kernel(WideArgs k)
{
    constexpr int R = 8, MG = 2, WM = 2;                       // a wave: two map tiles x 8 rows; two waves share a packed group
    using T = WideTile<8, KS, MG, R, XW>;
    extern __shared__ uint4v lds[];
    constexpr int RR = T::RT + KS - 1;
    constexpr int KR = big_rows<KS>(), RP = KS / KR, CF = KS / 4;             // rows of a step, steps of four columns: of one column step, all
    constexpr int TC = KS % 4, TR = TC ? 4 / TC : 1, TF = TC ? (KS + TR - 1) / TR : 0;   // columns left; kernel rows of their fragments, fragments
    constexpr int NS = CF * RP + (TC ? 1 : 0), CHUNK_BYTES = (CF * KS + TF) * 4096;
    static_assert(TC != 3 && TF <= KR, "the columns left are one step");
    constexpr int SLAB = KR * 4;                               // 1 KB weight fragments of a step
    constexpr int NW = (SLAB + 7) / 8;                         // weight loads of a wave per step

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4;
    const int wm = wave / T::PWV, pwv = wave % T::PWV;
    const int nslots = gridDim.x >> 3;
    const int t_end = (int)((long)k.w.total * ((blockIdx.x & 7) + 1) / 8);      // an XCD takes a contiguous eighth of the tiles
    const int t_first = (int)((long)k.w.total * (blockIdx.x & 7) / 8) + (int)(blockIdx.x >> 3);
    if (t_first >= t_end) return;

    const int pw = k.w.pw, oct_units = k.w.oct_units, last_blk = oct_units / 64 - 1;
    uint4v *const xbuf = lds, *const wbuf = lds + 2 * oct_units;
    float *const bias_lds = reinterpret_cast<float *>(wbuf + 3 * SLAB * 64);
    for (int q = tid; q < k.w.pgroups * 64; q += 512) bias_lds[q] = (k.a.bias && q < (k.a.c_out + 15) / 16 * 16) ? k.a.bias[q] : 0.f;

    const unsigned lane16 = lane * 16;
    const char *const zeros = reinterpret_cast<const char *>(k.a.zeros);
    struct Cursor {
        int t, ch;
        WidePos p;
        const char *x, *w;      // octet plane and weights of the chunk
        int o_in;               // the octet inside its group of octets
    };
    const int nchunks = k.w.nchunks, grp8 = k.a.grp8;
    const long plane = (long)k.a.H * k.a.W * 16, skip_bytes = (long)k.a.skip8 * plane;
    auto open_tile = [&](Cursor &c) {
        const WideArgs &q = *wide_args();
        c.p = wide_decode<KS, T>(q.w, q.a.n, c.t);
        c.ch = 0;
        c.o_in = 0;
        c.x = reinterpret_cast<const char *>(q.a.x) + (long)c.p.b * (q.a.xb8 > 0 ? q.a.xb8 : q.a.c8_in) * plane;
        c.w = reinterpret_cast<const char *>(q.a.wp) + (long)c.p.mg * q.w.nchunks * CHUNK_BYTES;
    };
    // the chunk after c; false at the end of this workgroup's list
    auto step_chunk = [&](Cursor &c) {
        if (++c.ch < nchunks) {
            c.x += plane;
            c.w += CHUNK_BYTES;
            if (grp8 > 0 && ++c.o_in == grp8) {
                c.o_in = 0;
                c.x += skip_bytes;
            }
            return true;
        }
        c.t += nslots;
        if (c.t >= t_end) return false;
        open_tile(c);
        return true;
    };

    // byte offsets inside an octet plane of the units this lane loads: outside the image the nearest sample, which no stored
    // output reads, or (PAD) ~0: zero
    unsigned xoff[NX];
    auto set_offsets = [&](const WidePos &p) {
        const WideArgs &q = *wide_args();
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const int unit = (wave + 8 * u < last_blk ? wave + 8 * u : last_blk) * 64 + lane;
            const int r = unit / pw, x = unit - r * pw;
            int gy = p.py + q.a.d * (p.ty * T::RT + r) - q.a.in_off, gx = p.x0 + x - q.a.in_off;
            const bool inside = r < RR && gy >= 0 && gy < q.a.H && gx >= 0 && gx < q.a.W;
            gy = gy < 0 ? 0 : (gy >= q.a.H ? q.a.H - 1 : gy);
            gx = gx < 0 ? 0 : (gx >= q.a.W ? q.a.W - 1 : gx);
            xoff[u] = PAD && !inside ? ~0u : (unsigned)(gy * q.a.W + gx) * 16u;
        }
    };
    int wblk[NW];
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        const int blk = wave + 8 * u;                          // (where eight waves do not divide the slab some load a fragment twice)
        wblk[u] = blk < SLAB ? blk : blk - (NW * 8 - SLAB);
    }
    auto load_x = [&](const Cursor &c, int buf, int u) {
        const int blk = wave + 8 * u < last_blk ? wave + 8 * u : last_blk;              // (spare loads repeat the last block)
        uint4v *dst = xbuf + buf * oct_units + blk * 64;
        if constexpr (PAD) wide_load_lds(xoff[u] != ~0u ? c.x + xoff[u] : zeros + lane16, dst);
        else wide_load_lds(c.x + xoff[u], dst);
    };
    // step s of a chunk: column step s / RP, kernel rows from (s % RP) * KR on; the last one: the columns left
    auto load_w = [&](const Cursor &c, int s, int sl, int u) {
        const int blk = TF < KR && TC && s == NS - 1 ? min(wblk[u], TF * 4 - 1) : wblk[u];
        wide_load_lds(c.w + s * (KR * 4096) + blk * 1024 + lane16, wbuf + (sl * SLAB + blk) * 64);
    };

    floatx4 acc[R][WM];
#pragma unroll
    for (int y = 0; y < R; ++y)
#pragma unroll
        for (int mt = 0; mt < WM; ++mt) acc[y][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int dil = k.a.d, col = (g >> 1) | ((g & 1) << 1);    // this lane group's kernel column within a column step
    const int pixel = (pwv / XW) * R * pw + (pwv % XW) * 16 + l16;
    const uint4v *const xfrag = xbuf + pixel + col * dil;
    // its tap of a fragment of the columns left: two columns of two rows, or four rows of one (where the last fragment of 5x5 has one row)
    const uint4v *const xtail = xbuf + pixel + (4 * CF + (TC == 2 ? g >> 1 : 0)) * dil + (TC == 2 ? g & 1 : g) * pw;
    const uint4v *const xend = xbuf + pixel + 4 * CF * dil + (KS - 1) * pw;
    const uint4v *const wfrag = wbuf + wm * WM * 64 + lane;
    // One step; its N loads for later steps go between the MFMAs.
    auto step = [&](bool act, int buf, auto si, int sl, auto loads, auto &&load) {
        constexpr int s = decltype(si)::value, N = decltype(loads)::value;
        constexpr bool TAIL = TC && s == NS - 1;
        // fragments of weights; input rows that a fragment reads and the one before it does not
        constexpr int FR = TAIL ? TF : KR, PR = TAIL ? (TC == 1 ? R : TR) : 1, GROUPS = FR * R, SPREAD = N > 0 ? GROUPS / std::max(N, 1) : 1;
        static_assert(N <= GROUPS, "one load per group of MFMAs at most");
        if (!act) {
#pragma unroll
            for (int q = 0; q < N; ++q) load(q);
            return;
        }
        const uint4v *wl = wfrag + sl * SLAB * 64;
        const uint4v *xl = (TAIL ? xtail : xfrag + (s / RP) * 4 * dil + (s % RP) * KR * pw) + buf * oct_units, *xe = xend + buf * oct_units;
        constexpr int NB = R + (FR - 1) * PR, NREAD = FR * WM + NB, HEAD = WM + 3;
        uint4v af[FR][WM], bf[NB];
        // fragments in the order of their use: the first's maps and input rows, then maps and the input rows that come on
        auto row = [&](int q) { bf[q] = TAIL && TC == 1 && q >= R ? xe[(q - R) * pw] : xl[q * pw]; };
        auto read = [&](int q) {
            if (q < WM) af[0][q] = wl[q * 64];
            else if (q < WM + R) row(q - WM);
            else {
                const int i = 1 + (q - WM - R) / (WM + PR), m = (q - WM - R) % (WM + PR);
                if (m < WM) af[i][m] = wl[(i * 4 + m) * 64];
                else row(R + (i - 1) * PR + m - WM);
            }
        };
#pragma unroll
        for (int q = 0; q < HEAD; ++q) read(q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
            const int i = q / R, y = q % R;
            if (HEAD + q < NREAD) read(HEAD + q);
#pragma unroll
            for (int mt = 0; mt < WM; ++mt) acc[y][mt] = wide_mfma<DT>(af[i][mt], bf[y + PR * i], acc[y][mt]);
            if (q % SPREAD == SPREAD - 1 && q / SPREAD < N) load(q / SPREAD);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    auto epilogue = [&](const Cursor &c) {
        const WideArgs &q = *wide_args();
        const int mt0 = c.p.mg * 4 + wm * WM;
        float bia[WM][4];
#pragma unroll
        for (int mt = 0; mt < WM; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) bia[mt][r] = bias_lds[(mt0 + mt) * 16 + 4 * g + r];
#pragma unroll
        for (int y = 0; y < R; y += 2) {
            const WideDst<OUT> dst = wide_dst<OUT, KS, R, XW, T>(q.a, c.p, pwv, y, l16, g, mt0);
#pragma unroll
            for (int mt = 0; mt < WM; ++mt) {
                wide_store<DT, OUT>(q.a, acc[y][mt], acc[y + 1][mt], bia[mt], dst, mt0, mt, g, uint4v{0u, 0u, 0u, 0u});
                acc[y][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
                acc[y + 1][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
    };

    const int Ho = k.a.Ho, Wo = k.a.Wo;
    auto wave_active = [&](const WidePos &p) { return p.x0 + (pwv % XW) * 16 < Wo && p.py + dil * (p.ty * T::RT + (pwv / XW) * R) < Ho; };

    Cursor cur;
    cur.t = t_first;
    open_tile(cur);
    set_offsets(cur.p);
    bool act = wave_active(cur.p);
#pragma unroll
    for (int u = 0; u < NX; ++u) load_x(cur, 0, u);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int u = 0; u < NW; ++u) load_w(cur, s, s, u);
    int buf = 0, sl = 0;                                       // sl: slot of the step's weights, the ring runs on over chunks
    wide_wait<NW>();
    Cursor nxt = cur;
    bool more = step_chunk(nxt);
    if (more && nxt.t != cur.t) set_offsets(nxt.p);
    while (more) {
        Cursor after = nxt;
        auto move = [&]() {
            more = step_chunk(after);
            if (more && after.t != nxt.t) set_offsets(after.p);
        };
        wide_for<NS>([&](auto si) {
            constexpr int s = decltype(si)::value;
            // input loads u = s, s + NS - 1, ... of the steps before the last
            constexpr int XN = s < NS - 1 ? (NX - s + NS - 2) / (NS - 1) : 0, XP = s >= 1 ? (NX - (s - 1) + NS - 2) / (NS - 1) : 0;
            const int ahead = sl == 0 ? 2 : sl - 1;            // slot of the step two on
            wide_barrier();
            // the cursor moves on while the other wave of the SIMD multiplies (its input loads are all under way)
            if (s == NS - 1 && wave < 4) move();
            step(act, buf, si, sl, std::integral_constant<int, NW + XN>{}, [&](int q) {
                if (q < NW) {
                    if (s + 2 < NS) load_w(cur, s + 2, ahead, q);
                    else load_w(nxt, s + 2 - NS, ahead, q);
                } else {
                    load_x(nxt, buf ^ 1, s + (q - NW) * (NS - 1));
                }
            });
            if (s == NS - 1 && wave >= 4) move();
            // the next step's weights (and, for a new chunk, its input) have landed; younger: what this step loaded and the
            // input loads of the one before
            if (s == NS - 1) wide_wait<NW>();
            else wide_wait<XP + NW + XN>();
            sl = sl == 2 ? 0 : sl + 1;
        });
        if (nxt.t != cur.t) {
            if (act) epilogue(cur);
            act = wave_active(nxt.p);
        }
        cur = nxt;
        nxt = after;
        buf ^= 1;
    }
    wide_for<NS>([&](auto si) {
        constexpr int s = decltype(si)::value, N = s + 2 < NS ? NW : 0;
        const int ahead = sl == 0 ? 2 : sl - 1;
        wide_barrier();
        step(act, buf, si, sl, std::integral_constant<int, N>{}, [&](int q) { load_w(cur, s + 2, ahead, q); });
        wide_wait<N>();
        sl = sl == 2 ? 0 : sl + 1;
    });
    if (act) epilogue(cur);
}

int tile_units(int pw, int rows) { return (rows * pw + 63) / 64 * 64; }

template <int KS>
size_t big_smem(const WideGeom &w)
{
    return (size_t)2 * w.oct_units * 16 + (size_t)3 * big_rows<KS>() * 4096 + (size_t)w.pgroups * 64 * sizeof(float);
}

// (the biases of all maps share the LDS with the tile: see conv_h_wide)
template <int KS>
bool big_fits(const WideGeom &w)
{
    return w.oct_units / 64 <= 48 && big_smem<KS>(w) <= 160 * 1024;
}

// input loads of a wave per chunk
int big_loads(int units) { return units / 64 <= 16 ? 2 : units / 64 <= 32 ? 4 : 6; }

template <int KS, int XW>
WideGeom big_geom(const ConvHArgs &a)
{
    using T = WideTile<8, KS, 2, 8, XW>;
    WideGeom w{};
    w.pgroups = w.mgroups = ((a.c_out + 15) / 16 + 3) / 4;
    w.nchunks = a.c8_in;
    w.split = 1;
    w.xtiles = (a.Wo + T::TX - 1) / T::TX;
    const int q = a.Ho / a.d;
    w.rem = a.Ho % a.d;
    w.tiles_hi = (q + 1 + T::RT - 1) / T::RT;
    w.tiles_lo = (q + T::RT - 1) / T::RT;
    w.ytiles = w.rem * w.tiles_hi + (a.d - w.rem) * w.tiles_lo;
    if (w.tiles_lo < 1) w.tiles_lo = 1;
    // Which tiles are taken stays with rows of whole column steps, for which it was measured (`fits`).  The two columns left of 6x6 and 10x10
    // need fewer, and neighbouring lane groups read them from neighbouring rows, which fall on different banks 16 units apart modulo 16
    // (see above)
    w.pw = T::TX + (4 * ((KS + 3) / 4) - 1) * a.d;
    w.oct_units = tile_units(w.pw, T::RT + KS - 1);
    const bool fits = big_fits<KS>(w);
    const int even = (T::TX + (KS - 1) * a.d + 15) / 16 * 16;
    if (KS % 4 == 2 && even <= w.pw) {
        w.pw = even;
        w.oct_units = tile_units(w.pw, T::RT + KS - 1);
    }
    const long tiles = (long)w.xtiles * w.ytiles * w.mgroups * a.n;
    w.tiles = w.total = !fits || tiles > 0x3fffffffL ? 0 : (int)tiles;
    return w;
}

template <int DT, int KS, int XW, int NX, bool PAD, int OUT>
hipError_t launch_big_n(const WideArgs &k, size_t smem, hipStream_t stream)
{
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_wide_big_h_kernel<DT, KS, XW, NX, PAD, OUT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int blocks = wide_cus() / 8 * 8;
    if (k.w.total < blocks) blocks = (k.w.total + 7) / 8 * 8;
    hipLaunchKernelGGL((conv_wide_big_h_kernel<DT, KS, XW, NX, PAD, OUT>), dim3(blocks), dim3(512), smem, stream, k);
    return hipGetLastError();
}

template <int DT, int KS, int XW, bool PAD, int OUT>
hipError_t launch_big_x(const ConvHArgs &a, hipStream_t stream)
{
    WideArgs k;
    k.a = a;
    k.w = big_geom<KS, XW>(a);
    const size_t smem = big_smem<KS>(k.w);
    if (k.w.tiles < 1 || !a.zeros) return hipErrorInvalidValue;
    if ((long)a.H * a.W * 16 >= 0xffffffffL || (long)(a.out_f32 ? a.c_out * 4L : a.c8_out_total * 16L) * a.OH * a.OW >= 0x7fffffffL) return hipErrorInvalidValue;
    switch (big_loads(k.w.oct_units)) {
    case 2: return launch_big_n<DT, KS, XW, 2, PAD, OUT>(k, smem, stream);
    case 4: return launch_big_n<DT, KS, XW, 4, PAD, OUT>(k, smem, stream);
    default: return launch_big_n<DT, KS, XW, 6, PAD, OUT>(k, smem, stream);
    }
}

// 16-column groups across a tile: 2 (32 x 16 output pixels) or 4 (64 x 8, which fits every kernel stride), the shape with fewer
// rounds of one tile per CU
template <int KS>
int big_columns(const ConvHArgs &a)
{
    if (a.out_f32) return 4;
    const WideGeom sq = big_geom<KS, 2>(a), flat = big_geom<KS, 4>(a);
    const int cus = wide_cus();
    return sq.tiles >= 1 && (sq.tiles + cus - 1) / cus <= (flat.tiles + cus - 1) / cus ? 2 : 4;
}

template <int DT, int KS>
hipError_t launch_big_k(const ConvHArgs &a, hipStream_t stream)
{
    if (a.out_f32) return a.in_off ? hipErrorInvalidValue : launch_big_x<DT, KS, 4, false, WV_F32>(a, stream);
    if (big_columns<KS>(a) == 2)
        return a.in_off ? launch_big_x<DT, KS, 2, true, WV_OCT>(a, stream) : launch_big_x<DT, KS, 2, false, WV_OCT>(a, stream);
    return a.in_off ? launch_big_x<DT, KS, 4, true, WV_OCT>(a, stream) : launch_big_x<DT, KS, 4, false, WV_OCT>(a, stream);
}

template <int KS>
ConvHPath big_path(const ConvHArgs &a)
{
    const int columns = big_columns<KS>(a);
    const WideGeom w = columns == 2 ? big_geom<KS, 2>(a) : big_geom<KS, 4>(a);
    return {w.tiles >= 1 ? 2 : -1, columns, 1, big_loads(w.oct_units)};
}

template <int DT>
hipError_t launch_big_dt(const ConvHArgs &a, hipStream_t stream)
{
    switch (a.k) {
    case 5: return launch_big_k<DT, 5>(a, stream);
    case 6: return launch_big_k<DT, 6>(a, stream);
    case 8: return launch_big_k<DT, 8>(a, stream);
    case 10: return launch_big_k<DT, 10>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

ConvHPath conv_wide_big_path(const ConvHArgs &a)
{
    switch (a.k) {
    case 5: return big_path<5>(a);
    case 6: return big_path<6>(a);
    case 8: return big_path<8>(a);
    default: return big_path<10>(a);
    }
}

hipError_t launch_conv_wide_big_h(const ConvHArgs &a, hipStream_t stream)
{
    if (a.mask || a.tap_maps) return hipErrorInvalidValue;
    if (a.dtype == 1) return launch_big_dt<1>(a, stream);
    if (a.dtype == 2) return launch_big_dt<2>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace sk
