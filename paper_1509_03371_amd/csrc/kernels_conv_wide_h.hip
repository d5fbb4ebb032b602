// 16-bit convolution with many output maps (1x1 and 3x3, 64 maps and more): MFMA 16x16x32 with wide register tiles.
//
// (3x3: 17 to 32 maps too.)  What bounds conv_h_kernel on these layers is LDS and the instructions around the MFMAs: its waves multiply 48 maps x 64 pixels,
// 45 fragments (1 KB each) read per 108 MFMAs of a 3x3 chunk -- with the staging writes about 126 of the 128 bytes a CU's LDS
// moves per cycle -- and every input sample passes through a register on its way to LDS.  Here a wave multiplies 64 maps x 32 to
// 128 pixels, 20 fragments per 72 MFMAs of a kernel column in the largest shape, and input and weights go from global memory
// straight into LDS (global_load_lds, 1 KB an instruction) with addresses that cost one or two instructions a load.
//
//   3x3: a step is one kernel column of one chunk of 32 input maps.  The weights of a step lie in a ring of three slots
//        (two steps ahead), the input tile of a chunk in one of two buffers (one chunk ahead).
//   1x1: a step is a chunk; pixels are taken linearly over the plane, so a tile has no ragged columns; input and weights
//        share a ring of S stages.
// One barrier per step; a wave waits for its own loads only (vmcnt with the exact number of younger ones) before it.
// A workgroup is 8 waves (1x1 also 4, two workgroups on a CU): MG map groups of 64 maps x pixel waves of 16 x R pixels (3x3: XW
// across, the rest down).
//
// Maps too small to give every CU a tile split the input maps over several workgroups (w.split): each writes its fp32
// sums in accumulator order, conv_wide_reduce_h_kernel adds them in a fixed order and does what the epilogue does.
//
// Measured (bf16, us, conv_h_kernel -> here; the reduction of a split included): 3x3 64 -> 64 at 570^2 46.5 -> 37.5 (0.63 PFLOP/s;
// 82 MB read and written, 16 us at the rate of a copy), 128 -> 128 at 282^2 46.8 -> 30 (0.77), 256 -> 256 at 138^2 64 -> 34,
// 1024 -> 1024 at 30^2 77 -> 35 (input maps split in four), 192 -> 128 at 516^2 186 -> 127 (0.91), 96 -> 128 at stride 4 on 64 slices
// of 136^2 325 -> 232 (1.0); 1x1 1024 -> 512 at 128^2 58 -> 37, 512 -> 256 at 202^2 103 -> 45, 1024 -> 2048 up-convolution at 28^2
// 52 -> 24.
// A step costs 0.52 / 0.93 / 1.20 us (tiles of 256 / 512 / 768 pixels x 64 maps) where its MFMAs are 0.32 / 0.64 / 0.96 at 2.4 GHz.
// A wave of the smallest tile multiplies 32 maps x 64 pixels, half of a packed group of map tiles: 12 fragments read for 24 MFMAs, 16 at
// 64 maps x 32 pixels (the U-Net's launches of it 28.5 -> 27.7 us, the 572^2 forward pass 668 -> 659).
// 17 to 32 output maps (conv_wide32): 32 maps x 64 x 12 pixels a tile, 14 fragments read for 36 MFMAs of a wave; weights packed as for
// conv_h_kernel.  128 -> 32 maps data gradient at stride 4 on 72 slices of 136^2 (295 GFLOP): 610 -> 384 us, 16 -> 32 at stride 2 on 74
// slices of 138^2 120 -> 94; the 3-D training step 3.03 -> 2.77 ms.
// Tried and dropped: 128 maps x 512 pixels a workgroup (1.63 us of 1.28; half as many tiles, and spills with masks), four waves
// and two workgroups a CU for 3x3 (within 5 % either way), the loads of a step issued together behind its barrier (5 to 10 %).
#include "conv_wide.h"

namespace sk {

namespace {

// NX: input loads of a wave per chunk; PAD: the launch reads zeros around the image (data gradient of a 3x3 layer)
template <int DT, int NWV, int KS, int MG, int R, int XW, int NX, bool PAD, int OUT, int S, int MT, int GT>
__global__ __launch_bounds__(64 * NWV, 2) void conv_wide_h_kernel(WideArgs k)
{
    using T = WideTile<NWV, KS, MG, R, XW, MT, GT>;
    extern __shared__ uint4v lds[];
    constexpr int RR = T::RT + KS - 1;
    constexpr int SLAB = KS * GT * MG;                         // 1 KB weight fragments of a step
    constexpr int NW = (SLAB + NWV - 1) / NWV;       // weight loads of a wave per step
    constexpr int NXB = KS == 3 ? 2 : S, NWB = KS == 3 ? 3 : S;   // input buffers, weight slots

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4;
    const int wm = wave / T::PWV, pwv = wave % T::PWV;         // map group and pixel wave
    const int nslots = gridDim.x >> 3;
    // workgroup ids go round-robin over the 8 XCDs: XCD x takes the x-th contiguous eighth of the items, so that neighbours
    // share input halo and weights in that XCD's L2
    const int t_end = (int)((long)k.w.total * ((blockIdx.x & 7) + 1) / 8);
    const int t_first = (int)((long)k.w.total * (blockIdx.x & 7) / 8) + (int)(blockIdx.x >> 3);
    if (t_first >= t_end) return;

    const int pw = k.w.pw, oct_units = k.w.oct_units;
    uint4v *const xbuf = lds, *const wbuf = lds + NXB * 4 * oct_units;
    float *const bias_lds = reinterpret_cast<float *>(wbuf + NWB * SLAB * 64);
    for (int q = tid; q < (k.w.split > 1 ? 0 : k.w.pgroups * GT * 16); q += 64 * NWV) bias_lds[q] = (k.a.bias && q < (k.a.c_out + 15) / 16 * 16) ? k.a.bias[q] : 0.f;

    // this wave loads one octet of a chunk, every LPO-th 64 units of it
    constexpr int LPO = NWV / 4;
    const int oct = wave / LPO, part = wave % LPO, units = KS == 1 ? T::TX : RR * pw, last_blk = (units - 1) / 64;
    const unsigned lane16 = lane * 16;
    const char *const zeros = reinterpret_cast<const char *>(k.a.zeros);

    // cursor over (item, chunk): an item is a tile and a range of its chunks
    struct Cursor {
        int t, ch, end;
        WidePos p;
        const char *x, *w;      // this wave's octet plane of the chunk, the chunk's weights
        int o_in;               // its octet inside the group of octets (WideArgs a.grp8)
        bool have;              // the octet exists (else zeros are read)
        long woff[NW];          // this wave's weight loads: bytes behind w
    };
    int wblk[NW];
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        const int blk = wave + NWV * u;                        // (where the waves do not divide the slab some load a fragment twice)
        wblk[u] = blk < SLAB ? blk : blk - (NW * NWV - SLAB);
    }
    auto open_item = [&](Cursor &c) {
        const WideArgs &q = *wide_args();
        const int sp = c.t / q.w.tiles;
        c.p = wide_decode<KS, T>(q.w, q.a.n, c.t - sp * q.w.tiles);
        c.ch = (int)((long)q.w.nchunks * sp / q.w.split);
        c.end = (int)((long)q.w.nchunks * (sp + 1) / q.w.split);
        const int o = c.ch * 4 + oct;
        const long plane = (long)q.a.H * q.a.W * 16;
        const int skips = q.a.grp8 > 0 ? o / q.a.grp8 : 0;
        c.o_in = o - skips * q.a.grp8;
        c.have = o < q.a.c8_in;
        c.x = reinterpret_cast<const char *>(q.a.x) + ((long)c.p.b * (q.a.xb8 > 0 ? q.a.xb8 : q.a.c8_in) + o + (long)skips * q.a.skip8) * plane;
        c.w = reinterpret_cast<const char *>(q.a.wp) + ((long)c.p.mg * MG * q.w.nchunks + c.ch) * (KS * KS * GT) * 1024;
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            const int h = wblk[u] / (KS * GT);
            // (beyond the last packed group: any weights that exist, nothing reads them)
            c.woff[u] = (wblk[u] - h * (KS * GT)) * 1024 + (c.p.mg * MG + h < q.w.pgroups ? h : 0) * ((long)q.w.nchunks * (KS * KS * GT) * 1024);
        }
    };
    const long plane4 = (long)k.a.H * k.a.W * 64;              // four octet planes
    const int c8_in = k.a.c8_in, grp8 = k.a.grp8;
    const long skip_bytes = (long)k.a.skip8 * k.a.H * k.a.W * 16;
    // the chunk after c; false at the end of this workgroup's list
    auto step_chunk = [&](Cursor &c) {
        if (++c.ch < c.end) {
            c.x += plane4;
            c.w += KS * KS * GT * 1024;
            c.have = c.ch * 4 + oct < c8_in;
            if (grp8 > 0) {
                c.o_in += 4;
                while (c.o_in >= grp8) {
                    c.o_in -= grp8;
                    c.x += skip_bytes;
                }
            }
            return true;
        }
        c.t += nslots;
        if (c.t >= t_end) return false;
        open_item(c);
        return true;
    };

    // byte offsets inside an octet plane of the units this lane loads for the tile at p.  Outside the image: the nearest
    // sample, which no stored output reads, or (PAD) ~0: zero
    unsigned xoff[NX];
    auto set_offsets = [&](const WidePos &p) {
        const WideArgs &q = *wide_args();
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const int unit = (part + LPO * u < last_blk ? part + LPO * u : last_blk) * 64 + lane;
            if (KS == 1) {
                const int i = p.x0 + unit, last = q.a.H * q.a.W - 1;
                xoff[u] = (unsigned)(i < last ? i : last) * 16u;
            } else {
                const int r = unit / pw, x = unit - r * pw;
                int gy = p.py + q.a.d * (p.ty * T::RT + r) - q.a.in_off, gx = p.x0 + x - q.a.in_off;
                const bool inside = r < RR && gy >= 0 && gy < q.a.H && gx >= 0 && gx < q.a.W;
                gy = gy < 0 ? 0 : (gy >= q.a.H ? q.a.H - 1 : gy);
                gx = gx < 0 ? 0 : (gx >= q.a.W ? q.a.W - 1 : gx);
                xoff[u] = PAD && !inside ? ~0u : (unsigned)(gy * q.a.W + gx) * 16u;
            }
        }
    };
    // load u of this wave's share of an input chunk / of the weights of kernel column cs (1 KB each)
    auto load_x = [&](const Cursor &c, int buf, int u) {
        const int blk = part + LPO * u < last_blk ? part + LPO * u : last_blk;      // (spare loads repeat the last block)
        uint4v *dst = xbuf + (buf * 4 + oct) * oct_units + blk * 64;
        if constexpr (PAD) {
            const char *src = c.have && xoff[u] != ~0u ? c.x + xoff[u] : zeros + lane16;
            wide_load_lds(src, dst);
        } else {
            wide_load_lds((c.have ? c.x : zeros) + (c.have ? xoff[u] : lane16), dst);
        }
    };
    auto load_w = [&](const Cursor &c, int cs, int sl, int u) {
        wide_load_lds(c.w + c.woff[u] + cs * (KS * GT * 1024) + lane16, wbuf + (sl * SLAB + wblk[u]) * 64);
    };

    floatx4 acc[R][MT];
#pragma unroll
    for (int y = 0; y < R; ++y)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[y][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    // One step: kernel column cs of the chunk in input buffer `buf` against the weights in slot sl.  load(q, n): the q-th of
    // the n loads the step issues for later ones; they go between the MFMAs, because eight waves that issue theirs together
    // behind the barrier stand in the memory pipeline's queue (16 cycles an instruction and more) while the matrix unit idles.
    const int xrow = KS == 1 ? pwv * 16 * R : (pwv / XW) * R * pw + (pwv % XW) * 16;
    const uint4v *const xfrag = xbuf + g * oct_units + l16 + xrow, *const wfrag = wbuf + (wm * MT / GT * KS * GT + wm * MT % GT) * 64 + lane;
    const int pitch = KS == 1 ? 16 : pw, dil = KS == 1 ? 0 : k.a.d, buf_units = 4 * oct_units;
    auto step = [&](bool act, int buf, int cs, int sl, auto loads, auto &&load) {
        constexpr int N = decltype(loads)::value, GROUPS = KS * R, SPREAD = N > 0 && GROUPS > N ? GROUPS / std::max(N, 1) : 1;
        if (!act) {                                            // a wave without pixels or maps in the tile only loads
#pragma unroll
            for (int q = 0; q < N; ++q) load(q);
            return;
        }
        const uint4v *wl = wfrag + sl * SLAB * 64;
        const uint4v *xl = xfrag + buf * buf_units + cs * dil;
        // fragments in the order the multiplication needs them: the map tiles of kernel row 0 and the input rows, then
        // the map tiles and one more input row per further kernel row
        constexpr int NB = R + KS - 1, NREAD = KS * MT + NB, HEAD = MT + (R < 3 ? R : 3), PER = R == 2 ? 3 : 2;
        uint4v af[KS][MT], bf[NB];
        auto read = [&](int q) {
            if (q < MT) af[0][q] = wl[q * 64];
            else if (q < MT + R) bf[q - MT] = xl[(q - MT) * pitch];
            else {
                const int i = 1 + (q - MT - R) / (MT + 1), m = (q - MT - R) % (MT + 1);
                if (m < MT) af[i][m] = wl[(i * GT + m) * 64];
                else bf[R + i - 1] = xl[(R + i - 1) * pitch];
            }
        };
#pragma unroll
        for (int q = 0; q < HEAD; ++q) read(q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
            const int i = q / R, y = q % R;
#pragma unroll
            for (int r = 0; r < PER; ++r)
                if (HEAD + q * PER + r < NREAD) read(HEAD + q * PER + r);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[y][mt] = wide_mfma<DT>(af[i][mt], bf[y + i], acc[y][mt]);
            if (q % SPREAD == SPREAD - 1 && q / SPREAD < N) load(q / SPREAD);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = GROUPS / SPREAD; q < N; ++q) load(q);
    };

    auto epilogue = [&](const Cursor &c) {
        const WideArgs &q = *wide_args();
        const int mt0 = c.p.mg * (MG * GT) + wm * MT;
        if (q.w.split > 1) {
            floatx4 *dst = reinterpret_cast<floatx4 *>(q.w.ws + (long)c.t * T::FLOATS) + (long)wave * R * MT * 64 + lane;
#pragma unroll
            for (int y = 0; y < R; ++y)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    dst[(y * MT + mt) * 64] = acc[y][mt];
                    acc[y][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            return;
        }
        constexpr bool MASK = OUT == WV_OCT_MASK;
        uint4v mk[MASK ? R / 2 : 1][MASK ? MT : 1];
        if constexpr (MASK) {
            // all masks in one batch: a load awaited between stores would wait for those stores too
            const long to_mask = reinterpret_cast<const char *>(q.a.mask) - reinterpret_cast<const char *>(q.a.y);     // laid out like y
#pragma unroll
            for (int y = 0; y < R; y += 2) {
                const WideDst<OUT> dst = wide_dst<OUT, KS, R, XW, T>(q.a, c.p, pwv, y, l16, g, mt0);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    mk[y / 2][mt] = uint4v{0u, 0u, 0u, 0u};
                    if (dst.ok[0] && (mt0 + mt) * 2 + (g >> 1) < q.a.c8_out)
                        mk[y / 2][mt] = *reinterpret_cast<const uint4v *>(dst.at[0] + to_mask + mt * 2 * ((long)q.a.OH * q.a.OW * 16));
                }
            }
        }
        float bia[MT][4];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) bia[mt][r] = bias_lds[(mt0 + mt) * 16 + 4 * g + r];
#pragma unroll
        for (int y = 0; y < R; y += 2) {
            const WideDst<OUT> dst = wide_dst<OUT, KS, R, XW, T>(q.a, c.p, pwv, y, l16, g, mt0);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                wide_store<DT, OUT>(q.a, acc[y][mt], acc[y + 1][mt], bia[mt], dst, mt0, mt, g, mk[MASK ? y / 2 : 0][MASK ? mt : 0]);
                acc[y][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
                acc[y + 1][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
    };

    // has this wave maps and pixels of the image in the tile?
    const int Ho = k.a.Ho, Wo = k.a.Wo, c_out = k.a.c_out;
    auto wave_active = [&](const WidePos &p) {
        if ((p.mg * (MG * GT) + wm * MT) * 16 >= c_out) return false;
        if (KS == 1) return p.x0 + pwv * R * 16 < Ho * Wo;
        return p.x0 + (pwv % XW) * 16 < Wo && p.py + dil * (p.ty * T::RT + (pwv / XW) * R) < Ho;
    };

    Cursor cur;
    cur.t = t_first;
    open_item(cur);
    set_offsets(cur.p);
    bool act = wave_active(cur.p);
    if constexpr (KS == 3) {
        constexpr int XE = (NX + 1) / 2, XO = NX / 2;          // the next chunk's input: even loads with step 0, odd ones with step 1
        using std::integral_constant;
#pragma unroll
        for (int u = 0; u < NX; ++u) load_x(cur, 0, u);
#pragma unroll
        for (int cs = 0; cs < 2; ++cs)
#pragma unroll
            for (int u = 0; u < NW; ++u) load_w(cur, cs, cs, u);
        int buf = 0;
        wide_wait<NW>();
        Cursor nxt = cur;
        bool more = step_chunk(nxt);
        if (more && nxt.t != cur.t) set_offsets(nxt.p);
        while (more) {
            wide_barrier();
            step(act, buf, 0, 0, integral_constant<int, NW + XE>{}, [&](int q) {
                if (q < NW) load_w(cur, 2, 2, q);
                else load_x(nxt, buf ^ 1, 2 * (q - NW));
            });
            wide_wait<NW + XE>();                              // W(1) of this chunk has landed; younger: what step 0 loaded
            wide_barrier();
            step(act, buf, 1, 1, integral_constant<int, NW + XO>{}, [&](int q) {
                if (q < NW) load_w(nxt, 0, 0, q);
                else load_x(nxt, buf ^ 1, 2 * (q - NW) + 1);
            });
            wide_wait<XE + NW + XO>();                         // W(2); younger: the next input and the next chunk's W(0)
            wide_barrier();
            // The cursor moves on while the other wave of the SIMD multiplies: the first half of the waves moves it before
            // its MFMAs, the second half after them (a new tile is some hundreds of scalar instructions).
            Cursor after = nxt;
            auto move = [&]() {
                more = step_chunk(after);
                if (more && after.t != nxt.t) set_offsets(after.p);
            };
            if (wave < NWV / 2) move();
            step(act, buf, 2, 2, integral_constant<int, NW>{}, [&](int q) { load_w(nxt, 1, 1, q); });
            if (wave >= NWV / 2) move();
            wide_wait<NW>();                                   // the next input and W(0); before the stores, which are younger
            if (cur.ch + 1 == cur.end && act) epilogue(cur);
            if (nxt.t != cur.t) act = wave_active(nxt.p);
            cur = nxt;
            nxt = after;
            buf ^= 1;
        }
        wide_barrier();
        step(act, buf, 0, 0, integral_constant<int, NW>{}, [&](int q) { load_w(cur, 2, 2, q); });
        wide_wait<NW>();
        wide_barrier();
        step(act, buf, 1, 1, integral_constant<int, 0>{}, [](int) {});
        wide_wait<0>();
        wide_barrier();
        step(act, buf, 2, 2, integral_constant<int, 0>{}, [](int) {});
    } else {
        Cursor iss = cur;
        bool pending = true;                                   // iss names a chunk that is not loaded yet
        int ahead = 0, ibuf = 0, buf = 0;                      // chunks loaded and not multiplied; stages of either cursor
        auto load = [&](int q) {
            if (!pending) return;                              // uniform
            if (q < NW) load_w(iss, 0, ibuf, q);
            else load_x(iss, ibuf, q - NW);
        };
        auto advance = [&]() {
            ++ahead;
            ibuf = ibuf + 1 == S ? 0 : ibuf + 1;
            const int before = iss.t;
            pending = step_chunk(iss);
            if (pending && iss.t != before) set_offsets(iss.p);
        };
#pragma unroll
        for (int j = 0; j < S - 1; ++j)
            if (pending) {
#pragma unroll
                for (int q = 0; q < NW + NX; ++q) load(q);
                advance();
            }
        while (true) {
            // this chunk's loads; those of the younger chunks may be in flight
            static_assert(S == 3 || S == 4, "up to two chunks behind the one that is waited for");
            if (S == 4 && ahead >= 3) wide_wait<2 * (NW + NX)>();
            else if (ahead == 2) wide_wait<NW + NX>();
            else wide_wait<0>();
            wide_barrier();
            step(act, buf, 0, buf, std::integral_constant<int, NW + NX>{}, load);
            if (pending) advance();
            --ahead;
            buf = buf + 1 == S ? 0 : buf + 1;
            if (cur.ch + 1 == cur.end) {
                if (act) epilogue(cur);
                cur.t += nslots;
                if (cur.t >= t_end) return;
                const WideArgs &q = *wide_args();
                const int sp = cur.t / q.w.tiles;
                cur.p = wide_decode<KS, T>(q.w, q.a.n, cur.t - sp * q.w.tiles);
                cur.ch = (int)((long)q.w.nchunks * sp / q.w.split);
                cur.end = (int)((long)q.w.nchunks * (sp + 1) / q.w.split);
                act = wave_active(cur.p);
            } else {
                ++cur.ch;
            }
        }
    }
    if (act) epilogue(cur);
}

// Sum of the partial sums of a split launch and its epilogue: a wave takes one pair of rows of one wave of one tile.
template <int DT, int NWV, int KS, int MG, int R, int XW, int OUT, int MT, int GT>
__global__ __launch_bounds__(256) void conv_wide_reduce_h_kernel(WideArgs k)
{
    const ConvHArgs &a = k.a;
    const WideGeom &w = k.w;
    using T = WideTile<NWV, KS, MG, R, XW, MT, GT>;
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const long unit = (long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = (int)(unit / (NWV * (R / 2))), rest = (int)(unit % (NWV * (R / 2)));
    const int wave = rest / (R / 2), y = rest % (R / 2) * 2;
    if (tile >= w.tiles) return;
    const int wm = wave / T::PWV, pwv = wave % T::PWV;
    const WidePos p = wide_decode<KS, T>(w, a.n, tile);
    const int mt0 = p.mg * (MG * GT) + wm * MT;
    if (mt0 * 16 >= a.c_out) return;
    if (KS == 1 ? p.x0 + pwv * R * 16 >= a.Ho * a.Wo : (p.x0 + (pwv % XW) * 16 >= a.Wo || p.py + a.d * (p.ty * T::RT + (pwv / XW) * R) >= a.Ho)) return;
    const WideDst<OUT> dst = wide_dst<OUT, KS, R, XW, T>(a, p, pwv, y, l16, g, mt0);
    uint4v mk[MT];
    float bia[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        mk[mt] = uint4v{0u, 0u, 0u, 0u};
        if constexpr (OUT == WV_OCT_MASK) {
            const long to_mask = reinterpret_cast<const char *>(a.mask) - reinterpret_cast<const char *>(a.y);
            if (dst.ok[0] && (mt0 + mt) * 2 + (g >> 1) < a.c8_out)
                mk[mt] = *reinterpret_cast<const uint4v *>(dst.at[0] + to_mask + mt * 2 * ((long)a.OH * a.OW * 16));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = (mt0 + mt) * 16 + 4 * g + r;
            bia[mt][r] = a.bias && o < (a.c_out + 15) / 16 * 16 ? a.bias[o] : 0.f;
        }
    }
    floatx4 v[2 * MT];
#pragma unroll
    for (int q = 0; q < 2 * MT; ++q) v[q] = floatx4{0.f, 0.f, 0.f, 0.f};
    const floatx4 *src = reinterpret_cast<const floatx4 *>(w.ws + (long)tile * T::FLOATS) + ((long)wave * R + y) * MT * 64 + lane;
#pragma unroll 2
    for (int sp = 0; sp < w.split; ++sp) {
#pragma unroll
        for (int q = 0; q < 2 * MT; ++q) v[q] += src[q * 64];
        src += (long)w.tiles * (T::FLOATS / 4);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) wide_store<DT, OUT>(a, v[mt], v[MT + mt], bia[mt], dst, mt0, mt, g, mk[mt]);
}

template <int NWV, int KS, int MG, int R, int XW, int MT, int GT>
WideGeom wide_geom(const ConvHArgs &a)
{
    using T = WideTile<NWV, KS, MG, R, XW, MT, GT>;
    WideGeom w{};
    w.pgroups = ((a.c_out + 15) / 16 + GT - 1) / GT;
    w.mgroups = (w.pgroups + MG - 1) / MG;
    w.nchunks = (a.c8_in + 3) / 4;
    w.split = 1;
    if (KS == 1) {
        w.xtiles = (int)(((long)a.Ho * a.Wo + T::TX - 1) / T::TX);
        w.ytiles = w.tiles_hi = w.tiles_lo = 1;
        w.pw = T::TX;
        w.oct_units = T::TX;
    } else {
        w.xtiles = (a.Wo + T::TX - 1) / T::TX;
        const int q = a.Ho / a.d;
        w.rem = a.Ho % a.d;
        w.tiles_hi = (q + 1 + T::RT - 1) / T::RT;
        w.tiles_lo = (q + T::RT - 1) / T::RT;
        w.ytiles = w.rem * w.tiles_hi + (a.d - w.rem) * w.tiles_lo;
        if (w.tiles_lo < 1) w.tiles_lo = 1;
        w.pw = T::TX + 2 * a.d;
        w.oct_units = ((T::RT + 2) * w.pw + 63) / 64 * 64;
    }
    const long tiles = (long)w.xtiles * w.ytiles * w.mgroups * a.n;
    w.tiles = w.total = tiles > 0x3fffffffL ? 0 : (int)tiles;
    return w;
}

template <int KS, int MG, int S, int GT>
size_t wide_smem(const WideGeom &w)
{
    const size_t x = (size_t)(KS == 3 ? 2 : S) * 4 * w.oct_units * 16, wt = (size_t)(KS == 3 ? 3 : S) * KS * GT * MG * 1024;
    return x + wt + (w.split > 1 ? 0 : (size_t)w.pgroups * GT * 16 * sizeof(float));
}

template <int NWV, int KS, int MG, int S, int GT>
bool wide_fits(const WideGeom &w)
{
    return w.tiles >= 1 && w.oct_units <= 64 * (NWV / 4) * WV_XQ && wide_smem<KS, MG, S, GT>(w) <= 160 * 1024;
}

// Input loads of a wave per chunk, 3x3: exact for the tile of kernel stride 1 (LEAST), one more up to about stride 4, the most for
// wider ones
template <class T, int LPO> struct WideLoads {
    static constexpr int LEAST = (((T::RT + 2) * (T::TX + 2) + 63) / 64 + LPO - 1) / LPO, MORE = LEAST + 1 < WV_XQ ? LEAST + 1 : WV_XQ;
    static int of(const WideGeom &w)
    {
        const int nx = ((w.oct_units + 63) / 64 + LPO - 1) / LPO;
        return nx <= LEAST ? LEAST : nx <= MORE ? MORE : WV_XQ;
    }
};

template <int DT, int NWV, int KS, int MG, int R, int XW, int NX, bool PAD, int OUT, int S, int MT, int GT>
hipError_t launch_wide_n(const WideArgs &k, size_t smem, hipStream_t stream)
{
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_wide_h_kernel<DT, NWV, KS, MG, R, XW, NX, PAD, OUT, S, MT, GT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int blocks = wide_cus() / 8 * 8 * (NWV == 4 && smem <= 80 * 1024 ? 2 : 1);
    if (k.w.total < blocks) blocks = (k.w.total + 7) / 8 * 8;
    hipLaunchKernelGGL((conv_wide_h_kernel<DT, NWV, KS, MG, R, XW, NX, PAD, OUT, S, MT, GT>), dim3(blocks), dim3(64 * NWV), smem, stream, k);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || k.w.split == 1) return e;
    const long waves = (long)k.w.tiles * NWV * (R / 2);
    hipLaunchKernelGGL((conv_wide_reduce_h_kernel<DT, NWV, KS, MG, R, XW, OUT, MT, GT>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, stream, k);
    return hipGetLastError();
}

template <int DT, int NWV, int KS, int MG, int R, int XW, int OUT, int S, int MT = 4, int GT = 4>
hipError_t launch_wide_m(const ConvHArgs &a, int split, hipStream_t stream)
{
    using T = WideTile<NWV, KS, MG, R, XW, MT, GT>;
    constexpr int LPO = NWV / 4;
    WideArgs k;
    k.a = a;
    k.w = wide_geom<NWV, KS, MG, R, XW, MT, GT>(a);
    WideGeom &w = k.w;
    if (split > w.nchunks) split = w.nchunks;
    while (split > 1 && (!a.ws || (long)w.tiles * split * T::FLOATS > a.ws_floats)) --split;
    w.split = split;
    w.ws = a.ws;
    const size_t smem = wide_smem<KS, MG, S, GT>(w);
    if (!wide_fits<NWV, KS, MG, S, GT>(w) || !a.zeros) return hipErrorInvalidValue;
    // (sample offsets inside an octet plane are 32-bit)
    if ((long)a.H * a.W * 16 >= 0xffffffffL || (long)(a.out_f32 ? a.c_out * 4L : a.c8_out_total * 16L) * a.OH * a.OW >= 0x7fffffffL) return hipErrorInvalidValue;
    if ((long)w.tiles * split > 0x3fffffffL) return hipErrorInvalidValue;
    w.total = w.tiles * split;
    if constexpr (KS == 1) {
        return launch_wide_n<DT, NWV, 1, MG, R, XW, T::TX / (64 * LPO), false, OUT, S, MT, GT>(k, smem, stream);
    } else {
        using L = WideLoads<T, LPO>;
        const int nx = L::of(w);
        if (a.in_off) {
            if (nx == L::LEAST) return launch_wide_n<DT, NWV, 3, MG, R, XW, L::LEAST, true, OUT, S, MT, GT>(k, smem, stream);
            if (nx == L::MORE) return launch_wide_n<DT, NWV, 3, MG, R, XW, L::MORE, true, OUT, S, MT, GT>(k, smem, stream);
            return launch_wide_n<DT, NWV, 3, MG, R, XW, WV_XQ, true, OUT, S, MT, GT>(k, smem, stream);
        }
        if (nx == L::LEAST) return launch_wide_n<DT, NWV, 3, MG, R, XW, L::LEAST, false, OUT, S, MT, GT>(k, smem, stream);
        if (nx == L::MORE) return launch_wide_n<DT, NWV, 3, MG, R, XW, L::MORE, false, OUT, S, MT, GT>(k, smem, stream);
        return launch_wide_n<DT, NWV, 3, MG, R, XW, WV_XQ, false, OUT, S, MT, GT>(k, smem, stream);
    }
}

template <int DT, int NWV, int KS, int MG, int R, int XW, int S, int MT = 4, int GT = 4>
hipError_t launch_wide(const ConvHArgs &a, int split, hipStream_t stream)
{
    return a.mask ? launch_wide_m<DT, NWV, KS, MG, R, XW, WV_OCT_MASK, S, MT, GT>(a, split, stream)
                  : launch_wide_m<DT, NWV, KS, MG, R, XW, WV_OCT, S, MT, GT>(a, split, stream);
}

// What a launch of one tile shape takes, roughly, in microseconds: `fit` the measured times of a step and of a tile's rest
// (epilogue, first loads) with a CU's workgroups busy, `lone` the same for a single tile per CU where two workgroups share one.
// A split adds the reduction's launch and the partial sums written and read once.
struct WideFit {
    double step, rest, lone_step, lone_rest;
};
template <int NWV, int KS, int MG, int R, int XW, int S, int MT = 4, int GT = 4>
double wide_cost(const ConvHArgs &a, int split, const WideFit &f)
{
    using T = WideTile<NWV, KS, MG, R, XW, MT, GT>;
    WideGeom w = wide_geom<NWV, KS, MG, R, XW, MT, GT>(a);
    w.split = split;
    if (split > w.nchunks || !wide_fits<NWV, KS, MG, S, GT>(w)) return 1e30;
    const double items = (double)w.tiles * split;
    if (split > 1 && (!a.ws || items * T::FLOATS > (double)a.ws_floats)) return 1e30;
    const int cus = wide_cus(), steps = KS * ((w.nchunks + split - 1) / split);
    const double rounds = std::ceil(items / cus);
    const double t = rounds == 1 ? steps * f.lone_step + f.lone_rest : rounds * (steps * f.step + f.rest);
    return t + (split > 1 ? 5 + items * T::FLOATS * 8 / 8e6 : 0);
}

struct WidePick {
    int shape, split;
};
WidePick wide_pick(const ConvHArgs &a)
{
    if (a.out_f32) return {0, 1};         // class planes: not where the time goes, one shape that fits every kernel stride
    // The shape and split with the least estimated time.  Which one that is turns on how the tiles fill the CUs: measured (us,
    // with the launch's own 5 to 8), 3x3 with 64 x 8 rows x 32 / 16 x 32 / 12 x 64 pixels --  64 -> 64 at 570^2: 38.6 / 38.6 / 37.0;
    // 256 -> 256 at 138^2: 38.3 / 31.3 / 39.4; 512 -> 256 at 104^2: 36.0 / 51.8 / 67.7; 1024 -> 1024 at 30^2: 61.9 / 95.4 /
    // 122.3, split in four, eight, eight 32.4 / 35.2 / 40.
    double best = 1e30;
    WidePick pick{-1, 1};
    auto take = [&](int s, int sp, double cost) {
        if (cost < best) {
            best = cost;
            pick = {s, sp};
        }
    };
    const int splits[] = {1, 2, 3, 4, 6, 8};
    for (int sp : splits) {
        if (a.k == 3) {
            take(0, sp, wide_cost<8, 3, 1, 4, 2, 3, 2>(a, sp, {0.52, 2.8, 0.52, 2.8}));
            take(1, sp, wide_cost<8, 3, 1, 4, 2, 3>(a, sp, {0.93, 4.6, 0.93, 4.6}));
            take(2, sp, wide_cost<8, 3, 1, 6, 4, 3>(a, sp, {1.20, 6.5, 1.20, 6.5}));
        } else {
            take(0, sp, wide_cost<8, 1, 2, 2, 1, 4>(a, sp, {0.36, 2.3, 0.36, 2.3}));
            take(1, sp, wide_cost<4, 1, 2, 4, 1, 4>(a, sp, {0.31, 1.8, 0.48, 3.0}));
            take(2, sp, wide_cost<4, 1, 2, 8, 1, 3>(a, sp, {0.42, 3.0, 0.60, 4.0}));
            take(3, sp, wide_cost<4, 1, 1, 4, 1, 3>(a, sp, {0.45, 2.7, 0.50, 3.0}));
        }
    }
    return pick;
}

template <int DT>
hipError_t launch_wide_dt(const ConvHArgs &a, hipStream_t stream)
{
    if (a.out_f32) {
        if (a.mask) return hipErrorInvalidValue;
        return a.k == 3 ? launch_wide_m<DT, 8, 3, 1, 4, 2, WV_F32, 3, 2>(a, 1, stream) : launch_wide_m<DT, 8, 1, 2, 2, 1, WV_F32, 4>(a, 1, stream);
    }
    const WidePick pick = wide_pick(a);
    const int split = pick.split;
    if (a.k == 3) {
        switch (pick.shape) {
        case 0: return launch_wide<DT, 8, 3, 1, 4, 2, 3, 2>(a, split, stream);
        case 1: return launch_wide<DT, 8, 3, 1, 4, 2, 3>(a, split, stream);
        case 2: return launch_wide<DT, 8, 3, 1, 6, 4, 3>(a, split, stream);
        }
    } else {
        switch (pick.shape) {
        case 0: return launch_wide<DT, 8, 1, 2, 2, 1, 4>(a, split, stream);
        case 1: return launch_wide<DT, 4, 1, 2, 4, 1, 4>(a, split, stream);
        case 2: return launch_wide<DT, 4, 1, 2, 8, 1, 3>(a, split, stream);
        case 3: return launch_wide<DT, 4, 1, 1, 4, 1, 3>(a, split, stream);
        }
    }
    return hipErrorInvalidValue;
}

template <int NWV, int KS, int MG, int R, int XW, int S, int MT = 4, int GT = 4>
ConvHPath wide_path(const ConvHArgs &a, const WidePick &p)
{
    using T = WideTile<NWV, KS, MG, R, XW, MT, GT>;
    const WideGeom w = wide_geom<NWV, KS, MG, R, XW, MT, GT>(a);
    const int loads = KS == 1 ? T::TX / (64 * (NWV / 4)) : WideLoads<T, NWV / 4>::of(w);
    return {wide_fits<NWV, KS, MG, S, GT>(w) ? 1 : -1, p.shape, p.split, loads};
}

}  // namespace

ConvHPath conv_wide_path(const ConvHArgs &a)
{
    const WidePick p = wide_pick(a);
    if (a.k == 3) {
        switch (p.shape) {
        case 0: return wide_path<8, 3, 1, 4, 2, 3, 2>(a, p);
        case 1: return wide_path<8, 3, 1, 4, 2, 3>(a, p);
        case 2: return wide_path<8, 3, 1, 6, 4, 3>(a, p);
        }
    } else {
        switch (p.shape) {
        case 0: return wide_path<8, 1, 2, 2, 1, 4>(a, p);
        case 1: return wide_path<4, 1, 2, 4, 1, 4>(a, p);
        case 2: return wide_path<4, 1, 2, 8, 1, 3>(a, p);
        case 3: return wide_path<4, 1, 1, 4, 1, 3>(a, p);
        }
    }
    return {-1, 0, 1, 0};
}

// 3x3 layers of 17 to 32 output maps (two map tiles, packed as conv_h_kernel's)
bool conv_wide32_applies(const ConvHArgs &a)
{
    if (a.k != 3 || a.c_out <= 16 || a.c_out > 32 || a.out_f32 || a.tap_maps || a.img || a.vpool || a.hd || (a.mt != 0 && a.mt != 2)) return false;
    const WideGeom w = wide_geom<8, 3, 1, 6, 4, 2, 2>(a);
    return a.c8_in >= 4 && wide_fits<8, 3, 1, 3, 2>(w);
}

ConvHPath conv_wide32_path(const ConvHArgs &a) { return wide_path<8, 3, 1, 6, 4, 3, 2, 2>(a, {3, 1}); }

hipError_t launch_conv_wide32_h(const ConvHArgs &a, hipStream_t stream)
{
    if (a.dtype == 1) return launch_wide<1, 8, 3, 1, 6, 4, 3, 2, 2>(a, 1, stream);
    if (a.dtype == 2) return launch_wide<2, 8, 3, 1, 6, 4, 3, 2, 2>(a, 1, stream);
    return hipErrorInvalidValue;
}

// At least 64 output maps with at most a fifth of the packed ones empty, and 32 input maps.  The biases of all maps lie in the LDS
// beside the tile: at 5x5, whose tile is the largest there, layers of more than 7168 maps stay on conv_h_kernel (at the widest
// kernel stride it takes, 18, they would not fit; the other kernel sizes fit wherever conv_h_kernel does).
bool conv_h_wide(int gemm_m, int gemm_c8, int k)
{
    if ((k != 1 && k != 3 && k != 5 && k != 6 && k != 8 && k != 10) || gemm_c8 < 4 || (k == 5 && gemm_m > 7168)) return false;
    const int m_tiles = (gemm_m + 15) / 16, pad = (m_tiles + 3) / 4 * 4 - m_tiles;
    return m_tiles >= 4 && 4 * pad <= m_tiles;
}

hipError_t launch_conv_wide_h(const ConvHArgs &a, hipStream_t stream)
{
    if (a.dtype == 1) return launch_wide_dt<1>(a, stream);
    if (a.dtype == 2) return launch_wide_dt<2>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace sk
