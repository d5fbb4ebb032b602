// Backward pass of the classification head in one kernel (gfx950, 16-bit storage):
//
//   h = ReLU(W1 x + b1)   z = W2 h + b2   loss = mean over labelled pixels of -log softmax(z)[label]
//
// (the 1x1 convolutions a9 / a10 of the SK-Net and the softmax loss of Section 4.3, with the label masking of
// Section 4.2).  Run layer by layer, the backward pass of these three moves the hidden maps five times between the
// GPU and its memory (200 maps per pixel against 48 of the input): written by the forward pass, read by the second
// convolution, by its weight gradient and as the ReLU mask, and their gradient written and read twice more.
// Here a workgroup of eight waves takes 64 pixels at a time and keeps everything but x and dx on the chip:
//   1. a wave owns a pair of hidden tiles (nets with few of them: a share of the pixels too) and keeps its fragments of
//      W1 and W2 in registers for the whole launch: h (recomputed from x, MFMA 16x16x32), rounded to LDS in the octet
//      layout, and the pair's share of z, fp32, to LDS;
//   2. every wave adds the shares and forms the softmax, one pixel per lane; dz = (p - onehot) / P; the loss term (one
//      wave); dh = (W2^T dz) * [h > 0] on the accumulator layout of h, to LDS in the octet layout (16-bit, rounded as
//      the layer-by-layer path rounds when it stores);
//   3. dx = W1^T dh with W1^T fragments in registers: a wave owns 16 input maps of half of the pixel groups;
//   4. the weight gradients contract over pixels: dW1 = dh x^T, dW2 = dz h^T, db1 = dh 1, db2 = dz 1, MFMA operands
//      read from those tiles with the transposing LDS read (ds_read_b64_tr_b16: lane 4r + q of a group of 16 names
//      maps 4q..4q+3 of pixel r and receives pixels 0..3 of map 4q + e); wave w owns the hidden-map tiles
//      w, w + 8, ... of dW1 and dW2 and keeps them in accumulators for the whole launch.
// The x of the next block is in flight during a block and lands in the second x tile, which holds the shares of z until then.
// Bound by LDS and the three barriers a block: about 400 KB of LDS traffic per 64 pixels (3200 cycles of a CU; the
// MFMAs take 1400).  With a wave per 16 pixels and all weights in LDS (four waves, one to a SIMD: 125 KB of LDS) nothing
// hid a load, a barrier or the per-pixel 64-bit divisions.  48 -> 200 -> 2, bf16, 8 x 1024^2 pixels: 2.73 -> 1.91 ms; 512^2:
// 101 -> 75 us.  128 pixels a block spill (82 registers).
// Each workgroup writes its sums once; head_train_reduce_kernel adds the workgroups' copies in a fixed order,
// scatters them to the two layers' dW / db and finishes the loss.
#include "reduce_copies.h"
#include "sk_kernels.h"

namespace sk {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int HB_WAVES = 8, HB_THREADS = 64 * HB_WAVES, HB_PIX = 64;

// bytes a pixel takes in an x tile, which also holds up to 8 partial z of 16 bytes
__host__ __device__ constexpr int x_row_bytes(int ksteps) { return ksteps * 64 + 16 > 128 ? ksteps * 64 + 16 : 128; }

template <int DT> __device__ __forceinline__ floatx4 mfma32(uint4v a, uint4v b, floatx4 c)
{
    if constexpr (DT == 1) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
}

template <int DT> __device__ __forceinline__ unsigned pack16x2(float lo, float hi)
{
    const floatx2 r = {lo, hi};
    if constexpr (DT == 1) return __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2));
    else return __builtin_bit_cast(unsigned, __builtin_convertvector(r, halfx2));
}

template <int DT> __device__ __forceinline__ unsigned short to16(float f)
{
    if constexpr (DT == 1) return __builtin_bit_cast(unsigned short, static_cast<__bf16>(f));
    else return __builtin_bit_cast(unsigned short, static_cast<_Float16>(f));
}

// one operand fragment from an LDS tile in the octet layout: this lane's 8 pixels of its map, two transposing reads
__device__ __forceinline__ uint4v read_frag(const char *lds_base, unsigned off_lo, unsigned off_hi)
{
    typedef short4v __attribute__((address_space(3))) *lds_s4;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(lds_base + off_lo));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(lds_base + off_hi));
    const uint2v l2 = __builtin_bit_cast(uint2v, lo), h2 = __builtin_bit_cast(uint2v, hi);
    return uint4v{l2[0], l2[1], h2[0], h2[1]};
}

// floats of one workgroup's sums: dW1 accumulators [HT][NT1][64][4], dW2 accumulators [HT][64][4], db1 [HT*16], db2 [16],
// the loss terms [1] (padded to a multiple of 4)
__host__ __device__ constexpr int copy_floats_of(int HT, int NT1) { return HT * NT1 * 256 + HT * 256 + HT * 16 + 16 + 4; }

template <int DT, int HT, int KSTEPS, int NT1>
__global__ __launch_bounds__(HB_THREADS) void head_train_bwd_h_kernel(HeadTrainArgs a)
{
    extern __shared__ uint4v smem16[];
    constexpr int HP = (HT + 1) / 2;                             // pairs of hidden tiles = K steps of the products over hidden maps
    constexpr int PH = HT * 32 + 16;                             // bytes of a pixel's row in the h / dh tiles (16 of padding)
    constexpr int PX = KSTEPS * 64 + 16;                         // ... in the x tiles
    constexpr int XB = HB_PIX * x_row_bytes(KSTEPS);                // bytes of an x tile (or of the partial z that share its place)
    constexpr int HSPLIT = HP > 4 ? 8 : HP > 2 ? 4 : 2;          // waves over the hidden pairs; the others split the pixels
    constexpr int NPG = HB_PIX / 16 * HSPLIT / HB_WAVES;            // 16-pixel groups of a wave in the pixel phases
    constexpr int SLOTS = (HT + HB_WAVES - 1) / HB_WAVES;        // hidden tiles of a wave in the weight gradients
    constexpr int XLD = HB_PIX * KSTEPS * 4 / HB_THREADS > 0 ? HB_PIX * KSTEPS * 4 / HB_THREADS : 1;    // octets of x a thread stages
    constexpr int NWG = HB_WAVES / NT1;                          // waves per 16 input maps of dx
    float *w2c = reinterpret_cast<float *>(smem16);              // [4][HT*16]         W2 rows, fp32
    float *b2 = w2c + 4 * HT * 16;                               // [4]
    float *red = b2 + 4;                                         // [16]               block sums
    char *hs = reinterpret_cast<char *>(red + 16);               // [HB_PIX][PH]
    char *dhs = hs + HB_PIX * PH;                                   // [HB_PIX][PH]
    char *xs0 = dhs + HB_PIX * PH;                                  // 2 x [HB_PIX][PX]; the next block's also holds [HP][HB_PIX][4] partial z
    char *dzs = xs0 + 2 * XB;                                    // [HB_PIX][16]  classes 0..3 in the first 8 bytes, zeros behind
    char *zero16 = dzs + HB_PIX * 16;                               // 16 bytes of zeros: the gradient's map quads 2 and 3

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hp = wave % HSPLIT, pg0 = wave / HSPLIT * NPG;     // this wave's hidden pair and first pixel group
    const bool has0 = 2 * hp < HT, has1 = 2 * hp + 1 < HT;       // ... and which of the pair's tiles there are

    // ---- weights: this wave's fragments into registers, W2 into LDS ----------------------------------------------
    uint4v w1[2][KSTEPS], w2f, w1t[HP];
    floatx4 b1[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = 2 * hp + i;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) w1[i][ks] = t < HT ? static_cast<const uint4v *>(a.w1p)[(t * KSTEPS + ks) * 64 + lane] : uint4v{0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < 4; ++r) b1[i][r] = 16 * t + 4 * g + r < a.hidden ? a.b1[16 * t + 4 * g + r] : 0.f;
    }
    {   // A fragment of z = W2 h: row = class, K value 8 g + e = hidden map 16 (2 hp + e / 4) + 4 g + e % 4 (the accumulators' order)
        unsigned short v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int h = 16 * (2 * hp + (e >> 2)) + 4 * g + (e & 3);
            v[e] = to16<DT>((l16 < a.classes && h < a.hidden) ? a.w2[l16 * a.hidden + h] : 0.f);
        }
        w2f = uint4v{v[0] | ((unsigned)v[1] << 16), v[2] | ((unsigned)v[3] << 16), v[4] | ((unsigned)v[5] << 16), v[6] | ((unsigned)v[7] << 16)};
    }
    const int xt = wave % NT1, xg0 = wave / NT1;                 // dx: this wave's input map tile, its first pixel group
#pragma unroll
    for (int pr = 0; pr < HP; ++pr) {   // A fragments of dx = W1^T dh: row = input map, K value 8 g + e = hidden map 32 pr + 8 g + e
        const int c = 16 * xt + l16;
        unsigned short v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int h = 32 * pr + 8 * g + e;
            v[e] = to16<DT>((c < a.c_in && h < a.hidden) ? a.w1[(long)h * a.c_in + c] : 0.f);
        }
        w1t[pr] = uint4v{v[0] | ((unsigned)v[1] << 16), v[2] | ((unsigned)v[3] << 16), v[4] | ((unsigned)v[5] << 16), v[6] | ((unsigned)v[7] << 16)};
    }
    for (int q = tid; q < 4 * HT * 16; q += HB_THREADS) {
        const int cls = q / (HT * 16), h = q - cls * (HT * 16);
        w2c[q] = (cls < a.classes && h < a.hidden) ? a.w2[cls * a.hidden + h] : 0.f;
    }
    if (tid < 4) b2[tid] = tid < a.classes ? a.b2[tid] : 0.f;
    for (int q = tid; q < HB_PIX * 4 + 4; q += HB_THREADS) reinterpret_cast<unsigned *>(dzs)[q] = 0u;       // dzs and zero16
    // labelled pixels P (exact: integers), the same sum in every thread
    long *cs = reinterpret_cast<long *>(red);                    // HB_WAVES longs = the 16 floats
    {
        long local = 0;
        for (int q = tid; q < a.ncounts; q += HB_THREADS) local += a.counts[q];
        for (int off = 32; off > 0; off >>= 1) local += __shfl_down(local, off, 64);
        if (lane == 0) cs[wave] = local;
    }
    __syncthreads();
    float invP;
    {
        long kept = 0;
#pragma unroll
        for (int w = 0; w < HB_WAVES; ++w) kept += cs[w];
        invP = 1.f / (float)(kept > 0 ? kept : 1);
    }

    const int plane = a.plane;
    const long total = (long)a.n * plane;
    const int c8 = (a.c_in + 7) / 8;
    const uint4v *xin = static_cast<const uint4v *>(a.x);
    const long nblocks = (total + HB_PIX - 1) / HB_PIX;

    // image and pixel of a block's first pixel, for the block at work and the one whose x is being loaded: a step of the
    // grid is added to them, so that no block costs a division
    const long step = (long)gridDim.x * HB_PIX, img_step = step / plane;
    const int pix_step = (int)(step - img_step * plane);
    auto advance = [&](long &img, int &pix) {
        img += img_step;
        const unsigned q = (unsigned)pix + (unsigned)pix_step;
        const bool over = q >= (unsigned)plane;
        pix = (int)(over ? q - (unsigned)plane : q);
        img += over ? 1 : 0;
    };
    auto locate = [&](long &img, int &pix, int off) {            // pixel `off` behind (img, pix); past the last one: the last one
        unsigned q = (unsigned)pix + (unsigned)off;
        if (plane >= HB_PIX) {
            const bool over = q >= (unsigned)plane;
            q -= over ? (unsigned)plane : 0u;
            img += over ? 1 : 0;
        } else {
            img += q / (unsigned)plane;
            q %= (unsigned)plane;
        }
        pix = img < a.n ? (int)q : plane - 1;
        img = img < a.n ? img : a.n - 1;
    };
    uint4v nx[XLD];
    auto load_x = [&](long img, int pix) {
#pragma unroll
        for (int i = 0; i < XLD; ++i) {
            const int q = tid + i * HB_THREADS, o = q / HB_PIX;
            long im = img;
            int px = pix;
            locate(im, px, q % HB_PIX);
            const uint4v v = xin[(im * c8 + (o < c8 ? o : c8 - 1)) * plane + px];
            nx[i] = o < c8 ? v : uint4v{0u, 0u, 0u, 0u};
        }
    };
    auto store_x = [&](char *xs) {
#pragma unroll
        for (int i = 0; i < XLD; ++i) {
            const int q = tid + i * HB_THREADS, o = q / HB_PIX;
            if (o < KSTEPS * 4) *reinterpret_cast<uint4v *>(xs + (q % HB_PIX) * PX + o * 16) = nx[i];
        }
    };

    // this lane's offsets into the tiles for the transposing reads (lane 4r + q of a 16-lane group: pixel r, map quad q)
    const int rr = l16 >> 2, q4 = l16 & 3;
    unsigned off_h[SLOTS], off_x[NT1], off_dz;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        int t = wave + HB_WAVES * s;
        t = t < HT ? t : HT - 1;
        off_h[s] = (unsigned)((8 * g + rr) * PH + (2 * t + (q4 >> 1)) * 16 + (q4 & 1) * 8);
    }
#pragma unroll
    for (int nt = 0; nt < NT1; ++nt) off_x[nt] = (unsigned)((8 * g + rr) * PX + (2 * nt + (q4 >> 1)) * 16 + (q4 & 1) * 8);
    off_dz = (unsigned)(q4 < 2 ? (dzs - hs) + (8 * g + rr) * 16 + q4 * 8 : (zero16 - hs));      // relative to hs
    const unsigned dz_step = q4 < 2 ? 16u : 0u;                 // bytes per pixel (the zeros do not move)

    floatx4 acc1[SLOTS][NT1], acc2[SLOTS], accb1[SLOTS], accb2 = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        acc2[s] = floatx4{0.f, 0.f, 0.f, 0.f};
        accb1[s] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nt = 0; nt < NT1; ++nt) acc1[s][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const unsigned one2 = DT == 1 ? 0x3F803F80u : 0x3C003C00u;  // two ones in the storage type
    const uint4v ones = uint4v{one2, one2, one2, one2};
    float loss_local = 0.f;

    // the grid has no more workgroups than there are blocks
    long bimg = (long)blockIdx.x * HB_PIX / plane, ximg = bimg;
    int bpix = (int)((long)blockIdx.x * HB_PIX - bimg * plane), xpix = bpix;
    load_x(ximg, xpix);
    store_x(xs0);
    advance(ximg, xpix);
    load_x(ximg, xpix);                                         // past the last pixel: that pixel, never used
    __syncthreads();
    int cur = 0;
    for (long blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        const char *xs = xs0 + cur * XB;
        char *xnext = xs0 + (cur ^ 1) * XB;
        const int lab = blk * HB_PIX + lane < total ? a.labels[blk * HB_PIX + lane] : -1;      // needed after the first barrier

        // ---- 1. h of the wave's hidden pair on its pixel groups, and the pair's share of z -------------------------
        floatx4 hacc[2][NPG];
        if (has0) {
#pragma unroll
            for (int j = 0; j < NPG; ++j) {
                const int px = 16 * (pg0 + j) + l16;
                hacc[0][j] = b1[0];
                hacc[1][j] = b1[1];
#pragma unroll
                for (int ks = 0; ks < KSTEPS; ++ks) {
                    const uint4v bv = *reinterpret_cast<const uint4v *>(xs + px * PX + (4 * ks + g) * 16);
                    hacc[0][j] = mfma32<DT>(w1[0][ks], bv, hacc[0][j]);
                    hacc[1][j] = mfma32<DT>(w1[1][ks], bv, hacc[1][j]);
                }
            }
#pragma unroll
            for (int j = 0; j < NPG; ++j) {
                // ReLU, rounding to the storage type (what the layer-by-layer path stores), z
                const int px = 16 * (pg0 + j) + l16;
                uint4v hv;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    hv[2 * i] = pack16x2<DT>(fmaxf(hacc[i][j][0], 0.f), fmaxf(hacc[i][j][1], 0.f));
                    hv[2 * i + 1] = pack16x2<DT>(fmaxf(hacc[i][j][2], 0.f), fmaxf(hacc[i][j][3], 0.f));
                }
                char *row = hs + px * PH + (4 * hp + (g >> 1)) * 16 + (g & 1) * 8;
                *reinterpret_cast<uint2v *>(row) = uint2v{hv[0], hv[1]};
                if (has1) *reinterpret_cast<uint2v *>(row + 32) = uint2v{hv[2], hv[3]};
                const floatx4 z = mfma32<DT>(w2f, hv, floatx4{0.f, 0.f, 0.f, 0.f});
                if (g == 0) *reinterpret_cast<floatx4 *>(xnext + (hp * HB_PIX + px) * 16) = z;
            }
        }
        __syncthreads();                                        // all shares of z are in LDS

        // ---- 2. softmax, loss term and dz = (p - onehot) / P, one pixel per lane, the same in every wave --------------
        floatx4 z = *reinterpret_cast<const floatx4 *>(b2);
#pragma unroll
        for (int pr = 0; pr < HP; ++pr) z += *reinterpret_cast<const floatx4 *>(xnext + (pr * HB_PIX + lane) * 16);
        const bool kept = lab >= 0 && lab < a.classes;
        float m = z[0];
#pragma unroll
        for (int c = 1; c < 4; ++c)
            if (c < a.classes) m = fmaxf(m, z[c]);
        float e[4], dz[4], sum = 0.f, zl = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            e[c] = 0.f;
            if (c < a.classes) e[c] = expf(z[c] - m);           // uniform
            sum += e[c];
            zl = c == lab ? z[c] : zl;
        }
        const float inv = 1.f / sum;
#pragma unroll
        for (int c = 0; c < 4; ++c) dz[c] = kept && c < a.classes ? (e[c] * inv - (c == lab ? 1.f : 0.f)) * invP : 0.f;
        if (wave == HB_WAVES - 1) {                             // (the wave with the least to do in phase 1)
            if (kept) loss_local -= zl - m - logf(sum);
            *reinterpret_cast<uint2v *>(dzs + lane * 16) = uint2v{pack16x2<DT>(dz[0], dz[1]), pack16x2<DT>(dz[2], dz[3])};
        }
        // dh = (W2^T dz) where h > 0, rounded to the storage type
        if (has0) {
            floatx4 v[2][NPG];
#pragma unroll
            for (int j = 0; j < NPG; ++j) v[0][j] = v[1][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (c >= a.classes) break;                      // uniform
                const float *wp = w2c + c * (HT * 16) + 32 * hp + 4 * g;
                const floatx4 wa = *reinterpret_cast<const floatx4 *>(wp), wb = has1 ? *reinterpret_cast<const floatx4 *>(wp + 16) : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < NPG; ++j) {
                    const float d = __shfl(dz[c], 16 * (pg0 + j) + l16, 64);
                    v[0][j] += wa * d;
                    v[1][j] += wb * d;
                }
            }
#pragma unroll
            for (int j = 0; j < NPG; ++j) {
                char *row = dhs + (16 * (pg0 + j) + l16) * PH + (4 * hp + (g >> 1)) * 16 + (g & 1) * 8;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[i][j][r] = hacc[i][j][r] > 0.f ? v[i][j][r] : 0.f;
                    if (i == 0 || has1) *reinterpret_cast<uint2v *>(row + 32 * i) = uint2v{pack16x2<DT>(v[i][j][0], v[i][j][1]), pack16x2<DT>(v[i][j][2], v[i][j][3])};
                }
            }
        }
        __syncthreads();                                        // h, dh and dz of the block are in LDS, the shares of z are read

        store_x(xnext);
        advance(ximg, xpix);
        load_x(ximg, xpix);                                     // in flight during the next block

        // ---- 3. dx = W1^T dh -----------------------------------------------------------------------------------------
        if (a.dx != nullptr && xg0 < NWG) {
            char *dxp = static_cast<char *>(a.dx);
            const int o8 = 2 * xt + (g >> 1);                   // lane (g, l16) holds input maps 16 xt + 4g .. + 3 of its pixel: half an octet
#pragma unroll
            for (int j = 0; j < (HB_PIX / 16 + NWG - 1) / NWG; ++j) {
                const int pg = xg0 + j * NWG;
                if (pg >= HB_PIX / 16) break;                      // uniform
                const char *row = dhs + (16 * pg + l16) * PH;
                floatx4 dxa = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int pr = 0; pr < HP; ++pr) {
                    const bool there = 4 * pr + 3 < 2 * HT || 4 * pr + g < 2 * HT;      // an odd number of tiles: no octets behind the last
                    uint4v dv = *reinterpret_cast<const uint4v *>(row + (there ? 4 * pr + g : 0) * 16);
                    if (!there) dv = uint4v{0u, 0u, 0u, 0u};
                    dxa = mfma32<DT>(w1t[pr], dv, dxa);
                }
                long img = bimg;
                int pix = bpix;
                const bool inside = blk * HB_PIX + 16 * pg + l16 < total;
                locate(img, pix, 16 * pg + l16);
                if (inside && o8 < c8)
                    *reinterpret_cast<uint2v *>(dxp + ((img * c8 + o8) * plane + pix) * 16 + (g & 1) * 8) =
                        uint2v{pack16x2<DT>(dxa[0], dxa[1]), pack16x2<DT>(dxa[2], dxa[3])};
            }
        }

        // ---- 4. weight gradients: contraction over the block's pixels (K steps of 32) ----------------------------------
#pragma unroll
        for (int ks = 0; ks < HB_PIX / 32; ++ks) {
            const uint4v adz = read_frag(hs, off_dz + ks * 32 * dz_step, off_dz + (ks * 32 + 4) * dz_step);
            if (wave == HB_WAVES - 1) accb2 = mfma32<DT>(adz, ones, accb2);
            if (wave >= HT) continue;                           // uniform
            uint4v bx[NT1];
#pragma unroll
            for (int nt = 0; nt < NT1; ++nt) bx[nt] = read_frag(xs, off_x[nt] + ks * 32 * PX, off_x[nt] + (ks * 32 + 4) * PX);
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                if (wave + HB_WAVES * s >= HT) break;           // uniform
                const uint4v adh = read_frag(dhs, off_h[s] + ks * 32 * PH, off_h[s] + (ks * 32 + 4) * PH);
                const uint4v bh = read_frag(hs, off_h[s] + ks * 32 * PH, off_h[s] + (ks * 32 + 4) * PH);
#pragma unroll
                for (int nt = 0; nt < NT1; ++nt) acc1[s][nt] = mfma32<DT>(adh, bx[nt], acc1[s][nt]);
                accb1[s] = mfma32<DT>(adh, ones, accb1[s]);
                acc2[s] = mfma32<DT>(adz, bh, acc2[s]);
            }
        }
        __syncthreads();                                        // the tiles are read and the next x is written
        advance(bimg, bpix);
        cur ^= 1;
    }

    // ---- this workgroup's sums -----------------------------------------------------------------------------------
    float *copy = a.scratch + (long)blockIdx.x * copy_floats_of(HT, NT1);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int t = wave + HB_WAVES * s;
        if (t >= HT) break;
#pragma unroll
        for (int nt = 0; nt < NT1; ++nt) *reinterpret_cast<floatx4 *>(copy + ((t * NT1 + nt) * 64 + lane) * 4) = acc1[s][nt];
        *reinterpret_cast<floatx4 *>(copy + HT * NT1 * 256 + (t * 64 + lane) * 4) = acc2[s];
        if (l16 == 0) *reinterpret_cast<floatx4 *>(copy + HT * NT1 * 256 + HT * 256 + t * 16 + 4 * g) = accb1[s];   // every column holds the same sums
    }
    if (wave == HB_WAVES - 1) {
        if (l16 == 0) *reinterpret_cast<floatx4 *>(copy + HT * NT1 * 256 + HT * 256 + HT * 16 + 4 * g) = accb2;
        for (int off = 32; off > 0; off >>= 1) loss_local += __shfl_down(loss_local, off, 64);
        if (lane == 0) copy[HT * NT1 * 256 + HT * 256 + HT * 16 + 16] = loss_local;
    }
}

// Sums the workgroups' copies element by element (fixed order) and scatters: dW1[h][c], dW2[class][h], db1, db2, loss.
__global__ void __launch_bounds__(256) head_train_reduce_kernel(HeadTrainArgs a, int copies, int HT, int NT1, int copy_floats)
{
    __shared__ __attribute__((aligned(16))) float sh[16][64];
    __shared__ long cnt[4];
    const int e = (int)blockIdx.x * 64 + (int)threadIdx.x;      // (threads 0 .. 63)
    if ((int)blockIdx.x == (int)gridDim.x - 1) {                // the last workgroup finishes the loss
        long local = 0;
        for (int q = threadIdx.x; q < a.ncounts; q += blockDim.x) local += a.counts[q];
        for (int off = 32; off > 0; off >>= 1) local += __shfl_down(local, off, 64);
        if ((threadIdx.x & 63) == 0) cnt[threadIdx.x >> 6] = local;
    }
    const float v = sum_copies64(a.scratch, copy_floats, (int)blockIdx.x * 64, copy_floats, copies, sh);     // (holds a barrier)
    if (threadIdx.x >= 64 || e >= copy_floats) return;
    const int n1 = HT * NT1 * 256, n2 = n1 + HT * 256, n3 = n2 + HT * 16, n4 = n3 + 16;
    if (e < n1) {               // ((t * NT1 + nt) * 64 + lane) * 4 + r: hidden map 16 t + 4 g + r, input map 16 nt + l16
        const int r = e & 3, ln = (e >> 2) & 63, tn = e >> 8, nt = tn % NT1, t = tn / NT1;
        const int h = 16 * t + 4 * (ln >> 4) + r, c = 16 * nt + (ln & 15);
        if (h < a.hidden && c < a.c_in) a.dw1[(long)h * a.c_in + c] = v;
    } else if (e < n2) {        // (t * 64 + lane) * 4 + r: class 4 g + r, hidden map 16 t + l16
        const int q = e - n1, r = q & 3, ln = (q >> 2) & 63, t = q >> 8;
        const int cls = 4 * (ln >> 4) + r, h = 16 * t + (ln & 15);
        if (cls < a.classes && h < a.hidden) a.dw2[(long)cls * a.hidden + h] = v;
    } else if (e < n3) {
        const int h = e - n2;
        if (h < a.hidden && a.db1) a.db1[h] = v;
    } else if (e < n4) {
        const int cls = e - n3;
        if (cls < a.classes && a.db2) a.db2[cls] = v;
    } else if (e == n4) {
        const long kept = cnt[0] + cnt[1] + cnt[2] + cnt[3];
        *a.loss = v / (float)(kept > 0 ? kept : 1);
    }
}

constexpr size_t smem_bytes(int HT, int KSTEPS)
{
    return (size_t)(4 * HT * 16 + 4 + 16) * 4 + (size_t)HB_PIX * (2 * (HT * 32 + 16) + 2 * x_row_bytes(KSTEPS) + 16) + 16;
}

template <int DT, int HT, int KSTEPS, int NT1>
hipError_t launch_t(const HeadTrainArgs &a, int blocks, hipStream_t stream)
{
    constexpr size_t smem = smem_bytes(HT, KSTEPS);
    static_assert(smem <= 160 * 1024, "LDS of a CU");
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&head_train_bwd_h_kernel<DT, HT, KSTEPS, NT1>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((head_train_bwd_h_kernel<DT, HT, KSTEPS, NT1>), dim3(blocks), dim3(HB_THREADS), smem, stream, a);
    return hipGetLastError();
}

template <int DT, int HT>
hipError_t launch_ht(const HeadTrainArgs &a, int nt1, int blocks, hipStream_t stream)
{
    switch (nt1) {
    case 1: return launch_t<DT, HT, 1, 1>(a, blocks, stream);
    case 2: return launch_t<DT, HT, 1, 2>(a, blocks, stream);
    case 3: return launch_t<DT, HT, 2, 3>(a, blocks, stream);
    default: return hipErrorInvalidValue;
    }
}

template <int DT>
hipError_t launch_dt(const HeadTrainArgs &a, int HT, int nt1, int blocks, hipStream_t stream)
{
    return HT == 4 ? launch_ht<DT, 4>(a, nt1, blocks, stream) : HT == 8 ? launch_ht<DT, 8>(a, nt1, blocks, stream) : launch_ht<DT, 13>(a, nt1, blocks, stream);
}

int tiles_of(int hidden)
{
    const int t = (hidden + 15) / 16;
    return t <= 4 ? 4 : t <= 8 ? 8 : 13;
}

}  // namespace

// Which heads this kernel takes: 16-bit storage, at most 48 input maps, 208 hidden maps and 4 classes
bool head_train_supported(int dtype, int c_in, int hidden, int classes)
{
    return (dtype == 1 || dtype == 2) && c_in >= 1 && c_in <= 48 && hidden >= 1 && hidden <= 208 && classes >= 1 && classes <= 4 &&
           head_supported(dtype, c_in, hidden, classes);
}

// floats of scratch: one copy of the sums for each of up to 512 workgroups
size_t head_train_scratch_floats(int c_in, int hidden)
{
    return (size_t)512 * copy_floats_of(tiles_of(hidden), (c_in + 15) / 16);
}

// labels: [n][plane]; counts: ncounts partial counts of the labelled pixels (launch_label_count); scratch: scratch_floats floats
hipError_t launch_head_train_bwd(HeadTrainArgs a, size_t scratch_floats, hipStream_t stream)
{
    if (!head_train_supported(a.dtype, a.c_in, a.hidden, a.classes) || a.n < 1 || a.plane < 1) return hipErrorInvalidValue;
    const int HT = tiles_of(a.hidden), NT1 = (a.c_in + 15) / 16, cf = copy_floats_of(HT, NT1);
    if ((a.c_in + 7) / 8 > (NT1 == 3 ? 8 : 4)) return hipErrorInvalidValue;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    const long total = (long)a.n * a.plane;
    const long nblocks = (total + HB_PIX - 1) / HB_PIX;
    long blocks = cus;
    if (blocks > nblocks) blocks = nblocks;
    if (blocks > (long)(scratch_floats / cf)) blocks = (long)(scratch_floats / cf);
    if (blocks < 1) return hipErrorInvalidValue;
    const hipError_t e = a.dtype == 1 ? launch_dt<1>(a, HT, NT1, (int)blocks, stream) : launch_dt<2>(a, HT, NT1, (int)blocks, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(head_train_reduce_kernel, dim3((cf + 63) / 64), dim3(256), 0, stream, a, (int)blocks, HT, NT1, cf);
    return hipGetLastError();
}

}  // namespace sk
