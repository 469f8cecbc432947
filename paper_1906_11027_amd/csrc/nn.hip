// nn.hip -- kernels of the learned warm start: a small convolutional net that
// maps droplet parameters plus a radial coordinate grid to the steady density
// field, trained and evaluated entirely on the GPU.
//
// Conventions: activations NCHW float32; weights [Cout][Cin][3][3] stored as
// bfloat16 for compute (FP32 master copy for the optimiser); every product
// accumulates in FP32.  Padding is circular (the droplet domain is periodic).
//
// The 3 x 3 convolutions are dense contractions and run on the matrix cores:
//   forward (32 output channels): out[co][p] = sum over 9 taps of
//     W_t[co][ci] x_t[ci][p], one 16 x 16 x 32 bf16 MFMA per (16 channels, 16
//     pixels, tap).  The FP32 activations enter as the exact sum of three bf16
//     parts (hi + mid + lo, 8 significant bits each), so each product is the
//     FP32 activation times the bf16 weight, exact, accumulated in FP32 --
//     three MFMAs per product, the price of keeping the activations in full
//     FP32.
//   backward-data: the forward kernel on the channel-transposed, spatially
//     flipped weights.
//   backward-weight: gW_t[co][ci] = sum_p g[co][p] x[ci][p + d_t], a
//     contraction over pixels with both operands FP32: split into three bf16
//     parts each (32 -> 32 channels) or on FP32 16 x 16 x 4 MFMAs (fewer).
//     Partial sums over a fixed share of the (tile, image) pairs, then a
//     column reduction in a fixed order (deterministic).
// The one-output-channel forward (the net's last layer) stays on the vector
// ALU: a 288-term dot product per pixel.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/sc_lbm.h"
#include "kernels.h"   // xcd_swizzle
#pragma clang fp contract(fast)

namespace sclbm {
namespace nn {

constexpr int TS = 16;      // pixel tile side
constexpr int CCH = 8;      // input channels per LDS chunk
constexpr int MAXC = 32;    // largest channel count

__device__ __forceinline__ float bf16_to_f(uint16_t h)
{
    return __uint_as_float((uint32_t)h << 16);
}

__device__ __forceinline__ uint16_t f_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);  // NaN
    u += 0x7fffu + ((u >> 16) & 1u);   // round to nearest even
    return (uint16_t)(u >> 16);
}

// v mod n for the halo coordinates of a tile: one add or subtract when v is
// within one period of [0, n), a full modulo otherwise (images narrower than
// the tile plus its halo)
__device__ __forceinline__ int wrapc(int v, int n)
{
    const int r = v < 0 ? v + n : (v >= n ? v - n : v);
    if (r >= 0 && r < n) return r;
    const int m = v % n;
    return m < 0 ? m + n : m;
}

template <int COUT>
__global__ void __launch_bounds__(TS* TS)
k_conv_fwd(const float* __restrict__ in, const uint16_t* __restrict__ w, const float* __restrict__ bias,
           float* __restrict__ out, int cin, int cout, int h, int wd)
{
    __shared__ float tile[CCH][TS + 2][TS + 3];
    __shared__ float ws[CCH][9][COUT];   // output channels contiguous: vector LDS reads
    const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * TS + tx;
    const int tiles_x = (wd + TS - 1) / TS;
    // XCD-aware order: the tiles one XCD runs together are neighbours, so
    // the cache lines two tiles share are fetched into one L2
    const int ntl = gridDim.x, L = xcd_swizzle(blockIdx.y * ntl + blockIdx.x, ntl * gridDim.y);
    const int tl = L % ntl, b = L / ntl;
    const int x0 = (tl % tiles_x) * TS, y0 = (tl / tiles_x) * TS;
    const int64_t plane = (int64_t)h * wd;
    const float* inb = in + (int64_t)b * cin * plane;
    float acc[COUT];
#pragma unroll
    for (int co = 0; co < COUT; ++co) acc[co] = (co < cout && bias) ? bias[co] : 0.f;
    for (int c0 = 0; c0 < cin; c0 += CCH) {
        const int nc = cin - c0 < CCH ? cin - c0 : CCH;
        for (int i = tid; i < CCH * (TS + 2) * (TS + 2); i += TS * TS) {
            const int c = i / ((TS + 2) * (TS + 2));
            const int r = i % ((TS + 2) * (TS + 2));
            const int ly = r / (TS + 2), lx = r % (TS + 2);
            float v = 0.f;
            if (c < nc) {
                const int gy = wrapc(y0 + ly - 1, h), gx = wrapc(x0 + lx - 1, wd);
                v = inb[(int64_t)(c0 + c) * plane + (int64_t)gy * wd + gx];
            }
            tile[c][ly][lx] = v;
        }
        for (int i = tid; i < COUT * CCH * 9; i += TS * TS) {
            const int co = i / (CCH * 9), r = i % (CCH * 9), c = r / 9, k = r % 9;
            ws[c][k][co] = (co < cout && c < nc) ? bf16_to_f(w[((int64_t)co * cin + c0 + c) * 9 + k]) : 0.f;
        }
        __syncthreads();
        for (int c = 0; c < nc; ++c) {
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const float v = tile[c][ty + k / 3][tx + k % 3];
#pragma unroll
                for (int co = 0; co < COUT; ++co) acc[co] += ws[c][k][co] * v;
            }
        }
        __syncthreads();
    }
    const int x = x0 + tx, y = y0 + ty;
    if (x < wd && y < h) {
        float* ob = out + (int64_t)b * cout * plane + (int64_t)y * wd + x;
#pragma unroll
        for (int co = 0; co < COUT; ++co)
            if (co < cout) ob[(int64_t)co * plane] = acc[co];
    }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// packed bf16 pairs (high halves) of two FP32 bit patterns: a in the low half
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// Exact split of an FP32 value into three bf16 parts, v = hi + mid + lo: each
// part truncates the remainder to its top 8 significant bits and the
// remainders are exact differences, so 24 bits are carried in all.  The parts
// are the top halves of u0, u1, u2.
__device__ __forceinline__ void split3_bits(float v, uint32_t& u0, uint32_t& u1, uint32_t& u2)
{
    u0 = __float_as_uint(v);
    const float r1 = v - __uint_as_float(u0 & 0xffff0000u);
    u1 = __float_as_uint(r1);
    u2 = __float_as_uint(r1 - __uint_as_float(u1 & 0xffff0000u));
}

constexpr int kPxSlot = 32;                     // bf16 per weight row in LDS: 64 B

// LDS slot s holds 32 bf16 channels as four 16-byte chunks; chunk k is
// stored at position k ^ ((s >> 2) & 3).  A quarter-wave reads one chunk of
// 16 consecutive slots, which then fall on 16 distinct bank quads.
__device__ __forceinline__ int slot_chunk(int s, int k) { return (k ^ (s >> 2)) & 3; }

// Epilogue applied to each output before it is stored (fusing the
// elementwise pass that would otherwise re-read the whole activation)
enum ConvEpi { kEpiNone = 0, kEpiTanh = 1, kEpiTanhGrad = 2 };

template <int EPI>
__device__ __forceinline__ float conv_epi(float v, float yv)
{
    if (EPI == kEpiTanh) return tanhf(v);
    if (EPI == kEpiTanhGrad) return v * (1.f - yv * yv);
    return v;
}

typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

// lane i of each 16 lanes takes src of lane i - 1 (lane 0: its own edge) or of
// lane i + 1 (lane 15: its own edge)
__device__ __forceinline__ u32x4 from_left(u32x4 edge, u32x4 src)
{
    u32x4 d;
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = __builtin_amdgcn_update_dpp(edge[i], src[i], 0x111, 0xf, 0xf, false);
    return d;
}
__device__ __forceinline__ u32x4 from_right(u32x4 edge, u32x4 src)
{
    u32x4 d;
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = __builtin_amdgcn_update_dpp(edge[i], src[i], 0x101, 0xf, 0xf, false);
    return d;
}

// 3 x 3 convolution to 32 channels (forward, and backward-data on the flipped,
// transposed weights) on bf16 MFMAs, the activations going from global memory
// to MFMA operands without LDS or barriers.
//
// A wave walks the rows of a 32-pixel strip.  The pixel operand's lane l holds
// 8 channels (8 (l / 16) ...) of one pixel: per channel one 8-byte load of the
// lane's two pixels x0 + 2 (l % 16) + {0, 1}, 128 contiguous bytes per channel.
// The two pixels are two operands ("phases"), each value split exactly into
// three bf16 parts; the three rows under the window stay in registers as
// parts, so a row is loaded and split once per segment.  For the taps one column
// to the left, phase 1's operand is phase 0 and phase 0's is phase 1 of the lane
// before (DPP within 16 lanes); to the right likewise.  The strip's two outer
// columns are a third operand (lane 0 of each 16 the left, the others the
// right), only there to feed lanes 0 and 15 of those moves.
//
// MFMA rows are output channels (two tiles of 16), so a lane ends with its two
// pixels of a channel: 8-byte stores, 128 bytes per channel.  The weights sit in
// LDS as [tap][co][ci], read as 16-byte operands.
//
// Work units are (image, strip, row segment), the segment height balanced over
// the resident waves (two per SIMD, so one's splits and epilogue run beside
// the other's products).  The last strip of a row is moved left to end at the
// image's edge and stores only its own pixels; NARROW: images narrower than a
// strip, whose columns are loaded one by one, wrapped.
//
// What bounds it: memory and vector issue.  32 -> 32 at batch 16, 256 x 256 reads
// and writes 268 MB (403 with the tanh derivative): 76 us plain (3.6 TB/s), 100
// with the tanh, 110 with its derivative, where 16 x 16 tiles staged through
// LDS took 110, 127 and 180; image sides that are no power of two run 10%
// faster still.  Every accumulator sums the same products in the same order
// as that kernel did: the outputs are the same to the bit.
constexpr int kCPx = 32;        // pixels of a strip
constexpr int kCWaves = 4;      // waves of a block, each with its own unit
constexpr int kCBlocks = 2;     // blocks per CU

template <bool ALL, int EPI, bool BWD, bool NARROW>
__global__ void __launch_bounds__(64 * kCWaves, kCBlocks)
k_conv_rows(const float* __restrict__ in, const uint16_t* __restrict__ w, const float* __restrict__ bias,
            float* __restrict__ out, const float* __restrict__ y, int batch, int cin, int h, int wd, int seg_h,
            int nseg)
{
    __shared__ __align__(16) uint16_t wsl[9 * MAXC * kPxSlot];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    const int64_t plane = (int64_t)h * wd;

    // weights: operand row co, k = ci; the backward pass reads w[ci][co] with
    // the taps reversed
    for (int j = threadIdx.x; j < 9 * MAXC * MAXC; j += 64 * kCWaves) {
        const int t = j >> 10, co = (j >> 5) & 31, ci = j & 31;
        const int sl = t * MAXC + co;
        const int64_t i = BWD ? ((int64_t)ci * MAXC + co) * 9 + 8 - t : ((int64_t)co * cin + ci) * 9 + t;
        wsl[sl * kPxSlot + slot_chunk(sl, ci >> 3) * 8 + (ci & 7)] = ci < cin ? w[i] : (uint16_t)0;
    }
    __syncthreads();
    f32x4 bv[2];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) bv[n][i] = bias ? bias[n * 16 + 4 * kq + i] : 0.f;

    const int strips = (wd + kCPx - 1) / kCPx;
    const int nunits = strips * nseg * batch;
    for (int u = xcd_swizzle(blockIdx.x, gridDim.x) * kCWaves + wv; u < nunits; u += gridDim.x * kCWaves) {
        const int b = u / (strips * nseg), q = u - b * (strips * nseg);
        const int sx = q / nseg, sy = q - sx * nseg;
        const int y0 = sy * seg_h, y1 = y0 + seg_h < h ? y0 + seg_h : h;
        const int xs = sx * kCPx;   // first pixel of the strip's own
        const int x0 = NARROW || xs + kCPx <= wd ? xs : wd - kCPx;
        const int p0 = x0 + 2 * r16;
        const int c0 = ALL ? 8 * kq : 0;
        const float* chan = in + ((int64_t)b * cin + c0) * plane;
        const int xh = wrapc(r16 ? x0 + kCPx : x0 - 1, wd);
        const int xa = NARROW ? wrapc(p0, wd) : p0, xb = NARROW ? wrapc(p0 + 1, wd) : p0 + 1;

        struct Raw {
            f32x2u v[8];
            float e[8];
        };
        // a row in [-1, h + 1]; rows past a segment are loaded ahead and dropped
        auto load = [&](int row, Raw& d) {
            const int wr = row < 0 ? row + h : (row >= h ? row - h : row);
            const float* pr = chan + (int64_t)(wr < h ? wr : h - 1) * wd;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float* p = pr + (ALL ? c : (8 * kq + c < cin ? 8 * kq + c : 0)) * plane;
                if (NARROW) d.v[c] = f32x2u{p[xa], p[xb]};
                else d.v[c] = *(const f32x2u*)(p + p0);
                d.e[c] = p[xh];
            }
        };
        u32x4 pt[3][3][3];   // [row slot][phase, 2 = outer columns][part]
        auto split = [&](const Raw& d, u32x4 (&o)[3][3]) {
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                uint32_t t[3][8];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    float v = f < 2 ? d.v[c][f & 1] : d.e[c];
                    if (!ALL) v = 8 * kq + c < cin ? v : 0.f;
                    split3_bits(v, t[0][c], t[1][c], t[2][c]);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    o[f][k] = u32x4{pack_hi(t[k][0], t[k][1]), pack_hi(t[k][2], t[k][3]), pack_hi(t[k][4], t[k][5]),
                                    pack_hi(t[k][6], t[k][7])};
            }
        };

        Raw raw;
        load(y0 - 1, raw);
        split(raw, pt[0]);
        load(y0, raw);
        split(raw, pt[1]);
        load(y0 + 1, raw);
        for (int r0 = y0; r0 < y1; r0 += 3) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const int r = r0 + s;
                if (r >= y1) continue;   // uniform
                // rows r - 1, r, r + 1 are in slots s, s + 1, s + 2 (mod 3)
                split(raw, pt[(s + 2) % 3]);
                load(r + 2, raw);
                const int64_t o0 = ((int64_t)b * MAXC + 4 * kq) * plane + (int64_t)r * wd + p0;
                f32x2u yv[2][4];
                if (EPI == kEpiTanhGrad)
#pragma unroll
                    for (int n = 0; n < 2; ++n)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float* yp = y + o0 + (n * 16 + i) * plane;
                            if (NARROW) yv[n][i] = f32x2u{p0 < wd ? yp[0] : 0.f, p0 + 1 < wd ? yp[1] : 0.f};
                            else yv[n][i] = *(const f32x2u*)yp;
                        }
                __builtin_amdgcn_sched_barrier(0);   // the loads are issued before the products

                f32x4 acc[2][2];   // [channel tile][phase]
#pragma unroll
                for (int n = 0; n < 2; ++n) acc[n][0] = acc[n][1] = bv[n];
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const int dx = t % 3, sr = (s + t / 3) % 3;
                    const int s0 = t * MAXC + r16, s1 = s0 + 16;
                    const bf16x8 w0 = *(const bf16x8*)(wsl + s0 * kPxSlot + slot_chunk(s0, kq) * 8);
                    const bf16x8 w1 = *(const bf16x8*)(wsl + s1 * kPxSlot + slot_chunk(s1, kq) * 8);
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const u32x4 a0 = pt[sr][0][k], a1 = pt[sr][1][k], ah = pt[sr][2][k];
                        const bf16x8 x0v = __builtin_bit_cast(bf16x8, dx == 0 ? from_left(ah, a1) : (dx == 1 ? a0 : a1));
                        const bf16x8 x1v = __builtin_bit_cast(bf16x8, dx == 0 ? a0 : (dx == 1 ? a1 : from_right(ah, a0)));
                        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x0v, acc[0][0], 0, 0, 0);
                        acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x0v, acc[1][0], 0, 0, 0);
                        acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x1v, acc[0][1], 0, 0, 0);
                        acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x1v, acc[1][1], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float* op = out + o0 + (n * 16 + i) * plane;
                        const float e0 = conv_epi<EPI>(acc[n][0][i], yv[n][i][0]);
                        const float e1 = conv_epi<EPI>(acc[n][1][i], yv[n][i][1]);
                        if (!NARROW && x0 == xs) {   // uniform
                            *(f32x2u*)op = f32x2u{e0, e1};
                        } else {
                            if (p0 >= xs && p0 < wd) op[0] = e0;
                            if (p0 + 1 >= xs && p0 + 1 < wd) op[1] = e1;
                        }
                    }
            }
        }
    }
}

// v with xcd_swizzle(v, nb) == L
__device__ __forceinline__ int xcd_unswizzle(int L, int nb)
{
    const int q = nb >> 3, r = nb & 7;
    if (L < r * (q + 1)) return (L % (q + 1)) * 8 + L / (q + 1);
    const int m = L - r * (q + 1);
    return (m % q) * 8 + r + m / q;
}

// Orders the LDS accesses of a wave's lanes: what any lane did before it, every
// lane sees after it.  The hardware runs a wave's LDS accesses in order, so this
// costs no instruction; it keeps the compiler, which follows one lane at a time,
// from exchanging a store and a load of different lanes' values.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// ---- weight gradients --------------------------------------------------
// gW_t[co][ci] = sum_p g[co][p] x[ci][p + d_t].  Partial row v sums the 16 x 16
// tiles xcd_swizzle(v) + k nblk, k = 0, 1, ..., of all images; it is
//   partial[v][(ci cout + co) 9 + t],  partial[v][cin cout 9 + co] (bias).
// A wave owns a 16 x 16 (co, ci) block of all nine taps of one partial row and
// takes its operands from an LDS patch of its own, so there is no barrier
// between staging and products: two image rows ("a pair") of 16 input and 16
// gradient channels at a time, FP32.  Input pair s of a tile holds rows
// y0 - 1 + 2s and y0 + 2s, s = 0 .. 8; the gradient rows that come with it are
// those of chunk s - 1, y0 + 2s - 2 and y0 + 2s - 1.
constexpr int kWXRow = 24;                     // floats per input channel row: pixel p at 4 + p, outer pixels at 3 and 20
constexpr int kWGRow = 20;                     // floats per gradient channel row
constexpr int kWPatch = 4 * 16 * kWXRow + 2 * 16 * kWGRow;   // floats of a wave: two input pairs, one gradient pair

// EDGE: the image width is not a multiple of 16.  Lanes of the last tile whose
// four pixels pass the image's edge load the row's last four and shift them;
// the pixel beyond the edge, the wrapped first one, is the outer pixel of that
// tile, and what lies past it meets a zero gradient.  kEdgeNarrow: fewer than
// four columns, loaded one by one.
enum WEdge { kEdgeNone = 0, kEdgeShift = 1, kEdgeNarrow = 2 };

// Loads and stages pairs.  Lane l loads 4 pixels from 4 (l & 3) of channel l / 4
// (four lanes a channel row's 64 bytes: with the operands' own layout, one
// channel per lane, every lane would be a cache line of its own) and an outer
// pixel of channel l & 15, row (l / 16) & 1, left or right by l / 32.
template <int EDGE>
struct PairStage {
    const float *in, *gout;
    int nwork, tiles, tiles_x, h, wd;
    int cin, cout, c0, g0;   // channels of an image, and the wave's first
    float* patch;

    struct Raw {
        f32x4 x[2], g[2];
        float o;
    };
    // a tile: the lane's channel rows at its columns (narrow images: column 0),
    // the first row, the columns inside the image and the lane's shift
    struct Tile {
        const float *x, *g, *o;
        int y0, width, sh, col;
        bool live;
    };

    // the patch starts as zeros: what a narrow last tile leaves unwritten has to
    // be a number (it meets zero gradients)
    __device__ __forceinline__ void clear(int lane) const
    {
        for (int i = lane; i < kWPatch; i += 64) patch[i] = 0.f;
        wave_lds_sync();
    }
    // channels that do not exist are read as channel 0
    __device__ __forceinline__ Tile tile(int at, int lane) const
    {
        Tile t;
        const int64_t plane = (int64_t)h * wd;
        const int wi = at < nwork ? at : nwork - 1;
        const int b = wi / tiles, tt = wi - b * tiles;
        const int x0 = (tt % tiles_x) * TS;
        auto chan = [&](const float* base, int nc, int c) { return base + ((int64_t)b * nc + (c < nc ? c : 0)) * plane; };
        const int xw = x0 + 4 * (lane & 3);   // wanted and loaded column
        const int xc = EDGE == kEdgeNarrow ? 0 : (EDGE == kEdgeShift && xw > wd - 4 ? wd - 4 : xw);
        t.y0 = (tt / tiles_x) * TS;
        t.width = EDGE != kEdgeNone && wd - x0 < TS ? wd - x0 : TS;
        t.sh = EDGE == kEdgeShift ? xw - xc : 0;
        t.col = xw;
        t.x = chan(in, cin, c0 + (lane >> 2)) + xc;
        t.g = chan(gout, cout, g0 + (lane >> 2)) + xc;
        t.o = chan(in, cin, c0 + (lane & 15)) + wrapc(lane & 32 ? x0 + t.width : x0 - 1, wd);
        t.live = at < nwork;
        return t;
    }
    // offset of input row r in [-1, TS h]: the wrapped row up to r = h; rows past
    // it meet zero gradients and any will do
    __device__ __forceinline__ int64_t row(int r) const
    {
        const int w = r < 0 ? h - 1 : (r == h ? 0 : (r < h ? r : h - 1));
        return (int64_t)w * wd;
    }
    __device__ __forceinline__ f32x4 four(const float* p, const Tile& t) const
    {
        if (EDGE == kEdgeNarrow)
            return f32x4{p[wrapc(t.col, wd)], p[wrapc(t.col + 1, wd)], p[wrapc(t.col + 2, wd)], p[wrapc(t.col + 3, wd)]};
        return (f32x4)*(const f32x4u*)p;
    }
    __device__ __forceinline__ Raw load(const Tile& t, int s, int lane) const
    {
        Raw v;
        int64_t xr[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            xr[i] = row(t.y0 - 1 + 2 * s + i);
            const int gy = t.y0 + 2 * s - 2 + i;   // s = 0 has no chunk: its gradient is dropped
            const int64_t gr = (int64_t)(gy < 0 ? 0 : (gy < h ? gy : h - 1)) * wd;
            v.x[i] = four(t.x + xr[i], t);
            v.g[i] = four(t.g + gr, t);
        }
        v.o = t.o[lane & 16 ? xr[1] : xr[0]];
        return v;
    }
    static __device__ __forceinline__ f32x4 shifted(f32x4 v, int sh)
    {
        if (EDGE != kEdgeShift) return v;
        const f32x4 a = sh & 1 ? f32x4{v[1], v[2], v[3], v[3]} : v;
        return sh & 2 ? f32x4{a[2], a[3], a[3], a[3]} : a;
    }
    // row i of pair slot k (0 or 1) and of the gradient pair, channel c
    __device__ __forceinline__ float* xrow(int k, int i, int c) const { return patch + ((2 * k + i) * 16 + c) * kWXRow + 4; }
    __device__ __forceinline__ float* grow(int i, int c) const { return patch + 4 * 16 * kWXRow + (i * 16 + c) * kWGRow; }

    // after the slot's last reads, and with the other lanes' values in place for
    // the next; in a ragged tile the outer pixel falls on another lane's row store
    __device__ __forceinline__ void stage(const Raw& v, const Tile& t, int slot, int lane) const
    {
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *(f32x4*)(xrow(slot, i, lane >> 2) + 4 * (lane & 3)) = shifted(v.x[i], t.sh);
            *(f32x4*)(grow(i, lane >> 2) + 4 * (lane & 3)) = shifted(v.g[i], t.sh);
        }
        wave_lds_sync();
        xrow(slot, (lane >> 4) & 1, lane & 15)[lane & 32 ? t.width : -1] = v.o;
        wave_lds_sync();
    }
    // whether gradient row i of pair s >= 1 counts
    __device__ __forceinline__ bool counts(const Tile& t, int s, int i) const
    {
        return t.live && t.y0 + 2 * s - 2 + i < h;
    }
};

// Layers with fewer than 32 channels on either side: FP32 16 x 16 x 4 MFMAs, k
// running over 4 consecutive pixels of a tile row.  NB waves per partial row,
// one per (co, ci) block, 4 / NB rows per block of four waves.
// What bounds it: latency beside the FP32 matrix rate.  36 MFMAs of 32 cycles per
// tile row and wave are 61 us at batch 16, 256 x 256 (2.4 GHz), 0.57 of the 106
// that 5 -> 32 and 32 -> 1 channels take; with one wave per SIMD nothing covers the
// loads, the patch and the bias sums (6 us).  Tiles staged by the whole block
// between two barriers took 150 and 197 us.  Each accumulator adds its products,
// and the bias its gradients, in the same order as then.
template <int NB, int EDGE>
__global__ void __launch_bounds__(256)
k_conv_bwd_w(const float* __restrict__ in, const float* __restrict__ gout, float* __restrict__ partial, int nblk,
             int batch, int cin, int cout, int h, int wd)
{
    constexpr int GR = 4 / NB;   // partial rows a block works on
    __shared__ __align__(16) float lds[4 * kWPatch];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wv / NB, blk = wv % NB;
    const int nci = cin > 16 ? 2 : 1;
    const int mt = blk / nci, nt = blk % nci;
    const int r16 = lane & 15, kq = lane >> 4;
    const int L0 = xcd_swizzle(blockIdx.x, gridDim.x) * GR + grp;   // this row's first tile
    const bool co_ok = mt * 16 + r16 < cout, ci_ok = nt * 16 + r16 < cin;
    using PS = PairStage<EDGE>;
    const int tiles_x = (wd + TS - 1) / TS, tiles = tiles_x * ((h + TS - 1) / TS);
    const PS st{in, gout, tiles * batch, tiles, tiles_x, h, wd, cin, cout, nt * 16, mt * 16, lds + wv * kWPatch};
    st.clear(lane);

    f32x4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum[2] = {0.f, 0.f};   // the bias's running sums of the lane's two row pairs
    // every wave of the block takes the same number of tiles, so that all meet
    // the barrier; without a tile of its own it adds zeros
    // Pair s goes through raw[s mod 3], its loads two pairs ahead: one wave per
    // SIMD has nothing else to cover them with.  Nor the LDS reads: row q of the
    // tile's 18 input rows sits in xw[q mod 3], and the next input row and
    // gradient row are read while this one's 36 products run.
    typename PS::Tile t = st.tile(L0, lane), nxt;
    typename PS::Raw raw[3] = {st.load(t, 0, lane), st.load(t, 1, lane), st.load(t, 2, lane)};
    float g[2][4], xw[3][4][3];   // [4 px group][dx]
    auto take_g = [&](int r, float (&d)[4]) {   // tile row r
        const bool row = co_ok && t.live && t.y0 + r < h;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float v = st.grow(r & 1, r16)[4 * j + kq];
            d[j] = row && (EDGE == kEdgeNone || 4 * j + kq < t.width) ? v : 0.f;
        }
    };
    // without a tile of its own the wave has a copy of the last one: its pixels must
    // not meet the zero gradients, an infinite one would give NaN
    auto take_x = [&](int q, float (&d)[4][3]) {
        const bool ok = ci_ok && t.live;
        const float* x = st.xrow((q >> 1) & 1, q & 1, r16) + kq - 1;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const float v = x[4 * j + dx];
                d[j][dx] = ok ? v : 0.f;
            }
    };
    // The bias sums a pair's 32 pixels one after the other, then the row's tiles:
    // chains that keep a sum of 10^5 values to a few 1e-10 of their magnitudes.
    // The lanes of quarter kq keep pairs 1 + kq and 5 + kq as they pass, so four
    // pairs are summed side by side (one pair at a time: 111 us for 5 -> 32).
    f32x4 hold[2][4];
    auto hold_g = [&](int s) {
        if (kq == ((s - 1) & 3))
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) hold[i][j] = *(const f32x4*)(st.grow(i, r16) + 4 * j);
    };
    auto sum_g = [&](int half) {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bool row = st.counts(t, 4 * half + kq + 1, i);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    sum += row && (EDGE == kEdgeNone || 4 * j + e < t.width) ? hold[i][j][e] : 0.f;
        }
        bsum[half] += sum;
    };
    for (int wi = L0; wi < st.nwork + grp; wi += nblk) {
        __builtin_amdgcn_s_barrier();
        st.stage(raw[0], t, 0, lane);
        raw[0] = st.load(t, 3, lane);
        take_x(0, xw[0]);
        take_x(1, xw[1]);
        st.stage(raw[1], t, 1, lane);
        raw[1] = st.load(t, 4, lane);
        take_x(2, xw[2]);
        take_g(0, g[0]);
        hold_g(1);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float xn[4][3];
            if (r == 9) nxt = st.tile(wi + nblk, lane);
            if (r < 15) {
                if (r & 1) {   // input row r + 3 and gradient row r + 1 open pair s
                    const int s = (r + 3) / 2;
                    st.stage(raw[s % 3], t, s & 1, lane);
                    raw[s % 3] = s < 6 ? st.load(t, s + 3, lane) : st.load(nxt, s - 6, lane);
                    hold_g(s);
                }
                if (r == 6 || r == 14) sum_g(r / 8);
                take_x(r + 3, xn);
                take_g(r + 1, g[(r + 1) & 1]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
                        acc[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x4f32(g[r & 1][j], xw[(r + dy) % 3][j][dx],
                                                                                acc[3 * dy + dx], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) xw[r % 3][j][dx] = r < 15 ? xn[j][dx] : 0.f;
            __builtin_amdgcn_sched_barrier(0);
        }
        t = nxt;
    }
    if (L0 >= nblk) return;
    const int E = cin * cout * 9;
    float* pb = partial + (int64_t)xcd_unswizzle(L0, nblk) * (E + cout);
    const int ci = nt * 16 + r16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int co = mt * 16 + 4 * kq + i;
        if (ci < cin && co < cout)
#pragma unroll
            for (int t = 0; t < 9; ++t) pb[(ci * cout + co) * 9 + t] = acc[t][i];
    }
    // bias: pairs 1 and 2, 3 and 4, ... of a channel, as a tree
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        bsum[k] += __shfl_xor(bsum[k], 16, 64);
        bsum[k] += __shfl_xor(bsum[k], 32, 64);
    }
    if (nt == 0 && kq == 0 && co_ok) pb[E + mt * 16 + r16] = bsum[0] + bsum[1];
}

// The 32 -> 32 weight gradient on bf16 MFMAs: both operands split exactly into
// three bf16 parts and the six part products whose weights reach 2^-24 summed
// (hi.hi, hi.mid, mid.hi, hi.lo, mid.mid, lo.hi): FP32 operands to within about
// 2^-24 of each product.  k runs over the 32 pixels of a chunk (two tile rows),
// 8 consecutive pixels of one row per lane; the splits are made in registers.
// Four waves per partial row, two rows per block.
//
// With input pairs P_s and M_s = the second row of P_(s-1) with the first of
// P_s, chunk c multiplies its gradient rows with P_c (dy = -1), M_(c+1) (dy =
// 0) and P_(c+1) (dy = +1).  The three column shifts of an operand are the same
// ten split values packed in pairs from three starts.  Software pipeline, per
// pair: pass the loaded rows through the patch, issue the next loads, then the
// products of the chunk before run beside the splits of this one.
//
// One barrier per tile keeps a block's waves on the same tiles: without it they
// drift apart and fetch each line twice (553 against 276 MB at batch 16,
// 256 x 256).
//
// What bounds it: vector issue and the matrix cores, 224 VALU instructions
// beside 54 MFMAs per step and wave.  At batch 16, 256 x 256 it takes 128 - 138
// us, where staging the parts of a whole tile through block-wide LDS took 223
// (16-bit stores, one block per CU).  Every accumulator sums the same products
// in the same order as that kernel did, so the weight gradients are the same to the
// bit; the bias gradients are summed in another order, in shorter chains.
constexpr int kWGroups = 2;                    // partial rows a block works on

template <int EDGE>
__global__ void __launch_bounds__(256 * kWGroups)
k_conv_bwd_w_bf16(const float* __restrict__ in, const float* __restrict__ gout, float* __restrict__ partial,
                  int nblk, int batch, int h, int wd)
{
    constexpr int E = MAXC * MAXC * 9;
    constexpr int RED = kWGroups * E > 4 * kWGroups * kWPatch ? kWGroups * E : 4 * kWGroups * kWPatch;
    __shared__ __align__(16) float lds[RED];
    __shared__ float redb[kWGroups * MAXC];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wv >> 2, mt = (wv >> 1) & 1, nt = wv & 1;
    const int r16 = lane & 15, kq = lane >> 4, rs = kq >> 1, c8 = 8 * (kq & 1);
    const int L0 = xcd_swizzle(blockIdx.x, gridDim.x) * kWGroups + grp;   // this row's first tile
    using PS = PairStage<EDGE>;
    const int tiles_x = (wd + TS - 1) / TS, tiles = tiles_x * ((h + TS - 1) / TS);
    const PS st{in, gout, tiles * batch, tiles, tiles_x, h, wd, MAXC, MAXC, nt * 16, mt * 16, lds + wv * kWPatch};
    st.clear(lane);

    f32x4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;

    auto take_g = [&](float (&d)[8]) {
        const float* g = st.grow(rs, r16) + c8;
        const f32x4 g0 = *(const f32x4*)g, g1 = *(const f32x4*)(g + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[j] = g0[j];
            d[4 + j] = g1[j];
        }
    };
    // rows (a, b) for the lanes of the first and the second row; row i of slot
    // k is 2 k + i
    auto take_x = [&](int a, int b, float (&d)[10]) {
        const float* p = st.xrow(0, rs ? b : a, r16) + c8;
        const f32x4 p0 = *(const f32x4*)p, p1 = *(const f32x4*)(p + 4);
        d[0] = p[-1];
        d[9] = p[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[1 + j] = p0[j];
            d[5 + j] = p1[j];
        }
    };
    // one part of an operand: pairs from pixel -1 (five) and from pixel 0 (four)
    struct Part {
        u32x4 ev, od;
        uint32_t el;
    };
    auto split_x = [&](const float (&v)[10], Part (&d)[3]) {
        uint32_t t[3][10];
#pragma unroll
        for (int j = 0; j < 10; ++j) split3_bits(v[j], t[0][j], t[1][j], t[2][j]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            d[k].ev = u32x4{pack_hi(t[k][0], t[k][1]), pack_hi(t[k][2], t[k][3]), pack_hi(t[k][4], t[k][5]),
                            pack_hi(t[k][6], t[k][7])};
            d[k].od = u32x4{pack_hi(t[k][1], t[k][2]), pack_hi(t[k][3], t[k][4]), pack_hi(t[k][5], t[k][6]),
                            pack_hi(t[k][7], t[k][8])};
            d[k].el = pack_hi(t[k][8], t[k][9]);
        }
    };
    // gradient outside the image and of s = 0 enters as zero
    auto split_g = [&](const float (&v)[8], const typename PS::Tile& t, int s, u32x4 (&d)[3]) {
        const bool row = st.counts(t, s, rs);
        uint32_t u[3][8];
        float m[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            m[j] = row && (EDGE == kEdgeNone || c8 + j < t.width) ? v[j] : 0.f;
            split3_bits(m[j], u[0][j], u[1][j], u[2][j]);
        }
        bsum += ((m[0] + m[1]) + (m[2] + m[3])) + ((m[4] + m[5]) + (m[6] + m[7]));
#pragma unroll
        for (int k = 0; k < 3; ++k)
            d[k] = u32x4{pack_hi(u[k][0], u[k][1]), pack_hi(u[k][2], u[k][3]), pack_hi(u[k][4], u[k][5]),
                         pack_hi(u[k][6], u[k][7])};
    };

    Part P[2][3], M[3];
    u32x4 G[2][3];
    auto products = [&](const Part (&x)[3], const u32x4 (&g)[3], int dy) {
#pragma unroll
        for (int xp = 0; xp < 3; ++xp) {
            const u32x4 e = x[xp].ev;
            const u32x4 v[3] = {e, x[xp].od, u32x4{e[1], e[2], e[3], x[xp].el}};
#pragma unroll
            for (int gp = 0; gp + xp < 3; ++gp)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    acc[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, g[gp]),
                                                                               __builtin_bit_cast(bf16x8, v[dx]),
                                                                               acc[3 * dy + dx], 0, 0, 0);
        }
    };
    auto mix = [] {   // one MFMA to a few VALU instructions
#pragma unroll
        for (int k = 0; k < 18; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // every wave of the block takes the same number of tiles, so that all meet
    // the barrier; without a tile of its own it adds zeros
    typename PS::Tile t = st.tile(L0, lane);
    typename PS::Raw raw = st.load(t, 0, lane);
    float gv[8], xv[10], mv[10];
    st.stage(raw, t, 0, lane);
    raw = st.load(t, 1, lane);
    take_x(0, 1, xv);
    split_x(xv, P[0]);
    for (int wi = L0; wi < st.nwork + grp; wi += nblk) {
        __builtin_amdgcn_s_barrier();
        // P[0] = P_0 of this tile.  Step s = 1 has no chunk before it.
        st.stage(raw, t, 1, lane);
        take_g(gv);
        take_x(2, 3, xv);
        take_x(1, 2, mv);
        raw = st.load(t, 2, lane);
        split_g(gv, t, 1, G[1]);
        split_x(xv, P[1]);
        split_x(mv, M);
        const typename PS::Tile nxt = st.tile(wi + nblk, lane);
        // step s, pair slot s & 1: the products of chunk s - 2 beside the splits of chunk s - 1
        auto step = [&](int slot, int s, const typename PS::Tile& ahead, int as) {
            st.stage(raw, t, slot, lane);
            take_g(gv);
            raw = st.load(ahead, as, lane);
            __builtin_amdgcn_sched_barrier(0);
            take_x(2 * slot, 2 * slot + 1, xv);
            products(P[slot], G[slot ^ 1], 0);
            split_g(gv, t, s, G[slot]);
            mix();
            take_x(2 * (slot ^ 1) + 1, 2 * slot, mv);
            products(M, G[slot ^ 1], 1);
            split_x(xv, P[slot]);
            mix();
            products(P[slot ^ 1], G[slot ^ 1], 2);
            split_x(mv, M);
            mix();
        };
#pragma unroll 1
        for (int s = 2; s < 8; s += 2) {
            step(0, s, t, s + 1);
            step(1, s + 1, t, s + 2);
        }
        step(0, 8, nxt, 0);
        // the last chunk beside the next tile's first pair
        st.stage(raw, nxt, 0, lane);
        raw = st.load(nxt, 1, lane);
        __builtin_amdgcn_sched_barrier(0);
        take_x(0, 1, xv);
        products(P[1], G[0], 0);
        products(M, G[0], 1);
        products(P[0], G[0], 2);
        split_x(xv, P[0]);
        t = nxt;
    }
    __syncthreads();   // every wave is done with its patch

    float* red = lds + grp * E;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < 9; ++t) red[((nt * 16 + r16) * MAXC + mt * 16 + 4 * kq + i) * 9 + t] = acc[t][i];
    // bias: the four pixel octets of a channel
    bsum += __shfl_xor(bsum, 16, 64);
    bsum += __shfl_xor(bsum, 32, 64);
    if (nt == 0 && kq == 0) redb[grp * MAXC + mt * 16 + r16] = bsum;
    __syncthreads();
    if (L0 >= nblk) return;
    float* pb = partial + (int64_t)xcd_unswizzle(L0, nblk) * (E + MAXC);
    const int t4 = threadIdx.x & 255;
    for (int e = t4; e < E; e += 256) pb[e] = red[e];
    if (t4 < MAXC) pb[E + t4] = redb[grp * MAXC + t4];
}

// Sum the per-block partials in a fixed order: gw[co][ci][k] from the
// ci-major partial entries, gbias[co] from the trailing bias columns.  A block
// covers 64 columns with 4 row groups (rows r = g mod 4), combined in group
// order through LDS.  A thread's additions are a chain; its loads run ahead of
// it (512 rows of 9,248 columns: 6.4 us, 20 with one load at a time).
constexpr int kSumCols = 64, kSumGroups = 4;
__global__ void __launch_bounds__(kSumCols* kSumGroups)
k_sum_partials(const float* __restrict__ m, int nrow, int cin, int cout, float* __restrict__ gw,
               float* __restrict__ gbias)
{
    __shared__ float part[kSumGroups][kSumCols];
    const int E = cin * cout * 9;
    const int ncol = E + cout;
    const int lc = threadIdx.x % kSumCols, g = threadIdx.x / kSumCols;
    const int j = blockIdx.x * kSumCols + lc;
    float s = 0.f;
    if (j < ncol) {
        // sixteen loads in flight; the additions keep their order
        int r = g;
        for (; r + 15 * kSumGroups < nrow; r += 16 * kSumGroups) {
            float v[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = m[(int64_t)(r + k * kSumGroups) * ncol + j];
#pragma unroll
            for (int k = 0; k < 16; ++k) s += v[k];
        }
        for (; r < nrow; r += kSumGroups) s += m[(int64_t)r * ncol + j];
    }
    part[g][lc] = s;
    __syncthreads();
    if (g != 0 || j >= ncol) return;
    s = ((part[0][lc] + part[1][lc]) + part[2][lc]) + part[3][lc];
    if (j < E) {
        const int ci = j / (cout * 9), rr = j % (cout * 9), co = rr / 9, k = rr % 9;
        gw[((int64_t)co * cin + ci) * 9 + k] = s;
    } else {
        gbias[j - E] = s;
    }
}

__global__ void k_tanh_fwd(float* __restrict__ x, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        x[i] = tanhf(x[i]);
}

__global__ void k_tanh_bwd(const float* __restrict__ y, float* __restrict__ g, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        g[i] *= 1.f - y[i] * y[i];
}

// grad = 2 (out - tgt) / n; partial[blk] = sum (out - tgt)^2 over the block's share
__global__ void __launch_bounds__(256)
k_mse(const float* __restrict__ out, const float* __restrict__ tgt, float* __restrict__ grad, int64_t n,
      double* __restrict__ partial)
{
    __shared__ double red[4];
    double s = 0.0;
    const float scale = 2.f / (float)n;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float d = out[i] - tgt[i];
        if (grad) grad[i] = scale * d;
        s += (double)d * d;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, uint16_t* __restrict__ pb, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        p[i] = pi;
        if (pb) pb[i] = f_to_bf16(pi);
    }
}

__global__ void k_to_bf16(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = f_to_bf16(x[i]);
}

// Input features of image b: channel 0 the distance to the domain centre
// scaled by 1/scale_r, channels 1..4 the image's four (already normalised)
// parameters broadcast over the grid.
__global__ void k_features(const float* __restrict__ prm, float* __restrict__ out, int batch, int h, int wd,
                           float scale_r)
{
    const int64_t plane = (int64_t)h * wd;
    const int64_t total = plane * batch;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int b = (int)(i / plane);
        const int64_t p = i % plane;
        const int y = (int)(p / wd), x = (int)(p % wd);
        const float dx = (float)(x - wd / 2), dy = (float)(y - h / 2);
        float* ob = out + (int64_t)b * 5 * plane + p;
        // distance to the centre relative to the radius carried in params[b][0]
        ob[0] = sqrtf(dx * dx + dy * dy) / scale_r - prm[b * 4];
        for (int c = 0; c < 4; ++c) ob[(int64_t)(c + 1) * plane] = prm[b * 4 + c];
    }
}

// Initial field of a learned start, one workgroup per image (n x n):
// v = mean over the 8 symmetries of the square about node (c, c), c = n/2,
// of base + inv_scale * resid; clamp to [lo, hi]; then shift uniformly to
// the target mass.  Sums in double.
constexpr int kStartThreads = 1024;

__global__ void __launch_bounds__(kStartThreads)
k_start_field(const float* __restrict__ resid, const double* __restrict__ base, const double* __restrict__ mass,
              double* __restrict__ out, int n, float inv_scale, double lo, double hi)
{
    __shared__ double red[kStartThreads / 64];
    __shared__ double shift;
    const int64_t plane = (int64_t)n * n;
    const float* r = resid + blockIdx.x * plane;
    const double* bs = base + blockIdx.x * plane;
    double* o = out + blockIdx.x * plane;
    const int c2 = 2 * (n / 2);
    double acc = 0.0;
    for (int64_t p = threadIdx.x; p < plane; p += blockDim.x) {
        const int i = (int)(p / n), j = (int)(p % n);
        const int ii[2] = {i, (c2 - i + n) % n};
        const int jj[2] = {j, (c2 - j + n) % n};
        double v = 0.0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) {
                const int64_t q0 = (int64_t)ii[a] * n + jj[b];
                const int64_t q1 = (int64_t)jj[b] * n + ii[a];
                v += (bs[q0] + (double)(inv_scale * r[q0])) + (bs[q1] + (double)(inv_scale * r[q1]));
            }
        v *= 0.125;
        v = v < lo ? lo : (v > hi ? hi : v);
        o[p] = v;
        acc += v;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < kStartThreads / 64; ++k) t += red[k];
        shift = (mass[blockIdx.x] - t) / (double)plane;
    }
    __syncthreads();
    const double d = shift;
    for (int64_t p = threadIdx.x; p < plane; p += blockDim.x) o[p] += d;
}

static int grid_for(int64_t n)
{
    int64_t g = (n + 255) / 256;
    return (int)(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

}  // namespace nn
}  // namespace sclbm

using namespace sclbm::nn;

static int nn_status(hipError_t e) { return e == hipSuccess ? SC_OK : SC_E_DEVICE; }

// compute units of the current device (cached per device): the persistent
// forward kernel runs two blocks per CU
static int cu_count()
{
    static int cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!cache[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        cache[dev] = n;
    }
    return cache[dev];
}

// 32 planes of an image hold fewer than 2^31 values (planes are addressed in 64
// bits, pixels, tiles and units counted in 32)
static bool conv_shape_ok(int batch, int cin, int cout, int h, int w)
{
    return batch >= 1 && cin >= 1 && cin <= MAXC && (cout == 1 || cout == MAXC) && h >= 1 && w >= 1 &&
           batch <= 65535 && (int64_t)h * w * MAXC < ((int64_t)1 << 31);
}

// Row-segment height of the row-walking convolution: `cols` strips of h rows
// over `slots` resident waves.  A wave walks ceil(cols nseg / slots) segments of
// H rows, each with about two rows' worth of start-up (the rows around it); the
// height with the least total is taken.
static int segment_height(int64_t cols, int h, int64_t slots)
{
    int best = h;
    int64_t least = INT64_MAX;
    const int64_t most = 4 * slots / cols + 4;   // beyond it every segment is start-up
    for (int n = 1; n <= h && n <= most; ++n) {
        const int H = (h + n - 1) / n;
        const int64_t cost = (cols * ((h + H - 1) / H) + slots - 1) / slots * (H + 2);
        if (cost < least) {
            least = cost;
            best = H;
        }
    }
    return best;
}

// the convolution to 32 channels with its epilogue; BWD: w is the forward
// weights of the layer whose input gradient this is
template <int EPI, bool BWD>
static hipError_t launch_rows(const float* in, const uint16_t* w, const float* bias, float* out, const float* y,
                              int batch, int cin, int h, int wd, hipStream_t s)
{
    const int cols = (wd + kCPx - 1) / kCPx * batch;
    const int64_t slots = (int64_t)cu_count() * kCBlocks * kCWaves;
    const int seg_h = segment_height(cols, h, slots), nseg = (h + seg_h - 1) / seg_h;
    const int64_t units = (int64_t)cols * nseg;
    const int nb = (int)std::min<int64_t>((units + kCWaves - 1) / kCWaves, (int64_t)cu_count() * kCBlocks);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(64 * kCWaves), 0, s, in, w, bias, out, y, batch, cin, h, wd, seg_h,
                           nseg);
    };
    if (wd < kCPx) launch(k_conv_rows<false, EPI, BWD, true>);
    else if (cin == MAXC) launch(k_conv_rows<true, EPI, BWD, false>);
    else launch(k_conv_rows<false, EPI, BWD, false>);
    return hipGetLastError();
}

extern "C" int sc_nn_conv3x3_fwd(const float* in, const uint16_t* w, const float* bias, float* out, int32_t batch,
                                 int32_t cin, int32_t cout, int32_t h, int32_t wd, void* stream)
{
    if (!in || !w || !out || !conv_shape_ok(batch, cin, cout, h, wd)) return SC_E_INVAL;
    if (cout == MAXC)
        return nn_status(
            launch_rows<kEpiNone, false>(in, w, bias, out, nullptr, batch, cin, h, wd, (hipStream_t)stream));
    const int tiles = ((wd + TS - 1) / TS) * ((h + TS - 1) / TS);
    dim3 grid(tiles, batch), block(TS, TS);
    hipLaunchKernelGGL(k_conv_fwd<1>, grid, block, 0, (hipStream_t)stream, in, w, bias, out, cin, cout, h, wd);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_conv3x3_fwd_tanh(const float* in, const uint16_t* w, const float* bias, float* out,
                                      int32_t batch, int32_t cin, int32_t cout, int32_t h, int32_t wd, void* stream)
{
    if (!in || !w || !out || !conv_shape_ok(batch, cin, cout, h, wd) || cout != MAXC) return SC_E_INVAL;
    return nn_status(launch_rows<kEpiTanh, false>(in, w, bias, out, nullptr, batch, cin, h, wd, (hipStream_t)stream));
}

// gradient w.r.t. the input: convolution of gout (cout channels) with the
// flipped, transposed weights (32 output channels), no bias; the kernel reads
// the weights that way itself, and wt_scratch is not written
extern "C" int sc_nn_conv3x3_bwd_data(const float* gout, const uint16_t* w, uint16_t* wt_scratch, float* gin,
                                      int32_t batch, int32_t cin, int32_t cout, int32_t h, int32_t wd, void* stream)
{
    if (!gout || !w || !wt_scratch || !gin || !conv_shape_ok(batch, cin, cout, h, wd) || cin != MAXC)
        return SC_E_INVAL;
    return nn_status(
        launch_rows<kEpiNone, true>(gout, w, nullptr, gin, nullptr, batch, cout, h, wd, (hipStream_t)stream));
}

extern "C" int sc_nn_conv3x3_bwd_data_tanh(const float* gout, const uint16_t* w, uint16_t* wt_scratch, const float* y,
                                           float* gin, int32_t batch, int32_t cin, int32_t cout, int32_t h, int32_t wd,
                                           void* stream)
{
    if (!gout || !w || !wt_scratch || !y || !gin || !conv_shape_ok(batch, cin, cout, h, wd) || cin != MAXC)
        return SC_E_INVAL;
    return nn_status(
        launch_rows<kEpiTanhGrad, true>(gout, w, nullptr, gin, y, batch, cout, h, wd, (hipStream_t)stream));
}

extern "C" int32_t sc_nn_bwd_weight_scratch_floats(int32_t cin, int32_t cout, int32_t nblk)
{
    return nblk * (cin * cout * 9 + cout);
}

extern "C" int sc_nn_conv3x3_bwd_weight(const float* in, const float* gout, float* partial_scratch, int32_t nblk,
                                        float* gw, float* gbias, int32_t batch, int32_t cin, int32_t cout, int32_t h,
                                        int32_t wd, void* stream)
{
    if (!in || !gout || !partial_scratch || !gw || !gbias || nblk < 1 || !conv_shape_ok(batch, cin, cout, h, wd))
        return SC_E_INVAL;
    const int E = cin * cout * 9;
    hipStream_t s = (hipStream_t)stream;
    const int edge = wd % TS == 0 ? kEdgeNone : (wd >= 4 ? kEdgeShift : kEdgeNarrow);
    if (cin == MAXC && cout == MAXC) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, (nblk + kWGroups - 1) / kWGroups, 256 * kWGroups, 0, s, in, gout, partial_scratch,
                               nblk, batch, h, wd);
        };
        if (edge == kEdgeNone) launch(k_conv_bwd_w_bf16<kEdgeNone>);
        else if (edge == kEdgeShift) launch(k_conv_bwd_w_bf16<kEdgeShift>);
        else launch(k_conv_bwd_w_bf16<kEdgeNarrow>);
    } else {
        const int nb = (cout > 16 ? 2 : 1) * (cin > 16 ? 2 : 1);   // waves per partial row
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, (nblk + 4 / nb - 1) / (4 / nb), 256, 0, s, in, gout, partial_scratch, nblk, batch,
                               cin, cout, h, wd);
        };
        auto pick = [&](auto none, auto shift, auto narrow) {
            if (edge == kEdgeNone) launch(none);
            else if (edge == kEdgeShift) launch(shift);
            else launch(narrow);
        };
        if (nb == 4) pick(k_conv_bwd_w<4, kEdgeNone>, k_conv_bwd_w<4, kEdgeShift>, k_conv_bwd_w<4, kEdgeNarrow>);
        else if (nb == 2) pick(k_conv_bwd_w<2, kEdgeNone>, k_conv_bwd_w<2, kEdgeShift>, k_conv_bwd_w<2, kEdgeNarrow>);
        else pick(k_conv_bwd_w<1, kEdgeNone>, k_conv_bwd_w<1, kEdgeShift>, k_conv_bwd_w<1, kEdgeNarrow>);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return nn_status(e);
    hipLaunchKernelGGL(k_sum_partials, (E + cout + kSumCols - 1) / kSumCols, kSumCols * kSumGroups, 0, s,
                       partial_scratch, nblk, cin, cout, gw, gbias);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_tanh_fwd(float* x, int64_t n, void* stream)
{
    if (!x || n < 0) return SC_E_INVAL;
    hipLaunchKernelGGL(k_tanh_fwd, grid_for(n), 256, 0, (hipStream_t)stream, x, n);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_tanh_bwd(const float* y, float* g, int64_t n, void* stream)
{
    if (!y || !g || n < 0) return SC_E_INVAL;
    hipLaunchKernelGGL(k_tanh_bwd, grid_for(n), 256, 0, (hipStream_t)stream, y, g, n);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_mse(const float* out, const float* tgt, float* grad, double* partial_scratch, int32_t nblk,
                         int64_t n, void* stream)
{
    if (!out || !tgt || !partial_scratch || nblk < 1 || n < 1) return SC_E_INVAL;
    hipLaunchKernelGGL(k_mse, nblk, 256, 0, (hipStream_t)stream, out, tgt, grad, n, partial_scratch);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_adam(float* p, const float* g, float* m, float* v, uint16_t* p_bf16, int64_t n, float lr,
                          float beta1, float beta2, float eps, int32_t t, void* stream)
{
    if (!p || !g || !m || !v || n < 0 || t < 1) return SC_E_INVAL;
    const float c1 = 1.f - powf(beta1, (float)t), c2 = 1.f - powf(beta2, (float)t);
    hipLaunchKernelGGL(k_adam, grid_for(n), 256, 0, (hipStream_t)stream, p, g, m, v, p_bf16, n, lr, beta1, beta2,
                       eps, c1, c2);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_to_bf16(const float* x, uint16_t* y, int64_t n, void* stream)
{
    if (!x || !y || n < 0) return SC_E_INVAL;
    hipLaunchKernelGGL(k_to_bf16, grid_for(n), 256, 0, (hipStream_t)stream, x, y, n);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_features(const float* params, float* out, int32_t batch, int32_t h, int32_t wd, float scale_r,
                              void* stream)
{
    if (!params || !out || batch < 1 || h < 1 || wd < 1 || !(scale_r > 0.f)) return SC_E_INVAL;
    hipLaunchKernelGGL(k_features, grid_for((int64_t)batch * h * wd), 256, 0, (hipStream_t)stream, params, out, batch,
                       h, wd, scale_r);
    return nn_status(hipGetLastError());
}

extern "C" int sc_nn_start_field(const float* resid, const double* base, const double* mass, double* out,
                                 int32_t batch, int32_t h, int32_t wd, float inv_scale, double lo, double hi,
                                 void* stream)
{
    if (!resid || !base || !mass || !out || batch < 1 || batch > 65535 || h < 1 || h != wd || !(lo <= hi) ||
        (int64_t)h * wd > ((int64_t)1 << 31))
        return SC_E_INVAL;
    hipLaunchKernelGGL(k_start_field, batch, kStartThreads, 0, (hipStream_t)stream, resid, base, mass, out, h,
                       inv_scale, lo, hi);
    return nn_status(hipGetLastError());
}
