// Blocked convolution on fp16 MFMA with float32 operands held as two fp16
// terms each (gfx950): the kernel for convolutions with enough work to be
// bound by the matrix units.
//
// A float32 value v, scaled by a power of two s, is written as
//   s v = h + 2^-11 l + e,  h = fp16(s v),  l = fp16(2^11 (s v - h)):
// 11 bits, then 11 more of the remainder, whose sign is a twelfth; the
// remainder has at most 12 bits and a sign, so |e| is at most one unit of v's
// last place and zero for three values in four.  A product is h h' + 2^-11
// (h l' + l h'); the dropped l l' lies below 2^-22 of it, with either sign.
// The two sums are kept in float32 accumulators of their own (so l needs no
// further bits of fp16's range) and joined at the end.  Three 32x32x16 fp16
// instructions (96 cycles) replace eight 32x32x2 float32 ones (512 cycles),
// and the sum is rounded once per 16 products instead of once per 2: against
// a float64 reference the result is closer than the float32 kernel's (the
// measured errors stand with the choice of the kernel, conv.hip).
//
// Range.  Filters are scaled per output channel, inputs per workgroup (and
// filters that arrive in float32 per wave): the scale puts the largest
// magnitude -- of the channel, or of the sampled operands: the first chunk of
// the reduction and one in its middle -- at 2^10 .. 2^11.  Values up to 2^5
// times that are exact as above; so are values down to 2^-22 of it, and
// smaller ones keep an absolute error of 2^-46 of it.  A value beyond the
// range (or an infinity or NaN) becomes infinite in h and makes every sum it
// enters non-finite: a wave that finds such a sum computes its tile again on
// float32 MFMA from memory.
//
// Tile.  A workgroup of four waves, WK along the output channels, computes
// 32 WK channels x 32 NP (4 / WK) pixels; a wave 32 channels x 32 NP pixels.
//   - Input: the patch that the tile's windows cover, a chunk of UC channel
//     blocks at a time, is loaded (float4 buffer loads, a zero-padding pixel
//     at an out-of-range offset), converted once and written to LDS; every
//     kernel entry then reads it there at its own pixel offset.  So a 3x3
//     layer loads and converts an input value once per chunk and not nine
//     times, and there is one barrier per chunk.  Two buffers: the next
//     chunk's loads are in flight during this chunk's matrix instructions.
//     LDS holds [term][half of the 16 channels][pixel][8 channels]: lane
//     (i, g) of the instruction's B operand reads the 16 bytes of half g at
//     its pixel.
//   - Filter: straight from memory into the instruction's lane order, no wave
//     reading what another one does; a ring of three or four steps in flight.  Plans
//     keep the filter as converted terms in that order (h2_split_filter), a
//     linear stream of 2 KB per step and 32 channels; a filter in float32
//     KCRS[16]c[16]k is converted as it is used.
// Inputs of at most four channels (network stems) keep four channels per patch
// pixel, and a step is a kernel row and four of its columns: lane (i, g) reads
// columns 2 g and 2 g + 1 of its pixel's window, two neighbouring patch pixels.
// The reduction runs over chunks, then the blocks of a chunk, then the kernel
// entries: the filter's own order.  It may be split over workgroups by
// chunks (partials, then split_reduce).
#pragma once

#include "conv_kernel.h"

namespace neo {
namespace conv_detail {

typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kH2Waves = 4;
// Filter steps in flight: as many as the registers hold.
constexpr int h2_ring(int np) { return np == 4 ? 3 : 4; }

// Channel blocks per chunk of a pointwise layer, by its patch pixels / 64 (up
// to eight float4 per thread in flight).
constexpr int h2_blocks(int ni) { return ni == 4 ? 2 : 4; }

// How a workgroup's pixels and its input patch are laid out.
enum { kH2Point = 0, kH2Rows = 1, kH2Block = 2 };
struct H2Args {
    ConvArgs a;
    const float* w32;  // the float32 filter: KCRS[16]c[16]k, or with a converted filter the kernel order
    const int* wexp;   // per output channel: the exponent of the converted filter's scale
    int w32_bytes;
    // kH2Point: consecutive pixels of a 1x1 layer, the patch is the pixels'
    // own inputs.  kH2Rows: consecutive pixels (n, oh, ow); the patch is the
    // input rows their windows touch, whole, image by image.  kH2Block: a
    // th x tw block of one image's pixels; the patch is its windows' input.
    int kind;
    int ltw, th;        // kH2Block: log2 of the block's width, its height
    int PW;             // patch row length in pixels
    int SF;             // kH2Rows: patch rows of a whole image
    FastDiv div_pw, div_sf;
    FastDiv div_tx, div_tpi;  // kH2Block: blocks per row of blocks, per image
    int chunks;         // chunks of the reduction
};

// The two terms of s v, s2 = 2^11 s.
__device__ inline void h2_terms(const v4f& x, float s, float s2, v4h& h, v4h& l) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        h[j] = (_Float16)__builtin_fmaf(x[j], s, 0.f);
        l[j] = (_Float16)__builtin_fmaf((float)h[j], -2048.f, x[j] * s2);
    }
}
__device__ inline v8h h2_join(const v4h& a, const v4h& b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

__device__ inline float h2_max(const v4f& x, float m) {
#pragma unroll
    for (int j = 0; j < 4; ++j) m = fmaxf(m, fabsf(x[j]));
    return m;
}
__device__ inline float h2_wave_max(float m) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
    return m;
}

// The exponent n of the scale 2^n that takes magnitude m (its float bits) to
// 2^10 .. 2^11; 0 for no magnitude, an infinity or NaN.
__device__ inline int h2_exponent(unsigned m) {
    const int e = (int)(m >> 23);
    if (m == 0 || e == 255) return 0;
    return min(137 - e, 110);
}

// The geometry of one workgroup's tile: where its pixels and patch pixels lie.
struct H2Tile {
    int m0;        // kH2Point, kH2Rows: the first pixel
    int n0, oh0, ow0;
    int S0;        // kH2Rows: patch rows of the first image
    int rows;      // patch rows in use
    // P: pixels of the tile
    __device__ void set(const H2Args& h, int pxt, int P) {
        const ConvArgs& a = h.a;
        const int ohw = a.OH * a.OW;
        if (h.kind == kH2Block) {
            n0 = fdiv(pxt, h.div_tpi);
            const int rem = pxt - n0 * h.div_tpi.d;
            const int ty = fdiv(rem, h.div_tx);
            oh0 = ty * h.th;
            ow0 = (rem - ty * h.div_tx.d) << h.ltw;
            m0 = 0;
            S0 = 0;
            rows = (h.th - 1) * a.sh + a.R;
        } else {
            m0 = pxt * P;
            n0 = fdiv(m0, a.div_ohw);
            oh0 = fdiv(m0 - n0 * ohw, a.div_ow);
            ow0 = 0;
            S0 = (a.OH - 1 - oh0) * a.sh + a.R;
            const int last = min(m0 + P, a.M) - 1;
            const int n1 = fdiv(last, a.div_ohw);
            rows = patch_row(h, n1, fdiv(last - n1 * ohw, a.div_ow)) + a.R;
        }
    }
    // first patch row of the windows of output row oh of image n (kH2Rows)
    __device__ int patch_row(const H2Args& h, int n, int oh) const {
        return n == n0 ? (oh - oh0) * h.a.sh : S0 + (n - n0 - 1) * h.SF + oh * h.a.sh;
    }
    // pixel p of the tile: image, position in the output map (-1: none) and
    // the patch pixel of its window's first entry
    __device__ void pixel(const H2Args& h, int p, int& n, int& pix, int& base) const {
        const ConvArgs& a = h.a;
        if (h.kind == kH2Block) {
            const int dy = p >> h.ltw, dx = p & ((1 << h.ltw) - 1);
            const int oh = oh0 + dy, ow = ow0 + dx;
            n = n0;
            pix = oh < a.OH && ow < a.OW ? oh * a.OW + ow : -1;
            base = dy * a.sh * h.PW + dx * a.sw;
            return;
        }
        const bool ok = m0 + p < a.M;
        const int m = ok ? m0 + p : m0;
        n = fdiv(m, a.div_ohw);
        const int rem = m - n * (a.OH * a.OW);
        pix = ok ? rem : -1;
        if (h.kind == kH2Point) {
            base = p;
        } else {
            const int oh = fdiv(rem, a.div_ow);
            base = patch_row(h, n, oh) * h.PW + (rem - oh * a.OW) * a.sw;
        }
    }
    // byte offset in the input (channel group 0, quad 0) of patch pixel j, or out of range
    template <bool XY>
    __device__ unsigned input(const H2Args& h, int j) const {
        const ConvArgs& a = h.a;
        int n, ih, iw;
        bool ok;
        if (h.kind == kH2Point) {
            const int m = m0 + j;
            ok = m < a.M;
            n = fdiv(ok ? m : 0, a.div_ohw);
            const int rem = (ok ? m : 0) - n * (a.OH * a.OW);
            const int oh = fdiv(rem, a.div_ow);
            ih = oh * a.sh - a.ph;
            iw = (rem - oh * a.OW) * a.sw - a.pw;
        } else {
            const int row = fdiv(j, h.div_pw), col = j - row * h.PW;
            ok = row < rows;
            iw = ow0 * a.sw - a.pw + col;
            if (h.kind == kH2Block || row < S0) {
                n = n0;
                ih = oh0 * a.sh - a.ph + row;
            } else {
                const int t = fdiv(row - S0, h.div_sf);
                n = n0 + 1 + t;
                ih = row - S0 - t * h.SF - a.ph;
            }
        }
        ok = ok && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
        return ok ? (unsigned)(((n * xblocks<XY>(a) * a.H + ih) * a.W + iw) * xpb_of<XY>(a)) : kOutOfRange;
    }
};

// Small-channel path: channels 0..3 of the pixel at byte offset off.
template <bool XY>
__device__ inline v4f h2_small_x(const ConvArgs& a, __amdgpu_buffer_rsrc_t xr, unsigned off) {
    if constexpr (XY) {
        if (a.xb == 1) {  // NCHW: the channels lie a plane apart; the rest are 0
            const int plane = __builtin_amdgcn_readfirstlane(a.H * a.W * 4);
            v4f v;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = t < a.XB ? ld1(xr, off, t * plane, 0) : 0.f;
            return v;
        }
    }
    return ld4(xr, off, 0, 0);
}

// The tile of one wave again in float32: chunk blocks [c_lo, c_hi) of the
// reduction, operands straight from memory (eight elements of a unit per
// lane, v_mfma_f32_32x32x2f32).
template <int NP, bool PRE, bool XY, bool SMALL>
__device__ inline void h2_again(const H2Args& h, const H2Tile& t, int kb, int p0, int c_lo, int c_hi, int lane,
                                v16f (&acc)[NP]) {
    const ConvArgs& a = h.a;
    const int i = lane & 31, g = lane >> 5;
    const __amdgpu_buffer_rsrc_t xr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), (short)0, a.x_bytes, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t wr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(h.w32), (short)0, h.w32_bytes, kRsrcWord3);
    int n[NP], ih0[NP], iw0[NP];
    bool in[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        int pix, base;
        t.pixel(h, p0 + p * 32 + i, n[p], pix, base);
        in[p] = pix >= 0;
        const int q = in[p] ? pix : 0, oh = fdiv(q, a.div_ow);
        ih0[p] = oh * a.sh - a.ph;
        iw0[p] = (q - oh * a.OW) * a.sw - a.pw;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[p][v] = 0.f;
    }
    const int k16 = 2 * kb + (i >> 4), li = i & 15;
    const bool kok = k16 < a.KB;
#pragma unroll 1
    for (int cb = c_lo; cb < c_hi; ++cb)
#pragma unroll 1
        for (int r = 0; r < a.R; ++r)
#pragma unroll 1
            for (int s = 0; s < (SMALL ? a.U : a.S); ++s) {
                v4f wv[2], xv[NP][2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int sc = SMALL ? 4 * s + 2 * g + e : s;  // kernel column
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        const int ih = ih0[p] + r, iw = iw0[p] + sc;
                        const bool ok =
                            in[p] && sc < a.S && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
                        const int at = ((n[p] * xblocks<XY>(a) * a.H + ih) * a.W + iw) * xpb_of<XY>(a);
                        if constexpr (SMALL)
                            xv[p][e] = h2_small_x<XY>(a, xr, ok ? (unsigned)at : kOutOfRange);
                        else
                            xv[p][e] = ld4(xr, ok ? (unsigned)(at + (XY ? xgroup(a, cb) : cb * a.H * a.W * 64) + 32 * g + 16 * e)
                                                  : kOutOfRange, 0, 0);
                    }
                    const int block = SMALL && PRE ? ((k16 * a.R + r) * a.U + s) * 1024
                                                   : ((k16 * a.CB + cb) * a.RS + r * a.S + sc) * 1024;
                    if constexpr (PRE) {
                        wv[e] = ld4(wr, kok ? (unsigned)(block + ((2 * g + e) * 16 + li) * 16) : kOutOfRange, 0, 0);
                    } else if constexpr (SMALL) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            wv[e][q] = ld1(wr, kok && sc < a.S ? (unsigned)(block + (q * 16 + li) * 4) : kOutOfRange, 0, 0);
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            wv[e][q] = ld1(wr, kok ? (unsigned)(block + ((8 * g + 4 * e + q) * 16 + li) * 4)
                                                   : kOutOfRange, 0, 0);
                    }
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        acc[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[q / 4][q % 4], xv[p][q / 4][q % 4], acc[p], 0, 0, 0);
            }
}

// NI: patch pixels per 64 (the patch has at most 64 NI pixels), per 256 on the
// small-channel path.
template <int NP, int WK, int NI, int UC, bool PRE, bool XY, bool SMALL>
__global__ __launch_bounds__(64 * kH2Waves, 2) void conv2d_h2(H2Args h) {
    constexpr int WP = kH2Waves / WK, kRing = h2_ring(NP);
    // v8h (small-channel path: v4h) of a plane; the 4 keep the halves' 8-byte
    // writes in different banks
    constexpr int kPlane = (SMALL ? 256 : 64) * NI + 4;
    __shared__ v8h xl[SMALL ? 1 : 2][SMALL ? 1 : UC][2][SMALL ? 1 : 2][SMALL ? kPlane / 2 : kPlane];
    __shared__ unsigned top[kH2Waves];
    // for the epilogue: image and position of the tile's pixels, its channels'
    // bias and scale exponents (loaded now: at the end each load would wait
    // for a full round trip to memory)
    __shared__ int where[2][NP * WP * 32];
    __shared__ __align__(16) float lbias[WK * 32];
    __shared__ int lexp[WK * 32];
    // the threads' patch offsets, read again for every chunk where the registers are full
    constexpr bool kOffLds = NP == 4 && !SMALL;
    __shared__ unsigned loff[kOffLds ? NI : 1][kOffLds ? 64 * kH2Waves : 1];
    const ConvArgs& a = h.a;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave % WK, wp = wave / WK;
    const int u = xcd_order();
    const int npx = a.div_npx.d, nkb = a.div_nkb.d;
    int pxt, kbt, z;
    if (a.kfirst) {
        const int t = fdiv(u, a.div_nkb);
        kbt = u - t * nkb;
        z = fdiv(t, a.div_npx);
        pxt = t - z * npx;
    } else {
        const int t = fdiv(u, a.div_npx);
        pxt = u - t * npx;
        z = fdiv(t, a.div_nkb);
        kbt = t - z * nkb;
    }
    H2Tile tile;
    tile.set(h, pxt, 32 * NP * WP);
    const int kb = kbt * WK + wk, p0 = wp * NP * 32;
    // this split's channel blocks
    const int c_lo = __builtin_amdgcn_readfirstlane(UC * (int)(((long)h.chunks * z) / a.split));
    const int c_hi = __builtin_amdgcn_readfirstlane(min(a.CB, UC * (int)(((long)h.chunks * (z + 1)) / a.split)));

    const __amdgpu_buffer_rsrc_t xr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), (short)0, a.x_bytes, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t wr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.w), (short)0, a.w_bytes, kRsrcWord3);

    float my_bias = 0.f;
    int my_exp = 0;
    {
        const int k = kbt * WK * 32 + threadIdx.x;
        const bool mine = threadIdx.x < WK * 32 && k < a.KB * 16;
        if (mine && a.bias && a.split == 1) my_bias = a.bias[k];
        if constexpr (PRE) {
            if (mine) my_exp = h.wexp[k];
        }
    }

    // ---- input: thread t loads quad t % 4 of patch pixels t / 4 + 64 j (the
    // small-channel path: pixels t + 256 j)
    const int xq = threadIdx.x & 3, xp = SMALL ? threadIdx.x : threadIdx.x >> 2;
    unsigned xoff[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) xoff[j] = tile.input<XY>(h, xp + (SMALL ? 256 : 64) * j) + (SMALL ? 0 : 16 * xq);
    if constexpr (kOffLds) {
#pragma unroll
        for (int j = 0; j < NI; ++j) loff[j][threadIdx.x] = xoff[j];
    }
    const int dx = __builtin_amdgcn_readfirstlane(a.H * a.W * 64);
    auto load_x = [&](v4f (&v)[UC][NI], int cb0) __attribute__((always_inline)) {
        unsigned o[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            if constexpr (kOffLds)
                o[j] = loff[j][threadIdx.x];
            else
                o[j] = xoff[j];
        }
#pragma unroll
        for (int c = 0; c < UC; ++c) {
            // (a block past the split's last is never multiplied)
            const int cb = min(cb0 + c, c_hi - 1);
            const int so = __builtin_amdgcn_readfirstlane(XY ? xgroup(a, cb) : cb * dx);
#pragma unroll
            for (int j = 0; j < NI; ++j) v[c][j] = SMALL ? h2_small_x<XY>(a, xr, o[j]) : ld4(xr, o[j], so, 0);
        }
    };
    auto max_x = [&](const v4f (&v)[UC][NI], float m) {
#pragma unroll
        for (int c = 0; c < UC; ++c)
#pragma unroll
            for (int j = 0; j < NI; ++j) m = h2_max(v[c][j], m);
        return m;
    };

    // ---- filter: a step is one channel block at one kernel entry, in its
    // own order (small-channel path: four columns of a kernel row)
    const int per_block = SMALL ? a.R * a.U : a.RS;
    const int f_lo = __builtin_amdgcn_readfirstlane(c_lo * per_block);
    const int f_hi = __builtin_amdgcn_readfirstlane(c_hi * per_block);
    const int li = lane & 15, k16 = 2 * kb + ((lane >> 4) & 1);
    const unsigned woff = PRE ? (2 * kb < a.KB ? (unsigned)(kb * a.CB * per_block * 2048 + lane * 16) : kOutOfRange)
                              : (k16 < a.KB ? (unsigned)(k16 * a.CB * a.RS * 1024 + li * 4 +
                                                         (SMALL ? (lane >> 5) * 2048 : (lane >> 5) * 512))
                                            : kOutOfRange);
    constexpr int kStep = PRE ? 2048 : 1024;
    const int w_end = __builtin_amdgcn_readfirstlane((f_hi - 1) * kStep);
    int w_at = __builtin_amdgcn_readfirstlane(f_lo * kStep);  // the next step's block (stays at the last one)
    int w_r = 0, w_u = 0;  // small-channel float32 filter: the next step's row and column group
    auto load_w = [&](v4f (&v)[2], int so) __attribute__((always_inline)) {
        if constexpr (PRE) {
            v[0] = ld4(wr, woff, so, 0);
            v[1] = ld4(wr, woff, so, 1024);
        } else if constexpr (SMALL) {
            // channels 0..3 of columns 4 u + 2 g + e: blocks of their own
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const bool ok = 4 * w_u + 2 * (lane >> 5) + e < a.S;
#pragma unroll
                for (int t = 0; t < 4; ++t) v[e][t] = ld1(wr, ok ? woff : kOutOfRange, so, e * 1024 + t * 64);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t / 4][t % 4] = ld1(wr, woff, so, t * 64);
        }
    };
    auto next_w = [&](v4f (&v)[2]) __attribute__((always_inline)) {
        if constexpr (SMALL && !PRE) {
            load_w(v, __builtin_amdgcn_readfirstlane((w_r * a.S + 4 * w_u) * 1024));
            const bool row = w_u + 1 == a.U, last = row && w_r + 1 == a.R;
            w_u = __builtin_amdgcn_readfirstlane(last ? w_u : row ? 0 : w_u + 1);
            w_r = __builtin_amdgcn_readfirstlane(row && !last ? w_r + 1 : w_r);
        } else {
            load_w(v, w_at);
            w_at = __builtin_amdgcn_readfirstlane(min(w_at + kStep, w_end));
        }
    };

    v4f wv[kRing][2], xv[UC][NI];
    // ---- scales
    int ew = 0, ex;
    {
        v4f mid = v4f{0.f, 0.f, 0.f, 0.f}, wmid[2] = {mid, mid};
        if constexpr (!SMALL) {
            const int cm = (c_lo + c_hi) / 2;
            mid = ld4(xr, xoff[NI / 2], __builtin_amdgcn_readfirstlane(XY ? xgroup(a, cm) : cm * dx), 0);
            if constexpr (!PRE) load_w(wmid, __builtin_amdgcn_readfirstlane((f_lo + f_hi) / 2 * kStep));
        }
        load_x(xv, c_lo);
#pragma unroll
        for (int d = 0; d < kRing; ++d) next_w(wv[d]);
        const float mx = h2_wave_max(max_x(xv, h2_max(mid, 0.f)));
        if (lane == 0) top[wave] = __float_as_uint(mx);
        if constexpr (!PRE) {
            float mw = h2_max(wmid[0], h2_max(wmid[1], 0.f));
#pragma unroll
            for (int d = 0; d < kRing; ++d) mw = h2_max(wv[d][0], h2_max(wv[d][1], mw));
            ew = __builtin_amdgcn_readfirstlane(h2_exponent(__float_as_uint(h2_wave_max(mw))));
        }
        __syncthreads();
        unsigned t = 0;
#pragma unroll
        for (int w = 0; w < kH2Waves; ++w) t = max(t, top[w]);
        ex = __builtin_amdgcn_readfirstlane(h2_exponent(t));
    }
    const float sclx = ldexpf(1.f, ex), sclx2 = sclx * 2048.f;
    const float sclw = ldexpf(1.f, ew), sclw2 = sclw * 2048.f;
    auto stage_one = [&](int buf, int c, int j) __attribute__((always_inline)) {
        v4h t[2];
        h2_terms(xv[c][j], sclx, sclx2, t[0], t[1]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if constexpr (SMALL)
                reinterpret_cast<v4h*>(&xl[0][0][e][0][0])[xp + 256 * j] = t[e];
            else
                reinterpret_cast<v4h*>(&xl[buf][c][e][xq >> 1][xp + 64 * j])[xq & 1] = t[e];
        }
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < UC; ++c)
#pragma unroll
            for (int j = 0; j < NI; ++j) stage_one(buf, c, j);
    };

    v16f acc[NP], accl[NP];
    // the lane's 16 bytes at its pixel's first window entry: v8h index from a
    // term's plane (small-channel path: v4h index of columns 2 g, 2 g + 1)
    int at[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int q = p0 + p * 32 + (lane & 31);
        int n, pix, base;
        tile.pixel(h, q, n, pix, base);
        where[0][q] = n;
        where[1][q] = pix;
        at[p] = (lane >> 5) * (SMALL ? 2 : kPlane) + (pix >= 0 ? base : 0);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[p][v] = 0.f;
            accl[p][v] = 0.f;
        }
    }

    v8h xh[NP], xlo[NP];
    if (threadIdx.x < WK * 32) {
        lbias[threadIdx.x] = my_bias;
        lexp[threadIdx.x] = my_exp;
    }
    const v8h* const x0 = &xl[0][0][0][0][0];
    constexpr int kBlock = 4 * kPlane, kBuffer = UC * kBlock;
    auto read = [&](int i, int e) __attribute__((always_inline)) {  // term e at index i
        if constexpr (SMALL) {
            const v4h* q = reinterpret_cast<const v4h*>(x0) + i + e * kPlane;
            return h2_join(q[0], q[1]);
        } else {
            return x0[i + e * 2 * kPlane];
        }
    };
    stage(0);
    if constexpr (!SMALL) load_x(xv, c_lo + UC);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        xh[p] = read(at[p], 0);
        xlo[p] = read(at[p], 1);
    }
    // off: the step's input from the lane's first (a chunk of one block walks
    // the kernel entries, a pointwise chunk its blocks); left: steps of the
    // chunk from this one on, at least two in a whole chunk
    const int per_chunk = UC > 1 ? UC : __builtin_amdgcn_readfirstlane(per_block);
    const int columns = SMALL ? a.U : a.S;  // steps of a kernel row
    constexpr int kColumn = SMALL ? 4 : 1;
    const int row_skip = __builtin_amdgcn_readfirstlane(h.PW - kColumn * columns);
    int buf = 0, off = 0, s = columns, left = per_chunk, cb = c_lo;
    auto advance = [&]() __attribute__((always_inline)) {
        if constexpr (UC > 1) {
            off += kBlock;
        } else {
            const bool row = --s == 0;
            off += row ? row_skip + kColumn : kColumn;
            s = row ? columns : s;
        }
        const bool end = --left == 0;  // (s is `columns` again)
        if constexpr (!SMALL) {
            buf ^= end ? 1 : 0;
            cb += end ? UC : 0;
        }
        off = end ? (buf ? kBuffer : 0) : off;
        left = end ? per_chunk : left;
    };
    // A step's 3 NP matrix instructions run back to back only if nothing that
    // they read is still on its way, so everything else stands between them, in
    // their shadow, held there by scheduling fences (left alone the scheduler
    // puts the LDS reads right before their use, and a wait in front of every
    // second instruction):
    //   - an operand of the next step's input is read from LDS as soon as this
    //     step's instructions have taken the last from its registers;
    //   - a float32 filter's next step is converted, a pair of elements a time.
    // A chunk's last step but one ends with the next chunk's input converted and
    // written to the other buffer, and the barrier; the last step then reads
    // ahead into the new chunk.  (Every wave's last reads of the other buffer
    // lie before the barrier one chunk earlier.)
    // Before and after: 256 -> 256 3x3 at 56x56 batch 8 118 -> 107 us (277
    // TFLOP/s), 64 -> 64 at 56x56 batch 32 39.0 -> 35.4 us, ResNet-50 batch 32
    // 1.76 -> 1.67 ms (1.79 -> 1.72 on another card); a float32 filter with one
    // or two workgroups on a CU (128 -> 128 at 28x28 batch 32) 38.3 -> 39.4 us.
    // The next chunk's conversions in a branch of each slot, between the
    // instructions, took 42.4 us there: a branch costs more than the shadow holds.
    v8h w[2];  // the step's filter terms
    auto convert_w = [&](const v4f (&v)[2], v8h (&o)[2], int pair) __attribute__((always_inline)) {
        if constexpr (!PRE) {
#pragma unroll
            for (int e = 2 * pair; e < 2 * pair + 2; ++e) {
                const float f = v[e / 4][e % 4];
                o[0][e] = (_Float16)__builtin_fmaf(f, sclw, 0.f);
                o[1][e] = (_Float16)__builtin_fmaf((float)o[0][e], -2048.f, f * sclw2);
            }
        }
    };
    auto step = [&](v4f (&wd)[2], const v4f (&wnext)[2]) __attribute__((always_inline)) {
        const bool stage_next = !SMALL && left == 2 && cb + UC < c_hi;
        if constexpr (PRE) {
            w[0] = __builtin_bit_cast(v8h, wd[0]);
            w[1] = __builtin_bit_cast(v8h, wd[1]);
        }
        v8h wn[2];
        const int other = buf ^ 1;
        advance();
        __builtin_amdgcn_sched_barrier(0);
        auto between = [&](int slot) __attribute__((always_inline)) {  // of 2 NP
            if (slot < 4) convert_w(wnext, wn, slot);
        };
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[0], xh[p], acc[p], 0, 0, 0);
            accl[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[1], xh[p], accl[p], 0, 0, 0);
            xh[p] = read(at[p] + off, 0);
            between(p);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            accl[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[0], xlo[p], accl[p], 0, 0, 0);
            xlo[p] = read(at[p] + off, 1);
            between(NP + p);
            __builtin_amdgcn_sched_barrier(0);
        }
        next_w(wd);
        if constexpr (!PRE) {
            w[0] = wn[0];
            w[1] = wn[1];
        }
        if (stage_next) {
            stage(other);
            load_x(xv, cb + 2 * UC);
            __syncthreads();
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (!PRE) {
#pragma unroll
        for (int q = 0; q < 4; ++q) convert_w(wv[0], w, q);
    }
    // (whole turns of the ring, then what remains: with an exit inside the turn
    // the waits for loads at the loop's head would count the ways that skip later loads)
    int f = f_lo;
    for (; f + kRing <= f_hi; f += kRing) {
#pragma unroll
        for (int d = 0; d < kRing; ++d) step(wv[d], wv[(d + 1) % kRing]);
    }
#pragma unroll
    for (int d = 0; d + 1 < kRing; ++d) {
        if (f + d >= f_hi) break;
        step(wv[d], wv[d + 1]);
    }

    // join the sums; a non-finite one means a value out of range
    float bad = 0.f;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[p][v] = __builtin_fmaf(accl[p][v], 1.f / 2048.f, acc[p][v]);
            bad = __builtin_fmaf(acc[p][v], 0.f, bad);
        }
    const bool again = __any(bad != bad);
    if (again) h2_again<NP, PRE, XY, SMALL>(h, tile, kb, p0, c_lo, c_hi, lane, acc);
    // Accumulator element 4 j + v of lane (i, g): channel 8 j + 4 g + v of the
    // block, pixel i.  Every operand of the epilogue is loaded before the first
    // store: a load after a store waits for its own round trip.
    const int k0 = kb * 32 + 4 * (lane >> 5);
    int n[NP], pix[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        n[p] = where[0][p0 + p * 32 + (lane & 31)];
        pix[p] = where[1][p0 + p * 32 + (lane & 31)];
    }
    // (channels past the last block read another's operands and store zeros or nothing)
    const int k_end = a.KB * 16;
    const bool whole = a.split == 1, res_on = whole && a.res;
    v4f bias[4], res[NP][4];
    int ex4[4][4];
    if (res_on) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = k0 + 8 * j < k_end ? k0 + 8 * j : 0;
                res[p][j] = *reinterpret_cast<const v4f*>(
                    a.res + yindex<XY>(a, n[p], rblocks<XY>(a), k, pix[p] >= 0 ? pix[p] : 0));
            }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int q = wk * 32 + 4 * (lane >> 5) + 8 * j;
        bias[j] = *reinterpret_cast<const v4f*>(&lbias[q]);
#pragma unroll
        for (int v = 0; v < 4; ++v) ex4[j][v] = again ? 0 : -ex - (PRE ? lexp[q + v] : ew);
    }
    const int ohw = a.OH * a.OW;
    const bool relu = a.act == NEO_ACT_RELU;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (pix[p] < 0) continue;
        float* part = a.ws + (long)z * a.N * a.KB * ohw * 16 + ((n[p] * a.KB + (k0 >> 4)) * ohw + pix[p]) * 16 + (k0 & 15);
        float* y0 = a.y + yindex<XY>(a, n[p], a.y_tot, a.y_off * (XY ? a.yb : 16) + k0, pix[p]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + 8 * j;
            v4f o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = __builtin_amdgcn_ldexpf(acc[p][4 * j + v], ex4[j][v]);
            if (!whole) {  // the raw partial sum of split z
                if (k < k_end) *reinterpret_cast<v4f*>(part + (j >> 1) * ohw * 16 + (j & 1) * 8) = o;
                continue;
            }
            if (a.bias) o += bias[j];
            if (res_on) o += res[p][j];
            if (relu) {
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = o[v] > 0.f ? o[v] : 0.f;
            }
            if constexpr (XY) {
                // (groups past the last real one are the last block's zero padding)
                if (k >= k_end) o = v4f{0.f, 0.f, 0.f, 0.f};
                if (k < kgroups<XY>(a) * 16)
                    *reinterpret_cast<v4f*>(a.y + yindex<XY>(a, n[p], a.y_tot, a.y_off * a.yb + k, pix[p])) = o;
            } else {
                if (k < k_end) *reinterpret_cast<v4f*>(y0 + (j >> 1) * ohw * 16 + (j & 1) * 8) = o;
            }
        }
    }
}

template <int NP, int WK, int NI, int UC, bool PRE, bool XY, bool SMALL = false>
hipError_t launch_h2_t(const H2Args& h, hipStream_t st) {
    const ConvArgs& a = h.a;
    const int wgs = a.div_npx.d * a.div_nkb.d * a.split;
    hipLaunchKernelGGL((conv2d_h2<NP, WK, NI, UC, PRE, XY, SMALL>), dim3(wgs), dim3(64 * kH2Waves), 0, st, h);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.split == 1) return e;
    const long total = (long)a.N * a.KBk * a.OH * a.OW * 4;
    const long blocks = std::min<long>(65536, (total + 255) / 256);
    hipLaunchKernelGGL(split_reduce<XY>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ni: patch pixels / 64 (a pointwise layer's are its tile's), / 256 on the
// small-channel path.
template <int NP, int WK, bool PRE, bool XY>
hipError_t dispatch_h2_patch(int ni, bool small, const H2Args& h, hipStream_t st) {
    if (small) {
        switch (ni) {
            case 2: return launch_h2_t<NP, WK, 2, 1, PRE, XY, true>(h, st);
            case 4: return launch_h2_t<NP, WK, 4, 1, PRE, XY, true>(h, st);
            case 6: return launch_h2_t<NP, WK, 6, 1, PRE, XY, true>(h, st);
            default: return hipErrorInvalidValue;
        }
    }
    constexpr int kOwn = NP * (kH2Waves / WK) / 2;
    if (h.kind == kH2Point) return launch_h2_t<NP, WK, kOwn, h2_blocks(kOwn), PRE, XY>(h, st);
    switch (ni) {
        case 2: return launch_h2_t<NP, WK, 2, 1, PRE, XY>(h, st);
        case 3: return launch_h2_t<NP, WK, 3, 1, PRE, XY>(h, st);
        case 5: return launch_h2_t<NP, WK, 5, 1, PRE, XY>(h, st);
        case 8: return launch_h2_t<NP, WK, 8, 1, PRE, XY>(h, st);
        default: return hipErrorInvalidValue;
    }
}

// Instantiated in conv_h2.hip (PRE) and conv_h2_raw.hip (a filter in KCRS[16]c[16]k).
template <bool PRE, bool XY>
hipError_t dispatch_h2(const ConvConfig& c, int ni, bool small, const H2Args& h, hipStream_t st) {
    switch (c.fk * 8 + c.fp) {
        case 2 * 8 + 2: return dispatch_h2_patch<2, 2, PRE, XY>(ni, small, h, st);
        case 2 * 8 + 4: return dispatch_h2_patch<4, 2, PRE, XY>(ni, small, h, st);
        case 4 * 8 + 2: return dispatch_h2_patch<2, 4, PRE, XY>(ni, small, h, st);
        case 4 * 8 + 4: return dispatch_h2_patch<4, 4, PRE, XY>(ni, small, h, st);
        default: return hipErrorInvalidValue;
    }
}

// Defined in conv_h2.hip.  A filter in kernel order as converted terms: for every 32 output channels,
// channel block and kernel entry 2 KB, term h then l, lane (i, g) the eight
// elements 8 g .. 8 g + 7 of channel i; then the channels' exponents.  One
// workgroup per output channel (of whole 32-channel blocks; the ones past K
// are zero).
hipError_t launch_h2_split(const float* w, int KB, int steps, void* out, int* wexp, hipStream_t st);

}  // namespace conv_detail
}  // namespace neo
