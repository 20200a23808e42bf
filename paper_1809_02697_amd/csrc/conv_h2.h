// Blocked convolution on fp16 MFMA with float32 operands held as two fp16
// terms each (gfx950): the kernel for convolutions with enough work to be
// bound by the matrix units.
//
// A float32 value v, scaled by a power of two s, is written as
//   s v = h + 2^-11 l + e,  h = fp16(s v),  l = fp16(2^11 (s v - h)):
// 11 bits, then 11 more of the remainder, whose sign is a twelfth; the
// remainder has at most 12 bits and a sign, so |e| is at most one unit of v's
// last place and zero for three values in four.  (Single precision from fp16
// products of two terms, the second scaled by 2^11: Markidis et al. 2018;
// Ootomo and Yokota 2022.)  A product is h h' + 2^-11 (h l' + l h'); the
// dropped l l' lies below 2^-22 of it, with either sign.
// The two sums are kept in float32 accumulators of their own (so l needs no
// further bits of fp16's range) and joined at the end.  Three 32x32x16 fp16
// instructions (96 cycles) replace eight 32x32x2 float32 ones (512 cycles),
// and the sum is rounded once per 16 products instead of once per 2: against
// a float64 reference the result is closer than the float32 kernel's from 24
// products on; shorter reductions keep that kernel (the measured errors stand
// at h2_long_enough, conv.hip).
//
// Range.  Filters are scaled per output channel, inputs per workgroup.  The
// scale puts the largest magnitude of a converted channel at 2^14 .. 2^15; of
// the input, and of a float32 filter's channels, it puts the largest of a
// sample at 2^10 .. 2^11: the input's first chunk and a float4 per thread in
// the middle of the reduction, the filter's first steps and its middle one.
//   - A value beyond the range (or an infinity or NaN) becomes infinite in h
//     and makes every sum it enters non-finite.
//   - A small value, below 2^-12 once scaled, keeps an error of up to 2^-36, which
//     is no longer a part of itself.  Small values are counted as they are
//     converted; at the end of the reduction the count bounds the error that
//     they can have left in a sum.
// A wave that finds a sum of its tile not finite, or not 2^20 times above that
// bound, computes the tile again on float32 MFMA from memory.  So every sum
// has a float32 sum's error for its own terms, whatever lies beside them.
// In a map of ordinary values a tile in fifty meets a small value, and one in
// millions of its sums lies as low as what a few of them leave.
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

typedef float v2f __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
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
    const int* wexp;   // per output channel of the converted filter: h2_channel()
    int w32_bytes;
    int K;             // output channels (without the last block's padding)
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

// The two terms of a pair of values scaled by s, s2 = 2^11 s: six instructions.
// (The empty statements keep the pair in one register: without them the
// compiler converts a value twice, or takes an instruction more for the second term.)
__device__ inline void h2_pair(float x0, float x1, float s2, v2h& h, v2h& l) {
    const float u0 = x0 * s2, u1 = x1 * s2;
    h = v2h{(_Float16)__builtin_fmaf(u0, 1.f / 2048.f, 0.f), (_Float16)__builtin_fmaf(u1, 1.f / 2048.f, 0.f)};
    asm("" : "+v"(h));
    _Float16 l0 = (_Float16)__builtin_fmaf((float)h[0], -2048.f, u0);
    asm("" : "+v"(l0));
    l = v2h{l0, (_Float16)__builtin_fmaf((float)h[1], -2048.f, u1)};
}
__device__ inline void h2_terms(const v4f& x, float s2, v4h& h, v4h& l) {
    v2h a[2], b[2];
    h2_pair(x[0], x[1], s2, a[0], b[0]);
    h2_pair(x[2], x[3], s2, a[1], b[1]);
    h = __builtin_shufflevector(a[0], a[1], 0, 1, 2, 3);
    l = __builtin_shufflevector(b[0], b[1], 0, 1, 2, 3);
}
__device__ inline v8h h2_join(const v4h& a, const v4h& b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

__device__ inline float h2_max(const v4f& x, float m) {
#pragma unroll
    for (int j = 0; j < 4; ++j) m = fmaxf(m, fabsf(x[j]));
    return m;
}
// min(m, |a|, |b|) in one instruction (fminf makes its operands canonical first).
__device__ inline float h2_min3(float m, float a, float b) {
    asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
    return m;
}
__device__ inline float h2_wave_max(float m) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
    return m;
}

// The magnitudes that the scales take the largest one to, 2^top .. 2^(top + 1):
// the largest of a sample (with room above), of a whole filter channel.
constexpr int kH2TopSample = 10, kH2TopAll = 14;

// The exponent n of the scale 2^n that takes magnitude m (its float bits) there;
// 0 for no magnitude, an infinity or NaN.
__device__ inline int h2_exponent(unsigned m, int top) {
    const int e = (int)(m >> 23);
    if (m == 0 || e == 255) return 0;
    return min(127 + top - e, 110);
}

// v is a small value if h2_key(v) < h2_key(h2_small(n)), n the exponent of its
// scale (a zero's key is the largest).
__device__ inline unsigned h2_key(float v) { return (__float_as_uint(v) << 1) - 1u; }
__device__ inline float h2_small(int n) { return ldexpf(1.f, -12 - n); }

// min(m, the values' keys), two keys an instruction.  The carry between the two
// moves the second by at most one, and a zero beside a negative value reads 0:
// the minimum lies below a limit wherever a small value does, and at times
// where none does (who counts them looks at the keys themselves).
__device__ inline unsigned h2_low(const v4f& x, unsigned m) {
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
        const v2f p = {x[j], x[j + 1]};
        const v2u k = __builtin_bit_cast(v2u, (__builtin_bit_cast(unsigned long, p) << 1) + 0xfffffffeffffffffUL);
        m = min(min(m, k[0]), k[1]);
    }
    return m;
}

// A filter channel's scale exponent and its number of small values (at most 65535).
__device__ inline int h2_channel(int exponent, int small) { return exponent * 65536 + min(small, 65535); }
__device__ inline int h2_channel_exponent(int c) { return c >> 16; }
__device__ inline int h2_channel_small(int c) { return c & 65535; }

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
// Workgroups per CU that the registers are kept for: three for two pixel blocks
// a wave and a small patch.
constexpr int h2_resident(int np, int items, bool pre, bool small) {
    return np == 2 && (small || items <= (pre ? 5 : 3)) ? 3 : 2;
}

template <int NP, int WK, int NI, int UC, bool PRE, bool XY, bool SMALL>
__global__ __launch_bounds__(64 * kH2Waves, h2_resident(NP, UC * NI, PRE, SMALL)) void conv2d_h2(H2Args h) {
    constexpr int WP = kH2Waves / WK, kRing = h2_ring(NP);
    // v8h (small-channel path: v4h) of a plane; the 4 keep the halves' 8-byte
    // writes in different banks
    constexpr int kPlane = (SMALL ? 256 : 64) * NI + 4;
    __shared__ v8h xl[SMALL ? 1 : 2][SMALL ? 1 : UC][2][SMALL ? 1 : 2][SMALL ? kPlane / 2 : kPlane];
    __shared__ unsigned top[kH2Waves], small[kH2Waves];
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
    // ---- scales: the input's exponent, and a float32 filter's of the lane's channel
    int ew = 0, ex;
    {
        v4f mid = v4f{0.f, 0.f, 0.f, 0.f}, wmid[2] = {mid, mid};
        if constexpr (!SMALL) {
            // (pixels that any but a short last tile has)
            const int cm = (c_lo + c_hi) / 2;
            mid = ld4(xr, xoff[(NI - 1) / 2], __builtin_amdgcn_readfirstlane(XY ? xgroup(a, cm) : cm * dx), 0);
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
            mw = fmaxf(mw, __shfl_xor(mw, 32, 64));
            mw = mw < __builtin_inff() ? mw : 0.f;
            // a channel whose sample is all zeros (or not finite) takes the largest of the wave's
            if (__any(mw == 0.f)) {
                const float wave_mw = h2_wave_max(mw);
                mw = mw > 0.f ? mw : wave_mw;
            }
            ew = h2_exponent(__float_as_uint(mw), kH2TopSample);
        }
        __syncthreads();
        unsigned t = 0;
#pragma unroll
        for (int w = 0; w < kH2Waves; ++w) t = max(t, top[w]);
        // (a sample of zeros, or with an infinity, says nothing: values about 1)
        if (t == 0 || t >= 0x7f800000u) t = 0x3f800000u;
        ex = __builtin_amdgcn_readfirstlane(h2_exponent(t, kH2TopSample));
    }
    const float sclx2 = ldexpf(1.f, ex + 11), sclw2 = ldexpf(1.f, ew + 11);
    const unsigned x_small = h2_key(h2_small(ex));
    const float w_small = h2_small(ew);
    // the wave's small input values; its small filter values (at most), and the
    // lanes (channels) that hold them
    int n_small = 0, nw_small = 0;
    unsigned long w_seen = 0;
    auto stage_one = [&](int at, int c, int j, unsigned& low) __attribute__((always_inline)) {  // at: the buffer's v8h
        v4h t[2];
        h2_terms(xv[c][j], sclx2, t[0], t[1]);
        low = h2_low(xv[c][j], low);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if constexpr (SMALL)
                reinterpret_cast<v4h*>(&xl[0][0][e][0][0])[xp + 256 * j] = t[e];
            else
                reinterpret_cast<v4h*>(&xl[0][c][e][xq >> 1][xp + 64 * j] + at)[xq & 1] = t[e];
        }
    };
    // (the barrier that follows makes the wave's count so far visible too)
    auto stage = [&](int at) __attribute__((always_inline)) {
        unsigned low = ~0u;
#pragma unroll
        for (int c = 0; c < UC; ++c)
#pragma unroll
            for (int j = 0; j < NI; ++j) stage_one(at, c, j, low);
        if (__any(low < x_small)) {
#pragma unroll
            for (int c = 0; c < UC; ++c)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) n_small += __popcll(__ballot(h2_key(xv[c][j][e]) < x_small));
            small[wave] = n_small;  // (by all lanes)
        }
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
        if constexpr (PRE) lexp[threadIdx.x] = my_exp;
    }
    small[wave] = 0;  // (read behind the barrier of the last staging)
    if constexpr (!PRE) {
        if (lane < 32) lexp[wk * 32 + lane] = h2_channel(ew, 0);
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
    unsigned w_low = 0;  // the wave's channels with small filter values
    if constexpr (PRE) w_low = (unsigned)__ballot(h2_channel_small(lexp[wk * 32 + (lane & 31)]) != 0);
    // off: the step's input from the lane's first (a chunk of one block walks
    // the kernel entries, a pointwise chunk its blocks); left: steps of the
    // chunk from this one on, at least two in a whole chunk
    const int per_chunk = UC > 1 ? UC : __builtin_amdgcn_readfirstlane(per_block);
    const int columns = SMALL ? a.U : a.S;  // steps of a kernel row
    constexpr int kColumn = SMALL ? 4 : 1;
    const int row_skip = __builtin_amdgcn_readfirstlane(h.PW - kColumn * columns);
    // base: the other buffer; next: the next chunk to stage, once `left` is stage_at
    int off = 0, s = columns, left = per_chunk, base = SMALL ? 0 : kBuffer, next = c_lo + UC;
    int stage_at = next < c_hi ? 2 : 0;
    auto advance = [&]() __attribute__((always_inline)) {
        if constexpr (UC > 1) {
            off += kBlock;
        } else {
            --s;
            off += s == 0 ? row_skip + kColumn : kColumn;
            s = s == 0 ? columns : s;
        }
        --left;
        off = left == 0 ? base : off;  // (s is `columns` again)
        if constexpr (!SMALL) base ^= left == 0 ? kBuffer : 0;
        left = left == 0 ? per_chunk : left;
    };
    // A step's 3 NP matrix instructions run back to back only if nothing that
    // they read is still on its way, so everything else stands between them, in
    // their shadow, held there by scheduling fences (left alone the scheduler
    // puts the LDS reads right before their use, and a wait in front of every
    // second instruction):
    //   - an operand of the next step's input is read from LDS as soon as this
    //     step's instructions have taken the last from its registers;
    //   - a float32 filter's own step is looked through for small values.
    // The filter's next step is converted behind them, where its loads have had
    // a whole step more (between the instructions: the same for 128 -> 128 at
    // 28x28, but spilt registers for large patches, 64 -> 64 at 56x56 75 us
    // against 37).
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
            v2h t[2];
            h2_pair(v[pair / 2][2 * pair % 4], v[pair / 2][2 * pair % 4 + 1], sclw2, t[0], t[1]);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                o[e][2 * pair] = t[e][0];
                o[e][2 * pair + 1] = t[e][1];
            }
        }
    };
    auto step = [&](v4f (&wd)[2], const v4f (&wnext)[2]) __attribute__((always_inline)) {
        const bool stage_next = !SMALL && left == stage_at;
        if constexpr (PRE) {
            w[0] = __builtin_bit_cast(v8h, wd[0]);
            w[1] = __builtin_bit_cast(v8h, wd[1]);
        }
        v8h wn[2];
        // The lowest of the lane's filter magnitudes, one instruction for two; only a
        // step with one below the limit, most often a zero, is looked at by keys
        // (always by keys: 128 -> 128 at 28x28 batch 32 45 us against 39).  Stems have
        // zeros in every step.
        float low = __builtin_inff();
        unsigned key = ~0u;
        advance();
        __builtin_amdgcn_sched_barrier(0);
        auto between = [&](int slot) __attribute__((always_inline)) {  // of 2 NP
            if constexpr (!PRE) {  // (the step's own values: the next one's are still on their way)
                if (slot < 4 && SMALL)
                    key = min(min(key, h2_key(wd[slot / 2][2 * slot % 4])), h2_key(wd[slot / 2][2 * slot % 4 + 1]));
                else if (slot < 4)
                    low = h2_min3(low, wd[slot / 2][2 * slot % 4], wd[slot / 2][2 * slot % 4 + 1]);
            }
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
        if constexpr (!PRE) {
            auto count = [&]() __attribute__((always_inline)) {
                const unsigned long m = __ballot(key < h2_key(w_small));
                w_seen |= m;
                nw_small += 8 * __popcll(m);
            };
            if constexpr (SMALL) {
                count();
            } else if (__any(low < w_small)) {  // (a zero, or a small value)
#pragma unroll
                for (int e = 0; e < 8; ++e) key = min(key, h2_key(wd[e / 4][e % 4]));
                count();
            }
        }
        next_w(wd);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!PRE) {
#pragma unroll
            for (int q = 0; q < 4; ++q) convert_w(wnext, wn, q);
            w[0] = wn[0];
            w[1] = wn[1];
        }
        if (stage_next) {
            stage(base);
            next += UC;
            stage_at = next < c_hi ? 2 : 0;
            load_x(xv, next);
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

    // (every wave's count stands since the barrier behind its last staging)
    unsigned x_count = 0;
#pragma unroll
    for (int w = 0; w < kH2Waves; ++w) x_count += small[w];
    x_count = __builtin_amdgcn_readfirstlane(x_count);
    // join the sums; a non-finite one means a value out of range
    float bad = 0.f;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[p][v] = __builtin_fmaf(accl[p][v], 1.f / 2048.f, acc[p][v]);
            bad = __builtin_fmaf(acc[p][v], 0.f, bad);
        }
    bool again = __any(bad != bad);
    if constexpr (!PRE) w_low = (unsigned)(w_seen | (w_seen >> 32));
    if (x_count | w_low) {
        // m small inputs leave a sum an error of at most m 2^-36 times the
        // largest weight (2^15, 2^16 from a sample), m small weights one of m
        // 2^-36 times the largest input (2^16); 2^20 of both:
        const float x_lim = (float)x_count * (PRE ? 0.5f : 1.f);
        bool few = false;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int c = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            const float m = PRE ? (float)h2_channel_small(lexp[wk * 32 + c]) : ((w_low >> c) & 1) ? (float)nw_small : 0.f;
            const float lim = kb * 32 + c < h.K ? x_lim + m : 0.f;
#pragma unroll
            for (int p = 0; p < NP; ++p)
                few |= (fabsf(acc[p][v]) < lim) & (where[1][p0 + p * 32 + (lane & 31)] >= 0);
        }
        again = again || __any(few);
    }
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
        for (int v = 0; v < 4; ++v) ex4[j][v] = again ? 0 : -ex - h2_channel_exponent(lexp[q + v]);
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
