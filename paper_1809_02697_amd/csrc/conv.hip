// Blocked convolution on fp32 MFMA (gfx950): launch configuration, cost model
// and launcher.  The kernels are in conv_kernel.h; this file instantiates the
// NCHW16c -> NCHW16c family, conv_xy.hip every other pair of blocks.
#include <array>
#include <map>
#include <mutex>
#include <new>

#include "conv_h2.h"

namespace neo {

using namespace conv_detail;

static_assert(kMaxGroup == kMaxGroupConvs, "group size");

extern template hipError_t conv_detail::dispatch_all<true>(const ConvConfig&, int, bool, bool,
                                                           const ConvArgs&, hipStream_t);
extern template hipError_t conv_detail::dispatch_h2<false, false>(const ConvConfig&, int, bool, const H2Args&, hipStream_t);
extern template hipError_t conv_detail::dispatch_h2<false, true>(const ConvConfig&, int, bool, const H2Args&, hipStream_t);
extern template hipError_t conv_detail::dispatch_h2<true, false>(const ConvConfig&, int, bool, const H2Args&, hipStream_t);
extern template hipError_t conv_detail::dispatch_h2<true, true>(const ConvConfig&, int, bool, const H2Args&, hipStream_t);

int conv_group(const ConvShape& s, const ConvConfig& c) {
    if (conv_small_c(s)) return 1;
    const int CB = cdiv(s.C, 16);
    int g = c.fk * c.fp == 1 ? 4 : (c.fk * c.fp == 2 ? 2 : 1);
    while (CB % g) g /= 2;
    return g;
}

int conv_steps(const ConvShape& s, const ConvConfig& c) {
    if (conv_small_c(s)) return s.R * cdiv(s.S, 4);
    return cdiv(s.C, 16) / conv_group(s, c) * s.R * s.S;
}

namespace {

// How the two-term kernel cuts the output pixels into tiles of P and the input
// patch of one: the patch pixels (at most), and the tiles.
struct H2Geometry {
    int kind, ltw, th, PW, patch;
    long tiles;
};

constexpr int kH2MaxPatch = 512, kH2MaxSmallPatch = 1536;

// Kernel columns that a patch row holds past its pixels' first: on the
// small-channel path whole groups of four.
int h2_columns(const ConvShape& s) { return conv_small_c(s) ? 4 * cdiv(s.S, 4) : s.S; }

// Whole rows of consecutive pixels (which may run over several images), or
// blocks of th x tw pixels of one image, whichever costs least: per channel
// block and tile the matrix instructions take 3 P cycles per kernel entry
// and a patch pixel's load, conversion and store about 1.5.  False if no patch
// fits.
bool h2_geometry(const ConvShape& s, int P, H2Geometry* out) {
    const long M = (long)s.N * s.OH * s.OW;
    const bool small = conv_small_c(s);
    const int S = h2_columns(s);
    if (s.R == 1 && s.S == 1 && !small) {
        *out = H2Geometry{kH2Point, 0, 0, 1, P, (M + P - 1) / P};
        return true;
    }
    double best = 1e300;
    auto consider = [&](int kind, int ltw, int th, long PW, long rows, long tiles) {
        if (PW * rows > (small ? kH2MaxSmallPatch : kH2MaxPatch)) return;
        const double cost = small ? (double)tiles * (3.0 * P * s.R * S / 4 + 0.4 * (double)(PW * rows))
                                  : (double)tiles * (3.0 * P * s.R * s.S + 1.5 * (double)(PW * rows));
        if (cost < best) {
            best = cost;
            *out = H2Geometry{kind, ltw, th, (int)PW, (int)(PW * rows), tiles};
        }
    };
    {
        // output rows that P consecutive pixels touch, and images those rows lie in
        const long nr = std::min<long>((P - 2) / s.OW + 2, (long)s.N * s.OH);
        const long ni = std::min<long>(nr < 2 ? 1 : (nr - 2) / s.OH + 2, s.N);
        consider(kH2Rows, 0, 0, (long)(s.OW - 1) * s.sw + S, nr * s.sh + ni * std::max(s.R - s.sh, 0), (M + P - 1) / P);
    }
    for (int ltw = 2; (1 << ltw) <= P; ++ltw) {
        const int tw = 1 << ltw, th = P / tw;
        consider(kH2Block, ltw, th, (long)(tw - 1) * s.sw + S, (long)(th - 1) * s.sh + s.R,
                 (long)s.N * cdiv(s.OH, th) * cdiv(s.OW, tw));
    }
    return best < 1e300;
}

// Patch pixels / 64 (/ 256 on the small-channel path) that the kernel is
// instantiated for.
int h2_patch_blocks(const ConvShape& s, const H2Geometry& g) {
    if (conv_small_c(s)) return cdiv(g.patch, 512) * 2;
    const int n = cdiv(g.patch, 64);
    return g.kind == kH2Point ? n : n <= 2 ? 2 : n <= 3 ? 3 : n <= 5 ? 5 : 8;
}

int h2_pixels(const ConvConfig& c) { return 32 * c.fp * (kH2Waves / c.fk); }

}  // namespace

// Short reductions keep the float32 kernel.  A two-term product is off by up to
// a few units of its last place, a sum of many is closer than the float32
// kernel's (it is rounded once per 16 products); where one outweighs the other
// was measured against float64, relative error in 1e-8, two-term and float32
// (a chain of one wave, as that kernel runs launches that fill the chip):
// 1 product 6.8 / 2.6, 9 8.4 / 5.3, 16 8.4 / 7.3, 20 8.3 / 8.2, 24 8.5 / 9.0,
// 32 8.6 / 10, 64 9.2 / 14, 576 17 / 42.  Of one or two channels, whose steps
// are mostly padding: 25 10.1 / 8.8, 36 10.8 / 10.7, 42 11.1 / 11.4, 49 11.9 / 12.2.
static bool h2_long_enough(const ConvShape& s) { return s.C * s.R * s.S >= (s.C < 3 ? 42 : 24); }

bool conv_h2_config_valid(const ConvShape& s, const ConvConfig& c) {
    // (the folded global pool needs the tile kernel's epilogue)
    if (!conv_h2(c) || !(c.fk == 2 || c.fk == 4) || !(c.fp == 2 || c.fp == 4) || c.split < 1 || c.split > 64 ||
        s.gap || (conv_small_c(s) && c.split > 1) || !h2_long_enough(s))
        return false;
    H2Geometry g;
    return h2_geometry(s, h2_pixels(c), &g) && g.tiles * cdiv(cdiv(s.K, s.yb) * s.yb, 32 * c.fk) * c.split < (1L << 30) &&
           h2_filter_floats(s) * 4 < (1L << 31);
}

int conv_h2_chunks(const ConvShape& s, const ConvConfig& c) {
    const int CB = cdiv(s.C, 16);
    return s.R == 1 && s.S == 1 && !conv_small_c(s) ? cdiv(CB, h2_blocks(h2_pixels(c) / 64)) : CB;
}

// Steps of the whole reduction.
static int h2_filter_steps(const ConvShape& s) {
    return conv_small_c(s) ? s.R * cdiv(s.S, 4) : cdiv(s.C, 16) * s.R * s.S;
}

long h2_filter_floats(const ConvShape& s) {
    const long kb = cdiv(cdiv(s.K, 16), 2);
    return kb * h2_filter_steps(s) * 512 + kb * 32;
}

hipError_t launch_h2_filter(const ConvShape& s, const float* w, float* out, hipStream_t st) {
    const int KB = cdiv(s.K, 16), steps = h2_filter_steps(s);
    return launch_h2_split(w, KB, steps, out, reinterpret_cast<int*>(out + (long)cdiv(KB, 2) * steps * 512), st);
}

bool conv_config_valid(const ConvConfig& c) {
    const bool tile = (c.fk == 1 || c.fk == 2 || c.fk == 4) && (c.fp == 1 || c.fp == 2 || c.fp == 4);
    const bool waves = c.waves == 1 || c.waves == 2 || c.waves == 4 ||
                       (c.waves == 8 && c.fk * c.fp <= 4) || (c.waves == 16 && c.fk * c.fp <= 2);
    return tile && waves && c.split >= 1 && c.split <= 64;
}

// Cost model for the launch configuration of one shape, in microseconds: a
// per-launch floor, plus the longest chain of reduction steps any wave walks
// (each step: its MFMAs, or the measured ~300-cycle bookkeeping-and-load
// chain when a SIMD has a single wave, shared between resident waves), plus
// the extra kernel and partial round trip of a split.
ConvConfig choose_tile_config(const ConvShape& s, double* us) {
    const int KB = cdiv(s.K, 16), MP = cdiv(s.N * s.OH * s.OW, 16);
    const double kClk = 2400.0;  // cycles per microsecond
    ConvConfig best{1, 1, 1, 4};
    double best_t = 1e30;
    static const int fks[] = {1, 2, 4}, fps[] = {1, 2, 4}, wvs[] = {1, 2, 4, 8, 16};
    static const int splits[] = {1, 2, 3, 4, 6, 8};
    for (int fk : fks) {
        if (fk > 1 && fk > KB) continue;
        for (int fp : fps) {
            if (fp > 1 && fp > MP) continue;
            const long tiles = (long)cdiv(MP, fp) * cdiv(KB, fk);
            for (int wv : wvs) {
                for (int sp : splits) {
                    const ConvConfig c{fk, fp, sp, wv};
                    if (!conv_config_valid(c)) continue;
                    const int T = conv_steps(s, c), G = conv_group(s, c);
                    if (sp > 1 && T / sp < wv) continue;
                    const long wgs = tiles * sp;
                    const double steps = std::ceil((double)T / sp / wv);
                    const double waves_per_simd = (double)wgs * wv / 1024.0;
                    const double resident = std::max(1.0, std::min(8.0, waves_per_simd));
                    const double rounds = std::max(1.0, std::ceil(waves_per_simd / 8.0));
                    const double mfma = 4.0 * G * fk * fp * 32.0;
                    const double chain = 300.0 + 40.0 * (fk + fp);
                    const double per_step = std::max(mfma * resident, chain);
                    double t = 3.5 + rounds * steps * per_step / kClk;
                    if (sp > 1) t += 2.0 + 2.0 * sp * s.N * KB * s.OH * s.OW * 64.0 / 4.0e6;
                    if (t < best_t * 0.98) {
                        best_t = t;
                        best = c;
                    }
                }
            }
        }
    }
    if (us) *us = best_t;
    return best;
}

namespace {

// Time of the two-term kernel in microseconds.  A workgroup alone on its CU
// walks a chain: per step 133 + 185 fp cycles, per chunk 337 for each float4 of
// a thread's patch, and 10,400 to set up, sample and store; several on one CU
// share its matrix and vector units, where a step takes 96 fp + 181 cycles and
// a float4 264.  The constants are a fit to 2,174 measured launches (220
// shapes of 1x1 to 7x7 kernels at batch 1 to 32, every tile, splits 1 to 8):
// mean deviation 11 %.  Against the kernel as it is now, over 30,701 launches of
// 3,357 other shapes: 12 %.  A new fit to those brings it to 9 % and makes the
// same choices (within 5 % of the best for 90 against 89 % of the shapes), so
// the constants stay.
double h2_time_us(const ConvShape& s, const ConvConfig& c) {
    H2Geometry g;
    if (!conv_h2_config_valid(s, c) || !h2_geometry(s, h2_pixels(c), &g)) return 1e30;
    const int CB = cdiv(s.C, 16), ni = h2_patch_blocks(s, g), uc = g.kind == kH2Point ? h2_blocks(ni) : 1;
    const int chunks = cdiv(conv_h2_chunks(s, c), c.split);
    const double steps = conv_small_c(s) ? h2_filter_steps(s) : (double)std::min(uc, CB) * s.R * s.S, items = uc * ni;
    const long lds = 2048 + (conv_small_c(s) ? 16L * (256 * ni + 4) : 2L * uc * 4 * (64 * ni + 4) * 16);
    const double occ = (double)std::max<long>(1, std::min<long>(c.fp == 4 ? 2 : 3, 163840 / lds));
    const double chain = chunks * (steps * (133.0 + 185.0 * c.fp) + 337.0 * items) + 10400.0;
    const double share = chunks * (steps * (181.0 + 96.0 * c.fp) + 264.0 * items) + 5600.0;
    const double per_cu = (double)g.tiles * cdiv(s.K, 32 * c.fk) * c.split / 256.0;
    const double full = std::floor(per_cu / occ), rest = std::ceil(per_cu - full * occ - 1e-9);
    double t = full * std::max(chain, occ * share);
    if (rest > 0) t += std::max(chain, rest * share);
    double us = 2.2 + t / 2400.0;
    if (c.split > 1) us += 1.3 + 2.0 * conv_workspace_bytes(s, c) / 3.8e6;
    return us;
}

// The tile kernel's model is too fast by 1.4 to 2.5 (the middle half of the 3,357
// shapes: 1.5 to 2.0), the two-term kernel's is not, so the line between them
// lies at 1.4 times the tile model's time: 1,393 of the shapes then take the
// two-term kernel, 1.66 times as fast on average, 14 of them more than 5 % slower
// (the worst 12 %).  At 1.3 that is 1 shape and 0.5 % more time on average, at
// 1.5 65 shapes and 0.2 % less.
constexpr double kH2Line = 1.4;

}  // namespace

namespace {

ConvConfig model_conv_config(const ConvShape& s) {
    double tile_us = 0;
    ConvConfig best = choose_tile_config(s, &tile_us);
    double best_us = kH2Line * tile_us;
    // never more partials than the tile kernel's choice asks for: a call that
    // needed no workspace (under stream capture, say) still needs none
    const size_t ws = conv_workspace_bytes(s, best);
    for (int fk : {2, 4})
        for (int fp : {2, 4})
            for (int sp : {1, 2, 4, 8}) {
                const ConvConfig c{fk, fp, sp, 0};
                if (sp > 1 && (conv_workspace_bytes(s, c) > ws || sp > conv_h2_chunks(s, c))) continue;
                const double us = h2_time_us(s, c);
                if (us < best_us) {
                    best_us = us;
                    best = c;
                }
            }
    return best;
}

// The models' choices of the last shapes asked for: evaluating them takes a few
// microseconds, about as long as a small layer runs.
constexpr size_t kMaxChoices = 1024;
std::mutex g_choices_mu;
std::map<std::array<int, 13>, ConvConfig> g_choices;

}  // namespace

ConvConfig choose_conv_config(const ConvShape& s) {
    const std::array<int, 13> key{s.N, s.C, s.H, s.W, s.K, s.R, s.S, s.sh, s.sw, s.ph, s.pw, s.gap, s.yb};
    {
        std::lock_guard<std::mutex> lk(g_choices_mu);
        const auto it = g_choices.find(key);
        if (it != g_choices.end()) return it->second;
    }
    const ConvConfig c = model_conv_config(s);
    try {
        std::lock_guard<std::mutex> lk(g_choices_mu);
        if (g_choices.size() >= kMaxChoices) g_choices.clear();
        g_choices[key] = c;
    } catch (const std::bad_alloc&) {  // kept for speed only
    }
    return c;
}

size_t conv_workspace_bytes(const ConvShape& s, const ConvConfig& c) {
    if (c.split <= 1) return 0;
    return (size_t)c.split * s.N * cdiv(s.K, 16) * s.OH * s.OW * 64;
}

namespace {

constexpr long kKFirstMinWgs = 1024;  // launches this large take channel tiles first

// Kernel arguments of one convolution for launch configuration c with G
// channel groups per reduction step.
ConvArgs make_args(const ConvShape& s, const ConvConfig& c, int G, const float* x, const float* w,
                   bool wmfma, const float* bias, const float* res, float* y, float* ws) {
    // a workgroup's tile in blocks of 16 (the two-term kernel: 32 fk channels)
    const int bk = conv_h2(c) ? 2 * c.fk : c.fk, bp = c.fp;
    ConvArgs a;
    a.x = x;
    a.w = w;
    a.bias = bias;
    a.res = res;
    a.y = y;
    a.ws = ws;
    a.N = s.N;
    a.CB = cdiv(s.C, 16);
    a.H = s.H;
    a.W = s.W;
    a.KB = cdiv(s.K, 16);
    a.R = s.R;
    a.S = s.S;
    a.RS = s.R * s.S;
    a.U = cdiv(s.S, 4);
    a.sh = s.sh;
    a.sw = s.sw;
    a.ph = s.ph;
    a.pw = s.pw;
    a.OH = s.OH;
    a.OW = s.OW;
    a.M = s.N * s.OH * s.OW;
    a.y_off = s.y_off;
    a.y_tot = s.y_tot;
    a.act = s.act;
    a.CBG = a.CB / G;
    a.T = conv_small_c(s) ? s.R * cdiv(s.S, 4) : a.CBG * s.R * s.S;
    a.split = (c.split > 1 && ws) ? std::min(c.split, a.T) : 1;
    a.xb = s.xb;
    a.XB = cdiv(s.C, s.xb);
    a.xpb = s.xb * 4;
    const int Q = s.xb >= 16 ? s.xb / 16 : 1;
    a.lq = ilog2(Q);
    a.qm = Q - 1;
    a.dblk = s.H * s.W * a.xpb;
    a.yb = s.yb;
    a.lyb = ilog2(s.yb);
    a.KY = cdiv(s.K, s.yb);
    a.KBk = a.KY * s.yb / 16;
    a.x_bytes = (int)((long)s.N * a.XB * s.H * s.W * a.xpb);
    a.w_bytes = (int)((wmfma ? kernel_filter_floats(s) : (long)a.KB * a.CB * a.RS * 256) * 4);
    a.div_ohw = make_fastdiv((unsigned)(s.OH * s.OW));
    a.div_ow = make_fastdiv((unsigned)s.OW);
    a.div_npx = make_fastdiv((unsigned)cdiv(a.M, 16 * bp));
    a.div_nkb = make_fastdiv((unsigned)cdiv(a.KBk, bk));
    // Large launches take channel tiles first: the workgroups that read one
    // input tile then run on one XCD and share its L2.  Measured on MI355X
    // (tuned, fused plans): from 1024 workgroups up, ResNet-50 batch 32 runs
    // 2.76 ms against 2.82 ms with pixel tiles first, batch 1 and VGG-16
    // batch 1 unchanged; from 512 up, batch 1 is 1.3 % slower.
    a.kfirst = (long)cdiv(a.M, 16 * bp) * cdiv(a.KBk, bk) >= kKFirstMinWgs;
    a.gap = s.gap;
    return a;
}

}  // namespace

hipError_t launch_conv2d(const ConvShape& s, const ConvConfig& c, const float* x, const float* w,
                         bool wmfma, const float* bias, const float* res, float* y, float* ws,
                         hipStream_t st, const float* wh2) {
    if (c.fp == 0) {  // the streaming pointwise kernel (filter in kernel order)
        if (!wmfma || !conv_stream_config_valid(s, c)) return hipErrorInvalidValue;
        return launch_conv_stream(s, c, x, w, bias, res, y, st);
    }
    if (conv_h2(c)) {
        H2Geometry g;
        if (!conv_h2_config_valid(s, c) || !conv_blocks_valid(s) || (wmfma && !wh2) ||
            !h2_geometry(s, h2_pixels(c), &g))
            return hipErrorInvalidValue;
        H2Args h;
        h.a = make_args(s, c, 1, x, wmfma ? wh2 : w, wmfma, bias, res, y, ws);
        ConvArgs& a = h.a;
        h.chunks = conv_h2_chunks(s, c);
        a.split = (c.split > 1 && ws) ? std::min(c.split, h.chunks) : 1;
        a.div_npx = make_fastdiv((unsigned)g.tiles);
        a.kfirst = g.tiles * a.div_nkb.d >= kKFirstMinWgs;
        h.w32 = w;
        h.w32_bytes = a.w_bytes;
        h.K = s.K;
        h.wexp = nullptr;
        if (wmfma) {
            const long blocks = (long)cdiv(a.KB, 2) * h2_filter_steps(s);
            a.w_bytes = (int)(blocks * 2048);
            h.wexp = reinterpret_cast<const int*>(wh2 + blocks * 512);
        }
        h.kind = g.kind;
        h.ltw = g.ltw;
        h.th = g.th;
        h.PW = g.PW;
        h.SF = (s.OH - 1) * s.sh + s.R;
        h.div_pw = make_fastdiv((unsigned)g.PW);
        h.div_sf = make_fastdiv((unsigned)h.SF);
        const int tx = g.kind == kH2Block ? cdiv(s.OW, 1 << g.ltw) : 1;
        h.div_tx = make_fastdiv((unsigned)tx);
        h.div_tpi = make_fastdiv((unsigned)(g.kind == kH2Block ? tx * cdiv(s.OH, g.th) : 1));
        const int n = h2_patch_blocks(s, g);
        const bool xy = s.xb != 16 || s.yb != 16, small = conv_small_c(s);
        if (wmfma) return xy ? dispatch_h2<true, true>(c, n, small, h, st) : dispatch_h2<true, false>(c, n, small, h, st);
        return xy ? dispatch_h2<false, true>(c, n, small, h, st) : dispatch_h2<false, false>(c, n, small, h, st);
    }
    if (!conv_config_valid(c) || !conv_blocks_valid(s)) return hipErrorInvalidValue;
    if (s.gap && s.N != 1) return hipErrorInvalidValue;
    const int G = conv_group(s, c);
    // a folded global pool writes its sums in the kernel's epilogue: no split
    const ConvArgs a = make_args(s, c, G, x, w, wmfma, bias, res, y, s.gap ? nullptr : ws);
    const bool small = conv_small_c(s);
    if (s.xb == 16 && s.yb == 16) return dispatch_all<false>(c, G, small, wmfma, a, st);
    return dispatch_all<true>(c, G, small, wmfma, a, st);
}

bool conv_group_eligible(const ConvShape& s) {
    return !conv_small_c(s) && s.xb == 16 && s.yb == 16 && !s.gap;
}

int conv_group_steps_min(const ConvShape* s, int n, const ConvConfig& c) {
    int G = 4, steps = 1 << 30;
    for (int i = 0; i < n; ++i) G = std::min(G, conv_group(s[i], c));
    for (int i = 0; i < n; ++i) steps = std::min(steps, cdiv(s[i].C, 16) / G * s[i].R * s[i].S);
    return steps;
}

bool conv_group_config_valid(const ConvShape* s, int n, const ConvConfig& c) {
    if (n < 1 || n > kMaxGroupConvs || c.split != 1 || !conv_config_valid(c)) return false;
    for (int i = 0; i < n; ++i) {
        if (!conv_group_eligible(s[i])) return false;
        const int KB = cdiv(s[i].K, 16), MP = cdiv(s[i].N * s[i].OH * s[i].OW, 16);
        if ((c.fk > 1 && c.fk > KB) || (c.fp > 1 && c.fp > MP)) return false;
    }
    return conv_group_steps_min(s, n, c) >= c.waves;
}

ConvConfig choose_group_config(const ConvShape* s, int n) {
    // the cost model's choice for the member with the most work, made valid
    // for every member (no split, a tile and wave count all can use)
    int big = 0;
    double most = -1;
    for (int i = 0; i < n; ++i) {
        const double f = (double)s[i].N * s[i].OH * s[i].OW * s[i].K * s[i].C * s[i].R * s[i].S;
        if (f > most) {
            most = f;
            big = i;
        }
    }
    ConvConfig c = choose_tile_config(s[big], nullptr);
    c.split = 1;
    for (int fk : {c.fk, 2, 1})
        for (int fp : {c.fp, 2, 1})
            for (int wv : {c.waves, 4, 2, 1}) {
                const ConvConfig t{fk, fp, 1, wv};
                if (conv_group_config_valid(s, n, t)) return t;
            }
    return ConvConfig{1, 1, 1, 1};
}

hipError_t launch_conv_group(const ConvShape* s, int n, const ConvConfig& c, const float* const* x,
                             const float* const* w, const float* const* bias,
                             const float* const* res, float* const* y, const GroupPool* pool,
                             hipStream_t st) {
    if (!conv_group_config_valid(s, n, c)) return hipErrorInvalidValue;
    // (a pool with an int8 copy runs in integer group launches only)
    if (pool && (!pow2_block(pool->s.xb) || !pool->x || !pool->y || pool->q.yq)) return hipErrorInvalidValue;
    int G = 4;
    for (int i = 0; i < n; ++i) G = std::min(G, conv_group(s[i], c));
    ConvGroupArgs ga;
    ga.n = n;
    ga.start[0] = 0;
    // Dispatch order: the members with the most reduction steps per tile
    // first (they finish last), ties in the given order.  Each member takes
    // a whole number of rounds over the XCDs.
    int order[kMaxGroup];
    for (int i = 0; i < n; ++i) order[i] = i;
    auto steps = [&](int i) { return cdiv(s[i].C, 16) / G * s[i].R * s[i].S; };
    std::stable_sort(order, order + n, [&](int p, int q) { return steps(p) > steps(q); });
    for (int j = 0; j < n; ++j) {
        const int i = order[j];
        ga.a[j] = make_args(s[i], c, G, x[i], w[i], true, bias[i], res[i], y[i], nullptr);
        ga.cnt[j] = cdiv(ga.a[j].M, 16 * c.fp) * cdiv(ga.a[j].KBk, c.fk);
        ga.start[j + 1] = ga.start[j] + cdiv(ga.cnt[j], kXcds) * kXcds;
    }
    for (int i = n; i < kMaxGroup; ++i) {
        ga.a[i] = ga.a[n - 1];
        ga.cnt[i] = 0;
        ga.start[i + 1] = ga.start[n];
    }
    PoolPart& pp = ga.pool;
    pp = PoolPart{};
    if (pool) {
        const PoolShape& ps = pool->s;
        pp.x = pool->x;
        pp.y = pool->y;
        pp.s = ps;
        pp.CB = cdiv(ps.C, ps.xb);
        pp.lq = ilog2(ps.xb / 4);
        const long total = ((long)ps.N * pp.CB * ps.OH * ps.OW) << pp.lq;
        if (total >= (1L << 31)) return hipErrorInvalidValue;
        pp.total = (int)total;
        pp.max = pool->max ? 1 : 0;
        pp.k33 = ps.R == 3 && ps.S == 3;
        // one output quad per thread, at most 1024 workgroups (then grid-stride)
        const long per = 64L * c.waves;
        pp.wgs = (int)std::min<long>(1024, std::max<long>(1, (total + per - 1) / per));
    }
    return dispatch_group(c, G, ga, ga.start[n] + pp.wgs, st);
}

}  // namespace neo
