// Planning and launching of conv_generic_kernel_tiled (conv_tiled.h).
#include "conv_tiled.h"

#include <cstdio>

namespace bs {
namespace tiled {
namespace {

TiledKernelFn pick(int a, int w, int cb, int c, bool xnor, bool req) {
    switch (a) {
        case 1: return pick_a<1>(w, cb, c, xnor, req);
        case 2: return pick_a<2>(w, cb, c, xnor, req);
        case 3: return pick_a<3>(w, cb, c, xnor, req);
        default: return pick_a<4>(w, cb, c, xnor, req);
    }
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct Plan {
    TiledKernelFn fn;
    TiledArgs g;
    dim3 grid;
    int a, w, cb, c;
    bool xnor;
};

int64_t act_image_bytes(const ConvShape& s) {
    return (int64_t)s.h * s.w * s.abits * ((s.c + 31) / 32) * 4;
}

// Images per launch within the kernel's 32-bit buffer offsets and pixel
// counts; 0 when one image is already too large.
int64_t images_per_launch(const ConvShape& s, bool req) {
    const int64_t lim = pix::kMaxBufferBytes;
    const int64_t act_img = act_image_bytes(s);
    const int64_t pix_img = (int64_t)s.oh * s.ow;
    int64_t n = s.n;
    if (n > lim / act_img) n = lim / act_img;
    if (!req && n > lim / (pix_img * s.oc * 4)) n = lim / (pix_img * s.oc * 4);
    if (n > (INT32_MAX - 64) / pix_img) n = (INT32_MAX - 64) / pix_img;
    while (n > 0 && ceil_div(n * pix_img, 64) * ceil_div(s.oc, 4) >=
                        INT32_MAX / 8)
        n /= 2;
    return n;
}

// The plan of one launch of shape s (n within images_per_launch), its int32
// output at element pixel * pix_step + channel * ch_step.
Plan make_plan(const ConvShape& s, const Requant* rq, int pix_step,
               int ch_step, int cus) {
    Plan pl{};
    TiledArgs& g = pl.g;
    const int cw = (s.c + 31) / 32;
    pl.a = group_planes(s.abits);
    pl.w = group_planes(s.wbits);
    Encoding e = encoding_terms(s);
    plane_weights(s.wbits, s.wenc, g.pw8);
    pl.xnor = s.aenc == kBipolar && s.abits == 1;
    if (pl.xnor && !e.xnor) {
        // aw sum_j pw_j (2 S_j - SW_j) = aw sum_j pw_j (SA - D_j)
        const int32_t aw = -e.csw;
        e.cs = -aw;
        for (int j = 0; j < s.wbits; ++j) e.csa += aw * g.pw8[j];
        e.csw = 0;
    }
    // words per chunk: 3 or 4, whichever reads fewer past the plane (4 when
    // equal: fewer steps)
    pl.cb = cw < 4 ? cw : ceil_div(cw, 3) * 3 < ceil_div(cw, 4) * 4 ? 3 : 4;
    g.h = s.h; g.w = s.w; g.oh = s.oh; g.ow = s.ow;
    g.sh = s.sh; g.sw = s.sw; g.ph = s.ph; g.pw = s.pw;
    g.kh = s.kh; g.kw = s.kw;
    g.cw = cw;
    g.c = s.c;
    g.oc = s.oc;
    g.npix = s.n * s.oh * s.ow;
    g.nch = (int32_t)ceil_div(cw, pl.cb);
    g.nsteps = s.kh * s.kw * g.nch;
    g.abits = s.abits; g.wbits = s.wbits;
    g.act_groups = plane_groups(s.abits);
    g.wt_groups = plane_groups(s.wbits);
    g.act_bytes = (int32_t)(s.n * act_image_bytes(s));
    g.wt_bytes = (int32_t)((int64_t)s.oc * s.kh * s.kw * s.wbits * cw * 4);
    g.out_bytes = rq ? 0 : (int32_t)((int64_t)g.npix * s.oc * 4);
    g.pix_step = pix_step;
    g.ch_step = ch_step;
    plane_weights(s.abits, s.aenc, g.pa);
    g.cs = e.cs; g.csa = e.csa; g.csw = e.csw; g.cn = e.cn;
    g.out_scale = rq ? rq->scale : 0.0f;
    g.out_bits = rq ? rq->bits : 0;
    g.out_qmax = rq ? (float)((1 << rq->bits) - 1) : 0.0f;
    g.out_words = (s.oc + 31) / 32;
    g.div_ow.init((uint32_t)s.ow);
    g.div_oh.init((uint32_t)s.oh);
    g.div_nch.init((uint32_t)g.nch);
    g.div_kw.init((uint32_t)s.kw);

    // The tile: the widest one, unless a quarter of its channels would be
    // padding.  Then more waves, each of which repeats a wave's set-up (about
    // 250 vector instructions): narrower units until there are 4 waves for every
    // SIMD; waves sharing a unit's steps, two until there are 4, or four until
    // there are 3.5, or either until there are 3 where a unit has less than 12
    // steps; and 4-channel tiles, which load each word four times as often,
    // until there are 3.
    //
    // Whole / shared units at 3 to 3.6 waves a SIMD: 44x20x20x192 -> 192 3x3 (18
    // steps) A2W1 37.6 / 32.4 us, A2W2 61.4 / 55.1; 178x14x14x64 -> 96 5x5 (25)
    // 36.7 / 33.4; 583x9x9x352 -> 70 (27) A1W2 64.2 / 60.1.  Over 233 random shapes,
    // rate shared / whole: two waves, 24 steps and more 1.04 to 1.19, less than 6
    // 0.88 to 0.99; four waves, 12 and more 1.00 to 1.13 up to 3.5 waves a SIMD,
    // 0.98 to 1.01 above, less than 12 0.87 to 0.98; narrower units 1.02 to 1.19.
    // 4 / 16 channels at 3.2 waves: 45x14x14x64 -> 96 5x5 A2W1 15.9 / 13.1 us, A1W2
    // 17.6 / 14.1, 129x9x9x352 -> 70 18.9 / 19.6.
    const int64_t groups = ceil_div(g.npix, 64);
    const int64_t simds = (int64_t)cus * 4;
    const int64_t want = simds * 4, few = simds * 3;
    const int least = rq ? 8 : 4;      // a packed byte is 8 channels
    pl.c = max_channels(pl.a, pl.w);
    if (4 * (int64_t)s.oc < 3 * ceil_div(s.oc, pl.c) * pl.c) pl.c = 4;
    int cols = kMaxCols;
    while (cols > pl.c && cols > least && ceil_div(s.oc, cols) * cols > s.oc &&
           ceil_div(s.oc, cols / 2) * (cols / 2) <
               ceil_div(s.oc, cols) * cols)
        cols /= 2;
    auto waves = [&]() { return groups * ceil_div(s.oc, cols) << g.ks_log2; };
    while (waves() < want && cols > pl.c && cols > least) cols /= 2;
    while (g.ks_log2 < 2 && g.nsteps >= 4 << g.ks_log2 &&
           waves() < (g.nsteps < 12 ? few
                      : g.ks_log2 == 0 ? want : simds * 7 / 2))
        ++g.ks_log2;
    while (waves() < few && pl.c > 4) {
        pl.c = 4;
        while (waves() < few && cols > pl.c && cols > least) cols /= 2;
    }
    g.unit_cols = cols;
    g.nsub = cols / pl.c;
    g.div_cols.init((uint32_t)ceil_div(s.oc, cols));
    g.units = (int32_t)(groups * ceil_div(s.oc, cols));
    const int per_block = kWaves >> g.ks_log2;
    pl.grid = dim3((uint32_t)ceil_div(g.units, per_block));
    pl.fn = pick(pl.a, pl.w, pl.cb, pl.c, pl.xnor, rq != nullptr);
    return pl;
}

// A 1x1 conv at stride 1 without padding is a matrix product, whose operands
// can change places: output channels on the lanes, pixels as the uniform
// rows.
ConvShape swapped(const ConvShape& s) {
    ConvShape t = s;
    t.n = t.h = t.oh = 1;
    t.w = t.ow = s.oc;
    t.oc = s.n * s.oh * s.ow;
    t.abits = s.wbits; t.wbits = s.abits;
    t.aenc = s.wenc; t.wenc = s.aenc;
    t.bipolar_w = t.wenc == kBipolar;
    return t;
}

bool fits(const ConvShape& s, bool req) {
    const int64_t cw = (s.c + 31) / 32;
    // the fold multiplies popcounts as 24-bit values
    if ((int64_t)s.kh * s.kw * s.c >= 1 << 23) return false;
    if ((int64_t)s.oc * s.kh * s.kw * s.wbits * cw * 4 > pix::kMaxBufferBytes)
        return false;
    return images_per_launch(s, req) >= 1;
}

// Lanes doing work, in 1/1024, with s's pixels on the lanes.
int64_t lane_share(const ConvShape& s) {
    const int64_t p = (int64_t)s.n * s.oh * s.ow;
    const int64_t chans = ceil_div(s.oc, 4) * 4;
    return 1024 * p * s.oc / (ceil_div(p, 64) * 64 * chans);
}

}  // namespace

bool prefer_swapped(const ConvShape& s) {
    if (s.kh != 1 || s.kw != 1 || s.sh != 1 || s.sw != 1 || s.ph || s.pw)
        return false;
    const int64_t p = (int64_t)s.n * s.oh * s.ow;
    if (p >= 64 || p * s.oc * 4 > pix::kMaxBufferBytes) return false;
    const ConvShape t = swapped(s);
    return lane_share(t) > lane_share(s) && fits(t, false);
}

bool covers(const ConvShape& s, bool req) { return fits(s, req); }

hipError_t launch_conv(const ConvShape& s, const uint32_t* act,
                       const uint32_t* wts, int32_t* out, const Requant* rq,
                       int cus, hipStream_t st) {
    if (!rq && prefer_swapped(s)) {
        const Plan pl = make_plan(swapped(s), nullptr, 1, s.oc, cus);
        return launch(pl.fn, pl.grid, dim3(kBlock), 0, st, wts, act, out,
                      pl.g);
    }
    const int64_t per = images_per_launch(s, rq != nullptr);
    const int64_t act_img = act_image_bytes(s) / 4;
    const int64_t out_img =
        (int64_t)s.oh * s.ow *
        (rq ? (int64_t)rq->bits * ((s.oc + 31) / 32) : (int64_t)s.oc);
    for (int64_t n0 = 0; n0 < s.n; n0 += per) {
        ConvShape c = s;
        c.n = (int32_t)(s.n - n0 < per ? s.n - n0 : per);
        const Plan pl = make_plan(c, rq, s.oc, 1, cus);
        const hipError_t e =
            launch(pl.fn, pl.grid, dim3(kBlock), 0, st, act + n0 * act_img,
                   wts, out + n0 * out_img, pl.g);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int describe(const ConvShape& s, const char* enc, int cus, char* buf,
             size_t len) {
    const bool sw = prefer_swapped(s);
    ConvShape c = sw ? swapped(s) : s;
    const int64_t per = images_per_launch(c, false);
    const int64_t launches = ceil_div(c.n, per);
    if (c.n > per) c.n = (int32_t)per;
    const Plan pl = make_plan(c, nullptr, 1, 1, cus);
    return snprintf(buf, len,
                    "conv_generic_kernel_tiled<A=%d,W=%d,CB=%d,C=%d%s> "
                    "A=%d W=%d %s%s grid=%u block=%d units=%d of %d channels "
                    "waves_per_unit=%d%s",
                    pl.a, pl.w, pl.cb, pl.c, pl.xnor ? ",xnor" : "", s.abits,
                    s.wbits, enc, sw ? " operands swapped" : "", pl.grid.x,
                    kBlock, pl.g.units, pl.g.unit_cols, 1 << pl.g.ks_log2,
                    launches > 1 ? " (per launch; batch split)" : "");
}

}  // namespace tiled
}  // namespace bs
