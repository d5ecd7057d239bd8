// Run-time-shaped bitserial conv kernel (conv_generic_kernel_tiled) for the
// shapes the specialised families do not cover: any window, stride and
// padding, any number of words per plane, any channel counts, 1-8 bits and
// every encoding.  Instantiated in conv_tiled_inst.hip.
//
// Mapping.  As in the pixels-on-lanes kernel, lane l owns one output pixel of
// a 64-pixel group and the filter words, uniform across the wave, are the
// SGPR operand of v_and_b32.  Here the reduction is the outer loop: a step is
// one tap and CB words of each plane.  A lane loads the step's A x CB words
// (raw buffer loads; taps in the padding read zeros), and they meet the
// filter words of C channels, whose A x W popcount accumulators per channel
// stay in VGPRs over all the steps.  Only the accumulators depend on a
// template argument; taps, chunks, strides and plane weights are arguments.
//
// What bounds it: the AND + popcount stream, as in the specialised kernels.
// Per step a wave issues 2 C A W CB of those against about 10 vector
// instructions of set-up, and C W scalar loads.  C is 16 channels while the
// accumulators (A W C) fit 64 VGPRs, then 8 and 4: enough products per
// loaded activation word that the loads (L1 and L2 hits) stay hidden.
// C = 4 also exists for every width, for problems too small to fill the chip
// with larger tiles, and the KS waves of a unit then split its steps.
//
// Measured against what served these shapes before (one output per thread):
// 32 x 27 x 27 x 96 -> 150 channels, 3x3, A2 x bipolar W1, quantize+pack
// included: 290 -> 25.7 us a pass; 100 x 784 x 1000 product, A2W2: 64.6 ->
// 14.2 us (of which the host takes most).
//
// Filter words come through s_buffer_load, whose range check makes the last
// channel tile and the over-read of a 3-word chunk safe without clamping.
// Words of a last, partial chunk: the chunk starts early enough to end with
// the plane, and the words the previous chunk already counted are cleared.
//
// Encodings.  With pa_i, pw_j the planes' weights (+-2^i) the result is
//   cs S + csa SA + csw SW + cn N,  S = sum_ij pa_i pw_j popcount(a_i AND w_j),
// SA, SW the weighted popcounts of the in-range activation and filter words
// and N the in-range channel values (conv_pix.h has the derivation).  SW is S
// of an activation plane of ones on the in-range taps, computed by a pass of
// the same loop.  +-1 activations need no such pass: with
// D_j = popcount((a XOR w_j) AND in-range), D_j = SA + SW_j - 2 S_j, so
//   2 S_j - SW_j = SA - D_j
// and one pass over D_j (the XOR and the mask are one instruction) replaces
// those over S and SW, each as long.  (+-1 filters too: N - 2 D.)
// Measured, packing included, with the pass over SW and without (A1, +-1):
// 32 x 27 x 27 x 96 -> 150, 3x3, W2 43.0 -> 27.9 us; 64 x 28 x 28 x 128 -> 128,
// 3x3, W2 70.0 -> 46.7 us; 64 x 28 x 28 x 160 -> 200, 1x1, signed W3 35.4 ->
// 25.1 us; 4 x 14 x 14 x 96 -> 64, 5x5, W2 13.9 -> 13.9 us (host-bound).
#pragma once

#include <type_traits>

#include "bs_internal.h"
#include "conv_pix.h"

namespace bs {
namespace tiled {

using pix::kOutOfRange;
using pix::kXcds;
using pix::Rsrc;

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kMaxCols = 16;                 // output channels of a unit
constexpr int kStride = kMaxCols + 1;        // words per tile row (padded)
constexpr int kTileWords = 64 * kStride;
constexpr int kSliceWords = 16;              // filter words per SGPR slice

struct TiledArgs {
    int32_t h, w, oh, ow, sh, sw, ph, pw, kh, kw;
    int32_t cw;            // words per plane
    int32_t c;             // input channels
    int32_t oc;            // output channels
    int32_t npix;          // n * oh * ow
    int32_t nch;           // chunks per tap: ceil(cw / CB)
    int32_t nsteps;        // kh * kw * nch
    int32_t units, unit_cols, nsub, ks_log2;
    int32_t abits, wbits;
    int32_t act_groups, wt_groups;   // groups of A (W) planes
    int32_t act_bytes, wt_bytes;
    int32_t out_bytes;     // int32 output (0: packed output)
    int32_t pix_step, ch_step;       // int32 output strides, in elements
    int32_t pa[8], pw8[8];           // plane weights, 0 past the last plane
    int32_t cs, csa, csw, cn;
    FastDiv div_ow, div_oh, div_cols, div_nch, div_kw;
    // requantized output
    float out_scale, out_qmax;
    int32_t out_bits, out_words;
};

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

// Scalar buffer loads of wave-uniform words (the compiler has no builtin for
// them): words past the resource's size read zeros.
extern "C" __device__ v4i bs_sbuffer_load4(v4i rsrc, int off, int aux) __asm(
    "llvm.amdgcn.s.buffer.load.v4i32");
extern "C" __device__ v2i bs_sbuffer_load2(v4i rsrc, int off, int aux) __asm(
    "llvm.amdgcn.s.buffer.load.v2i32");
extern "C" __device__ int bs_sbuffer_load1(v4i rsrc, int off, int aux) __asm(
    "llvm.amdgcn.s.buffer.load.i32");

// Channels per accumulator tile of an A x W kernel.
constexpr int max_channels(int a, int w) {
    return a * w <= 4 ? 16 : a * w <= 8 ? 8 : 4;
}

// Channels per SGPR slice: the largest power of two whose words fit, at most
// half of the tile's, so that a step takes an even number of slices and the
// two buffers alternate the same way in every step.
template <int W, int CB, int C>
constexpr int slice_channels() {
    constexpr int per = W * (CB == 3 ? 4 : CB);
    int sc = C / 2;
    while (sc > 1 && sc * per > kSliceWords) sc >>= 1;
    return sc;
}

template <int W, int CB, int SC>
struct Slice {
    uint32_t w[SC][W][CB];
};

template <int W, int CB, int SC>
__device__ __forceinline__ void load_slice(Slice<W, CB, SC>& f, v4i rw,
                                           uint32_t off, uint32_t ch_bytes,
                                           const uint32_t (&plane)[W]) {
#pragma unroll
    for (int o = 0; o < SC; ++o) {
#pragma unroll
        for (int j = 0; j < W; ++j) {
            if constexpr (CB == 1) {
                f.w[o][j][0] =
                    (uint32_t)bs_sbuffer_load1(rw, (int)(off + plane[j]), 0);
            } else if constexpr (CB == 2) {
                const v2i x = bs_sbuffer_load2(rw, (int)(off + plane[j]), 0);
                f.w[o][j][0] = (uint32_t)x[0];
                f.w[o][j][1] = (uint32_t)x[1];
            } else {
                const v4i x = bs_sbuffer_load4(rw, (int)(off + plane[j]), 0);
#pragma unroll
                for (int k = 0; k < CB; ++k) f.w[o][j][k] = (uint32_t)x[k];
            }
        }
        off += ch_bytes;
    }
}

// The lane's window: its top-left input pixel and that pixel's byte offset
// (wrapped when it lies in the padding; in-range taps add up to true
// offsets).
struct Window {
    int iy0, ix0;
    uint32_t base;
};

// Position in the reduction: tap (r, s), first word c0 of the chunk as
// numbered, cs as read (a last partial chunk starts early), all uniform, and
// the lane's offset of the tap's pixel.
struct Step {
    int r, s, c0, cs;
    uint32_t voff;
    bool in;
};

template <int CB>
__device__ __forceinline__ void set_tap(Step& st, const TiledArgs& g,
                                        const Window& win) {
    const uint32_t pixb = 4u * (uint32_t)(g.abits * g.cw);
    st.in = (unsigned)(win.iy0 + st.r) < (unsigned)g.h &&
            (unsigned)(win.ix0 + st.s) < (unsigned)g.w;
    st.voff = st.in ? win.base + (uint32_t)(st.r * g.w + st.s) * pixb
                    : kOutOfRange;
}

template <int CB>
__device__ __forceinline__ void next_step(Step& st, const TiledArgs& g,
                                          const Window& win) {
    st.c0 += CB;
    if (st.c0 >= g.cw) {
        st.c0 = 0;
        if (++st.s == g.kw) {
            st.s = 0;
            ++st.r;
        }
        set_tap<CB>(st, g, win);
    }
    st.cs = min(st.c0, g.cw - CB);
}

template <int A, int CB, bool ONES>
__device__ __forceinline__ void load_words(uint32_t (&p)[A][CB], Rsrc act,
                                           const Step& st,
                                           const uint32_t (&plane)[A]) {
#pragma unroll
    for (int i = 0; i < A; ++i) {
        if constexpr (ONES) {
#pragma unroll
            for (int k = 0; k < CB; ++k) p[i][k] = st.in ? ~0u : 0u;
            continue;
        }
        const uint32_t so = plane[i] + 4u * (uint32_t)st.cs;
        if constexpr (CB == 4) {
            const auto x =
                __builtin_amdgcn_raw_buffer_load_b128(act, st.voff, so, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) p[i][k] = x[k];
        } else if constexpr (CB == 3) {
            const auto x =
                __builtin_amdgcn_raw_buffer_load_b96(act, st.voff, so, 0);
#pragma unroll
            for (int k = 0; k < 3; ++k) p[i][k] = x[k];
        } else if constexpr (CB == 2) {
            const auto x =
                __builtin_amdgcn_raw_buffer_load_b64(act, st.voff, so, 0);
            p[i][0] = x[0];
            p[i][1] = x[1];
        } else {
            p[i][0] = __builtin_amdgcn_raw_buffer_load_b32(act, st.voff, so, 0);
        }
    }
}

// Steps [t0, t1) over A activation planes (byte offsets ap within a pixel)
// and W filter planes (byte offsets wp within a tap) for the C channels from
// filter byte offset ch0: adds to the lane's tile row (or, with `first`, sets
// it to)
//   add + sum_ij scale pa[i] pw[j] popcount(a_i AND w_j)
//       + csa sum_i pa[i] popcount(a_i).
template <int A, int W, int CB, int C, bool XN, bool ONES>
__device__ __forceinline__ void reduce(
    uint32_t* trow, bool first, uint32_t add, const TiledArgs& g,
    const Window& win, Rsrc act, v4i rw, int t0, int t1,
    const uint32_t (&ap)[A], const uint32_t (&wp)[W], uint32_t ch0,
    const int (&pa)[A], const int (&pw)[W], int scale, int csa) {
    constexpr int SC = slice_channels<W, CB, C>();
    constexpr int NSL = C / SC;
    static_assert(NSL % 2 == 0, "slice buffers alternate within a step");
    const uint32_t ch_bytes =
        4u * (uint32_t)(g.kh * g.kw) * (uint32_t)(g.wbits * g.cw);
    const uint32_t tap_bytes = 4u * (uint32_t)(g.wbits * g.cw);
    uint32_t acc[C][A][W];
#pragma unroll
    for (int o = 0; o < C; ++o)
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int j = 0; j < W; ++j) acc[o][i][j] = 0;

    uint32_t sa = 0;
    Step st;
    const int tap = (int)g.div_nch.div((uint32_t)t0);
    st.r = (int)g.div_kw.div((uint32_t)tap);
    st.s = tap - st.r * g.kw;
    st.c0 = (t0 - tap * g.nch) * CB;
    st.cs = min(st.c0, g.cw - CB);
    set_tap<CB>(st, g, win);

    uint32_t p[A][CB], pn[A][CB];
    Slice<W, CB, SC> f[2];
    load_words<A, CB, ONES>(p, act, st, ap);
    uint32_t fbase = ch0 + (uint32_t)(st.r * g.kw + st.s) * tap_bytes +
                     4u * (uint32_t)st.cs;
    load_slice<W, CB, SC>(f[0], rw, fbase, ch_bytes, wp);

    // a step's first filter slice is in (or on its way to) f[0]; the next
    // step's words and first slice are requested on the way (for the last
    // step, its own again)
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
        const int dup = st.c0 - st.cs;       // words the last chunk counted
        [[maybe_unused]] const bool in = st.in;
        if (t + 1 < t1) next_step<CB>(st, g, win);
        load_words<A, CB, ONES>(pn, act, st, ap);
        const uint32_t fnext = ch0 +
                               (uint32_t)(st.r * g.kw + st.s) * tap_bytes +
                               4u * (uint32_t)st.cs;
        if (dup > 0) {
#pragma unroll
            for (int k = 0; k < CB; ++k) {
                const uint32_t m = k < dup ? 0u : ~0u;
#pragma unroll
                for (int i = 0; i < A; ++i) p[i][k] &= m;
            }
        }
        if (csa != 0) {
#pragma unroll
            for (int i = 0; i < A; ++i) {
                uint32_t n = 0;
#pragma unroll
                for (int k = 0; k < CB; ++k)
                    n += (uint32_t)__builtin_popcount(p[i][k]);
                sa += (uint32_t)__mul24((int)n, pa[i]);
            }
        }
        [[maybe_unused]] uint32_t keep[CB];
        if constexpr (XN) {
#pragma unroll
            for (int k = 0; k < CB; ++k)
                keep[k] = in && k >= dup ? ~0u : 0u;
        }
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) {
            pix::wait_scalar_loads();
            if (sl + 1 < NSL)
                load_slice<W, CB, SC>(
                    f[(sl + 1) & 1], rw,
                    fbase + (uint32_t)((sl + 1) * SC) * ch_bytes, ch_bytes,
                    wp);
            else
                load_slice<W, CB, SC>(f[0], rw, fnext, ch_bytes, wp);
            __builtin_amdgcn_sched_barrier(0);
            const Slice<W, CB, SC>& fs = f[sl & 1];
#pragma unroll
            for (int k = 0; k < CB; ++k)
#pragma unroll
                for (int j = 0; j < W; ++j)
#pragma unroll
                    for (int i = 0; i < A; ++i)
#pragma unroll
                        for (int o = 0; o < SC; ++o) {
                            uint32_t& n = acc[sl * SC + o][i][j];
                            if constexpr (XN)
                                pix::bcnt_acc(n, pix::xor_keep(
                                                     p[i][k], keep[k],
                                                     fs.w[o][j][k]));
                            else
                                pix::and_bcnt_acc<false>(n, p[i][k],
                                                         fs.w[o][j][k]);
                        }
            __builtin_amdgcn_sched_barrier(0);
        }
        fbase = fnext;
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int k = 0; k < CB; ++k) p[i][k] = pn[i][k];
    }
    if (csa != 0) add += (uint32_t)csa * sa;
#pragma unroll
    for (int o = 0; o < C; ++o) {
        uint32_t v = add;
        if (!first) v += trow[o];
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int j = 0; j < W; ++j)
                v += (uint32_t)__mul24((int)acc[o][i][j],
                                       scale * pa[i] * pw[j]);
        trow[o] = v;
    }
}

template <int A, int W, int CB, int C, bool XN, bool REQ>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_num_sgpr(96)))
void conv_generic_kernel_tiled(const uint32_t* __restrict__ act,
                               const uint32_t* __restrict__ wts,
                               int32_t* __restrict__ out, TiledArgs g) {
    static_assert(!XN || A == 1, "+-1 activations");
    __shared__ uint32_t lds[kWaves * kTileWords];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ks = wv & ((1 << g.ks_log2) - 1);
    const int u = pix::xcd_block() * (kWaves >> g.ks_log2) +
                  (wv >> g.ks_log2);
    const bool live = u < g.units;
    uint32_t* tile = lds + wv * kTileWords;
    const int grp = (int)g.div_cols.div((uint32_t)(live ? u : 0));
    const int col0 = ((live ? u : 0) - grp * (int)g.div_cols.d) * g.unit_cols;
    const int pix0 = grp * 64;

    if (live) {
        const Rsrc ract = pix::make_rsrc(act, g.act_bytes);
        v4i rw;
        rw[0] = (int)(uint32_t)(uintptr_t)wts;
        rw[1] = (int)((uint32_t)((uintptr_t)wts >> 32) & 0xFFFFu);
        rw[2] = g.wt_bytes;
        rw[3] = pix::kRsrcWord3;
        const uint32_t p = (uint32_t)min(pix0 + lane, g.npix - 1);
        const uint32_t row = g.div_ow.div(p);
        const int ox = (int)(p - row * (uint32_t)g.ow);
        const uint32_t img = g.div_oh.div(row);
        const int oy = (int)(row - img * (uint32_t)g.oh);
        Window win;
        win.iy0 = oy * g.sh - g.ph;
        win.ix0 = ox * g.sw - g.pw;
        win.base = ((img * (uint32_t)g.h + (uint32_t)win.iy0) *
                        (uint32_t)g.w + (uint32_t)win.ix0) *
                   (4u * (uint32_t)(g.abits * g.cw));
        // the term of the window's in-range channel values
        uint32_t konst = 0;
        if (g.cn != 0 && ks == 0) {
            const int nr = max(min(win.iy0 + g.kh, g.h) - max(win.iy0, 0), 0);
            const int nc = max(min(win.ix0 + g.kw, g.w) - max(win.ix0, 0), 0);
            konst = (uint32_t)g.cn * (uint32_t)(nr * nc) * (uint32_t)g.c;
        }
        // this wave's steps (at least one: the host shares them out so)
        const int t0 = (int)((int64_t)g.nsteps * ks >> g.ks_log2);
        const int t1 = (int)((int64_t)g.nsteps * (ks + 1) >> g.ks_log2);
        const uint32_t ch_bytes =
            4u * (uint32_t)(g.kh * g.kw) * (uint32_t)(g.wbits * g.cw);
#pragma unroll 1
        for (int sub = 0; sub < g.nsub; ++sub) {
            uint32_t* trow = tile + lane * kStride + sub * C;
            bool first = true;
            const uint32_t ch0 = (uint32_t)(col0 + sub * C) * ch_bytes;
#pragma unroll 1
            for (int wg = 0; wg < g.wt_groups; ++wg) {
                uint32_t wp[W];
                int pw[W];
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    pw[j] = g.pw8[wg * W + j];
                    wp[j] =
                        4u * (uint32_t)(min(wg * W + j, g.wbits - 1) * g.cw);
                }
#pragma unroll 1
                for (int ag = 0; ag < g.act_groups; ++ag) {
                    uint32_t ap[A];
                    int pa[A];
#pragma unroll
                    for (int i = 0; i < A; ++i) {
                        pa[i] = g.pa[ag * A + i];
                        ap[i] = 4u * (uint32_t)(
                                    min(ag * A + i, g.abits - 1) * g.cw);
                    }
                    reduce<A, W, CB, C, XN, false>(
                        trow, first, first ? konst : 0u, g, win, ract, rw, t0,
                        t1, ap, wp, ch0, pa, pw, g.cs, wg == 0 ? g.csa : 0);
                    first = false;
                }
                if constexpr (!XN) {
                    if (g.csw != 0) {
                        const uint32_t none[1] = {0};
                        const int one[1] = {1};
                        reduce<1, W, CB, C, false, true>(
                            trow, false, 0u, g, win, ract, rw, t0, t1, none,
                            wp, ch0, one, pw, g.csw, 0);
                    }
                }
            }
        }
    }
    // the unit's tiles: one per wave that took part of its steps
    if (g.ks_log2 > 0) __syncthreads();
    else pix::wave_lds_sync();
    if (!live) return;
    const int nks = 1 << g.ks_log2;
    const uint32_t* t = lds + (wv - ks) * kTileWords;
    // N consecutive channels of one pixel, summed over the unit's waves
    auto values = [&](auto& v, int row, int col) __attribute__((always_inline)) {
        constexpr int N = sizeof(v) / sizeof(v[0]);
        const uint32_t* e = t + row * kStride + col;
#pragma unroll
        for (int o = 0; o < N; ++o) v[o] = e[o];
#pragma unroll 1
        for (int k = 1; k < nks; ++k) {
            e += kTileWords;
#pragma unroll
            for (int o = 0; o < N; ++o) v[o] += e[o];
        }
    };
    const int cols = g.unit_cols;
    if constexpr (REQ) {
        // lane = pixel; 8 channels make one byte of each plane
        const int p = pix0 + lane;
        const int last = (g.oc + 7) / 8 - 1;
        for (int b8 = ks; b8 < cols / 8; b8 += nks) {
            const int k8 = col0 / 8 + b8;
            if (k8 > last) break;
            uint32_t codes[2] = {0, 0};
            uint32_t v[8];
            values(v, lane, b8 * 8);
#pragma unroll
            for (int o = 0; o < 8; ++o)
                codes[o >> 2] = quant_insert(
                    (float)(int32_t)v[o], g.out_scale, g.out_qmax,
                    (uint32_t)(o & 3), codes[o >> 2]);
            // channels past the last one have code 0
            const int n = g.oc - 8 * k8;
            if (n < 8) codes[1] &= n > 4 ? ~0u >> 8 * (8 - n) : 0u;
            if (n < 4) codes[0] &= ~0u >> 8 * (4 - n);
            if (p >= g.npix) continue;
            uint8_t* dst = reinterpret_cast<uint8_t*>(out) +
                           (size_t)p * (uint32_t)(4 * g.out_bits *
                                                  g.out_words) +
                           (uint32_t)k8;
            // the last byte also clears the rest of its word
            const int pad = k8 == last ? 3 - (k8 & 3) : 0;
            for (int b = 0; b < g.out_bits; ++b) {
                uint8_t* d = dst + (size_t)b * (uint32_t)(4 * g.out_words);
                d[0] = (uint8_t)plane_byte(codes[0], codes[1], b);
                for (int z = 1; z <= pad; ++z) d[z] = 0;
            }
        }
    } else {
        const Rsrc rout = pix::make_rsrc(out, g.out_bytes);
        if (g.ch_step != 1) {
            // channel rows: 64 consecutive results per store
            const int p = pix0 + lane;
            for (int c = ks; c < cols; c += nks) {
                uint32_t v[1];
                values(v, lane, c);
                const bool in = p < g.npix && col0 + c < g.oc;
                const uint32_t off =
                    4u * ((uint32_t)(col0 + c) * (uint32_t)g.ch_step +
                          (uint32_t)p);
                __builtin_amdgcn_raw_buffer_store_b32(
                    v[0], rout, in ? off : kOutOfRange, 0, 0);
            }
        } else if (g.oc % 4 == 0 || col0 + cols <= g.oc) {
            // whole quads of channels (dword-aligned 16-byte stores)
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const int nq = cols >> 2;            // quads per pixel: 1, 2, 4
            const int lg = nq == 4 ? 2 : nq == 2 ? 1 : 0;
            const int q = lane & (nq - 1), pr = lane >> lg;
            for (int r = ks; r < nq; r += nks) {
                const int rowi = r * (64 >> lg) + pr, p = pix0 + rowi;
                uint32_t x[4];
                values(x, rowi, 4 * q);
                const u32x4 v = {x[0], x[1], x[2], x[3]};
                const bool in = p < g.npix && col0 + 4 * q < g.oc;
                const uint32_t off =
                    4u * ((uint32_t)p * (uint32_t)g.pix_step +
                          (uint32_t)(col0 + 4 * q));
                __builtin_amdgcn_raw_buffer_store_b128(
                    v, rout, in ? off : kOutOfRange, 0, 0);
            }
        } else {
            const int lg = cols == 16 ? 4 : cols == 8 ? 3 : 2;
            const int c = lane & (cols - 1), pr = lane >> lg;
            for (int r = ks; r < cols; r += nks) {
                const int rowi = r * (64 >> lg) + pr, p = pix0 + rowi;
                uint32_t v[1];
                values(v, rowi, c);
                const bool in = p < g.npix && col0 + c < g.oc;
                const uint32_t off = 4u * ((uint32_t)p * (uint32_t)g.pix_step +
                                           (uint32_t)(col0 + c));
                __builtin_amdgcn_raw_buffer_store_b32(
                    v[0], rout, in ? off : kOutOfRange, 0, 0);
            }
        }
    }
}

using TiledKernelFn = void (*)(const uint32_t*, const uint32_t*, int32_t*,
                               TiledArgs);

// Kernel for A x W planes at a time, chunks of cb words, c channels per
// accumulator tile (max_channels or 4); xnor: +-1 activations.
template <int A>
TiledKernelFn pick_a(int w, int cb, int c, bool xnor, bool req);
template <> TiledKernelFn pick_a<1>(int, int, int, bool, bool);
template <> TiledKernelFn pick_a<2>(int, int, int, bool, bool);
template <> TiledKernelFn pick_a<3>(int, int, int, bool, bool);
template <> TiledKernelFn pick_a<4>(int, int, int, bool, bool);

template <int A, int W, int CB, bool XN>
TiledKernelFn pick_c(int c, bool req) {
    constexpr int M = max_channels(A, W);
    if (c == 4)
        return req ? conv_generic_kernel_tiled<A, W, CB, 4, XN, true>
                   : conv_generic_kernel_tiled<A, W, CB, 4, XN, false>;
    if (c == M)
        return req ? conv_generic_kernel_tiled<A, W, CB, M, XN, true>
                   : conv_generic_kernel_tiled<A, W, CB, M, XN, false>;
    return nullptr;
}

template <int A, int W, bool XN>
TiledKernelFn pick_cb(int cb, int c, bool req) {
    switch (cb) {
        case 1: return pick_c<A, W, 1, XN>(c, req);
        case 2: return pick_c<A, W, 2, XN>(c, req);
        case 3: return pick_c<A, W, 3, XN>(c, req);
        default: return pick_c<A, W, 4, XN>(c, req);
    }
}

template <int A>
TiledKernelFn pick_for_a(int w, int cb, int c, bool xnor, bool req) {
    if constexpr (A == 1)
        if (xnor) switch (w) {
                case 1: return pick_cb<1, 1, true>(cb, c, req);
                case 2: return pick_cb<1, 2, true>(cb, c, req);
                case 3: return pick_cb<1, 3, true>(cb, c, req);
                default: return pick_cb<1, 4, true>(cb, c, req);
            }
    switch (w) {
        case 1: return pick_cb<A, 1, false>(cb, c, req);
        case 2: return pick_cb<A, 2, false>(cb, c, req);
        case 3: return pick_cb<A, 3, false>(cb, c, req);
        default: return pick_cb<A, 4, false>(cb, c, req);
    }
}

// ---- host side (conv_tiled.hip) --------------------------------------------

// True when the kernel covers the shape (sizes within its 32-bit offsets);
// req: with requantized, packed output.
bool covers(const ConvShape& s, bool req);

// True for a matrix product (1x1, stride 1, no padding) with so few rows that
// most lanes would idle with pixels on the lanes: the call then runs with
// the operands' roles exchanged, output channels on the lanes.
bool prefer_swapped(const ConvShape& s);

// Launches the kernel (covers() must hold); cus: the device's compute units.
hipError_t launch_conv(const ConvShape& s, const uint32_t* act,
                       const uint32_t* wts, int32_t* out, const Requant* rq,
                       int cus, hipStream_t st);

// The launch as text (snprintf semantics); enc names the encodings.
int describe(const ConvShape& s, const char* enc, int cus, char* buf,
             size_t len);

}  // namespace tiled
}  // namespace bs
