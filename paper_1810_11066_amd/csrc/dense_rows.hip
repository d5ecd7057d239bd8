// Matrix products of few rows (out[r][o] = sum_k value(a[r][k]) value(w[o][k]),
// bs_dense and 1x1 convs of few pixels): the reduction across the lanes.
//
// With pixels (or output channels) on the lanes such a product leaves most
// lanes without work, or reads every lane's operand row at a stride, and a
// wave walks the whole reduction alone.  Here lane l takes words l, l + 64, ..
// of every plane, so the loads of an operand row are consecutive words, and a
// wave computes a tile of R rows x NB output channels whose A x W popcounts
// per output it keeps in registers; one cross-lane sum per output ends it.
//
// What bounds it: reading the weights once (one row), latency otherwise.  A
// wave has the NB W + R A loads of a chunk in flight at once, two chunks
// deep.  One row of 4096 x 4096 at A2W2 takes 4.2 us a launch (13.1 us with
// pixels on the lanes), about what an empty launch takes; dense_rows.h has the
// other sizes.
//
// The encodings' corrections are sums over the words too (conv_tiled.h names
// them), so they are added per lane before the cross-lane sum.
#include <cstdio>

#include "bs_internal.h"
#include "conv_pix.h"
#include "dense_rows.h"

namespace bs {
namespace rows {
namespace {

using pix::kOutOfRange;
using pix::Rsrc;

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

struct RowsArgs {
    int32_t m, n;          // rows, output channels
    int32_t cw, c;         // words per plane, values per row
    int32_t abits, wbits;
    int32_t act_groups, wt_groups;
    int32_t act_bytes, wt_bytes, out_bytes;
    int32_t pa[8], pw[8];  // plane weights, 0 past the last plane
    int32_t cs, csa, csw, cn;
    int32_t tiles_n;       // tiles along n
    int32_t tiles;
    FastDiv div_tiles;
};

// Sum over the 64 lanes of four values: row 0 of the result (lanes 0-15)
// holds v0's, row 1 v2's, row 2 v1's and row 3 v3's, in every lane.
// permlane32_swap exchanges the upper half of its first operand with the
// lower half of its second, permlane16_swap the odd 16-lane rows of the first
// with the even ones of the second, so each swap and add halves two values
// into one register.
template <int CTRL>
__device__ __forceinline__ uint32_t add_dpp(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF,
                                                     true);
}

__device__ __forceinline__ uint32_t sum4(uint32_t v0, uint32_t v1, uint32_t v2,
                                         uint32_t v3) {
    const auto a = __builtin_amdgcn_permlane32_swap(v0, v1, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(v2, v3, false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0] + a[1], b[0] + b[1],
                                                    false, false);
    uint32_t s = c[0] + c[1];
    s = add_dpp<0x128>(s);     // row_ror:8
    s = add_dpp<0x124>(s);     // row_ror:4
    s = add_dpp<0x122>(s);     // row_ror:2
    return add_dpp<0x121>(s);  // row_ror:1
}

template <int A, int W, int R, int NB, bool XN>
__global__ __launch_bounds__(kBlock) void dense_rows_kernel(
    const uint32_t* __restrict__ act, const uint32_t* __restrict__ wts,
    int32_t* __restrict__ out, RowsArgs g) {
    static_assert(R * NB % 4 == 0, "outputs are summed four at a time");
    constexpr int V = R * NB;
    const int lane = threadIdx.x & 63;
    const int tile = __builtin_amdgcn_readfirstlane(
        (int)(blockIdx.x * kWaves + (threadIdx.x >> 6)));
    if (tile >= g.tiles) return;
    const int tr = (int)g.div_tiles.div((uint32_t)tile);
    const int r0 = tr * R, n0 = (tile - tr * g.tiles_n) * NB;
    const Rsrc ra = pix::make_rsrc(act, g.act_bytes);
    const Rsrc rw = pix::make_rsrc(wts, g.wt_bytes);
    uint32_t total[V];
#pragma unroll
    for (int v = 0; v < V; ++v) total[v] = 0;

#pragma unroll 1
    for (int wg = 0; wg < g.wt_groups; ++wg) {
#pragma unroll 1
        for (int ag = 0; ag < g.act_groups; ++ag) {
            uint32_t acc[V][A][W];
            uint32_t sa[R], sw[NB];
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int i = 0; i < A; ++i)
#pragma unroll
                    for (int j = 0; j < W; ++j) acc[v][i][j] = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) sa[r] = 0;
#pragma unroll
            for (int o = 0; o < NB; ++o) sw[o] = 0;
#pragma unroll 2
            for (int t = lane; t - lane < g.cw; t += 64) {
                // words past the plane, rows past m and channels past n load
                // out of range and read zeros
                const bool in = t < g.cw;
                uint32_t a[R][A], w[NB][W];
#pragma unroll
                for (int o = 0; o < NB; ++o)
#pragma unroll
                    for (int j = 0; j < W; ++j) {
                        const int pl = wg * W + j;
                        const uint32_t off =
                            4u * (uint32_t)(((n0 + o) * g.wbits +
                                             min(pl, g.wbits - 1)) * g.cw + t);
                        w[o][j] = __builtin_amdgcn_raw_buffer_load_b32(
                            rw, in && n0 + o < g.n ? off : kOutOfRange, 0, 0);
                    }
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int i = 0; i < A; ++i) {
                        const int pl = ag * A + i;
                        const uint32_t off =
                            4u * (uint32_t)(((r0 + r) * g.abits +
                                             min(pl, g.abits - 1)) * g.cw + t);
                        a[r][i] = __builtin_amdgcn_raw_buffer_load_b32(
                            ra, in && r0 + r < g.m ? off : kOutOfRange, 0, 0);
                    }
                if (g.csa != 0 && wg == 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int i = 0; i < A; ++i)
                            sa[r] += (uint32_t)__mul24(
                                __builtin_popcount(a[r][i]), g.pa[ag * A + i]);
                }
                if (g.csw != 0 && ag == 0) {
#pragma unroll
                    for (int o = 0; o < NB; ++o)
#pragma unroll
                        for (int j = 0; j < W; ++j)
                            sw[o] += (uint32_t)__mul24(
                                __builtin_popcount(w[o][j]), g.pw[wg * W + j]);
                }
#pragma unroll
                for (int o = 0; o < NB; ++o)
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int i = 0; i < A; ++i)
#pragma unroll
                            for (int j = 0; j < W; ++j)
                                pix::bcnt_acc(acc[o * R + r][i][j],
                                              XN ? a[r][i] ^ w[o][j]
                                                 : a[r][i] & w[o][j]);
            }
#pragma unroll
            for (int o = 0; o < NB; ++o)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    uint32_t s = total[o * R + r];
#pragma unroll
                    for (int i = 0; i < A; ++i)
#pragma unroll
                        for (int j = 0; j < W; ++j)
                            s += (uint32_t)__mul24(
                                (int)acc[o * R + r][i][j],
                                g.cs * g.pa[ag * A + i] * g.pw[wg * W + j]);
                    s += (uint32_t)g.csa * sa[r] + (uint32_t)g.csw * sw[o];
                    total[o * R + r] = s;
                }
        }
    }
    // output v = 4 q + {0, 2, 1, 3}[lane / 16] ends in register q; lane
    // 16 x + q stores that of its row x
    const int lq = lane & 15, x = lane >> 4;
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < V / 4; ++q) {
        const uint32_t s = sum4(total[4 * q], total[4 * q + 1],
                                total[4 * q + 2], total[4 * q + 3]);
        mine = lq == q ? s : mine;
    }
    const int v = 4 * lq + ((x & 1) << 1 | x >> 1);
    const int o = v / R, r = v - o * R;
    const bool in = lq < V / 4 && r0 + r < g.m && n0 + o < g.n;
    const uint32_t off = 4u * (uint32_t)((r0 + r) * g.n + n0 + o);
    const Rsrc ro = pix::make_rsrc(out, g.out_bytes);
    __builtin_amdgcn_raw_buffer_store_b32(
        mine + (uint32_t)g.cn * (uint32_t)g.c, ro, in ? off : kOutOfRange, 0,
        0);
}

using Fn = void (*)(const uint32_t*, const uint32_t*, int32_t*, RowsArgs);

// Rows per wave for products of more than two rows: the A x W counters of
// R x 4 outputs within 64 registers.
constexpr int wide_rows(int a, int w) {
    return a * w <= 4 ? 4 : a * w <= 8 ? 2 : 1;
}
constexpr int kTileCols = 4;

template <int A, int W>
Fn pick_r(int r, bool xnor) {
    constexpr int R = wide_rows(A, W);
    if constexpr (A == 1 && W == 1)
        if (xnor)
            return r == 1 ? dense_rows_kernel<1, 1, 1, kTileCols, true>
                          : dense_rows_kernel<1, 1, R, kTileCols, true>;
    return r == 1 ? dense_rows_kernel<A, W, 1, kTileCols, false>
                  : dense_rows_kernel<A, W, R, kTileCols, false>;
}

template <int A>
Fn pick_w(int w, int r, bool xnor) {
    switch (w) {
        case 1: return pick_r<A, 1>(r, xnor);
        case 2: return pick_r<A, 2>(r, xnor);
        case 3: return pick_r<A, 3>(r, xnor);
        default: return pick_r<A, 4>(r, xnor);
    }
}

Fn pick(int a, int w, int r, bool xnor) {
    switch (a) {
        case 1: return pick_w<1>(w, r, xnor);
        case 2: return pick_w<2>(w, r, xnor);
        case 3: return pick_w<3>(w, r, xnor);
        default: return pick_w<4>(w, r, xnor);
    }
}

// Rows of a wave's tile.
int tile_rows(const ConvShape& s) {
    return (int64_t)s.n * s.oh * s.ow <= 2
               ? 1
               : wide_rows(group_planes(s.abits), group_planes(s.wbits));
}

struct Plan {
    Fn fn;
    RowsArgs g;
    dim3 grid;
    int a, w, r;
};

Plan make_plan(const ConvShape& s) {
    Plan pl{};
    RowsArgs& g = pl.g;
    const int cw = (s.c + 31) / 32;
    pl.a = group_planes(s.abits);
    pl.w = group_planes(s.wbits);
    const Encoding e = encoding_terms(s);
    g.m = s.n * s.oh * s.ow;
    g.n = s.oc;
    g.cw = cw;
    g.c = s.c;
    g.abits = s.abits;
    g.wbits = s.wbits;
    g.act_groups = plane_groups(s.abits);
    g.wt_groups = plane_groups(s.wbits);
    g.act_bytes = (int32_t)((int64_t)g.m * s.abits * cw * 4);
    g.wt_bytes = (int32_t)((int64_t)g.n * s.wbits * cw * 4);
    g.out_bytes = (int32_t)((int64_t)g.m * g.n * 4);
    plane_weights(s.abits, s.aenc, g.pa);
    plane_weights(s.wbits, s.wenc, g.pw);
    g.cs = e.cs; g.csa = e.csa; g.csw = e.csw; g.cn = e.cn;
    pl.r = tile_rows(s);
    g.tiles_n = (g.n + kTileCols - 1) / kTileCols;
    g.tiles = g.tiles_n * ((g.m + pl.r - 1) / pl.r);
    g.div_tiles.init((uint32_t)g.tiles_n);
    pl.fn = pick(pl.a, pl.w, pl.r, e.xnor);
    pl.grid = dim3((uint32_t)((g.tiles + kWaves - 1) / kWaves));
    return pl;
}

// Waves per SIMD up to which the kernel is the faster one.  A wave's tile ends
// with a cross-lane sum per output and reads each weight word for R rows only,
// so with many tiles of short rows (large n) the kernels with pixels or output
// channels on the lanes win.
//
// pixel: the pixel kernel would serve the call.  It leaves most lanes idle and
// takes as long for 1 row as for 64, so the rows count.  Rate against it, at
// waves per SIMD: k = 1024, 16 rows, A2W2 1.23 at 2, 0.93 at 4, A4W4 1.45 at 8,
// 0.85 at 16; 9 rows A2W2 1.09 at 3, A4W4 1.32 at 9, 1.10 at 36; 8 rows A2W2 1.23
// at 32; one bit a pair, 8 rows, 0.98 at 2, 0.94 at 4; k = 2048, 16 rows, one bit
// 1.06 at 4, 0.97 at 8, A2W1 1.09 at 32; k = 4096, 32 rows, one bit 1.02 at 12,
// 0.88 at 16, A2W1 1.12 at 16, 0.88 at 64, A4W4 1.23 at 32, 1.00 at 64; 24 rows,
// one bit 1.01 at 24, 0.87 at 48, A4W4 1.21 at 96.
//
// Otherwise the tiled kernel would, with the output channels on the lanes: k =
// 768, 16 rows, A2W2 1.25 at 2, 0.96 at 4, 0.63 at 8, A4W4 1.10 at 8, 0.65 at 16;
// k = 1024, A8W8 1.25 at 4.5, 0.85 at 8; k = 3072, 32 rows, A2W1 1.02 at 6, 0.85
// at 8, A4W4 1.46 at 8, 0.94 at 17; k = 4096 A8W8 1.13 at 17, 0.91 at 24.  One row
// leaves its lanes idle: k = 768 A2W2 1.04 at 8, 0.74 at 16.
int waves_per_simd(const ConvShape& s, int m, int cw, int rows, bool pixel) {
    constexpr int kAny = 1 << 20;
    const bool wide = rows == 4;
    if (pixel) {
        if (s.abits * s.wbits == 1)
            return m <= 4 ? kAny : cw < 64 ? 2 : cw < 128 ? 4
                                 : m > 24 ? 12 : m > kFewRows ? 24 : kAny;
        if (m <= (wide ? 8 : 10)) return kAny;
        if (cw < 64) return wide ? 3 : 8;
        if (m <= (wide ? kFewRows : 24)) return kAny;
        return wide ? 32 : 64;
    }
    if (m <= 2) return cw < 96 ? 8 : 64;
    if (cw < 64) return wide ? 2 : cw < 32 ? 8 : 6;
    if (cw < 96) return wide ? 4 : 8;
    if (cw < 128) return wide ? 6 : 12;
    return !wide ? 20 : m > kFewRows ? 12 : 16;
}

}  // namespace

bool covers(const ConvShape& s, int cus, bool pixel) {
    if (s.kh != 1 || s.kw != 1 || s.sh != 1 || s.sw != 1 || s.ph || s.pw)
        return false;
    const int64_t m = (int64_t)s.n * s.oh * s.ow, cw = (s.c + 31) / 32;
    if (!(m <= kFewRows && cw >= kFewWords) &&
        !(m <= kMoreRows && cw >= kMoreWords))
        return false;
    const int r = tile_rows(s);
    const int64_t waves =
        (m + r - 1) / r * (((int64_t)s.oc + kTileCols - 1) / kTileCols);
    if (waves >
        (int64_t)waves_per_simd(s, (int)m, (int)cw, r, pixel) * 4 * cus)
        return false;
    // popcounts are folded as 24-bit values
    if (s.c >= 1 << 23) return false;
    return (int64_t)s.oc * s.wbits * cw * 4 <= pix::kMaxBufferBytes &&
           m * s.abits * cw * 4 <= pix::kMaxBufferBytes &&
           m * s.oc * 4 <= pix::kMaxBufferBytes;
}

hipError_t launch_rows(const ConvShape& s, const uint32_t* act,
                       const uint32_t* wts, int32_t* out, hipStream_t st) {
    const Plan pl = make_plan(s);
    return launch(pl.fn, pl.grid, dim3(kBlock), 0, st, act, wts, out, pl.g);
}

int describe(const ConvShape& s, const char* enc, char* buf, size_t len) {
    const Plan pl = make_plan(s);
    return snprintf(buf, len,
                    "dense_rows_kernel<A=%d,W=%d,R=%d,NB=%d> A=%d W=%d %s "
                    "grid=%u block=%d tiles=%d",
                    pl.a, pl.w, pl.r, kTileCols, s.abits, s.wbits, enc,
                    pl.grid.x, kBlock, pl.g.tiles);
}

}  // namespace rows
}  // namespace bs
