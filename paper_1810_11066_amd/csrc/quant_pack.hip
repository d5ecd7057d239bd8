// Quantize and bit-pack kernels for gfx950 (wave64).
//
// quantize       float32 -> uint8 codes (Sec. 3.1 quantization operator)
// pack           uint8 codes -> bit-planes packed into uint32 words along the
//                reduction axis, layout [rows][bits][ceil(k/32)] (Sec. 2.2,
//                Sec. 3.1, MBK')
// quantize_pack  both in one pass over the float32 data
//
// All three stream HBM once and do a few integer ops per element, so they
// are bound by memory bandwidth.  Every load is a 16-byte vector load with
// consecutive lanes reading consecutive addresses; the bits of one packed
// word are gathered in registers and joined across lanes with DPP ORs (or
// wave ballots in the any-k fallback).
//
// Inputs are read once, with non-temporal loads: they do not push out of the
// caches what the surrounding kernels leave there -- in particular the int32
// output of a preceding convolution, whose write-back to HBM then overlaps
// the next convolution (bound by the vector ALUs) instead of this kernel.
// Measured on the ResNet-18 layers at batch 128: quantize+pack+conv steps
// 4-17 % shorter.
#include <type_traits>

#include "bs_internal.h"

namespace bs {
namespace {

__device__ __forceinline__ uint4 stream_load(const uint4* p) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 t =
        __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ float4 stream_load(const float4* p) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 t =
        __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    return make_float4(t[0], t[1], t[2], t[3]);
}

constexpr int kBlock = 256;
constexpr int kMaxBlocks = 8192;

// ENC: kUnipolar, kBipolar or kSigned (qmax as for quant_code_enc)
template <int ENC>
__device__ __forceinline__ uint32_t code_of(float x, float scale, float qmax) {
    return quant_code_enc<ENC>(x, scale, qmax);
}

template <int ENC>
__device__ __forceinline__ uint32_t codes4(float4 f, float scale, float qmax) {
    if constexpr (ENC == kUnipolar) {
        uint32_t c4 = quant_insert(f.x, scale, qmax, 0, 0u);
        c4 = quant_insert(f.y, scale, qmax, 1, c4);
        c4 = quant_insert(f.z, scale, qmax, 2, c4);
        return quant_insert(f.w, scale, qmax, 3, c4);
    }
    return code_of<ENC>(f.x, scale, qmax) |
           (code_of<ENC>(f.y, scale, qmax) << 8) |
           (code_of<ENC>(f.z, scale, qmax) << 16) |
           (code_of<ENC>(f.w, scale, qmax) << 24);
}

// ---------------------------------------------------------------------------
// quantize: 16 elements per thread per step (four 16-byte loads, one 16-byte
// store); the n % 16 tail is done one element per thread.
template <int ENC>
__global__ __launch_bounds__(kBlock) void quantize_kernel(
    const float* __restrict__ x, uint8_t* __restrict__ q, int64_t n,
    float scale, float qmax) {
    const int64_t nvec = n >> 4;
    const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t nthr = (int64_t)gridDim.x * kBlock;
    const float4* xv = reinterpret_cast<const float4*>(x);
    uint4* qv = reinterpret_cast<uint4*>(q);
    for (int64_t v = tid; v < nvec; v += nthr) {
        float4 f0 = stream_load(xv + 4 * v + 0);
        float4 f1 = stream_load(xv + 4 * v + 1);
        float4 f2 = stream_load(xv + 4 * v + 2);
        float4 f3 = stream_load(xv + 4 * v + 3);
        qv[v] = make_uint4(codes4<ENC>(f0, scale, qmax),
                           codes4<ENC>(f1, scale, qmax),
                           codes4<ENC>(f2, scale, qmax),
                           codes4<ENC>(f3, scale, qmax));
    }
    const int64_t tail = nvec << 4;
    if (tid < n - tail)
        q[tail + tid] = (uint8_t)code_of<ENC>(x[tail + tid], scale, qmax);
}

// ---------------------------------------------------------------------------
// Cross-lane OR with a DPP lane permutation (all source lanes are inside the
// 8-lane group, so every lane reads a defined value).
constexpr int kDppQuadXor1 = 0xB1;     // quad_perm [1,0,3,2]: lane ^ 1
constexpr int kDppQuadXor2 = 0x4E;     // quad_perm [2,3,0,1]: lane ^ 2
constexpr int kDppHalfMirror = 0x141;  // row_half_mirror: lane i <-> 7 - i

template <int CTRL>
__device__ __forceinline__ uint32_t or_dpp(uint32_t v) {
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF,
                                                     false);
}

// pack, k % 32 == 0: a wave packs 128 consecutive words of the flat
// [rows][k / 32] word array (4096 codes, which never split a word across
// rows).  Load j (0..3) reads 16 codes per lane, lanes consecutive, so every
// load is one coalesced 1 KiB.  Lanes 2p, 2p+1 of load j hold the two halves
// of word 32 j + p: each gathers its 16 bits of plane b in registers and one
// DPP OR joins the halves.  Lane 2p + i keeps word 32 j + p when j % 2 == i
// (slot j / 2); one ds_bpermute per plane and slot then moves word w to lane
// w % 64, so the stores write 64 consecutive words.
template <int A>
__global__ __launch_bounds__(kBlock) void pack_dpp_kernel(
    const uint8_t* __restrict__ q, uint32_t* __restrict__ packed,
    uint32_t nwords, FastDiv kwdiv) {
    const int lane = threadIdx.x & 63;
    const uint32_t kw = kwdiv.d;
    const uint4* src = reinterpret_cast<const uint4*>(q);
    const uint32_t wave0 = (blockIdx.x * kBlock + threadIdx.x) >> 6;
    const uint32_t nwaves = (gridDim.x * kBlock) >> 6;
    // lane l's words (l and 64 + l of the chunk) come from lane 2 (l % 32) +
    // l / 32, which holds them in slots 0 and 1
    const int from = (2 * (lane & 31) + (lane >> 5)) * 4;
    for (uint32_t base = wave0 * 128u; base < nwords; base += nwaves * 128u) {
        const uint32_t left = nwords - base;
        uint4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // this lane's 16 codes belong to word 32 j + lane / 2
            const bool ok = (uint32_t)(32 * j + (lane >> 1)) < left;
            v[j] = ok ? stream_load(src + (size_t)base * 2 + 64 * j + lane)
                      : make_uint4(0, 0, 0, 0);
        }
        uint32_t keep[A][2];
#pragma unroll
        for (int b = 0; b < A; ++b) keep[b][0] = keep[b][1] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int b = 0; b < A; ++b) {
                uint32_t h = nibble_of(v[j].x, b) | nibble_of(v[j].y, b) << 4 |
                             nibble_of(v[j].z, b) << 8 |
                             nibble_of(v[j].w, b) << 12;
                h <<= 16 * (lane & 1);
                h = or_dpp<kDppQuadXor1>(h);
                if ((lane & 1) == (j & 1)) keep[b][j >> 1] = h;
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const uint32_t wi = base + 64 * s + lane;
            uint32_t word[A];
#pragma unroll
            for (int b = 0; b < A; ++b)
                word[b] = (uint32_t)__builtin_amdgcn_ds_bpermute(
                    from, (int)keep[b][s]);
            if (wi < nwords) {
                const uint32_t row = kwdiv.div(wi), t = wi - row * kw;
                uint32_t* dst = packed + (size_t)row * A * kw + t;
#pragma unroll
                for (int b = 0; b < A; ++b) dst[(size_t)b * kw] = word[b];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Wave-ballot packing, any k and any alignment, used when k is not a multiple
// of 32.  A chunk is 64 elements of one row; lane l holds element 64 c + l and
// the wave ballot of bit b is exactly the two packed words 2c, 2c+1 of plane b
// (bit l <- lane l), so no per-lane bit shuffling is needed.  A wave takes
// kChunks consecutive chunks (of one or several rows) at a time: their loads
// are in flight together, and the ballots, moved into lanes with writelane,
// leave by one store of 2 kChunks words per plane.  Bound by memory: with one
// chunk (one load of 4 or 1 bytes per lane) in flight and a 64-bit division
// for each, 104749 rows of 101 floats took 27.9 us (now 12.2 us, 3.7 TB/s) and
// 4096 rows of 1000 floats 10.4 us (now 5.4 us).  WIDE: 64-bit chunk numbers.
//
// A wave of few chunks takes one: its serial ballots count until the waves of
// one chunk each are 6 on a SIMD.  One / eight chunks per wave: 1000 rows of 100
// codes (2000 chunks) at 8 bits 2.6 / 3.3 us, 5000 chunks 3.0 / 3.2, 8192 3.4 /
// 3.2, 16384 4.7 / 3.7; floats at 2 bits 2000 chunks 2.4 / 2.7, 8192 3.0 / 2.7.
constexpr int kChunks = 8;
constexpr int64_t kFewChunks = 6144;

// old with `lane` (uniform) set to the uniform value (v_writelane_b32; the
// compiler has no builtin for it)
extern "C" __device__ int bs_writelane(int value, int lane, int old) __asm(
    "llvm.amdgcn.writelane.i32");

template <bool FROM_FLOAT, int ENC, bool WIDE, int CHUNKS>
__global__ __launch_bounds__(kBlock) void pack_ballot_kernel(
    const void* __restrict__ src, uint32_t* __restrict__ packed, int64_t k,
    int64_t nchunks, int64_t total, FastDiv div_chunks, int bits, float scale,
    float qmax) {
    using Index = std::conditional_t<WIDE, int64_t, int32_t>;
    constexpr uint32_t kSize = FROM_FLOAT ? 4 : 1;
    constexpr uint32_t kOutOfRange = 0x80000000u;
    constexpr int kNonTemporal = 2;          // buffer load cache policy
    const int lane = threadIdx.x & 63;
    const int64_t kw = (k + 31) >> 5;
    const Index nc = (Index)nchunks, end = (Index)total;
    const Index nwaves = (Index)gridDim.x * (kBlock / 64);
    const Index wave = __builtin_amdgcn_readfirstlane(
        (int)(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)));
    auto row_of = [&](Index chunk) -> Index {
        if constexpr (WIDE) return chunk / nc;
        else return (Index)div_chunks.div((uint32_t)chunk);
    };
    for (Index first = wave * CHUNKS; first < end; first += nwaves * CHUNKS) {
        const Index row = row_of(first);
        Index c = first - row * nc;
        // every chunk starts where the one before it ends, so the buffer is
        // based at the first chunk and the others are at most 64 elements
        // apart; lanes past a chunk's end read out of range, i.e. zeros
        const __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t*>(static_cast<const uint8_t*>(src)) +
                ((int64_t)row * k + (int64_t)c * 64) * kSize,
            (short)0, 64 * CHUNKS * kSize, 0x00020000);
        uint32_t raw[CHUNKS], code[CHUNKS];
        int count[CHUNKS];
        uint32_t at = 0;
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            const int64_t left = k - (int64_t)c * 64;
            const int n = first + u < end ? (left < 64 ? (int)left : 64) : 0;
            const uint32_t off =
                lane < n ? (at + (uint32_t)lane) * kSize : kOutOfRange;
            if constexpr (FROM_FLOAT)
                raw[u] = __builtin_amdgcn_raw_buffer_load_b32(buf, off, 0,
                                                              kNonTemporal);
            else
                raw[u] = __builtin_amdgcn_raw_buffer_load_b8(buf, off, 0,
                                                             kNonTemporal);
            count[u] = n;
            at += (uint32_t)n;
            if (++c == nc) c = 0;
        }
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            code[u] = raw[u];
            if constexpr (FROM_FLOAT) {
                code[u] = code_of<ENC>(__builtin_bit_cast(float, raw[u]),
                                       scale, qmax);
                // 0 is code 0 except under the sign quantizer
                if constexpr (ENC == kBipolar)
                    code[u] = lane < count[u] ? code[u] : 0u;
            }
        }
        // lane 2 u + h stores word 2 c + h of chunk u
        const Index mine = first + (lane >> 1);
        const Index mrow = row_of(mine < end ? mine : first);
        const int64_t t = 2 * ((int64_t)mine - (int64_t)mrow * nc) + (lane & 1);
        const bool stores = lane < 2 * CHUNKS && mine < end && t < kw;
        uint32_t* dst = packed + (int64_t)mrow * bits * kw + t;
        for (int b = 0; b < bits; ++b) {
            uint32_t word = 0;
#pragma unroll
            for (int u = 0; u < CHUNKS; ++u) {
                const uint64_t m = __ballot((code[u] >> b) & 1u);
                word = (uint32_t)bs_writelane((int)(uint32_t)m, 2 * u,
                                              (int)word);
                word = (uint32_t)bs_writelane((int)(uint32_t)(m >> 32),
                                              2 * u + 1, (int)word);
            }
            if (stores) dst[(int64_t)b * kw] = word;
        }
    }
}

// ---------------------------------------------------------------------------
// quantize_pack, k % 32 == 0: a wave produces 64 consecutive words of the
// flat [rows][k / 32] word array (2048 floats).  Load j (0..7) reads one
// float4 per lane, lanes consecutive (coalesced 1 KiB).  The 8 lanes
// 8m .. 8m+7 of load j hold word 8 j + m, 4 elements each: every lane
// quantizes its 4 values, places their plane-b bits at 4 (lane % 8), and
// three DPP ORs combine the group.  Lane 8m + i keeps word 8 j + m when
// j == i; a ds_bpermute per plane then moves word w to lane w.
template <int A, int ENC>
__global__ __launch_bounds__(kBlock) void quantize_pack_dpp_kernel(
    const float* __restrict__ x, uint32_t* __restrict__ packed,
    uint32_t nwords, FastDiv kwdiv, float scale, float qmax) {
    const int lane = threadIdx.x & 63;
    const uint32_t kw = kwdiv.d;
    const float4* xv = reinterpret_cast<const float4*>(x);
    const uint32_t wave0 = (blockIdx.x * kBlock + threadIdx.x) >> 6;
    const uint32_t nwaves = (gridDim.x * kBlock) >> 6;
    // word l is held by lane 8 (l % 8) + l / 8
    const int from = (8 * (lane & 7) + (lane >> 3)) * 4;
    for (uint32_t base = wave0 * 64u; base < nwords; base += nwaves * 64u) {
        const uint32_t left = nwords - base;
        float4 f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool ok = (uint32_t)(8 * j + (lane >> 3)) < left;
            f[j] = ok ? stream_load(xv + (size_t)base * 8 + 64 * j + lane)
                      : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        uint32_t keep[A];
#pragma unroll
        for (int b = 0; b < A; ++b) keep[b] = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t c4 = codes4<ENC>(f[j], scale, qmax);
#pragma unroll
            for (int b = 0; b < A; ++b) {
                uint32_t h = nibble_of(c4, b) << (4 * (lane & 7));
                h = or_dpp<kDppQuadXor1>(h);
                h = or_dpp<kDppQuadXor2>(h);
                h = or_dpp<kDppHalfMirror>(h);
                if ((lane & 7) == j) keep[b] = h;
            }
        }
        uint32_t word[A];
#pragma unroll
        for (int b = 0; b < A; ++b)
            word[b] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)keep[b]);
        const uint32_t wi = base + lane;
        if (wi < nwords) {
            const uint32_t row = kwdiv.div(wi), t = wi - row * kw;
            uint32_t* dst = packed + (size_t)row * A * kw + t;
#pragma unroll
            for (int b = 0; b < A; ++b) dst[(size_t)b * kw] = word[b];
        }
    }
}

// ---------------------------------------------------------------------------
// pack_ex: the codes viewed as [outer][k][inner], the reduction axis k at
// stride `inner` (NCHW activations, OIHW filters).  A thread builds word t of
// every plane for V consecutive rows i0 .. i0+V-1 of one outer index: it makes
// the word's 32 V-byte loads (neighbouring threads take neighbouring rows, so
// a load instruction reads one contiguous span) before it uses any of them,
// transposes the bytes of every 4 loads to 4 codes of one row per dword, and
// gathers each plane's bits with plane_word.  The words are stored where the
// layout puts them.
//
// A workgroup takes a tile of 256 V / TT rows x TT words (TT a power of two up
// to 8, or 64 where a row's codes are contiguous, at most the words per plane)
// and stores it through LDS, so that consecutive lanes store consecutive words
// of the packed rows; they do without it where a row's codes are contiguous,
// and for BMK with one word per plane and row (1000 x 4096 contiguous codes at 8
// bits, BMK, 10.4 us, with LDS 11.4; 64 x 3 x 12544 at 4 bits 9.8, with LDS 12.2).
//
// Bound by memory latency at small sizes and by the loads otherwise: with the
// loads waited for one by one, every bit moved by an extract and a shift-or
// and single words stored at the packed rows' stride, 128 x 256 x 196 codes at
// 3 bits took 21.3 us (now 5.6 us, an empty launch 4 us), 128 x 256 x 784 ones
// 46.8 us (now 12.2 us) and 2 x 128 x 100 ones 13.6 us (now 4.0 us).
//
// V = 4 needs inner >= 4; the last group of a row length that is no multiple
// of 4 starts early and skips the rows the previous group stores.  Its dword
// loads may then be unaligned, which global loads allow.  WIDE: 64-bit tile
// numbers.
struct StridedArgs {
    int64_t k, inner, kw, rows;
    int64_t iv, groups;            // row groups of one outer index, of all
    int64_t tiles_t, total;        // tiles along the words, of all
    FastDiv div_iv, div_t, div_row;    // div_row: words of a tile row
    int bits, layout, tt_log2;
};

// Where word i of a tile sits in LDS: one padding word in 32, so that the
// rows of neighbouring threads start in different banks.
__host__ __device__ inline int strided_slot(int i) { return i + (i >> 5); }

template <int V, bool WIDE>
__global__ __launch_bounds__(kBlock) void pack_strided_kernel(
    const uint8_t* __restrict__ q, uint32_t* __restrict__ packed,
    StridedArgs g) {
    typedef uint32_t __attribute__((aligned(1))) dword_any;
    // the tile in the order of its layout: [row][bits][TT] (MBK),
    // [row][TT][bits] (MKB) or [bits][row][TT] (BMK)
    extern __shared__ uint32_t lds[];
    const int tt_log2 = g.tt_log2;
    const int lines = 1 << tt_log2, threads_i = kBlock >> tt_log2;
    const int tile_rows = threads_i * V;
    const int row_words = g.bits << tt_log2;
    // steps of a tile word's index per row, plane and word
    const bool mkb = g.layout == kLayoutMKB, bmk = g.layout == kLayoutBMK;
    const int by_row = bmk ? lines : row_words;
    const int by_plane = bmk ? tile_rows << tt_log2 : mkb ? 1 : lines;
    const int by_word = mkb ? g.bits : 1;
    // neighbouring threads take neighbouring rows, or words where the codes of
    // a row are contiguous
    const bool along = g.inner == 1;
    const int qi = along ? threadIdx.x >> tt_log2
                         : threadIdx.x & (threads_i - 1);
    const int tt = along ? threadIdx.x & (lines - 1) : threadIdx.x / threads_i;
    // consecutive threads hold consecutive words of a plane, or whole words of
    // it `bits` apart: stored without LDS
    const bool direct = along || (bmk && g.kw == 1);
    // outer index and first row of group n of V rows
    auto locate = [&](int64_t n, int64_t* o) -> int64_t {
        if constexpr (WIDE) *o = n / g.iv;
        else *o = g.div_iv.div((uint32_t)n);
        return (n - *o * g.iv) * V;
    };
    for (int64_t f = blockIdx.x; f < g.total; f += gridDim.x) {
        int64_t tq, o;
        if constexpr (WIDE) tq = f / g.tiles_t;
        else tq = g.div_t.div((uint32_t)f);
        const int64_t tw = f - tq * g.tiles_t;
        const int64_t n0 = tq * threads_i, n = n0 + qi;
        const int64_t t = (tw << tt_log2) + tt;
        // the tile's rows: those of its groups, consecutive across outer
        // indices
        int64_t i = locate(n0, &o);
        const int64_t r0 = o * g.inner + i;
        i = locate((n0 + threads_i < g.groups ? n0 + threads_i : g.groups) - 1,
                   &o);
        const int rows_here = (int)(
            o * g.inner + (i + V < g.inner ? i + V : g.inner) - r0);
        if (n < g.groups && t < g.kw) {
            const int64_t want = locate(n, &o);
            const int64_t i0 = want < g.inner - V ? want : g.inner - V;
            const int64_t left = g.k - 32 * t;
            const int u_end = left < 32 ? (int)left : 32;
            const uint8_t* src = q + (o * g.k + 32 * t) * g.inner + i0;
            uint32_t x[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                // past the last element: read it again, then drop it
                const uint8_t* p = src + (int64_t)min(u, u_end - 1) * g.inner;
                if constexpr (V == 4)
                    x[u] = *reinterpret_cast<const dword_any*>(p);
                else
                    x[u] = *p;
            }
#pragma unroll
            for (int u = 0; u < 32; ++u) x[u] = u < u_end ? x[u] : 0u;
            uint32_t d[V][8];
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint32_t x0 = x[4 * m], x1 = x[4 * m + 1],
                               x2 = x[4 * m + 2], x3 = x[4 * m + 3];
                if constexpr (V == 4) {
                    // 4 x 4 byte transpose
                    const uint32_t a =
                        __builtin_amdgcn_perm(x1, x0, 0x05010400u);
                    const uint32_t b =
                        __builtin_amdgcn_perm(x1, x0, 0x07030602u);
                    const uint32_t c =
                        __builtin_amdgcn_perm(x3, x2, 0x05010400u);
                    const uint32_t e =
                        __builtin_amdgcn_perm(x3, x2, 0x07030602u);
                    d[0][m] = __builtin_amdgcn_perm(c, a, 0x05040100u);
                    d[1][m] = __builtin_amdgcn_perm(c, a, 0x07060302u);
                    d[2][m] = __builtin_amdgcn_perm(e, b, 0x05040100u);
                    d[3][m] = __builtin_amdgcn_perm(e, b, 0x07060302u);
                } else {
                    d[0][m] = x0 | x1 << 8 | x2 << 16 | x3 << 24;
                }
            }
            // row i0 + v of outer index o; the rows before `want` are the
            // previous group's
            const int at = (int)(o * g.inner + i0 - r0);
            const int skip = (int)(want - i0);
            if (direct) {
                const int64_t row = o * g.inner + i0;
                uint32_t* dst =
                    packed + (mkb ? (row * g.kw + t) * g.bits
                                  : row * g.kw + t);
                const int64_t by_b = mkb ? 1 : g.rows * g.kw;
                for (int b = 0; b < g.bits; ++b, dst += by_b)
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        if (v >= skip) dst[v] = plane_word(d[v], b);
                continue;
            }
            for (int b = 0; b < g.bits; ++b)
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if (v >= skip)
                        lds[strided_slot((at + v) * by_row + b * by_plane +
                                         tt * by_word)] = plane_word(d[v], b);
        }
        if (direct) continue;
        __syncthreads();
        // the tile's words, at the same order in memory: rows of row_words
        // words every kw * bits (MBK: pieces of TT words every kw)
        const int64_t left_t = g.kw - (tw << tt_log2);
        const int words = left_t < lines ? (int)left_t : lines;
        const int64_t t0 = tw << tt_log2;
        if (bmk) {
            constexpr int PLANE = kBlock * V;      // words of a tile's plane
            uint32_t* dst = packed + r0 * g.kw + t0;
#pragma unroll 4
            for (int e = threadIdx.x; e < g.bits * PLANE; e += kBlock) {
                const int b = e / PLANE, r = (e % PLANE) >> tt_log2;
                const int w = e & (lines - 1);
                if (r < rows_here && w < words)
                    dst[((int64_t)b * g.rows + r) * g.kw + w] =
                        lds[strided_slot(e)];
            }
        } else if (words == g.kw && words == lines) {
            // whole rows: one contiguous piece of memory
            uint32_t* dst = packed + r0 * g.bits * g.kw;
#pragma unroll 4
            for (int e = threadIdx.x; e < rows_here * row_words; e += kBlock)
                dst[e] = lds[strided_slot(e)];
        } else {
            uint32_t* dst = packed + r0 * g.bits * g.kw + (mkb ? t0 * g.bits
                                                               : t0);
            for (int e = threadIdx.x; e < rows_here * row_words; e += kBlock) {
                if (mkb) {
                    const int r = (int)g.div_row.div((uint32_t)e);
                    const int j = e - r * row_words;
                    if (j < words * g.bits)
                        dst[(int64_t)r * g.kw * g.bits + j] =
                            lds[strided_slot(e)];
                } else {
                    const int w = e & (lines - 1);
                    if (w < words)
                        dst[(int64_t)(e >> tt_log2) * g.kw + w] =
                            lds[strided_slot(e)];
                }
            }
        }
        __syncthreads();
    }
}

int grid_for(int64_t work_items, int per_block) {
    int64_t b = (work_items + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > kMaxBlocks) b = kMaxBlocks;
    return (int)b;
}

template <int A>
hipError_t launch_pack32(const uint8_t* q, uint32_t* packed, uint32_t nwords,
                         const FastDiv& d, hipStream_t st) {
    // 128 words per wave, 4 waves per block
    return launch(pack_dpp_kernel<A>, dim3(grid_for(nwords, 512)),
                  dim3(kBlock), 0, st, q, packed, nwords, d);
}

template <int A, int ENC>
hipError_t launch_qpack(const float* x, uint32_t* packed, uint32_t nwords,
                        const FastDiv& d, float scale, float qmax,
                        hipStream_t st) {
    // 64 words per wave, 4 waves per block
    return launch(quantize_pack_dpp_kernel<A, ENC>,
                  dim3(grid_for(nwords, 256)), dim3(kBlock), 0, st, x, packed,
                  nwords, d, scale, qmax);
}

template <bool FROM_FLOAT, int ENC, int CHUNKS>
hipError_t launch_chunks(const void* src, uint32_t* packed, int64_t k,
                         int64_t total, int bits, float scale, float qmax,
                         hipStream_t st) {
    const int64_t nchunks = (k + 63) / 64;
    const dim3 grid(grid_for(total, 4 * CHUNKS));
    FastDiv d{};
    // the last step past the end stays within 32 bits
    if (total > INT32_MAX - (int64_t)kMaxBlocks * 4 * CHUNKS)
        return launch(pack_ballot_kernel<FROM_FLOAT, ENC, true, CHUNKS>, grid,
                      dim3(kBlock), 0, st, src, packed, k, nchunks, total, d,
                      bits, scale, qmax);
    d.init((uint32_t)nchunks);
    return launch(pack_ballot_kernel<FROM_FLOAT, ENC, false, CHUNKS>, grid,
                  dim3(kBlock), 0, st, src, packed, k, nchunks, total, d, bits,
                  scale, qmax);
}

// Any k, 4 waves per block.
template <bool FROM_FLOAT, int ENC>
hipError_t launch_ballot(const void* src, uint32_t* packed, int64_t rows,
                         int64_t k, int bits, float scale, float qmax,
                         hipStream_t st) {
    const int64_t total = rows * ((k + 63) / 64);
    if (total <= kFewChunks)
        return launch_chunks<FROM_FLOAT, ENC, 1>(src, packed, k, total, bits,
                                                 scale, qmax, st);
    return launch_chunks<FROM_FLOAT, ENC, kChunks>(src, packed, k, total, bits,
                                                   scale, qmax, st);
}

}  // namespace

// qmax of an encoding: the top unipolar code, the top signed value
static float enc_qmax(int bits, int enc) {
    return enc == kSigned ? (float)((1 << (bits - 1)) - 1)
                          : (float)((1 << bits) - 1);
}

hipError_t launch_quantize(const float* x, uint8_t* q, int64_t n, float scale,
                           int bits, int enc, hipStream_t st) {
    const float qmax = enc_qmax(bits, enc);
    const dim3 grid(grid_for((n >> 4) + 1, kBlock));
    if (enc == kBipolar)
        return launch(quantize_kernel<kBipolar>, grid, dim3(kBlock), 0, st, x,
                      q, n, scale, qmax);
    if (enc == kSigned)
        return launch(quantize_kernel<kSigned>, grid, dim3(kBlock), 0, st, x,
                      q, n, scale, qmax);
    return launch(quantize_kernel<kUnipolar>, grid, dim3(kBlock), 0, st, x, q,
                  n, scale, qmax);
}

hipError_t launch_pack(const uint8_t* q, uint32_t* packed, int64_t rows,
                       int64_t k, int bits, hipStream_t st) {
    const int64_t kw = (k + 31) / 32;
    const int64_t groups = rows * kw;
    if (k % 32 == 0 && groups < (int64_t)INT32_MAX - 128) {
        FastDiv d;
        d.init((uint32_t)kw);
        switch (bits) {
            case 1: return launch_pack32<1>(q, packed, (uint32_t)groups, d, st);
            case 2: return launch_pack32<2>(q, packed, (uint32_t)groups, d, st);
            case 3: return launch_pack32<3>(q, packed, (uint32_t)groups, d, st);
            case 4: return launch_pack32<4>(q, packed, (uint32_t)groups, d, st);
            case 5: return launch_pack32<5>(q, packed, (uint32_t)groups, d, st);
            case 6: return launch_pack32<6>(q, packed, (uint32_t)groups, d, st);
            case 7: return launch_pack32<7>(q, packed, (uint32_t)groups, d, st);
            default: return launch_pack32<8>(q, packed, (uint32_t)groups, d, st);
        }
    }
    return launch_ballot<false, kUnipolar>(q, packed, rows, k, bits, 0.0f,
                                           0.0f, st);
}

template <int V>
static hipError_t launch_strided(const uint8_t* q, uint32_t* packed,
                                 int64_t outer, int64_t k, int64_t inner,
                                 int bits, int layout, hipStream_t st) {
    StridedArgs g{};
    g.k = k;
    g.inner = inner;
    g.kw = (k + 31) / 32;
    const int most = inner == 1 ? 6 : 3;
    while (g.tt_log2 < most && 2 << g.tt_log2 <= g.kw) ++g.tt_log2;
    g.iv = (inner + V - 1) / V;
    g.groups = outer * g.iv;
    g.tiles_t = (g.kw + (1 << g.tt_log2) - 1) >> g.tt_log2;
    const int64_t per_tile = kBlock >> g.tt_log2;
    g.total = (g.groups + per_tile - 1) / per_tile * g.tiles_t;
    g.rows = outer * inner;
    g.bits = bits;
    g.layout = layout;
    g.div_row.init((uint32_t)(bits << g.tt_log2));
    const dim3 grid(grid_for(g.total, 1));
    const size_t lds = (size_t)(strided_slot(kBlock * V * bits - 1) + 1) * 4;
    // group and tile numbers, the last tile's past the end included, in 32
    // bits
    if (g.groups > INT32_MAX - kBlock || g.total > INT32_MAX)
        return launch(pack_strided_kernel<V, true>, grid, dim3(kBlock), lds,
                      st, q, packed, g);
    g.div_iv.init((uint32_t)g.iv);
    g.div_t.init((uint32_t)g.tiles_t);
    return launch(pack_strided_kernel<V, false>, grid, dim3(kBlock), lds, st,
                  q, packed, g);
}

hipError_t launch_pack_ex(const uint8_t* q, uint32_t* packed, int64_t outer,
                          int64_t k, int64_t inner, int bits, int layout,
                          hipStream_t st) {
    if (inner == 1 && layout == kLayoutMBK)
        return launch_pack(q, packed, outer, k, bits, st);
    // four rows to a thread wherever a row's neighbours exist and the grid
    // keeps a workgroup for every other CU (workgroups of 4 x 256 rows x
    // words); below that a thread's serial work counts: 8 bits, one row / four:
    // 64 x 512 x 9 codes (12 workgroups) 6.4 / 11.2 us, 128 x 512 x 49 (104) 7.2 /
    // 11.4, 64 x 128 x 196 (49) 4.4 / 6.1; 64 x 3 x 12544 (784) 21.3 / 18.7
    const int64_t blocks =
        outer * ((inner + 3) / 4) * ((k + 31) / 32) / kBlock;
    return inner >= 4 && 2 * blocks >= device_cus()
               ? launch_strided<4>(q, packed, outer, k, inner, bits, layout,
                                   st)
               : launch_strided<1>(q, packed, outer, k, inner, bits, layout,
                                   st);
}

namespace {

template <int ENC>
hipError_t quantize_pack_enc(const float* x, uint32_t* packed, int64_t rows,
                             int64_t k, float scale, int bits, float qmax,
                             hipStream_t st) {
    const int64_t nwords = rows * ((k + 31) / 32);
    if (k % 32 == 0 && nwords < (int64_t)INT32_MAX - 64) {
        FastDiv d;
        d.init((uint32_t)(k / 32));
        const uint32_t nw = (uint32_t)nwords;
        switch (bits) {
            case 1: return launch_qpack<1, ENC>(x, packed, nw, d, scale, qmax, st);
            case 2: return launch_qpack<2, ENC>(x, packed, nw, d, scale, qmax, st);
            case 3: return launch_qpack<3, ENC>(x, packed, nw, d, scale, qmax, st);
            case 4: return launch_qpack<4, ENC>(x, packed, nw, d, scale, qmax, st);
            case 5: return launch_qpack<5, ENC>(x, packed, nw, d, scale, qmax, st);
            case 6: return launch_qpack<6, ENC>(x, packed, nw, d, scale, qmax, st);
            case 7: return launch_qpack<7, ENC>(x, packed, nw, d, scale, qmax, st);
            default: return launch_qpack<8, ENC>(x, packed, nw, d, scale, qmax, st);
        }
    }
    return launch_ballot<true, ENC>(x, packed, rows, k, bits, scale, qmax, st);
}

}  // namespace

hipError_t launch_quantize_pack(const float* x, uint32_t* packed,
                                int64_t rows, int64_t k, float scale, int bits,
                                int enc, hipStream_t st) {
    const float qmax = enc_qmax(bits, enc);
    if (enc == kBipolar)
        return quantize_pack_enc<kBipolar>(x, packed, rows, k, scale, 1, qmax,
                                           st);
    if (enc == kSigned)
        return quantize_pack_enc<kSigned>(x, packed, rows, k, scale, bits,
                                          qmax, st);
    return quantize_pack_enc<kUnipolar>(x, packed, rows, k, scale, bits, qmax,
                                        st);
}

}  // namespace bs
