// any-n GEMM (n = 4, 3, 2) for a few dozen rows of x (17 <= M <= 128: token generation with many sequences
// in flight): codes become matrix-core operands in registers, activations pass through LDS.
//
// y[m][n] = sum_k x[m][k] * (LUT[n][code[n][k]] * scale[n][k/128] + offset[n][k/128])
// (any4 paper, section 4.2 for y = x w^T with on-the-fly dequantisation, sections 2.4.1 and 2.5.2 for
// the per-row table and alpha * w_Q + beta).
//
// Lookup.  A lane keeps to one weight row (row lane % 32 of its wavefront's 32), whose table sits in eight
// registers (any4_regtable.h): codes are loaded from memory straight into the lane that uses them and leave
// the lookup as the B operand of v_mfma_f32_32x32x16.  Lane half h owns codes 32 h .. 32 h + 31 of every 64, so
// operand kk of a group pairs chunk 8 (kk / 4) + 4 h + kk % 4 (eight weights) with the same chunk of x.
//
// Scale and offset never touch weights: a group's products are summed by themselves and enter the result
// with one fma each; the offset term is a matrix instruction per eight groups over (group sum of x, split into a
// high and a low 16-bit part) x (offset).  The group sums come from a matrix instruction with an operand of
// ones, one (32 rows, group) per wavefront, alternating between the halves of the block.
//
// Work split.  A block takes 32 MT rows of x (all of them: MT = ceil(M / 32)), 32 WN rows of weights and a slab of
// K; its 8 wavefronts are WN along n and WK = 8 / WN along k (alternate groups).  A step is one group per k part.
// x of the coming steps is copied straight into a ring of LDS buffers, three steps ahead, and the codes are loaded into
// registers, four steps ahead; a step waits for what step t + 2 needs, so the first operand of the next step can be
// prepared before the barrier.  The parts meet in LDS, slabs of K in the workspace (fp32, added in slab order by the blocks of the tile, see meet).
//
// Order of the sums.  A block starts at a step of its own along K (see `rot`), so the last bit of an output can depend on
// the place of its row of weights in the matrix.
//
// What bounds it: no unit by itself.  28672 x 4096 at M = 64 (16 steps, 224 blocks, 38 us under the counters, 1.93 GHz): a
// wavefront issues 310 vector instructions (20 of them matrix) and 24 LDS instructions a step; vector issue is
// busy 54 % of the time, the matrix cores of the SIMDs that hold a block 28 %, the LDS pipe 18 %, and wavefronts wait 39 % of
// theirs.  A step takes 1.8 us.  The rest of a launch is fixed: 5 - 14 us for start and end of a block (32 .. 128 rows of x),
// and where slabs meet 3 - 6 us for their sums (any4_batch.hip has the constants).  The four linears of an 8B layer at M = 24 / 64 / 128:
// 81 / 96 / 147 us; with one block adding all the sums of a tile and all first loads at once 84 / 106 / 183.
#pragma once
#include "any4_device.h"
#include "any4_internal.h"
#include "any4_lds_copy.h"
#include "any4_regtable.h"
#include "any4_splitk.h"
#include <type_traits>

namespace any4 {
namespace batch {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x4* lds_u4;
typedef __attribute__((address_space(3))) uint32_t* lds_u32;
typedef __attribute__((address_space(3))) uint16_t* lds_u16;
typedef __attribute__((address_space(3))) float* lds_f32;

constexpr int kWaves = 8, kThreads = kWaves * 64;
constexpr int kRowBytes = kGroup * 2;                 // one group of one row of x in LDS
constexpr int kLdsPerCu = 160 * 1024;
// wavefronts along n: with up to 64 rows of x four (128 rows of weights a block) and two k parts; above, eight -
// the activations of a step are then those of one group, which is what the LDS buffers hold
constexpr int wn_of(int mt) { return mt <= 2 ? 4 : 8; }

// MT: 32-row tiles of x per block; WN: wavefronts along n (32 rows of weights each), WK = 8 / WN along k
template <int MT, int WN> struct Shape {
    static constexpr int WK = kWaves / WN, ROWS = 32 * MT, BN = 32 * WN;
    static constexpr int XBUF = WK * ROWS * kRowBytes;            // x of one step: one group per k part
    static constexpr int DEPTH = 3;                               // steps from the issue of x's loads to their use
    static constexpr int CODE_DEPTH = MT == 4 ? 3 : 4;            // ... of the codes' (a fourth set does not fit next to four tiles)
    static constexpr int XS = (DEPTH + 1) * XBUF;                 // group sums of x: [2][WK][ROWS][8] packed hi, lo
    static constexpr int XS_SET = WK * ROWS * 32;
    static constexpr int SC = XS + 2 * XS_SET;                    // the slab's scales, then its offsets: [BN] rows of sc_stride bytes
    static constexpr int lds_bytes(int sc_stride) { return SC + 2 * BN * sc_stride; }
    // bytes from a row of staged scales to the next: an odd number of 4-byte words, so that 32 rows lie in 32 banks
    static constexpr int sc_stride(int values) { return ((values + 1) / 2 | 1) * 4; }
    static constexpr int DMA = XBUF / (kWaves * 1024);            // 1 KB pieces of x per wavefront and step
    // the most values a slab may have per row of weights (a row of staged values is an odd number of words)
    static constexpr int MAX_VALUES = 2 * (((kLdsPerCu - SC) / (8 * BN) - 1) | 1);
    static_assert(XBUF % (kWaves * 1024) == 0, "every wavefront moves whole pieces");
    static_assert(MT * WK <= kWaves, "at most one group sum task per wavefront and step");
    static_assert(MT * WK * WN * 4096 * (WK > 1) <= XS, "the combination of the k parts fits the x buffers");
};

struct Params {
    const uint16_t* x;
    const uint32_t* codes;
    const uint16_t* lut;
    const uint16_t* scale;
    const uint16_t* offset;
    uint16_t* y;
    float* partial;                  // [tiles][slabs][ROWS * BN] fp32, slabs > 1 only
    unsigned long long* words;       // a meeting word every word_step words per tile, slabs > 1 only
    int word_step;
    int64_t N, K, ldy;               // N: rows of weights of this launch; ldy: values from a row of y to the next
    int M, G;                        // G = K / 128
    int lr;                          // log2(group size / 128), 0 with groups of 64
    int flags;                       // 1: re-laid-out codes, 2: one table for all rows
    int slabs, tiles_n;              // grid = (tiles_n * slabs, blocks of ROWS rows of x)
    int parts;                       // in how many parts the sums of a tile's slabs are added: 1, or one for each of up to 8 slabs
    int sc_stride;                   // Shape::sc_stride of the largest slab
};

template <int BITS, int MT, int WN, bool F16, bool FINE>
__device__ __forceinline__ void batch_body(const Params& p) {
    using S = Shape<MT, WN>;
    constexpr int WK = S::WK, ROWS = S::ROWS, BN = S::BN, D = S::DEPTH, CD = S::CODE_DEPTH;
    auto mma = [](const u32x4& a, const u32x4& b, const f32x16& c) -> f32x16 {
        if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    };
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave % WN, wk = wave / WN, r32 = lane & 31, h = lane >> 5;
    // (32-bit divisions: G < 2^17, at most 64 slabs)
    const int tile = (int)(blockIdx.x / (unsigned)p.slabs), slab = (int)blockIdx.x - tile * p.slabs;
    const int G = p.G, g_lo = (int)((unsigned)(slab * G) / (unsigned)p.slabs), g_hi = (int)((unsigned)((slab + 1) * G) / (unsigned)p.slabs);
    const int T = (g_hi - g_lo + WK - 1) / WK;                    // steps
    // A block starts at a step of its own and wraps around: rows lie powers of two apart, and blocks that
    // walked along K together would all ask the same few memory channels at a time.
    const int rot = tile % T;
    auto group_of = [&](int t, int part) -> int {                 // the group of part `part` at step t (>= g_hi: none)
        const int s = t + rot;
        return g_lo + (s >= T ? s - T : s) * WK + part;
    };
    const int64_t n0 = (int64_t)tile * BN, m0 = (int64_t)blockIdx.y * ROWS;
    const bool repacked = p.flags & 1, one_table = p.flags & 2;
    const int64_t row = min(n0 + wn * 32 + r32, p.N - 1);         // rows past N are computed, never stored

    // ---- where this lane's data comes from
    // codes: half i of a group, this lane's 32 codes of it: BITS words
    const int64_t RW = row_words(p.K, BITS), GS = FINE ? 2 * (int64_t)G : G >> p.lr;           // words of codes / scales per row
    const int rloc = (int)(row - n0);
    const char* const cbase = reinterpret_cast<const char*>(p.codes + n0 * RW);
    const uint32_t coff = (uint32_t)(repacked ? ((rloc >> 4) * G * 64 + h * 16 + (rloc & 15)) * BITS : rloc * (int)RW + h * BITS) * 4u;
    const uint32_t cgroup = (repacked ? 64 * BITS : 4 * BITS) * 4, chalf = (repacked ? 32 * BITS : 2 * BITS) * 4;   // bytes to the next group / half
    // x: piece i of this wavefront = 4 rows of one group; LDS position c of row r holds the 16-byte
    // chunk c ^ (r % 16), so that the 16 lanes LDS serves together read 16 different columns
    uint32_t xoff[S::DMA];
#pragma unroll
    for (int i = 0; i < S::DMA; ++i) {
        const int r = ((wave * S::DMA + i) * 4 + (lane >> 4)) % ROWS;
        const int64_t m = min((int64_t)r, p.M - 1 - m0);
        xoff[i] = (uint32_t)(m * p.K * 2) + (uint32_t)((lane & 15) ^ (r & 15)) * 16u;
    }
    auto fetch_x = [&](int t) {
        const uint32_t buf = (uint32_t)(t % (D + 1)) * S::XBUF;
#pragma unroll
        for (int i = 0; i < S::DMA; ++i) {
            const int piece = wave * S::DMA + i;                  // a buffer is [WK][ROWS] rows of 256 bytes
            const int g = min(group_of(t, piece / (ROWS / 4)), g_hi - 1);
            copy_to_lds(buf + (uint32_t)piece * 1024u, reinterpret_cast<const char*>(p.x + m0 * p.K) + (int64_t)g * kRowBytes, xoff[i]);
        }
    };
    using words = std::conditional_t<BITS == 4, u32x4, std::conditional_t<BITS == 3, u32x3, u32x2>>;
    struct Codes { words w[2]; };
    auto fetch_codes = [&](Codes& c, int t) {                     // (past the last step: a piece of the slab once more)
        const int g = min(group_of(t, wk), g_hi - 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            struct packed { uint32_t v[BITS]; };
            const packed v = *reinterpret_cast<const packed*>(cbase + (int64_t)g * cgroup + i * chalf + coff);
#pragma unroll
            for (int j = 0; j < BITS; ++j) c.w[i][j] = v.v[j];
        }
    };
    // (the compiler's wait for these codes goes here: after the copies of x that follow it would be for some of them, too)
    auto landed = [&](Codes& c) { asm volatile("" : "+v"(c.w[0]), "+v"(c.w[1])); };
    constexpr int kLoads = 2 + S::DMA;                            // load instructions per wavefront and step

    // Scales and offsets of the slab are staged in LDS once, with loads as wide as their alignment allows: a
    // load of one value from each of 32 rows costs the memory pipeline as much as one of their codes.
    const int s_lo = FINE ? 2 * g_lo : g_lo >> p.lr, s_n = (FINE ? 2 * g_hi : ((g_hi - 1) >> p.lr) + 1) - s_lo;
    auto stage_pieces = [&](auto unit, auto flight_, int chunks, int total) {
        using V = decltype(unit);
        constexpr int PER = sizeof(V) / 2, FLIGHT = decltype(flight_)::value;
        for (int base = threadIdx.x; base < total; base += kThreads * FLIGHT) {
            V v[2][FLIGHT];
            uint32_t to[FLIGHT];
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) {
                const int idx = min(base + u * kThreads, total - 1), r = idx / chunks, c = idx - r * chunks;
                const int64_t from = min(n0 + r, p.N - 1) * GS + s_lo + c * PER;
                v[0][u] = *reinterpret_cast<const V*>(p.scale + from);
                v[1][u] = *reinterpret_cast<const V*>(p.offset + from);
                to[u] = (uint32_t)(S::SC + r * p.sc_stride + c * (int)sizeof(V));
            }
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u)                      // (past the end: the last piece once more)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const uint32_t a = to[u] + k * BN * p.sc_stride;
                    if constexpr (sizeof(V) == 16) {
#pragma unroll
                        for (int d = 0; d < 4; ++d) *reinterpret_cast<lds_u32>(a + 4 * d) = v[k][u][d];
                    } else *reinterpret_cast<__attribute__((address_space(3))) V*>(a) = v[k][u];
                }
        }
    };
    auto stage_scales = [&](auto unit) {
        constexpr int PER = sizeof(unit) / 2;
        const int chunks = (s_n + PER - 1) / PER, total = BN * chunks;
        if (total <= kThreads) stage_pieces(unit, std::integral_constant<int, 1>{}, chunks, total);
        else if (total <= 2 * kThreads) stage_pieces(unit, std::integral_constant<int, 2>{}, chunks, total);
        else stage_pieces(unit, std::integral_constant<int, 4>{}, chunks, total);
    };

    // the row's table and the codes of the first steps
    using table_words = std::conditional_t<BITS == 2, u32x2, u32x4>;
    table_words tw[BITS == 4 ? 2 : 1];
    if (p.lut) {
        const table_words* const src = reinterpret_cast<const table_words*>(p.lut + (one_table ? 0 : row << BITS));
        tw[0] = src[0];
        if constexpr (BITS == 4) tw[1] = src[1];
    }
    // (Loads are taken only as fast as earlier ones are served - the first 160 KB of a block took 10 - 14 000 cycles to be taken - so
    // what the first step does not need is asked for behind what it waits for: two steps, the scales, a third step, and the rest
    // after the wait.  6144 / 4096 / 28672 x 4096 at M = 64 17.9 / 16.5 / 40.1 -> 17.0 / 15.7 / 38.5 us; without the third step before the wait 17.5 /
    // 16.4 / 39.3.)
    Codes cq[CD];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        fetch_codes(cq[t], min(t, T - 1));
        if (t < T) fetch_x(t);
    }
    if (((GS | s_lo | s_n) & 7) == 0) stage_scales(u32x4{});
    else if (((GS | s_lo) & 1) == 0) stage_scales(uint32_t{});
    else stage_scales(uint16_t{});
    fetch_codes(cq[2], min(2, T - 1));
    if (2 < T) fetch_x(2);
    for (uint32_t a = threadIdx.x * 16; a < 2 * S::XS_SET; a += kThreads * 16) *reinterpret_cast<lds_u4>(S::XS + a) = u32x4{0, 0, 0, 0};
    const uint32_t srow = (uint32_t)(S::SC + (wn * 32 + r32) * p.sc_stride);   // this lane's staged scales; offsets BN rows on
    auto staged = [&](uint32_t at, int g) -> uint32_t {           // FINE: the pair of the group's halves
        if constexpr (FINE) return *reinterpret_cast<lds_u32>(at + (g - g_lo) * 4);
        else return *reinterpret_cast<lds_u16>(at + ((g >> p.lr) - s_lo) * 2);
    };

    RowTable<BITS> table;
    f32x16 zero;
#pragma unroll
    for (int v = 0; v < 16; ++v) zero[v] = 0.f;
    f32x16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i] = zero;
    const uint32_t one2 = F16 ? 0x3C003C00u : 0x3F803F80u;
    const u32x4 ones = {one2, one2, one2, one2};
    // operand kk of a group = its chunk 8 (kk / 4) + 4 h + kk % 4 (8 activations): a lane's 32 codes of a half
    // group are 4 operands.  LDS address of that chunk of row r32 of tile i of part k of a buffer:
    const uint32_t xrd = (uint32_t)(r32 * kRowBytes + ((4 * h) ^ (r32 & 15)) * 16);
    auto read_x = [&](uint32_t base, int i, int kk) -> u32x4 {
        return *reinterpret_cast<lds_u4>((base ^ (uint32_t)((8 * (kk >> 2) + (kk & 3)) * 16)) + (uint32_t)(i * 32 * kRowBytes));
    };
    // The offsets times the group sums of x of (up to) eight of this part's groups, those of steps t0 ..: one
    // matrix instruction per tile; half h of the wavefront brings four of the groups (FINE: two, two values each)
    auto offset_term = [&](int t0, int set) {
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < (FINE ? 2 : 4); ++j) {
            const int t = t0 + (FINE ? 2 : 4) * h + j, g = group_of(t, wk);
            const bool in = t < T && g < g_hi;
            const uint32_t v = staged(srow + BN * p.sc_stride, in ? g : g_lo);
            if constexpr (FINE) {
                o[2 * j] = in ? (v & 0xFFFFu) | (v << 16) : 0u;
                o[2 * j + 1] = in ? (v >> 16) | (v & 0xFFFF0000u) : 0u;
            } else o[j] = in ? v | (v << 16) : 0u;
        }
        const u32x4 b = {o[0], o[1], o[2], o[3]};
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const u32x4 a = *reinterpret_cast<lds_u4>(S::XS + set * S::XS_SET + (wk * ROWS + i * 32 + r32) * 32 + h * 16);
            acc[i] = mma(a, b, acc[i]);
        }
    };
    constexpr int kPer = FINE ? 4 : 8;                            // groups of 128 per offset term

    // The step's matrix instructions go operand by operand (kk), interleaved with the lookups of the next
    // operand and the reads of its activations; the last operand of a step prepares the first one of the next
    // step, whose activations and codes have landed a step early for that.
    u32x4 a[2][MT], b[2];
    auto prepare = [&](const Codes& c, uint32_t xm, int kk) {
#pragma unroll
        for (int i = 0; i < MT; ++i) a[kk & 1][i] = read_x(xm, i, kk);
        uint32_t w[BITS], d[4];
#pragma unroll
        for (int j = 0; j < BITS; ++j) w[j] = c.w[kk >> 2][j];
        table.eight(w, kk & 3, d);
        b[kk & 1] = u32x4{d[0], d[1], d[2], d[3]};
    };
    auto xbase = [&](int t) -> uint32_t { return xrd + (uint32_t)(t % (D + 1)) * S::XBUF + (uint32_t)(wk * ROWS * kRowBytes); };
    auto work = [&](const Codes& c, const Codes& next, int t) {
        if (t + D < T) fetch_x(t + D);
        if (t > 0 && t % kPer == 0) offset_term(t - kPer, (t - 1) / kPer & 1);
        const int slot = t % kPer, set = t / kPer & 1;
        uint32_t xm = xbase(t), xn = xbase(t + 1);                // opaque: their variants are not kept in registers
        asm volatile("" : "+v"(xm), "+v"(xn));
        // group sums of x, one (tile, part) for some of the wavefronts: with an operand of ones every row of the
        // product holds the sums of its columns
        const int task = (wave + 4 * (t & 1)) & 7;
        if (task < MT * WK) {
            const int i = task % MT, k = task / MT;
            f32x16 d = zero, e = zero;
            uint32_t xt = xrd + (uint32_t)(t % (D + 1)) * S::XBUF + (uint32_t)((k * ROWS + i * 32) * kRowBytes);
            asm volatile("" : "+v"(xt));
            u32x4 v[8];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) v[kk] = read_x(xt, 0, kk);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                if (FINE && kk >= 4) e = mma(ones, v[kk], e);
                else d = mma(ones, v[kk], d);
            }
            auto split = [&](float s) -> uint32_t {
                const uint32_t hi = f32_to_h16<F16>(s);
                return hi | (f32_to_h16<F16>(s - h16_to_f32<F16>(hi)) << 16);
            };
            const uint32_t to = S::XS + set * S::XS_SET + (k * ROWS + i * 32 + r32) * 32;
            if constexpr (FINE) *reinterpret_cast<lds_u32>(to + slot * 8 + h * 4) = split(h ? e[0] : d[0]);
            else *reinterpret_cast<lds_u32>(to + slot * 4) = split(d[0]);
        }
        if (group_of(t, wk) < g_hi) {
            const uint32_t cs = staged(srow, group_of(t, wk));
            f32x16 part[MT];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                prepare(kk < 7 ? c : next, kk < 7 ? xm : xn, (kk + 1) & 7);
#pragma unroll
                for (int i = 0; i < MT; ++i) part[i] = mma(a[kk & 1][i], b[kk & 1], kk == 0 || (FINE && kk == 4) ? zero : part[i]);
                __builtin_amdgcn_sched_group_barrier(0x102, MT + 1, 0);        // the reads first (and their address) ...
#pragma unroll
                for (int i = 0; i < MT; ++i) {                    // ... then matrix instructions among the lookups
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 24 / MT, 0);
                }
                if (kk == 7 || (FINE && kk == 3)) {
                    const float s = FINE ? h16_to_f32<F16>(kk == 3 ? cs & 0xFFFFu : cs >> 16) : h16_to_f32<F16>(cs);
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[i][v] = __builtin_fmaf(part[i][v], s, acc[i][v]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else prepare(next, xn, 0);
    };
    auto step = [&](Codes& c, Codes& next, int t) {
        landed(next);
        if (t < T) work(c, next, t);
        fetch_codes(c, t + CD);
        // x of step t + 2 has landed; this step's loads (x of step t + 3, codes of step t + CD) stay in flight
        if (t + D < T) loads_left<kLoads>();
        else if (t + 2 < T) loads_left<2>();
        lds_barrier();
    };
    static_assert(D == 3, "the waits");
    if (2 < T) loads_left<kLoads>(); else loads_left<2>();
    landed(cq[0]);
    landed(cq[1]);
    {
        constexpr int L = 1 << BITS, W = BITS == 2 ? 2 : 4;       // entries; dwords per load
        uint32_t d[L / 2];
        if (p.lut) {
#pragma unroll
            for (int i = 0; i < L / 2; ++i) d[i] = tw[i / W][i % W];
        } else {
#pragma unroll
            for (int i = 0; i < L / 2; ++i)                       // the integer grid
                d[i] = f32_to_h16<F16>((float)(2 * i - L / 2)) | (f32_to_h16<F16>((float)(2 * i + 1 - L / 2)) << 16);
        }
        table.load(d);
    }
    lds_barrier();
#pragma unroll
    for (int t = 3; t < CD; ++t) {
        fetch_codes(cq[t], min(t, T - 1));
    }
    prepare(cq[0], xbase(0), 0);
    // (whole turns: a step past the last does nothing.  With a way out in the middle of a turn, or loads left out, the
    // compiler's wait at the top of the loop would be for all the codes in flight)
    for (int t = 0; t < T; t += CD) {
#pragma unroll
        for (int u = 0; u < CD; ++u) step(cq[u], cq[(u + 1) % CD], t + u);
    }
    offset_term((T - 1) / kPer * kPer, (T - 1) / kPer & 1);

    // ---- the WK parts of every tile meet in LDS; part i % WK finishes tile i
    if constexpr (WK > 1) {
        lds_barrier();                                            // the last step's buffers and group sums have been read
        auto slotaddr = [&](int i, int k) -> uint32_t { return (uint32_t)((((i * WK + k) * WN + wn) * 16) * 64 + lane) * 4u; };
#pragma unroll
        for (int i = 0; i < MT; ++i)
            if (wk != i % WK) {
#pragma unroll
                for (int v = 0; v < 16; ++v) *reinterpret_cast<lds_f32>(slotaddr(i, wk) + v * 256) = acc[i][v];
            }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < MT; ++i)
            if (wk == i % WK) {
                f32x16 sum = zero;
#pragma unroll
                for (int k = 0; k < WK; ++k) {
                    if (k == i % WK) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) sum[v] += acc[i][v];
                    } else {
#pragma unroll
                        for (int v = 0; v < 16; ++v) sum[v] += *reinterpret_cast<lds_f32>(slotaddr(i, k) + v * 256);
                    }
                }
                acc[i] = sum;
            }
    }
    // accumulator element v of a lane: row 8 (v / 4) + 4 h + v % 4 of its tile, column lane % 32
    const int64_t n = n0 + wn * 32 + r32;
    auto store_tile = [&](int i, const f32x16& r) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t m = m0 + i * 32 + (v >> 2) * 8 + h * 4 + (v & 3);
            if (m < p.M && n < p.N) p.y[m * p.ldy + n] = (uint16_t)f32_to_h16<F16>(r[v]);
        }
    };
    if (p.slabs == 1) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
            if (wk == i % WK) store_tile(i, acc[i]);
        return;
    }
    // ---- K slabs: fp32 sums to the workspace, where the tile's blocks meet and add them in slab order, each its part (one of them all, where
    //      they do not share the adding)
    const int64_t btile = (int64_t)blockIdx.y * p.tiles_n + tile;
    // (16 bytes per lane: four accumulator elements)
    float* const all = p.partial + btile * p.slabs * (ROWS * BN);
    const __amdgpu_buffer_rsrc_t ares = __builtin_amdgcn_make_buffer_rsrc(all, 0, p.slabs * (ROWS * BN) * 4, 0x00020000);
    auto quad = [&](int i, int v4) -> uint32_t { return (uint32_t)((((i * WN + wn) * 4 + v4) * 64 + lane) * 16); };
    constexpr int kAgent = 16;                                    // cache policy: coherent over the whole device
#pragma unroll
    for (int i = 0; i < MT; ++i)
        if (wk == i % WK) {
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const u32x4 q = {__float_as_uint(acc[i][4 * v4]), __float_as_uint(acc[i][4 * v4 + 1]), __float_as_uint(acc[i][4 * v4 + 2]), __float_as_uint(acc[i][4 * v4 + 3])};
                // (no scalar offset: with one the compiler takes it that the next instruction may overwrite the registers of the
                // data, which in the large-M kernel sent other values out)
                __builtin_amdgcn_raw_buffer_store_b128(q, ares, quad(i, v4) + (uint32_t)slab * (ROWS * BN * 4), 0, kAgent);
            }
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (threadIdx.x == 0) *reinterpret_cast<lds_u32>(0u) = meet(p.words + btile * p.word_step, p.slabs, p.parts, slab);
    lds_barrier();
    const uint32_t mine = __builtin_amdgcn_readfirstlane(*reinterpret_cast<lds_u32>(0u));
    // A unit is 1 KB, one wavefront's quads, numbered as they lie; part k has units k U / parts ..  UNITS of them at a time
    // are added over all slabs and stored.
    constexpr int U = MT * WN * 4;
    auto add_units = [&](auto units_, auto flight_, const int (&unit)[4]) {
        constexpr int UNITS = decltype(units_)::value, FLIGHT = decltype(flight_)::value;      // slabs whose loads are in flight together
        float sum[UNITS][4];
#pragma unroll
        for (int k = 0; k < UNITS; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[k][e] = 0.f;
        for (int sl = 0; sl < p.slabs; sl += FLIGHT) {
            u32x4 q[FLIGHT][UNITS];
#pragma unroll
            for (int f = 0; f < FLIGHT; ++f)
#pragma unroll
                for (int k = 0; k < UNITS; ++k)                // (not there: an offset beyond the buffer, 0 without a read)
                    q[f][k] = __builtin_amdgcn_raw_buffer_load_b128(ares, sl + f < p.slabs && unit[k] < U ? (uint32_t)((sl + f) * (ROWS * BN * 4) + unit[k] * 1024 + lane * 16) : 0x80000000u, 0, kAgent);
#pragma unroll
            for (int f = 0; f < FLIGHT; ++f)                   // (otherwise each load is put in front of its addition)
#pragma unroll
                for (int k = 0; k < UNITS; ++k) asm volatile("" : "+v"(q[f][k]));
#pragma unroll
            for (int f = 0; f < FLIGHT; ++f)
                if (sl + f < p.slabs)
#pragma unroll
                    for (int k = 0; k < UNITS; ++k)
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[k][e] += __uint_as_float(q[f][k][e]);
        }
#pragma unroll
        for (int k = 0; k < UNITS; ++k) {
            if (unit[k] >= U) break;
            const int64_t col = n0 + (unit[k] >> 2) % WN * 32 + r32;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t m = m0 + (unit[k] >> 2) / WN * 32 + (unit[k] & 3) * 8 + h * 4 + e;
                if (m < p.M && col < p.N) p.y[m * p.ldy + col] = (uint16_t)f32_to_h16<F16>(sum[k][e]);
            }
        }
    };
    int at = wave - kWaves;
    auto next_unit = [&]() -> int {
        do at += kWaves; while (at < U && !(mine >> (at * p.parts / U) & 1u));
        return at;
    };
    for (;;) {
        const int first = next_unit();
        if (first >= U) break;
        const int second = next_unit();
        if (second >= U) {
            add_units(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{}, {first, U, U, U});
            break;
        }
        const int third = next_unit(), fourth = next_unit();
        if (p.slabs <= 2) add_units(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{}, {first, second, third, fourth});
        else add_units(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{}, {first, second, third, fourth});
    }
}

template <int BITS, int MT, int WN, bool F16, bool FINE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void batch_kernel(const Params p) {
    batch_body<BITS, MT, WN, F16, FINE>(p);
}

// One translation unit per code width instantiates and launches the variants.
template <int BITS, int MT, bool F16, bool FINE> hipError_t launch_variant(const Params& p, int blocks_m, hipStream_t stream) {
    using S = Shape<MT, wn_of(MT)>;
    constexpr auto kernel = batch_kernel<BITS, MT, wn_of(MT), F16, FINE>;
    const hipError_t e = ensure_lds<kernel>(kLdsPerCu);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(p.tiles_n * p.slabs), (unsigned)blocks_m), dim3(kThreads), S::lds_bytes(p.sc_stride), stream, p);
    return hipGetLastError();
}
template <int BITS> hipError_t launch_bits(const Params& p, int mt, int blocks_m, bool f16, bool fine, hipStream_t stream) {
    auto go = [&](auto m) -> hipError_t {
        constexpr int MT = decltype(m)::value;
        return f16 ? launch_variant<BITS, MT, true, false>(p, blocks_m, stream)
             : fine ? launch_variant<BITS, MT, false, true>(p, blocks_m, stream) : launch_variant<BITS, MT, false, false>(p, blocks_m, stream);
    };
    switch (mt) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 3: return go(std::integral_constant<int, 3>{});
        default: return go(std::integral_constant<int, 4>{});
    }
}

}  // namespace batch

hipError_t launch_batch_bits4(const batch::Params& p, int mt, int blocks_m, bool f16, bool fine, hipStream_t stream);
hipError_t launch_batch_bits3(const batch::Params& p, int mt, int blocks_m, bool f16, bool fine, hipStream_t stream);
hipError_t launch_batch_bits2(const batch::Params& p, int mt, int blocks_m, bool f16, bool fine, hipStream_t stream);

}  // namespace any4
