// Compute-bound any-n GEMM for large M (prompt processing): table lookup in registers, looked-up tiles in LDS
// feeding bf16 matrix-core (MFMA) tiles with fp32 accumulation.
//
// y[m][n] = sum_k x[m][k] * w[n][k],  w[n][k] = LUT[n][code] * scale[n][k/128] + offset[n][k/128]
// (any4 paper, section 4.2: weights are dequantised on the fly before the matrix instruction;
// sections 2.4.1 / 2.5.2 define the table lookup and alpha * w_Q + beta).  The paper's own
// kernels stop at M = 16; this path is the large-M counterpart for CDNA4.
//
// Rounding a dequantised weight to bf16 costs up to 2^-8 relative per weight (1.7e-3 rms of the
// output, ~1e-2 * rms at the worst of a few million outputs), which is too much for the
// 1e-2 * rms output bound.  The kernel therefore never forms w.  Per group g of 128 weights it uses
//     sum_{k in g} x[m][k] w[n][k] = scale[n][g] * sum_{k in g} x[m][k] LUT[n][code[n][k]]
//                                  + offset[n][g] * X[m][g],      X[m][g] = sum_{k in g} x[m][k]
// The first sum multiplies two exact bf16 operands on the matrix cores (fp32 accumulate) and is
// scaled in fp32 on the vector ALU; the second term is a small extra GEMM over the "group"
// dimension whose left operand X is precomputed in fp32 and split into a bf16 high and low part
// (relative error 2^-16), and whose right operand is the bf16 offset itself.
//
// Block tile 256 (m) x 128 (n), K step 64, eight wavefronts in a 4 x 2 arrangement, each owning a
// 64 x 64 sub-tile as 2 x 2 v_mfma_f32_32x32x16_bf16 accumulators.  x, codes and scales are copied straight to LDS, three
// steps (groups) to a ring; a thread keeps to one weight row, whose table sits in its registers (any4_regtable.h), and
// turns 16 codes of a step into a piece of the looked-up tile, two steps to a ring.
//
// What bounds it: no unit by itself.  A K step takes a block 1500 cycles, of which the matrix cores are busy 1024, vector issue 900
// (a SIMD's two wavefronts: 46 lookup, 32 scale fold and 2 other instructions of 4 cycles each, and 16 matrix instructions, which
// hold the issue port for 8) and the LDS pipe about 1000 (700 for operands, codes and looked-up weights, the rest the copies): two
// thirds each, so the order of the instructions decides.
//   - Operands are read half a step ahead, the barrier stands in the middle of a step, between matrix instructions that
//     both have their operands: nothing waits behind it.
//   - A tile's two instructions of a half step follow each other, so that a finished group's sums have six matrix
//     instructions' time to be scaled before the next group writes their registers.
//   - Lookups, reads, writes and copies are spread over the instructions of a step.  Four copies at once at its start
//     held every wavefront until the address unit had taken them: 530 cycles a step.  The reads of a half step that ends at the
//     barrier come in its first four instructions: read one by one, the last held everybody there (1 %).
// The order is pinned by scheduling barriers, one per four matrix instructions (one per two: 1 % slower; none, and the
// compiler emits "all MFMAs, then all staging").  With x and codes through registers into padded LDS, operands read behind the
// barrier, and the fold at a group's end a step took 1940 cycles; a loop of nothing but this mix of matrix, vector and LDS
// instructions takes 1280.  The clock was 1.84 GHz then and is 1.5 - 1.65 now, by box.  N = 28672, K = 4096 at M = 2048: 540 -> 470 us;
// the four linears of an 8B layer at M = 2048 / 512: 1035 / 337 -> 908 / 296 us.
#include "any4_device.h"
#include "any4_internal.h"
#include "any4_lds_copy.h"
#include "any4_regtable.h"
#include "any4_splitk.h"
#include <type_traits>

namespace any4 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x4* lds_u4;
typedef __attribute__((address_space(3))) u32x2* lds_u2;
typedef __attribute__((address_space(3))) uint32_t* lds_u32;

constexpr int PBM = 256, PBN = 128, PBK = 64;
constexpr int PTHREADS = 512;
// LDS, bytes.  A tile is 64 rows of 64 values (one K step).  Its row r holds 16-byte chunk c at place c ^ place(r): the 16 lanes
// that LDS serves together in a read, one chunk of 16 rows, find it in 16 different columns of 256 bytes, and the 8 lanes of a
// write, the even or the odd chunks of two rows, in 8 different ones of 128.
constexpr uint32_t kTile = 64 * PBK * 2;
constexpr uint32_t kXSlots = 3, kWSlots = 2, kRing = 3;           // steps of x, steps of looked-up weights; groups of codes and scales
constexpr uint32_t kWAt = (PBM / 64) * kXSlots * kTile;           // x: [rows / 64][slot], then looked-up weights: [rows / 64][slot]
constexpr uint32_t kCAt = kWAt + (PBN / 64) * kWSlots * kTile;    // a group's codes of the block's 128 rows: [slot]
constexpr uint32_t kCSlot = PBN * kGroup / 2;
constexpr uint32_t kSAt = kCAt + kRing * kCSlot;                  // a group's scales of a wavefront's 64 columns, one a word: [slot][wavefront]
constexpr uint32_t kSSlot = 8 * 256;
constexpr uint32_t kLdsBytes = kSAt + kRing * kSSlot;
static_assert(kLdsBytes <= 160 * 1024);
__device__ __forceinline__ int place(int row) { return ((row >> 1) & 7) ^ (row & 1); }
// Longest rows whose offsets inside a wavefront are kept in 32 bits (31 rows of x, the furthest apart, stay below 2^31 bytes); WIDE
// kernels beyond, which form a 64-bit address at every copy and take longer for it: 300 x 2048, K = 132096 303 us, by a WIDE kernel 349.
// (With the line at 2^17 calls beyond were 1 - 3 % slower than with x and codes through registers, now 4 - 25 % faster on both sides.
// WIDE launches without K slices take 80 GB of operands at least.)
constexpr int64_t kNarrowK = 1 << 25;
constexpr int64_t furthest(int64_t K) { return 31 * 2 * K + PBK * 2; }
static_assert(furthest(kNarrowK) < ((int64_t)1 << 31) && furthest(2 * kNarrowK) > ((int64_t)1 << 31), "a power of two, as large as it goes");

#define ANY4_SB() __builtin_amdgcn_sched_barrier(0)

// X[m][g] = sum of the 128 activations of group g, in fp32, stored as two bf16 (high part,
// remainder) at xs[m][2g], xs[m][2g+1]; columns 2G .. KP-1 are zero.  16 lanes per (m, g).
// `fine`: groups of 64 activations, 8 lanes each.
// Also sets the words of K slices, so that those find no earlier call's leftovers: to an empty meeting (kMeetTag) where the slices
// meet, `word_step` words apart, otherwise to counts of 0.  Claiming such words by compare-and-swap, as the other kernels do, has
// every part of every slice of a tile queue up at one word (four linears at M = 512, scratch allocated by the call: 314 us against 295).
template <bool F16>
__global__ __launch_bounds__(256) void group_sums_kernel(const uint16_t* __restrict__ x, int64_t M,
                                                         int64_t K, int KP, int fine, uint16_t* __restrict__ xs,
                                                         unsigned long long* __restrict__ counters, int ncounters, int word_step) {
    for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < ncounters; c += (int64_t)gridDim.x * 256) counters[c * word_step] = word_step > 1 ? kMeetTag : 0ull;
    const int lanes = fine ? 8 : 16;
    const int64_t G = K / (8 * lanes);
    const int64_t unit = ((int64_t)blockIdx.x * 256 + threadIdx.x) / lanes;  // (m, g), g fastest
    const int sub = threadIdx.x & (lanes - 1);
    const bool live = unit < M * G;
    const int64_t u = live ? unit : 0;
    const uint4 v = reinterpret_cast<const uint4*>(x + u * (8 * lanes))[sub];    // x is [M][G][8 * lanes]
    float s = ((h16lo_to_f32<F16>(v.x) + h16hi_to_f32<F16>(v.x)) + (h16lo_to_f32<F16>(v.y) + h16hi_to_f32<F16>(v.y))) +
              ((h16lo_to_f32<F16>(v.z) + h16hi_to_f32<F16>(v.z)) + (h16lo_to_f32<F16>(v.w) + h16hi_to_f32<F16>(v.w)));
    // rotations inside rows of 16 lanes: after 1, 2, 4 a lane holds the sum of itself and the 7 lanes
    // before it (the last lane of a group of 8: its group); after 8, every lane holds the row's sum
    s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x121, 0xF, 0xF, false));
    s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x122, 0xF, 0xF, false));
    s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x124, 0xF, 0xF, false));
    if (!fine) s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x128, 0xF, 0xF, false));
    if (!live) return;
    const int64_t m = u / G, g = u % G;
    if (sub == lanes - 1) {
        const uint32_t hi = f32_to_h16<F16>(s);
        const uint32_t lo = f32_to_h16<F16>(s - h16_to_f32<F16>(hi));
        *reinterpret_cast<uint32_t*>(xs + m * KP + 2 * g) = hi | (lo << 16);
    }
    // zero padding of the row tail, done by the lanes of the row's last group
    if (g == G - 1)
        for (int c = (int)(2 * G) + sub; c < KP; c += lanes) xs[m * KP + c] = 0;
}

// FINE: groups of 64 weights - every K step is a group of its own (scale index 2g, 2g + 1 for the two
// steps of chunk g; the offset phase runs over 64-weight groups).  Otherwise groups of 128 << lr.
// F16: activations, table, scales, offsets and output are fp16 instead of bf16.
// NOLUT: 4-bit codes on the uniform grid (value = code - 8, the int4 format the paper compares with in
// section 4.2, last paragraph) without any table: a code c becomes the bf16 number 128 + c by OR-ing it
// into the mantissa of 128.0 (0x4300 | c) - two shifts and two and-or per pair of weights, 16 vector
// instructions for eight codes where the table takes 23 - and the surplus 136 * scale * X (X = the
// group sum of the activations) is taken off in the offset phase by two more passes over the same
// group sums whose right operands are the exact bf16 numbers -128 * scale and -8 * scale.
template <int BITS, bool FINE, bool F16, bool NOLUT, bool WIDE>
__global__ __launch_bounds__(PTHREADS, 1) void prefill_kernel(
    const uint16_t* __restrict__ x, const uint32_t* __restrict__ codes,
    const uint16_t* __restrict__ lut, const uint16_t* __restrict__ scale,
    const uint16_t* __restrict__ offset, const uint16_t* __restrict__ xsums, int KP,
    int64_t M, int64_t N, int64_t K, int lr, int flags, int gm, int tail_first, int tail_s, int word_step,
    unsigned long long* __restrict__ counters, float* __restrict__ partial, uint16_t* __restrict__ y) {
    constexpr int L = 1 << BITS;
    const bool repacked = flags & 1, one_table = flags & 2;     // re-laid-out codes / one table for all rows
    static_assert(!(F16 && FINE), "fp16 comes with groups of 128 and more");
    static_assert(!NOLUT || (BITS == 4 && !F16 && !FINE), "the table-free path: 4-bit codes, bf16, groups of 128");
    using op16x8 = std::conditional_t<F16, f16x8, bf16x8>;
    auto mma = [](const op16x8& a, const op16x8& b, const f32x16& c) -> f32x16 {
        if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    };
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, r32 = lane & 31, h = lane >> 5;
    const int64_t G = K / kGroup, RW = row_words(K, BITS);
    // Blocks below tail_first own a whole output tile.  The tiles of the last, partly filled round
    // of blocks are cut along K into tail_s slices of whole groups, one block each, so that the
    // round keeps every compute unit busy for 1 / tail_s of a tile's time; the slices' fp32 results
    // meet in the workspace and are added in slice order.
    int tile = blockIdx.x, slice = -1;
    int g_lo = 0, g_hi = (int)G;
    if (tile >= tail_first) {
        const int idx = tile - tail_first;
        tile = tail_first + idx / tail_s;
        slice = idx % tail_s;
        g_lo = (int)(slice * G / tail_s);
        g_hi = (int)((slice + 1) * G / tail_s);
    }
    const int64_t m0 = (int64_t)(tile % gm) * PBM, n0 = (int64_t)(tile / gm) * PBN;   // m fastest: an XCD keeps its rows of x
    const int T = 2 * g_hi;                                               // the block's K steps end here
    const int64_t GS = FINE ? 2 * G : G >> lr;                            // scales / offsets per row

    // ---- copies to LDS.  Rows past M or N are clamped (computed, never stored).  A lane's address is a base of its
    //      wavefront and a 32-bit offset; WIDE: an offset holds (row << 10 | bytes in the row).
    auto copy16 = [&](uint32_t lds, const void* base, uint32_t off, int64_t stride) {
        if constexpr (!WIDE) copy_to_lds(lds, base, off);
        else {
            asm volatile("" : "+v"(off));                      // (64-bit addresses are not kept in registers)
            copy_to_lds_from(lds, static_cast<const char*>(base) + (int64_t)(off >> 10) * stride + (off & 1023));
        }
    };
    auto offset_of = [&](int64_t row, int64_t stride, int bytes) -> uint32_t {
        return WIDE ? (uint32_t)(row << 10) + (uint32_t)bytes : (uint32_t)(row * stride) + (uint32_t)bytes;
    };
    // x: a wavefront moves 32 rows of a step, 8 to a copy
    const int64_t xrow = min(m0 + wave * 32, M - 1);
    const char* const xbase = reinterpret_cast<const char*>(x + xrow * K);
    auto x_offset = [&](int i, int l) -> uint32_t {
        return offset_of(min(m0 + wave * 32 + i * 8 + (l >> 3), M - 1) - xrow, 2 * K, ((l & 7) ^ place(i * 8 + (l >> 3))) * 16);
    };
    uint32_t xoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) xoff[i] = x_offset(i, lane);
    auto fetch_x = [&](int step, uint32_t slot, int i) {
        uint32_t off = xoff[i];
        if constexpr (WIDE) {                                  // (four registers less to keep)
            int l = lane;
            asm volatile("" : "+v"(l));
            off = x_offset(i, l);
        }
        copy16((wave >> 1) * (kXSlots * kTile) + slot * kTile + ((wave & 1) * 4 + i) * 1024, xbase + (int64_t)min(step, T - 1) * (PBK * 2), off, 2 * K);
    };
    // codes: pieces of 16 bytes, BITS to a row and group, one behind the other (re-laid-out: as they lie in units of
    // 16 rows); with less than 4 bits the last wavefronts repeat what the first ones copy
    const int cwave = wave % (2 * BITS), cpiece = cwave * 64 + lane, ufirst = cwave * 64 / (16 * BITS), rfirst = cwave * 64 / BITS;
    const int64_t units = (N + 15) >> 4;
    const int64_t crow = repacked ? min((n0 >> 4) + ufirst, units - 1) : min(n0 + rfirst, N - 1);
    const int64_t cstride = repacked ? G * (256 * BITS) : RW * 4;         // bytes from a unit / row to the next
    const char* const cbase = reinterpret_cast<const char*>(codes) + crow * cstride;
    const uint32_t coff = repacked ? offset_of(min((n0 >> 4) + cpiece / (16 * BITS), units - 1) - crow, cstride, cpiece % (16 * BITS) * 16)
                                   : offset_of(min(n0 + cpiece / BITS, N - 1) - crow, cstride, cpiece % BITS * 16);
    auto fetch_codes = [&](int g, uint32_t slot) {
        copy16(kCAt + slot * kCSlot + cwave * 1024, cbase + (int64_t)min(g, g_hi - 1) * (repacked ? 256 * BITS : 16 * BITS), coff, cstride);
    };
    // scales of the wavefront's columns (FINE: the pair of the group's halves, 4 bytes: rows are a whole number of pairs)
    const int64_t srow = min(n0 + wn * 64, N - 1);
    const uint16_t* const sbase = scale + srow * GS;
    uint32_t soff = (uint32_t)(min(n0 + wn * 64 + lane, N - 1) - srow);   // WIDE: the row alone
    if constexpr (!WIDE) soff *= (uint32_t)GS * 2;
    auto fetch_scales = [&](int g, uint32_t slot) {
        const int gg = min(g, g_hi - 1);
        const uint32_t lds = kSAt + slot * kSSlot + wave * 256;
        const uint16_t* const from = sbase + (FINE ? 2 * gg : gg >> lr);
        if constexpr (!WIDE) copy_values_to_lds<FINE>(lds, from, soff);
        else {
            uint32_t row = soff;
            asm volatile("" : "+v"(row));
            copy_values_to_lds_from<FINE>(lds, from + (int64_t)row * GS);
        }
    };

    // ---- where this lane reads and writes LDS (the kernel has no static LDS: dynamic LDS starts at 0)
    uint32_t ard[4], brd[4];                                              // operand kk of a step; + slot, + 32-row tile
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const uint32_t at = r32 * (PBK * 2) + (((2 * kk + h) ^ place(r32)) << 4);
        ard[kk] = wm * (kXSlots * kTile) + at;
        brd[kk] = kWAt + wn * (kWSlots * kTile) + at;
    }
    // looking up: thread -> (weight row, 16-code quarter of the K step)
    const int wrow = tid >> 2, wq = tid & 3;
    const int64_t wn_glob = min(n0 + wrow, N - 1);
    const uint32_t wwr = kWAt + (wrow >> 6) * (kWSlots * kTile) + (wrow & 63) * (PBK * 2);
    const uint32_t wwr0 = wwr + (((2 * wq) ^ place(wrow)) << 4), wwr1 = wwr + (((2 * wq + 1) ^ place(wrow)) << 4);
    // The thread's 16 codes inside a group: plain layout, word (2 * BITS) * (step % 2) + qword of the row (any3: from
    // bit qshift of it).  Tile-major layout (any4_repack): one half of piece 16 * q + n, q = 2 * (step % 2) + wq / 2, n = row % 16.
    const int qword = BITS == 4 ? 2 * wq : (BITS == 2 ? wq : (6 * wq) >> 2), qshift = BITS == 3 ? ((6 * wq) & 3) * 8 : 0;
    const uint32_t crd0 = kCAt + 4 * (repacked ? (wrow >> 4) * 64 * BITS + ((wq >> 1) * 16 + (wrow & 15)) * BITS + (BITS == 4 ? 2 : 1) * (wq & 1)
                                               : wrow * 4 * BITS + qword);
    const uint32_t crd1 = crd0 + 4 * (repacked ? 32 * BITS : 2 * BITS);

    f32x16 acc[2][2], part[2][2];
    f32x16 zero;
#pragma unroll
    for (int v = 0; v < 16; ++v) zero[v] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) { acc[i][j] = zero; part[i][j] = zero; }

    // NOLUT: codes 2p, 2p + 1 of a word of eight as the bf16 pair (128 + c, 128 + c')
    auto grid_pair = [&](uint32_t w, int pi) -> uint32_t {
        const uint32_t t = w >> (8 * pi);
        return (t & 0xFu) | ((t << 12) & 0xF0000u) | 0x43004300u;
    };
    RowTable<BITS> table;
    struct Words { uint32_t lo, hi; };                                    // a thread's 16 codes of a step
    auto read_codes = [&](uint32_t slot, int odd) -> Words {
        const uint32_t at = (odd ? crd1 : crd0) + slot * kCSlot;
        if constexpr (BITS == 4) {
            const u32x2 v = *reinterpret_cast<lds_u2>(at);
            return {v[0], v[1]};
        } else if constexpr (BITS == 3) {
            return {*reinterpret_cast<lds_u32>(at), *reinterpret_cast<lds_u32>(at + 4)};
        } else return {*reinterpret_cast<lds_u32>(at), 0u};
    };
    auto aligned = [&](const Words& q) -> Words {
        if constexpr (BITS != 3) return q;
        const unsigned long long v = (((unsigned long long)q.hi << 32) | q.lo) >> qshift;
        return {(uint32_t)v, (uint32_t)(v >> 32)};
    };
    // values of codes 8 c + 4 s .. + 3 of the thread's 16
    auto lookup = [&](const Words& q, int c, int s, uint32_t (&d)[4]) {
        if constexpr (NOLUT) {
            d[2 * s] = grid_pair(c ? q.hi : q.lo, 2 * s);
            d[2 * s + 1] = grid_pair(c ? q.hi : q.lo, 2 * s + 1);
        } else {
            const uint32_t w[2] = {q.lo, q.hi};
            table.half(w, c, s, d[2 * s], d[2 * s + 1]);
        }
    };
    auto write_chunk = [&](uint32_t slot, int c, const uint32_t (&d)[4]) {
        *reinterpret_cast<lds_u4>((c ? wwr1 : wwr0) + slot * kTile) = u32x4{d[0], d[1], d[2], d[3]};
    };

    // ---- first loads: the thread's table row and its first offsets, the first group sums, the codes of two groups and x
    //      of the first step; then what is waited for later
    const uint16_t* const trow = lut + (one_table ? 0 : wn_glob * L);     // (rows past N are clamped: they are never stored)
    uint32_t td[L / 2];
    if (!NOLUT && lut) {
#pragma unroll
        for (int i = 0; i < L / 4; ++i) { const u32x2 v = reinterpret_cast<const u32x2*>(trow)[i]; td[2 * i] = v[0]; td[2 * i + 1] = v[1]; }
    }
    const int og_lo = FINE ? 2 * g_lo : g_lo, og_hi = FINE ? 2 * g_hi : g_hi;      // this block's groups, in the units of xsums
    const bool by16 = (GS & 7) == 0 && (FINE || lr == 0);      // a thread's 8 offsets are one aligned piece
    const int64_t orow = wn_glob * GS;
    auto fetch8 = [&](const uint16_t* from, int g0) -> u32x4 { // groups g0 .. g0 + 7 of the thread's row (past the last: masked below)
        u32x4 v = {0, 0, 0, 0};
        if (by16) {
            v = *reinterpret_cast<const u32x4*>(from + orow + (g0 < og_hi ? g0 : 0));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int gg = min(g0 + e, og_hi - 1);
                v[e >> 1] |= (uint32_t)from[orow + (FINE ? gg : gg >> lr)] << (16 * (e & 1));
            }
        }
        return v;
    };
    auto fetch_sums = [&](int c0) {                            // 64 columns of the group sums of 32 rows of x
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t m = min(m0 + wave * 32 + i * 8 + (lane >> 3), M - 1);
            const int col = 2 * c0 + 8 * ((lane & 7) ^ place(i * 8 + (lane >> 3)));
            copy_to_lds_from((wave >> 1) * (kXSlots * kTile) + 2 * kTile + ((wave & 1) * 4 + i) * 1024, xsums + m * KP + (col < KP ? col : 0));
        }
    };
    const int oc_lo = og_lo / 32 * 32;
    u32x4 vo = fetch8(offset, oc_lo + 8 * wq), vs = {0, 0, 0, 0};
    if constexpr (NOLUT) vs = fetch8(scale, oc_lo + 8 * wq);
    fetch_sums(oc_lo);
    fetch_codes(g_lo, 0);
    fetch_codes(g_lo + 1, 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) fetch_x(2 * g_lo, 0, i);
    fetch_scales(g_lo, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) fetch_x(2 * g_lo + 1, 1, i);
    fetch_codes(g_lo + 2, 2);
    fetch_scales(g_lo + 1, 1);
    constexpr int kLater = 7;
    if constexpr (!NOLUT) {
        if (!lut) {
#pragma unroll
            for (int i = 0; i < L / 2; ++i)                    // no table: the integer grid
                td[i] = f32_to_h16<F16>((float)(2 * i - L / 2)) | (f32_to_h16<F16>((float)(2 * i + 1 - L / 2)) << 16);
        }
        table.load(td);
    }
    op16x8 a[2][2][2], b[2][2][2];                             // [set][operand][32-row tile]
    // operands kk = 2 * half + k of a step, n: 0 .. 7 in the order of their use
    auto read_op = [&](int set, uint32_t xslot, uint32_t wslot, int half, int n) {
        const int k = n < 4 ? n >> 1 : n & 1, i = n >> 2, kk = 2 * half + k;
        if (n < 4 ? !(n & 1) : n >= 6) a[set][k][i] = __builtin_bit_cast(op16x8, *reinterpret_cast<lds_u4>(ard[kk] + xslot * kTile + i * (kTile / 2)));
        else b[set][k][i] = __builtin_bit_cast(op16x8, *reinterpret_cast<lds_u4>(brd[kk] + wslot * kTile + i * (kTile / 2)));
    };
    // ---- offset term, while the first copies are on their way: K steps over the group dimension (activation group sums
    //      split into bf16 hi + lo in columns 2g, 2g + 1; both columns meet offset[n][g]); unscaled
    // NOLUT: three products over the group sums - right operand offset, then -128 * scale and -8 * scale (the
    // bf16 scale with 7 / 3 added to its exponent and the sign flipped: exact)
    constexpr int kKinds = NOLUT ? 3 : 1;
    auto look_up_step = [&](int odd) {                         // the weights of one of the first two steps
        const Words q = aligned(read_codes(0, odd));
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint32_t v[4];
            lookup(q, c, 0, v);
            lookup(q, c, 1, v);
            write_chunk(odd, c, v);
        }
    };
    for (int c0 = oc_lo;;) {
#pragma unroll
        for (int kind = 0; kind < kKinds; ++kind) {
            uint32_t d[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int gg = c0 + 8 * wq + e;
                uint32_t t = ((kind == 0 ? vo : vs)[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
                if (kind > 0) t = (t + (kind == 1 ? 0x0380u : 0x0180u)) ^ 0x8000u;
                d[e] = gg >= og_lo && gg < og_hi ? (t & 0xFFFFu) | (t << 16) : 0u;
            }
            *reinterpret_cast<lds_u4>(wwr0 + kTile) = u32x4{d[0], d[1], d[2], d[3]};
            *reinterpret_cast<lds_u4>(wwr1 + kTile) = u32x4{d[4], d[5], d[6], d[7]};
            if (c0 == oc_lo) loads_left<kLater>();
            else loads_left<0>();
            lds_barrier();
            if (kind == 0 && c0 == oc_lo) look_up_step(0);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int n = 0; n < 8; ++n) read_op(0, 2, 1, half, n);
#pragma unroll
                for (int n = 0; n < 8; ++n) {
                    const int k = n >> 2, i = (n >> 1) & 1, j = n & 1;
                    acc[i][j] = mma(a[0][k][i], b[0][k][j], acc[i][j]);
                }
            }
            lds_barrier();
        }
        c0 += 32;
        if (c0 >= og_hi) break;
        vo = fetch8(offset, c0 + 8 * wq);
        if constexpr (NOLUT) vs = fetch8(scale, c0 + 8 * wq);
        fetch_sums(c0);
    }
    fetch_x(2 * g_lo + 2, 2, 0);
    fetch_x(2 * g_lo + 2, 2, 1);
    look_up_step(1);                                           // (read behind the first barrier of the main loop)

    // ---- main loop.  Operands are read half a K step (32 values) ahead of the matrix instructions, into two sets of
    //      registers; a barrier stands between the instructions of a step's first half and those of its second.
    // One half of a step: eight matrix instructions, each tile's two one after the other, and what `between` puts
    // behind each of them
    auto half_step = [&](auto set_, auto first_, auto between) {
        constexpr int SET = decltype(set_)::value;
        constexpr bool FIRST = decltype(first_)::value;
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int i = n >> 2, j = (n >> 1) & 1, k = n & 1;
            // the wavefront that is behind in the phase goes first: both of a SIMD reach the barrier together
            if constexpr (SET == 1) {
                if (n == 0) __builtin_amdgcn_s_setprio(3);
                if (n == 4) __builtin_amdgcn_s_setprio(2);
            } else {
                if (n == 0) __builtin_amdgcn_s_setprio(1);
                if (n == 4) __builtin_amdgcn_s_setprio(0);
            }
            part[i][j] = mma(a[SET][k][i], b[SET][k][j], FIRST && k == 0 ? zero : part[i][j]);
            between(n);
            if ((n & 3) == 3) ANY4_SB();
        }
    };
    // elements lo .. hi - 1 of the 64 sums of a finished group enter the result
    float s0 = 0.f, s1 = 0.f;
    uint32_t sraw0 = 0, sraw1 = 0;
    auto fold = [&](int lo, int hi) {
#pragma unroll
        for (int e = lo; e < hi; ++e) {
            const int i = e >> 5, j = (e >> 4) & 1, v = e & 15;
            acc[i][j][v] = __builtin_fmaf(part[i][j][v], j ? s1 : s0, acc[i][j][v]);
        }
    };
    auto read_scales = [&](uint32_t slot) {
        const uint32_t at = kSAt + slot * kSSlot + wave * 256 + r32 * 4;
        sraw0 = *reinterpret_cast<lds_u32>(at);
        sraw1 = *reinterpret_cast<lds_u32>(at + 128);
    };
    auto widen_scales = [&](int odd) {
        s0 = h16_to_f32<F16>(FINE && odd ? sraw0 >> 16 : sraw0 & 0xFFFFu);
        s1 = h16_to_f32<F16>(FINE && odd ? sraw1 >> 16 : sraw1 & 0xFFFFu);
    };
    // the sums are folded between the last instructions on them (n >= 4 of the old half) and the next on the same registers
    auto pin = [&]() {                                         // (or the additions move to where their results are used)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) asm volatile("" : "+v"(acc[i][j]));
    };
    auto fold_old = [&](int n) { if (n >= 4) fold((n - 4) * 26 / 4, (n - 3) * 26 / 4); };
    auto fold_new = [&](int n) { if (n < 6) fold(26 + n * 38 / 6, 26 + (n + 1) * 38 / 6); };
    // end of a phase: the copies of x and codes issued before this phase have landed (six younger ones may be on their way)
    auto next_phase = [&]() {
        loads_left<6>();
        lds_barrier();
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using C2 = std::integral_constant<int, 2>;
    using Yes = std::true_type;
    using No = std::false_type;
    uint32_t wpk[4], held[4];
    // a group, steps 2g and 2g + 1; U: its place in the rings of three
    auto group = [&](auto u_, int g) {
        constexpr uint32_t U = decltype(u_)::value, X0 = 2 * U % 3, X1 = (2 * U + 1) % 3, X2 = (2 * U + 2) % 3, NEXT = (U + 1) % 3, AFTER = (U + 2) % 3;
        Words q, qn;
        // first half of step 2g
        half_step(C0{}, Yes{}, [&](int n) {
            if (n < 4) { read_op(1, X0, 0, 1, 2 * n); read_op(1, X0, 0, 1, 2 * n + 1); }
            if (n == 4) q = read_codes(NEXT, 0);
            if ((n & 3) == 1) fetch_x(2 * g + 2, X2, 2 + (n >> 2));
            fold_new(n);
        });
        pin();
        next_phase();
        // second half of step 2g; the first half of the weights of step 2g + 2
        q = aligned(q);
        half_step(C1{}, No{}, [&](int n) {
            read_op(0, X1, 1, 0, n);
            if (FINE && n == 0) read_scales(U);
            if (FINE && n == 4) widen_scales(0);
            if (FINE) fold_old(n);
            if (n == 1) lookup(q, 0, 0, wpk);
            if (n == 3) { lookup(q, 0, 1, wpk); write_chunk(0, 0, wpk); }
            if (n == 5) qn = read_codes(NEXT, 1);
            if ((n & 3) == 1) fetch_x(2 * g + 3, X0, n >> 2);
        });
        // first half of step 2g + 1; the second half of the weights of step 2g + 2, the first of those of 2g + 3
        half_step(C0{}, std::integral_constant<bool, FINE>{}, [&](int n) {
            if (n < 4) { read_op(1, X1, 1, 1, 2 * n); read_op(1, X1, 1, 1, 2 * n + 1); }
            if (FINE) fold_new(n);
            if (n == 1) lookup(q, 1, 0, wpk);
            if (n == 3) { lookup(q, 1, 1, wpk); write_chunk(0, 1, wpk); }
            if (n == 5) { qn = aligned(qn); lookup(qn, 0, 0, held); }
            if (n == 7) lookup(qn, 0, 1, held);
            if ((n & 3) == 1) fetch_x(2 * g + 3, X0, 2 + (n >> 2));
            if (n == 6) fetch_codes(g + 3, U);
            if (n == 7) fetch_scales(g + 2, AFTER);
        });
        next_phase();
        // second half of step 2g + 1
        half_step(C1{}, No{}, [&](int n) {
            read_op(0, X2, 0, 0, n);
            if (n == 0) { write_chunk(1, 0, held); if (!FINE) read_scales(U); }
            if (n == 1) lookup(qn, 1, 0, wpk);
            if (n == 3) { lookup(qn, 1, 1, wpk); write_chunk(1, 1, wpk); }
            if (n == 4) widen_scales(1);
            if ((n & 3) == 1) fetch_x(2 * g + 4, X1, n >> 2);
            fold_old(n);
        });
        pin();
    };
#pragma unroll
    for (int n = 0; n < 8; ++n) read_op(0, 0, 0, 0, n);
    for (int g = g_lo;;) {
        group(C0{}, g);
        if (++g == g_hi) break;
        group(C1{}, g);
        if (++g == g_hi) break;
        group(C2{}, g);
        if (++g == g_hi) break;
    }
    fold(26, 64);
    loads_left<0>();                                           // (what was copied past the last step)

    lds_barrier();                                             // LDS is free: the whole block's copies have landed, its operands have been read

    // ---- store (accumulator element v of a lane is row 8*(v/4) + 4*(lane/32) + v%4, column lane%32 of its
    //      32 x 32 tile)
    // Rows of y that are whole 16-byte pieces take 8 stores of 16 bytes per lane through LDS: 64 stores of 2 bytes took a block
    // 10 000 cycles, 8 % of its time at K = 4096, in which nothing else runs on the compute unit.
    const bool by8 = (N & 7) == 0;
    constexpr uint32_t kRow = 64 * 2 + 16, kWaveOut = 64 * kRow;          // a wavefront's 64 x 64 outputs, rows spread over the banks
    auto put_tile = [&](int i, int j, const f32x16& r) {
        // two rows (v, v + 1) of one column -> two columns of one row: even lanes keep row v, odd ones row v + 1
        const uint32_t sel = lane & 1 ? 0x03020706u : 0x05040100u;
        const uint32_t at = wave * kWaveOut + (i * 32 + 4 * h + (lane & 1)) * kRow + j * 64 + (r32 >> 1) * 4;
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            const uint32_t own = f32x2_to_h16x2<F16>(r[v], r[v + 1]);
            const uint32_t other = __builtin_amdgcn_update_dpp(0, own, 0xB1 /*quad_perm 1 0 3 2*/, 0xF, 0xF, false);
            *reinterpret_cast<lds_u32>(at + ((v >> 2) * 8 + (v & 3)) * kRow) = vperm(other, own, sel);
        }
    };
    // 16 bytes of a row of them to y (the wavefront's own part of LDS)
    auto store_piece = [&](int row, int chunk) {
        const u32x4 v = *reinterpret_cast<lds_u4>(wave * kWaveOut + row * kRow + chunk * 16);
        const int64_t m = m0 + wm * 64 + row, n = n0 + wn * 64 + chunk * 8;
        if (m < M && n < N) *reinterpret_cast<u32x4*>(y + m * N + n) = v;
    };
    auto store_tile = [&](int i, int j, const f32x16& r) {
        const int64_t n = n0 + wn * 64 + j * 32 + r32;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t m = m0 + wm * 64 + i * 32 + (v >> 2) * 8 + h * 4 + (v & 3);
            if (m < M && n < N) y[m * N + n] = (uint16_t)f32_to_h16<F16>(r[v]);
        }
    };
    auto finish = [&](int i, int j, const f32x16& r) {
        if (by8) put_tile(i, j, r);
        else store_tile(i, j, r);
    };
    if (slice < 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) finish(i, j, acc[i][j]);
        if (by8) {
#pragma unroll
            for (int p = 0; p < 8; ++p) store_piece(p * 8 + (lane >> 3), lane & 7);
        }
        return;
    }
    // ---- a K slice: its fp32 sums go to the workspace, where those of all slices are added.  Done by the last block alone that took
    //      22 000 cycles for four slices, nearly as long as their loop over K at K = 4096 (a compute unit reads 17 - 20 bytes a cycle of
    //      what others wrote).  Where the words have cache lines of their own (not with groups of 64) the slices meet and share the adding (any4_splitk.h).
    //      Otherwise the four 32 x 32 tiles of the wavefronts are four parts (two of two slices), which the last slice to arrive with one adds up, and
    //      the slices bring the parts in different orders, so that blocks that end together share the adding too; a part costs a trip to memory.
    //      Parts by the last to bring them -> a meeting, us: 4096 x 4096 at M = 200 (eight slices) 30.1 -> 28.0, at M = 512 (four) 38.7 -> 38.0, 6144 x 4096
    //      at M = 512 (two) 48.7 -> 47.2, 1000 x 4096 at M = 777 35.6 -> 29.7.
    float* const all = partial + (int64_t)(tile - tail_first) * tail_s * (PBM * PBN);
    const __amdgpu_buffer_rsrc_t ares = __builtin_amdgcn_make_buffer_rsrc(all, 0, tail_s * (PBM * PBN) * 4, 0x00020000);
    auto quad = [&](int part, int v4) -> uint32_t { return (uint32_t)((((part * 4 + v4) * 8 + wave) * 64 + lane) * 16); };   // 16 bytes: four elements
    constexpr int kAgent = 16;                                 // cache policy: coherent over the whole device
    // (a word per tile, word_step words apart, set by group_sums_kernel; without a meeting a count of 16 bits per part)
    unsigned long long* const word = counters + (tile - tail_first) * word_step;
    unsigned long long before = 0;
    auto arrive = [&](int part) { before = __hip_atomic_fetch_add(word, 1ull << (16 * part), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> (16 * part); };
    const bool shared = word_step > 1;
    const int sh = shared ? 2 : tail_s == 2 ? 1 : 0, parts = 4 >> sh;    // part p: tiles p << sh ..
#pragma unroll 1
    for (int r = 0; r < parts; ++r) {
        // (the arrival with the part before: its trip to memory goes with that of this part's stores)
        if (r > 0 && tid == (r - 1) * 64) arrive((r - 1 + slice) & (parts - 1));
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k >> sh == ((r + slice) & (parts - 1))) {
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    // through an opaque copy: with the accumulator vector itself as the source of the
                    // stores the compiler copies all 64 accumulators inside the main loop on every iteration
                    const f32x16& c = acc[k >> 1][k & 1];
                    u32x4 q = {__float_as_uint(c[4 * v4]), __float_as_uint(c[4 * v4 + 1]), __float_as_uint(c[4 * v4 + 2]), __float_as_uint(c[4 * v4 + 3])};
                    asm volatile("" : "+v"(q));
                    // (no scalar offset: with one the compiler takes it that the next instruction may overwrite the registers of
                    // the data, and the upper halves of some lanes' did not get out)
                    __builtin_amdgcn_raw_buffer_store_b128(q, ares, quad(k, v4) + (uint32_t)slice * (PBM * PBN * 4), 0, kAgent);
                }
            }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this thread's sums are out
        lds_barrier();                                         // ... and so are the whole block's
    }
    uint32_t todo = 0;                                         // the wavefront's 32 x 32 tiles (bits) that it is to add up
    if (shared) {
        // the tiles of all wavefronts, numbered wavefront by wavefront, are as many parts as there are slices
        if (tid == 0) *reinterpret_cast<lds_u32>(0u) = meet(word, tail_s, tail_s, slice);
        lds_barrier();
        const uint32_t mine = __builtin_amdgcn_readfirstlane(*reinterpret_cast<lds_u32>(0u));
#pragma unroll
        for (int k = 0; k < 4; ++k) todo |= (mine >> (((k * 8 + wave) * tail_s) >> 5) & 1u) << k;
    } else {
        if (tid == (parts - 1) * 64) arrive((parts - 1 + slice) & (parts - 1));
        if (lane == 0 && wave < parts) *reinterpret_cast<lds_u32>((uint32_t)((wave + slice) & (parts - 1)) * 4u) = (before & 0xFFFFull) == (unsigned long long)(tail_s - 1) ? 1u : 0u;
        lds_barrier();
        const u32x4 mine = *reinterpret_cast<lds_u4>(0u);      // the parts that this block was the last to bring
#pragma unroll
        for (int k = 0; k < 4; ++k) todo |= __builtin_amdgcn_readfirstlane(sh ? mine[k >> 1] : mine[k]) << k;
    }
    lds_barrier();                                             // (the outputs go over it)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (!(todo >> k & 1u)) continue;
        f32x16 sum = zero;
        constexpr int FLIGHT = 4;                              // slices whose loads are in flight together
        for (int sl = 0; sl < tail_s; sl += FLIGHT) {
            u32x4 q[FLIGHT][4];
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u)                   // (past the last slice: an offset beyond the buffer, 0 without a read)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const bool in = sl + u < tail_s;           // (the scalar offset takes no part in the check of the range)
                    q[u][v4] = __builtin_amdgcn_raw_buffer_load_b128(ares, in ? quad(k, v4) : 0x80000000u, in ? (sl + u) * (PBM * PBN) * 4 : 0, kAgent);
                }
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u)                   // (otherwise each load is put in front of its addition)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) asm volatile("" : "+v"(q[u][v4]));
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[v] += __uint_as_float(q[u][v >> 2][v & 3]);
        }
        finish(k >> 1, k & 1, sum);
        if (by8) {
#pragma unroll
            for (int p = 0; p < 2; ++p) store_piece((k >> 1) * 32 + p * 16 + (lane >> 2), (k & 1) * 4 + (lane & 3));
        }
    }
}

// Work split: whole tiles, and K slices for the tiles of a last round that would leave more than
// half of the compute units idle (also the only round of a small problem).
PrefillPlan plan_prefill(int64_t M, int64_t N, int64_t K, int cus) {
    PrefillPlan p{};
    const int64_t gm = (M + PBM - 1) / PBM, gn = (N + PBN - 1) / PBN, G = K / kGroup;
    p.gm = gm;
    p.tiles = gm * gn;
    p.tail_tiles = 0;
    p.tail_s = 1;
    const int64_t r = p.tiles % cus;
    if (r > 0) {
        int64_t sl = cus / r;
        if (sl > 8) sl = 8;
        if (sl > G / 4) sl = G / 4;                            // at least four groups (eight K steps) per slice
        if (sl >= 2) { p.tail_tiles = r; p.tail_s = (int)sl; }
    }
    // (sized for groups of 64, the largest case: the workspace does not depend on the group size)
    p.xsums_bytes = ((size_t)M * (size_t)prefill_kp(K, true) * sizeof(uint16_t) + 255) / 256 * 256;
    p.partial_bytes = (size_t)p.tail_tiles * (size_t)p.tail_s * (PBM * PBN) * sizeof(float);
    p.counter_bytes = p.tail_tiles ? splitk_counter_bytes(p.tail_tiles) : 0;
    return p;
}

hipError_t launch_prefill(const uint16_t* x, const uint32_t* codes, const uint16_t* lut,
                          const uint16_t* scale, const uint16_t* offset,
                          int64_t M, int64_t N, int64_t K, int bits, int lr, bool repacked, bool f16, bool one_table, int cus,
                          uint16_t* y, void* workspace, hipStream_t stream) {
    const PrefillPlan pp = plan_prefill(M, N, K, cus);
    const bool fine = lr < 0;
    if (lr < -1 || (f16 && fine)) return hipErrorInvalidValue;
    const int64_t sblocks = (M * (K / 8) + 255) / 256;         // one lane per 8 activations
    const int64_t nblocks = pp.tiles - pp.tail_tiles + pp.tail_tiles * pp.tail_s;
    if (pp.gm > 0x7FFFFFFF || nblocks > 0x7FFFFFFF || sblocks > 0x7FFFFFFF || K / kGroup > 0x1FFFFFFF) return hipErrorInvalidValue;
    const int KP = prefill_kp(K, fine);
    uint16_t* xsums = static_cast<uint16_t*>(workspace);
    unsigned long long* counters = reinterpret_cast<unsigned long long*>(static_cast<char*>(workspace) + pp.xsums_bytes);
    float* partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + pp.xsums_bytes + pp.counter_bytes);
    // A cache line of 64 bytes to a tile's word where the group sums leave room for it (they are half as many with groups of 128 and
    // more): with eight tiles' words in one, all of whose slices come at once, 4096 x 4096 at M = 200 took 34.0 us, 31.2 so; 6144 x 4096
    // at M = 512 49.2, 48.7.
    int word_step = 1;
    const size_t sums = ((size_t)M * KP * sizeof(uint16_t) + 255) / 256 * 256;
    if (sums + (size_t)pp.tail_tiles * 64 <= pp.xsums_bytes) {
        word_step = 8;
        counters = reinterpret_cast<unsigned long long*>(static_cast<char*>(workspace) + sums);
    }
    const dim3 grid((unsigned)nblocks), block(PTHREADS);
    const int gm = (int)pp.gm, tail_first = (int)(pp.tiles - pp.tail_tiles), tail_s = pp.tail_s;
    // the LDS limit first: whatever can be refused is refused before anything is enqueued
    hipError_t e = hipSuccess;
#define ANY4_PREFILL_F(B, F, H, NL, W)                                                                              \
    do {                                                                                                          \
        e = ensure_lds<prefill_kernel<B, F, H, NL, W>>((int)kLdsBytes);                                    \
        if (e != hipSuccess) return e;                                                                            \
        if (f16) hipLaunchKernelGGL(group_sums_kernel<true>, dim3((unsigned)sblocks), dim3(256), 0, stream, x, M, K, KP, 0, xsums, counters, (int)pp.tail_tiles, word_step); \
        else hipLaunchKernelGGL(group_sums_kernel<false>, dim3((unsigned)sblocks), dim3(256), 0, stream, x, M, K, KP, fine ? 1 : 0, xsums, counters, (int)pp.tail_tiles, word_step); \
        e = hipGetLastError();                                                                                    \
        if (e != hipSuccess) return e;                                                                            \
        hipLaunchKernelGGL((prefill_kernel<B, F, H, NL, W>), grid, block, kLdsBytes, stream, x, codes, lut, scale, \
                           offset, xsums, KP, M, N, K, F ? 0 : lr, (repacked ? 1 : 0) | (one_table ? 2 : 0), gm, tail_first, tail_s, word_step, counters, partial, y); \
    } while (0)
#define ANY4_PREFILL_W(B, W)                                                                                      \
    do {                                                                                                          \
        if (B == 4 && !lut && !f16 && !fine && lr == 0) ANY4_PREFILL_F(4, false, false, true, W);                 \
        else if (f16) ANY4_PREFILL_F(B, false, true, false, W);                                                   \
        else if (fine) ANY4_PREFILL_F(B, true, false, false, W);                                                  \
        else ANY4_PREFILL_F(B, false, false, false, W);                                                           \
    } while (0)
#define ANY4_PREFILL(B)                                                                                           \
    do {                                                                                                          \
        if (K > kNarrowK) ANY4_PREFILL_W(B, true);                                                                \
        else ANY4_PREFILL_W(B, false);                                                                            \
    } while (0)
    switch (bits) {
        case 4: ANY4_PREFILL(4); break;
        case 3: ANY4_PREFILL(3); break;
        default: ANY4_PREFILL(2); break;
    }
#undef ANY4_PREFILL_F
#undef ANY4_PREFILL_W
#undef ANY4_PREFILL
    return hipGetLastError();
}

}  // namespace any4
