// Host side of the kernel for a few dozen rows of x (any4_batch.h): its work split and the launch.
#include "any4.h"
#include "any4_batch.h"

namespace any4 {

// values of scales (and of offsets) per row of weights that a slab may have: what LDS holds
template <int MT> constexpr int max_slab_values() {
    using S = batch::Shape<MT, batch::wn_of(MT)>;
    static_assert(S::lds_bytes(S::sc_stride(S::MAX_VALUES)) <= batch::kLdsPerCu);
    static_assert(S::lds_bytes(S::sc_stride(S::MAX_VALUES + 1)) > batch::kLdsPerCu);
    return S::MAX_VALUES;
}
constexpr int kMaxSlabValues[4] = {max_slab_values<1>(), max_slab_values<2>(), max_slab_values<3>(), max_slab_values<4>()};

// The blocks of a tile share the adding of their slabs' sums where all blocks of a launch run at once and there is room for its words.
static size_t tile_sum_bytes(int mt) { return (size_t)(32 * mt) * (32 * batch::wn_of(mt)) * sizeof(float); }
static bool shares(int mt, int t, int s, int cus) {
    return (int64_t)t * s <= cus && splitk_counter_bytes(t) + (size_t)t * (s + 1) * tile_sum_bytes(mt) <= (size_t)ANY4_NOALLOC_SCRATCH_BYTES;
}

// Time in us of a launch of t tiles with s slabs of G groups.  Per round of blocks: their start and end (more with the
// chip full: `crowd`), four steps whose loads come with the start, and the rest, which take longer from a quarter of the chip
// on; a round that fills the chip to the last compute unit took longer by `even`.  Where slabs meet and share the adding: a meeting, more
// beyond eight slabs (whose parts the first eight add), and the traffic of all sums; where the last adds alone: four slabs at a time, and
// the traffic.  Up to 32 rows of x: constants fitted to times of 2100 matrices of 512 .. 60000 rows of weights, K = 1024 .. 28672.  The others:
// to 44 000 times of 10 000 matrices of 16 .. 60000 rows, K = 128 .. 28672, 6 - 7 % rms; the count taken is on average
// 0.4 (64 rows), 0.8 (96) and 1.2 % (128) slower than the best of those timed, below K = 1024 0.7 at most.  (Constants from K = 1024 on had
// shorter rows cut where they are faster in one piece: 9954 x 640 at M = 75 19.9 us for 15.5.)
struct Cost {
    double block, crowd, first, rest, rest_busy, even;
    double meeting, more, per_mb;          // the adding is shared
    double more_alone, per_mb_alone;       // it is not
};
constexpr Cost kCost[4] = {{4.94, 0.49, 1.45, 1.24, 1.38, 0.11, 2.08, 0.93, 0.43, 0.66, 0.79}, {5.23, 2.05, 1.49, 1.53, 1.77, 0.12, 2.59, 0.59, 0.30, 1.07, 0.47},
                           {6.80, 5.47, 1.54, 1.62, 1.80, 0.14, 3.40, 1.34, 0.15, 3.63, 0.36}, {7.46, 6.63, 1.85, 1.78, 2.05, 0.83, 3.46, 1.51, 0.12, 1.55, 0.34}};
static double meet_us(int mt, int t, int s, int cus) {
    const Cost& c = kCost[mt - 1];
    const double mb = (double)t * s * (double)tile_sum_bytes(mt) * 1e-6;
    if (s == 1) return 0.0;
    return shares(mt, t, s, cus) ? c.meeting + c.more * (double)((s - 1) / 8) + c.per_mb * mb : c.more_alone * (double)((s - 1) / 4) + c.per_mb_alone * mb;
}
static double launch_us(int mt, int t, int s, int G, int cus) {
    const Cost& c = kCost[mt - 1];
    const int wk = batch::kWaves / batch::wn_of(mt), steps = ((G + s - 1) / s + wk - 1) / wk, blocks = t * s, rounds = (blocks + cus - 1) / cus;
    const double busy = blocks < cus ? (double)blocks / cus : 1.0, quarter = busy < 0.25 ? 4 * busy : 1.0;
    const int first = steps < 4 ? steps : 4;
    return (double)rounds * (c.block + c.crowd * busy + c.first * first + (c.rest + (c.rest_busy - c.rest) * quarter) * (steps - first)) +
           (blocks % cus == 0 ? c.even : 0.0) + meet_us(mt, t, s, cus);
}

// Work split for groups of 128 and more and for groups of 64 (twice the scales to keep in LDS); a pure function of its arguments.
// A block takes 32 mt rows of x, 32 * wn rows of weights and one of `slabs` parts of K; a launch takes `tiles_n` times
// 32 * wn rows of weights.
//
// The sums of slabs stay within what any4_gemm_noalloc has, so that it takes every call.  Where those of the whole
// matrix do not fit, the rows of weights are cut into launches that follow each other in the same workspace, each as many
// whole rounds of blocks as fit.
static BatchPlans plan(int64_t M, int64_t N, int64_t K, int cus, bool whole) {
    BatchPlans both{};
    if (M < 1 || M > kBatchMaxM || cus < 1) return both;
    const int mt = (int)((M + 31) / 32), rows = 32 * mt, wn = batch::wn_of(mt), wk = batch::kWaves / wn, bn = 32 * wn;
    // 32-bit offsets inside a block's rows
    if (K * bn >= ((int64_t)1 << 31) || K * 2 * rows >= ((int64_t)1 << 31) || (N + bn - 1) / bn > ((int64_t)1 << 24)) return both;
    const int G = (int)(K / kGroup), tiles = (int)((N + bn - 1) / bn), most = kMaxSlabValues[mt - 1];   // values per row in LDS
    const int first = (G + most - 1) / most, first_fine = (2 * G + most / 2 * 2 - 1) / (most / 2 * 2);
    const size_t tile_bytes = tile_sum_bytes(mt);
    // Rows of up to 384 weights are faster in one piece whatever their number (measured 0.96 .. 1.00 of the best cut, 24 x 384 at M = 100 10.5 us and
    // 12.8).  Above 96 rows of x a matrix of up to 1024 x 1024 is not cut so that its calls go on needing no workspace, at the price of speed (23 us at 128
    // rows; in eight slabs 14).
    const bool whole_k = whole || G <= 3 || (mt > 3 && N <= 1024 && K <= 1024);
    auto take = [&](BatchPlan& pl, int part, int s, double us) {
        if (pl.ok && (whole_k || us >= pl.us)) return;
        pl = BatchPlan{};
        pl.ok = true;
        pl.mt = mt; pl.rows = rows;
        pl.tiles_n = part; pl.slabs = s;
        pl.us = us;
    };
    for (int s = first; s <= 64 && s <= (G + wk - 1) / wk; ++s) {
        // no slab count from here on can be better once as many rounds of blocks take too long
        const double rounds = (double)tiles * s / cus;
        if (both.fine.ok && kCost[mt - 1].block * (rounds > 1.0 ? rounds : 1.0) > (both.fine.us > both.plain.us ? both.fine.us : both.plain.us)) break;
        int part = tiles;
        if (s > 1 && (size_t)tiles * (s * tile_bytes + 8) + 256 > (size_t)ANY4_NOALLOC_SCRATCH_BYTES) {
            const int fit = (int)((ANY4_NOALLOC_SCRATCH_BYTES - 256) / (s * tile_bytes + 8)), full = fit * s / cus * cus;
            part = full >= s ? full / s : fit;
        }
        double us = launch_us(mt, part, s, G, cus);
        if (part < tiles) us = us * (tiles / part) + (tiles % part ? launch_us(mt, tiles % part, s, G, cus) : 0.0);
        take(both.plain, part, s, us);
        if (s >= first_fine) take(both.fine, part, s, us);
    }
    for (const bool fine : {false, true}) {
        BatchPlan& pl = fine ? both.fine : both.plain;
        if (!pl.ok) continue;
        // Up to 64 rows of x several launches have an alternative, blocks of 32 rows of x without slabs, which need no
        // workspace: taken unless the launches are clearly faster (100000 x 8192 at M = 64: 347 us, in two launches 270).
        if (mt == 2 && pl.tiles_n < tiles && (fine ? 2 * G : G) <= kMaxSlabValues[0]) {
            const double whole = launch_us(1, 2 * tiles, 1, G, cus);
            if (0.78 * whole <= pl.us) {
                pl.mt = 1; pl.rows = 32;
                pl.tiles_n = tiles; pl.slabs = 1;
                pl.us = whole;
            }
        }
        if (pl.slabs > 1) {
            const size_t sums = (size_t)pl.tiles_n * pl.slabs * tile_bytes;
            pl.counter_bytes = pl.sums_at = splitk_counter_bytes(pl.tiles_n);
            pl.shared = shares(mt, pl.tiles_n, pl.slabs, cus);
            if (pl.shared) {                                   // words in lines of their own, in the room of one more slab
                // (64 bytes a tile would do; so the size stays one counter and whole slabs of sums per tile, as it has always been)
                pl.counter_bytes = ((size_t)pl.tiles_n * kWordBytes + 255) / 256 * 256;
                pl.sums_at += (size_t)pl.tiles_n * tile_bytes;
            }
            pl.workspace = pl.sums_at + sums;
        }
    }
    return both;
}
BatchPlans plan_batch(int64_t M, int64_t N, int64_t K, int cus) { return plan(M, N, K, cus, false); }

// Calls without a workspace.  Until slabs shared their adding, rows of up to 18 groups were cut along K for few tiles only, or not at all: from how many
// tiles on they went without, for each number of groups (0: never; two gaps at 128 rows of x).  Longer rows did where they fit one piece and there
// are many tiles (not all of them; they may now).  Cutting is the faster way for some of them since, up to 1.7x, and any4_gemm_workspace_bytes
// asks for what that takes; a caller who brings none is served in one piece, in the time that it took then.
static int whole_mt(int64_t M, int G) {                          // height of the blocks, 0: no block holds the scales of a row
    const int mt = (int)((M + 31) / 32);
    return 2 * G <= kMaxSlabValues[mt - 1] / 2 * 2 ? mt : mt == 2 && 2 * G <= kMaxSlabValues[0] ? 1 : 0;
}
bool batch_goes_without(int64_t M, int64_t N, int64_t K) {
    constexpr unsigned char kFrom[4][18] = {{1, 1, 1, 1, 1, 1, 11, 11, 31, 31, 71, 71, 91, 91, 129, 129, 129, 129},
                                            {1, 1, 1, 1, 1, 1, 1, 1, 16, 16, 43, 43, 68, 68, 115, 115, 115, 115},
                                            {1, 1, 1, 1, 1, 1, 1, 3, 13, 26, 49, 79, 79, 90, 90, 118, 118, 128},
                                            {1, 1, 1, 1, 1, 1, 1, 1, 1, 8, 80, 0, 0, 0, 0, 0, 0, 0}};
    if (M <= 16 || M > kBatchMaxM || K > 128 * kGroup) return false;
    const int G = (int)(K / kGroup), mt = (int)((M + 31) / 32);
    const int64_t bn = 32 * batch::wn_of(mt), tiles = (N + bn - 1) / bn;
    if (G > 18) return tiles > 128 && whole_mt(M, G) > 0;
    if (mt == 4 && (G == 9 || G == 10) && tiles > (G == 9 ? 55 : 36) && tiles <= 64) return false;
    const int from = kFrom[mt - 1][G - 1];
    return from > 0 && tiles >= from;
}
BatchPlans plan_batch_whole(int64_t M, int64_t N, int64_t K, int cus) {
    BatchPlans p = plan(M, N, K, cus, true);
    const int mt = whole_mt(M, (int)(K / kGroup));
    if (p.plain.ok && mt > 0 && mt < p.plain.mt) {               // blocks of 32 rows of x for up to 64
        p.plain = plan(32, N, K, cus, true).plain;
        p.fine = p.plain;
    }
    return p;
}

hipError_t launch_batch(const uint16_t* x, const uint32_t* codes, const uint16_t* lut, const uint16_t* scale,
                        const uint16_t* offset, int64_t M, int64_t N, int64_t K, int bits, int lr, bool repacked, bool f16,
                        bool one_table, const BatchPlan& pl, uint16_t* y, void* workspace, hipStream_t stream) {
    const bool fine = lr < 0;
    if (!pl.ok || lr < -1 || (f16 && fine) || (pl.slabs > 1 && !workspace)) return hipErrorInvalidValue;
    batch::Params p{};
    p.x = x;
    p.words = static_cast<unsigned long long*>(workspace);
    p.word_step = pl.shared ? kWordBytes / 8 : 1;
    p.parts = pl.shared ? (pl.slabs < kMaxParts ? pl.slabs : kMaxParts) : 1;
    p.partial = pl.slabs > 1 ? reinterpret_cast<float*>(static_cast<char*>(workspace) + pl.sums_at) : nullptr;
    p.K = K; p.ldy = N; p.M = (int)M; p.G = (int)(K / kGroup);
    p.lr = fine ? 0 : lr;
    p.flags = (repacked ? 1 : 0) | (one_table ? 2 : 0);
    p.slabs = pl.slabs;
    const int groups = (p.G + pl.slabs - 1) / pl.slabs;           // of the largest slab
    p.sc_stride = batch::Shape<1, 4>::sc_stride(fine ? 2 * groups : groups);
    const int blocks_m = (int)((M + pl.rows - 1) / pl.rows);
    const int64_t bn = 32 * batch::wn_of(pl.mt), GS = fine ? 2 * (int64_t)p.G : p.G >> p.lr;   // scales per row
    // (launches follow each other on the stream and leave the workspace's counters clean)
    for (int64_t n0 = 0; n0 < N; n0 += pl.tiles_n * bn) {
        p.N = N - n0 < pl.tiles_n * bn ? N - n0 : pl.tiles_n * bn;
        p.tiles_n = (int)((p.N + bn - 1) / bn);
        p.codes = codes + n0 * row_words(K, bits);                // (both layouts: n0 is a multiple of 128 rows)
        p.lut = lut && !one_table ? lut + (n0 << bits) : lut;
        p.scale = scale + n0 * GS; p.offset = offset + n0 * GS; p.y = y + n0;
        const hipError_t e = bits == 4 ? launch_batch_bits4(p, pl.mt, blocks_m, f16, fine, stream)
                           : bits == 3 ? launch_batch_bits3(p, pl.mt, blocks_m, f16, fine, stream)
                                       : launch_batch_bits2(p, pl.mt, blocks_m, f16, fine, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace any4
