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

// Work split; a pure function of its arguments.  A block takes 32 mt rows of x, 32 * wn rows of weights and one
// of `slabs` parts of K.
BatchPlan plan_batch(int64_t M, int64_t N, int64_t K, bool fine, int cus) {
    BatchPlan pl{};
    if (M < 1 || M > kBatchMaxM || cus < 1) return pl;
    pl.mt = (int)((M + 31) / 32);
    pl.rows = 32 * pl.mt;
    const int wn = batch::wn_of(pl.mt), wk = batch::kWaves / wn, bn = 32 * wn;
    const int64_t G = K / kGroup, tiles = (N + bn - 1) / bn;
    const int values = kMaxSlabValues[pl.mt - 1];
    const int64_t most = fine ? values / 2 : values;              // groups whose scales and offsets LDS holds
    // 32-bit offsets inside a block's rows
    if (K * bn >= ((int64_t)1 << 31) || K * 2 * pl.rows >= ((int64_t)1 << 31) || tiles > ((int64_t)1 << 24)) return pl;
    // Time in us of a launch with s slabs: per round of blocks their start and end, and their steps (which take longer
    // the more of the chip is busy); where slabs meet, a wait for their sums, eight slabs at a time, and the traffic of
    // all sums; a flight of seven or eight slabs takes longer by `full`.  Constants fitted to 1100 problems of 128 .. 128256
    // rows of weights, K = 128 .. 28672, each with up to 14 slab counts: times within 7 % rms, the count taken on
    // average 1 % slower than the best, 10 % at worst.
    struct Cost { double block, step_idle, step_busy, flight, more, full, per_mb; int64_t least; };   // (more: flights after the first; least: steps)
    constexpr Cost cost[4] = {{6.0, 1.1, 1.3, 2.1, 1.0, 0.45, 1.15, 1}, {8.7, 0.9, 1.62, 2.2, 4.8, 0.7, 0.59, 2},
                              {9.2, 1.4, 1.94, 7.8, 7.2, 1.0, 0.32, 1}, {11.7, 1.45, 2.3, 8.6, 8.3, 1.9, 0.23, 1}};
    const auto meet_us = [&](int64_t t, int64_t s) -> double {
        const Cost& c = cost[pl.mt - 1];
        return s == 1 ? 0.0 : c.flight + c.more * (double)((s - 1) / 8) + (s % 8 == 0 || s % 8 == 7 ? c.full : 0.0) + c.per_mb * (double)(t * s * pl.rows * bn) * 4e-6;
    };
    const auto launch_us = [&](int64_t t, int64_t s) -> double {
        const Cost& c = cost[pl.mt - 1];
        const int64_t own = ((G + s - 1) / s + wk - 1) / wk, steps = own > c.least ? own : c.least, rounds = (t * s + cus - 1) / cus;
        const double busy = t * s < cus ? (double)(t * s) / cus : 1.0;
        return (double)rounds * (c.block + (c.step_idle + (c.step_busy - c.step_idle) * busy) * (double)steps) + meet_us(t, s);
    };
    // (no slab count from here on can be better once its sums alone take too long)
    for (int64_t s = (G + most - 1) / most; s <= 64 && s <= (G + wk - 1) / wk && !(pl.ok && meet_us(tiles, s) > pl.us); ++s) {
        const double t = launch_us(tiles, s);
        if (!pl.ok || t < pl.us) {
            pl.ok = true;
            pl.us = t;
            pl.slabs = (int)s;
        }
    }
    if (!pl.ok) return pl;
    pl.tiles_n = (int)tiles;
    if (pl.slabs > 1) {
        pl.counter_bytes = splitk_counter_bytes(tiles);
        pl.workspace = pl.counter_bytes + (size_t)tiles * pl.slabs * pl.rows * bn * sizeof(float);
    }
    // The sums of slabs stay within what any4_gemm_noalloc has, so that it takes what the kernels before this one
    // took.  Beyond (100000 rows of weights and more, at up to 64 rows of x) blocks of 32 rows of x go without slabs;
    // the weights are then read twice, still less than the matrix-core kernel's four-fold padding of x costs.
    if (pl.workspace > (size_t)ANY4_NOALLOC_SCRATCH_BYTES) {
        const int v1 = kMaxSlabValues[0];
        if (M > 64 || G > (fine ? v1 / 2 : v1)) return BatchPlan{};
        pl.mt = 1;
        pl.rows = 32;
        pl.slabs = 1;
        pl.counter_bytes = pl.workspace = 0;
    }
    return pl;
}

hipError_t launch_batch(const uint16_t* x, const uint32_t* codes, const uint16_t* lut, const uint16_t* scale,
                        const uint16_t* offset, int64_t M, int64_t N, int64_t K, int bits, int lr, bool repacked, bool f16,
                        bool one_table, const BatchPlan& pl, uint16_t* y, void* workspace, hipStream_t stream) {
    const bool fine = lr < 0;
    if (!pl.ok || lr < -1 || (f16 && fine) || (pl.slabs > 1 && !workspace)) return hipErrorInvalidValue;
    batch::Params p{};
    p.x = x; p.codes = codes; p.lut = lut; p.scale = scale; p.offset = offset; p.y = y;
    p.counters = static_cast<unsigned long long*>(workspace);
    p.partial = pl.slabs > 1 ? reinterpret_cast<float*>(static_cast<char*>(workspace) + pl.counter_bytes) : nullptr;
    p.N = N; p.K = K; p.M = (int)M; p.G = (int)(K / kGroup);
    p.lr = fine ? 0 : lr;
    p.flags = (repacked ? 1 : 0) | (one_table ? 2 : 0);
    p.slabs = pl.slabs; p.tiles_n = pl.tiles_n;
    const int groups = (p.G + pl.slabs - 1) / pl.slabs;           // of the largest slab
    p.sc_stride = batch::Shape<1, 4>::sc_stride(fine ? 2 * groups : groups);
    const int blocks_m = (int)((M + pl.rows - 1) / pl.rows);
    if (bits == 4) return launch_batch_bits4(p, pl.mt, blocks_m, f16, fine, stream);
    if (bits == 3) return launch_batch_bits3(p, pl.mt, blocks_m, f16, fine, stream);
    return launch_batch_bits2(p, pl.mt, blocks_m, f16, fine, stream);
}

}  // namespace any4
