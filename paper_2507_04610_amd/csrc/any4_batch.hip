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
    // Time in us of a launch with s slabs, constants measured with 4096 .. 28672 rows of weights and K = 4096 ..
    // 14336: start and end of a block, a step of its main loop, and where sums of slabs meet through memory
    // a wait for them and a share per slab (of a tile of 32 mt * bn sums).
    const double step[4] = {1.25, 1.65, 2.1, 2.6};
    const double per_slab = 0.9 * pl.mt * wn / 8.0;
    double best = 0;
    // (no slab count from here on can be better once its sums alone take too long)
    for (int64_t s = (G + most - 1) / most; s <= 64 && s <= (G + wk - 1) / wk && !(pl.ok && per_slab * (double)s > best); ++s) {
        const int64_t steps = ((G + s - 1) / s + wk - 1) / wk, rounds = (tiles * s + cus - 1) / cus;
        const double t = (double)rounds * (7.5 + step[pl.mt - 1] * (double)steps) + (s > 1 ? per_slab * (double)s : 0.0);
        if (!pl.ok || t < best) {
            best = t;
            pl.ok = true;
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
