// Host side of the packed-activation kernel for M <= 4 (any4_decode_pack.h): which problems it takes,
// its work split and the launch.
#include "any4_decode_pack.h"

namespace any4 {

// Whether and how the packed-activation kernel takes a problem; a pure function of its arguments.
PackPlan plan_pack(int64_t M, int64_t N, int64_t K, int bits, bool one_table, int cus) {
    PackPlan pl{};
    const int64_t G = K / kGroup;
    const int64_t tiles = (N + pack::kTile - 1) / pack::kTile;
    // (any2 tables are fetched 16 bytes at a time)
    if (M < 1 || M > 4 || tiles > 0x7FFFFFFF || cus < 1 || N * (2 << bits) < 16) return pl;
    // the kernel addresses every array with 32-bit offsets (padded to whole tiles for the re-laid-out codes)
    if (tiles * pack::kTile * (K * bits / 8) >= ((int64_t)1 << 31)) return pl;
    const int mp = M == 1 ? 1 : (M == 2 ? 2 : 4);
    const int passes = (int)((G + 4 * pack::kWaves - 1) / (4 * pack::kWaves));
    // K <= 4096 (one unit per wavefront and tile): nothing to gain over the streaming kernel, which needs no K
    // slabs there either and is 5 - 10 % faster on such shapes
    if (passes < 2) return pl;
    // K no multiple of 1024.  One block has all of a tile's K, so with few tiles most of the chip idles through it, where the streaming
    // kernel spreads its slabs: 195 x 28160 at M = 1 13.0 us, by the streaming kernel 8.3, 39 x 13952 at M = 2 9.4 and 6.8, 39 x 7424 at M = 4
    // 7.2 and 6.1; but 4096 x 4224 at M = 1 6.7 and 9.1, 28672 x 4224 19.9 and 26.6, 4096 x 14464 9.8 and 12.6.  The line lies where the two met
    // for each number of register sets (11 000 matrices of 16 .. 20000 rows, 0.4 % from the better of the two on average); any2, whose
    // tables cost the streaming kernel more, stays longer.  Long rows whose second round of tiles is nearly empty are not taken either
    // (4578 x 24064 22.9, 19.4).
    if (G % 8 != 0) {
        const int few = bits == 2 ? (mp == 1 ? (passes <= 4 ? 0 : cus * 3 / 16) : mp == 2 && passes > 2 ? cus / 4 : 0)
                      : mp == 1 ? (passes == 2 ? 0 : passes <= 4 ? cus / 4 : cus / 2)
                      : mp == 2 ? (passes == 2 ? cus / 16 : cus * 3 / 8) : cus / 4;
        if (tiles <= few || (bits != 2 && passes >= 5 && tiles > cus && tiles <= cus * 5 / 4)) return pl;
    }
    // the activations of a wavefront's groups must fit two register sets
    if (passes > 8 / mp) return pl;
    pl.mp = mp;
    pl.passes = passes;
    pl.tiles = tiles;
    if (pack::lds_bytes(bits, mp, passes, (int)G) > pack::kLdsPerCu) return pl;
    // as many blocks as the device holds at once (one or two per compute unit): more, started as others
    // finish, measured 5 - 25 % slower (every block pays for its first tile's latency)
    const int64_t slots = (int64_t)cus * (pack::two_blocks(bits, mp, passes) ? 2 : 1);
    pl.nblocks = (int)(tiles < slots ? tiles : slots);
    pl.ok = true;
    return pl;
}

hipError_t launch_decode_pack(const uint16_t* x, const uint32_t* codes, const uint16_t* lut,
                              const uint16_t* scale, const uint16_t* offset, int64_t M, int64_t N,
                              int64_t K, int bits, bool repacked, bool one_table, const PackPlan& pl, uint16_t* y,
                              hipStream_t stream) {
    if (!pl.ok || !lut) return hipErrorInvalidValue;
    pack::Params p{};
    p.x = x; p.codes = codes; p.lut = lut; p.scale = scale; p.offset = offset; p.y = y;
    p.N = N; p.K = K; p.M = (int)M; p.G = (int)(K / kGroup);
    p.tiles = (int)pl.tiles;
    p.nblocks = pl.nblocks;
    p.tpb = (int)(pl.tiles / pl.nblocks); p.trem = (int)(pl.tiles % pl.nblocks);
    p.codes_bytes = (int)((repacked ? pl.tiles * pack::kTile : N) * (K * bits / 8));
    p.lut_bytes = (int)((one_table ? 1 : N) * (2 << bits));
    p.one_table = one_table ? 1 : 0;
    p.so_bytes = (int)(N * (K / kGroup) * 2);
    if (bits == 4) return launch_pack_bits4(p, pl, repacked, stream);
    if (bits == 3) return launch_pack_bits3(p, pl, repacked, stream);
    return launch_pack_bits2(p, pl, repacked, stream);
}

}  // namespace any4
