// How the tiles of two products are shared out over the blocks of one launch (host only, plain C++: a test compiles it too).
#pragma once
#include <stdint.h>

namespace quartet {

// `tiles` tiles of two products at `cost` each on `blocks` blocks.  early = tiles[0] % blocks blocks have one tile of the first product more
// than the others, the late ones, which take tiles of the second for `extra` rounds alone before all blocks do (TileWalk); the partial
// last round falls on the late blocks first.
struct PairLevel {
    int64_t extra, early;
    double early_load, late_load;
    double busiest() const { return early_load > late_load ? early_load : late_load; }
};

// the most rounds that the second product's tiles can fill
inline int64_t pair_most_extra(const int64_t (&tiles)[2], int64_t blocks) {
    const int64_t late = blocks - tiles[0] % blocks;
    return (tiles[1] + late - 1) / late;
}

inline PairLevel pair_loads(const int64_t (&tiles)[2], const double (&cost)[2], int64_t blocks, int64_t extra) {
    const int64_t r = tiles[0] % blocks, late = blocks - r, few = tiles[0] / blocks;
    const int64_t rest = tiles[1] > extra * late ? tiles[1] - extra * late : 0, full = rest / blocks, part = rest % blocks;
    const int64_t late_tiles = rest > 0 ? extra + full + (part > 0) : pair_most_extra(tiles, blocks), early_tiles = full + (part > late);
    return PairLevel{extra, r, r > 0 ? (double)(few + 1) * cost[0] + (double)early_tiles * cost[1] : 0.0,
                     (double)few * cost[0] + (double)late_tiles * cost[1]};
}

// The extra rounds with the smallest load of the busiest block.  An early block's tile more makes up for cost[0] / cost[1] tiles of the
// second product, or for all of them where there are fewer: the best of the rounds around that number is the best of all (a test compares).
// Without that limit no extra round was left where the tiles are most unequal; backward passes of layers (tokens, in, out; us):
// 16640 x 1280 x 256 80.8 -> 73.2, 13856 x 5888 x 384 154.7 -> 140.4, Hadamard blocks of 256 16640 x 1280 x 256 98.3 -> 81.8, 15872 x 512 x 768 87.8 -> 78.0.
inline PairLevel pair_level(const int64_t (&tiles)[2], const double (&cost)[2], int64_t blocks) {
    PairLevel best = pair_loads(tiles, cost, blocks, 0);
    if (best.early == 0) return best;
    const int64_t most = pair_most_extra(tiles, blocks);
    const double rounds = cost[0] / cost[1];
    const int64_t level = rounds < (double)most ? (int64_t)rounds : most;
    for (int64_t x = level - 1; x < level + 3; ++x) {
        if (x < 1 || x > most) continue;
        const PairLevel here = pair_loads(tiles, cost, blocks, x);
        if (here.busiest() < best.busiest()) best = here;
    }
    return best;
}

}  // namespace quartet
