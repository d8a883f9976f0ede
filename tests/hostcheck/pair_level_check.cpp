// pair_level (csrc/pair_level.h) against every number of extra rounds, over tile counts and costs of the launcher's range: prints the cases
// where another number gives the busiest block less, and returns their count (at most 255).
#include <cstdio>
#include <random>

#include "pair_level.h"

int main() {
    std::mt19937 rng(7);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    int bad = 0, extended = 0;
    for (int n = 0; n < 60000; ++n) {
        const int64_t blocks = n % 3 == 0 ? 512 : n % 3 == 1 ? 256 : 8 + (int64_t)(u(rng) * 300);
        const int64_t tiles[2] = {1 + (int64_t)(u(rng) * u(rng) * 1500), 1 + (int64_t)(u(rng) * u(rng) * 3000)};
        const double cost[2] = {1.0 + 60.0 * u(rng) * u(rng), 1.0 + 60.0 * u(rng) * u(rng)};
        const int64_t used = tiles[0] + tiles[1] < blocks ? tiles[0] + tiles[1] : blocks;
        const quartet::PairLevel got = quartet::pair_level(tiles, cost, used);
        const int64_t most = quartet::pair_most_extra(tiles, used);
        double best = quartet::pair_loads(tiles, cost, used, 0).busiest();
        if (tiles[0] % used != 0)
            for (int64_t x = 1; x <= most; ++x) {
                const double here = quartet::pair_loads(tiles, cost, used, x).busiest();
                if (here < best) best = here;
            }
        extended += got.extra > 0 && cost[0] / cost[1] > (double)most + 1.0;
        if (got.extra < 0 || got.extra > most || got.busiest() > best * (1.0 + 1e-12)) {
            if (++bad < 5) std::printf("tiles %ld %ld, cost %g %g, blocks %ld: %ld rounds %g, best %g\n", (long)tiles[0], (long)tiles[1], cost[0], cost[1], (long)used, (long)got.extra, got.busiest(), best);
        }
    }
    if (extended < 100) std::printf("only %d cases beyond what the second product can fill\n", extended);
    return bad + (extended < 100) > 255 ? 255 : bad + (extended < 100);
}
