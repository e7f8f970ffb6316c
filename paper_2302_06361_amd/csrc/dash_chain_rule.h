// dash_chain_rule.h -- how the tiles of a batch of carry gates are dealt to waves (host code)
#pragma once
#include <stdint.h>

namespace dash {

// Waves per unit (batch and repetition) of tiles: a multiple of the quantum that keeps the rounds of the resident waves full.  With V waves a unit
// the launch takes r = ceil(units V / resident) rounds of ceil(tiles / V) tiles each and half a tile's time of start and end: the smallest V of
// the least  r (ceil(tiles / V) + 1/2).  Only the largest V of each number of rounds is looked at: within a round the cost does not
// grow with V, and r rounds cost at least  units tiles / resident + r / 2,  which ends the search after a few (all multiples of the quantum up
// to 4 resident: 10 900 of them for m = 96, 45 us of host time a launch; this way 0.02 to 0.3 for up to 60 units).
inline uint32_t chain_waves(uint64_t tiles, uint32_t units, uint32_t quantum, uint32_t resident, uint32_t* tried = nullptr) {
    auto up = [&](uint64_t v) { return (v + quantum - 1) / quantum * quantum; };
    const uint64_t cap = up(tiles) < 4ull * resident ? up(tiles) : 4ull * resident / quantum * quantum;
    uint64_t best = quantum;
    double cost = 1e300;
    uint32_t looked = 0;
    for (uint64_t r = 1; (double)units * (double)tiles / resident + 0.5 * (double)r < cost; r++) {
        uint64_t V = r * resident / units / quantum * quantum;
        if (V > cap) V = cap;
        if (V == 0) {                                     // not even a quantum in r rounds
            r = ((uint64_t)units * quantum + resident - 1) / resident - 1;
            continue;
        }
        looked++;
        const uint64_t share = (tiles + V - 1) / V, rounds = (units * V + resident - 1) / resident;
        const double c = (double)rounds * ((double)share + 0.5);
        if (c < cost) { cost = c; best = up((tiles + share - 1) / share); }
        if (V == cap) break;
    }
    if (tried) *tried = looked;
    return (uint32_t)best;
}

}  // namespace dash
