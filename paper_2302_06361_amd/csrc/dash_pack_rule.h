// dash_pack_rule.h -- how the tiles of packed table rows are dealt to waves (host code)
#pragma once
#include <stdint.h>

namespace dash {

struct PackShape {
    uint32_t run_log2;       // a wave takes 2^run_log2 tiles at a time
    uint32_t max_blocks;     // of four waves
};
// tiles: of all segments of the launch, 64 rows each (rows of one digit: 1024).
//
// A wave's cost is its walk past the segments (up to 96 of them, some 0.1 us each) and its tiles, one after the other.
// Few tiles: a wave each, then two.  (Four for all sizes, 4 primes, 300 values: unpacking 20.7 us instead of 9.6, packing 9.4 and 7.1.)
// More: no more waves than fit at a time, or the walk is paid over and over (12 primes, 1 000 values, 1024 blocks instead of up to 4096: packing 131 -> 44 us).
// Unpacking has seven blocks per CU (12 primes, 40 000 values: 1 277 us with 1024 blocks, 1 132 with 1792, 1 166 with 4096).  Where the walk
// is short (ReLU with 4 primes: 27 segments) a tile a wave, 4096 blocks (4 primes, ReLU, 10 000 values, 88 us in runs and 1792 blocks, 76 in tiles), and with
// up to 15 segments as many blocks as there are (2 primes, ReLU, 40 000 values, 40 us in runs and 1792 blocks, 30 in tiles; scaling, 160 000, 110 and 94;
// the other way round with 24: 5 primes, scaling, 10 000, 69 us in 4096 blocks and 92).
// Packing has eight per CU, but half of them read as fast: 8 primes, 5 000 values, 39 us with 1024 and 41 with 2048.  1536 from 2^16 tiles on (10 primes,
// 12 000 values: 299 us with 1024, 275 with 1536), 4096 where a wave has a tile for five or six segments: the ends of the waves even out
// (6 primes, ReLU, 20 000 values: 133 us with 1536, 126 with 4096; 12 primes, 5 000 values, the other way round: 147 and 188).
inline PackShape pack_shape(uint64_t tiles, uint32_t nseg, bool pack) {
    const uint32_t run = tiles >= 16384 ? 2u : tiles >= 8192 ? 1u : 0u;
    if (pack) return PackShape{run, tiles < 1u << 16 ? 1024u : tiles < 3072ull * nseg ? 1536u : 4096u};
    if (nseg <= 27) return PackShape{0u, nseg <= 15 ? 32768u : 4096u};
    return PackShape{run, 1792u};
}

}  // namespace dash
