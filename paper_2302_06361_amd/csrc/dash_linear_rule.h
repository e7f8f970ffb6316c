// dash_linear_rule.h -- which kernel takes a dense or convolution layer, as a function of its sizes alone (host code)
#pragma once
#include <stdint.h>

namespace dash {

enum LinearForm { LINEAR_BY_SHAPE = 0, LINEAR_TILE4 = 1, LINEAR_TILE8 = 2, LINEAR_SPLIT = 3, LINEAR_MFMA = 4 };

struct LinearShape {
    int64_t npx, chunks;      // output pixels of the batch; 16-digit chunks of all primes together
    int nch;                  // ... and of the prime with the most
    int out_c, K;             // output channels, length of the reduction
    bool mfma;                // dense_mfma_wanted
};

// A grid holds fewer than 2^32 lanes, and k_linear_split has a wave of them per (output pixel, chunk, 8 channels); its unit index,
// 64 times smaller, then also stays within its 32-bit products.
inline bool linear_split_fits(const LinearShape& S) { return S.npx * ((S.out_c + 7) / 8) * S.nch < (1ll << 26); }

// Times in us, from runs over the shapes of the benchmark's and the paper's networks at batches of 1 to 64.
//   k_linear_split: about 3 + instructions of all its waves / 290 000: 190 per 256 of K, 360 for the addition over the wave
//   k_dense_mfma:   about 6 + 0.6 per round and 64 of K, 8 more per further round of 256 tiles (where its tiles fit the layer at all)
//   k_linear_tile:  0.6 per four of K (a chain of loads) while its waves are one round of the chip; eight channels per lane from 256
//                   waves on (6x6 over 28x28x1 -> 16, 139 waves: 11.4 with four, 14 with eight; 2x2 over 28x28x32 -> 32, 355 waves:
//                   50 and 33; 3x3 over 30x30x32 -> 32, 1420 waves: 226 and 114)
inline int linear_form_by_shape(const LinearShape& S) {
    const int64_t blocks8 = (S.out_c + 7) / 8;
    const double split = 3 + (double)S.npx * blocks8 * S.chunks * ((S.K + 255) / 256 * 190 + 360) / 290e3;
    if (S.mfma) {
        const int64_t tiles = (S.npx * S.chunks + 31) / 32 * ((S.out_c + 127) / 128), rounds = (tiles + 255) / 256;
        return split < 6 + 0.6 * rounds * ((S.K + 63) / 64) + 8 * (rounds - 1) ? LINEAR_SPLIT : LINEAR_MFMA;
    }
    const int64_t waves8 = S.npx * S.chunks * blocks8 / 64;
    const double tile = 4 + 0.6 * ((S.K + 3) / 4) * (1 + waves8 / 2048);
    if (split < tile) return LINEAR_SPLIT;
    return waves8 < 256 ? LINEAR_TILE4 : LINEAR_TILE8;
}

// forced: the tuning and test hook's form; k_dense_mfma only for layers that it can be chosen for.  Whichever way k_linear_split is
// chosen, it takes the layer only if a grid holds it.
inline int linear_form(int forced, const LinearShape& S) {
    const int f = forced && (forced != LINEAR_MFMA || S.mfma) ? forced : linear_form_by_shape(S);
    return f == LINEAR_SPLIT && !linear_split_fits(S) ? LINEAR_TILE8 : f;
}

}  // namespace dash
