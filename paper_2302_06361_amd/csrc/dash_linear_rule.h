// dash_linear_rule.h -- which kernel takes a dense or convolution layer, as a function of its sizes alone (host code)
#pragma once
#include <stdint.h>

namespace dash {

// k_linear_tile with 4, 8, 1 channels per lane; k_linear_split with a wave and 8 channels; k_dense_mfma; k_linear_split with a row of 16
// lanes and 1, 2, 4 channels
enum LinearForm { LINEAR_BY_SHAPE = 0, LINEAR_TILE4 = 1, LINEAR_TILE8 = 2, LINEAR_SPLIT = 3, LINEAR_MFMA = 4, LINEAR_TILE1 = 5, LINEAR_ROW1 = 6,
                  LINEAR_ROW2 = 7, LINEAR_ROW4 = 8 };
inline int linear_form_channels(int f) { return f == LINEAR_TILE1 || f == LINEAR_ROW1 ? 1 : f == LINEAR_ROW2 ? 2 : f == LINEAR_TILE4 || f == LINEAR_ROW4 ? 4 : 8; }
inline int linear_split_lanes(int f) { return f == LINEAR_SPLIT ? 64 : f >= LINEAR_ROW1 ? 16 : 0; }      // 0: not a form of k_linear_split

struct LinearShape {
    int64_t npx, chunks;      // output pixels of the batch; 16-digit chunks of all primes together
    int nch;                  // ... and of the prime with the most
    int out_c, K, in_c;       // output channels, length of the reduction, input channels
    bool mfma;                // dense_mfma_wanted
};

// A grid holds fewer than 2^32 lanes, and k_linear_split has 64 or 16 of them per (output pixel, chunk, block of channels); its unit
// index, as many times smaller, then also stays within its 32-bit products.
inline bool linear_split_fits(int f, const LinearShape& S) {
    const int co = linear_form_channels(f);
    return S.npx * ((S.out_c + co - 1) / co) * S.nch < (1ll << 32) / linear_split_lanes(f);
}

// Times in us, from runs over the shapes of the benchmark's and the paper's networks at batches of 1 to 64.
//   k_linear_split: about 3 + instructions of all its waves / 290 000: 190 per 256 of K, 360 for the addition over the wave
//   k_dense_mfma:   about 6 + 0.6 per round and 64 of K, 8 more per further round of 256 tiles (where its tiles fit the layer at all)
//   k_linear_tile:  0.6 per four of K (a chain of loads) while its waves are one round of the chip; eight channels per lane from 256
//                   waves on (6x6 over 28x28x1 -> 16, 139 waves: 11.4 with four, 14 with eight; 2x2 over 28x28x32 -> 32, 355 waves:
//                   50 and 33; 3x3 over 30x30x32 -> 32, 1420 waves: 226 and 114)
// Up to four channels, where eight per lane are mostly multiplications for nobody:
//   rows of lanes:  as k_linear_split, a quarter of the waves, 62 + 16 per channel instructions per 64 of K and 60 + 45 per channel for
//                   the addition, but not below 5 + 0.6 per 64 of K, the chain of loads (4096 -> 1, batch 1: 43, with a wave 18)
//   k_linear_tile:  0.8 to 20 per four of K as its waves fill the chip; a lane's time is the fetch of the input, so one channel costs what
//                   eight do (3x3 over 128x128x16, 12 primes: 258 with eight channels per lane, 301 with one, whose many waves crowd
//                   each other's lines out) unless neighbouring pixels share a line of 128 bytes, in_c <= 8 (5x5 over 28x28x1, batch 64,
//                   8 primes: to one channel 118 with eight, 69 with four, 52 with one; to two 124, 75 and 102)
// To one, two and four channels, before (eight or four per lane) and now: 3x3 over 28x28x32, 8 primes 61, 62, 64 -> 17, 18, 23; the same
// at batch 4 105, 106, 107 -> 44, 53, 68; 3x3 over 32x32x64, batch 2, 12 primes 201, 202, 203 -> 81, 75, 90; 100 inputs, batch 2048, 8
// primes 44, 45, 47 -> 20, 22, 29; 5x5 over 28x28x1, batch 64, 8 primes 115, 124, 139 -> 52, 75, 86.
inline int linear_form_by_shape(const LinearShape& S) {
    const int64_t blocks8 = (S.out_c + 7) / 8;
    const double split = 3 + (double)S.npx * blocks8 * S.chunks * ((S.K + 255) / 256 * 190 + 360) / 290e3;
    if (S.mfma) {
        const int64_t tiles = (S.npx * S.chunks + 31) / 32 * ((S.out_c + 127) / 128), rounds = (tiles + 255) / 256;
        return split < 6 + 0.6 * rounds * ((S.K + 63) / 64) + 8 * (rounds - 1) ? LINEAR_SPLIT : LINEAR_MFMA;
    }
    if (S.out_c <= 4) {
        const int co = S.out_c == 3 ? 4 : S.out_c, steps = (S.K + 63) / 64;
        const double chain = 5 + 0.6 * steps, issue = 3 + (double)S.npx * S.chunks / 4 * (steps * (62 + 16 * co) + 60 + 45 * co) / 290e3;
        const double row = chain > issue ? chain : issue;
        const double waves = (double)S.npx * S.chunks / 64, group = 0.3 + 0.0008 * waves;
        const double tile = 4 + (S.K + 3) / 4 * (group > 0.8 ? group : 0.8) * (S.out_c == 1 && S.in_c <= 8 ? 0.5 : 1);
        if (row < tile && row < split) return co == 1 ? LINEAR_ROW1 : co == 2 ? LINEAR_ROW2 : LINEAR_ROW4;
        if (split < tile) return LINEAR_SPLIT;
        return S.in_c > 8 && waves >= 256 ? LINEAR_TILE8 : S.out_c == 1 ? LINEAR_TILE1 : LINEAR_TILE4;
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
    return linear_split_lanes(f) && !linear_split_fits(f, S) ? LINEAR_TILE8 : f;
}

}  // namespace dash
