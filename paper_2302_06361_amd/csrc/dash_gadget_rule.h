// dash_gadget_rule.h -- which kernels garble the gates of a sign gadget (host code)
#pragma once
#include <stdint.h>

namespace dash {

// Digit gates of a gadget that is not one of few rows: the AES tables once per bank (blocks of 1024 lanes, 64 KB), or one copy.
// typed: the digit set has compile-time code; uniform: all digits behind the first have one modulus; k: primes of the base.
//
// Bank-replicated tables look up twice as fast, and with them a gadget is faster from the first launch that is not one of few rows on: one repetition
// of 12 000 values, compile-time set of 8 primes, 269 us instead of 344; run-time sets: 10 primes 913 and 956, 6 primes 267 and 287, 12 primes with
// different digits (20 000 values) 546 and 634, 5 primes with equal ones 273 and 284.
// The other way round with different digits of few primes, whose lanes read many output labels (a tile of a small prime has many values) and the offset
// multiples of every digit's modulus, for twice as many waves at a time: (2, 12, 25, 20) of 5 primes, 20 000 values, 564 us and 546; (4, 15, 14) of 4
// primes, 40 000, 620 and 594; (2, 5, 9) of 3 primes, ReLU, 60 000, 675 and 628.
inline bool digits_banked(bool typed, bool uniform, int k) { return typed || uniform || k > 5; }

// A caller's gates on the mod-2 wire (bits: their number; others: of its other gates; rows: of all of them), where they don't share the launch of the
// carry gates: whether they have the kernel for one mod-2 wire.  few: all of them together are few rows and would share launches of up to max_jobs
// gates; else they would have a launch per output modulus.
//
// Of few rows a launch is paid for more than its rows.  So: where it is none more than without it (ReLU, 7 primes, 5 000 values: 156 us, 166 without; 12
// primes, 1 000: 185 and 189; one launch more: 9 primes, 2 000, 163 and 160; 4 primes, 7 000, 153 and 147; 10 primes, 1 000, 214 and 210) or the
// rows are 600 000 and up (2 primes, 60 000: 309 and 334; 9 primes, 7 000: 297 and 302), and for four gates on, which the 64 KB of its tables take
// to pay (scaling, 3 casts, 9 500 values: 190 and 188; 7 casts: 218 and 221).
inline bool bits_own_launch(uint32_t bits, uint32_t others, uint64_t rows, bool few, uint32_t max_jobs) {
    auto launches = [&](uint32_t n) { return (n + max_jobs - 1) / max_jobs; };
    if (!few) return bits > 0;
    return bits >= 4 && (rows >= 600000 || launches(bits) + launches(others) <= launches(bits + others));
}

}  // namespace dash
