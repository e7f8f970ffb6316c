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

}  // namespace dash
