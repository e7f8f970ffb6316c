// dash_proj_rule.h -- how the evaluator launches independent projection gates, as a function of their sizes alone (host code)
#pragma once
#include <stdint.h>

namespace dash {

// The PROJ calls of one layer id that have the same output modulus.
struct ProjRun {
    uint32_t q;            // output modulus
    uint64_t calls, gates;
    bool bits_only;        // every input modulus is 2
    bool alone;            // there are no calls with another output modulus
};

// Whether they have launches of their own (k_proj_eval with this output modulus' compile-time code, up to 16 calls each) or share those of all
// moduli (k_proj_eval_many, 64 calls each).  Sharing saves launches and their ends: 1 000 gates over the 144 pairs of the 12-prime base 66 ->
// 35 us, 4.2 M 315 -> 256.  Where there is one output modulus, or an output modulus has gates enough to fill the chip by itself, that leaves the
// kernels themselves (us, own and shared, one pair of moduli):
//   q = 2: the shared kernel fetches the 128 bytes of a row behind the hash with half the waves per SIMD.  100 000 gates 37 -> 2: 11 and 12; 400 000:
//     23 and 44; 4.2 M: 288 and 402.  2 -> 2: 12 and 13, 28 and 46, 348 and 458.
//     Beside others from 2^18 gates on: a mix of 1.05 M gates, 87 000 or 131 000 of them with q = 2, 86 instead of 81 (12 primes) and 61
//     instead of 58 (8 primes) with a launch of their own, 4.2 M (350 000, 524 000) 239 instead of 243 and 238 instead of 245.
//   q = 3, 5: rows before the hash hide the gather.  4.2 M gates 37 -> 3: 309 and 288, 5 -> 5: 264 and 245; 400 000: 28 and 25, 24 and 23.
//   q >= 7: the hashes count, and own launches have bank-replicated tables from banked_min on.  4.2 M gates 2 -> 37: 180 and 199, 13 -> 17: 175 and 187,
//     37 -> 37: 187 and 196; 2.1 M: 91 and 100, 90 and 94, 95 and 98; 1.05 M: 40 and 46, 40 and 37, 43 and 40 (with rows of two values, one or
//     two lines, earlier than with more); below, the same.
//   One launch either way (20 000 gates and fewer, any moduli): 9.4 to 9.7 and 9.5 to 10.6, the smaller kernel and argument block.
inline bool proj_own_launches(const ProjRun& R, uint64_t banked_min) {
    const uint64_t launches = (R.calls + 15) / 16;
    if (R.alone && launches == 1 && (R.q == 2 || R.gates < 1u << 18)) return true;
    if (R.q == 2) return R.gates >= launches << 18;
    return R.q >= 7 && R.gates / launches / (R.bits_only ? 1 : 2) >= banked_min;
}

}  // namespace dash
