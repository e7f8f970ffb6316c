// dash_core.h -- per-lane arithmetic of the garbling hash: modulus constants, packed-digit
// arithmetic, label compression (Horner, Sec. Implementation), AES-128 on little-endian column
// words with T-tables (FIPS-197; the paper's fixed-key permutation, Sec. Garbled Circuit
// Optimizations) and base-q digit extraction (label decompression, Sec. LabelTensors).
//
// Everything here is a forceinline host+device function with no memory access of its own except
// through the functors it is given, so the same code is exercised by a host self-check.
//
// Every routine is a template over the modulus description: either the runtime ModInfo (any
// modulus 2..255, loops with wave-uniform trip counts) or CMod<m, lam> whose fields are
// compile-time constants, so that the same source unrolls completely and all divisions become
// multiplications by literals.
#pragma once
#include <stdint.h>

#include <type_traits>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define DASH_HD __host__ __device__ __forceinline__
#else
#define DASH_HD inline
#endif

namespace dash {

// Constants of one modulus m (2..255), computed on the host (dash_hostconst.h).
struct ModInfo {
    uint32_t m;       // modulus
    uint32_t lam;     // digits per label
    uint32_t nchunk;  // ceil(lam / 16): 16-digit chunks of a LabelTensor
    uint32_t ndw;     // ceil(lam / 4): dwords of a table row (pitch / 4)
    uint32_t mmagic;  // ceil(2^32 / m): floor(n / m) = mulhi(n, mmagic) for n < 2^24
    uint32_t m4;      // m replicated in 4 bytes
    uint32_t c4;      // (128 - m) replicated (m <= 128), else 0
    uint32_t gc;      // dwords (4 digits each) per 32-bit super-digit of compress: m^(4 gc) < 2^32
    uint32_t Qc;      // m^(4 gc)
    // decompress: m = 2^tw * mo (mo odd).  A super-digit of gd digits is h mod m^gd; dividing by
    // m^gd = 2^(tw gd) * mo^gd is a shift by dsh = tw*gd bits and a long division by Qd = mo^gd <= 2^15.
    uint32_t tw;      // number of factors 2 in m
    uint32_t omagic;  // ceil(2^32 / mo): floor(n / mo) = mulhi(n, omagic) for n < 2^24; 0 when mo = 1
    uint32_t gd;      // digits per super-digit
    uint32_t dsh;     // tw * gd
    uint32_t Qd;      // mo^gd
    uint32_t Qdmagic; // ceil(2^(31+L) / Qd), L = ceil(log2 Qd): floor(n / Qd) = mulhi(n, Qdmagic) >> (L-1), n < 2^31
    uint32_t Qdshift; // L - 1
    uint32_t Qdbits;  // dsh + floor(log2 Qd): every super-digit shortens the dividend by at least this many bits
    const uint32_t* dtab;  // device: [a = 0..m-1][ndw] packed digits of a * R_m mod m
};

// ---- the same constants at compile time ---------------------------------------------------------
namespace cm {
constexpr uint32_t ceil_log2(uint64_t v) { uint32_t l = 0; while ((1ull << l) < v) l++; return l; }
constexpr uint32_t floor_log2(uint64_t v) { uint32_t l = 0; while ((2ull << l) <= v) l++; return l; }
constexpr uint64_t ipow(uint64_t b, uint32_t e) { uint64_t r = 1; for (uint32_t i = 0; i < e; i++) r *= b; return r; }
constexpr uint32_t gc_of(uint32_t m) { uint32_t g = 0; while (g < 8 && ipow(m, 4 * (g + 1)) < (1ull << 32)) g++; return g; }
constexpr uint32_t twos_of(uint32_t m) { uint32_t t = 0; while (!(m & 1)) { m >>= 1; t++; } return t; }
constexpr uint32_t bits_of(uint64_t v) { uint32_t b = 0; while (v) { b++; v >>= 1; } return b; }   // v < 2^bits_of(v)
// largest g with mo^g <= 2^15, the super-digit (mo^g - 1) * 2^(tw g) + ... below 2^32 and, for the digit
// extraction, (m^g >> tw) below 2^24 (powers of two: at most 24 bits per super-digit)
constexpr bool gd_ok(uint32_t m, uint32_t g) {
    const uint32_t tw = twos_of(m);
    const uint64_t mo = m >> tw, qo = ipow(mo, g);
    if (qo > (1ull << 15)) return false;
    if (tw * g + ceil_log2(qo) > 32) return false;
    if (mo == 1 && tw * g > 24) return false;
    return (ipow(m, g) >> tw) < (1ull << 24);
}
constexpr uint32_t gd_of(uint32_t m) { uint32_t g = 1; while (gd_ok(m, g + 1)) g++; return g; }
// label length of modulus m under the ceil rule: smallest lam with m^lam >= 2^128
constexpr uint32_t lam_ceil(uint32_t m) { uint32_t l = 0; for (unsigned __int128 v = ~(unsigned __int128)0; v; v /= m) l++; return l; }
// ... and under the floor rule (largest lam with m^lam <= 2^128)
constexpr uint32_t lam_of(uint32_t m, bool floor_rule) { return lam_ceil(m) - (floor_rule && (m & (m - 1)) != 0 ? 1u : 0u); }

// ---- constants of the base conversion (decompress), see there
struct Big { uint32_t w[10]; };      // 320-bit number
constexpr void big_mul(Big& b, uint32_t m) { uint64_t c = 0; for (int i = 0; i < 10; i++) { c += (uint64_t)b.w[i] * m; b.w[i] = (uint32_t)c; c >>= 32; } }
constexpr bool big_ge(const Big& a, const Big& b) { for (int i = 9; i >= 0; i--) if (a.w[i] != b.w[i]) return a.w[i] > b.w[i]; return true; }
constexpr void big_sub(Big& a, const Big& b) { uint64_t br = 0; for (int i = 0; i < 10; i++) { uint64_t t = (uint64_t)a.w[i] - b.w[i] - br; a.w[i] = (uint32_t)t; br = (t >> 32) & 1; } }
constexpr void big_dbl(Big& a, uint32_t in) { for (int i = 9; i > 0; i--) a.w[i] = (a.w[i] << 1) | (a.w[i - 1] >> 31); a.w[0] = (a.w[0] << 1) | in; }
constexpr Big big_recip(uint32_t s, const Big& D) {      // 2^s / D to the nearest integer
    Big q{}, r{};
    for (uint32_t i = 0; i <= s; i++) {
        big_dbl(r, i == 0 ? 1u : 0u);
        big_dbl(q, 0);
        if (big_ge(r, D)) { big_sub(r, D); q.w[0] |= 1; }
    }
    big_dbl(r, 0);
    if (big_ge(r, D)) for (int i = 0; i < 10; i++) if (++q.w[i]) break;
    return q;
}
constexpr double big_double(const Big& b) { double d = 0; for (int i = 9; i >= 0; i--) d = d * 4294967296.0 + b.w[i]; return d; }
constexpr double pow2(int e) { double d = 1; for (int i = 0; i < e; i++) d *= 2; for (int i = 0; i > e; i--) d *= 0.5; return d; }

struct FracPlan {
    uint32_t ns, top;        // super-digits of gc dwords, dwords of the (shorter) top one
    Big R;                   // 2^256 / D, D = m^(digits below the top super-digit)
    uint32_t c0;             // lowest 32-bit column of h R that is formed
    uint32_t bcol, bword;    // start value: bword in column bcol, about R / 2
    uint32_t w[16];          // words of the fraction before extraction k
    double low, high;        // distance of the worst errors from the ends of the window that gives exact digits
};
constexpr FracPlan frac_plan(uint32_t m) {
    FracPlan P{};
    const uint32_t ndw = (lam_ceil(m) + 3) / 4, gc = gc_of(m);
    P.ns = (ndw + gc - 1) / gc;
    P.top = ndw - (P.ns - 1) * gc;
    Big D{};
    D.w[0] = 1;
    for (uint32_t i = 0; i < (P.ns - 1) * gc * 4; i++) big_mul(D, m);
    P.R = big_recip(256, D);
    const double R = big_double(P.R), Q = (double)ipow(m, 4 * gc);
    Big half = P.R;
    for (int i = 0; i < 9; i++) half.w[i] = (half.w[i] >> 1) | (half.w[i + 1] << 31);
    P.bcol = half.w[4] ? 4 : 3;
    P.bword = half.w[P.bcol];
    const double pos = P.bword * pow2(32 * (int)P.bcol) / R, rounding = 0.5 * pow2(128) / R;      // h times the rounding of R
    double loss = rounding, drop = 0;
    int rw = 0;
    for (int i = 0; i < 10; i++) if (P.R.w[i]) rw = i + 1;
    for (int c = 0; c < 4; c++) {
        double n = 0;
        for (int i = 0; i < 4; i++) if (c - i >= 0 && c - i < rw) n += 1;
        const double d = n * pow2(64 + 32 * c) / R;
        if (drop + d > 0.03) break;
        drop += d;
        P.c0 = (uint32_t)c + 1;
    }
    loss += drop;
    double Dk = big_double(D);
    for (uint32_t k = 0; k + 1 < P.ns; k++) {
        uint32_t w = 1;
        while (Dk * pow2(-32 * (int)w) > 0.05) w++;
        const uint32_t have = k == 0 ? 8 - P.c0 : P.w[k - 1];
        P.w[k] = w < have ? w : have;
        if (w < have) loss += Dk * pow2(-32 * (int)w);
        Dk /= Q;
    }
    P.low = pos - loss;
    P.high = 1.0 - pos - rounding;
    return P;
}
// smallest shift s for which floor(n / D) = mulhi(n, ceil(2^(32 + s) / D)) >> s for all n <= nmax; 32 if there is none
constexpr uint32_t magic_shift(uint64_t nmax, uint64_t D) {
    for (uint32_t s = 0; s < 32; s++) {
        const unsigned __int128 t = (unsigned __int128)1 << (32 + s), M = (t + D - 1) / D;
        if (M >> 32 == 0 && nmax * (M * D - t) < t) return s;
    }
    return 32;
}
constexpr uint32_t magic_mul(uint32_t s, uint64_t D) { return (uint32_t)((((unsigned __int128)1 << (32 + s)) + D - 1) / D); }
// smallest shift s for which floor(x / m) = (x * ceil(2^s / m)) >> s for all x < m^2
constexpr uint32_t small_shift(uint32_t m) {
    for (uint32_t s = 1; s < 24; s++) if ((uint64_t)(m * m - 1) * ((((1ull << s) + m - 1) / m) * m - (1ull << s)) < (1ull << s)) return s;
    return 24;
}
}  // namespace cm

template <uint32_t MOD, uint32_t LAM>
struct CMod {
    static constexpr uint32_t m = MOD, lam = LAM, nchunk = (LAM + 15) / 16, ndw = (LAM + 3) / 4;
    static constexpr uint32_t mmagic = (uint32_t)(((1ull << 32) + MOD - 1) / MOD);
    static constexpr uint32_t m4 = MOD * 0x01010101u, c4 = MOD <= 128 ? (128 - MOD) * 0x01010101u : 0;
    static constexpr uint32_t gc = cm::gc_of(MOD), Qc = (uint32_t)cm::ipow(MOD, 4 * gc);
    const uint32_t* dtab;
};

// the modulus of a compile-time description, 0 for the run-time one
template <class T> struct cmod_m { static constexpr uint32_t value = 0; };
template <uint32_t MOD, uint32_t LAM> struct cmod_m<CMod<MOD, LAM>> { static constexpr uint32_t value = MOD; };
// dwords per label of a compile-time description, 1 for the run-time one (array sizes)
template <class T> struct cmod_ndw { static constexpr uint32_t value = 1; };
template <uint32_t MOD, uint32_t LAM> struct cmod_ndw<CMod<MOD, LAM>> { static constexpr uint32_t value = (LAM + 3) / 4; };

struct U128 { uint32_t w[4]; };

DASH_HD uint32_t mulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
// 24-bit multiply (both operands below 2^24, product below 2^32).
// Measured issue cost of a wave64 instruction on this chip, in cycles per SIMD: and / or / xor / add / sub / shift right /
// three-input bit operation 2; shift left, byte permute, sub-dword selects, three-operand integer forms, 24-bit and 32-bit
// multiplies (low and high half alike), 64-bit multiply-add, byte dot product 4.
DASH_HD uint32_t mul24(uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __umul24(a, b);
#else
    return a * b;
#endif
}
// sum of byte products a.b0*b.b0 + .. + a.b3*b.b3
DASH_HD uint32_t dot4(uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__) && __has_builtin(__builtin_amdgcn_udot4)
    return __builtin_amdgcn_udot4(a, b, 0u, false);
#else
    uint32_t s = 0;
    for (int i = 0; i < 4; i++) s += ((a >> (8 * i)) & 0xff) * ((b >> (8 * i)) & 0xff);
    return s;
#endif
}
// load through a pointer that is known to address device global memory (pointers that were themselves
// loaded from memory would otherwise be dereferenced with flat instructions, which also occupy the LDS queue)
DASH_HD uint32_t gload32(const uint32_t* p) {
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const __attribute__((address_space(1))) uint32_t*)p;
#else
    return *p;
#endif
}
// record of a modulus: the table of moduli is never written while a kernel runs, so a wave-uniform index is a scalar load
DASH_HD ModInfo ld_mod(const ModInfo* mods, uint32_t m) {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(sizeof(ModInfo) % 8 == 0, "copied in 8-byte words");
    const auto* src = (const __attribute__((address_space(4))) uint64_t*)(mods + m);
    union { uint64_t w[sizeof(ModInfo) / 8]; ModInfo M; } u;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(ModInfo) / 8); i++) u.w[i] = src[i];
    return u.M;
#else
    return mods[m];
#endif
}
template <class MI> DASH_HD uint32_t div_m(uint32_t n, const MI& M) { return mulhi(n, M.mmagic); }           // n < 2^24
template <class MI> DASH_HD uint32_t mod_m(uint32_t n, const MI& M) { return n - mul24(div_m(n, M), M.m); }  // n < 2^24
// floor(n / m) for n <= 2^32 - m (wave-uniform n: scalar unit): the rounded-up reciprocal is too large by at most one, and q m must not
// pass 2^32 (callers: the first row of a tile, a multiple of 256 below 2^32)
template <class MI> DASH_HD uint32_t div_any(uint32_t n, const MI& M) { const uint32_t q = mulhi(n, M.mmagic); return q - (q * M.m > n ? 1u : 0u); }
DASH_HD uint32_t byte_of(uint32_t w, int b) { return (w >> (8 * b)) & 0xffu; }

// Packed modular addition and subtraction on 4 digits, for kernels that are bound by the number of vector instructions: four for
// a sum, five for a difference.  Moduli below 128: the bytes of u = a + b + (128 - m) reach 128 where a + b >= m, and then u - 128 is
// the result; where they do not, it is u - 128 + m.  The flags stay where they are (bit 7 of each byte): the high half of
// flags * (m << 25) is m in each flagged byte.  Every byte of the result lies in [0, m), so the carries and borrows between the bytes of
// the intermediate dwords cancel.  (Bringing the flags down to bit 0 and multiplying by m took five and seven.)
constexpr uint32_t kOnes = 0x01010101u, kTops = 0x80808080u;
// ~a & b (one v_bitop3_b32 on gfx950, kept from being folded into the additions around it)
DASH_HD uint32_t andn(uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__) && __has_builtin(__builtin_amdgcn_bitop3_b32)
    return __builtin_amdgcn_bitop3_b32(a, b, b, 0x0c);
#else
    return ~a & b;
#endif
}
// u - 128 in every byte, + m where the byte is below 128 (m < 128).  (u is kept as it is: the compiler would take the constants of its
// sum and of this one together, which costs an instruction more.)
DASH_HD uint32_t settle4(uint32_t u, uint32_t m) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+v"(u));
#endif
    return u + mulhi(andn(u, kTops), m << 25) - kTops;
}
// per byte (a + b + (r & 1)) >> 1, without carries between bytes
DASH_HD uint32_t lerp4(uint32_t a, uint32_t b, uint32_t r) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_lerp(a, b, r);
#else
    uint32_t w = 0;
    for (int i = 0; i < 32; i += 8) w |= ((((a >> i) & 0xffu) + ((b >> i) & 0xffu) + ((r >> i) & 1u)) >> 1) << i;
    return w;
#endif
}
// (a + b) mod m on 4 packed digits, a, b < m per byte.
template <class MI>
DASH_HD uint32_t addmod4(uint32_t a, uint32_t b, const MI& M) {
    if constexpr (cmod_m<MI>::value == 2) return a ^ b;          // digits are bits (one per byte)
    if (M.m < 128) return settle4(a + b + M.c4, M.m);
    const uint32_t t = a + b;
    // moduli from 128 up: the sum need not fit a byte, its half does.  a + b >= m iff (a + b + (m odd)) / 2 >= ceil(m / 2).
    const uint32_t h = lerp4(a, b, (M.m & 1u) * kOnes) + (128u - (M.m + 1u) / 2u) * kOnes;
    return t - ((h >> 7) & kOnes) * M.m;
}
// the same with b prepared once for several sums: offset4(b) = b + (128 - m) where that fits a byte
template <class MI> DASH_HD uint32_t offset4(uint32_t b, const MI& M) { return cmod_m<MI>::value != 2 && M.m < 128 ? b + M.c4 : b; }
template <class MI>
DASH_HD uint32_t addmod4_off(uint32_t a, uint32_t b_off, const MI& M) {
    return cmod_m<MI>::value != 2 && M.m < 128 ? settle4(a + b_off, M.m) : addmod4(a, b_off, M);
}
// (a - b) mod m on 4 packed digits.
template <class MI>
DASH_HD uint32_t submod4(uint32_t a, uint32_t b, const MI& M) {
    if constexpr (cmod_m<MI>::value == 2) return a ^ b;
    // (Run-time descriptions take the form for all moduli, without a branch per dword: their callers are the evaluator's chains of hashes.  13 primes,
    // 100 values, six repetitions: 912 us with the branch, 855 without.)
    if (cmod_m<MI>::value != 0 && M.m < 128) return settle4((a ^ kTops) - b, M.m);      // a - b + 128: no borrow between bytes
    const uint32_t t = a - b;
    return t + andn(lerp4(a, ~b, kOnes) >> 7, kOnes) * M.m;                        // top bit of a byte: a >= b
}
// (a + c * b) mod m on 4 packed digits, c < m.
template <class MI>
DASH_HD uint32_t axpymod4(uint32_t a, uint32_t c, uint32_t b, const MI& M) {
    if constexpr (cmod_m<MI>::value == 2) return a ^ (b & (0u - (c & 1u)));
    uint32_t r = 0;
    for (int b8 = 0; b8 < 4; b8++) r |= mod_m(byte_of(a, b8) + mul24(c, byte_of(b, b8)), M) << (8 * b8);
    return r;
}

// acc = acc * mul + add  (mod 2^128)
DASH_HD void muladd128(U128& a, uint32_t mul, uint32_t add) {
    uint64_t t = (uint64_t)a.w[0] * mul + add;
    a.w[0] = (uint32_t)t; t >>= 32;
    t += (uint64_t)a.w[1] * mul; a.w[1] = (uint32_t)t; t >>= 32;
    t += (uint64_t)a.w[2] * mul; a.w[2] = (uint32_t)t; t >>= 32;
    t += (uint64_t)a.w[3] * mul; a.w[3] = (uint32_t)t;
}

// acc = acc * mul + add (mod 2^128) for an accumulator known to fit W words: W multiplications
template <int W>
DASH_HD void muladd128_w(U128& a, uint32_t mul, uint32_t add) {
    uint64_t t = add;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (i < W) { t += (uint64_t)a.w[i] * mul; a.w[i] = (uint32_t)t; t >>= 32; }
        else if (i == W) a.w[i] = (uint32_t)t;
    }
}
// compile-time descriptions: super-digit T (counted from the top) and all below it.  Before it is folded in, the
// accumulator is below Qc^T, so only the words that can be non-zero are multiplied.
template <class MI, int T, class LoadDw>
DASH_HD void compress_from(U128& acc, LoadDw& dw, uint32_t& w0) {
    constexpr int NS = ((int)MI::ndw + (int)MI::gc - 1) / (int)MI::gc;
    if constexpr (T < NS) {
        constexpr int top = (int)MI::ndw - (NS - 1) * (int)MI::gc;        // dwords of the top super-digit (may be short)
        constexpr int cnt = T == 0 ? top : (int)MI::gc;
        constexpr int hi = T == 0 ? (int)MI::ndw - 1 : (int)MI::ndw - 1 - top - (T - 1) * (int)MI::gc;
        constexpr uint32_t wlo = 1u | (MI::m << 8), whi = (1u << 16) | (MI::m << 24), m2 = MI::m * MI::m, m4 = m2 * m2;
        uint32_t S = 0;
#pragma unroll
        for (int c = 0; c < cnt; c++) {
            const uint32_t w = dw(hi - c);
            if (hi - c == 0) w0 = w;
            const uint32_t v = dot4(w, wlo) + mul24(m2, dot4(w, whi));     // < m^4; both factors below 2^17
            S = c == 0 ? v : (MI::Qc < (1u << 24) ? mul24(S, m4) : S * m4) + v;
        }
        constexpr int wbits = T * (int)cm::bits_of((uint64_t)MI::Qc - 1);
        constexpr int W = T == 0 ? 0 : (wbits + 31) / 32 > 4 ? 4 : (wbits + 31) / 32;
        muladd128_w<W>(acc, MI::Qc, S);
        compress_from<MI, T + 1>(acc, dw, w0);
    }
}

// compress(l) = sum_j l[j] m^j mod 2^128 (Horner from the top digit).  dw(i) returns packed digits
// 4i..4i+3 of the label, digits past lam zero.  *colour receives digit 0.
// Four digits at a time: v = d0 + m d1 + m^2 d2 + m^3 d3 by two byte dot products; gc such values
// make one 32-bit super-digit; the 128-bit accumulator is multiplied once per super-digit.  The top
// dword may hold fewer than 4 digits: its missing digits are zero, which Horner ignores.
template <class MI, class LoadDw>
DASH_HD U128 compress(const MI& M, LoadDw dw, uint32_t* colour) {
    U128 acc = {{0, 0, 0, 0}};
    if constexpr (cmod_m<MI>::value == 2) {   // digits are bits: pack them (compile-time description only:
                                                        // with run-time trip counts the word index would be dynamic)
        uint32_t w0 = 0;
#pragma unroll
        for (int i = (int)M.ndw - 1; i >= 0; i--) {
            uint32_t w = dw(i);
            if (i == 0) w0 = w;
            acc.w[i >> 3] |= dot4(w, 0x08040201u) << (4 * (i & 7));
        }
        *colour = w0 & 0xffu;
        return acc;
    }
    if constexpr (cmod_m<MI>::value > 2) {
        uint32_t w0 = 0;
        compress_from<MI, 0>(acc, dw, w0);
        *colour = w0 & 0xffu;
        return acc;
    }
    const uint32_t wlo = 1u | (M.m << 8), whi = (1u << 16) | (M.m << 24), m2 = M.m * M.m, m4 = m2 * m2;
    uint32_t S = 0, w0 = 0;
    uint32_t left = M.ndw % M.gc;        // dwords still to take into the current super-digit;
    if (left == 0) left = M.gc;          // the first (top) group may be short: acc is still 0
#pragma unroll
    for (int i = (int)M.ndw - 1; i >= 0; i--) {
        uint32_t w = dw(i);
        if (i == 0) w0 = w;
        uint32_t v = dot4(w, wlo) + mul24(m2, dot4(w, whi));     // < m^4; both factors below 2^17
        S = (M.Qc < (1u << 24) ? mul24(S, m4) : S * m4) + v;     // S < Qc / m^4
        if (--left == 0) { muladd128(acc, M.Qc, S); S = 0; left = M.gc; }
    }
    *colour = w0 & 0xffu;
    return acc;
}

// ---------------------------------------------------------------------------------------------
// AES-128 encryption.  The state is four little-endian column words: word c holds bytes
// in[4c..4c+3], which are exactly the four 32-bit limbs of the 128-bit block read as a little-endian
// integer.  T[r][x] = column r of MixColumns times S[x]; T[r] = T[0] rotated left by 8r bits.
// rk: 44 round-key words in the same byte order.
// ---------------------------------------------------------------------------------------------
// three-input exclusive or (one v_bitop3_b32 on gfx950)
DASH_HD uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__) && __has_builtin(__builtin_amdgcn_bitop3_b32)
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
    return a ^ b ^ c;
#endif
}

// Tab: the T-tables.  T.template at<R, B>(w) is entry (byte B of w) of table R; the accessor gets the whole
// word so that a table layout can build its address from the byte in place.  A layout with
// Tab::two_tables holds T0 and T1 only: T2 = rot16(T0), T3 = rot16(T1), and one rotation serves both.
template <class Tab, class = void> struct tab_two : std::false_type {};
template <class Tab> struct tab_two<Tab, std::enable_if_t<Tab::two_tables>> : std::true_type {};
DASH_HD uint32_t rot16(uint32_t v) { return (v << 16) | (v >> 16); }

// (Tab::rotated_keys: the caller hands over the keys of rounds 1..9 rotated by 16 bits already, see rotate_round_keys.)
template <class Tab, class = void> struct tab_rot : std::false_type {};
template <class Tab> struct tab_rot<Tab, std::enable_if_t<Tab::rotated_keys>> : std::true_type {};
DASH_HD void rotate_round_keys(uint32_t rk[44]) { for (int i = 4; i < 40; i++) rk[i] = rot16(rk[i]); }

// one column of a round: bytes 0..3 of a0..a3 through T0..T3, and the round key.  With two tables the key goes in before the
// rotation that T2 and T3 need, so that every step is a three-input exclusive-or: 7 instructions a column with the four addresses
// instead of 8.
template <class Tab>
DASH_HD uint32_t aes_column(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t rk, const Tab& T) {
    if constexpr (tab_two<Tab>::value) {
        const uint32_t k = tab_rot<Tab>::value ? rk : rot16(rk);
        return xor3(T.template at<0, 0>(a0), T.template at<1, 1>(a1), rot16(xor3(T.template at<0, 2>(a2), T.template at<1, 3>(a3), k)));
    } else {
        return xor3(xor3(T.template at<0, 0>(a0), T.template at<1, 1>(a1), T.template at<2, 2>(a2)), T.template at<3, 3>(a3), rk);
    }
}
// bytes of two words by a selector: 0..3 bytes of lo, 4..7 bytes of hi, 0x0c zero (one v_perm_b32)
DASH_HD uint32_t pick_bytes(uint32_t hi, uint32_t lo, uint32_t sel) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_perm(hi, lo, sel);
#else
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    uint32_t w = 0;
    for (int i = 0; i < 4; i++) { const uint32_t b = (sel >> (8 * i)) & 0xffu; if (b < 8) w |= (uint32_t)((v >> (8 * b)) & 0xffu) << (8 * i); }
    return w;
#endif
}
// a column of the last round (SubBytes and ShiftRows only): S[x] sits in bytes 1 and 2 of T0.  Two byte permutes and an exclusive-or
// instead of four maskings and an exclusive-or
template <class Tab>
DASH_HD uint32_t last_column(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t rk, const Tab& T) {
    return xor3(pick_bytes(T.template at<0, 1>(a1), T.template at<0, 0>(a0), 0x0c0c0501u), pick_bytes(T.template at<0, 3>(a3), T.template at<0, 2>(a2), 0x06020c0cu), rk);
}
// rounds R0..10 on the state a
template <int R0, class Tab>
DASH_HD void aes_rounds(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t s[4], const uint32_t* rk, const Tab& T) {
#pragma unroll
    for (int r = R0; r < 10; r++) {
        const uint32_t b0 = aes_column(a0, a1, a2, a3, rk[4 * r + 0], T), b1 = aes_column(a1, a2, a3, a0, rk[4 * r + 1], T);
        const uint32_t b2 = aes_column(a2, a3, a0, a1, rk[4 * r + 2], T), b3 = aes_column(a3, a0, a1, a2, rk[4 * r + 3], T);
        a0 = b0; a1 = b1; a2 = b2; a3 = b3;
    }
    s[0] = last_column(a0, a1, a2, a3, rk[40], T); s[1] = last_column(a1, a2, a3, a0, rk[41], T);
    s[2] = last_column(a2, a3, a0, a1, rk[42], T); s[3] = last_column(a3, a0, a1, a2, rk[43], T);
}
template <class Tab>
DASH_HD void aes128_encrypt(uint32_t s[4], const uint32_t* rk, const Tab& T) {
    aes_rounds<1>(s[0] ^ rk[0], s[1] ^ rk[1], s[2] ^ rk[2], s[3] ^ rk[3], s, rk, T);
}

// AES-128 by the FOUR lanes of a quad (lanes 4i .. 4i + 3 of a wave) together: all four call with the same s, all four
// return with the same result.  Lane c keeps column c of the state; a round takes the neighbours' columns with three
// quad permutes and does 4 look-ups instead of 16: a third of the instructions per lane, for kernels whose run time is
// the chain of one lane (few elements).  The four lanes must be active together.  (Host build: each caller encrypts
// on its own.)
// Q: the lane's words of the key schedule, k[r] = rk[4 r + c] (rotated keys for tables that want them).  (Picking them per round with selects from the whole schedule
// was turned into branches around scalar loads: 2.0 instead of 1.1 us per gate of a carry chain.)
struct QuadKey { uint32_t k[11]; };
DASH_HD QuadKey quad_key(const uint32_t* rk, uint32_t c) {
    QuadKey Q;
#pragma unroll
    for (int r = 0; r < 11; r++) Q.k[r] = rk[4 * r + c];
    return Q;
}
// Columns: the columns go to the neighbours, before the look-ups; else the entries, after them.
template <bool Columns = false, class Tab>
DASH_HD void aes128_encrypt_quad(uint32_t s[4], const QuadKey& Q, const uint32_t* rk, const Tab& T) {
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t c = __lane_id() & 3u;
    // value of the lane 1, 2, 3 places up in the quad (cyclic), and of lane i of the quad
    auto up1 = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x39, 0xf, 0xf, true); };    // quad_perm:[1,2,3,0]
    auto up2 = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true); };    // quad_perm:[2,3,0,1]
    auto up3 = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x93, 0xf, 0xf, true); };    // quad_perm:[3,0,1,2]
    const uint32_t s01 = c & 1u ? s[1] : s[0], s23 = c & 1u ? s[3] : s[2];
    uint32_t a = (c & 2u ? s23 : s01) ^ Q.k[0];
#pragma unroll
    for (int r = 1; r < 10; r++) {
        // A lane looks up the bytes of its own column, and the entries, not the columns, go to their neighbours: as the operand of the
        // exclusive-or that takes them (keep: or the compiler makes three-input operations of them, which have no such operand).  With the columns
        // exchanged before the look-ups every round had three moves and their wait states more (one launch per layer, scaling, 1 000 values: 7 primes
        // 21.2 us instead of 20.5, 12 primes 37.7 and 35.2).  In the kernel of a carry chain alone the columns are the faster way: signs of 1 000 values,
        // 8 primes, 26.5 us instead of 27.0, 9 primes 29.9 and 30.7.
        auto keep = [](uint32_t v) { asm("" : "+v"(v)); return v; };
        if constexpr (Columns) {
            const uint32_t a1 = up1(a), a2 = up2(a), a3 = up3(a);
            a = aes_column(a, a1, a2, a3, Q.k[r], T);
        } else if constexpr (tab_two<Tab>::value) {
            const uint32_t k = tab_rot<Tab>::value ? Q.k[r] : rot16(Q.k[r]);
            const uint32_t t0 = T.template at<0, 0>(a), t1 = T.template at<1, 1>(a), t2 = T.template at<0, 2>(a), t3 = T.template at<1, 3>(a);
            uint32_t w = keep(up2(t2) ^ k);
            w = keep(up3(t3) ^ w);
            const uint32_t v = keep(up1(t1) ^ t0);
            a = v ^ rot16(w);
        } else {
            const uint32_t t0 = T.template at<0, 0>(a), t1 = T.template at<1, 1>(a), t2 = T.template at<2, 2>(a), t3 = T.template at<3, 3>(a);
            a = keep(t0 ^ Q.k[r]);
            a = keep(up1(t1) ^ a);
            a = keep(up2(t2) ^ a);
            a = up3(t3) ^ a;
        }
    }
    {
        const uint32_t a1 = up1(a), a2 = up2(a), a3 = up3(a);
        a = last_column(a, a1, a2, a3, Q.k[10], T);
    }
    s[0] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0x00, 0xf, 0xf, true);      // quad_perm:[0,0,0,0]
    s[1] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0x55, 0xf, 0xf, true);
    s[2] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0xAA, 0xf, 0xf, true);
    s[3] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0xFF, 0xf, 0xf, true);
#else
    aes128_encrypt(s, rk, T);
#endif
}

// value that lane I (0..3) of the caller's quad holds (all four lanes active)
template <int I> DASH_HD uint32_t quad_lane(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, I * 0x55, 0xf, 0xf, true);      // quad_perm:[I,I,I,I]
#else
    return v;
#endif
}

// h = AES(X) xor X with X = K xor tweak; tweak = elem:u64 | slot:u32 | layer:u16 | 0:u16.
template <class Tab>
DASH_HD U128 hash_block(const U128& K, uint64_t elem, uint32_t slot, uint32_t layer, const uint32_t* rk, const Tab& T) {
    uint32_t x[4] = {K.w[0] ^ (uint32_t)elem, K.w[1] ^ (uint32_t)(elem >> 32), K.w[2] ^ slot, K.w[3] ^ (layer & 0xffffu)};
    uint32_t s[4] = {x[0], x[1], x[2], x[3]};
    aes128_encrypt(s, rk, T);
    U128 h = {{s[0] ^ x[0], s[1] ^ x[1], s[2] ^ x[2], s[3] ^ x[3]}};
    return h;
}
// Several hashes of ONE label whose slots differ in the low byte only (the digit gates of a residue): that byte is one byte of
// the state, it reaches one column in round 1 and one byte of every column in round 2.  Everything else of the two rounds is done
// once: each further hash looks up 5 entries in them instead of 32.
struct SlotHash { uint32_t x[4], b2, c[4]; };      // hash input; column 2 after round 1 and the columns after round 2, without what the slot's low byte contributes
// (from the hash input, its slot's low byte zero)
template <class Tab>
DASH_HD SlotHash slot_hash_start(const uint32_t x[4], const uint32_t* rk, const Tab& T) {
    SlotHash S;
    S.x[0] = x[0]; S.x[1] = x[1]; S.x[2] = x[2]; S.x[3] = x[3];
    const uint32_t a0 = S.x[0] ^ rk[0], a1 = S.x[1] ^ rk[1], a2 = S.x[2] ^ rk[2], a3 = S.x[3] ^ rk[3];
    const uint32_t b0 = aes_column(a0, a1, a2, a3, rk[4], T), b1 = aes_column(a1, a2, a3, a0, rk[5], T), b3 = aes_column(a3, a0, a1, a2, rk[7], T);
    if constexpr (tab_two<Tab>::value) {
        auto key = [&](int i) { return tab_rot<Tab>::value ? rk[i] : rot16(rk[i]); };
        auto T0 = [&](auto B, uint32_t w) { return T.template at<0, decltype(B)::value>(w); };
        auto T1 = [&](auto B, uint32_t w) { return T.template at<1, decltype(B)::value>(w); };
        typedef std::integral_constant<int, 0> B0; typedef std::integral_constant<int, 1> B1; typedef std::integral_constant<int, 2> B2; typedef std::integral_constant<int, 3> B3;
        S.b2 = T1(B1{}, a3) ^ rot16(xor3(T0(B2{}, a0), T1(B3{}, a1), key(6)));
        S.c[0] = xor3(T0(B0{}, b0), T1(B1{}, b1), rot16(T1(B3{}, b3) ^ key(8)));
        S.c[1] = T0(B0{}, b1) ^ rot16(xor3(T0(B2{}, b3), T1(B3{}, b0), key(9)));
        S.c[2] = T1(B1{}, b3) ^ rot16(xor3(T0(B2{}, b0), T1(B3{}, b1), key(10)));
        S.c[3] = xor3(T0(B0{}, b3), T1(B1{}, b0), rot16(T0(B2{}, b1) ^ key(11)));
    } else {
        S.b2 = xor3(T.template at<1, 1>(a3), T.template at<2, 2>(a0), T.template at<3, 3>(a1)) ^ rk[6];
        S.c[0] = xor3(T.template at<0, 0>(b0), T.template at<1, 1>(b1), T.template at<3, 3>(b3)) ^ rk[8];
        S.c[1] = xor3(T.template at<0, 0>(b1), T.template at<2, 2>(b3), T.template at<3, 3>(b0)) ^ rk[9];
        S.c[2] = xor3(T.template at<1, 1>(b3), T.template at<2, 2>(b0), T.template at<3, 3>(b1)) ^ rk[10];
        S.c[3] = xor3(T.template at<0, 0>(b3), T.template at<1, 1>(b0), T.template at<2, 2>(b1)) ^ rk[11];
    }
    return S;
}
template <class Tab>
DASH_HD SlotHash slot_hash_start(const U128& K, uint64_t elem, uint32_t slot, uint32_t layer, const uint32_t* rk, const Tab& T) {
    const uint32_t x[4] = {K.w[0] ^ (uint32_t)elem, K.w[1] ^ (uint32_t)(elem >> 32), K.w[2] ^ (slot & ~0xffu), K.w[3] ^ (layer & 0xffffu)};
    return slot_hash_start(x, rk, T);
}
// the hash for a slot with the same upper 24 bits
template <class Tab>
DASH_HD U128 slot_hash(const SlotHash& S, uint32_t slot, const uint32_t* rk, const Tab& T) {
    const uint32_t x2 = S.x[2] ^ (slot & 0xffu);
    const uint32_t b2 = S.b2 ^ T.template at<0, 0>(x2 ^ rk[2]);
    uint32_t s[4];
    if constexpr (tab_two<Tab>::value)
        aes_rounds<3>(S.c[0] ^ rot16(T.template at<0, 2>(b2)), S.c[1] ^ T.template at<1, 1>(b2), S.c[2] ^ T.template at<0, 0>(b2),
                      S.c[3] ^ rot16(T.template at<1, 3>(b2)), s, rk, T);
    else
        aes_rounds<3>(S.c[0] ^ T.template at<2, 2>(b2), S.c[1] ^ T.template at<1, 1>(b2), S.c[2] ^ T.template at<0, 0>(b2), S.c[3] ^ T.template at<3, 3>(b2),
                      s, rk, T);
    U128 h = {{s[0] ^ S.x[0], s[1] ^ S.x[1], s[2] ^ x2, s[3] ^ S.x[3]}};
    return h;
}
// the same by the four lanes of a quad together (aes128_encrypt_quad): same arguments and same result in all four
template <bool Columns = false, class Tab>
DASH_HD U128 hash_block_quad(const U128& K, uint64_t elem, uint32_t slot, uint32_t layer, const QuadKey& Q, const uint32_t* rk, const Tab& T) {
    uint32_t x[4] = {K.w[0] ^ (uint32_t)elem, K.w[1] ^ (uint32_t)(elem >> 32), K.w[2] ^ slot, K.w[3] ^ (layer & 0xffffu)};
    uint32_t s[4] = {x[0], x[1], x[2], x[3]};
    aes128_encrypt_quad<Columns>(s, Q, rk, T);
    U128 h = {{s[0] ^ x[0], s[1] ^ x[1], s[2] ^ x[2], s[3] ^ x[3]}};
    return h;
}
// PRG block: AES_seed(elem:u64 | slot:u32 | layer:u16 | domain:u8 | m:u8), no feed-forward.
template <class Tab>
DASH_HD U128 prg_block(uint64_t elem, uint32_t slot, uint32_t layer, uint32_t domain, uint32_t m, const uint32_t* rk, const Tab& T) {
    uint32_t s[4] = {(uint32_t)elem, (uint32_t)(elem >> 32), slot, (layer & 0xffffu) | (domain << 16) | (m << 24)};
    aes128_encrypt(s, rk, T);
    U128 h = {{s[0], s[1], s[2], s[3]}};
    return h;
}

// ---------------------------------------------------------------------------------------------
// decompress: digits floor(h / m^j) mod m, j = 0..lam-1, delivered as packed dwords emit(i, w)
// for i = 0..ndw-1 (in any order).  Run-time description: with m = 2^tw * mo, a super-digit of gd digits is taken off the 128-bit number by
// a shift (its low dsh bits) and a long division by Qd = mo^gd <= 2^15 over 16-bit half-words (every
// partial dividend r * 2^16 + half is below 2^31, where the magic division is exact):
//     h mod m^gd = ((h >> dsh) mod Qd) << dsh | (h & (2^dsh - 1)),   h div m^gd = (h >> dsh) div Qd.
// After each super-digit the number is shorter by Qdbits bits; half-words known to be zero are skipped.
// ---------------------------------------------------------------------------------------------
template <class MI>
DASH_HD uint32_t take_superdigit(U128& x, const MI& M, uint32_t bits) {
    uint32_t low = 0;
    if (M.dsh) {
        low = x.w[0] & ((1u << M.dsh) - 1u);
#pragma unroll
        for (int i = 0; i < 3; i++) x.w[i] = (x.w[i] >> M.dsh) | (x.w[i + 1] << (32 - M.dsh));
        x.w[3] >>= M.dsh;
        bits = bits > M.dsh ? bits - M.dsh : 0;
    }
    if (M.Qd == 1) return low;                       // power of two: nothing left to divide
    const uint32_t nh = (bits + 15) / 16;            // significant half-words
    uint32_t r = 0;
#pragma unroll
    for (int i = 3; i >= 0; i--) {
        if ((uint32_t)(2 * i) >= nh) continue;
        uint32_t w = x.w[i], q1 = 0;
        if ((uint32_t)(2 * i + 1) < nh) {
            uint32_t cur = (r << 16) | (w >> 16);
            q1 = mulhi(cur, M.Qdmagic) >> M.Qdshift;
            r = cur - mul24(q1, M.Qd);
        }
        uint32_t cur = (r << 16) | (w & 0xffffu);
        uint32_t q0 = mulhi(cur, M.Qdmagic) >> M.Qdshift;
        r = cur - mul24(q0, M.Qd);
        x.w[i] = (q1 << 16) | q0;
    }
    return (r << M.dsh) | low;
}

// Compile-time descriptions.  The number is turned into a fraction once and the super-digits (gc dwords of 4 digits each, below
// 2^32) come off its TOP end:  with D = m^(digits below the top super-digit) and R = 2^256 / D,  h R / 2^256 = h / D  has the top
// super-digit as its integer part; multiplying the fraction by Q = m^(4 gc) gives the next one, and so on, on ever fewer words.
// Exactness: any fraction in [x / D, (x + 1) / D) gives the digits of x.  The product starts at about R / 2, the middle of that
// window, and what the rounding of R, the columns that are never formed and the words that are dropped can move it by is added
// up at compile time (FracPlan) and must stay below half the window.
// Against the long division over 16-bit half-words that the run-time description below uses, this is a 32 x 32 -> 64-bit
// multiply-add per word instead of two steps of five instructions, with super-digits up to 2^32 instead of 2^15 times a power of
// two: 83 vector instructions instead of 197 for m = 96 (20 digits), 104 instead of 283 for m = 204, 122 instead of 333 for m = 37.
template <uint32_t MOD> struct Frac { static constexpr cm::FracPlan P = cm::frac_plan(MOD); };

// acc += a * b, b the same in all lanes (see mad64_carries)
DASH_HD void mad64(uint64_t& acc, uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_mad_u64_u32 %0, vcc, %1, %2, %0" : "+v"(acc) : "v"(a), "s"(b) : "vcc");
#else
    acc += (uint64_t)a * b;
#endif
}
// acc += a[0] b[0] + .. + a[N-1] b[N-1]; the number of times that the 64-bit sum overflows.  (As assembly because the compiler forms a carry
// by a comparison and takes sums of products apart: 6 vector instructions more for the conversion of m = 96, 10 for m = 13, 14 for m = 22.)
// Two wait states must pass between a vector instruction that writes a carry and one that reads it, and nothing watches over that inside
// an assembly block: the carries are added up behind the products, and where these are fewer than three, s_nop fills the rest.
template <int N>
DASH_HD uint32_t mad64_carries(uint64_t& acc, const uint32_t* a, const uint32_t* b) {
    static_assert(N >= 1 && N <= 3, "no modulus has a column with more");
    uint32_t over = 0;
#if defined(__HIP_DEVICE_COMPILE__)
    uint64_t c0, c1;
    if constexpr (N == 1)
        asm("v_mad_u64_u32 %0, vcc, %2, %3, %0\n\ts_nop 1\n\tv_addc_co_u32_e64 %1, vcc, 0, 0, vcc"
            : "+v"(acc), "=v"(over) : "v"(a[0]), "s"(b[0]) : "vcc");
    else if constexpr (N == 2)
        asm("v_mad_u64_u32 %0, %2, %3, %5, %0\n\tv_mad_u64_u32 %0, vcc, %4, %6, %0\n\ts_nop 0\n\t"
            "v_addc_co_u32_e64 %1, %2, 0, 0, %2\n\tv_addc_co_u32_e32 %1, vcc, 0, %1, vcc"
            : "+v"(acc), "=v"(over), "=&s"(c0) : "v"(a[0]), "v"(a[1]), "s"(b[0]), "s"(b[1]) : "vcc");
    else
        asm("v_mad_u64_u32 %0, %2, %4, %7, %0\n\tv_mad_u64_u32 %0, %3, %5, %8, %0\n\tv_mad_u64_u32 %0, vcc, %6, %9, %0\n\t"
            "v_addc_co_u32_e64 %1, %2, 0, 0, %2\n\tv_addc_co_u32_e64 %1, %3, 0, %1, %3\n\tv_addc_co_u32_e32 %1, vcc, 0, %1, vcc"
            : "+v"(acc), "=v"(over), "=&s"(c0), "=&s"(c1) : "v"(a[0]), "v"(a[1]), "v"(a[2]), "s"(b[0]), "s"(b[1]), "s"(b[2]) : "vcc");
#else
    for (int i = 0; i < N; i++) {
        const uint64_t p = (uint64_t)a[i] * b[i];
        acc += p;
        over += acc < p;
    }
#endif
    return over;
}
// products h.w[I..3] * R.w[C - I] of column C, and how often the 64-bit sum overflows: counted from the first product on after which
// the constants allow an overflow
template <uint32_t MOD, int C>
struct FracColumn {
    static constexpr uint32_t r(int I) { return C - I >= 0 && C - I < 10 ? Frac<MOD>::P.R.w[C - I] : 0u; }
    static constexpr int first_carry() {
        unsigned __int128 b = (unsigned __int128)1 << 35;        // carry from the column before and the start value
        for (int I = 0; I < 4; I++) {
            b += (unsigned __int128)0xffffffffu * r(I);
            if ((b >> 64) != 0) return I;
        }
        return 4;
    }
    static constexpr int carries() { int n = 0; for (int I = first_carry(); I < 4; I++) n += r(I) != 0; return n; }
};
template <uint32_t MOD, int C>
DASH_HD uint32_t frac_column(const U128& h, uint64_t& acc) {
    typedef FracColumn<MOD, C> F;
    constexpr int first = F::first_carry(), N = F::carries();
    uint32_t a[4], b[4];
    int n = 0;
#pragma unroll
    for (int I = 0; I < 4; I++) {
        if (F::r(I) == 0) continue;
        if (I < first) mad64(acc, h.w[I], F::r(I));
        else { a[n] = h.w[I]; b[n] = F::r(I); n++; }
    }
    if constexpr (N > 0) return mad64_carries<N>(acc, a, b);
    else return 0;
}
// columns C..8 of h R: columns 8 - w[0] .. 7 are the fraction, column 8 the top super-digit
template <uint32_t MOD, int C>
DASH_HD void frac_product(const U128& h, uint64_t acc, uint32_t* f, uint32_t& top) {
    constexpr cm::FracPlan P = Frac<MOD>::P;
    if constexpr (C == 8) {
        top = (uint32_t)acc;
    } else {
        if constexpr (C == (int)P.bcol) acc += P.bword;
        const uint32_t over = frac_column<MOD, C>(h, acc);
        if constexpr (C >= 8 - (int)P.w[0]) f[C - (8 - (int)P.w[0])] = (uint32_t)acc;
        frac_product<MOD, C + 1>(h, (acc >> 32) | ((uint64_t)over << 32), f, top);
    }
}
// floor(v / m^E) for v <= VMAX
template <uint32_t MOD, uint32_t E, uint64_t VMAX>
DASH_HD uint32_t div_pow(uint32_t v) {
    constexpr uint32_t tw = E * cm::twos_of(MOD), plain = cm::magic_shift(VMAX, cm::ipow(MOD, E));
    constexpr uint64_t D = cm::ipow(MOD, E) >> tw;
    if constexpr (D == 1) return v >> tw;
    else if constexpr (plain == 0) return mulhi(v, cm::magic_mul(0, cm::ipow(MOD, E)));      // no shift at all
    else {
        constexpr uint32_t sh = cm::magic_shift(VMAX >> tw, D);
        static_assert(sh < 32, "multiply-high division out of range");
        return mulhi(v >> tw, cm::magic_mul(sh, D)) >> sh;
    }
}
// the four digits of v < m^4, packed: v = lo + m^2 hi, then each half into its two digits.  The digits are put in place by adding
// multiples of (256 - m) and (2^16 - m^2) to v: one multiply-add each, no shifts.
template <uint32_t MOD>
DASH_HD uint32_t split_dword(uint32_t v) {
    constexpr uint32_t m2 = MOD * MOD;
    const uint32_t hi = div_pow<MOD, 2, (uint64_t)m2 * m2 - 1>(v);
    if constexpr (MOD <= 13) {       // both halves in 16-bit fields of one word: m^2 times the reciprocal fits a field
        constexpr uint32_t s = cm::small_shift(MOD), M = ((1u << s) + MOD - 1) / MOD;
        static_assert(s < 16 && (m2 - 1) * M < 65536u && ((m2 - 1) << 16) < (1u << 24), "16-bit fields out of range");
        const uint32_t x = v + mul24(hi, 65536u - m2);
        return x + mul24((mul24(x, M) >> s) & ((0xffffu >> s) * 0x00010001u), 256u - MOD);
    } else {
        const uint32_t lo = v - mul24(hi, m2);
        const uint32_t t1 = div_pow<MOD, 1, m2 - 1>(hi), t0 = div_pow<MOD, 1, m2 - 1>(lo);
        return v + mul24(hi, 65536u - m2) + mul24(t0, 256u - MOD) + mul24(t1, (256u - MOD) << 16);
    }
}
// super-digit S < m^(4 N) into N dwords, the first at index i
template <uint32_t MOD, int N, class Emit>
DASH_HD void split_super(uint32_t S, int i, Emit& emit) {
    if constexpr (N == 1) {
        emit(i, split_dword<MOD>(S));
    } else {
        constexpr int N1 = N / 2;
        const uint32_t hi = div_pow<MOD, 4 * N1, cm::ipow(MOD, 4 * N) - 1>(S);
        split_super<MOD, N1>(S - hi * (uint32_t)cm::ipow(MOD, 4 * N1), i, emit);
        split_super<MOD, N - N1>(hi, i + N1, emit);
    }
}
// extraction K: super-digit ns - 2 - K off the top of the fraction f (w[K] words, least significant first)
template <uint32_t MOD, int K, class Emit>
DASH_HD void frac_extract(const uint32_t* f, Emit& emit) {
    constexpr cm::FracPlan P = Frac<MOD>::P;
    if constexpr (K + 1 < (int)P.ns) {
        constexpr int w = (int)P.w[K], wn = K + 2 < (int)P.ns ? (int)P.w[K + 1] : 0, gc = (int)cm::gc_of(MOD);
        constexpr uint32_t Q = (uint32_t)cm::ipow(MOD, 4 * gc);
        uint32_t g[w], c = 0;
#pragma unroll
        for (int i = 0; i < w; i++) {
            const uint64_t t = (uint64_t)f[i] * Q + c;
            g[i] = (uint32_t)t; c = (uint32_t)(t >> 32);
        }
        split_super<MOD, gc>(c, ((int)P.ns - 2 - K) * gc, emit);
        frac_extract<MOD, K + 1>(g + (w - wn), emit);
    }
}

template <class MI, class Emit>
DASH_HD void decompress(const MI& M, const U128& h, Emit emit) {
    if constexpr (cmod_m<MI>::value > 2) {
        constexpr uint32_t m = cmod_m<MI>::value;
        constexpr cm::FracPlan P = Frac<m>::P;
        static_assert(P.low > 0 && P.high > 0, "errors leave the window of exact digits");
        static_assert(MI::lam <= cm::lam_ceil(m), "digits past 2^128");
        // shorter labels (the floor rule) are the same digits without the last ones
        auto put = [&](int i, uint32_t w) {
            if (MI::lam < cm::lam_ceil(m) && (MI::lam & 3) && i == (int)(MI::lam >> 2)) w &= (1u << (8 * (MI::lam & 3))) - 1u;
            if (i < (int)MI::ndw) emit(i, w);
        };
        uint32_t f[8], top;
        frac_product<m, (int)P.c0>(h, 0, f, top);
        split_super<m, (int)P.top>(top, (int)((P.ns - 1) * cm::gc_of(m)), put);
        frac_extract<m, 0>(f, put);
    } else if constexpr (cmod_m<MI>::value == 2) {   // digits are bits: spread 4 bits into 4 bytes
#pragma unroll
        for (int i = 0; i < (int)M.ndw; i++) {
            uint32_t nib = (h.w[i >> 3] >> (4 * (i & 7))) & 0xfu;
            emit(i, mul24(nib, 0x00204081u) & 0x01010101u);
        }
    } else {
        U128 x = h;
        uint32_t S = 0, have = 0;     // digits left in the current super-digit
        uint32_t bits = 128;          // the number is below 2^bits
        uint32_t w = 0;
#pragma unroll
        for (uint32_t j = 0; j < M.lam; j++) {
            if (have == 0) {
                S = take_superdigit(x, M, bits);
                bits = bits > M.Qdbits ? bits - M.Qdbits : 0;
                have = M.gd;
            }
            uint32_t q = M.omagic ? mulhi(S >> M.tw, M.omagic) : (S >> M.tw);   // S div m = (S >> tw) div mo; omagic = 0: mo = 1
            uint32_t d = S - mul24(q, M.m);
            S = q; have--;
            w |= d << (8 * (j & 3));
            if ((j & 3) == 3) { emit((int)(j >> 2), w); w = 0; }
        }
        if (M.lam & 3) emit((int)(M.lam >> 2), w);
    }
}

struct Limbs { uint32_t l[8]; };
DASH_HD Limbs to_limbs(const U128& h) {
    Limbs x;
#pragma unroll
    for (int i = 0; i < 4; i++) { x.l[2 * i] = h.w[i] & 0xffffu; x.l[2 * i + 1] = h.w[i] >> 16; }
    return x;
}

// digit 0 alone: h mod m
template <class MI>
DASH_HD uint32_t mod_u128(const U128& h, const MI& M) {
    Limbs x = to_limbs(h);
    uint32_t r = 0;
#pragma unroll
    for (int i = 7; i >= 0; i--) r = mod_m((r << 16) | x.l[i], M);    // r < 256, (r<<16)|limb < 2^24
    return r;
}

// The moduli with a compile-time description: the CRT primes up to 37 and the accumulation moduli of the default digit sets, with
// their label lengths under one of the two rules.  The gate sources are compiled once per rule (DASH_RULE_FLOOR: the floor rule, else
// the ceil rule), each in an inline namespace of its own; the launch functions carry the rule in their name (DASH_FN) and are picked
// by the context's rule (dash_internal.h).
#define DASH_PASTE2(a, b) a##b
#define DASH_PASTE(a, b) DASH_PASTE2(a, b)
#if defined(DASH_RULE_FLOOR)
#define DASH_RULE_NS floor_rule
#define DASH_RULE_IS_FLOOR true
#define DASH_FN(name) DASH_PASTE(name, _floor)
#define DASH_HOT_MODS(X) \
    X(2, 128) X(3, 80) X(5, 55) X(7, 45) X(11, 37) X(13, 34) X(17, 31) X(19, 30) X(23, 28) X(29, 26) X(31, 25) X(37, 24) \
    X(26, 27) X(96, 19) X(46, 23) X(204, 16) X(10, 38) X(91, 19) X(22, 28) X(90, 19)
#else
#define DASH_RULE_NS ceil_rule
#define DASH_RULE_IS_FLOOR false
#define DASH_FN(name) DASH_PASTE(name, _ceil)
#define DASH_HOT_MODS(X) \
    X(2, 128) X(3, 81) X(5, 56) X(7, 46) X(11, 38) X(13, 35) X(17, 32) X(19, 31) X(23, 29) X(29, 27) X(31, 26) X(37, 25) \
    X(26, 28) X(96, 20) X(46, 24) X(204, 17) X(10, 39) X(91, 20) X(22, 29) X(90, 20)
#endif

inline namespace DASH_RULE_NS {
constexpr bool kFloorRule = DASH_RULE_IS_FLOOR;
// f(description of M): compile-time description for the hot moduli, run-time otherwise
template <class F>
DASH_HD void with_mod(const ModInfo& M, F&& f) {
#define DASH_MOD_CASE(MOD, LAM) case MOD: if (M.lam == LAM) { f(CMod<MOD, LAM>{M.dtab}); return; } break;
    switch (M.m) {
        DASH_HOT_MODS(DASH_MOD_CASE)
        default: break;
    }
#undef DASH_MOD_CASE
    f(M);
}

// description of type QD (ModInfo itself, or a CMod) built from the run-time record
template <class QD> struct make_mod { static DASH_HD QD from(const ModInfo& M) { return QD{M.dtab}; } };
template <> struct make_mod<ModInfo> { static DASH_HD ModInfo from(const ModInfo& M) { return M; } };

// index of the compile-time description that fits M (1..), 0 if none
DASH_HD int hot_mod_index(const ModInfo& M) {
    int idx = 0;
#define DASH_MOD_IDX(MOD, LAM) idx++; if (M.m == MOD && M.lam == LAM) return idx;
    DASH_HOT_MODS(DASH_MOD_IDX)
#undef DASH_MOD_IDX
    return 0;
}

// Digit sets (d_1; d, .., d) of the sign gadget whose kernels exist with compile-time moduli, as (m_c, lambda, m_1, lambda):
// m_1 = d_1 the accumulation modulus of digit 1, m_c = k d that of the others.  The default sets of the 8-, 12-, 7- and
// 9-prime bases (the bases of the paper's models).
#if defined(DASH_RULE_FLOOR)
#define DASH_DIGIT_SETS(X) X(96, 19, 26, 27) X(204, 16, 46, 23) X(91, 19, 10, 38) X(90, 19, 22, 28)
#else
#define DASH_DIGIT_SETS(X) X(96, 20, 26, 28) X(204, 17, 46, 24) X(91, 20, 10, 39) X(90, 20, 22, 29)
#endif
template <class MC_, class M1_> struct DigitSet { typedef MC_ MC; typedef M1_ M1; };
// index (1..) of the set with these two moduli, 0 if none
DASH_HD int digit_set_index(const ModInfo& Mc, const ModInfo& M1) {
    int idx = 0;
#define DASH_SET_IDX(MC, LC, M1_, L1) idx++; if (Mc.m == MC && Mc.lam == LC && M1.m == M1_ && M1.lam == L1) return idx;
    DASH_DIGIT_SETS(DASH_SET_IDX)
#undef DASH_SET_IDX
    return 0;
}
// f(DigitSet of compile-time descriptions) for index 1.., f(DigitSet<ModInfo, ModInfo>) for 0
template <class F>
void with_digit_set(int index, F&& f) {
    int idx = 0;
#define DASH_SET_CASE(MC, LC, M1_, L1) if (++idx == index) { f(DigitSet<CMod<MC, LC>, CMod<M1_, L1>>{}); return; }
    DASH_DIGIT_SETS(DASH_SET_CASE)
#undef DASH_SET_CASE
    f(DigitSet<ModInfo, ModInfo>{});
}

}  // inline namespace
}  // namespace dash
