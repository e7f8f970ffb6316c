// dash_act_eval.hip -- the evaluator's side of a whole ReLU or scaling layer in ONE launch (Appendix, Approximated Garbled Sign,
// Garbled Mixed-Radix Addition, mixed-modulus half gates; Sec. The Scaling Operation).
//
// The values of an activation layer are independent, so a block takes EPB of them through the gadget with a wave per residue and
// barriers between its steps; the wires in between (digit wires and their sums, carries, the halved residues, the sign bit, the
// shifted mod-2 wire) stay in registers and LDS.  Against one launch per step of the gadget (digit gates, sums, carry chain, half
// gates; times the repetitions of the scaling gadget) this saves the launches of small layers, whose time is a chain of short
// dependent kernels with cold instruction caches, and half of the memory traffic of large ones, whose time is the gather of table
// rows (a row of 20 bytes moves a 128-byte line) plus the digit wires that were written and read back.
//
//   step 1  wave = residue i: [scaling: cast of the mod-2 wire into Z_p, b = (x - cast) / 2]; the label is compressed and its n digit
//           gates evaluated; their output labels are added into LDS, digit by digit in 16-bit fields
//   step 2  all lanes: the sums mod m_j, packed
//   step 3  four lanes per value walk the n dependent gates of the mixed-radix addition and share each AES; the sign bit's label
//           stays packed (128 digits of modulus 2 = 128 bits)
//   step 4  ReLU: wave = residue: both half gates and z = V + beta x - U
//
// Three forms.  Deep (EPB = 64): a lane owns (value, residue) and works through the n digit gates.  Shallow (EPB = 16): four lanes do,
// every fourth digit each.  Tiny (EPB = 2 or 1): four lanes own (value, residue, digit) and share the AES, for layers so small that
// their time is the latency of one value.
// The deep form is bound by the hashes of its waves (vector issue 0.7 of the cycles that a CU is busy; two blocks per CU).  With one copy of
// T0..T3 two thirds of its LDS cycles were bank collisions; with HalfTab 75 264 values of the 8-prime base take 152 us a repetition instead
// of 168, 9 216 (one block per CU) 36 instead of 45.
// For digit sets with compile-time moduli over the first NP primes; anything else takes the launches of dash_layers.hip one by one.
// Compiled once per digit set (DASH_SET = number of primes) and label-length rule.
#include <algorithm>

#include "dash_tabs.h"

#ifndef DASH_SET
#error "DASH_SET: number of primes of the digit set"
#endif

namespace dash {
inline namespace DASH_RULE_NS {
namespace {

#if DASH_SET == 7
typedef CMod<91, cm::lam_of(91, kFloorRule)> MC; typedef CMod<10, cm::lam_of(10, kFloorRule)> M1;
#elif DASH_SET == 8
typedef CMod<96, cm::lam_of(96, kFloorRule)> MC; typedef CMod<26, cm::lam_of(26, kFloorRule)> M1;
#elif DASH_SET == 9
typedef CMod<90, cm::lam_of(90, kFloorRule)> MC; typedef CMod<22, cm::lam_of(22, kFloorRule)> M1;
#elif DASH_SET == 12
typedef CMod<204, cm::lam_of(204, kFloorRule)> MC; typedef CMod<46, cm::lam_of(46, kFloorRule)> M1;
#endif
constexpr int kNP = DASH_SET;
constexpr uint32_t kPrimeMax = kNP == 7 ? 17 : kNP == 8 ? 19 : kNP == 9 ? 23 : 37;
// Deep form: dwords of digit sums (whole digits) that lie beside the table and behind it in rows as beside it; the digits after them take the
// half of the rows behind the table that these leave free.
constexpr uint32_t kSpanSums = 64, kCut = M1::ndw + (75 - M1::ndw) / MC::ndw * MC::ndw;
static_assert(kSpanSums + M1::ndw + (kMaxChain - 1) * MC::ndw - kCut <= 78, "two deep blocks fit a CU");
constexpr int kMaxX = 24;                           // dwords of the longest label of an odd prime (81 digits in six chunks)

// f(description) for the primes of the base; bit labels (p = 2) only where the caller asks for them
template <bool Two, class F>
__device__ __forceinline__ void with_prime(const ModInfo& M, F&& f) {
#define DASH_PRIME_CASE(MOD, LAM) case MOD: if constexpr ((MOD <= 37 && MOD != 26 && MOD != 10 && MOD != 22) && MOD <= kPrimeMax && (Two || MOD > 2)) f(CMod<MOD, LAM>{M.dtab}); break;
    switch (M.m) { DASH_HOT_MODS(DASH_PRIME_CASE) default: break; }
#undef DASH_PRIME_CASE
}

// 32 digits of modulus 2 (32 bytes) as 32 bits and back
__device__ __forceinline__ uint32_t pack_bits(const uint32_t* w) {
    uint32_t b = 0;
#pragma unroll
    for (int i = 0; i < 8; i++) b |= dot4(w[i], 0x08040201u) << (4 * i);
    return b;
}
__device__ __forceinline__ uint32_t pack_bits_at(const uint8_t* p) {
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; i++) w[i] = *(const uint32_t*)(p + 4 * i);
    return pack_bits(w);
}
// bits w of the digits 32 c .. 32 c + 31 of element e
__device__ __forceinline__ void store_bits(const LView& v, uint32_t e, int c, uint32_t w) {
#pragma unroll
    for (int ch = 0; ch < 2; ch++) {
        Dw4 d;
#pragma unroll
        for (int q = 0; q < 4; q++) d.w[q] = mul24((w >> (16 * ch + 4 * q)) & 0xfu, 0x00204081u) & kOnes;
        st_chunk(v, e, 2 * c + ch, d);
    }
}

template <bool RELU, int EPB, int Q>
__global__ __launch_bounds__(64 * (RELU ? kNP : kNP - 1), EPB == 64 ? (kNP == 12 ? 3 : 4) : 1) void k_act_eval(const ActLaunch) {
    constexpr int JL = 64 / (EPB * Q), NW = RELU ? kNP : kNP - 1, T = 64 * NW;
    constexpr bool Deep = EPB == 64;
    // The arguments are read through the constant address space: with the by-value parameter the compiler kept a copy in scratch memory.
    const auto& L = *(const __attribute__((address_space(4))) ActLaunch*)__builtin_amdgcn_kernarg_segment_ptr();
    auto view = [](const __attribute__((address_space(4))) LView& v) __attribute__((always_inline)) { return LView{v.p, v.cs, v.es}; };
    __shared__ uint32_t tt[Deep ? 1 : kTabWords];
    __shared__ __attribute__((aligned(16))) uint32_t bt_static[Deep ? 4 : kBankTabWords];
    __shared__ uint32_t kb[4][EPB];                 // the mod-2 wire of the repetition (scaling) or the sign bit (ReLU): 128 bits per value
    static_assert(!Deep || sizeof(kb) == HalfTab::base, "the static LDS in front of the table");
    // Dynamic LDS.  Deep form: the table's span (dynamic, so that the compiler, which takes 64 KB of it for a limit of the blocks per CU,
    // keeps to 128 registers: two blocks, 36 instead of 64 us for a repetition of 25 088 values of the 7-prime base); else the digit sums.
    extern __shared__ __attribute__((aligned(16))) uint32_t acc[];
    uint32_t* const bt = Deep ? acc : bt_static;
    // sums over the residues, two digits per word: word (digit dword i, even or odd digits h, value v) at sum0[at_dword(i) + h * kS + at(v)].
    // Deep form: in the half of the table's span that HalfTab leaves free, and behind the span (a 16-digit set needs 77 KB this way, two blocks
    // per CU; 87 KB in rows as beside the table: 75 264 values of 8 primes 409 us a repetition in 87, 276 in 77).
    uint32_t* const sum0 = Deep ? acc + HalfTab::hole : acc;
    constexpr int kS = Deep ? 2 * EPB : EPB;
    auto at_dword = [](uint32_t i) __attribute__((always_inline)) { return i * (2 * kS) + (Deep && i >= kCut ? (kSpanSums - kCut) * (2 * kS) - HalfTab::hole : 0u); };
    auto at = [](uint32_t v) __attribute__((always_inline)) { return Deep ? (v & 32u) + v : v; };      // (64 values: two rows of 32 words, 64 apart)
    const int n = (int)L.n;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    const uint32_t c = lane % Q, el = lane / Q % EPB, jl = lane / (Q * EPB);      // lane of the quad, value, digit
    const uint32_t e_raw = blockIdx.x * EPB + el, e = e_raw < L.n_elem ? e_raw : L.n_elem - 1;      // lanes past the end repeat the last value and store nothing
    const auto& RA = L.res[wave];
    struct { uint32_t digit_slot, hg_slot, cast_slot; const uint8_t *digit_table, *g_table, *e_table, *s_table, *cast_table, *shift; LView in, out; } R = {
        RA.digit_slot, RA.hg_slot, RA.cast_slot, RA.digit_table, RA.g_table, RA.e_table, RA.s_table, RA.cast_table, RA.shift, view(RA.in), view(RA.out)};
    const uint32_t* const rk = (const uint32_t*)L.key_rot.rk;              // of step 1's and step 4's hashes
    const uint32_t* const crk = (const uint32_t*)(Deep ? L.key_rot.rk : L.key.rk);      // of the carry chain's
    const ModInfo Mp = ld_mod(L.mods, RA.p);

    // lanes of the carry chain: four per value
    const bool chain_lane = threadIdx.x < 4 * EPB;
    const uint32_t cel = (threadIdx.x >> 2) % EPB, cc = threadIdx.x & 3u;
    const uint32_t ce_raw = blockIdx.x * EPB + cel, ce = ce_raw < L.n_elem ? ce_raw : L.n_elem - 1;
    const QuadKey qk = quad_key(crk, cc), qs = Q == 4 ? quad_key(rk, c) : QuadKey{};
    uint32_t x[kMaxX];                                                      // scaling: the residue (with the constants of the repetition before)
    uint32_t one = 0, up0 = 0;                                              // scaling, chain lanes: 32 bits of the constant-one wire and of the first mod-2 wire
    if constexpr (!RELU) {
        with_prime<false>(Mp, [&](auto P) __attribute__((always_inline)) {
#pragma unroll
            for (int ch = 0; ch < (int)P.nchunk; ch++) {
                const Dw4 d = ld_chunk(R.in, e, ch);
#pragma unroll
                for (int q = 0; q < 4; q++) x[4 * ch + q] = d.w[q];
            }
        });
        if (chain_lane) {
            const LView in2 = view(L.in2);
            one = pack_bits_at(L.one2 + 32 * cc);
            uint32_t w[8];
#pragma unroll
            for (int ch = 0; ch < 2; ch++) { const Dw4 d = ld_chunk(in2, ce, 2 * (int)cc + ch); w[4 * ch] = d.w[0]; w[4 * ch + 1] = d.w[1]; w[4 * ch + 2] = d.w[2]; w[4 * ch + 3] = d.w[3]; }
            up0 = pack_bits(w) ^ one;                                       // ShiftUp: + 1 on the mod-2 residue
        }
    }
    const uint32_t sums = M1::ndw + (uint32_t)(n - 1) * MC::ndw;           // dwords of the n digit sums
    for (uint32_t i = threadIdx.x; i < sums * 2 * EPB; i += T) sum0[at_dword(i / (2 * EPB)) + i / EPB % 2 * kS + at(i % EPB)] = 0;
    if (chain_lane && !RELU) kb[cc][cel] = up0;
    auto step_table = [&]() __attribute__((always_inline)) {               // (ends with a barrier)
        if constexpr (Deep) return load_halftab(bt, L.ttab);
        else return load_banktab(bt, L.ttab);
    };
    const auto tab = step_table();
    auto chain_table = [&]() __attribute__((always_inline)) {
        if constexpr (Deep) return tab;
        else return load_ttab(tt, L.ttab);
    };
    const auto ctab = chain_table();

    // a hash of step 1 or 4: by the lane, or by the four lanes of its quad together
    auto hash = [&](const U128& key, uint32_t slot) __attribute__((always_inline)) {
        if constexpr (Q == 4) return hash_block_quad(key, L.elem_base + e, slot, L.layer, qs, rk, tab);
        else return hash_block(key, L.elem_base + e, slot, L.layer, rk, tab);
    };
    U128 K = {{0, 0, 0, 0}};
    uint32_t colour = 0;
    for (int rep = 0; rep < (int)L.repeat; rep++) {
        const uint64_t toff = (uint64_t)rep * L.rep_bytes;                  // tables of this repetition
        const uint32_t soff = (uint32_t)rep * L.rep_slots;
        // ---- step 1: digit gates
        if constexpr (RELU) {
            with_prime<true>(Mp, [&](auto P) __attribute__((always_inline)) { K = compress(P, [&](int i) __attribute__((always_inline)) { return ld_dw(R.in, e, i); }, &colour); });
        } else {
            // (the hash stands outside the dispatch on the prime: one copy of its code)
            const U128 Ky = {{kb[0][el], kb[1][el], kb[2][el], kb[3][el]}};
            uint32_t rw[kMaxX];
            auto load_row = [&](auto P) __attribute__((always_inline)) {
                const uint32_t* row = (const uint32_t*)(R.cast_table + toff + ((size_t)e * 2 + (Ky.w[0] & 1u)) * (P.ndw * 4));
#pragma unroll
                for (int i = 0; i < (int)P.ndw; i++) rw[i] = row[i];
            };
            // (shallow form: the row's loads go out before the hash; deep form: registers are short and other waves hide them)
            if constexpr (!Deep) with_prime<false>(Mp, load_row);
            const U128 h = hash(Ky, R.cast_slot + soff);
            with_prime<false>(Mp, [&](auto P) __attribute__((always_inline)) {
                typedef decltype(P) PD;
                if constexpr (Deep) load_row(P);
                decompress(P, h, [&](int i, uint32_t hd) __attribute__((always_inline)) { x[i] = halve4(x[i], submod4(rw[i], hd, P), (PD::m + 1) / 2, P); });
                K = compress(P, [&](int i) __attribute__((always_inline)) { return x[i]; }, &colour);
                // ShiftDown: the constant that the next repetition's halving, or the layer's output, takes with it (digits past lambda: 0 + 0)
#pragma unroll
                for (int i = 0; i < (int)PD::ndw; i++) x[i] = addmod4(x[i], *(const uint32_t*)(R.shift + 4 * i), P);
            });
        }
        {
            SlotHasher H(K, L.elem_base + e, L.layer);
            const uint8_t* seg0 = R.digit_table + toff;
            const uint64_t rows = (uint64_t)L.n_elem * Mp.m;                // rows of a digit's segment
            const uint64_t mine = (uint64_t)e * Mp.m + colour;
            for (int j = 1 + (int)jl; j <= n; j += JL) {
                const uint32_t slot = R.digit_slot + soff + (uint32_t)(j - 1);
                uint32_t rw[M1::ndw > MC::ndw ? M1::ndw : MC::ndw];
                const uint32_t* row = (const uint32_t*)(j == 1 ? seg0 + mine * (M1::ndw * 4)
                                                               : seg0 + rows * (M1::ndw * 4 + (uint32_t)(j - 2) * (MC::ndw * 4)) + mine * (MC::ndw * 4));
#pragma unroll
                for (int i = 0; i < (int)MC::ndw; i++) rw[i] = row[i];
                if (j == 1) {
#pragma unroll
                    for (int i = (int)MC::ndw; i < (int)M1::ndw; i++) rw[i] = row[i];
                }
                const U128 h = Deep ? H.get(slot, rk, tab) : hash(K, slot);
                uint32_t* a = sum0 + at_dword(j == 1 ? 0u : M1::ndw + (uint32_t)(j - 2) * MC::ndw) + at(el);
                auto put = [&](int i, uint32_t w) __attribute__((always_inline)) {
                    if (Q == 4 && c != (uint32_t)(i & 3)) return;           // (the lanes of a quad hold the same label)
                    sum_add(a + 2 * kS * i, w & 0x00ff00ffu);
                    sum_add(a + 2 * kS * i + kS, (w >> 8) & 0x00ff00ffu);
                };
                if (j == 1) { const M1 M{nullptr}; decompress(M, h, [&](int i, uint32_t hd) __attribute__((always_inline)) { put(i, submod4(rw[i], hd, M)); }); }
                else { const MC M{nullptr}; decompress(M, h, [&](int i, uint32_t hd) __attribute__((always_inline)) { put(i, submod4(rw[i], hd, M)); }); }
            }
        }
        __syncthreads();
        // ---- step 2: the sums mod m_j (fields below 16 * 255)
        for (uint32_t t = threadIdx.x; t < sums * EPB; t += T) {
            const uint32_t i = t / EPB, c = t % EPB;
            uint32_t* a = sum0 + at_dword(i) + at(c);
            const uint32_t ev = a[0], od = a[kS];
            auto reduce = [&](auto M) __attribute__((always_inline)) { return mod_m(ev & 0xffffu, M) | (mod_m(ev >> 16, M) << 16) | (mod_m(od & 0xffffu, M) << 8) | (mod_m(od >> 16, M) << 24); };
            a[0] = i < M1::ndw ? reduce(M1{nullptr}) : reduce(MC{nullptr});
            a[kS] = 0;
        }
        __syncthreads();
        // ---- step 3: the carry chain.  One loop over its n gates, one copy of the hash; the sum of the next digit is fetched under the
        // hash of the current one.
        if (chain_lane) {
            const MC Mc{nullptr};
            const M1 Mf{nullptr};
            constexpr int kIn = (int)(M1::ndw > MC::ndw ? M1::ndw : MC::ndw);
            uint32_t cw[kIn] = {}, sm[kIn];
            auto fetch = [&](int j) __attribute__((always_inline)) {                                   // packed sum of digit j; cleared for the next repetition
                uint32_t* a = sum0 + at_dword(j == 1 ? 0u : M1::ndw + (uint32_t)(j - 2) * MC::ndw) + at(cel);
#pragma unroll
                for (int i = 0; i < kIn; i++) if (i < (int)MC::ndw || j == 1) { sm[i] = a[i * 2 * kS]; DASH_WAVE_POINT(); a[i * 2 * kS] = 0; }
            };
            wave_priority<3>();
            fetch(n);
#pragma unroll 1
            for (int j = n; j >= 1; j--) {
                uint32_t in[kIn], rw[kIn > 8 ? kIn : 8], col;
                const uint8_t* table = L.chain_table[j] + toff;
                U128 k;
                if (j > 1) {
#pragma unroll
                    for (int i = 0; i < (int)MC::ndw; i++) in[i] = addmod4(sm[i], cw[i], Mc);
                    const uint32_t ndw = j > 2 ? MC::ndw : M1::ndw;
                    const uint32_t* row = (const uint32_t*)(table + ((size_t)ce * MC::m + (in[0] & 0xffu)) * (ndw * 4));
#pragma unroll
                    for (int i = 0; i < (int)MC::ndw; i++) rw[i] = row[i];
                    if (j == 2) {
#pragma unroll
                        for (int i = (int)MC::ndw; i < (int)M1::ndw; i++) rw[i] = row[i];
                    }
                    fetch(j - 1);
                    k = compress(Mc, [&](int i) __attribute__((always_inline)) { return in[i]; }, &col);
                } else {                                                    // final gate: the lane's 32 of the 128 bits
#pragma unroll
                    for (int i = 0; i < (int)M1::ndw; i++) in[i] = addmod4(sm[i], cw[i], Mf);
                    const uint32_t* row = (const uint32_t*)(table + ((size_t)ce * M1::m + (in[0] & 0xffu)) * 128 + 32 * cc);
#pragma unroll
                    for (int i = 0; i < 8; i++) rw[i] = row[i];
                    k = compress(Mf, [&](int i) __attribute__((always_inline)) { return in[i]; }, &col);
                }
                const uint32_t slot = L.chain_slot + soff + (uint32_t)(j > 1 ? j - 2 : n - 1);
                const U128 h = hash_block_quad(k, L.elem_base + ce, slot, L.layer, qk, crk, ctab);
                if (j > 2) {
                    decompress(Mc, h, [&](int i, uint32_t hd) __attribute__((always_inline)) { cw[i] = submod4(rw[i], hd, Mc); });
                } else if (j == 2) {
                    decompress(Mf, h, [&](int i, uint32_t hd) __attribute__((always_inline)) { cw[i] = submod4(rw[i], hd, Mf); });
                } else {
                    const uint32_t h01 = cc & 1u ? h.w[1] : h.w[0], h23 = cc & 1u ? h.w[3] : h.w[2];
                    uint32_t bit = pack_bits(rw) ^ (cc & 2u ? h23 : h01);
                    if constexpr (!RELU) {
                        const bool last = rep + 1 == (int)L.repeat;
                        if (last ? L.last_coef : L.up_coef) bit ^= one;
                        if (last && ce_raw < L.n_elem) store_bits(view(L.out2), ce, (int)cc, bit);
                    }
                    kb[cc][cel] = bit;
                }
            }
            wave_priority<0>();
        }
        __syncthreads();
    }
    if constexpr (!RELU) {
        if (jl == 0 && c == 0 && e_raw < L.n_elem) {
            with_prime<false>(Mp, [&](auto P) __attribute__((always_inline)) {
#pragma unroll
                for (int ch = 0; ch < (int)P.nchunk; ch++) {
                    Dw4 d;
#pragma unroll
                    for (int q = 0; q < 4; q++) d.w[q] = 4 * ch + q < (int)P.ndw ? x[4 * ch + q] : 0u;
                    st_chunk(R.out, e, ch, d);
                }
            });
        }
    } else {
        // ---- step 4: z = V + beta x - U.  Role 0: U (garbler half, from the label of x), role 1: V (evaluator half, from the sign
        // bit's label), role 2: beta.  Shallow form: the roles side by side in three lanes of the value.
        const U128 Ky = {{kb[0][el], kb[1][el], kb[2][el], kb[3][el]}};
        const uint32_t cy = Ky.w[0] & 1u;
        U128 hu, hv, hb;
        if constexpr (JL >= 3) {
            const uint32_t role = jl < 2 ? jl : 2u;
            const U128 key = {{role ? Ky.w[0] : K.w[0], role ? Ky.w[1] : K.w[1], role ? Ky.w[2] : K.w[2], role ? Ky.w[3] : K.w[3]}};
            hu = hash(key, R.hg_slot + role);
            hv = hb = hu;
        } else {
#pragma unroll 1
            for (uint32_t role = 0; role < 3; role++) {                     // (one copy of the hash)
                const U128 key = {{role ? Ky.w[0] : K.w[0], role ? Ky.w[1] : K.w[1], role ? Ky.w[2] : K.w[2], role ? Ky.w[3] : K.w[3]}};
                const U128 h = hash(key, R.hg_slot + role);
                if (role == 0) hu = h;
                else if (role == 1) hv = h;
                else hb = h;
            }
        }
        with_prime<true>(Mp, [&](auto P) __attribute__((always_inline)) {
            typedef decltype(P) PD;
            constexpr bool bits = PD::m == 2;
            constexpr int ndw = bits ? 4 : (int)PD::ndw, nch = (int)PD::nchunk;       // bit labels stay packed
            const int64_t g_off = (R.g_table - R.e_table) + (int64_t)(((uint64_t)e * PD::m + colour) * (PD::ndw * 4));
            const int64_t e_off = (int64_t)(((uint64_t)e * 2 + cy) * (PD::ndw * 4));
            auto half = [&](int64_t off, const U128& h, uint32_t* w) __attribute__((always_inline)) {            // output label: its row minus the hash
                const uint8_t* row = R.e_table + off;
                if constexpr (bits) {
#pragma unroll
                    for (int c = 0; c < 4; c++) w[c] = pack_bits_at(row + 32 * c) ^ h.w[c];
                } else {
                    uint32_t rw[ndw];
#pragma unroll
                    for (int i = 0; i < ndw; i++) rw[i] = ((const uint32_t*)row)[i];
                    decompress(P, h, [&](int i, uint32_t hd) __attribute__((always_inline)) { w[i] = submod4(rw[i], hd, P); });
                }
            };
            const uint32_t s = *(const uint32_t*)(R.s_table + ((size_t)e * 2 + cy) * 4);
            uint32_t u[ndw], v[ndw], beta = mod_m(s + PD::m - mod_u128(hb, P), P);
            if constexpr (JL >= 3) {
                half(jl == 0 ? g_off : e_off, hu, u);
#pragma unroll
                for (int i = 0; i < ndw; i++) v[i] = (uint32_t)__shfl((int)u[i], (int)(Q * (el + EPB)), 64);
                beta = (uint32_t)__shfl((int)beta, (int)(Q * (el + 2 * EPB)), 64);
            } else {
                half(g_off, hu, u);
                half(e_off, hv, v);
            }
            if (jl != 0 || c != 0 || e_raw >= L.n_elem) return;
            if constexpr (bits) {
#pragma unroll
                for (int c = 0; c < 4; c++) store_bits(R.out, e, c, u[c] ^ v[c] ^ (beta ? K.w[c] : 0u));
            } else {
#pragma unroll
                for (int ch = 0; ch < nch; ch++) {
                    const Dw4 xw = ld_chunk(R.in, e, ch);
                    Dw4 z;
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const int i = 4 * ch + q;
                        z.w[q] = i < ndw ? submod4(axpymod4(v[i < ndw ? i : 0], beta, xw.w[q], P), u[i < ndw ? i : 0], P) : 0u;
                    }
                    st_chunk(R.out, e, ch, z);
                }
            }
        });
    }
}

}  // namespace

// see launch_act_eval in dash_layers.hip, which has checked that the digit set and the primes are this file's
int DASH_FN(DASH_PASTE(launch_act_eval_, DASH_SET))(const dash_ctx* c, ActLaunch& L, bool relu, hipStream_t s) {
    static_assert(sizeof(ActLaunch) <= 4096, "kernel argument block");
    constexpr int kShallow = 16, kTiny = kNP >= 9 ? 1 : 2;                  // values per block (tiny: 16 or 8 digits of 4 lanes each)
    // Tiny and shallow blocks have a CU each (64 KB of tables), so a form is taken while its blocks are one round of the 256 CUs: a
    // second round costs the whole latency again (320 values of the 9-prime base: 50 us in 320 tiny blocks, 28 in shallow ones).
    // From two rounds of shallow blocks on the deep form is the faster one (6 400 values, us a repetition, scaling: 44 shallow and 39 deep on
    // the 8-prime base, 45 and 37 on 7, 54 and 48 on 9, 73 and 65 on 12; 4 096 values: 24 and 39 on 8).
    // The deep form's digit sums lie in the table's span, which holds 64 dwords of them (the default sets have 35 to 56), and go on behind it.
    const uint32_t sums = M1::ndw + (L.n - 1) * MC::ndw;
    const int form = L.n_elem < c->act_shallow_min_elems && L.n_elem <= 256u * kTiny ? ACT_TINY
                   : L.n_elem < c->act_deep_min_elems ? ACT_SHALLOW : ACT_DEEP;
    const uint32_t epb = form == ACT_DEEP ? 64 : form == ACT_SHALLOW ? kShallow : kTiny;
    const dim3 grid((L.n_elem + epb - 1) / epb), block(64 * (relu ? kNP : kNP - 1));
    static_assert(HalfTab::words == kSpanSums * 4 * 64, "rows of the deep form");
    const uint32_t rows = sums <= kSpanSums ? kSpanSums : sums <= kCut ? sums : std::max(kCut, kSpanSums + sums - kCut);
    const size_t lds = form == ACT_DEEP ? (size_t)rows * 4 * epb * 4 : (size_t)sums * 2 * epb * 4;
    if (form == ACT_DEEP) {      // the kernel reads its table at HalfTab::base, whatever static LDS it was built with
        hipFuncAttributes attr;
        DASH_HIP(hipFuncGetAttributes(&attr, relu ? (const void*)k_act_eval<true, 64, 1> : (const void*)k_act_eval<false, 64, 1>));
        if (attr.sharedSizeBytes != HalfTab::base) return DASH_EUNSUPPORTED;
    }
    if (relu) {
        if (form == ACT_DEEP) hipLaunchKernelGGL((k_act_eval<true, 64, 1>), grid, block, lds, s, L);
        else if (form == ACT_SHALLOW) hipLaunchKernelGGL((k_act_eval<true, kShallow, 1>), grid, block, lds, s, L);
        else hipLaunchKernelGGL((k_act_eval<true, kTiny, 4>), grid, block, lds, s, L);
    } else {
        if (form == ACT_DEEP) hipLaunchKernelGGL((k_act_eval<false, 64, 1>), grid, block, lds, s, L);
        else if (form == ACT_SHALLOW) hipLaunchKernelGGL((k_act_eval<false, kShallow, 1>), grid, block, lds, s, L);
        else hipLaunchKernelGGL((k_act_eval<false, kTiny, 4>), grid, block, lds, s, L);
    }
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

}  // inline namespace
}  // namespace dash
