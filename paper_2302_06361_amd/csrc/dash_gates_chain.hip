// dash_gates_chain.hip -- the garbler's kernel for large batches of carry gates of the sign gadget (Appendix, Garbled Mixed-Radix Addition):
// many gates with one function table, over the accumulation moduli of the digit sets with compile-time kernels.
//
// Bound by vector issue like k_proj_garble, which takes these batches where this file's kernels do not apply; a row costs it the index
// of its gate and value, four loads of labels and tables and their addresses on top.  Here a lane keeps its value a (chain_garble_rows),
// and the labels of the next tile are fetched under the hash of the current one.
#include "dash_chain_rule.h"
#include "dash_tabs.h"

namespace dash {
inline namespace DASH_RULE_NS {

// Units (repetition, batch) of V waves each, one after the other over the grid's waves.
template <class MP, class QD>
__global__ __launch_bounds__(kBigThreads, 8) void k_chain_garble(const GateLaunch, uint32_t V) {
    // (the arguments through the constant address space, as in k_act_eval)
    const auto& L = *(const __attribute__((address_space(4))) GateLaunch*)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ uint32_t tt[kBankTabWords];
    const BankTab T = load_banktab(tt, L.ttab);
    const uint32_t reps = L.reps.n ? L.reps.n : 1u, njobs = L.njobs, units = njobs * reps, waves = gridDim.x * (kBigThreads / 64);
    const MP P{ld_mod(L.mods, MP::m).dtab};
    const QD Q{ld_mod(L.mods, QD::m).dtab};
    auto keys = [&]() __attribute__((always_inline)) { return read_again(L.key.rk); };
    const uint32_t share = ((uint32_t)(((uint64_t)L.jobs[0].n_elem * MP::m + 63) / 64) + V - 1) / V;      // tiles of a unit's wave, at most
    Pace pace((units * V + waves - 1) / waves * share);
    for (uint32_t vw = blockIdx.x * (kBigThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64); vw < units * V; vw += waves) {
        const uint32_t unit = __builtin_amdgcn_readfirstlane(vw / V), rep = __builtin_amdgcn_readfirstlane(unit / njobs);
        const auto& J = L.jobs[unit - rep * njobs];
        const int64_t wires = (int64_t)rep * L.reps.wires;
        const ChainRows R{J.in.p + wires, J.out.p + wires, J.phi, J.in.cs, J.out.cs, J.table + (int64_t)rep * L.reps.tables,
                          J.elem_base, J.n_elem, J.slot + rep * L.reps.slots, L.layer};
        chain_garble_rows(R, P, Q, V, vw - unit * V, threadIdx.x & 63u, keys, T, [&]() __attribute__((always_inline)) { pace.tick(); });
    }
}

// Final gates: 16 KB of LDS beside the tables for the tile's bits, so that two blocks fit a CU.  (Rows kept in registers and staged as 32
// dwords a lane, with 140 KB of LDS and one block per CU: 115 us for the 1.96 M rows of 75 264 gates; this form takes 69.)
template <class MP>
__global__ __launch_bounds__(kBigThreads, 8) void k_chain_garble_bits(const GateLaunch, uint32_t V) {
    const auto& L = *(const __attribute__((address_space(4))) GateLaunch*)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ uint32_t tt[kBankTabWords];
    __shared__ __attribute__((aligned(16))) uint32_t stage[kBigThreads * 4];
    const BankTab T = load_banktab(tt, L.ttab);
    const uint32_t reps = L.reps.n ? L.reps.n : 1u, njobs = L.njobs, units = njobs * reps, waves = gridDim.x * (kBigThreads / 64);
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t* const st = stage + (threadIdx.x & ~63u) * 4;
    const MP P{ld_mod(L.mods, MP::m).dtab};
    U128 R2;                                            // the offset label of modulus 2
    {
        const uint32_t* d = ld_mod(L.mods, 2).dtab + 32;
        uint32_t colour;
        R2 = compress(CMod<2, 128>{nullptr}, [&](int i) { return gload32(d + i); }, &colour);
#pragma unroll
        for (int i = 0; i < 4; i++) R2.w[i] = __builtin_amdgcn_readfirstlane(R2.w[i]);
    }
    auto keys = [&]() __attribute__((always_inline)) { return read_again(L.key.rk); };
    const uint32_t share = ((uint32_t)(((uint64_t)L.jobs[0].n_elem * MP::m + 63) / 64) + V - 1) / V;      // tiles of a unit's wave, at most
    Pace pace((units * V + waves - 1) / waves * share);
    for (uint32_t vw = blockIdx.x * (kBigThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64); vw < units * V; vw += waves) {
        const uint32_t unit = __builtin_amdgcn_readfirstlane(vw / V), rep = __builtin_amdgcn_readfirstlane(unit / njobs), t0 = vw - unit * V;
        const auto& J = L.jobs[unit - rep * njobs];
        const int64_t wires = (int64_t)rep * L.reps.wires;
        const ChainRows R{J.in.p + wires, J.out.p + wires, J.phi, J.in.cs, J.out.cs, J.table + (int64_t)rep * L.reps.tables,
                          J.elem_base, J.n_elem, J.slot + rep * L.reps.slots, L.layer};
        constexpr int NP = (int)MP::ndw;
        const uint32_t n = R.n, tiles = (uint32_t)(((uint64_t)n * MP::m + 63) / 64), step = 64 * V / MP::m;
        if (t0 >= tiles) continue;
        const BitsLane B = chain_bits_lane(R, P, t0, lane);
        uint32_t gb = t0 * 64 / MP::m, z[NP];
        auto eo = [&](uint32_t b) __attribute__((always_inline)) { return 16 * (B.dg < n - b ? B.dg : n - 1 - b); };      // (past the end: the last gate, never stored)
        ld_label<NP>(R.in + (uint64_t)gb * 16, R.in_cs, eo(gb), z);
        for (uint32_t t = t0; t < tiles; t += V) {
            const uint32_t next = t + V < tiles ? gb + step : gb;
            pace.tick();
            uint32_t row;
            const U128 w = chain_bits_row(R, P, R2, B, gb, z, keys(), T, row);
            ld_label<NP>(R.in + (uint64_t)next * 16, R.in_cs, eo(next), z);
            *(uint4*)(st + lane * 4) = make_uint4(w.w[0], w.w[1], w.w[2], w.w[3]);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            uint32_t sl = lane;               // (opaque: its products are formed here and not held over the hash)
#if defined(__HIP_DEVICE_COMPILE__)
            asm volatile("" : "+v"(sl));
#endif
            const uint32_t part = sl & 7u;
#pragma unroll
            for (uint32_t half = 0; half < 2; half++) {               // four loads at a time
                uint32_t r[4], bits[4];
                Dw4 d[4];
#pragma unroll
                for (uint32_t i = 0; i < 4; i++) {
                    const uint32_t k = half * 32 + i * 8 + (sl >> 3);
                    r[i] = (uint32_t)__shfl((int)row, (int)k, 64);
                    d[i] = chain_bits_label<MP::m>(R, gb, r[i], part);
                    bits[i] = ((const uint16_t*)st)[k * 8 + part];
                }
#pragma unroll
                for (uint32_t i = 0; i < 4; i++) chain_bits_store<MP::m>(R, gb, r[i], part, bits[i], d[i]);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            gb = next;
        }
    }
}

int DASH_FN(launch_chain_garble)(const dash_ctx* c, GateLaunch& L, int njobs, hipStream_t s, bool* done) {
    *done = false;
    const GateJob& J0 = L.jobs[0];
    const uint64_t rows = (uint64_t)J0.n_elem * J0.p;
    for (int j = 0; j < njobs; j++) {
        const GateJob& J = L.jobs[j];
        if (J.mode != PAY_PHI || J.phi_stride != 0 || J.p != J0.p || J.q != J0.q || J.n_elem != J0.n_elem || J.in.es != 16u || J.out.es != 16u) return DASH_OK;
    }
    const ModInfo &Mp = c->mods[J0.p], &Mq = c->mods[J0.q];
    constexpr uint32_t kBlocks = 512;                   // two per CU
    const uint32_t units = (uint32_t)njobs * rep_count(L.reps);
    const uint32_t V = chain_waves((rows + 63) / 64, units, chain_quantum(J0.p), kBlocks * (kBigThreads / 64));
    if (rows + 64ull * V >= (1ull << 32) || (uint64_t)units * V >= (1ull << 31)) return DASH_OK;
    const uint32_t need = (units * V + kBigThreads / 64 - 1) / (kBigThreads / 64);
    const dim3 grid(need < kBlocks ? need : kBlocks), block(kBigThreads);
#define DASH_CHAIN(MC, LC, M1, L1)                                                                                                        \
    if (!*done && J0.p == MC && Mp.lam == LC && J0.q == MC) {                                                                             \
        hipLaunchKernelGGL((k_chain_garble<CMod<MC, LC>, CMod<MC, LC>>), grid, block, 0, s, L, V);                                        \
        *done = true;                                                                                                                     \
    }                                                                                                                                     \
    if (!*done && J0.p == MC && Mp.lam == LC && J0.q == M1 && Mq.lam == L1) {                                                             \
        hipLaunchKernelGGL((k_chain_garble<CMod<MC, LC>, CMod<M1, L1>>), grid, block, 0, s, L, V);                                        \
        *done = true;                                                                                                                     \
    }                                                                                                                                     \
    if (!*done && J0.p == M1 && Mp.lam == L1 && J0.q == 2 && Mq.lam == 128) {                                                             \
        hipLaunchKernelGGL((k_chain_garble_bits<CMod<M1, L1>>), grid, block, 0, s, L, V);                                                 \
        *done = true;                                                                                                                     \
    }
    DASH_DIGIT_SETS(DASH_CHAIN)
#undef DASH_CHAIN
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

}  // inline namespace
}  // namespace dash
