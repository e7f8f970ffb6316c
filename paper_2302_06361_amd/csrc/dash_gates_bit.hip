// dash_gates_bit.hip -- the garbler's gates on one wire of modulus 2: the casts of the scaling gadget's mod-2 wire into the odd primes (Sec. The
// Scaling Operation), the evaluator's halves and known inputs of the half gates (Appendix, mixed-modulus half gate).
//
// These gates have two rows each and an output modulus per prime.  In a launch per output modulus they are short kernels one after the other,
// each with a round of one hash per lane, the copy of the tables and the packing of 128-byte labels: the seven casts of 75 264 values
// took 115 us a repetition.  Here one launch takes all of them, a lane per (value, row) that forms its label once and goes through the jobs: 42 us.
// (Held to 64 registers, two blocks per CU, it spills 50 of them; on 147 CUs, four tiles a block, 60 us.)
#include "dash_tabs.h"

namespace dash {
inline namespace DASH_RULE_NS {

// groups: the jobs are dealt out to so many lanes per (value, row)
template <bool Half>
__global__ __launch_bounds__(kBigThreads, 4) void k_bit_garble(const GateLaunch, uint32_t groups) {
    const auto& L = *(const __attribute__((address_space(4))) GateLaunch*)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ uint32_t tt[kBankTabWords];
    const BankTab T = load_banktab(tt, L.ttab);
    U128 R2;                                            // the offset label of modulus 2
    {
        const uint32_t* d = ld_mod(L.mods, 2).dtab + 32;
        uint32_t colour;
        R2 = compress(CMod<2, 128>{nullptr}, [&](int i) { return ld_const(d + i); }, &colour);
#pragma unroll
        for (int i = 0; i < 4; i++) R2.w[i] = __builtin_amdgcn_readfirstlane(R2.w[i]);
    }
    const uint32_t njobs = L.njobs, per = (njobs + groups - 1) / groups, reps = L.reps.n ? L.reps.n : 1u;
    const uint32_t tiles = (2 * L.jobs[0].n_elem + kThreads - 1) / kThreads, total = tiles * groups * reps;
    const uint32_t sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tx = threadIdx.x % kThreads;
    const uint32_t first = sub * gridDim.x + blockIdx.x, step = gridDim.x * (kBigThreads / kThreads);
    auto keys = [&]() __attribute__((always_inline)) { return read_again(L.key.rk); };
    Pace pace(first, total, step, per);
    for (uint32_t t = first; t < total; t += step) {
        const uint32_t unit = __builtin_amdgcn_readfirstlane(t / tiles), rep = __builtin_amdgcn_readfirstlane(unit / groups), j0 = (unit - rep * groups) * per;
        bit_garble_body<Half>(L, t - unit * tiles, rep, j0, j0 + per < njobs ? j0 + per : njobs, tx, R2, T, keys, [&]() __attribute__((always_inline)) { pace.tick(); });
    }
}

// One block fits a CU (registers): 1024 tiles at a time.  Where the values have fewer, the jobs are shared out to groups of lanes, none of them empty.
// tiles: of all repetitions
inline uint32_t bit_groups(uint64_t tiles, uint32_t njobs) {
    const uint64_t wanted = tiles < 1024 ? 1024 / tiles : 1;
    const uint32_t groups = wanted < njobs ? (uint32_t)wanted : njobs, per = (njobs + groups - 1) / groups;
    return (njobs + per - 1) / per;
}

int DASH_FN(launch_bit_garble)(const dash_ctx* c, GateLaunch& L, int njobs, hipStream_t s, bool* done) {
    *done = false;
    if (njobs < 1 || njobs > kMaxJobs) return DASH_EINVAL;
    const GateJob& J0 = L.jobs[0];
    if (c->mods[2].lam != 128 || !c->mods[2].dtab || J0.n_elem > (1u << 28)) return DASH_OK;
    double bytes = 0;
    for (int j = 0; j < njobs; j++) {
        const GateJob& J = L.jobs[j];
        if (J.p != 2 || J.mode == PAY_MULR || (J.mode == PAY_PHI) != (J0.mode == PAY_PHI) || J.phi_stride != 0 || J.n_elem != J0.n_elem || J.elem_base != J0.elem_base || J.in.p != J0.in.p || J.in.cs != J0.in.cs ||
            J.in.es != 16u || (J.mode != PAY_SHORT && J.out.es != 16u) || (J.mode == PAY_EHALF && J.x0.es != 16u) || J.q < 2 || J.q > 255 || !hot_mod_index(c->mods[J.q]))
            return DASH_OK;
        const double lq = J.mode == PAY_SHORT ? 1 : c->mods[J.q].lam;
        bytes += (double)J.n_elem * (128 + lq + 2 * lq + (J.mode == PAY_EHALF ? lq : 0));
    }
    *done = true;
    if (J0.n_elem == 0) return DASH_OK;
    const uint32_t reps = rep_count(L.reps);
    const uint64_t tiles = ((uint64_t)J0.n_elem * 2 + kThreads - 1) / kThreads * reps;
    const uint32_t groups = bit_groups(tiles, (uint32_t)njobs);
    if (tiles * groups > 0x7fffffffull) { *done = false; return DASH_OK; }
    L.key = c->fixed_rot; L.ttab = c->d_ttab; L.mods = c->d_mods; L.njobs = (uint32_t)njobs;
    ProfScope ps(c->prof, DASH_PROF_GARBLE, s, 2.0 * J0.n_elem * njobs * reps, bytes * reps);
    const dim3 grid((uint32_t)(tiles * groups < 256 ? tiles * groups : 256));      // (a tile on every CU before a second one on any)
    if (J0.mode == PAY_PHI) hipLaunchKernelGGL(k_bit_garble<false>, grid, dim3(kBigThreads), 0, s, L, groups);
    else hipLaunchKernelGGL(k_bit_garble<true>, grid, dim3(kBigThreads), 0, s, L, groups);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

}  // inline namespace
}  // namespace dash
