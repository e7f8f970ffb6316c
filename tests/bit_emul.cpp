// The garbler's kernel for gates on one wire of modulus 2 (dash_gates_bit.hip) through tests/simt: every prime with a compile-time description, casts
// and both gates of the half gates, several repetitions, jobs dealt out to groups of lanes, over exactly-sized buffers under the sanitizers;
// against garble_body on the same gates, every table byte.  Test code, not part of libdash.
// usage: bit_emul <gates> <jobs> <repetitions> <first slot> <seed> [<groups> <blocks>]
// groups, blocks: the kernel itself with its jobs dealt out to so many lanes per (value, row), in so many blocks (0 0: the launcher, which has to
// give a lane more than one job), over both assignments of the half gates' modes to the primes and masks of all digits.
#define SIMT_MAIN
#include <hip/hip_runtime.h>

#include "../paper_2302_06361_amd/csrc/dash_gates_bit.hip"
#include "../paper_2302_06361_amd/csrc/dash_hostconst.h"

using namespace dash;
using namespace dash::hostconst;

static uint32_t TT[1024];
struct HostTab {
    template <int R, int B> uint32_t at(uint32_t w) const { return TT[R * 256 + ((w >> (8 * B)) & 0xffu)]; }
};
static uint64_t rng_state;
static uint32_t rnd() { rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(rng_state >> 33); }

static dash_ctx ctx;
static uint32_t n, jobs, reps, slot0;
static bool forced = false;                     // groups and blocks were given
static uint32_t groups = 0, blocks = 0;
static AesKey fixed, fixed_rot;

static std::vector<uint8_t> labels(const ModInfo& M, uint32_t count) {
    std::vector<uint8_t> v((size_t)count * M.nchunk * n * 16, 0);
    for (uint32_t u = 0; u < count; u++)
        for (uint32_t e = 0; e < n; e++)
            for (uint32_t d = 0; d < M.lam; d++) v[(size_t)u * M.nchunk * n * 16 + ((size_t)(d / 16) * n + e) * 16 + d % 16] = (uint8_t)(rnd() % M.m);
    return v;
}

// half: every second job the evaluator's half of a half gate, every other the known input, from the first on or (shift) from the second; else casts
static bool same(bool half, uint32_t shift = 0) {
    static const uint32_t primes[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
    // all wires of a repetition are one step apart: the widest label, of modulus 2
    const int64_t step = (int64_t)8 * n * 16, tstep = (int64_t)n * 2 * 128;
    std::vector<std::vector<uint8_t>> wires(1 + 2 * jobs), want(jobs), got(jobs);
    auto spread = [&](const ModInfo& M) {                       // labels of the repetitions, step bytes apart, the last one exactly sized
        const std::vector<uint8_t> all = labels(M, reps);
        const size_t one = all.size() / reps;
        std::vector<uint8_t> v((size_t)(reps - 1) * step + one, 0);
        for (uint32_t r = 0; r < reps; r++) memcpy(v.data() + r * step, all.data() + r * one, one);
        return v;
    };
    std::vector<uint8_t> mask((size_t)n), phi(2 * jobs);
    std::vector<std::vector<uint8_t>> masks(jobs);      // of every digit of the job's prime (forced)
    GateLaunch L;
    memset(&L, 0, sizeof(L));
    L.mods = ctx.d_mods; L.layer = 9; L.njobs = jobs; L.ttab = TT;
    L.reps = Reps{reps, 300, step, tstep};
    wires[0] = spread(ctx.mods[2]);
    for (auto& v : mask) v = (uint8_t)rnd();
    for (uint32_t j = 0; j < jobs; j++) {
        GateJob& J = L.jobs[j];
        J.p = 2; J.q = primes[(j + (half ? 0 : 1)) % 12]; J.slot = slot0 + j;
        J.mode = !half ? PAY_PHI : (j + shift) % 2 ? PAY_SHORT : PAY_EHALF;
        J.elem_base = (1ull << 32) - 3; J.n_elem = n;
        J.in = LView{wires[0].data(), (int64_t)16 * n, 16u};
        const ModInfo& M = ctx.mods[J.q];
        wires[1 + j] = spread(M);
        J.out = LView{wires[1 + j].data(), (int64_t)16 * n, 16u};
        if (half) {
            for (uint32_t e = 0; e < n; e++) mask[e] %= 2;      // a digit of every prime
            J.r = mask.data();
            if (forced) {
                masks[j].resize(n);
                for (uint32_t e = 0; e < n; e++) masks[j][e] = (uint8_t)(e < 2 ? (J.q - 1) * (1 - e) : rnd() % J.q);
                J.r = masks[j].data();
            }
            wires[1 + jobs + j] = spread(M);
            J.x0 = LView{wires[1 + jobs + j].data(), (int64_t)16 * n, 16u};
        } else {
            phi[2 * j] = (uint8_t)(rnd() % J.q); phi[2 * j + 1] = (uint8_t)(rnd() % J.q);
            J.phi = phi.data() + 2 * j;
        }
        const size_t bytes = (size_t)(reps - 1) * tstep + (size_t)n * 2 * (J.mode == PAY_SHORT ? 4 : M.ndw * 4);
        want[j].assign(bytes, 0xDD); got[j].assign(bytes, 0xDD);
    }
    L.key = fixed;
    for (uint32_t j = 0; j < jobs; j++) L.jobs[j].table = want[j].data();
    for (uint32_t r = 0; r < reps; r++)
        for (uint32_t j = 0; j < jobs; j++)
            for (uint32_t bx = 0; bx < (2 * n + kThreads - 1) / kThreads; bx++)
                for (uint32_t tx = 0; tx < (uint32_t)kThreads; tx++) { DirectSink sink; garble_body<PerJobMod>(L, bx, j, tx, HostTab(), sink, r); }
    for (uint32_t j = 0; j < jobs; j++) L.jobs[j].table = got[j].data();
    bool done = false;
    if (forced && groups) {
        L.key = fixed_rot;
        if (half) hipLaunchKernelGGL(k_bit_garble<true>, dim3(blocks), dim3(kBigThreads), 0, nullptr, L, groups);
        else hipLaunchKernelGGL(k_bit_garble<false>, dim3(blocks), dim3(kBigThreads), 0, nullptr, L, groups);
        for (uint32_t j = 0; j < jobs; j++)
            if (got[j] != want[j]) { fprintf(stderr, "job %u (q %u, mode %u), forced: tables differ\n", j, L.jobs[j].q, L.jobs[j].mode); return false; }
        return true;
    }
    if (forced && bit_groups(((uint64_t)n * 2 + kThreads - 1) / kThreads * reps, jobs) >= jobs) { fprintf(stderr, "one job per lane\n"); return false; }
    if (DASH_FN(launch_bit_garble)(&ctx, L, (int)jobs, nullptr, &done) != DASH_OK || !done) { fprintf(stderr, "not launched\n"); return false; }
    for (uint32_t j = 0; j < jobs; j++)
        if (got[j] != want[j]) { fprintf(stderr, "job %u (q %u, mode %u): tables differ\n", j, L.jobs[j].q, L.jobs[j].mode); return false; }
    // what is not the kernel's is left alone
    for (int k = 0; k < 4; k++) {
        GateLaunch N = L;
        if (k == 0) N.jobs[jobs - 1].p = 3;
        if (k == 1) N.jobs[jobs - 1].q = 97;
        if (k == 2) N.jobs[jobs - 1].out.es = 0, N.jobs[jobs - 1].mode = half ? PAY_EHALF : PAY_PHI;
        if (k == 3) { if (jobs < 2) continue; N.jobs[jobs - 1].n_elem = n + 1; }
        bool taken = true;
        if (DASH_FN(launch_bit_garble)(&ctx, N, (int)jobs, nullptr, &taken) != DASH_OK || taken) { fprintf(stderr, "case %d taken\n", k); return false; }
    }
    return true;
}

int main(int argc, char** argv) {
    if (argc != 6 && argc != 8) return 2;
    forced = argc == 8;
    if (forced) { groups = (uint32_t)atoi(argv[6]); blocks = (uint32_t)atoi(argv[7]); }
    n = (uint32_t)atoi(argv[1]); jobs = (uint32_t)atoi(argv[2]); reps = (uint32_t)atoi(argv[3]); slot0 = (uint32_t)atoi(argv[4]);
    rng_state = (uint64_t)atoll(argv[5]);
    if (jobs < 1 || jobs > (uint32_t)kMaxJobs || reps < 1 || (groups != 0) != (blocks != 0)) return 2;
    uint8_t S[256], key[16];
    make_sbox(S);
    make_ttab(S, TT);
    for (int i = 0; i < 16; i++) key[i] = (uint8_t)(i * 7 + 1);
    expand_key(key, S, fixed.rk);
    fixed_rot = fixed;
    rotate_round_keys(fixed_rot.rk);
    ctx.fixed = fixed; ctx.fixed_rot = fixed_rot; ctx.d_ttab = TT;
    std::vector<std::vector<uint32_t>> dtab(256);
    for (int m = 2; m < 256; m++) {
        ModInfo& M = ctx.mods[m];
        fill_modinfo(M, m, kFloorRule);
        dtab[m].assign((size_t)M.m * M.ndw, 0);
        for (uint32_t d = 0; d < M.lam; d++) {
            const uint32_t r = d == 0 ? 1u : rnd() % M.m;
            for (uint32_t a = 0; a < M.m; a++) dtab[m][(size_t)a * M.ndw + d / 4] |= (a * r % M.m) << (8 * (d % 4));
        }
        M.dtab = dtab[m].data();
    }
    ctx.d_mods = ctx.mods;
    const bool ok = same(false) && same(true) && (!forced || same(true, 1));
    if (ok) printf("ok\n");
    return ok ? 0 : 1;
}
