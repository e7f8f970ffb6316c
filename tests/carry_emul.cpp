// The garbler's kernels for large batches of carry gates (dash_gates_chain.hip) through tests/simt: units of several repetitions and batches,
// waves that walk over several tiles and several units, the tile's rows handed over in LDS, over exactly-sized buffers under the
// sanitizers; against garble_body on the same gates, every table byte.  Test code, not part of libdash.
// usage: carry_emul <gates> <quanta of tiles per wave round; 0: launch_chain_garble's own> <blocks> <jobs> <repetitions> <seed>
#define SIMT_MAIN
#include <hip/hip_runtime.h>

#include "../paper_2302_06361_amd/csrc/dash_gates_chain.hip"
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
static uint32_t n, quanta, blocks, jobs, reps;
static AesKey fixed, fixed_rot;

// one batch per job, the labels of a repetition one after the other in an arena, the tables likewise
template <class MP, class QD, class Launch>
static bool same(Launch launch) {
    const ModInfo &Mp = ctx.mods[MP::m], &Mq = ctx.mods[QD::m];
    if (Mp.lam != MP::lam || Mq.lam != QD::lam) { fprintf(stderr, "label lengths\n"); return false; }
    const size_t lin = (size_t)Mp.nchunk * n * 16, lout = (size_t)Mq.nchunk * n * 16, rows = (size_t)n * MP::m * Mq.ndw * 4;
    std::vector<uint8_t> wires(reps * jobs * (lin + lout), 0), want(reps * jobs * rows, 0xDD), got(want.size(), 0xEE);
    std::vector<uint8_t> phi(jobs * MP::m);
    for (auto& v : phi) v = (uint8_t)(rnd() % QD::m);
    auto fill = [&](uint8_t* at, const ModInfo& M) {
        for (uint32_t e = 0; e < n; e++)
            for (uint32_t d = 0; d < M.lam; d++) at[((size_t)(d / 16) * n + e) * 16 + d % 16] = (uint8_t)(rnd() % M.m);
    };
    for (uint32_t u = 0; u < reps * jobs; u++) { fill(wires.data() + u * (lin + lout), Mp); fill(wires.data() + u * (lin + lout) + lin, Mq); }
    GateLaunch L;
    memset(&L, 0, sizeof(L));
    L.mods = ctx.d_mods; L.layer = 11; L.njobs = jobs; L.ttab = TT;
    L.reps = Reps{reps, 1000, (int64_t)(jobs * (lin + lout)), (int64_t)(jobs * rows)};
    for (uint32_t j = 0; j < jobs; j++) {
        GateJob& J = L.jobs[j];
        uint8_t* w = wires.data() + j * (lin + lout);
        J.p = MP::m; J.q = QD::m; J.slot = 57 + j; J.mode = PAY_PHI; J.elem_base = (1ull << 32) - 3; J.n_elem = n;
        J.in = LView{w, (int64_t)16 * n, 16u}; J.out = LView{w + lin, (int64_t)16 * n, 16u}; J.phi = phi.data() + j * MP::m;
    }
    L.key = fixed;
    for (uint32_t j = 0; j < jobs; j++) L.jobs[j].table = want.data() + j * rows;
    for (uint32_t r = 0; r < reps; r++)
        for (uint32_t j = 0; j < jobs; j++)
            for (uint32_t bx = 0; bx < ((uint64_t)n * MP::m + kThreads - 1) / kThreads; bx++)
                for (uint32_t tx = 0; tx < (uint32_t)kThreads; tx++) { DirectSink sink; garble_body<QD>(L, bx, j, tx, HostTab(), sink, r); }
    L.key = fixed_rot;
    for (uint32_t j = 0; j < jobs; j++) L.jobs[j].table = got.data() + j * rows;
    bool done = true;
    if (quanta) launch(L, quanta * chain_quantum(MP::m));
    else if (DASH_FN(launch_chain_garble)(&ctx, L, (int)jobs, nullptr, &done) != DASH_OK) return false;
    if (!done || got != want) { fprintf(stderr, "%u -> %u: %s\n", MP::m, QD::m, done ? "tables differ" : "not launched"); return false; }
    return true;
}
template <class MP, class QD> static bool rows() {
    return same<MP, QD>([](GateLaunch& L, uint32_t V) { hipLaunchKernelGGL((k_chain_garble<MP, QD>), dim3(blocks), dim3(kBigThreads), 0, nullptr, L, V); });
}
template <class MP> static bool bits() {
    return same<MP, CMod<2, 128>>([](GateLaunch& L, uint32_t V) { hipLaunchKernelGGL((k_chain_garble_bits<MP>), dim3(blocks), dim3(kBigThreads), 0, nullptr, L, V); });
}

int main(int argc, char** argv) {
    if (argc != 7) return 2;
    n = (uint32_t)atoi(argv[1]); quanta = (uint32_t)atoi(argv[2]); blocks = (uint32_t)atoi(argv[3]); jobs = (uint32_t)atoi(argv[4]); reps = (uint32_t)atoi(argv[5]);
    rng_state = (uint64_t)atoll(argv[6]);
    if (jobs < 1 || jobs > (uint32_t)kMaxJobs || reps < 1) return 2;
    uint8_t S[256], key[16];
    make_sbox(S);
    make_ttab(S, TT);
    for (int i = 0; i < 16; i++) key[i] = (uint8_t)(i * 7 + 1);
    expand_key(key, S, fixed.rk);
    fixed_rot = fixed;
    rotate_round_keys(fixed_rot.rk);
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
    bool ok = true;
#define PAIR(MC, LC, M1, L1) ok = ok && rows<CMod<MC, LC>, CMod<MC, LC>>() && rows<CMod<MC, LC>, CMod<M1, L1>>() && bits<CMod<M1, L1>>();
    DASH_DIGIT_SETS(PAIR)
#undef PAIR
    if (ok) printf("ok\n");
    return ok ? 0 : 1;
}
