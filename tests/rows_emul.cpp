// Host emulation of the bodies of the garbler's kernels for batches of carry gates (the kernels themselves: carry_emul.cpp) and of the
// evaluator's for gates of any moduli: chain_garble_rows and the helpers of the final gates, wave by wave and lane by lane over
// exactly-sized buffers under the sanitizers, against garble_body on the same gates, every table byte, for the pairs of moduli that the
// kernels are compiled for; eval_many_body against eval_body.  Test code, not part of libdash.
// usage: rows_emul <gates> <quanta of tiles per round of waves> <seed>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "../paper_2302_06361_amd/csrc/dash_bodies.h"
#include "../paper_2302_06361_amd/csrc/dash_hostconst.h"

using namespace dash;
using namespace dash::hostconst;

static uint32_t TT[1024];
struct HostTab {
    template <int R, int B> uint32_t at(uint32_t w) const { return TT[R * 256 + ((w >> (8 * B)) & 0xffu)]; }
};
static uint64_t rng_state;
static uint32_t rnd() { rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(rng_state >> 33); }

static std::vector<ModInfo> mods(256);
static uint32_t n, quanta;
static GateLaunch G;

static std::vector<uint8_t> labels(const ModInfo& M) {
    std::vector<uint8_t> v((size_t)M.nchunk * n * 16, 0);
    for (uint32_t e = 0; e < n; e++)
        for (uint32_t d = 0; d < M.lam; d++) v[((size_t)(d / 16) * n + e) * 16 + d % 16] = (uint8_t)(rnd() % M.m);
    return v;
}
template <class MP, class QD>
static bool same() {
    const ModInfo &Mp = mods[MP::m], &Mq = mods[QD::m];
    if (Mp.lam != MP::lam || Mq.lam != QD::lam) { fprintf(stderr, "label lengths\n"); return false; }
    std::vector<uint8_t> in = labels(Mp), out0 = labels(Mq), phi(MP::m), want((size_t)n * MP::m * Mq.ndw * 4, 0xDD), got(want.size(), 0xEE);
    for (auto& v : phi) v = (uint8_t)(rnd() % QD::m);
    GateJob& J = G.jobs[0];
    memset(&J, 0, sizeof(J));
    J.p = MP::m; J.q = QD::m; J.slot = 57; J.mode = PAY_PHI; J.elem_base = (1ull << 32) - 3; J.n_elem = n;
    J.in = LView{in.data(), (int64_t)16 * n, 16u}; J.out = LView{out0.data(), (int64_t)16 * n, 16u};
    J.phi = phi.data(); J.table = want.data();
    const uint32_t blocks = (uint32_t)(((uint64_t)n * MP::m + kThreads - 1) / kThreads);
    for (uint32_t bx = 0; bx < blocks; bx++)
        for (uint32_t tx = 0; tx < (uint32_t)kThreads; tx++) { DirectSink sink; garble_body<QD>(G, bx, 0, tx, HostTab(), sink); }
    const uint32_t V = quanta * chain_quantum(MP::m);
    if (64 * V % MP::m) { fprintf(stderr, "quantum of %u\n", MP::m); return false; }
    const ChainRows R{in.data(), out0.data(), phi.data(), (int64_t)16 * n, (int64_t)16 * n, got.data(), J.elem_base, n, J.slot, G.layer};
    for (uint32_t t0 = 0; t0 < V; t0++)
        for (uint32_t lane = 0; lane < 64; lane++)
            chain_garble_rows(R, MP{Mp.dtab}, QD{Mq.dtab}, V, t0, lane, [] { return (const uint32_t*)G.key.rk; }, HostTab());
    if (got != want) { fprintf(stderr, "%u -> %u: tables differ\n", MP::m, QD::m); return false; }
    return true;
}

// the final gates: rows of bits, written 16 bytes a lane
template <class MP>
static bool same_bits() {
    const ModInfo &Mp = mods[MP::m], &M2 = mods[2];
    std::vector<uint8_t> in = labels(Mp), out0 = labels(M2), phi(MP::m), want((size_t)n * MP::m * 128, 0xDD), got(want.size(), 0xEE);
    for (auto& v : phi) v = (uint8_t)(rnd() % 2);
    GateJob& J = G.jobs[0];
    memset(&J, 0, sizeof(J));
    J.p = MP::m; J.q = 2; J.slot = 91; J.mode = PAY_PHI; J.elem_base = (1ull << 32) - 2; J.n_elem = n;
    J.in = LView{in.data(), (int64_t)16 * n, 16u}; J.out = LView{out0.data(), (int64_t)16 * n, 16u};
    J.phi = phi.data(); J.table = want.data();
    const uint32_t blocks = (uint32_t)(((uint64_t)n * MP::m + kThreads - 1) / kThreads);
    for (uint32_t bx = 0; bx < blocks; bx++)
        for (uint32_t tx = 0; tx < (uint32_t)kThreads; tx++) { DirectSink sink; garble_body<CMod<2, 128>>(G, bx, 0, tx, HostTab(), sink); }
    const uint32_t V = quanta * chain_quantum(MP::m), tiles = (n * MP::m + 63) / 64;
    const ChainRows R{in.data(), out0.data(), phi.data(), (int64_t)16 * n, (int64_t)16 * n, got.data(), J.elem_base, n, J.slot, G.layer};
    uint32_t colour;
    const U128 R2 = compress(CMod<2, 128>{nullptr}, [&](int i) { return M2.dtab[32 + i]; }, &colour);
    for (uint32_t t0 = 0; t0 < V; t0++)
        for (uint32_t t = t0, gb = t0 * 64 / MP::m; t < tiles; t += V, gb += 64 * V / MP::m) {
            U128 bits[64];
            uint32_t row[64];
            for (uint32_t lane = 0; lane < 64; lane++) {
                const BitsLane B = chain_bits_lane(R, MP{Mp.dtab}, t0, lane);
                uint32_t z[MP::ndw];
                ld_label<(int)MP::ndw>(in.data() + (uint64_t)gb * 16, R.in_cs, 16 * (B.dg < n - gb ? B.dg : n - 1 - gb), z);
                bits[lane] = chain_bits_row(R, MP{Mp.dtab}, R2, B, gb, z, G.key.rk, HostTab(), row[lane]);
            }
            for (uint32_t i = 0; i < 8; i++)
                for (uint32_t lane = 0; lane < 64; lane++) {
                    const uint32_t k = i * 8 + lane / 8, part = lane % 8, b16 = (bits[k].w[part / 2] >> (16 * (part % 2))) & 0xffffu;
                    chain_bits_store<MP::m>(R, gb, row[k], part, b16, chain_bits_label<MP::m>(R, gb, row[k], part));
                }
        }
    if (got != want) { fprintf(stderr, "%u -> 2: tables differ\n", MP::m); return false; }
    return true;
}

// the evaluator's gates of any moduli (eval_many_body) against eval_body
static bool same_eval(uint32_t p, uint32_t q) {
    const ModInfo &Mp = mods[p], &Mq = mods[q];
    std::vector<uint8_t> in = labels(Mp), table((size_t)n * p * Mq.ndw * 4, 0), want((size_t)Mq.nchunk * n * 16, 0xDD), got(want.size(), 0xEE);
    for (size_t r = 0; r < (size_t)n * p; r++)
        for (uint32_t d = 0; d < Mq.lam; d++) table[r * Mq.ndw * 4 + d] = (uint8_t)(rnd() % q);
    GateJob& J = G.jobs[0];
    memset(&J, 0, sizeof(J));
    J.p = p; J.q = q; J.mode = PAY_PHI; J.elem_base = (1ull << 32) - 5; J.n_elem = n;
    J.in = LView{in.data(), (int64_t)16 * n, 16u}; J.out = LView{want.data(), (int64_t)16 * n, 16u}; J.table = table.data();
    const EvalGate E{in.data(), table.data(), got.data(), (int64_t)16 * n, (int64_t)16 * n, J.elem_base, n, p, q};
    for (uint32_t bx = 0; bx < (n + kThreads - 1) / kThreads; bx++)
        for (uint32_t tx = 0; tx < (uint32_t)kThreads; tx++) {
            eval_body<ModInfo>(G, bx, 0, tx, HostTab());
            eval_many_body(E, mods.data(), G.layer, G.key.rk, bx, tx, HostTab());
        }
    if (got != want) { fprintf(stderr, "eval %u -> %u: labels differ\n", p, q); return false; }
    return true;
}

int main(int argc, char** argv) {
    if (argc != 4) return 2;
    n = (uint32_t)atoi(argv[1]); quanta = (uint32_t)atoi(argv[2]);
    rng_state = (uint64_t)atoll(argv[3]);
    uint8_t S[256], fixed[16];
    make_sbox(S);
    make_ttab(S, TT);
    for (int i = 0; i < 16; i++) fixed[i] = (uint8_t)(i * 7 + 1);
    memset(&G, 0, sizeof(G));
    expand_key(fixed, S, G.key.rk);
    std::vector<std::vector<uint32_t>> dtab(256);
    for (int m = 2; m < 256; m++) {
        fill_modinfo(mods[m], m, kFloorRule);
        ModInfo& M = mods[m];
        dtab[m].assign((size_t)M.m * M.ndw, 0);
        for (uint32_t d = 0; d < M.lam; d++) {
            const uint32_t r = d == 0 ? 1u : rnd() % M.m;
            for (uint32_t a = 0; a < M.m; a++) dtab[m][(size_t)a * M.ndw + d / 4] |= (a * r % M.m) << (8 * (d % 4));
        }
        M.dtab = dtab[m].data();
    }
    G.mods = mods.data(); G.layer = 11; G.njobs = 1;
    bool ok = true;
#define PAIR(MC, LC, M1, L1) ok = ok && same<CMod<MC, LC>, CMod<MC, LC>>() && same<CMod<MC, LC>, CMod<M1, L1>>() && same_bits<CMod<M1, L1>>();
    DASH_DIGIT_SETS(PAIR)
#undef PAIR
    static const int primes[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
    for (int i = 0; i < 12; i++) ok = ok && same_eval(primes[i], primes[(i + 5) % 12]) && same_eval(primes[(i + 1) % 12], primes[i]);
    if (ok) printf("ok\n");
    return ok ? 0 : 1;
}
