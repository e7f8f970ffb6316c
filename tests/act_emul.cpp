// The library on the CPU through tests/simt: contexts, the evaluator's one-launch activation layers, the repacking of tables and the
// linear layers without matrix instructions, driven through the C ABI over exactly-sized buffers, for the address and undefined-behaviour sanitizers.  Test code, not part of libdash.
//
// One source, three kinds of object:
//   -DPART_ACT -DDASH_SET=k [-DDASH_RULE_FLOOR]   dash_act_eval.hip
//   -DPART_GATES [-DDASH_RULE_FLOOR]              draws, free gates and repacking of dash_gates.hip; the launches of the step-by-step
//                                                 path are absent and refuse
//   (none)                                        context, layer pipelines and main()
//
// usage: act_emul act  <in> <out>      in : int32 k rule kind n repeat layer in_place n_digits; uint64 elem_base; u16 primes[k] digits[n_digits];
//                                           u8 seed[16], labels per residue [n][lam], tables
//                                      out: u8 labels per residue [n][lam]
//        act_emul pack <in> <out>      the same in; out: u8 packed tables, tables unpacked from them
//        act_emul linear <in> <out>    in : int32 k rule batch in_h in_w in_c out_c kh stride pad bias garble shift n_digits; u16 primes[k]
//                                           digits[n_digits]; u8 seed[16], labels per residue [n_in][lam]; int32 weights[out_c][K], bias[out_c]
//                                      out: u8 labels per residue [n_out][lam].  Prepared weights start shift bytes past an aligned address.
#if !defined(PART_ACT) && !defined(PART_GATES)
#define SIMT_MAIN
#endif
#include <hip/hip_runtime.h>

#if defined(PART_ACT)

#include "../paper_2302_06361_amd/csrc/dash_act_eval.hip"
namespace dash { inline namespace DASH_RULE_NS { namespace {
thread_local uint32_t acc[85 * 256];                     // the kernel's dynamic LDS
const simt::dynamic_lds announce(acc, sizeof(acc));
} } }

#elif defined(PART_GATES)

#include "../paper_2302_06361_amd/csrc/dash_tabs.h"
// (the garbling kernels are not launched here: four instantiations instead of twenty, for the repacking of rows of bits and of one, two and
// four tiles at a time; the other moduli take its form for any modulus)
#undef DASH_HOT_MODS
#if defined(DASH_RULE_FLOOR)
#define DASH_HOT_MODS(X) X(2, 128) X(3, 80) X(26, 27) X(96, 19)
#else
#define DASH_HOT_MODS(X) X(2, 128) X(3, 81) X(26, 28) X(96, 20)
#endif
#include "../paper_2302_06361_amd/csrc/dash_gates.hip"
namespace dash { inline namespace DASH_RULE_NS {
#define ABSENT(ret, name, ...) ret DASH_FN(name)(__VA_ARGS__) { fprintf(stderr, "act_emul: " #name " is not part of this program\n"); abort(); }
ABSENT(int, launch_eval, const dash_ctx*, GateLaunch&, int, hipStream_t)
ABSENT(int, launch_eval_many, const dash_ctx*, EvalManyLaunch&, int, hipStream_t)
ABSENT(int, launch_chain_garble, const dash_ctx*, GateLaunch&, int, hipStream_t, bool*)
ABSENT(int, launch_bit_garble, const dash_ctx*, GateLaunch&, int, hipStream_t, bool*)
ABSENT(int, launch_chain_eval, const dash_ctx*, ChainLaunch&, hipStream_t)
ABSENT(int, launch_digits_eval, const dash_ctx*, DigitsLaunch&, hipStream_t)
ABSENT(int, launch_digits_garble, const dash_ctx*, DigitsLaunch&, hipStream_t)
ABSENT(int, launch_cast_halve, const dash_ctx*, CastLaunch&, int, hipStream_t)
ABSENT(int, launch_cast_digits_eval, const dash_ctx*, CastLaunch&, int, DigitsLaunch&, hipStream_t)
ABSENT(int, launch_hg_finish, const dash_ctx*, HgLaunch&, int, hipStream_t)
ABSENT(bool, hg_eval_quad_wanted, const dash_ctx*, uint32_t)
ABSENT(int, launch_hg_eval_quad, const dash_ctx*, HgLaunch&, int, hipStream_t)
} }

#else

#include "../paper_2302_06361_amd/csrc/dash_ctx.hip"
#include "../paper_2302_06361_amd/csrc/dash_layers.hip"

#include "../paper_2302_06361_amd/csrc/dash_linear.hip"

namespace dash {          // (the MFMA kernel is not part of this program)
bool dense_mfma_wanted(const dash_layer*, int64_t) { return false; }
int dense_mfma(dash_ctx*, const dash_layer*, bool, const dash_labels*, dash_labels*, hipStream_t) { abort(); }
}

static std::vector<uint8_t> slurp(const char* name) {
    FILE* f = fopen(name, "rb");
    if (!f) exit(2);
    std::vector<uint8_t> v;
    uint8_t buf[65536];
    for (size_t n; (n = fread(buf, 1, sizeof(buf), f)) > 0;) v.insert(v.end(), buf, buf + n);
    fclose(f);
    return v;
}
static void check(int st, const char* what) { if (st) { fprintf(stderr, "%s: %s\n", what, dash_strerror(st)); exit(4); } }

// a bundle of labels, every residue in a buffer of its own of exactly nchunk * n * 16 bytes
struct Bundle {
    dash_labels c;
    Bundle(dash_ctx* ctx, int64_t n) {
        memset(&c, 0, sizeof(c));
        c.n_elem = n;
        for (int i = 0; i < ctx->k; i++) {
            const size_t bytes = (size_t)ctx->mods[ctx->prime[i]].nchunk * n * 16;
            if (hipMalloc(&c.data[i], bytes)) exit(3);
            memset(c.data[i], 0, bytes);
            c.chunk_stride[i] = 16 * n;
        }
    }
    uint8_t* at(int i, int64_t e, uint32_t j) { return (uint8_t*)c.data[i] + (j / 16) * c.chunk_stride[i] + e * 16 + j % 16; }
    // the labels, residue after residue; false if a digit past the label's length is not zero
    bool read(dash_ctx* ctx, std::vector<uint8_t>& out) {
        for (int i = 0; i < ctx->k; i++) {
            const ModInfo& M = ctx->mods[ctx->prime[i]];
            for (int64_t e = 0; e < c.n_elem; e++) {
                for (uint32_t j = 0; j < M.lam; j++) out.push_back(*at(i, e, j));
                for (uint32_t j = M.lam; j < M.nchunk * 16; j++) if (*at(i, e, j)) return false;
            }
        }
        return true;
    }
};

static bool write_out(const char* name, const std::vector<uint8_t>& out) {
    FILE* f = fopen(name, "wb");
    return f && fwrite(out.data(), 1, out.size(), f) == out.size() && !fclose(f);
}

template <class Take> static int linear_main(const char* fout, Take take) {
    int32_t hd[14];
    memcpy(hd, take(sizeof(hd)), sizeof(hd));
    const int k = hd[0], nd = hd[13];
    std::vector<uint16_t> primes(k), digits(nd);
    memcpy(primes.data(), take(2 * k), 2 * k);
    memcpy(digits.data(), take(2 * nd), 2 * nd);
    const uint8_t* seed = take(16);
    dash_ctx* ctx = nullptr;
    check(dash_ctx_create(&ctx, primes.data(), k, hd[1], nullptr, seed, digits.data(), nd, 0), "dash_ctx_create");
    dash_layer L;
    memset(&L, 0, sizeof(L));
    L.kind = hd[3] == 1 && hd[4] == 1 && hd[7] == 1 ? DASH_DENSE : DASH_CONV2D;
    L.layer_id = 1; L.n_elem = hd[2]; L.in_h = hd[3]; L.in_w = hd[4]; L.in_c = hd[5]; L.out_c = hd[6]; L.kh = L.kw = hd[7]; L.stride = hd[8]; L.pad = hd[9];
    const int64_t n_in = (int64_t)hd[2] * hd[3] * hd[4] * hd[5];
    const int K = hd[7] * hd[7] * hd[5];
    Bundle a(ctx, n_in);
    for (int i = 0; i < k; i++)
        for (int64_t e = 0; e < n_in; e++)
            for (uint32_t j = 0; j < ctx->mods[primes[i]].lam; j++) *a.at(i, e, j) = *take(1);
    std::vector<int32_t> w((size_t)hd[6] * K), bias(hd[6]);
    memcpy(w.data(), take(4 * w.size()), 4 * w.size());
    memcpy(bias.data(), take(4 * bias.size()), 4 * bias.size());
    uint8_t* prepared;
    if (hipMalloc(&prepared, hd[12] + dash_weights_bytes(ctx, hd[6], K))) return 3;
    check(dash_weights_prepare(ctx, w.data(), hd[6], K, prepared + hd[12], nullptr), "dash_weights_prepare");
    L.weights = prepared + hd[12];
    L.bias = hd[10] ? bias.data() : nullptr;
    int64_t oe;
    check(dash_layer_sizes(ctx, &L, &oe, nullptr, nullptr), "dash_layer_sizes");
    Bundle o(ctx, oe * hd[2]);
    check(hd[11] ? dash_garble_layer(ctx, &L, &a.c, &o.c, nullptr, nullptr, nullptr) : dash_eval_layer(ctx, &L, &a.c, nullptr, &o.c, nullptr, nullptr), "layer");
    std::vector<uint8_t> out;
    return o.read(ctx, out) && write_out(fout, out) ? 0 : 5;
}

int main(int argc, char** argv) {
    if (argc != 4) return 2;
    const std::vector<uint8_t> in = slurp(argv[2]);
    const uint8_t* p = in.data();
    auto take = [&](size_t n) { if (p + n > in.data() + in.size()) exit(2); const uint8_t* at = p; p += n; return at; };
    if (!strcmp(argv[1], "linear")) return linear_main(argv[3], take);
    int32_t hd[8];
    uint64_t elem_base;
    memcpy(hd, take(32), 32);
    memcpy(&elem_base, take(8), 8);
    const int k = hd[0], n = hd[3], nd = hd[7];
    std::vector<uint16_t> primes(k), digits(nd);
    memcpy(primes.data(), take(2 * k), 2 * k);
    memcpy(digits.data(), take(2 * nd), 2 * nd);
    const uint8_t* seed = take(16);
    dash_ctx* ctx = nullptr;
    check(dash_ctx_create(&ctx, primes.data(), k, hd[1], nullptr, seed, digits.data(), nd, 0), "dash_ctx_create");
    dash_layer L;
    memset(&L, 0, sizeof(L));
    L.kind = hd[2]; L.layer_id = hd[5]; L.elem_base = (int64_t)elem_base; L.n_elem = n; L.repeat = hd[4];
    int64_t oe;
    size_t tb, sb;
    check(dash_layer_sizes(ctx, &L, &oe, &tb, &sb), "dash_layer_sizes");
    Bundle a(ctx, n), other(ctx, n);
    for (int i = 0; i < k; i++)
        for (int e = 0; e < n; e++)
            for (uint32_t j = 0; j < ctx->mods[primes[i]].lam; j++) *a.at(i, e, j) = *take(1);
    // the tables end where the buffer ends and begin 4 bytes past a 16-byte address: all that the interface promises
    const size_t gap = 4;
    std::vector<uint8_t> out;
    uint8_t* buf;
    if (hipMalloc(&buf, gap + tb)) return 3;
    uint8_t* tables = buf + gap;
    memcpy(tables, take(tb), tb);
    if (p != in.data() + in.size()) return 2;
    if (!strcmp(argv[1], "act")) {
        uint8_t* scratch;
        if (hipMalloc(&scratch, sb + 256)) return 3;
        Bundle& o = hd[6] ? a : other;
        check(dash_eval_layer(ctx, &L, &a.c, tables, &o.c, scratch, nullptr), "dash_eval_layer");
        if (!o.read(ctx, out)) { fprintf(stderr, "pad digits not zero\n"); return 5; }
        free(scratch);
    } else {
        size_t pb = 0;
        check(dash_tables_packed_bytes(ctx, &L) ? 0 : DASH_EUNSUPPORTED, "dash_tables_packed_bytes");
        pb = dash_tables_packed_bytes(ctx, &L);
        uint8_t* packed;
        if (hipMalloc(&packed, pb)) return 3;
        check(dash_tables_pack(ctx, &L, tables, packed, nullptr), "dash_tables_pack");
        memset(tables, 0xEE, tb);
        check(dash_tables_unpack(ctx, &L, packed, tables, nullptr), "dash_tables_unpack");
        out.assign(packed, packed + pb);
        out.insert(out.end(), tables, tables + tb);
        free(packed);
    }
    if (!write_out(argv[3], out)) return 2;
    free(buf);
    for (int i = 0; i < k; i++) { free(a.c.data[i]); free(other.c.data[i]); }
    dash_ctx_destroy(ctx);
    return 0;
}
#endif
