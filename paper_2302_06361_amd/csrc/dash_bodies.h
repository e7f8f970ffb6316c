// dash_bodies.h -- the per-lane bodies of the gate kernels, as host+device templates over the AES
// table accessor.  The __global__ kernels in dash_gates.hip call them with (blockIdx, threadIdx) and
// the LDS copy of the tables; the CPU test suite runs the very same bodies lane by lane under a
// sanitizer, against host memory.
#pragma once
#include "dash_core.h"
#include "dash_launch.h"

namespace dash {
inline namespace DASH_RULE_NS {

// dword i (digits 4i..4i+3) of element e of a label view
// The chunk base is wave-uniform (scalar registers); the lane part is a 32-bit byte offset, so the
// access is "scalar base + 32-bit vector offset" (elements per view are limited to 2^28 for this).
DASH_HD uint32_t lane_off(const LView& v, uint32_t e) { return v.es ? e << 4 : 0u; }   // es is 16 or 0
DASH_HD uint32_t ld_dw(const LView& v, uint32_t e, int i) {
    const uint8_t* base = v.p + (int64_t)(i >> 2) * v.cs + (i & 3) * 4;
    return *(const uint32_t*)(base + lane_off(v, e));
}
DASH_HD void st_dw(const LView& v, uint32_t e, int i, uint32_t w) {
    uint8_t* base = v.p + (int64_t)(i >> 2) * v.cs + (i & 3) * 4;
    *(uint32_t*)(base + lane_off(v, e)) = w;
}

// a whole 16-digit chunk of element e at once (label tensors are 16-byte aligned): one 16-byte access
struct alignas(16) Dw4 { uint32_t w[4]; };
DASH_HD Dw4 ld_chunk(const LView& v, uint32_t e, int ch) { return *(const Dw4*)(v.p + (int64_t)ch * v.cs + lane_off(v, e)); }
DASH_HD void st_chunk(const LView& v, uint32_t e, int ch, const Dw4& d) { *(Dw4*)(v.p + (int64_t)ch * v.cs + lane_off(v, e)) = d; }

// N dwords at base + off (base the same in all lanes: scalar base and 32-bit offset), 4-byte aligned, as wide as the hardware takes them
template <int N> DASH_HD void ld_dwords(const void* base, uint32_t off, uint32_t* w) {
#if defined(__HIP_DEVICE_COMPILE__)
    const auto* src = (const __attribute__((address_space(1))) uint8_t*)base + off;
#pragma unroll
    for (int i = 0; i < N; i++) w[i] = *(const __attribute__((address_space(1))) uint32_t*)(src + 4 * i);
#else
    const uint32_t* src = (const uint32_t*)((const uint8_t*)base + off);
    for (int i = 0; i < N; i++) w[i] = src[i];
#endif
}
// a dword of a table that is never written while a kernel runs, at an address that is the same in all lanes (a scalar load)
DASH_HD uint32_t ld_const(const uint32_t* p) {
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const __attribute__((address_space(4))) uint32_t*)p;
#else
    return *p;
#endif
}
// 16 bytes at base + off, 16-byte aligned
DASH_HD Dw4 ld_dw4(const uint8_t* base, uint32_t off) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = *(const __attribute__((address_space(1))) u32x4*)((const __attribute__((address_space(1))) uint8_t*)base + off);
    return Dw4{{v.x, v.y, v.z, v.w}};
#else
    return *(const Dw4*)(base + off);
#endif
}
// dword i of a row at base + off
DASH_HD void st_row(uint8_t* base, uint32_t off, int i, uint32_t w) {
#if defined(__HIP_DEVICE_COMPILE__)
    *(__attribute__((address_space(1))) uint32_t*)((__attribute__((address_space(1))) uint8_t*)base + off + 4 * i) = w;
#else
    *(uint32_t*)(base + off + 4 * i) = w;
#endif
}
// dwords 0..N-1 of the label at element offset eo (16 bytes an element) of a tensor of chunk stride cs, es = 16
template <int N> DASH_HD void ld_label(const uint8_t* p, int64_t cs, uint32_t eo, uint32_t* w) {
#pragma unroll
    for (int ch = 0; ch < (N + 3) / 4; ch++) {
        const Dw4 d = ld_dw4(p + (int64_t)ch * cs, eo);
#pragma unroll
        for (int q = 0; q < 4; q++) if (4 * ch + q < N) w[4 * ch + q] = d.w[q];
    }
}
// the same number, of which nothing is known (what is formed from it is formed where it stands); the same in all lanes
DASH_HD uint32_t opaque(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v));
#endif
    return v;
}
// the same for a number of each lane's
DASH_HD uint32_t opaque_lane(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(v));
#endif
    return v;
}
// keeps what stands before it from being moved behind what follows, and the other way round (loads ahead of a hash)
DASH_HD void schedule_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// compressed label and colour of a wire of modulus 2 (a sign bit or a mod-2 residue): the 128-digit description
// when that is the context's label length of modulus 2, the run-time record otherwise
template <class LoadDw>
DASH_HD U128 compress_mod2(const ModInfo* mods, LoadDw dw, uint32_t* colour) {
    if (ld_mod(mods, 2).lam == 128) return compress(CMod<2, 128>{nullptr}, dw, colour);
    const ModInfo M2 = ld_mod(mods, 2);
    return compress(M2, dw, colour);
}

// PRG labels: one lane per (job, element)
template <class Tab>
DASH_HD void draw_body(const DrawLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T) {
    const DrawJob& J = L.jobs[by];
    uint32_t e = bx * kThreads + tx;
    if (e >= J.n_elem) return;
    const ModInfo M = ld_mod(L.mods, J.m);
    U128 h = prg_block(J.elem_base + e, J.slot, L.layer, J.domain, J.m, L.key.rk, T);
    if (J.digit0_only) { J.out.p[e] = (uint8_t)mod_u128(h, M); return; }
    with_mod(M, [&](auto Q) {
        decompress(Q, h, [&](int i, uint32_t w) { st_dw(J.out, e, i, w); });
        for (int i = (int)Q.ndw; i < (int)Q.nchunk * 4; i++) st_dw(J.out, e, i, 0);
    });
}

// ... of a gadget's gates: one lane per (job, element)
template <class Tab>
DASH_HD void draw_many_body(const DrawManyLaunch& L, uint32_t bx, uint32_t by, uint32_t rep, uint32_t tx, const Tab& T) {
    const DrawManyJob& J = L.jobs[by];
    const uint32_t e = bx * kThreads + tx;
    if (e >= L.n_elem) return;
    const U128 h = prg_block(L.elem_base + e, J.slot + rep * L.reps.slots, L.layer, DOM_GATE, J.m, L.key.rk, T);
    const LView out{L.base + J.off + rep * L.reps.wires, 16 * (int64_t)L.n_elem, 16u};
    with_mod(ld_mod(L.mods, J.m), [&](auto Q) {
        decompress(Q, h, [&](int i, uint32_t w) { st_dw(out, e, i, w); });
        for (int i = (int)Q.ndw; i < (int)Q.nchunk * 4; i++) st_dw(out, e, i, 0);
    });
}

// free gates: out = sum_t coef_t * term_t mod m.  One lane per (element, 16-digit chunk): a 16-byte load
// per term.  Sums with unit coefficients (the mixed-radix additions of the sign gadget) accumulate two
// digits per 32-bit word in 16-bit fields; general coefficients go digit by digit.
DASH_HD void affine_body(const AffineLaunch& L, uint32_t bx, uint32_t by, uint32_t tx) {
    const AffineJob& J = L.jobs[by];
    const ModInfo M = ld_mod(L.mods, J.m);
    const uint64_t idx = (uint64_t)bx * kThreads + tx;
    if (idx >= (uint64_t)L.n_elem * M.nchunk) return;
    const uint32_t ch = (uint32_t)(idx / L.n_elem), e = (uint32_t)(idx - (uint64_t)ch * L.n_elem);
    const Term* T = L.terms + J.term_first;
    uint32_t out[4];
    if (J.unit) {
        uint32_t ev[4] = {0, 0, 0, 0}, od[4] = {0, 0, 0, 0};      // digits 0,2 / 1,3 of each dword, 16 bits each
        for (uint32_t t = 0; t < J.term_count; t++) {
            const uint32_t* src = (const uint32_t*)(T[t].v.p + (int64_t)ch * T[t].v.cs + lane_off(T[t].v, e));
            for (int q = 0; q < 4; q++) { uint32_t w = src[q]; ev[q] += w & 0x00ff00ffu; od[q] += (w >> 8) & 0x00ff00ffu; }
        }
        for (int q = 0; q < 4; q++)
            out[q] = mod_m(ev[q] & 0xffffu, M) | (mod_m(od[q] & 0xffffu, M) << 8) | (mod_m(ev[q] >> 16, M) << 16) | (mod_m(od[q] >> 16, M) << 24);
    } else {
        for (int q = 0; q < 4; q++) {
            uint32_t acc[4] = {0, 0, 0, 0};
            for (uint32_t t = 0; t < J.term_count; t++) {
                const uint32_t* src = (const uint32_t*)(T[t].v.p + (int64_t)ch * T[t].v.cs + lane_off(T[t].v, e));
                uint32_t w = src[q], cf = T[t].coef;
                for (int b = 0; b < 4; b++) acc[b] += mul24(cf, byte_of(w, b));      // <= 16 * 254 * 254 < 2^24
            }
            out[q] = mod_m(acc[0], M) | (mod_m(acc[1], M) << 8) | (mod_m(acc[2], M) << 16) | (mod_m(acc[3], M) << 24);
        }
    }
    uint32_t* dst = (uint32_t*)(J.out.p + (int64_t)ch * J.out.cs + lane_off(J.out, e));
    for (int q = 0; q < 4; q++) dst[q] = out[q];
}

// (x - cast) * 2^-1 mod p on four digits (scaling gadget)
template <class P>
DASH_HD uint32_t halve4(uint32_t x, uint32_t cast, uint32_t inv2, const P& Pm) {
    if (Pm.m <= 127) {
        // four digits at once (p odd): t = (x - cast) mod p, then t / 2 for even t and (t + p) / 2 for odd t.  Bytes stay
        // below 2p <= 254, and the bit that the shift brings in from the byte above is masked off.
        const uint32_t t = submod4(x, cast, Pm);
        const uint32_t odd = t & 0x01010101u;
        return ((t + odd * Pm.m) >> 1) & 0x7f7f7f7fu;
    }
    uint32_t b = 0;
    // digits past lambda: x and cast are 0 there, and inv2 * p = 0 mod p
    for (int b8 = 0; b8 < 4; b8++) b |= mod_m(mul24(inv2, byte_of(x, b8) + Pm.m - byte_of(cast, b8)), Pm) << (8 * b8);
    return b;
}
// the same view t repetitions on
DASH_HD LView rep_view(const LView& v, const Reps& R, uint32_t t) { return LView{v.p + (int64_t)t * R.wires, v.cs, v.es}; }

// garbler, scaling gadget: by < n the sum of digit by + 1 (one repetition per call); by = n the mod-2 wire and by > n the halving of an odd
// residue, whose repetitions follow from each other and are walked by the lane.  One lane per (element, 16-digit chunk).
DASH_HD void scale_free_body(const ScaleFreeLaunch& L, uint32_t bx, uint32_t by, uint32_t rep, uint32_t tx) {
    const uint32_t reps = rep_count(L.reps);
    if (by >= L.n && rep != 0) return;
    const HalveJob& J = L.halve[by > L.n ? by - L.n - 1 : 0];
    const ModInfo M = ld_mod(L.mods, by < L.n ? L.m[by + 1] : by == L.n ? 2u : J.p);
    const uint64_t idx = (uint64_t)bx * kThreads + tx;
    if (idx >= (uint64_t)L.n_elem * M.nchunk) return;
    const uint32_t ch = (uint32_t)(idx / L.n_elem), e = (uint32_t)(idx - (uint64_t)ch * L.n_elem);
    if (by < L.n) {
        const uint32_t j = by + 1;
        const int64_t at = (int64_t)rep * L.reps.wires + (int64_t)ch * L.cs + (int64_t)e * 16;
        uint32_t ev[4] = {0, 0, 0, 0}, od[4] = {0, 0, 0, 0};          // digits 0, 2 / 1, 3 of each dword, 16 bits each
        auto add = [&](const uint8_t* p) {
            const Dw4 d = *(const Dw4*)(p + at);
            for (int q = 0; q < 4; q++) { ev[q] += d.w[q] & 0x00ff00ffu; od[q] += (d.w[q] >> 8) & 0x00ff00ffu; }
        };
        for (uint32_t i = 0; i < L.nres; i++) add(L.a1 + L.a_prefix[j] + (int64_t)i * L.res_step);
        if (j < L.n) add(L.C[j]);
        Dw4 out;
        for (int q = 0; q < 4; q++)
            out.w[q] = mod_m(ev[q] & 0xffffu, M) | (mod_m(od[q] & 0xffffu, M) << 8) | (mod_m(ev[q] >> 16, M) << 16) | (mod_m(od[q] >> 16, M) << 24);
        *(Dw4*)(L.S[j] + at) = out;
    } else if (by == L.n) {
        const Dw4 one = ld_chunk(L.one2, e, (int)ch);
        auto plus = [&](Dw4 d, uint32_t coef) {
            for (int q = 0; q < 4; q++) d.w[q] ^= coef ? one.w[q] : 0u;
            return d;
        };
        st_chunk(L.up, e, (int)ch, plus(ld_chunk(L.x0, e, (int)ch), L.x0_coef));
        for (uint32_t t = 0; t < reps; t++) {
            const Dw4 bit = ld_chunk(rep_view(L.bit, L.reps, t), e, (int)ch);
            if (t + 1 < reps) st_chunk(rep_view(L.up, L.reps, t + 1), e, (int)ch, plus(bit, L.up_coef));
            else st_chunk(L.last, e, (int)ch, plus(bit, L.last_coef));
        }
    } else {
        const Dw4 one = ld_chunk(J.one, e, (int)ch);
        const uint32_t inv2 = (M.m + 1) / 2;
        Dw4 x = ld_chunk(J.x, e, (int)ch), shift;
        for (int q = 0; q < 4; q++) {
            shift.w[q] = axpymod4(0u, J.addc, one.w[q], M);
            if (J.addc0) x.w[q] = axpymod4(x.w[q], J.addc0, one.w[q], M);
        }
        for (uint32_t t = 0; t < reps; t++) {
            const Dw4 cast = ld_chunk(rep_view(J.cast, L.reps, t), e, (int)ch);
            Dw4 b;
            for (int q = 0; q < 4; q++) { b.w[q] = halve4(x.w[q], cast.w[q], inv2, M); x.w[q] = addmod4(b.w[q], shift.w[q], M); }
            st_chunk(rep_view(J.b, L.reps, t), e, (int)ch, b);
        }
        if (J.out.p) st_chunk(J.out, e, (int)ch, x);
    }
}

// Where a finished ciphertext row goes.  DirectSink stores it dword by dword at its place in the table;
// the kernel for long rows stages rows in LDS instead and writes them out cooperatively.
struct DirectSink {
    uint32_t* row;
    DASH_HD void begin(uint8_t* table, uint64_t row_index, uint32_t pitch) { row = (uint32_t*)(table + row_index * pitch); }
    DASH_HD void put(int i, uint32_t w) { row[i] = w; }
};

// tag: the output modulus' compile-time description is chosen per job inside the kernel
struct PerJobMod {};

// garble: one lane per ciphertext row r = gate * p + a.  QD: description type of the output modulus
// (every job of a launch has the same output modulus), fixed at compile time for the hot moduli.
// keys(): the round keys.
template <class QD, class Tab, class Sink, class Keys>
DASH_HD void garble_body(const GateLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T, Sink& sink, uint32_t rep, Keys keys) {
    const GateJob& J = L.jobs[by];
    const LView Jin = rep_view(J.in, L.reps, rep), Jout = rep_view(J.out, L.reps, rep);
    uint8_t* const table = J.table + (int64_t)rep * L.reps.tables;
    const ModInfo Mp = ld_mod(L.mods, J.p), Mq = ld_mod(L.mods, J.q);
    // The block's first row is divided once (scalar unit; rows of a job are below 2^32); the lane's offset from it is small
    // enough for the 24-bit magic division.
    const uint32_t r0 = bx * kThreads;
    if ((uint64_t)bx * kThreads >= (uint64_t)J.n_elem * Mp.m) return;
    const uint32_t g0 = div_any(r0, Mp), off = r0 - g0 * Mp.m + tx;
    const uint32_t dg = div_m(off, Mp);
    const uint32_t g = g0 + dg, a = off - dg * Mp.m;
    if (g >= J.n_elem) return;

    // label of value a on the input wire: zero label + a * R_p (row a of the table of offset multiples)
    uint32_t colour = 0;
    U128 K = {{0, 0, 0, 0}};
    with_mod(Mp, [&](auto P) {
        const uint32_t* da = P.dtab + a * P.ndw;
        K = compress(P, [&](int i) { return addmod4(ld_dw(Jin, g, i), gload32(da + i), P); }, &colour);
    });
    U128 h = hash_block(K, J.elem_base + g, J.slot + rep * L.reps.slots, L.layer, keys(), T);

    // the output modulus: the kernel's compile-time description, or the run-time record (the instantiation for any
    // modulus, which also serves launches that mix output moduli; choosing a compile-time description per job inside
    // it, as eval_body does, was measured much slower on large launches: the kernel then needs the registers of its
    // largest case), or, QD = PerJobMod, that choice per job: for launches of few rows, where a lane's run time and
    // not the number of waves in flight decides)
    auto finish = [&](const auto& Q) {
        typedef std::decay_t<decltype(Q)> QT;
        if (J.mode == PAY_SHORT) {
            uint32_t v = mod_m(a + J.r[g] + mod_u128(h, Q), Q);
            *(uint32_t*)(table + ((size_t)g * Mp.m + colour) * 4) = v;
            return;
        }
        sink.begin(table, (uint64_t)g * Mp.m + colour, Q.ndw * 4);
        if (J.mode == PAY_EHALF) {
            uint32_t cf = mod_m(a + J.r[g], Q);
            cf = cf ? Q.m - cf : 0;                          // minus (a + r) * x0
            decompress(Q, h, [&](int i, uint32_t hd) {
                uint32_t pay = axpymod4(ld_dw(Jout, g, i), cf, ld_dw(J.x0, g, i), Q);
                sink.put(i, addmod4(pay, hd, Q));
            });
            return;
        }
        uint32_t f;
        if (J.mode == PAY_MULR) f = mod_m(a * J.r[g], Q);
        else f = J.phi[(size_t)g * J.phi_stride + a];
        const uint32_t* df = Q.dtab + f * Q.ndw;
        if constexpr (cmod_m<QT>::value != 0) {
            // payload first (its loads do not wait behind the row stores), then one pass over the hash digits
            uint32_t pay[QT::ndw];
#pragma unroll
            for (int i = 0; i < (int)QT::ndw; i++) pay[i] = addmod4(ld_dw(Jout, g, i), gload32(df + i), Q);
            decompress(Q, h, [&](int i, uint32_t hd) { sink.put(i, addmod4(pay[i], hd, Q)); });
        } else {
            decompress(Q, h, [&](int i, uint32_t hd) {
                sink.put(i, addmod4(addmod4(ld_dw(Jout, g, i), gload32(df + i), Q), hd, Q));
            });
        }
    };
    if constexpr (cmod_m<QD>::value != 0) finish(make_mod<QD>::from(Mq));
    else if constexpr (std::is_same<QD, PerJobMod>::value) with_mod(Mq, finish);
    else finish(Mq);
}

template <class QD, class Tab, class Sink>
DASH_HD void garble_body(const GateLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T, Sink& sink, uint32_t rep = 0) {
    garble_body<QD>(L, bx, by, tx, T, sink, rep, [&] { return (const uint32_t*)L.key.rk; });
}

// Garbler, a batch of gates of one input modulus and one function table (carry gates of the sign gadget): the lane keeps its value a.
// The rows of a batch, gate * m + a in order, are dealt to V waves in tiles of 64, and V tiles are a multiple of the input modulus m: a, with it
// the multiple of R_p that forms the label and the one of R_q that the row carries, stays the same from tile to tile and is held in
// registers, and so is the lane's place relative to the tile's first gate.  What is left per row is the label's addition and
// compression, the hash, and two packed additions.  keys(): the round keys; tick(): called once per tile.
struct ChainRows {
    const uint8_t *in, *out0, *phi;      // zero labels of the input and the output wires; function table
    int64_t in_cs, out_cs;
    uint8_t* table;
    uint64_t elem_base;
    uint32_t n, slot, layer;             // gates
};
struct NoTick { DASH_HD void operator()() const {} };
template <class MP, class QD, class Keys, class Tab, class Tick = NoTick>
DASH_HD void chain_garble_rows(const ChainRows& J, const MP& P, const QD& Q, uint32_t V, uint32_t t0, uint32_t lane, Keys keys, const Tab& T, Tick tick = Tick()) {
    constexpr uint32_t m = MP::m, pitch = QD::ndw * 4;
    constexpr int NP = (int)MP::ndw, NQ = (int)QD::ndw;
    const uint32_t n = J.n, tiles = (uint32_t)(((uint64_t)n * m + 63) / 64);
    if (t0 >= tiles) return;
    const uint32_t off = t0 * 64 % m + lane;                          // (rows of a batch are below 2^32)
    const uint32_t dg = off / m, a = off - dg * m, step = 64 * V / m;
    uint32_t da[NP], df[NQ];
    ld_dwords<NP>(P.dtab, a * (MP::ndw * 4), da);
    ld_dwords<NQ>(Q.dtab, J.phi[a] * pitch, df);
#pragma unroll
    for (int i = 0; i < NP; i++) da[i] = offset4(da[i], P);
#pragma unroll
    for (int i = 0; i < NQ; i++) df[i] = offset4(df[i], Q);
    const uint32_t row0 = dg * m;
    uint32_t gb = t0 * 64 / m, z[NP], o[NQ];                          // first gate of the tile
    // the lane's gate as an offset from gate b; past the end the last one (read, never stored)
    auto eo = [&](uint32_t b) { return 16 * (dg < n - b ? dg : n - 1 - b); };
    ld_label<NP>(J.in + (uint64_t)gb * 16, J.in_cs, eo(gb), z);
    for (uint32_t t = t0; t < tiles; t += V) {
        const uint32_t next = t + V < tiles ? gb + step : gb;
        tick();
        ld_label<NQ>(J.out0 + (uint64_t)gb * 16, J.out_cs, eo(gb), o);
        uint32_t colour;
        const U128 K = compress(P, [&](int i) { return addmod4_off(z[i], da[i], P); }, &colour);
        ld_label<NP>(J.in + (uint64_t)next * 16, J.in_cs, eo(next), z);
        schedule_fence();
        const U128 h = hash_block(K, J.elem_base + gb + dg, J.slot, J.layer, keys(), T);
#pragma unroll
        for (int i = 0; i < NQ; i++) o[i] = offset4(addmod4_off(o[i], df[i], Q), Q);
        uint8_t* rows = J.table + (uint64_t)gb * (m * pitch);
        const uint32_t ro = (row0 + colour) * pitch;
        if (dg < n - gb) decompress(Q, h, [&](int i, uint32_t hd) { st_row(rows, ro, i, addmod4_off(hd, o[i], Q)); });
        gb = next;
    }
}
// The same for the final gates (output modulus 2, rows of 128 bytes), in two steps.  A lane forms its row as 128 bits without the output
// wire's zero label; then the wave writes the tile's rows, 16 bytes a lane and eight lanes a row, and each lane spreads its 16 bits and puts the
// 16 digits of the zero label to them, so that nobody handles a row of 32 dwords.
struct BitsLane { uint32_t da[10], f, dg, row0; };                  // (labels of m_1 have at most ten dwords)
template <class MP>
DASH_HD BitsLane chain_bits_lane(const ChainRows& J, const MP& P, uint32_t t0, uint32_t lane) {
    static_assert(MP::ndw <= 10, "BitsLane");
    BitsLane B;
    const uint32_t off = t0 * 64 % MP::m + lane, a = off % MP::m;
    B.dg = off / MP::m; B.row0 = B.dg * MP::m;
    ld_dwords<(int)MP::ndw>(P.dtab, a * (MP::ndw * 4), B.da);
#pragma unroll
    for (int i = 0; i < (int)MP::ndw; i++) B.da[i] = offset4(B.da[i], P);
    B.f = 0u - (J.phi[a] & 1u);
    return B;
}
// z: zero label of the lane's gate gb + dg.  Bits of the row, and its index past the rows of gate gb
template <class MP, class Tab>
DASH_HD U128 chain_bits_row(const ChainRows& J, const MP& P, const U128& R2, const BitsLane& B, uint32_t gb, const uint32_t* z, const uint32_t* rk, const Tab& T, uint32_t& row) {
    uint32_t colour;
    const U128 K = compress(P, [&](int i) { return addmod4_off(z[i], B.da[i], P); }, &colour);
    const U128 h = hash_block(K, J.elem_base + gb + B.dg, J.slot, J.layer, rk, T);
    row = B.row0 + colour;
    return U128{{h.w[0] ^ (R2.w[0] & B.f), h.w[1] ^ (R2.w[1] & B.f), h.w[2] ^ (R2.w[2] & B.f), h.w[3] ^ (R2.w[3] & B.f)}};
}
// digits 16 part .. 16 part + 15 of the row with that index past the rows of gate gb: what the row adds to its bits, and the row's piece
// (stored if its gate is one of the batch's)
template <uint32_t m>
DASH_HD Dw4 chain_bits_label(const ChainRows& J, uint32_t gb, uint32_t row, uint32_t part) {
    const uint32_t dg = row / m, last = J.n - 1 - gb;
    return ld_dw4(J.out0 + (int64_t)part * J.out_cs + (uint64_t)gb * 16, (dg < last ? dg : last) * 16);
}
template <uint32_t m>
DASH_HD void chain_bits_store(const ChainRows& J, uint32_t gb, uint32_t row, uint32_t part, uint32_t bits16, Dw4 d) {
#pragma unroll
    for (int q = 0; q < 4; q++) d.w[q] ^= mul24((bits16 >> (4 * q)) & 0xfu, 0x00204081u) & kOnes;
    uint8_t* rows = J.table + (uint64_t)gb * (m * 128u);
    if (row / m < J.n - gb) {
#pragma unroll
        for (int q = 0; q < 4; q++) st_row(rows, row * 128 + part * 16, q, d.w[q]);
    }
}
// tiles of 64 rows after which a lane comes back to its value
DASH_HD uint32_t chain_quantum(uint32_t m) { uint32_t q = m; for (int i = 0; i < 6 && !(q & 1); i++) q /= 2; return q; }

// eval: one lane per gate
template <class QD, class Tab>
DASH_HD void eval_body(const GateLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T) {
    const GateJob& J = L.jobs[by];
    const ModInfo Mp = ld_mod(L.mods, J.p), Mq = ld_mod(L.mods, J.q);
    uint32_t g = bx * kThreads + tx;
    if (g >= J.n_elem) return;
    uint32_t colour = ld_dw(J.in, g, 0) & 0xffu;
    U128 K = {{0, 0, 0, 0}};
    with_mod(Mp, [&](auto P) { K = compress(P, [&](int i) { return ld_dw(J.in, g, i); }, &colour); });
    // (the output modulus as in garble_body; the row is named by the colour, digit 0 of the label: its loads are issued
    // before the hash, not after)
    auto finish = [&](const auto& Q) {
        typedef std::decay_t<decltype(Q)> QT;
        const uint32_t* row = (const uint32_t*)(J.table + ((size_t)g * Mp.m + colour) * (Q.ndw * 4));
        uint32_t rw[cmod_ndw<QT>::value];
        if constexpr (cmod_m<QT>::value != 0) {
#pragma unroll
            for (int i = 0; i < (int)QT::ndw; i++) rw[i] = row[i];
        }
        U128 h = hash_block(K, J.elem_base + g, J.slot, L.layer, L.key.rk, T);
        if constexpr (cmod_m<QT>::value != 0) {
            decompress(Q, h, [&](int i, uint32_t hd) { st_dw(J.out, g, i, submod4(rw[i], hd, Q)); });
        } else {
            decompress(Q, h, [&](int i, uint32_t hd) { st_dw(J.out, g, i, submod4(row[i], hd, Q)); });
        }
        for (int i = (int)Q.ndw; i < (int)Q.nchunk * 4; i++) st_dw(J.out, g, i, 0);
    };
    if constexpr (cmod_m<QD>::value != 0) finish(make_mod<QD>::from(Mq));
    else with_mod(Mq, finish);
}

// The same for launches that mix output moduli, all of them with compile-time descriptions: the hash stands between two dispatches on the
// output modulus (one copy of its code), the first of which sends the row's loads out.  (Rows of bits are loaded after the hash: 32
// dwords held over it would halve the waves per SIMD.)  J: a job of the launch.
struct EvalGate {
    const uint8_t *in, *table;       // label tensor and segment
    uint8_t* out;
    int64_t in_cs, out_cs;
    uint64_t elem_base;
    uint32_t n, p, q;
};
template <class Tab>
DASH_HD void eval_many_body(const EvalGate& J, const ModInfo* mods, uint32_t layer, const uint32_t* rk, uint32_t bx, uint32_t tx, const Tab& T) {
    const uint32_t g0 = bx * kThreads;
    if (g0 + tx >= J.n) return;
    const ModInfo Mp = ld_mod(mods, J.p), Mq = ld_mod(mods, J.q);
    const uint8_t *in = J.in + (uint64_t)g0 * 16, *rows = J.table + (uint64_t)g0 * (Mp.m * Mq.ndw * 4);     // of the tile
    uint8_t* out = J.out + (uint64_t)g0 * 16;
    const uint32_t eo = tx * 16;
    uint32_t colour = 0;
    U128 K = {{0, 0, 0, 0}};
    with_mod(Mp, [&](auto P) {
        typedef decltype(P) PT;
        if constexpr (cmod_m<PT>::value != 0) {
            uint32_t x[PT::ndw];
            ld_label<(int)PT::ndw>(in, J.in_cs, eo, x);
            K = compress(P, [&](int i) { return x[i]; }, &colour);
        }
    });
    const uint32_t row = (tx * Mp.m + colour) * (Mq.ndw * 4);
    constexpr int kMax = 21;                // dwords of the longest row but those of bits
    uint32_t rw[kMax];
    with_mod(Mq, [&](auto Q) {
        typedef decltype(Q) QT;
        if constexpr (cmod_m<QT>::value > 2) { static_assert(QT::ndw <= kMax, "row"); ld_dwords<(int)QT::ndw>(rows, row, rw); }
    });
    schedule_fence();
    const U128 h = hash_block(K, J.elem_base + g0 + tx, 0, layer, rk, T);
    with_mod(Mq, [&](auto Q) {
        typedef decltype(Q) QT;
        if constexpr (cmod_m<QT>::value == 2) {
#pragma unroll
            for (int ch = 0; ch < 8; ch++) {
                uint32_t r[4];
                ld_dwords<4>(rows, row + 16 * ch, r);
                Dw4 w;
#pragma unroll
                for (int q = 0; q < 4; q++) w.w[q] = r[q] ^ (mul24((h.w[ch >> 1] >> (16 * (ch & 1) + 4 * q)) & 0xfu, 0x00204081u) & kOnes);
                *(Dw4*)(out + (int64_t)ch * J.out_cs + eo) = w;
            }
        } else if constexpr (cmod_m<QT>::value != 0) {
            Dw4 w[QT::nchunk] = {};
            decompress(Q, h, [&](int i, uint32_t hd) { w[i >> 2].w[i & 3] = submod4(rw[i], hd, Q); });
#pragma unroll
            for (int ch = 0; ch < (int)QT::nchunk; ch++) *(Dw4*)(out + (int64_t)ch * J.out_cs + eo) = w[ch];
        }
    });
}

// ---- evaluator, carry chain of the sign gadget ------------------------------------------------
// One gate of the chain for element e: the input label comes dword by dword from in_dw, the output label
// goes dword by dword to out.
// QUAD: the four lanes of a quad work on the same element and share the AES (hash_block_quad).
template <bool QUAD = false, class MI, class MO, class Tab, class In, class Out>
DASH_HD void chain_gate(const ChainLaunch& L, const MI& Mi, const MO& Mo, uint32_t e, int j, In in_dw, Out out, const Tab& T, const QuadKey& Q = QuadKey{}) {
    uint32_t colour = in_dw(0) & 0xffu;       // the row's loads go out before the hash
    const uint32_t* row = (const uint32_t*)(L.table[j] + ((size_t)e * Mi.m + colour) * (Mo.ndw * 4));
    uint32_t rw[cmod_ndw<MO>::value];
    if constexpr (cmod_m<MO>::value != 0) {
#pragma unroll
        for (int i = 0; i < (int)MO::ndw; i++) rw[i] = row[i];
    }
    U128 K = compress(Mi, in_dw, &colour);
    U128 h = QUAD ? hash_block_quad<cmod_m<MO>::value != 0>(K, L.elem_base + e, L.slot[j], L.layer, Q, L.key.rk, T)
                  : hash_block(K, L.elem_base + e, L.slot[j], L.layer, L.key.rk, T);
    if constexpr (cmod_m<MO>::value != 0) {
        decompress(Mo, h, [&](int i, uint32_t hd) { out(i, submod4(rw[i], hd, Mo)); });
    } else {
        decompress(Mo, h, [&](int i, uint32_t hd) { out(i, submod4(row[i], hd, Mo)); });
    }
}

// dword i of the final gate's output: the sign bit wire, and (scaling gadget) the same wire plus a constant
DASH_HD void chain_out(const ChainLaunch& L, uint32_t e, int i, uint32_t w) {
    st_dw(L.bit, e, i, w);
    if (L.up.p) st_dw(L.up, e, i, L.up_coef ? addmod4(w, ld_dw(L.up_one, e, i), CMod<2, 128>{nullptr}) : w);
}

// Digit sets whose digits 2..n share one accumulation modulus (description MC) and whose first digit has
// description M1, both fixed at compile time: the carry label stays in registers from gate to gate.  The output
// wire has modulus 2 and 128 digits (the launcher takes the generic body for any other label length of modulus 2).
// QUAD (layers of few elements, where the chain of one lane is the run time): four neighbouring lanes per element; they
// do everything alike except the AES, which they share, and the stores, which the first of them does.
template <class MC, class M1, bool QUAD = false, class Tab>
DASH_HD void chain_eval_body(const ChainLaunch& L, uint32_t bx, uint32_t tx, const Tab& T) {
    const uint32_t lane = bx * kThreads + tx;
    const uint32_t e = QUAD ? lane >> 2 : lane;
    const bool writer = !QUAD || (lane & 3u) == 0;
    if (e >= L.n_elem) return;
    const QuadKey Q = QUAD ? quad_key(L.key.rk, lane & 3u) : QuadKey{};
    const MC Mc{nullptr};
    const M1 Mf{nullptr};
    const CMod<2, 128> M2{nullptr};
    uint32_t cw[MC::ndw], c1[M1::ndw];
#pragma unroll
    for (int i = 0; i < (int)MC::ndw; i++) cw[i] = 0;
    const int n = (int)L.n;
    // The digit sums do not depend on the chain: the sum of the next digit is fetched before the hash of the current
    // gate, so that its latency passes under the hash (a lane has nothing else to overlap it with).
    uint32_t sm[MC::ndw], s1[M1::ndw];
#pragma unroll
    for (int i = 0; i < (int)MC::ndw; i++) sm[i] = ld_dw(L.sum[n], e, i);
    for (int j = n; j >= 3; j--) {                  // carry out of digit j into digit j-1, same modulus
        uint32_t in[MC::ndw];
#pragma unroll
        for (int i = 0; i < (int)MC::ndw; i++) in[i] = addmod4(sm[i], cw[i], Mc);   // cw = 0 at j = n
#pragma unroll
        for (int i = 0; i < (int)MC::ndw; i++) sm[i] = ld_dw(L.sum[j - 1], e, i);
        chain_gate<QUAD>(L, Mc, Mc, e, j, [&](int i) { return in[i]; }, [&](int i, uint32_t w) { cw[i] = w; }, T, Q);
    }
    {                                               // digit 2 -> carry into digit 1 (modulus of the first digit)
        uint32_t in[MC::ndw];
#pragma unroll
        for (int i = 0; i < (int)MC::ndw; i++) in[i] = addmod4(sm[i], cw[i], Mc);
#pragma unroll
        for (int i = 0; i < (int)M1::ndw; i++) s1[i] = ld_dw(L.sum[1], e, i);
        chain_gate<QUAD>(L, Mc, Mf, e, 2, [&](int i) { return in[i]; }, [&](int i, uint32_t w) { c1[i] = w; }, T, Q);
    }
    {                                               // final gate: digit 1 -> the sign bit
        uint32_t in[M1::ndw];
#pragma unroll
        for (int i = 0; i < (int)M1::ndw; i++) in[i] = addmod4(s1[i], c1[i], Mf);
        Dw4 bits[8];                                // the 128 digits of the output wire: stored 16 bytes at a time
        chain_gate<QUAD>(L, Mf, M2, e, 1, [&](int i) { return in[i]; }, [&](int i, uint32_t w) { bits[i >> 2].w[i & 3] = w; }, T, Q);
        if (!writer) return;
#pragma unroll
        for (int ch = 0; ch < 8; ch++) st_chunk(L.bit, e, ch, bits[ch]);
        if (L.up.p) {
#pragma unroll
            for (int ch = 0; ch < 8; ch++) {
                if (L.up_coef) {
                    const Dw4 ow = ld_chunk(L.up_one, e, ch);
#pragma unroll
                    for (int q = 0; q < 4; q++) bits[ch].w[q] = addmod4(bits[ch].w[q], ow.w[q], M2);
                }
                st_chunk(L.up, e, ch, bits[ch]);
            }
        }
    }
}

// Any digit set, run-time constants: the carry label goes through its buffer in memory (written and read
// back by the same lane).
template <class Tab>
DASH_HD void chain_eval_generic_body(const ChainLaunch& L, uint32_t bx, uint32_t tx, const Tab& T) {
    const uint32_t e = bx * kThreads + tx;
    if (e >= L.n_elem) return;
    const int n = (int)L.n;
    for (int j = n; j >= 1; j--) {
        const ModInfo Mi = ld_mod(L.mods, L.m[j]);
        const bool has_carry = j < n;
        auto in_dw = [&](int i) {
            uint32_t w = ld_dw(L.sum[j], e, i);
            return has_carry ? addmod4(w, ld_dw(L.carry[j], e, i), Mi) : w;
        };
        if (j >= 2) {
            const ModInfo Mo = ld_mod(L.mods, L.m[j - 1]);
            chain_gate(L, Mi, Mo, e, j, in_dw, [&](int i, uint32_t w) { st_dw(L.carry[j - 1], e, i, w); }, T);
            for (int i = (int)Mo.ndw; i < (int)Mo.nchunk * 4; i++) st_dw(L.carry[j - 1], e, i, 0);
        } else if (ld_mod(L.mods, 2).lam == 128) {
            const CMod<2, 128> M2{nullptr};
            chain_gate(L, Mi, M2, e, 1, in_dw, [&](int i, uint32_t w) { chain_out(L, e, i, w); }, T);
        } else {                                // another label length of modulus 2: run-time constants
            const ModInfo M2 = ld_mod(L.mods, 2);
            chain_gate(L, Mi, M2, e, 1, in_dw, [&](int i, uint32_t w) { chain_out(L, e, i, w); }, T);
            for (int i = (int)M2.ndw; i < (int)M2.nchunk * 4; i++) chain_out(L, e, i, 0);
        }
    }
}

// ---- evaluator, digit gates of the sign gadget -------------------------------------------------
// The hashes of one label under the slots of its digit gates, one after the other: what they share (slot_hash_start) is
// formed at the first and again only where the slots' upper 24 bits change (the same for all lanes).
struct SlotHasher {
    const U128 K; const uint64_t elem; const uint32_t layer;
    SlotHash S; uint32_t hi = 0; bool started = false;
    DASH_HD SlotHasher(const U128& K_, uint64_t elem_, uint32_t layer_) : K(K_), elem(elem_), layer(layer_) {}
    template <class Tab> DASH_HD U128 get(uint32_t slot, const uint32_t* rk, const Tab& T) {
        if (!started || (slot >> 8) != hi) { S = slot_hash_start(K, elem, slot, layer, rk, T); hi = slot >> 8; started = true; }
        return slot_hash(S, slot, rk, T);
    }
};
// gate (residue, digit j) of element e: hash(slot) gives the hash of its input label, colour is the label's colour (it names the
// row, whose loads go out before the hash)
template <class MO, class Hash>
DASH_HD void digit_gate(const DigitsLaunch& L, const DigitsRes& R, const MO& Mo, uint32_t colour, uint32_t e, int j, Hash hash) {
    const uint8_t* seg = R.table + (size_t)L.n_elem * R.p * L.row_prefix[j];
    const uint32_t* row = (const uint32_t*)(seg + ((size_t)e * R.p + colour) * (Mo.ndw * 4));
    const LView out{R.out + L.out_prefix[j], L.out_cs, 16u};
    const uint32_t slot = R.slot0 + (uint32_t)(j - 1);
    if constexpr (cmod_m<MO>::value != 0) {
        uint32_t rw[MO::ndw];
#pragma unroll
        for (int i = 0; i < (int)MO::ndw; i++) rw[i] = row[i];
        const U128 h = hash(slot);
        Dw4 w[MO::nchunk] = {};
        decompress(Mo, h, [&](int i, uint32_t hd) { w[i >> 2].w[i & 3] = submod4(rw[i], hd, Mo); });
#pragma unroll
        for (int ch = 0; ch < (int)MO::nchunk; ch++) st_chunk(out, e, ch, w[ch]);
    } else {
        const U128 h = hash(slot);
        decompress(Mo, h, [&](int i, uint32_t hd) { st_dw(out, e, i, submod4(row[i], hd, Mo)); });
        for (int i = (int)Mo.ndw; i < (int)Mo.nchunk * 4; i++) st_dw(out, e, i, 0);
    }
}
// the same gate with its output label handed to put(dword index, packed digits) instead of stored (compile-time moduli)
template <class MO, class Tab, class Put>
DASH_HD void digit_gate_to(const DigitsLaunch& L, const DigitsRes& R, const MO& Mo, const U128& K, uint32_t colour, uint32_t e, int j, const Tab& T,
                           Put put) {
    const uint8_t* seg = R.table + (size_t)L.n_elem * R.p * L.row_prefix[j];
    const uint32_t* row = (const uint32_t*)(seg + ((size_t)e * R.p + colour) * (MO::ndw * 4));
    uint32_t rw[MO::ndw];
#pragma unroll
    for (int i = 0; i < (int)MO::ndw; i++) rw[i] = row[i];
    U128 h = hash_block(K, L.elem_base + e, R.slot0 + (uint32_t)(j - 1), L.layer, L.key.rk, T);
    decompress(Mo, h, [&](int i, uint32_t hd) { put(i, submod4(rw[i], hd, Mo)); });
}

// MC, M1: descriptions of the accumulation moduli of digits 2..n and of digit 1 (compile time), or ModInfo for
// both (any digit set: then every digit's constants are read from the table of moduli)
template <class MC, class M1, class Tab>
DASH_HD void digits_eval_body(const DigitsLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T) {
    const DigitsRes& R = L.res[by];
    const uint32_t e = bx * kThreads + tx;
    if (e >= L.n_elem) return;
    const ModInfo Mp = ld_mod(L.mods, R.p);
    uint32_t colour = 0;
    U128 K = {{0, 0, 0, 0}};
    with_mod(Mp, [&](auto P) { K = compress(P, [&](int i) { return ld_dw(R.in, e, i); }, &colour); });
    SlotHasher H(K, L.elem_base + e, L.layer);
    auto hash = [&](uint32_t slot) { return H.get(slot, L.key.rk, T); };
    if constexpr (cmod_m<MC>::value != 0) {
        digit_gate(L, R, M1{nullptr}, colour, e, 1, hash);
        for (int j = 2; j <= (int)L.n; j++) digit_gate(L, R, MC{nullptr}, colour, e, j, hash);
    } else {
        for (int j = 1; j <= (int)L.n; j++) {
            const ModInfo Mo = ld_mod(L.mods, L.m[j]);      // a copy in registers: through the reference every use is a load
            digit_gate(L, R, Mo, colour, e, j, hash);
        }
    }
}

// The same gates with one lane per (element, residue, digit j): every lane compresses the label again, but a lane's
// chain is one hash instead of n.  For gadgets over few elements, whose time is the length of that chain.
template <class MC, class M1, class Tab>
DASH_HD void digits_eval_wide_body(const DigitsLaunch& L, uint32_t bx, uint32_t by, uint32_t j, uint32_t tx, const Tab& T) {
    const DigitsRes& R = L.res[by];
    const uint32_t e = bx * kThreads + tx;
    if (e >= L.n_elem || j < 1 || j > L.n) return;
    const ModInfo Mp = ld_mod(L.mods, R.p);
    uint32_t colour = 0;
    U128 K = {{0, 0, 0, 0}};
    with_mod(Mp, [&](auto P) { K = compress(P, [&](int i) { return ld_dw(R.in, e, i); }, &colour); });
    auto hash = [&](uint32_t slot) { return hash_block(K, L.elem_base + e, slot, L.layer, L.key.rk, T); };
    if constexpr (cmod_m<MC>::value != 0) {
        if (j == 1) digit_gate(L, R, M1{nullptr}, colour, e, 1, hash);
        else digit_gate(L, R, MC{nullptr}, colour, e, (int)j, hash);
    } else {
        const ModInfo Mo = ld_mod(L.mods, L.m[j]);
        digit_gate(L, R, Mo, colour, e, (int)j, hash);
    }
}

// ---- garbler, digit gates of the sign gadget ---------------------------------------------------
// One lane per (element g, value a) of a residue: the label of a is formed and compressed once, then one
// ciphertext row per digit: rows[colour] = out0 + phi_j(a) R_{m_j} + H_{m_j}(label, slot_j).
DASH_HD void digit_row(const DigitsLaunch& L, const DigitsRes& R, const ModInfo& Mo, const U128& h, uint32_t f, uint32_t colour, uint32_t g, int j, uint32_t rep) {
    uint8_t* seg = R.table + (int64_t)rep * L.reps.tables + (size_t)L.n_elem * R.p * L.row_prefix[j];
    uint32_t* row = (uint32_t*)(seg + ((size_t)g * R.p + colour) * (Mo.ndw * 4));
    const LView out0{R.out + (int64_t)rep * L.reps.wires + L.out_prefix[j], L.out_cs, 16u};
    const uint32_t* df = Mo.dtab + f * Mo.ndw;
    decompress(Mo, h, [&](int i, uint32_t hd) { row[i] = addmod4(addmod4(ld_dw(out0, g, i), gload32(df + i), Mo), hd, Mo); });
}
// Compile-time moduli: the rows of digits j0..j1 (j0 = 1 or 2 and up) of one (element, value a).  Everything but the hash costs as little as can be, the
// kernel being bound by vector issue: the tile's first element is in the scalar base addresses and the lane's part in 32-bit offsets
// that serve every digit; what a row adds to its hash is fetched before the hash.
template <class MO, class Tab, class Tick>
DASH_HD void digit_rows(const DigitsLaunch& L, const uint8_t* phi, uint32_t p, const uint8_t* out0, int64_t out_step, uint8_t* seg, int64_t seg_step, const MO& Mo,
                        SlotHash& S, uint32_t& hi, uint32_t& slot, int count, uint32_t a, uint32_t eo, uint32_t row, const Tab& T, Tick tick) {
    constexpr int N = (int)MO::ndw;
    const uint32_t ro = row * (MO::ndw * 4);
    uint32_t f = phi[a];
    for (int j = 0; j < count; j++) {
        uint32_t pay[N], o[N];
        tick();
        ld_label<N>(out0, L.out_cs, eo, o);
        ld_dwords<N>(Mo.dtab, f * (MO::ndw * 4), pay);
        phi += p;
        if (j + 1 < count) f = phi[a];
        schedule_fence();
        if ((slot & ~0xffu) != hi) {                // another upper part of the slot: what the hashes share is formed again
            S.x[2] ^= hi ^ (slot & ~0xffu);
            hi = slot & ~0xffu;
            S = slot_hash_start(S.x, L.key.rk, T);
        }
        const U128 h = slot_hash(S, slot, L.key.rk, T);
        slot++;
#pragma unroll
        for (int i = 0; i < N; i++) pay[i] = offset4(addmod4(o[i], pay[i], Mo), Mo);
        decompress(Mo, h, [&](int i, uint32_t hd) { st_row(seg, ro, i, addmod4_off(hd, pay[i], Mo)); });
        out0 += out_step; seg += seg_step;
    }
}
// j0 = 0: all n digits of the lane's (element, value); j0 = 1..n: digit j0 only (gadgets over few elements: a lane per
// row, a chain of one hash).  tick(): called once per digit (of compile-time moduli)
template <class MC, class M1, class Tab, class Tick = NoTick>
DASH_HD void digits_garble_body(const DigitsLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T, uint32_t j0 = 0, uint32_t rep = 0, Tick tick = Tick()) {
    const DigitsRes& R = L.res[by];
    const LView in = rep_view(R.in, L.reps, rep);
    const uint32_t slot0 = R.slot0 + rep * L.reps.slots;
    const ModInfo Mp = ld_mod(L.mods, R.p);
    const uint32_t r0 = bx * kThreads;
    if ((uint64_t)bx * kThreads >= (uint64_t)L.n_elem * Mp.m) return;
    const uint32_t g0 = div_any(r0, Mp), off = r0 - g0 * Mp.m + tx;
    const uint32_t dg = div_m(off, Mp);
    const uint32_t g = g0 + dg, a = off - dg * Mp.m;
    if (g >= L.n_elem) return;
    uint32_t colour = 0;
    U128 K = {{0, 0, 0, 0}};
    with_mod(Mp, [&](auto P) {
        const uint32_t* da = P.dtab + a * P.ndw;
        K = compress(P, [&](int i) { return addmod4(ld_dw(in, g, i), gload32(da + i), P); }, &colour);
    });
    const int jlo = j0 ? (int)j0 : 1, jhi = j0 ? (int)j0 : (int)L.n;
    if constexpr (cmod_m<MC>::value != 0) {
        const uint64_t elem = L.elem_base + g;
        const uint32_t s0 = slot0 + (uint32_t)(jlo - 1);
        const uint32_t x[4] = {K.w[0] ^ (uint32_t)elem, K.w[1] ^ (uint32_t)(elem >> 32), K.w[2] ^ (s0 & ~0xffu), K.w[3] ^ (L.layer & 0xffffu)};
        SlotHash S = slot_hash_start(x, L.key.rk, T);
        uint32_t slot = s0, hi = s0 & ~0xffu;
        const uint32_t eo = dg * 16, row = dg * Mp.m + colour;
        uint8_t* seg = R.table + (int64_t)rep * L.reps.tables;
        const uint8_t* out0 = R.out + (int64_t)rep * L.reps.wires + (uint64_t)g0 * 16;
        const int64_t rows = (int64_t)L.n_elem * Mp.m, before = (int64_t)g0 * Mp.m;       // of a segment; before the tile's first element
        int j = jlo;
        if (j == 1) {
            const M1 Mf{ld_mod(L.mods, L.m[1]).dtab};
            digit_rows(L, R.phi, R.p, out0, 0, seg + before * (int64_t)(M1::ndw * 4), 0, Mf, S, hi, slot, 1, a, eo, row, T, tick);
            j = 2;
        }
        if (j <= jhi) {
            const MC Mc{ld_mod(L.mods, L.m[2]).dtab};
            const int64_t step = rows * (int64_t)(MC::ndw * 4);
            digit_rows(L, R.phi + (uint32_t)(j - 1) * R.p, R.p, out0 + L.out_prefix[j], (int64_t)(L.out_prefix[j < (int)L.n ? j + 1 : j] - L.out_prefix[j]),
                       seg + rows * (int64_t)(M1::ndw * 4) + (j - 2) * step + before * (int64_t)(MC::ndw * 4), step, Mc, S, hi, slot, jhi - j + 1, a, eo, row, T, tick);
        }
        return;
    }
    SlotHasher H(K, L.elem_base + g, L.layer);
    for (int j = jlo; j <= jhi; j++) {
        const uint32_t f = R.phi[(size_t)(j - 1) * R.p + a];
        const U128 h = H.get(slot0 + (uint32_t)(j - 1), L.key.rk, T);
        const ModInfo Mo = ld_mod(L.mods, L.m[j]);      // a copy in registers: through the reference every use is a load
        digit_row(L, R, Mo, h, f, colour, g, j, rep);
    }
}

// Garbler, gates on ONE wire of modulus 2 (128 digits): the casts of the scaling gadget, the evaluator's halves and known inputs of the half gates.
// A lane has (element, value a): it packs and forms the label of a once, and the hashes of its jobs j0 .. j1 - 1, whose slots are
// neighbours, share their first two rounds.  The jobs have compile-time output moduli, labels of 16-byte elements, and in, n_elem and elem_base
// in common; the hash stands between two dispatches on the output modulus, the first of which sends the loads of the output wire's label out.
// R2: the offset label of modulus 2.  keys(): the round keys; tick(): called once per job.  Half: the jobs are PAY_EHALF and PAY_SHORT, else
// PAY_PHI.
template <bool Half, class Launch, class Tab, class Keys, class Tick = NoTick>
DASH_HD void bit_garble_body(const Launch& L, uint32_t tile, uint32_t rep, uint32_t j0, uint32_t j1, uint32_t tx, const U128& R2, const Tab& T, Keys keys, Tick tick = Tick()) {
    constexpr int kMax = 12;                // labels of more dwords (moduli 2, 3 and 5) are loaded after the hash: registers
    const uint32_t n = L.jobs[j0].n_elem, e0 = tile * (kThreads / 2), e = e0 + (tx >> 1), a = tx & 1u, eo = (tx >> 1) * 16;
    if (e >= n) return;
    const int64_t wires = (int64_t)rep * L.reps.wires;
    const uint64_t elem = L.jobs[j0].elem_base + e;
    const uint8_t* in = L.jobs[j0].in.p + wires + (uint64_t)e0 * 16;
    const int64_t in_cs = L.jobs[j0].in.cs;
    U128 K;
#pragma unroll
    for (int c = 0; c < 4; c++) {
        uint32_t w = 0;
#pragma unroll
        for (int ch = 0; ch < 2; ch++) {
            const Dw4 d = ld_dw4(in + (2 * c + ch) * in_cs, eo);
#pragma unroll
            for (int q = 0; q < 4; q++) w |= dot4(d.w[q], 0x08040201u) << (16 * ch + 4 * q);
        }
        K.w[c] = w ^ (R2.w[c] & (0u - a));
    }
    const uint32_t row = (tx & ~1u) | (K.w[0] & 1u);                     // past the tile's first row
    uint32_t hi = L.jobs[j0].slot + rep * L.reps.slots & ~0xffu;
    const uint32_t x[4] = {K.w[0] ^ (uint32_t)elem, K.w[1] ^ (uint32_t)(elem >> 32), K.w[2] ^ hi, K.w[3] ^ (L.layer & 0xffffu)};
    SlotHash S = slot_hash_start(x, keys(), T);
    for (uint32_t j = j0; j < j1; j++) {
        const auto& J = L.jobs[j];
        const uint32_t slot = J.slot + rep * L.reps.slots;
        const bool digit = Half && J.mode == PAY_SHORT;                  // one digit and no output label
        tick();
        uint32_t o[kMax], r = 0;
        if (Half) r = J.r[e];
        if (!digit) with_mod(ld_mod(L.mods, J.q), [&](auto Q) {
            typedef decltype(Q) QT;
            if constexpr (cmod_m<QT>::value != 0) { if constexpr (QT::ndw <= kMax) ld_label<(int)QT::ndw>(J.out.p + wires + (uint64_t)e0 * 16, J.out.cs, eo, o); }
        });
        schedule_fence();
        if ((slot & ~0xffu) != hi) {
            S.x[2] ^= hi ^ (slot & ~0xffu);
            hi = slot & ~0xffu;
            S = slot_hash_start(S.x, keys(), T);
        }
        const U128 h = slot_hash(S, slot, keys(), T);
        const auto& A = L.jobs[opaque(j)];                               // (J, read again: its fields don't stay in registers over the hash)
        with_mod(ld_mod(L.mods, A.q), [&](auto Q) {
            typedef decltype(Q) QT;
            if constexpr (cmod_m<QT>::value != 0) {
                constexpr uint32_t m = QT::m, pitch = QT::ndw * 4;
                uint8_t* const table = A.table + (int64_t)rep * L.reps.tables;
                const uint8_t* const out0 = A.out.p + wires + (uint64_t)e0 * 16;
                const int64_t out_cs = A.out.cs;
                if (digit) { st_row(table + (uint64_t)e0 * 8, row * 4, 0, mod_m(a + r + mod_u128(h, Q), Q)); return; }
                uint8_t* const rows = table + (uint64_t)e0 * (2 * pitch);
                // PAY_PHI: phi(a) R_q, its two values the same in all lanes; PAY_EHALF: - (a + r) x0
                const uint32_t f0 = Half ? 0u : A.phi[0], f1 = Half ? 0u : A.phi[1], s = mod_m(a + r, Q), cf = s ? m - s : 0u;
                const uint32_t *df0 = Q.dtab + f0 * QT::ndw, *df1 = Q.dtab + f1 * QT::ndw;
                const uint8_t* const x0 = Half ? A.x0.p + (uint64_t)e0 * 16 : nullptr;
                auto payload = [&](int i, uint32_t z, uint32_t xd) { return Half ? axpymod4(z, cf, xd, Q) : addmod4(z, a ? ld_const(df1 + i) : ld_const(df0 + i), Q); };
                if constexpr (m == 2) {
#pragma unroll
                    for (int ch = 0; ch < 8; ch++) {
                        const Dw4 d = ld_dw4(out0 + (int64_t)ch * out_cs, eo);
                        Dw4 xd = {};
                        if (Half) xd = ld_dw4(x0 + (int64_t)ch * A.x0.cs, eo);
#pragma unroll
                        for (int q = 0; q < 4; q++)
                            st_row(rows, row * pitch, 4 * ch + q, payload(4 * ch + q, d.w[q], xd.w[q]) ^ (mul24((h.w[ch >> 1] >> (16 * (ch & 1) + 4 * q)) & 0xfu, 0x00204081u) & kOnes));
                    }
                } else {
                    uint32_t z[QT::ndw], xd[QT::ndw] = {};
                    if constexpr (QT::ndw <= kMax) {
#pragma unroll
                        for (int i = 0; i < (int)QT::ndw; i++) z[i] = o[i];
                    } else ld_label<(int)QT::ndw>(out0, out_cs, eo, z);
                    if (Half) ld_label<(int)QT::ndw>(x0, A.x0.cs, eo, xd);
#pragma unroll
                    for (int i = 0; i < (int)QT::ndw; i++) z[i] = payload(i, z[i], xd[i]);
                    decompress(Q, h, [&](int i, uint32_t hd) { st_row(rows, row * pitch, i, addmod4(hd, z[i], Q)); });
                }
            }
        });
    }
}

// evaluator, scaling gadget: cast = rows[colour(y)] - H_p(y) (two-row gate Z_2 -> Z_p, identity function), then
// b = (x + addc * one - cast) * 2^-1 mod p.  The cast label itself is not stored.
// compile-time label length: b of element e in registers (xw: its chunks), 16-byte loads
template <class PD>
DASH_HD void cast_halve_regs(const CastJob& J, const PD& P, uint32_t e, uint32_t colour, const U128& h, Dw4* xw) {
    constexpr int ndw = (int)PD::ndw, nch = (int)PD::nchunk;
    const uint32_t inv2 = (J.p + 1) / 2;
    const uint32_t* row = (const uint32_t*)(J.table + ((size_t)e * 2 + colour) * (P.ndw * 4));
    uint32_t rw[ndw];
#pragma unroll
    for (int i = 0; i < ndw; i++) rw[i] = row[i];
#pragma unroll
    for (int ch = 0; ch < nch; ch++) xw[ch] = ld_chunk(J.x, e, ch);
    if (J.addc) {
#pragma unroll
        for (int ch = 0; ch < nch; ch++) {
            const Dw4 ow = ld_chunk(J.one, e, ch);
#pragma unroll
            for (int q = 0; q < 4; q++) xw[ch].w[q] = J.addc == 1 ? addmod4(xw[ch].w[q], ow.w[q], P) : axpymod4(xw[ch].w[q], J.addc, ow.w[q], P);
        }
    }
    decompress(P, h, [&](int i, uint32_t hd) { xw[i >> 2].w[i & 3] = halve4(xw[i >> 2].w[i & 3], submod4(rw[i], hd, P), inv2, P); });
#pragma unroll
    for (int i = ndw; i < nch * 4; i++) xw[i >> 2].w[i & 3] = 0;
}
template <class Tab>
DASH_HD void cast_halve_body(const CastLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T) {
    const CastJob& J = L.jobs[by];
    const uint32_t e = bx * kThreads + tx;
    if (e >= L.n_elem) return;
    const ModInfo Mp = ld_mod(L.mods, J.p);
    uint32_t colour = 0;
    U128 K = compress_mod2(L.mods, [&](int i) { return ld_dw(L.y, e, i); }, &colour);
    U128 h = hash_block(K, L.elem_base + e, J.slot, L.layer, L.key.rk, T);
    const uint32_t inv2 = (J.p + 1) / 2;
    with_mod(Mp, [&](auto P) {
        typedef decltype(P) PD;
        if constexpr (cmod_m<PD>::value != 0) {
            Dw4 xw[PD::nchunk];
            cast_halve_regs(J, P, e, colour, h, xw);
#pragma unroll
            for (int ch = 0; ch < (int)PD::nchunk; ch++) st_chunk(J.out, e, ch, xw[ch]);
        } else {
            const uint32_t* row = (const uint32_t*)(J.table + ((size_t)e * 2 + colour) * (P.ndw * 4));
            decompress(P, h, [&](int i, uint32_t hd) {
                const uint32_t cast = submod4(row[i], hd, P);
                uint32_t x = ld_dw(J.x, e, i);
                if (J.addc) x = J.addc == 1 ? addmod4(x, ld_dw(J.one, e, i), P) : axpymod4(x, J.addc, ld_dw(J.one, e, i), P);
                st_dw(J.out, e, i, halve4(x, cast, inv2, P));
            });
            for (int i = (int)P.ndw; i < (int)P.nchunk * 4; i++) st_dw(J.out, e, i, 0);
        }
    });
}

// The cast step and ONE digit gate per lane: lane (element, odd prime, digit j) forms b as above (the lanes of
// digit 1 store it), compresses it from its registers and evaluates digit gate j: a chain of two hashes, for
// gadgets over few elements.  Only for primes with a compile-time description (the launcher checks).
template <class MC, class M1, class Tab>
DASH_HD void cast_digit_wide_body(const CastLaunch& C, const DigitsLaunch& L, uint32_t bx, uint32_t by, uint32_t j, uint32_t tx, const Tab& T) {
    const CastJob& J = C.jobs[by];
    const DigitsRes& R = L.res[by];
    const uint32_t e = bx * kThreads + tx;
    if (e >= L.n_elem || j < 1 || j > L.n) return;
    const ModInfo Mp = ld_mod(C.mods, J.p);
    uint32_t colour = 0;
    U128 K2 = compress_mod2(C.mods, [&](int i) { return ld_dw(C.y, e, i); }, &colour);
    U128 h = hash_block(K2, C.elem_base + e, J.slot, C.layer, C.key.rk, T);
    with_mod(Mp, [&](auto P) {
        typedef decltype(P) PD;
        if constexpr (cmod_m<PD>::value != 0) {
            Dw4 xw[PD::nchunk];
            cast_halve_regs(J, P, e, colour, h, xw);
            if (j == 1) {
#pragma unroll
                for (int ch = 0; ch < (int)PD::nchunk; ch++) st_chunk(J.out, e, ch, xw[ch]);
            }
            uint32_t cb = 0;
            const U128 K = compress(P, [&](int i) { return xw[i >> 2].w[i & 3]; }, &cb);
            auto hash = [&](uint32_t slot) { return hash_block(K, L.elem_base + e, slot, L.layer, L.key.rk, T); };
            if constexpr (cmod_m<MC>::value != 0) {
                if (j == 1) digit_gate(L, R, M1{nullptr}, cb, e, 1, hash);
                else digit_gate(L, R, MC{nullptr}, cb, e, (int)j, hash);
            } else {
                const ModInfo Mo = ld_mod(L.mods, L.m[j]);
                digit_gate(L, R, Mo, cb, e, (int)j, hash);
            }
        }
    });
}

// ---- evaluator, few elements: digit gates that add up their outputs --------------------------
// A block takes 64 elements and one digit j; wave w of it takes residue w.  Every lane evaluates its digit gate (the
// scaling gadget's lanes do the cast step first, as in cast_digit_wide_body) and adds the output label into the block's
// accumulator, two digits per 32-bit word in 16-bit fields (phase 1); after a barrier the first wave reduces the sums
// mod m_j and stores the wire S_j (phase 2).  The digit wires themselves are not stored, and the launch that added them
// up is not needed.  Digit sets with compile-time moduli only.
constexpr int kSumDw = 10;                  // dwords per label of the longest such modulus (39 digits)
constexpr int kSumElems = 64;
DASH_HD void sum_add(uint32_t* a, uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    atomicAdd(a, v);
#else
    *a += v;
#endif
}
struct NoCast {};       // in place of the CastLaunch: the digit gates of a plain sign gadget
template <class MC, class M1, class CastT, class Tab>
DASH_HD void digits_sum_phase1(const CastT& C, const DigitsLaunch& L, uint32_t bx, uint32_t by, uint32_t j, uint32_t el, const Tab& T,
                               uint32_t* acc) {
    static_assert(MC::ndw <= kSumDw && M1::ndw <= kSumDw, "accumulator rows");
    const DigitsRes& R = L.res[by];
    const uint32_t e = bx * kSumElems + el;
    if (e >= L.n_elem || j < 1 || j > L.n) return;
    const ModInfo Mp = ld_mod(L.mods, R.p);
    uint32_t colour = 0;
    U128 K = {{0, 0, 0, 0}};
    if constexpr (std::is_same<CastT, CastLaunch>::value) {        // scaling gadget: b of this residue first (stored by the lanes of digit 1)
        const CastJob& J = C.jobs[by];
        uint32_t c2 = 0;
        const U128 K2 = compress_mod2(C.mods, [&](int i) { return ld_dw(C.y, e, i); }, &c2);
        const U128 h = hash_block(K2, C.elem_base + e, J.slot, C.layer, C.key.rk, T);
        with_mod(Mp, [&](auto P) {
            typedef decltype(P) PD;
            if constexpr (cmod_m<PD>::value != 0) {
                Dw4 xw[PD::nchunk];
                cast_halve_regs(J, P, e, c2, h, xw);
                if (j == 1) {
#pragma unroll
                    for (int ch = 0; ch < (int)PD::nchunk; ch++) st_chunk(J.out, e, ch, xw[ch]);
                }
                K = compress(P, [&](int i) { return xw[i >> 2].w[i & 3]; }, &colour);
            }
        });
    } else {
        with_mod(Mp, [&](auto P) { K = compress(P, [&](int i) { return ld_dw(R.in, e, i); }, &colour); });
    }
    uint32_t* row = acc + (size_t)el * (kSumDw * 2);
    auto put = [&](int i, uint32_t w) {
        sum_add(row + 2 * i, w & 0x00ff00ffu);
        sum_add(row + 2 * i + 1, (w >> 8) & 0x00ff00ffu);
    };
    if (j == 1) digit_gate_to(L, R, M1{nullptr}, K, colour, e, 1, T, put);
    else digit_gate_to(L, R, MC{nullptr}, K, colour, e, (int)j, T, put);
}
template <class MO>
DASH_HD void digits_sum_store(const DigitsLaunch& L, const MO& Mo, uint32_t e, uint32_t j, const uint32_t* row) {
    const LView out{L.sum1 + L.sum_prefix[j], L.out_cs, 16u};
#pragma unroll
    for (int ch = 0; ch < (int)MO::nchunk; ch++) {
        Dw4 z;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int i = 4 * ch + q;
            uint32_t w = 0;
            if (i < (int)MO::ndw) {      // fields below 16 * 255 < 2^24
                const uint32_t ev = row[2 * i], od = row[2 * i + 1];
                w = mod_m(ev & 0xffffu, Mo) | (mod_m(ev >> 16, Mo) << 16) | (mod_m(od & 0xffffu, Mo) << 8) | (mod_m(od >> 16, Mo) << 24);
            }
            z.w[q] = w;
        }
        st_chunk(out, e, ch, z);
    }
}
template <class MC, class M1>
DASH_HD void digits_sum_phase2(const DigitsLaunch& L, uint32_t bx, uint32_t j, uint32_t el, const uint32_t* acc) {
    const uint32_t e = bx * kSumElems + el;
    if (e >= L.n_elem || j < 1 || j > L.n) return;
    const uint32_t* row = acc + (size_t)el * (kSumDw * 2);
    if (j == 1) digits_sum_store(L, M1{nullptr}, e, j, row);
    else digits_sum_store(L, MC{nullptr}, e, j, row);
}

// evaluator side of the mixed-modulus half gate: z = V + beta * x - U
template <class Tab>
DASH_HD void hg_finish_body(const HgLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T) {
    const HgJob& J = L.jobs[by];
    const ModInfo Mp = ld_mod(L.mods, J.p);
    uint32_t e = bx * kThreads + tx;
    if (e >= L.n_elem) return;
    uint32_t colour = 0;
    U128 K = compress_mod2(L.mods, [&](int i) { return ld_dw(J.y, e, i); }, &colour);
    U128 h = hash_block(K, L.elem_base + e, J.slot, L.layer, L.key.rk, T);
    uint32_t s = *(const uint32_t*)(J.S + ((size_t)e * 2 + colour) * 4);
    uint32_t beta = mod_m(s + Mp.m - mod_u128(h, Mp), Mp);
    with_mod(Mp, [&](auto P) {
        typedef decltype(P) PD;
        if constexpr (cmod_m<PD>::value != 0) {
            // compile-time label length: all loads first, 16 bytes each, then the arithmetic in registers
            constexpr int nch = (int)PD::nchunk;
            Dw4 v[nch], x[nch], u[nch];
#pragma unroll
            for (int ch = 0; ch < nch; ch++) { v[ch] = ld_chunk(J.V, e, ch); x[ch] = ld_chunk(J.x, e, ch); u[ch] = ld_chunk(J.U, e, ch); }
#pragma unroll
            for (int ch = 0; ch < nch; ch++) {
#pragma unroll
                for (int q = 0; q < 4; q++) v[ch].w[q] = submod4(axpymod4(v[ch].w[q], beta, x[ch].w[q], P), u[ch].w[q], P);
                st_chunk(J.z, e, ch, v[ch]);
            }
        } else {
            for (int i = 0; i < (int)P.nchunk * 4; i++) {
                uint32_t v = axpymod4(ld_dw(J.V, e, i), beta, ld_dw(J.x, e, i), P);
                st_dw(J.z, e, i, submod4(v, ld_dw(J.U, e, i), P));
            }
        }
    });
}

// The whole evaluator side of the mixed-modulus half gate (Appendix) for layers of few elements, where three dependent
// launches cost more than their work: the four lanes of a quad take one (element, prime).  Lane 0 evaluates the garbler
// half (U, from the label of x), lane 1 the evaluator half (V, from the sign bit's label), lane 2 the row that carries
// beta: three hashes side by side; lane 0 then collects V and beta from its neighbours and stores z = V + beta x - U.
// Primes with compile-time descriptions only (the launcher checks).  On the host a caller with role 0 works through
// the three roles itself.
template <class Tab>
DASH_HD void hg_eval_quad_body(const HgLaunch& L, uint32_t bx, uint32_t by, uint32_t tx, const Tab& T) {
    const HgJob& J = L.jobs[by];
    const ModInfo Mp = ld_mod(L.mods, J.p);
    const uint32_t lane = bx * kThreads + tx, e = lane >> 2, c = lane & 3u;
    if (e >= L.n_elem) return;
    with_mod(Mp, [&](auto P) {
        typedef decltype(P) PD;
        if constexpr (cmod_m<PD>::value != 0) {
            constexpr int ndw = (int)PD::ndw, nch = (int)PD::nchunk;
            Dw4 x[nch];
            // one role: w = the gate's output label (roles 0 and 1), beta (role 2; role 3 repeats it and is not used)
            auto run_role = [&](uint32_t role, uint32_t* w, uint32_t& beta) {
                uint32_t colour = 0;
                U128 K;
                if (role == 0) {
#pragma unroll
                    for (int ch = 0; ch < nch; ch++) x[ch] = ld_chunk(J.x, e, ch);
                    K = compress(P, [&](int i) { return x[i >> 2].w[i & 3]; }, &colour);
                } else {
                    K = compress_mod2(L.mods, [&](int i) { return ld_dw(J.y, e, i); }, &colour);
                }
                const uint32_t rows = role == 0 ? Mp.m : 2u;
                const uint8_t* table = role == 0 ? J.G : J.Eh;
                uint32_t rw[ndw];
                uint32_t srow = 0;
                if (role < 2) {
                    const uint32_t* row = (const uint32_t*)(table + ((size_t)e * rows + colour) * (ndw * 4));
#pragma unroll
                    for (int i = 0; i < ndw; i++) rw[i] = row[i];
                } else {
                    srow = *(const uint32_t*)(J.S + ((size_t)e * 2 + colour) * 4);
                }
                const uint32_t slot = J.slot - 2 + (role < 2 ? role : 2u);
                const U128 h = hash_block(K, L.elem_base + e, slot, L.layer, L.key.rk, T);
                if (role < 2) decompress(P, h, [&](int i, uint32_t hd) { w[i] = submod4(rw[i], hd, P); });
                else beta = mod_m(srow + Mp.m - mod_u128(h, Mp), Mp);
            };
            uint32_t u[ndw], v[ndw], beta = 0;
#if defined(__HIP_DEVICE_COMPILE__)
            run_role(c, u, beta);
#pragma unroll
            for (int i = 0; i < ndw; i++) v[i] = quad_lane<1>(u[i]);
            beta = quad_lane<2>(beta);
            if (c != 0) return;
#else
            if (c != 0) return;
            uint32_t unused = 0;
            run_role(1, v, unused);
            run_role(2, u, beta);
            run_role(0, u, unused);
#endif
#pragma unroll
            for (int ch = 0; ch < nch; ch++) {
                Dw4 z;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int i = 4 * ch + q;
                    z.w[q] = i < ndw ? submod4(axpymod4(v[i], beta, x[ch].w[q], P), u[i], P) : 0u;
                }
                st_chunk(J.z, e, ch, z);
            }
        }
    });
}

}  // inline namespace
}  // namespace dash
