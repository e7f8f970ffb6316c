// dash_gates.hip -- gate-level kernels over LabelTensors.
//
//   k_draw        : PRG labels (fresh zero labels of gate outputs, input wires, masks)
//   k_affine      : free gates: out = sum_t coef_t * term_t mod m   (Sec. Arithmetic Garbled Circuits)
//   k_proj_garble : one lane per ciphertext row: hash the label of value a, add the payload, store
//                   the row at the position its colour names            (projection gates, point-and-permute)
//   (the fused digit gates of the sign gadget: dash_gates_digits.hip; the evaluator's kernels: dash_gates_eval.hip,
//   dash_gates_digits_eval.hip, dash_gates_cast.hip)
//
// A launch carries up to 16 homogeneous gate batches ("jobs", blockIdx.y); every lane of a block
// works on the same pair of moduli, so all modulus-dependent control flow is wave-uniform.  The
// moduli that carry nearly all of the work (the CRT primes and the accumulation moduli of the
// default digit sets, with the label lengths of the rule this file is compiled for) run through compile-time
// descriptions; any other modulus or length takes the same code with run-time constants.
#include "dash_pack_rule.h"
#include "dash_tabs.h"

namespace dash {
inline namespace DASH_RULE_NS {

// ------------------------------------------------------------------------------------------ draw
template <bool Banked>
__global__ __launch_bounds__(gate_tab<Banked>::threads) void k_draw(const DrawLaunch L) {
    constexpr int kGateTiles = gate_tab<Banked>::threads / kThreads;
    __shared__ uint32_t tt[gate_tab<Banked>::words];
    const auto T = gate_tab<Banked>::load(tt, L.ttab);
    const uint32_t tiles = (L.jobs[blockIdx.y].n_elem + kThreads - 1) / kThreads;
    const uint32_t sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tx = threadIdx.x % kThreads;      // (the same in all lanes of a wave: scalar unit)
    for (uint32_t tile = blockIdx.x * kGateTiles + sub; tile < tiles; tile += gridDim.x * kGateTiles) draw_body(L, tile, blockIdx.y, tx, T);
}

int DASH_FN(launch_draw)(const dash_ctx* c, DrawLaunch& L, int njobs, hipStream_t s) {
    static_assert(sizeof(DrawLaunch) <= 4096, "kernel argument block");
    if (njobs < 1 || njobs > kMaxDrawJobs) return DASH_EINVAL;
    uint64_t lanes = 0;
    uint32_t nmax = 0;
    for (int j = 0; j < njobs; j++) {
        if (L.jobs[j].n_elem > (1u << 28)) return DASH_ESIZE;      // lane offsets into a chunk are 32-bit byte offsets
        lanes += L.jobs[j].n_elem;
        nmax = L.jobs[j].n_elem > nmax ? L.jobs[j].n_elem : nmax;
    }
    if (nmax == 0) return DASH_OK;
    const bool banked = lanes >= c->banked_min_lanes;
    L.key = banked ? c->seed_rot : c->seed; L.ttab = c->d_ttab; L.mods = c->d_mods;
    dim3 grid(gate_grid_x_for((nmax + kThreads - 1) / kThreads, njobs, banked), njobs);
    if (banked) hipLaunchKernelGGL(k_draw<true>, grid, dim3(kBigThreads), 0, s, L);
    else hipLaunchKernelGGL(k_draw<false>, grid, dim3(kThreads), 0, s, L);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

// the same for the zero labels of a gadget's gates (few: blockIdx.y = label, blockIdx.z = repetition)
template <bool Banked>
__global__ __launch_bounds__(gate_tab<Banked>::threads, Banked ? 8 : 1) void k_draw_many(const DrawManyLaunch L) {
    constexpr int kGateTiles = gate_tab<Banked>::threads / kThreads;
    __shared__ uint32_t tt[gate_tab<Banked>::words];
    const auto T = gate_tab<Banked>::load(tt, L.ttab);
    const uint32_t tiles = (L.n_elem + kThreads - 1) / kThreads;
    const uint32_t sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tx = threadIdx.x % kThreads;
    if constexpr (Banked) {      // one-dimensional grid over the tiles of all labels and repetitions: two blocks per CU, one round
        const uint32_t njobs = L.njobs, total = tiles * njobs * rep_count(L.reps), first = sub * gridDim.x + blockIdx.x, step = gridDim.x * kGateTiles;
        Pace pace(first, total, step);
        for (uint32_t t = first; t < total; t += step) {
            pace.tick();
            const uint32_t unit = __builtin_amdgcn_readfirstlane(t / tiles), rep = __builtin_amdgcn_readfirstlane(unit / njobs);
            draw_many_body(L, t - unit * tiles, unit - rep * njobs, rep, tx, T);
        }
    } else {
        for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) draw_many_body(L, tile, blockIdx.y, blockIdx.z, tx, T);
    }
}

int DASH_FN(launch_draw_many)(const dash_ctx* c, DrawManyLaunch& L, int njobs, hipStream_t s) {
    static_assert(sizeof(DrawManyLaunch) <= 4096, "kernel argument block");
    if (njobs < 1 || njobs > kMaxDrawMany) return DASH_EINVAL;
    if (L.n_elem == 0) return DASH_OK;
    if (L.n_elem > (1u << 28)) return DASH_ESIZE;      // lane offsets into a chunk are 32-bit byte offsets
    const uint32_t reps = rep_count(L.reps);
    const bool banked = (uint64_t)L.n_elem * njobs * reps >= c->banked_min_lanes;
    L.key = banked ? c->seed_rot : c->seed; L.ttab = c->d_ttab; L.mods = c->d_mods;
    const uint64_t tiles = (L.n_elem + kThreads - 1) / kThreads, all = tiles * njobs * reps;
    if (all > 0x7fffffffull) return DASH_ESIZE;
    L.njobs = (uint32_t)njobs;
    const dim3 grid = banked ? dim3((uint32_t)(all < 512 ? all : 512)) : dim3(grid_x_for(tiles, njobs * (int)reps), njobs, reps);
    if (banked) hipLaunchKernelGGL(k_draw_many<true>, grid, dim3(kBigThreads), 0, s, L);
    else hipLaunchKernelGGL(k_draw_many<false>, grid, dim3(kThreads), 0, s, L);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

// ------------------------------------------------------------------ free gates of the scaling gadget, garbler
__global__ __launch_bounds__(kThreads) void k_scale_free(const ScaleFreeLaunch L) {
    scale_free_body(L, blockIdx.x, blockIdx.y, blockIdx.z, threadIdx.x);
}

int DASH_FN(launch_scale_free)(const dash_ctx* c, ScaleFreeLaunch& L, hipStream_t s) {
    static_assert(sizeof(ScaleFreeLaunch) <= 4096, "kernel argument block");
    if (L.n < 1 || L.n > (uint32_t)kMaxChain || L.nres < 1 || L.nres > 14) return DASH_EINVAL;
    if (L.n_elem == 0) return DASH_OK;
    if (L.n_elem > (1u << 28)) return DASH_ESIZE;      // lane offsets into a chunk are 32-bit byte offsets
    L.mods = c->d_mods;
    uint32_t nchunk = c->mods[2].nchunk;
    for (uint32_t j = 1; j <= L.n; j++) {
        if (L.m[j] < 2 || L.m[j] > 255 || !L.S[j] || (j < L.n && !L.C[j])) return DASH_EINVAL;
        nchunk = c->mods[L.m[j]].nchunk > nchunk ? c->mods[L.m[j]].nchunk : nchunk;
    }
    for (uint32_t i = 0; i < L.nres; i++) {
        if (L.halve[i].p < 3 || L.halve[i].p > 255) return DASH_EINVAL;
        nchunk = c->mods[L.halve[i].p].nchunk > nchunk ? c->mods[L.halve[i].p].nchunk : nchunk;
    }
    const dim3 grid((uint32_t)(((uint64_t)L.n_elem * nchunk + kThreads - 1) / kThreads), L.n + 1 + L.nres, rep_count(L.reps));
    hipLaunchKernelGGL(k_scale_free, grid, dim3(kThreads), 0, s, L);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

// ---------------------------------------------------------------------------------------- affine
__global__ __launch_bounds__(kThreads) void k_affine(const AffineLaunch L) {
    affine_body(L, blockIdx.x, blockIdx.y, threadIdx.x);
}

int DASH_FN(launch_affine)(const dash_ctx* c, AffineLaunch& L, int njobs, hipStream_t s) {
    static_assert(sizeof(AffineLaunch) <= 4096, "kernel argument block");
    if (njobs < 1 || njobs > kMaxJobs) return DASH_EINVAL;
    if (L.n_elem == 0) return DASH_OK;
    if (L.n_elem > (1u << 28)) return DASH_ESIZE;      // lane offsets into a chunk are 32-bit byte offsets
    L.mods = c->d_mods;
    uint32_t nchunk = 1;
    for (int j = 0; j < njobs; j++) {
        AffineJob& J = L.jobs[j];
        if (J.m < 2 || J.m > 255 || J.term_count == 0 || J.term_first + J.term_count > (uint32_t)kMaxTerms) return DASH_EINVAL;
        J.unit = 1;
        for (uint32_t t = 0; t < J.term_count; t++) if (L.terms[J.term_first + t].coef != 1) J.unit = 0;
        nchunk = c->mods[J.m].nchunk > nchunk ? c->mods[J.m].nchunk : nchunk;
    }
    dim3 grid((uint32_t)(((uint64_t)L.n_elem * nchunk + kThreads - 1) / kThreads), njobs);
    hipLaunchKernelGGL(k_affine, grid, dim3(kThreads), 0, s, L);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

// ------------------------------------------------------------------------------- packed table rows
// Working format [pitch_q bytes, one digit each] <-> 16-byte integer sum_j row[j] q^j.  What the kernel has to do is move bytes (36 per 20-byte
// row).  The segments of a layer differ in length by a factor of 50, so the waves share the concatenation of their tiles of 64 rows, a run of up to
// four at a time (dash_pack_rule.h), neighbouring waves neighbouring runs (a contiguous range for each wave was 16 384 streams through 8 GB: 2.7
// ms instead of 2.3 below).
// Packing: a lane reads its own row and has those of up to four tiles in flight.  (Rows through LDS, a dword per lane, one tile at a time and the
// segment looked for at every tile: 2.5 TB/s, 3.4 ms for the 5.1 GB of tables of a LeNet batch of 4; this way 1.8 ms, 4.6 TB/s.)
// Packing: 64 registers, eight waves per SIMD.  A modulus without compile-time code reads its row in pieces of four dwords (dword by dword, with so many
// waves beside each other: 4 primes, 160 000 values, 913 us; 387 this way).
// Unpacking: a wave brings its 64 rows through LDS, so that every access to them is a dword per lane, consecutive lanes consecutive dwords,
// whatever the pitch; the 16-byte rows of two tiles are read at a time (one, two: 4.22, 3.88 ms with the evaluation behind it).  The lane's number
// is taken anew for every run: else the addresses that follow from it, for all moduli, are formed before the loop, 128 registers and 88 bytes of
// scratch memory a lane (65 and none this way, seven waves per SIMD instead of four: 12 primes, ReLU, 20 000 values, 795 us and 634; 2 primes, 40 000, 48 and 30).
// Rows of bits (q = 2): 16 digits are 16 bits, a lane moves 16 bytes on one side and 2 on the other.
template <bool Pack>
__global__ __launch_bounds__(kThreads, Pack ? 8 : 7) void k_rows_repack(const PackLaunch L) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef u32x4 u32x4_at4 __attribute__((aligned(4)));              // of table rows: tables, and with rows of 20 bytes their segments, are 4-byte aligned
    const uint32_t lg = L.run_log2;                                   // a wave takes 2^lg tiles at a time
    constexpr int kMaxDw = 21;                                        // dwords of the longest row that goes through LDS (81 digits)
    __shared__ uint32_t stage[Pack ? 1 : kThreads / 64][Pack ? 1 : 64 * kMaxDw];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t* st = stage[Pack ? 0 : wave];
    auto rows_of = [&](uint32_t i) { return (uint64_t)L.n_elem * L.seg[i].rows_per_gate; };
    // one-digit rows: 1024 bytes of the packed segment per tile (padded with zeros to a multiple of 16 bytes)
    auto tiles_of = [&](uint32_t i) { return L.seg[i].q ? (rows_of(i) + 63) / 64 : (rows_of(i) + 1023) / 1024; };
    auto runs_of = [&](uint32_t i) { return (tiles_of(i) + (1u << lg) - 1) >> lg; };
    const uint64_t waves = (uint64_t)gridDim.x * (kThreads / 64);
    uint32_t seg = 0;
    uint64_t base = 0, next = runs_of(0);
    for (uint64_t run = (uint64_t)blockIdx.x * (kThreads / 64) + wave; run < L.runs; run += waves) {
        while (run >= next) {
            base = next;
            next += runs_of(++seg);
        }
        const uint32_t lane = Pack ? threadIdx.x & 63u : opaque_lane(threadIdx.x & 63u);
        const PackSeg& S = L.seg[seg];
        const uint64_t rows = rows_of(seg), first = (run - base) << lg, last = tiles_of(seg), stop = first + (1u << lg) < last ? first + (1u << lg) : last;
        if (S.q == 0) {
            for (uint64_t tile = first; tile < stop; tile++) {
                const uint64_t r0 = tile * 1024 + lane * 16, padded = (rows + 15) & ~(uint64_t)15;
                for (int k = 0; k < 16 && r0 + k < padded; k++) {
                    const uint64_t r = r0 + k;
                    if (Pack) S.packed[r] = r < rows ? S.rows[r * 4] : 0;
                    else if (r < rows) *(uint32_t*)(const_cast<uint8_t*>(S.rows) + r * 4) = S.packed[r];
                }
            }
            continue;
        }
        with_mod(ld_mod(L.mods, S.q), [&](auto M) {
            typedef decltype(M) MD;
            if constexpr (cmod_m<MD>::value == 2) {
                for (uint64_t tile = first; tile < stop; tile++) {
                    const uint64_t r0 = tile * 64;
                    const uint32_t n = rows - r0 < 64 ? (uint32_t)(rows - r0) : 64u;
                    uint16_t* bits = (uint16_t*)(S.packed + r0 * 16);
                    u32x4_at4* digits = (u32x4_at4*)(const_cast<uint8_t*>(S.rows) + r0 * 128);
                    uint32_t v16[8];
                    u32x4 v[8];
#pragma unroll
                    for (uint32_t i = 0; i < 8; i++) {                   // piece i * 64 + lane: row / 8, 16 digits of it
                        const uint32_t d = i * 64 + lane < n * 8 ? i * 64 + lane : 0;
                        if (Pack) v[i] = digits[d];
                        else v16[i] = bits[d];
                    }
#pragma unroll
                    for (uint32_t i = 0; i < 8; i++) {
                        if (i * 64 + lane >= n * 8) continue;
                        if (Pack) {
                            uint32_t w = 0;
#pragma unroll
                            for (int q = 0; q < 4; q++) w |= dot4(v[i][q], 0x08040201u) << (4 * q);
                            bits[i * 64 + lane] = (uint16_t)w;
                        } else {
                            u32x4 w;
#pragma unroll
                            for (int q = 0; q < 4; q++) w[q] = mul24((v16[i] >> (4 * q)) & 0xfu, 0x00204081u) & kOnes;
                            digits[i * 64 + lane] = w;
                        }
                    }
                }
            } else if constexpr (cmod_m<MD>::value != 0) {
                constexpr uint32_t ndw = MD::ndw, stride = ndw | 1;      // (odd: a lane's own row without bank conflicts)
                static_assert(stride <= kMaxDw, "stage");
                constexpr uint32_t U = !Pack ? 2 : ndw <= 5 ? 4 : ndw <= 10 ? 2 : 1;      // tiles in flight
                for (uint64_t tile = first; tile < stop; tile += U) {
                    const uint64_t r0 = tile * 64, left = (stop * 64 < rows ? stop * 64 : rows) - r0;
                    const uint32_t n = left < U * 64 ? (uint32_t)left : U * 64;      // rows; lanes past them read the last one and store nothing
                    uint8_t* const rowbase = const_cast<uint8_t*>(S.rows) + r0 * (ndw * 4);
                    uint8_t* const packed = S.packed + r0 * 16;
                    if constexpr (Pack) {
                        uint32_t v[U][ndw];
#pragma unroll
                        for (uint32_t u = 0; u < U; u++) ld_dwords<(int)ndw>(rowbase, (u * 64 + lane < n ? u * 64 + lane : n - 1) * (ndw * 4), v[u]);
                        schedule_fence();
#pragma unroll
                        for (uint32_t u = 0; u < U; u++) {
                            uint32_t colour;
                            const U128 x = compress(M, [&](int i) { return v[u][i]; }, &colour);
                            if (u * 64 + lane < n) *(u32x4*)(packed + (u * 64 + lane) * 16) = u32x4{x.w[0], x.w[1], x.w[2], x.w[3]};
                        }
                    } else {
                        u32x4 v[U];
#pragma unroll
                        for (uint32_t u = 0; u < U; u++) v[u] = *(const u32x4*)(packed + (u * 64 + lane < n ? u * 64 + lane : n - 1) * 16);
                        schedule_fence();
#pragma unroll 1
                        for (uint32_t u = 0; u * 64 < n; u++) {
                            decompress(M, U128{{v[0].x, v[0].y, v[0].z, v[0].w}}, [&](int i, uint32_t w) { st[lane * stride + i] = w; });
#pragma unroll
                            for (uint32_t k = 0; k + 1 < U; k++) v[k] = v[k + 1];
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                            __builtin_amdgcn_wave_barrier();
                            DASH_WAVE_POINT();
                            const uint32_t m = n - u * 64 < 64 ? n - u * 64 : 64u;
#pragma unroll
                            for (uint32_t i = 0; i < ndw; i++) {
                                const uint32_t d = i * 64 + lane;
                                if (d < m * ndw) *(uint32_t*)(rowbase + (u * (64 * ndw) + d) * 4) = st[(d / ndw) * stride + d % ndw];
                            }
                            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                            __builtin_amdgcn_wave_barrier();
                            DASH_WAVE_POINT();
                        }
                    }
                }
            } else {                                                     // any other modulus or length: run-time constants, a row per lane
                for (uint64_t tile = first; tile < stop; tile++) {
                    const uint64_t r = tile * 64 + lane;
                    if (r >= rows) continue;
                    uint32_t* row = (uint32_t*)(const_cast<uint8_t*>(S.rows) + r * (M.ndw * 4));
                    u32x4* packed = (u32x4*)(S.packed + r * 16);
                    if (Pack) {
                        uint32_t colour;
                        U128 x;
                        if (M.ndw >= 4) {                                // from the top, the last piece overlapping the one before
                            u32x4 piece = {};
                            int at = 0;
                            x = compress(M, [&](int i) {
                                if ((((int)M.ndw - 1 - i) & 3) == 0) { at = i >= 3 ? i - 3 : 0; piece = *(const u32x4_at4*)(row + at); }
                                const int q = i - at;
                                return q & 2 ? (q & 1 ? piece[3] : piece[2]) : (q & 1 ? piece[1] : piece[0]);
                            }, &colour);
                        } else x = compress(M, [&](int i) { return row[i]; }, &colour);
                        *packed = u32x4{x.w[0], x.w[1], x.w[2], x.w[3]};
                    } else {
                        const u32x4 v = *packed;
                        decompress(M, U128{{v.x, v.y, v.z, v.w}}, [&](int i, uint32_t w) { row[i] = w; });
                    }
                }
            }
        });
    }
}

int DASH_FN(launch_pack)(const dash_ctx* c, PackLaunch& L, bool pack, hipStream_t s) {
    static_assert(sizeof(PackLaunch) <= 4096, "kernel argument block");
    if (L.nseg < 1 || L.nseg > (uint32_t)kMaxPackSegs) return DASH_EINVAL;
    if (L.n_elem == 0) return DASH_OK;
    L.mods = c->d_mods;
    auto tiles_of = [&](uint32_t i) {
        const uint64_t rows = (uint64_t)L.n_elem * L.seg[i].rows_per_gate;
        return L.seg[i].q ? (rows + 63) / 64 : (rows + 1023) / 1024;
    };
    uint64_t tiles = 0;
    for (uint32_t i = 0; i < L.nseg; i++) tiles += tiles_of(i);
    const PackShape shape = pack_shape(tiles, L.nseg, pack);
    L.run_log2 = c->pack_run_log2 < 0 ? shape.run_log2 : (uint32_t)c->pack_run_log2;
    L.runs = 0;
    for (uint32_t i = 0; i < L.nseg; i++) L.runs += (tiles_of(i) + (1u << L.run_log2) - 1) >> L.run_log2;
    const uint64_t blocks = (L.runs + kThreads / 64 - 1) / (kThreads / 64);
    const dim3 grid((uint32_t)(blocks < shape.max_blocks ? blocks : shape.max_blocks));
    if (pack) hipLaunchKernelGGL(k_rows_repack<true>, grid, dim3(kThreads), 0, s, L);
    else hipLaunchKernelGGL(k_rows_repack<false>, grid, dim3(kThreads), 0, s, L);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

// ---------------------------------------------------------------------------------------- garble
// One instantiation per output-modulus description: QD = ModInfo (any modulus, run-time constants) or
// CMod<m, lam> for the hot moduli.  The input modulus is dispatched inside (its code is small).
// Rows of 64 bytes or more (pitch a multiple of 16): a lane that stored its own row dword by dword would
// touch 64 different cache lines with every store instruction.  Such rows are staged in LDS (row stride
// one word more than the pitch, so the column accesses spread over the banks) and written by the whole
// block, each lane 16 consecutive bytes, consecutive lanes consecutive pieces of a row.
template <class QD> struct stage_rows { static constexpr bool value = false; static constexpr int ndw = 1; };
template <uint32_t MOD, uint32_t LAM> struct stage_rows<CMod<MOD, LAM>> {
    static constexpr int ndw = (LAM + 3) / 4;
    static constexpr bool value = ndw >= 16 && ndw % 16 == 0;
};
struct StagedSink {
    uint32_t* st;        // this lane's row in LDS
    uint32_t* slot;      // where the row index goes
    __device__ __forceinline__ void begin(uint8_t*, uint64_t row_index, uint32_t) { *slot = (uint32_t)row_index; }
    __device__ __forceinline__ void put(int i, uint32_t w) { st[i] = w; }
};

// a row kept in the lane's registers, with the address it goes to (0: the lane has no row to stage)
template <int NDW> struct RegSink {
    uint32_t w[NDW];
    uint64_t addr = 0;
    __device__ __forceinline__ void begin(uint8_t* table, uint64_t row_index, uint32_t pitch) { addr = (uint64_t)(table + row_index * pitch); }
    __device__ __forceinline__ void put(int i, uint32_t v) { w[i] = v; }
};

template <class QD, bool Banked>
__global__ __launch_bounds__(gate_tab<Banked>::threads, Banked ? 8 : 1) void k_proj_garble(const GateLaunch L) {
    constexpr int kGateTiles = gate_tab<Banked>::threads / kThreads;
    const uint64_t rows = (uint64_t)L.jobs[blockIdx.y].n_elem * L.jobs[blockIdx.y].p;      // (unused by the one-dimensional banked forms)
    const uint32_t tiles = (uint32_t)((rows + kThreads - 1) / kThreads);
    if constexpr (stage_rows<QD>::value && Banked) {
        // Long rows with the bank-replicated tables: 64 KB of tables leave room to stage 16 dwords per lane, so a lane keeps
        // its row in registers and its wave writes the rows out in ndw / 16 passes of 64 bytes per row, 16 bytes per lane,
        // consecutive lanes consecutive pieces.  One-dimensional grid over the tiles of all jobs.
        constexpr int ndw = stage_rows<QD>::ndw, kPass = 16, stride = kPass + 1, pieces = kPass / 4;
        static_assert(ndw % kPass == 0, "whole passes");
        __shared__ uint32_t tt[kBankTabWords];
        __shared__ uint32_t stage[kBigThreads * stride];
        __shared__ uint64_t sdst[kBigThreads];
        const BankTab T = load_banktab(tt, L.ttab);
        const uint32_t sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tx = threadIdx.x % kThreads;      // (the same in all lanes of a wave: scalar unit)
        const int lane = threadIdx.x & 63, w0 = threadIdx.x & ~63;       // this wave's rows: w0 .. w0 + 63
        auto tiles_of = [&](uint32_t j) { return (uint32_t)(((uint64_t)L.jobs[j].n_elem * L.jobs[j].p + kThreads - 1) / kThreads); };
        uint32_t total = 0;
        for (uint32_t j = 0; j < L.njobs; j++) total += tiles_of(j);
        total *= rep_count(L.reps);
        uint32_t job = 0, rep = 0, base = 0, next = tiles_of(0);
        // (every wave stages and writes out its own 64 rows: no barrier between waves)
        const uint32_t rounds = (total + gridDim.x * kGateTiles - 1) / (gridDim.x * kGateTiles);
        Pace pace(rounds);
        for (uint32_t r = 0; r < rounds; r++) {
            const uint32_t t = (r * kGateTiles + sub) * gridDim.x + blockIdx.x;
            RegSink<ndw> sink;
            pace.tick();
            if (t < total) {
                while (t >= next) { if (++job == L.njobs) { job = 0; rep++; } base = next; next += tiles_of(job); }
                garble_body<QD>(L, t - base, job, tx, T, sink, rep);
            }
            sdst[threadIdx.x] = sink.addr;
#pragma unroll
            for (int pass = 0; pass < ndw / kPass; pass++) {
                if (sink.addr) {
#pragma unroll
                    for (int i = 0; i < kPass; i++) stage[threadIdx.x * stride + i] = sink.w[pass * kPass + i];
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                for (int id = lane; id < 64 * pieces; id += 64) {
                    const int k = w0 + id / pieces, part = id % pieces;
                    const uint64_t d = sdst[k];
                    if (d) {
                        const uint32_t* src = stage + k * stride + part * 4;
                        uint32_t* dst = (uint32_t*)(d + (uint64_t)pass * (kPass * 4) + part * 16);
                        uint32_t v0 = src[0], v1 = src[1], v2 = src[2], v3 = src[3];
                        dst[0] = v0; dst[1] = v1; dst[2] = v2; dst[3] = v3;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    } else if constexpr (stage_rows<QD>::value) {
        // Long rows, shared tables: every WAVE stages its 64 rows in its own part of LDS and writes them out itself, 16 bytes
        // per lane, eight consecutive lanes one row: no barrier between waves (a wave's LDS accesses complete in order).
        __shared__ uint32_t tt[kTabWords];
        const LdsTab T = load_ttab(tt, L.ttab);
        constexpr int ndw = stage_rows<QD>::ndw, stride = ndw + 1, pieces = ndw / 4;
        __shared__ uint32_t stage[kThreads * stride];
        __shared__ uint32_t srow[kThreads];
        uint8_t* table = L.jobs[blockIdx.y].table + (int64_t)blockIdx.z * L.reps.tables;
        const int lane = threadIdx.x & 63, w0 = threadIdx.x & ~63;       // this wave's rows: w0 .. w0 + 63
        for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
            srow[threadIdx.x] = 0xffffffffu;
            StagedSink sink{stage + threadIdx.x * stride, srow + threadIdx.x};
            garble_body<QD>(L, tile, blockIdx.y, threadIdx.x, T, sink, blockIdx.z);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int id = lane; id < 64 * pieces; id += 64) {
                const int k = w0 + id / pieces, part = id % pieces;
                const uint32_t r = srow[k];
                if (r != 0xffffffffu) {
                    const uint32_t* src = stage + k * stride + part * 4;
                    uint32_t* dst = (uint32_t*)(table + (uint64_t)r * (ndw * 4) + part * 16);
                    uint32_t v0 = src[0], v1 = src[1], v2 = src[2], v3 = src[3];
                    dst[0] = v0; dst[1] = v1; dst[2] = v2; dst[3] = v3;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        __shared__ uint32_t tt[gate_tab<Banked>::words];
        const auto T = gate_tab<Banked>::load(tt, L.ttab);
        const uint32_t sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tx = threadIdx.x % kThreads;      // (the same in all lanes of a wave: scalar unit)
        // Run-time modulus: its record and the round keys together are more than the scalar registers hold, and 826 places of the code brought one
        // back from a vector register (61 with the keys read again; a repetition of 40 000 values of 10 primes garbled in 3.0 ms instead of 4.9).
        auto body = [&](uint32_t tile, uint32_t job, uint32_t rep) __attribute__((always_inline)) {
            DirectSink sink;
            if constexpr (std::is_same<QD, ModInfo>::value)
                garble_body<QD>(L, tile, job, tx, T, sink, rep, [] { return read_again(((const __attribute__((address_space(4))) GateLaunch*)__builtin_amdgcn_kernarg_segment_ptr())->key.rk); });
            else
                garble_body<QD>(L, tile, job, tx, T, sink, rep);
        };
        if constexpr (Banked) {
            // one-dimensional grid: the jobs differ in length (n_elem * p rows), so the blocks share the
            // concatenation of all jobs' tiles evenly.  job, base and next are the same in all lanes of a wave.
            auto tiles_of = [&](uint32_t j) { return (uint32_t)(((uint64_t)L.jobs[j].n_elem * L.jobs[j].p + kThreads - 1) / kThreads); };
            uint32_t total = 0;
            for (uint32_t j = 0; j < L.njobs; j++) total += tiles_of(j);
            total *= rep_count(L.reps);
            uint32_t job = 0, rep = 0, base = 0, next = tiles_of(0);
            // (one tile of each block, then the next of each: what is left over for a last, partial round lies on as many CUs as it has tiles)
            const uint32_t first = sub * gridDim.x + blockIdx.x, step = gridDim.x * kGateTiles;
            Pace pace(first, total, step);
            for (uint32_t t = first; t < total; t += step) {
                pace.tick();
                while (t >= next) { if (++job == L.njobs) { job = 0; rep++; } base = next; next += tiles_of(job); }
                body(t - base, job, rep);
            }
        } else {
            for (uint32_t tile = blockIdx.x * kGateTiles + sub; tile < tiles; tile += gridDim.x * kGateTiles) body(tile, blockIdx.y, blockIdx.z);
        }
    }
}

#define DASH_GARBLE_K(MOD, LAM) k_proj_garble<CMod<MOD, LAM>, false>,
static const GateKernel kGarbleKernels[] = {k_proj_garble<ModInfo, false>, DASH_HOT_MODS(DASH_GARBLE_K)};
#undef DASH_GARBLE_K
// with BankTab
#define DASH_GARBLE_KB(MOD, LAM) k_proj_garble<CMod<MOD, LAM>, true>,
static const GateKernel kGarbleKernelsBanked[] = {k_proj_garble<ModInfo, true>, DASH_HOT_MODS(DASH_GARBLE_KB)};
#undef DASH_GARBLE_KB
#define DASH_GARBLE_S(MOD, LAM) stage_rows<CMod<MOD, LAM>>::value,
static const bool kGarbleStaged[] = {false, DASH_HOT_MODS(DASH_GARBLE_S)};
#undef DASH_GARBLE_S


int DASH_FN(launch_garble)(const dash_ctx* c, GateLaunch& L, int njobs, hipStream_t s) {
    if (njobs < 1 || njobs > kMaxJobs) return DASH_EINVAL;
    L.key = c->fixed; L.ttab = c->d_ttab; L.mods = c->d_mods;
    uint64_t rows = 0, tiles_sum = 0;      // rows of the largest job; tiles of all jobs
    double units = 0, bytes = 0;
    for (int j = 0; j < njobs; j++) {
        const GateJob& J = L.jobs[j];
        if (J.n_elem > (1u << 28)) return DASH_ESIZE;      // lane offsets into a chunk are 32-bit byte offsets
        if (J.n_elem == 0) continue;
        if (J.p < 2 || J.p > 255 || J.q < 2 || J.q > 255 || !c->mods[J.p].dtab || !c->mods[J.q].dtab) return DASH_EINVAL;
        if (!J.in.p || !J.table) return DASH_EINVAL;
        const uint64_t r = (uint64_t)J.n_elem * J.p;
        rows = r > rows ? r : rows;
        tiles_sum += (r + kThreads - 1) / kThreads;
        const double lp = c->mods[J.p].lam, lq = J.mode == PAY_SHORT ? 1 : c->mods[J.q].lam;
        units += (double)r;
        bytes += (double)J.n_elem * (lp + (J.phi_stride ? J.p : 0) + lq + J.p * lq + (J.mode == PAY_EHALF ? lq : 0));
    }
    if (rows == 0) return DASH_OK;
    const uint32_t reps = rep_count(L.reps);
    units *= reps; bytes *= reps; tiles_sum *= reps;
    const uint64_t blocks = (rows + kThreads - 1) / kThreads;
    if (blocks > 0x7fffffffull || tiles_sum > 0x7fffffffull) return DASH_ESIZE;
    // jobs with one output modulus run its instantiation; a mix of output moduli (many small batches
    // in one launch) runs the instantiation with run-time constants
    const uint32_t q = common_q(L, njobs);
    if (rows >= (1ull << 32)) return DASH_ESIZE;      // staged rows carry a 32-bit row index
    const int ki = q ? hot_mod_index(c->mods[q]) : 0;
    const bool staged = kGarbleStaged[ki];
    const bool banked = (uint64_t)units >= c->banked_min_lanes;
    if (banked) L.key = c->fixed_rot;
    L.njobs = (uint32_t)njobs;
    dim3 grid(gate_grid_x_for(blocks, njobs * (int)reps, banked), njobs, reps);
    if (banked) {       // one-dimensional: all jobs' tiles, 1024 lanes (4 tiles) per block at a time, two blocks per CU
        const uint64_t nb = (tiles_sum + 3) / 4;
        const uint64_t cap = staged ? 256 : 512;      // (long rows also stage in LDS: one block per CU)
        grid = dim3((uint32_t)(nb < cap ? nb : cap));
    }
    ProfScope ps(c->prof, DASH_PROF_GARBLE, s, units, bytes);
    // carry gates: kernels of their own, whose blocks have the bank-replicated tables.  (665 600 rows of the final gate: 46 us in
    // k_proj_garble with one copy of the tables, 31 in k_chain_garble_bits.)
    if ((uint64_t)units >= c->banked_min_lanes / 4) {
        L.key = c->fixed_rot;
        bool done = false;
        const int st = DASH_FN(launch_chain_garble)(c, L, njobs, s, &done);
        if (st || done) return st;
        if (!banked) L.key = c->fixed;
    }
    GateKernel k = banked ? kGarbleKernelsBanked[ki] : kGarbleKernels[ki];
    if (ki == 0 && !banked && (uint64_t)units <= c->few_rows_max) k = k_proj_garble<PerJobMod, false>;      // few rows: see garble_body
    hipLaunchKernelGGL(k, grid, dim3(banked ? kBigThreads : kThreads), 0, s, L);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

}  // inline namespace
}  // namespace dash
