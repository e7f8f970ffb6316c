// dash_linear.hip -- the "free" linear layers on LabelTensors (Sec. Arithmetic Garbled Circuits: free
// addition and multiplication by a public constant; Sec. System-level Architecture: Dense and Conv2D;
// the Conv2D figure of Sec. LabelTensors): per CRT prime p
//     out[b][oy][ox][co][digit] = sum_{ky,kx,ci} (W[co][ky][kx][ci] mod p) * in[b][iy][ix][ci][digit]
//                                 (+ (bias[co] mod p) * one[digit])        mod p
// The garbler applies it to zero labels, the evaluator to active labels; the arithmetic is the same.
//
//   k_weights_prepare : int32 weights -> per-prime int8 residues in [0, p), rows padded to 64
//   k_linear_tile     : any shape; one lane per (output pixel, 16-digit chunk) and CO output channels
//   k_linear_split    : few outputs or few channels; a wave or 16 lanes per (output pixel, 16-digit chunk) and CO output channels
//   (dense layers that fill MFMA tiles go to k_dense_mfma in dash_gemm.hip)
//   k_sumpool         : 2x2 sum, stride 2
#include <string.h>

#include "dash_internal.h"
#include "dash_linear_rule.h"

namespace dash {

constexpr int kKpad = 64;   // weight rows are padded to a multiple of 64 entries

__host__ __device__ inline int64_t kpad_of(int K) { return ((int64_t)K + kKpad - 1) / kKpad * kKpad; }
__host__ __device__ inline int64_t mpad_of(int M) { return ((int64_t)M + 31) / 32 * 32; }

struct PrepArgs {
    const int32_t* w;
    int8_t* out;
    int M, K, k;
    uint32_t prime[DASH_MAX_PRIMES];
};

__global__ __launch_bounds__(kThreads) void k_weights_prepare(const PrepArgs A) {
    const int64_t Kp = kpad_of(A.K), Mp = mpad_of(A.M);
    int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (idx >= Mp * Kp) return;
    int64_t row = idx / Kp, col = idx - row * Kp;
    int32_t w = (row < A.M && col < A.K) ? A.w[row * A.K + col] : 0;
    for (int i = 0; i < A.k; i++) {
        int32_t p = (int32_t)A.prime[i];
        int32_t r = w % p;
        if (r < 0) r += p;
        A.out[(int64_t)i * Mp * Kp + idx] = (int8_t)r;
    }
}

struct LinPrime {
    uint32_t p;
    const int8_t* w;        // [Mpad][Kpad] residues of this prime
    const uint8_t* one;     // chunked label of the constant-one wire (zero or active), or NULL
    LView in, out;
};
struct LinArgs {
    const ModInfo* mods;
    const int32_t* bias;    // [out_c] or NULL
    int64_t kpad;
    int batch, in_h, in_w, in_c, out_c, kh, kw, stride, pad, out_h, out_w, co_first;
    LinPrime pr[DASH_MAX_PRIMES];
};

// Four consecutive entries k0 .. k0 + 3 of the reduction index against CO weight rows: the four 16-byte label words are turned around
// with byte permutes, so that a dword holds one digit of the four taps, and one byte dot product takes the four weights of an output.
// The permutes (32) and the loads are shared by the CO outputs, 16 dot products each.
template <int CO>
__device__ __forceinline__ void dot_group(const uint4* v, const uint32_t* w4, uint32_t acc[CO][16]) {
    const uint32_t vq[4][4] = {{v[0].x, v[1].x, v[2].x, v[3].x}, {v[0].y, v[1].y, v[2].y, v[3].y}, {v[0].z, v[1].z, v[2].z, v[3].z}, {v[0].w, v[1].w, v[2].w, v[3].w}};
#pragma unroll
    for (int q = 0; q < 4; q++) {
        // v_perm_b32(hi, lo, sel): byte i of the result = byte sel.i of the 8 bytes {hi:lo}
        const uint32_t ab02 = __builtin_amdgcn_perm(vq[q][1], vq[q][0], 0x06020400u), ab13 = __builtin_amdgcn_perm(vq[q][1], vq[q][0], 0x07030501u);
        const uint32_t cd02 = __builtin_amdgcn_perm(vq[q][3], vq[q][2], 0x06020400u), cd13 = __builtin_amdgcn_perm(vq[q][3], vq[q][2], 0x07030501u);
        const uint32_t d0 = __builtin_amdgcn_perm(cd02, ab02, 0x05040100u), d1 = __builtin_amdgcn_perm(cd13, ab13, 0x05040100u);
        const uint32_t d2 = __builtin_amdgcn_perm(cd02, ab02, 0x07060302u), d3 = __builtin_amdgcn_perm(cd13, ab13, 0x07060302u);
#pragma unroll
        for (int c = 0; c < CO; c++) {
            acc[c][4 * q + 0] = __builtin_amdgcn_udot4(d0, w4[c], acc[c][4 * q + 0], false);
            acc[c][4 * q + 1] = __builtin_amdgcn_udot4(d1, w4[c], acc[c][4 * q + 1], false);
            acc[c][4 * q + 2] = __builtin_amdgcn_udot4(d2, w4[c], acc[c][4 * q + 2], false);
            acc[c][4 * q + 3] = __builtin_amdgcn_udot4(d3, w4[c], acc[c][4 * q + 3], false);
        }
    }
}
// an accumulator ((p-1)^2 K < 2^31 is checked on the host) mod p, in two steps so that the magic division applies (n < 2^24)
__device__ __forceinline__ uint32_t reduce_acc(uint32_t a, const ModInfo& M) { return mod_m(mod_m(a >> 12, M) * (4096u % M.m) + (a & 4095u), M); }
__device__ __forceinline__ uint32_t bias_of(const int32_t* bias, int co, const ModInfo& M) {
    if (!bias) return 0;
    const int32_t r = bias[co] % (int32_t)M.m;
    return (uint32_t)(r < 0 ? r + (int32_t)M.m : r);
}

// One lane per (output pixel, chunk), CO output channels; blockIdx.y = prime, blockIdx.z = block of CO channels.  The taps are the same
// for all lanes: their offsets, the weights and the loop run on the scalar unit.  Bound by vector issue: 32 permutes and 16 CO dot
// products per four taps.  (One lane per output value repeated loads, permutes and 64-bit address arithmetic for every channel:
// 6 -> 16 channels, 5 x 5, 14 x 14, batch 16, 8 primes: 131 us; CO = 8: 49 us.)  CO = 1 and 4 serve few channels.
// D: groups of four taps in flight.  Two where the accumulators fill the registers; four for CO = 1 (5 x 5 over 28 x 28 x 6 -> 1, batch
// 16, 8 primes: 139 us with two, 121 with four).
template <int CO, bool Aligned, int D>
__global__ __launch_bounds__(kThreads) void k_linear_tile(const LinArgs A) {
    const LinPrime& P = A.pr[blockIdx.y];
    const ModInfo M = ld_mod(A.mods, P.p);
    const uint32_t n_px = (uint32_t)A.batch * A.out_h * A.out_w;
    const uint64_t idx = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    if (idx >= (uint64_t)n_px * M.nchunk) return;
    const uint32_t ch = (uint32_t)(idx / n_px), px = (uint32_t)(idx - (uint64_t)ch * n_px);
    const uint32_t row = px / (uint32_t)A.out_w, ox = px - row * A.out_w, b = row / (uint32_t)A.out_h, oy = row - b * A.out_h;
    const int iy0 = (int)oy * A.stride - A.pad, ix0 = (int)ox * A.stride - A.pad;
    const int base = (((int)b * A.in_h + iy0) * A.in_w + ix0) * A.in_c;      // (below 2^31; may be negative before the tap is added)
    const uint8_t* inc = P.in.p + (int64_t)ch * P.in.cs;
    const int co0 = A.co_first + (int)blockIdx.z * CO;
    const int8_t* wrow = P.w + (int64_t)co0 * A.kpad;                       // rows past out_c are there (padded to 32) and zero
    typedef const __attribute__((address_space(4))) uint32_t* sptr;         // weights are wave-uniform and not written by the kernel: scalar loads
    uint32_t acc[CO][16] = {};
    const int K = A.kh * A.kw * A.in_c;
    int ky = 0, kx = 0, ci = 0;
    struct Group { uint4 v[4]; uint32_t w4[CO]; };
    auto load = [&](int k0, Group& g) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CO; c++) {
            const int8_t* w = wrow + (int64_t)c * A.kpad + k0;
            if constexpr (Aligned) g.w4[c] = *(sptr)w;
            else __builtin_memcpy(&g.w4[c], w, 4);                         // (a scalar load drops the low two bits of its address)
        }
#pragma unroll
        for (int t = 0; t < 4; t++) {
            g.v[t] = make_uint4(0, 0, 0, 0);
            if (k0 + t < K) {
                const bool ok = A.pad == 0 || ((uint32_t)(iy0 + ky) < (uint32_t)A.in_h && (uint32_t)(ix0 + kx) < (uint32_t)A.in_w);
                if (ok) g.v[t] = *(const uint4*)(inc + ((uint64_t)(uint32_t)(base + (ky * A.in_w + kx) * A.in_c + ci) << 4));
                if (++ci == A.in_c) { ci = 0; if (++kx == A.kw) { kx = 0; ky++; } }
            }
        }
    };
    // the next groups' loads go out before the current one is multiplied (few waves fit beside 16 CO accumulators)
    Group g[D];
#pragma unroll
    for (int d = 0; d + 1 < D; d++) if (4 * d < K) load(4 * d, g[d]);
    for (int k0 = 0; k0 < K; k0 += 4 * D) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            if (k0 + 4 * d >= K) break;
            if (k0 + 4 * (d + D - 1) < K) load(k0 + 4 * (d + D - 1), g[(d + D - 1) % D]);
            dot_group<CO>(g[d].v, g[d].w4, acc);
        }
    }
    uint32_t one[4] = {0, 0, 0, 0};
    if (A.bias) { const uint4 o = *(const uint4*)(P.one + 16 * ch); one[0] = o.x; one[1] = o.y; one[2] = o.z; one[3] = o.w; }
    uint8_t* dst = P.out.p + (int64_t)ch * P.out.cs + ((uint64_t)px * A.out_c + co0) * 16;
#pragma unroll
    for (int c = 0; c < CO; c++) {
        if (co0 + c >= A.out_c) return;
        const uint32_t bm = bias_of(A.bias, co0 + c, M);
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            w[q] = 0;
#pragma unroll
            for (int d = 0; d < 4; d++) {
                uint32_t r = reduce_acc(acc[c][4 * q + d], M);
                if (bm) r = mod_m(r + mul24(bm, byte_of(one[q], d)), M);
                w[q] |= r << (8 * d);
            }
        }
        *(uint4*)(dst + 16 * c) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// S lanes (a wave, or a row of 16 lanes) per (output pixel, chunk), CO output channels; blockIdx.y = prime.  The lanes deal the reduction
// index out in groups of four; the 16 CO sums are then added up over the S lanes so that lane l ends with 16 CO / S consecutive ones of
// the CO x 16 (channel, digit).
// S = 64, CO = 8: layers whose outputs do not fill the chip.  The loop is 64 times shorter than a lane per output's, at about 300
// instructions for the addition.  (3 x 3 over 3 x 3 x 128 -> 128, 7 primes: 21 -> 11 us, the rate of the host's calls; 4096 -> 256, 12
// primes: 46 -> 33 us.)
// S = 16, CO = 1, 2, 4: layers of up to four output channels.  The 16 lanes read 1024 consecutive bytes of a pixel's channels, where
// neighbouring lanes of k_linear_tile read a word of different pixels each (times at linear_form_by_shape).
template <int CO, int S>
__global__ __launch_bounds__(kThreads) void k_linear_split(const LinArgs A) {
    static_assert(S == 64 || S == 16, "a wave or a row of lanes");
    const LinPrime& P = A.pr[blockIdx.y];
    const ModInfo M = ld_mod(A.mods, P.p);
    const uint32_t lane = threadIdx.x % S, n_px = (uint32_t)A.batch * A.out_h * A.out_w, njb = ((uint32_t)A.out_c + CO - 1) / CO;
    const uint32_t sub = threadIdx.x / S, unit = blockIdx.x * (kThreads / S) + (S == 64 ? __builtin_amdgcn_readfirstlane(sub) : sub);
    if (unit >= n_px * njb * M.nchunk) return;                              // (n_px * njb * nchunk < 2^32 / S: linear_split_fits)
    const uint32_t ch = unit / (n_px * njb), u = unit - ch * (n_px * njb), px = u / njb, co0 = (u - px * njb) * CO;
    const uint32_t row = px / (uint32_t)A.out_w, ox = px - row * A.out_w, b = row / (uint32_t)A.out_h, oy = row - b * A.out_h;
    const int iy0 = (int)oy * A.stride - A.pad, ix0 = (int)ox * A.stride - A.pad;
    const int base = (((int)b * A.in_h + iy0) * A.in_w + ix0) * A.in_c;
    const uint8_t* inc = P.in.p + (int64_t)ch * P.in.cs;
    const int8_t* wrow = P.w + (int64_t)co0 * A.kpad;
    uint32_t acc[CO][16] = {};
    const uint32_t K = (uint32_t)A.kh * A.kw * A.in_c;
    for (uint32_t k0 = 4 * lane; k0 < K; k0 += 4 * S) {
        uint32_t w4[CO];
#pragma unroll
        for (int c = 0; c < CO; c++) __builtin_memcpy(&w4[c], wrow + (int64_t)c * A.kpad + k0, 4);      // (at any address)
        uint32_t tap = A.kh * A.kw > 1 ? k0 / (uint32_t)A.in_c : 0u, ci = k0 - tap * A.in_c, ky = A.kw > 1 ? tap / (uint32_t)A.kw : tap, kx = tap - ky * A.kw;
        uint4 v[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const bool ok = k0 + t < K && (uint32_t)(iy0 + (int)ky) < (uint32_t)A.in_h && (uint32_t)(ix0 + (int)kx) < (uint32_t)A.in_w;
            v[t] = make_uint4(0, 0, 0, 0);
            if (ok) v[t] = *(const uint4*)(inc + ((uint64_t)(uint32_t)(base + (int)((ky * A.in_w + kx) * A.in_c + ci)) << 4));
            if (++ci == (uint32_t)A.in_c) { ci = 0; if (++kx == (uint32_t)A.kw) { kx = 0; ky++; } }
        }
        dot_group<CO>(v, w4, acc);
    }
    // add up over the S lanes: halves of the wave, halves of 32 lanes (swaps), then within rows of 16 lanes; each lane keeps the half of
    // its sums that its bit names
    uint32_t* s = &acc[0][0];
    if constexpr (S == 64) {
#pragma unroll
        for (int i = 0; i < 8 * CO; i++) { const auto r = __builtin_amdgcn_permlane32_swap(s[i], s[i + 8 * CO], false, false); s[i] = r[0] + r[1]; }
#pragma unroll
        for (int i = 0; i < 4 * CO; i++) { const auto r = __builtin_amdgcn_permlane16_swap(s[i], s[i + 4 * CO], false, false); s[i] = r[0] + r[1]; }
    }
#pragma unroll
    for (int d = 8, n = 128 * CO / S; d >= 1; d >>= 1, n >>= 1) {
        const uint32_t up = (lane & d) ? ~0u : 0u;         // (a mask: selects were turned into a search for the index i + n or i in registers)
#pragma unroll
        for (int i = 0; i < n; i++) {
            const uint32_t keep = (s[i + n] & up) | (s[i] & ~up), send = (s[i] & up) | (s[i + n] & ~up);
            uint32_t got;
            if (d == 8) got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x128, 0xf, 0xf, true);         // row_ror:8
            else if (d == 4) got = (uint32_t)__builtin_amdgcn_ds_swizzle((int)send, (4 << 10) | 0x1f);           // lane ^ 4
            else if (d == 2) got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x4E, 0xf, 0xf, true);     // quad_perm:[2,3,0,1]
            else got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0xB1, 0xf, 0xf, true);                 // quad_perm:[1,0,3,2]
            s[i] = keep + got;
        }
    }
    constexpr uint32_t kSums = 16 * CO / S;
    const int co = (int)(co0 + lane * kSums / 16), dg = (int)(lane * kSums % 16);
    if (co >= A.out_c) return;
    const uint32_t bm = A.bias ? bias_of(A.bias, co, M) : 0;
    uint32_t w = 0;
#pragma unroll
    for (uint32_t i = 0; i < kSums; i++) {
        uint32_t r = reduce_acc(s[i], M);
        if (A.bias) r = mod_m(r + mul24(bm, P.one[16 * ch + dg + i]), M);
        w |= r << (8 * i);
    }
    // neighbouring lanes put a dword together for one store
    if constexpr (kSums < 4) {
        w <<= 8 * (dg % 4);
        w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xf, 0xf, true);                              // quad_perm:[1,0,3,2]
        if constexpr (kSums == 1) w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xf, 0xf, true);    // quad_perm:[2,3,0,1]
        if (dg % 4) return;
    }
    *(uint32_t*)(P.out.p + (int64_t)ch * P.out.cs + ((uint64_t)px * A.out_c + co) * 16 + dg) = w;
}

struct PoolPrime { uint32_t p; LView in, out; };
struct PoolArgs {
    const ModInfo* mods;
    int batch, in_h, in_w, ch;
    PoolPrime pr[DASH_MAX_PRIMES];
};
// blockIdx.y = prime
__global__ __launch_bounds__(kThreads) void k_sumpool(const PoolArgs AA) {
    struct { uint32_t p; LView in, out; int batch, in_h, in_w, ch; } A;
    A.p = AA.pr[blockIdx.y].p; A.in = AA.pr[blockIdx.y].in; A.out = AA.pr[blockIdx.y].out;
    A.batch = AA.batch; A.in_h = AA.in_h; A.in_w = AA.in_w; A.ch = AA.ch;
    const ModInfo M = AA.mods[A.p];
    const int oh = A.in_h / 2, ow = A.in_w / 2;
    const int64_t n_out = (int64_t)A.batch * oh * ow * A.ch;
    int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (idx >= n_out * M.nchunk) return;
    const uint32_t chunk = (uint32_t)(idx / n_out);
    const int64_t o = idx - (int64_t)chunk * n_out;
    int c = (int)(o % A.ch);
    int64_t t = o / A.ch;
    int ox = (int)(t % ow); t /= ow;
    int oy = (int)(t % oh);
    int b = (int)(t / oh);
    uint32_t w[4] = {0, 0, 0, 0};
    for (int dy = 0; dy < 2; dy++)
        for (int dx = 0; dx < 2; dx++) {
            int64_t e = (((int64_t)b * A.in_h + 2 * oy + dy) * A.in_w + 2 * ox + dx) * A.ch + c;
            uint4 v = *(const uint4*)(A.in.p + (int64_t)chunk * A.in.cs + e * 16);
            w[0] = addmod4(w[0], v.x, M); w[1] = addmod4(w[1], v.y, M);
            w[2] = addmod4(w[2], v.z, M); w[3] = addmod4(w[3], v.w, M);
        }
    *(uint4*)(A.out.p + (int64_t)chunk * A.out.cs + o * 16) = make_uint4(w[0], w[1], w[2], w[3]);
}

int linear_layer(dash_ctx* c, const dash_layer* L, bool garble, const dash_labels* in, dash_labels* out, hipStream_t s) {
    int64_t per_out = 0;
    int st = layer_sizes(c, L, &per_out, nullptr, nullptr);
    if (st) return st;
    const int64_t batch = L->n_elem;
    if (batch == 0) return DASH_OK;
    int in_h = L->in_h, in_w = L->in_w, kh = L->kh, kw = L->kw, stride = L->stride, pad = L->pad, out_c = L->out_c;
    if (L->kind == DASH_DENSE) { in_h = in_w = kh = kw = stride = 1; pad = 0; }
    if (L->kind == DASH_SUMPOOL) out_c = L->in_c;
    const int64_t n_in = (int64_t)batch * in_h * in_w * L->in_c, n_out = batch * per_out;
    if (n_in > 0x7fffffff || n_out > 0x7fffffff) return DASH_ESIZE;
    if (!in || !out || in->n_elem < n_in || out->n_elem < n_out) return DASH_EINVAL;
    for (int i = 0; i < c->k; i++) {
        if (!in->data[i] || !out->data[i] || ((uintptr_t)in->data[i] & 15) || ((uintptr_t)out->data[i] & 15)) return DASH_EINVAL;
        if ((in->chunk_stride[i] & 15) || (out->chunk_stride[i] & 15) || in->chunk_stride[i] < 16 * n_in || out->chunk_stride[i] < 16 * n_out)
            return DASH_EINVAL;
    }
    if (L->kind == DASH_SUMPOOL) {
        PoolArgs A;
        memset(&A, 0, sizeof(A));
        A.mods = c->d_mods; A.batch = (int)batch; A.in_h = in_h; A.in_w = in_w; A.ch = L->in_c;
        int64_t lanes = 0;          // of the prime with the most chunks; the others' surplus blocks exit
        for (int i = 0; i < c->k; i++) {
            A.pr[i] = PoolPrime{(uint32_t)c->prime[i], view_of(in, i), view_of(out, i)};
            const int64_t l = n_out * c->mods[c->prime[i]].nchunk;
            lanes = l > lanes ? l : lanes;
        }
        hipLaunchKernelGGL(k_sumpool, dim3((uint32_t)((lanes + kThreads - 1) / kThreads), c->k), dim3(kThreads), 0, s, A);
        DASH_HIP(hipGetLastError());
        return DASH_OK;
    }
    if (!L->weights) return DASH_EINVAL;
    const int K = kh * kw * L->in_c;
    const int64_t Kp = kpad_of(K), Mp = mpad_of(out_c);
    for (int i = 0; i < c->k; i++) {
        uint64_t p1 = (uint64_t)(c->prime[i] - 1);
        if (p1 * p1 * (uint64_t)K >= (1ull << 31)) return DASH_ESIZE;      // int32 accumulators must not overflow
    }
    const int out_h = (in_h + 2 * pad - kh) / stride + 1, out_w = (in_w + 2 * pad - kw) / stride + 1;
    const int64_t npx = batch * out_h * out_w;
    int64_t chunks = 0;
    int nch = 1;                // chunks of all primes, of the prime with the most (the others' surplus blocks exit)
    for (int i = 0; i < c->k; i++) { chunks += c->mods[c->prime[i]].nchunk; nch = (int)c->mods[c->prime[i]].nchunk > nch ? (int)c->mods[c->prime[i]].nchunk : nch; }
    const int f = linear_form(c->linear_form, LinearShape{npx, chunks, nch, out_c, K, L->in_c, dense_mfma_wanted(L, batch)});
    if (f == LINEAR_MFMA) return dense_mfma(c, L, garble, in, out, s);
    LinArgs A;
    memset(&A, 0, sizeof(A));
    A.mods = c->d_mods; A.bias = L->bias; A.kpad = Kp;
    A.batch = (int)batch; A.in_h = in_h; A.in_w = in_w; A.in_c = L->in_c; A.out_c = out_c;
    A.kh = kh; A.kw = kw; A.stride = stride; A.pad = pad; A.out_h = out_h; A.out_w = out_w;
    double macs = 0, bytes = 0;
    for (int i = 0; i < c->k; i++) {
        LinPrime& P = A.pr[i];
        P.p = c->prime[i];
        P.w = (const int8_t*)L->weights + (int64_t)i * Mp * Kp;
        P.one = L->bias ? (garble ? c->d_one0[i] : c->d_one[i]) : nullptr;
        P.in = view_of(in, i); P.out = view_of(out, i);
        const double lam = c->mods[c->prime[i]].lam;
        macs += (double)n_out * K * lam;
        bytes += ((double)n_in + n_out) * lam + (double)out_c * K;
    }
    {
        ProfScope ps(c->prof, DASH_PROF_LINEAR, s, macs, bytes);
        const bool aligned = !((uintptr_t)L->weights & 3);
        const int lanes = linear_split_lanes(f), co = !lanes && !aligned ? 8 : linear_form_channels(f), blocks = (out_c + co - 1) / co;
        if (lanes) {
            const dim3 grid((uint32_t)((npx * blocks * nch * lanes + kThreads - 1) / kThreads), c->k);
            auto kernel = f == LINEAR_ROW1 ? k_linear_split<1, 16> : f == LINEAR_ROW2 ? k_linear_split<2, 16> : f == LINEAR_ROW4 ? k_linear_split<4, 16> : k_linear_split<8, 64>;
            hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, A);
        } else for (int at = 0; at < blocks; at += 65535) {                 // (the grid's third dimension ends at 65535)
            A.co_first = at * co;
            const dim3 grid((uint32_t)((npx * nch + kThreads - 1) / kThreads), c->k, blocks - at < 65535 ? blocks - at : 65535);
            auto kernel = !aligned ? k_linear_tile<8, false, 2> : co == 1 ? k_linear_tile<1, true, 4> : co == 4 ? k_linear_tile<4, true, 2> : k_linear_tile<8, true, 2>;
            hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, A);
        }
    }
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

}  // namespace dash

extern "C" {

size_t dash_weights_bytes(const dash_ctx* c, int out_c, int K) {
    if (!c || out_c < 1 || K < 1) return 0;
    return (size_t)c->k * (size_t)dash::mpad_of(out_c) * (size_t)dash::kpad_of(K);
}

int dash_weights_prepare(dash_ctx* c, const int32_t* w, int out_c, int K, void* prepared, void* stream) {
    if (!c || !w || !prepared || out_c < 1 || K < 1) return DASH_EINVAL;
    dash::PrepArgs A;
    memset(&A, 0, sizeof(A));
    A.w = w; A.out = (int8_t*)prepared; A.M = out_c; A.K = K; A.k = c->k;
    for (int i = 0; i < c->k; i++) A.prime[i] = c->prime[i];
    int64_t n = dash::mpad_of(out_c) * dash::kpad_of(K);
    if ((n + dash::kThreads - 1) / dash::kThreads > 0x7fffffff) return DASH_ESIZE;
    hipLaunchKernelGGL(dash::k_weights_prepare, dim3((uint32_t)((n + dash::kThreads - 1) / dash::kThreads)), dim3(dash::kThreads), 0,
                       (hipStream_t)stream, A);
    DASH_HIP(hipGetLastError());
    return DASH_OK;
}

}  // extern "C"
