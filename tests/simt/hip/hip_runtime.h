// Host stand-in for the HIP runtime: a kernel launch runs on the CPU, block after block, a fiber per lane, so that the kernels
// themselves (index arithmetic, barriers, LDS) can be compiled with the address and undefined-behaviour sanitizers.  Covers what the
// sources that are built with it use, and nothing else.  Test code, not part of libdash.
//
// A lane runs until it meets a barrier of its block or of its wave, or ends; a barrier opens when every lane of the block or wave that
// has not ended stands at it.  Lanes run in ascending or (SIMT_REVERSE set)
// descending order between barriers: a result that depends on the order shows a missing barrier.
// SIMT_TRACE set: a line per launch on stderr.
// Dynamic LDS is the array whose name the source gives it, at namespace scope; simt::dynamic_lds announces it, and what a launch does
// not ask for is poisoned.
#pragma once
#include <math.h>
#include <sanitizer/asan_interface.h>
#include <sanitizer/common_interface_defs.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <functional>
#include <vector>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ thread_local      // one program thread: static storage, one copy for all lanes
#define address_space(n) may_alias   // __attribute__((address_space(4))): constant memory is ordinary memory

struct dim3 { uint32_t x, y, z; dim3(uint32_t x_ = 1, uint32_t y_ = 1, uint32_t z_ = 1) : x(x_), y(y_), z(z_) {} };
struct __attribute__((aligned(16))) uint4 { uint32_t x, y, z, w; };
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return uint4{x, y, z, w}; }

namespace simt {
constexpr size_t kStack = 512 << 10;
enum { RUN, AT_WAVE, AT_BLOCK, ENDED };
struct Lane { void* sp; char* stack; void* fake; uint32_t id; int state; int value; bool there; };
inline std::vector<Lane> lanes;
inline Lane* cur;
inline void* main_sp;
inline void* main_fake;
inline const void* main_stack;
inline size_t main_size;
inline dim3 block_idx, block_dim, grid_dim;
inline const void* kernarg;
inline std::function<void()>* body;
struct Dynamic { char* p; size_t size; };
inline std::vector<Dynamic>& dynamic() { static std::vector<Dynamic> d; return d; }
struct dynamic_lds { dynamic_lds(void* p, size_t size) { dynamic().push_back({(char*)p, size}); } };

// saves the callee's registers and the stack pointer, goes on where another fiber did (swapcontext changes the signal mask with a system
// call, and the sanitizer's version of it clears the shadow of the whole stack every time)
extern "C" void simt_switch(void** save, void* to);
#if defined(SIMT_MAIN)
asm(R"(
.globl simt_switch
.type simt_switch,@function
simt_switch:
    pushq %rbp
    pushq %rbx
    pushq %r12
    pushq %r13
    pushq %r14
    pushq %r15
    movq %rsp, (%rdi)
    movq %rsi, %rsp
    popq %r15
    popq %r14
    popq %r13
    popq %r12
    popq %rbx
    popq %rbp
    retq
)");
#endif

inline void enter() {
    __sanitizer_finish_switch_fiber(nullptr, &main_stack, &main_size);
    (*body)();
    cur->state = ENDED;
    __sanitizer_start_switch_fiber(nullptr, main_stack, main_size);
    simt_switch(&cur->sp, main_sp);
}
inline void wait(int state) {
    Lane* me = cur;
    me->state = state;
    __sanitizer_start_switch_fiber(&me->fake, main_stack, main_size);
    simt_switch(&me->sp, main_sp);
    __sanitizer_finish_switch_fiber(me->fake, &main_stack, &main_size);
}
inline void resume(Lane& l) {
    cur = &l;
    __sanitizer_start_switch_fiber(&main_fake, l.stack, kStack);
    simt_switch(&main_sp, l.sp);
    __sanitizer_finish_switch_fiber(main_fake, nullptr, nullptr);
}
// opens a barrier of the lanes first .. first + n - 1 if all that are left stand at it (a barrier of a wave: all that are in the same
// branch, i.e. not at a barrier of the block already)
inline bool open(uint32_t first, uint32_t n, int state) {
    bool any = false;
    for (uint32_t i = first; i < first + n; i++) {
        if (lanes[i].state == ENDED || (state == AT_WAVE && lanes[i].state == AT_BLOCK)) continue;
        if (lanes[i].state != state) return false;
        any = true;
    }
    for (uint32_t i = first; any && i < first + n; i++) if (lanes[i].state == state) lanes[i].state = RUN;
    return any;
}
inline void run_block() {
    const uint32_t n = block_dim.x;
    const bool reverse = getenv("SIMT_REVERSE") != nullptr;
    while (lanes.size() < n) {
        char* s = (char*)mmap(nullptr, kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (s == MAP_FAILED) { perror("mmap"); exit(3); }
        lanes.push_back(Lane{});
        lanes.back().stack = s;
    }
    for (uint32_t i = 0; i < n; i++) {
        Lane& l = lanes[i];
        l.id = i; l.state = RUN; l.fake = nullptr; l.there = false;
        void** top = (void**)(l.stack + kStack) - 1;              // first switch: six registers, then a return into enter()
        *top = nullptr;
        *--top = (void*)enter;
        for (int r = 0; r < 6; r++) *--top = nullptr;
        l.sp = top;
    }
    for (;;) {
        for (uint32_t i = 0; i < n; i++) { Lane& l = lanes[reverse ? n - 1 - i : i]; if (l.state == RUN) resume(l); }
        bool opened = false, left = false;
        for (uint32_t i = 0; i < n; i++) left = left || lanes[i].state != ENDED;
        if (!left) return;
        for (uint32_t w = 0; w < n; w += 64) opened = open(w, n - w < 64 ? n - w : 64, AT_WAVE) || opened;
        if (!opened) opened = open(0, n, AT_BLOCK);
        if (!opened) { fprintf(stderr, "simt: lanes of a block stand at different barriers\n"); abort(); }
    }
}
template <class K, class... A>
void launch(K* kernel, dim3 grid, dim3 block, size_t lds, void*, const A&... args) {
    grid_dim = grid; block_dim = block;
    if (getenv("SIMT_TRACE")) fprintf(stderr, "simt: grid %u %u %u block %u lds %zu\n", grid.x, grid.y, grid.z, block.x, lds);
    const void* ptrs[] = {(const void*)&args...};
    kernarg = ptrs[0];
    std::function<void()> f = [&] { kernel(args...); };
    body = &f;
    for (Dynamic& d : dynamic()) {
        if (lds > d.size) { fprintf(stderr, "simt: dynamic LDS\n"); abort(); }
        __asan_unpoison_memory_region(d.p, d.size);
        __asan_poison_memory_region(d.p + lds, d.size - lds);
    }
    for (uint32_t z = 0; z < grid.z; z++) for (uint32_t y = 0; y < grid.y; y++) for (uint32_t x = 0; x < grid.x; x++) {
        block_idx = dim3(x, y, z);
        for (Dynamic& d : dynamic()) memset(d.p, 0xC5, lds);
        run_block();
    }
}
inline int shfl(int v, int src) {
    cur->value = v;
    cur->there = true;
    Lane* wave = &lanes[cur->id & ~63u];
    wait(AT_WAVE);
    if (src < 0 || src > 63 || !wave[src].there) { fprintf(stderr, "simt: shuffle from a lane that is not there\n"); abort(); }
    const int r = wave[src].value;
    wait(AT_WAVE);
    cur->there = false;
    return r;
}
// v_perm_b32
inline uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    uint32_t r = 0;
    for (int i = 0; i < 4; i++) {
        const uint32_t s = (sel >> (8 * i)) & 0xffu;
        if (s < 8) r |= (uint32_t)((v >> (8 * s)) & 0xffu) << (8 * i);
        else if (s != 0x0c) { fprintf(stderr, "simt: permute selector\n"); abort(); }
    }
    return r;
}
inline uint32_t lane_id() { return cur->id & 63u; }
// v_permlane32_swap / v_permlane16_swap: the upper half (odd rows of 16) of a against the lower half (even rows) of b
struct Pair { uint32_t v[2]; uint32_t operator[](int i) const { return v[i]; } };
inline Pair swap(uint32_t a, uint32_t b, uint32_t n) {
    const int l = (int)lane_id(), other = l ^ (int)n;
    const uint32_t oa = (uint32_t)shfl((int)a, other), ob = (uint32_t)shfl((int)b, other);
    return l & (int)n ? Pair{{ob, b}} : Pair{{a, oa}};
}
// the data-parallel permutes that the sources use: row_ror:8 and quad_perm
inline uint32_t dpp(uint32_t v, int ctrl) {
    const int l = (int)lane_id();
    if (ctrl == 0x128) return (uint32_t)shfl((int)v, (l & ~15) | ((l + 8) & 15));
    if (ctrl < 0x100) return (uint32_t)shfl((int)v, (l & ~3) | ((ctrl >> (2 * (l & 3))) & 3));
    abort();
}
// ds_swizzle in bit mode: lane = ((lane & and) | or) ^ xor within 32 lanes
inline uint32_t swizzle(uint32_t v, int pattern) {
    const int l = (int)lane_id();
    return (uint32_t)shfl((int)v, (l & 32) | (((l & pattern & 31) | ((pattern >> 5) & 31)) ^ ((pattern >> 10) & 31)));
}
inline uint32_t udot4(uint32_t a, uint32_t b, uint32_t c) {
    for (int i = 0; i < 32; i += 8) c += ((a >> i) & 0xffu) * ((b >> i) & 0xffu);
    return c;
}
struct Tid { uint32_t x, y, z; };
inline Tid thread_idx() { return Tid{cur->id, 0, 0}; }
}  // namespace simt

#define threadIdx simt::thread_idx()
#define blockIdx simt::block_idx
#define blockDim simt::block_dim
#define gridDim simt::grid_dim
#define hipLaunchKernelGGL(K, G, B, LDS, S, ...) simt::launch(K, G, B, LDS, S, __VA_ARGS__)
#define __syncthreads() simt::wait(simt::AT_BLOCK)
#define __shfl(v, src, width) simt::shfl(v, src)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_perm simt::perm
#define __builtin_amdgcn_udot4(a, b, c, clamp) simt::udot4(a, b, c)
#define __builtin_amdgcn_permlane32_swap(a, b, fi, bc) simt::swap(a, b, 32)
#define __builtin_amdgcn_permlane16_swap(a, b, fi, bc) simt::swap(a, b, 16)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, bc) simt::dpp((uint32_t)(v), ctrl)
#define __builtin_amdgcn_ds_swizzle(v, pattern) simt::swizzle((uint32_t)(v), pattern)
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() simt::wait(simt::AT_WAVE)
#define DASH_WAVE_POINT() simt::wait(simt::AT_WAVE)
#define __builtin_amdgcn_kernarg_segment_ptr() simt::kernarg

typedef int hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;
enum { hipSuccess = 0, hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
#define HIP_SYMBOL(x) x
inline hipError_t hipGetLastError() { return 0; }
// static LDS of a kernel as the device's build has it (SIMT_STATIC_LDS: another)
struct hipFuncAttributes { size_t sharedSizeBytes; };
inline hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
    const char* e = getenv("SIMT_STATIC_LDS");
    a->sharedSizeBytes = e ? (size_t)atoll(e) : 1024;
    return 0;
}
inline hipError_t hipSetDevice(int) { return 0; }
inline hipError_t hipDeviceSynchronize() { return 0; }
template <class T> hipError_t hipMalloc(T** p, size_t n) { void* v; const int st = posix_memalign(&v, 256, n); *p = (T*)v; return st; }
inline hipError_t hipFree(void* p) { free(p); return 0; }
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
inline hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
template <class T> hipError_t hipGetSymbolAddress(void** p, T& sym) { *p = (void*)&sym; return 0; }
inline hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return 0; }
inline hipError_t hipEventDestroy(hipEvent_t) { return 0; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return 0; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return 0; }
inline hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0; return 0; }
