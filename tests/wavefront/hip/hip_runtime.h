// A wavefront of 64 lanes on the CPU: enough of the HIP language to compile a kernel of one-wavefront blocks from its own source
// and to run it lane by lane with every access to LDS checked.  Test infrastructure; never part of the library.
//
// Each lane is a fiber.  It runs until its next operation that involves other lanes (ballot, shuffle, DPP move, barrier) and
// waits there; the lanes that wait at the place that comes first in the program go on together, as lanes of a wavefront whose
// paths have parted do.  "First in the program" is the order of the return addresses from the kernel's frame inward, which is
// the order of the source without optimisation (build with -O0).
//
// LDS is reached through lds_at.  Reported, with the first of them kept as text: accesses past the allocation or not aligned to
// their type, reads of bytes that nobody has written and, if asked for, bytes used as two types neither of which may alias the other.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

typedef int hipError_t;
typedef void *hipStream_t;
constexpr hipError_t hipSuccess = 0;
inline hipError_t hipGetLastError() { return hipSuccess; }
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
struct int4 { int x, y, z, w; };
inline int4 make_int4(int x, int y, int z, int w) { return int4{x, y, z, w}; }
inline struct { unsigned x, y, z; } threadIdx, blockIdx, gridDim, blockDim;

namespace emu {

constexpr int kLanes = 64, kDepth = 24;
constexpr size_t kStack = 128 * 1024;

struct Lane {
    void *sp;
    char *stack;
    bool done;
    uintptr_t *frame;                    // of the function that calls the kernel
    uintptr_t key[kDepth];               // return addresses from the kernel's frame inward
    int depth;
    uint32_t give;                       // operand of the operation it waits in
};
inline Lane lanes[kLanes];
inline void *scheduler_sp;
inline int self;                         // the lane that runs
inline uint64_t group;                   // lanes that take the operation together
inline uint32_t given[kLanes];
inline void (*body)(void *);
inline void *body_arg;

// ---- what a test asks for and learns
inline int64_t waits, reads, wait_limit;  // operations, reads of LDS by one lane since the last of its own; most operations a launch may take
constexpr int64_t kReadLimit = 1 << 20;  // most such reads
inline bool backwards;                   // lanes between two operations run in falling order
inline int32_t *clear;                    // a word of memory that becomes 0 after so many operations (null: none)
inline int64_t clear_at;
inline int64_t poke_at, poke_place, poke_value, poke_size;   // after so many operations (0: never) some bytes of LDS are overwritten
inline bool types;                                   // report bytes used as two types
inline int faults;
inline char first_fault[256];
inline bool stopped;

inline std::vector<unsigned char> lds;
inline std::vector<const void *> type_of;            // per byte: the type it is used as (null: never written)
inline std::vector<char> aliases;

inline void fault(const char *what, int64_t at, int size)
{
    if (faults++ == 0) snprintf(first_fault, sizeof first_fault, "%s: %d bytes at %lld of %zu, lane %d", what, size, static_cast<long long>(at), lds.size(), self);
}

// switches stacks; callee-saved registers travel on them
__attribute__((naked)) inline void swap_stacks(void ** /* keep */, void * /* next */)
{
    __asm__("pushq %rbp\n pushq %rbx\n pushq %r12\n pushq %r13\n pushq %r14\n pushq %r15\n movq %rsp, (%rdi)\n movq %rsi, %rsp\n"
            "popq %r15\n popq %r14\n popq %r13\n popq %r12\n popq %rbx\n popq %rbp\n retq\n");
}

__attribute__((noinline)) inline void lane_main()
{
    Lane &l = lanes[self];
    l.frame = static_cast<uintptr_t *>(__builtin_frame_address(0));
    body(body_arg);
    lanes[self].done = true;
    swap_stacks(&lanes[self].sp, scheduler_sp);
    abort();
}

__attribute__((noinline)) inline void wait_here(uint32_t give)
{
    Lane &l = lanes[self];
    uintptr_t chain[kDepth];
    int n = 0;
    for (uintptr_t *f = static_cast<uintptr_t *>(__builtin_frame_address(0)); f != l.frame && n < kDepth; f = reinterpret_cast<uintptr_t *>(f[0]))
        chain[n++] = f[1];
    l.depth = n;
    for (int i = 0; i < n; ++i) l.key[i] = chain[n - 1 - i];
    l.give = give;
    swap_stacks(&l.sp, scheduler_sp);
}

inline int compare(const Lane &a, const Lane &b)
{
    for (int i = 0; i < a.depth && i < b.depth; ++i)
        if (a.key[i] != b.key[i]) return a.key[i] < b.key[i] ? -1 : 1;
    return a.depth - b.depth;
}

inline void run_wavefront()
{
    for (int i = 0; i < kLanes; ++i) {
        Lane &l = lanes[i];
        if (!l.stack) l.stack = static_cast<char *>(malloc(kStack));
        void **top = reinterpret_cast<void **>(reinterpret_cast<uintptr_t>(l.stack + kStack) & ~uintptr_t(63)) - 2;
        *--top = nullptr;                                        // lane_main's return address (never used)
        *--top = reinterpret_cast<void *>(&lane_main);
        for (int r = 0; r < 6; ++r) *--top = nullptr;
        l.sp = top;
        l.done = false; l.depth = 0;
    }
    uint64_t next = ~uint64_t(0);
    while (next != 0) {
        group = next;
        for (int i = 0; i < kLanes; ++i) given[i] = lanes[i].give;
        for (int k = 0; k < kLanes; ++k) {
            const int i = backwards ? kLanes - 1 - k : k;
            if (!(next >> i & 1)) continue;
            self = i; threadIdx.x = static_cast<unsigned>(i);
            reads = 0;
            swap_stacks(&scheduler_sp, lanes[i].sp);
            if (stopped) return;
        }
        int first = -1;
        next = 0;
        for (int i = 0; i < kLanes; ++i) {
            if (lanes[i].done) continue;
            const int c = first < 0 ? -1 : compare(lanes[i], lanes[first]);
            if (c < 0) { first = i; next = 0; }
            if (c <= 0) next |= uint64_t(1) << i;
        }
        ++waits;
        if (clear != nullptr && waits >= clear_at) *clear = 0;
        if (poke_at != 0 && waits == poke_at) memcpy(lds.data() + poke_place, &poke_value, static_cast<size_t>(poke_size));
        if (waits > wait_limit) { stopped = true; return; }
    }
}

template <typename F> inline void launch(dim3 grid, dim3 block, size_t lds_bytes, F kernel)
{
    if (block.x != kLanes) { fault("launch of a block that is no wavefront", 0, static_cast<int>(block.x)); return; }
    body = [](void *f) { (*static_cast<F *>(f))(); };
    body_arg = &kernel;
    gridDim.x = grid.x; blockDim.x = block.x;
    for (unsigned b = 0; b < grid.x && !stopped; ++b) {
        lds.assign(lds_bytes, 0xA5);
        type_of.assign(lds_bytes, nullptr);
        aliases.assign(lds_bytes, 0);
        blockIdx.x = b;
        run_wavefront();
    }
}

// ---- LDS
template <typename T> inline const void *type_id() { static const char id = 0; return &id; }
template <typename T> struct MayAlias { static constexpr bool value = std::is_class<T>::value || !std::is_arithmetic<T>::value; };   // structures and vectors declared so
template <typename T> inline bool reachable(int64_t at, const char *what)
{
    if (at < 0 || at + static_cast<int64_t>(sizeof(T)) > static_cast<int64_t>(lds.size())) { fault(what, at, sizeof(T)); return false; }
    if (at % static_cast<int64_t>(sizeof(T) < 8 ? sizeof(T) : 8) != 0) fault("not aligned", at, sizeof(T));
    return true;
}
template <typename T> struct Ref {
    int64_t at;
    operator T() const
    {
        if (++reads > kReadLimit) { stopped = true; swap_stacks(&lanes[self].sp, scheduler_sp); }      // and never comes back
        T v{};
        if (!reachable<T>(at, "read past the end")) return v;
        for (size_t i = 0; i < sizeof(T); ++i) {
            if (!type_of[at + i]) { fault("read of what nobody wrote", at, sizeof(T)); break; }
            if (types && type_of[at + i] != type_id<T>() && !MayAlias<T>::value && !aliases[at + i]) { fault("read as another type", at, sizeof(T)); break; }
        }
        memcpy(&v, lds.data() + at, sizeof(T));
        return v;
    }
    const Ref &operator=(T v) const
    {
        if (!reachable<T>(at, "write past the end")) return *this;
        for (size_t i = 0; i < sizeof(T); ++i) {
            if (types && type_of[at + i] && type_of[at + i] != type_id<T>() && !MayAlias<T>::value && !aliases[at + i]) { fault("written as another type", at, sizeof(T)); break; }
            if (!type_of[at + i] || !MayAlias<T>::value) { type_of[at + i] = type_id<T>(); aliases[at + i] = MayAlias<T>::value; }
        }
        memcpy(lds.data() + at, &v, sizeof(T));
        return *this;
    }
    const Ref &operator=(const Ref &o) const { return *this = static_cast<T>(o); }
};
template <typename T> struct Ptr { int64_t at; Ref<T> operator*() const { return Ref<T>{at}; } };

// ---- operations that involve other lanes
inline bool taking(int i) { return i >= 0 && i < kLanes && (group >> i & 1) != 0; }
__attribute__((noinline)) inline uint64_t ballot(int pred)
{
    wait_here(pred != 0);
    uint64_t m = 0;
    for (int i = 0; i < kLanes; ++i) if (taking(i) && given[i]) m |= uint64_t(1) << i;
    return m;
}
__attribute__((noinline)) inline uint32_t from(uint32_t v, int lane)      // of a lane that does not take part: 0
{
    wait_here(v);
    return taking(lane) ? given[lane] : 0;
}
__attribute__((noinline)) inline uint32_t from_first(uint32_t v)
{
    wait_here(v);
    return given[__builtin_ctzll(group)];
}
__attribute__((noinline)) inline int dpp(int v, int ctrl)
{
    const int row = self & ~15, in = self & 15;
    int src = -1;
    if (ctrl < 0x100) src = (self & ~3) | (ctrl >> (2 * (self & 3)) & 3);
    else if (ctrl > 0x120 && ctrl < 0x130) src = row | ((in - (ctrl & 15)) & 15);
    else if (ctrl == 0x134) src = (self + 1) & 63;
    else if (ctrl == 0x13C) src = (self - 1) & 63;
    else fault("DPP control that is not emulated", ctrl, 0);
    return static_cast<int>(from(static_cast<uint32_t>(v), src));
}
__attribute__((noinline)) inline void barrier() { wait_here(0); }
inline int mbcnt(uint32_t mask, int base) { return __builtin_popcount(mask & (self - base >= 32 ? ~0u : self - base <= 0 ? 0u : (1u << (self - base)) - 1)); }

}  // namespace emu

#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
    do { (void)(stream); emu::launch(grid, block, lds, [&] { (kernel)(__VA_ARGS__); }); } while (0)

#define __ballot(p) emu::ballot(p)
#define __syncthreads() emu::barrier()
#define __popcll(v) __builtin_popcountll(v)
template <typename T> inline T __shfl(T v, int lane, int width = 64)
{
    static_assert(sizeof(T) == 4, "32-bit values");
    return static_cast<T>(emu::from(static_cast<uint32_t>(v), (emu::self & ~(width - 1)) | (lane & (width - 1))));
}
template <typename T> inline T __shfl_up(T v, int n, int = 64) { abort(); (void)n; return v; }
template <typename T> inline T __shfl_xor(T v, int n, int = 64) { abort(); (void)n; return v; }
template <typename T, typename U> inline T atomicAdd(T *p, U v) { const T old = *p; *p = static_cast<T>(old + v); return old; }
#define __builtin_amdgcn_wave_barrier() emu::barrier()
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, zero) emu::dpp(v, ctrl)
#define __builtin_amdgcn_readfirstlane(v) static_cast<int>(emu::from_first(static_cast<uint32_t>(v)))
#define __builtin_amdgcn_readlane(v, lane) static_cast<int>(emu::from(static_cast<uint32_t>(v), lane))
#define __builtin_amdgcn_mbcnt_lo(mask, add) (emu::mbcnt(mask, 0) + (add))
#define __builtin_amdgcn_mbcnt_hi(mask, add) (emu::mbcnt(mask, 32) + (add))
#define __builtin_amdgcn_ubfe(v, at, n) (static_cast<uint32_t>(v) >> ((at) & 31) & ((1u << (n)) - 1))
#define __hip_atomic_load(p, order, scope) (*(p))

#define PRS_LDS_AT
namespace prs { template <typename T> inline emu::Ptr<T> lds_at(int32_t at) { return emu::Ptr<T>{at}; } }
