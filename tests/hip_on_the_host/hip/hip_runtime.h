// Stand-in for the HIP runtime header with which clang++ compiles a .hip file of this library for the host, so that a kernel can be
// run without a GPU, on whatever its scratch memory holds.  The workgroups of a launch run one after the other; the threads of a
// workgroup are coroutines that run until they meet a barrier or an operation of the whole wave (a ballot, a DPP move), where they
// wait for the others of the workgroup or the wave.  __shared__ variables are static ones.  Only what the kernels under test use.
// Of one range of memory (on_host::cached) atomic loads of a workgroup's scope see what a cache may hold: workgroup b belongs to cache b
// modulo 8, which keeps a line of 128 bytes as it was when it was first loaded in the launch, until the same cache's workgroups store there.
#pragma once
#include <setjmp.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <string.h>

#include <functional>
#include <unordered_map>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define asm                         // (barriers of the optimiser, `asm volatile("" : "+v"(x))`: nothing)
#define volatile(...)

typedef int hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;
constexpr hipError_t hipSuccess = 0, hipErrorInvalidValue = 1;
enum hipMemcpyKind { hipMemcpyDefault = 4 };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* to, const void* from, size_t bytes, hipMemcpyKind, hipStream_t) {
    memmove(to, from, bytes);
    return hipSuccess;
}

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
inline dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace on_host {
constexpr unsigned kLanes = 64;
struct Meeting {                    // of the threads that are left of a workgroup or a wave
    unsigned left = 0, here = 0, turn = 0;
    int64_t value[2][kLanes];       // by parity of the turn, so that a thread may still read one while the next fills
    uint64_t lanes[2] = {0, 0};
    void arrive_all() {
        if (here == 0 || here < left) return;
        here = 0;
        ++turn;
        lanes[turn & 1] = 0;
    }
};
struct Thread {
    ucontext_t first;
    jmp_buf at;
    bool begun, done;
};
constexpr size_t kStack = 64 << 10;
inline std::vector<Thread> threads;
inline std::vector<char> stacks;
inline Meeting group;
inline std::vector<Meeting> waves;
inline jmp_buf scheduler;
inline unsigned now;
inline const std::function<void()>* body;

constexpr unsigned kCaches = 8;
constexpr uintptr_t kLine = 128;
struct Line {
    char bytes[kLine];
    bool there = false;
};
inline std::unordered_map<const char*, Line> caches[kCaches];
inline struct { const char *begin = nullptr, *end = nullptr; } cached;

inline void give_way() {
    if (_setjmp(threads[now].at) == 0) _longjmp(scheduler, 1);
}
inline unsigned meet(Meeting& m) {
    const unsigned turn = m.turn;
    ++m.here;
    m.arrive_all();
    while (m.turn == turn) give_way();
    return turn & 1;
}
// every lane's value, and which lanes there are
inline const int64_t* exchange(int64_t v, uint64_t* lanes) {
    Meeting& m = waves[now / kLanes];
    m.value[m.turn & 1][now % kLanes] = v;
    m.lanes[m.turn & 1] |= uint64_t{1} << (now % kLanes);
    const unsigned which = meet(m);
    *lanes = m.lanes[which];
    return m.value[which];
}
inline void run_thread() {
    (*body)();
    threads[now].done = true;
    for (Meeting* m : {&group, &waves[now / kLanes]}) {
        --m->left;
        m->arrive_all();
    }
    _longjmp(scheduler, 1);
}
inline void run_workgroup(unsigned block, unsigned grid, unsigned size, const std::function<void()>& f) {
    body = &f;
    threads.resize(size);
    stacks.resize(size * kStack);
    waves.assign((size + kLanes - 1) / kLanes, Meeting{});
    group = Meeting{};
    group.left = size;
    for (unsigned t = 0; t < size; ++t) {
        waves[t / kLanes].left += 1;
        threads[t].begun = threads[t].done = false;
        getcontext(&threads[t].first);
        threads[t].first.uc_stack.ss_sp = stacks.data() + t * kStack;
        threads[t].first.uc_stack.ss_size = kStack;
        threads[t].first.uc_link = nullptr;
        makecontext(&threads[t].first, run_thread, 0);
    }
    blockDim = dim3(size);
    gridDim = dim3(grid);
    blockIdx = dim3(block);
    while (group.left > 0) {
        for (now = 0; now < threads.size(); ++now) {
            if (threads[now].done) continue;
            threadIdx = dim3(now);
            if (_setjmp(scheduler) != 0) continue;           // it has given way, or has ended
            if (threads[now].begun) _longjmp(threads[now].at, 1);
            threads[now].begun = true;
            setcontext(&threads[now].first);
        }
    }
}
template <class F>
void launch(dim3 grid, dim3 block, const F& f) {
    const std::function<void()> g = f;
    for (auto& c : caches) c.clear();
    for (unsigned b = 0; b < grid.x; ++b) run_workgroup(b, grid.x, block.x, g);
}
}  // namespace on_host

#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) on_host::launch(grid, block, [=]() { (kernel)(__VA_ARGS__); })

inline void __syncthreads() { on_host::meet(on_host::group); }
inline uint64_t __ballot(bool v) {
    uint64_t lanes, ones = 0;
    const int64_t* all = on_host::exchange(v, &lanes);
    for (unsigned l = 0; l < on_host::kLanes; ++l)
        if (((lanes >> l) & 1) && all[l]) ones |= uint64_t{1} << l;
    return ones;
}
inline int on_host_readlane(int v, int lane) {
    uint64_t lanes;
    return static_cast<int>(on_host::exchange(v, &lanes)[lane]);
}
inline int on_host_dpp(int old, int v, int ctrl, int row_mask, int bank_mask, bool) {
    uint64_t lanes;
    const int64_t* all = on_host::exchange(v, &lanes);
    const int lane = static_cast<int>(on_host::now % on_host::kLanes), row = lane / 16, in_row = lane % 16;
    int from = -1;
    if (ctrl > 0x110 && ctrl < 0x120) from = in_row >= ctrl - 0x110 ? lane - (ctrl - 0x110) : -1;       // row_shr
    else if (ctrl == 0x142) from = row > 0 ? row * 16 - 1 : -1;                                         // row_bcast:15
    else if (ctrl == 0x143) from = row >= 2 ? 31 : -1;                                                  // row_bcast:31
    else if (ctrl >= 0x150 && ctrl < 0x160) from = row * 16 + (ctrl - 0x150);                           // row_newbcast
    else abort();
    const bool on = ((row_mask >> row) & 1) && ((bank_mask >> (in_row / 4)) & 1);
    return on && from >= 0 && ((lanes >> from) & 1) ? static_cast<int>(all[from]) : old;
}
inline unsigned on_host_mbcnt(unsigned mask, unsigned v, unsigned first) {
    const unsigned lane = on_host::now % on_host::kLanes;
    const unsigned below = lane <= first ? 0u : lane - first >= 32 ? ~0u : (1u << (lane - first)) - 1u;
    return v + static_cast<unsigned>(__builtin_popcount(mask & below));
}
#define __builtin_amdgcn_readlane on_host_readlane
#define __builtin_amdgcn_readfirstlane(v) (v)                  // (used on values that are the same in all lanes, unless the test has its own)
#define __builtin_amdgcn_update_dpp on_host_dpp
#define __builtin_amdgcn_mbcnt_lo(mask, v) on_host_mbcnt(mask, v, 0)
#define __builtin_amdgcn_mbcnt_hi(mask, v) on_host_mbcnt(mask, v, 32)
#define __builtin_amdgcn_s_sleep(n) on_host::give_way()
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)on_host::meet(on_host::waves[on_host::now / on_host::kLanes]))
template <class T>
T __shfl_xor(T v, int d, int) {
    uint64_t lanes;
    return static_cast<T>(on_host::exchange(v, &lanes)[(on_host::now % on_host::kLanes) ^ d]);
}
template <class T>
T __shfl_up(T v, unsigned d, int) {
    uint64_t lanes;
    const unsigned lane = on_host::now % on_host::kLanes;
    const int64_t* all = on_host::exchange(v, &lanes);
    return lane < d ? v : static_cast<T>(all[lane - d]);
}
inline int on_host_sbfe(int v, unsigned at, unsigned bits) { return (v << (32 - at - bits)) >> (32 - bits); }
inline uint32_t on_host_bitop3(uint32_t x, uint32_t y, uint32_t z, int table) {
    uint32_t r = 0;
    for (int q = 0; q < 8; ++q)
        if ((table >> q) & 1) r |= (q & 4 ? x : ~x) & (q & 2 ? y : ~y) & (q & 1 ? z : ~z);
    return r;
}
#define __builtin_amdgcn_sbfe on_host_sbfe
#define __builtin_amdgcn_bitop3_b32 on_host_bitop3
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }
inline uint64_t wall_clock64() { return 0; }
template <class T>
T min(T a, T b) { return a < b ? a : b; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return static_cast<uint32_t>((static_cast<uint64_t>(a) * b) >> 32); }
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __HIP_MEMORY_SCOPE_AGENT 1
#define __HIP_MEMORY_SCOPE_SYSTEM 2
#define __hip_atomic_load(p, order, scope) on_host::load(p, scope)
#define __hip_atomic_store(p, v, order, scope) on_host::store(p, v)
#define __hip_atomic_fetch_add(p, v, order, scope) atomicAdd(p, v)
namespace on_host {
template <class T>
T load(const T* p, int scope) {
    const char* at = reinterpret_cast<const char*>(p);
    if (scope != __HIP_MEMORY_SCOPE_WORKGROUP || at < cached.begin || at >= cached.end) return *p;
    const uintptr_t offset = reinterpret_cast<uintptr_t>(p) % kLine;
    Line& line = caches[blockIdx.x % kCaches].try_emplace(at - offset).first->second;
    if (!line.there) memcpy(line.bytes, at - offset, kLine);
    line.there = true;
    T v;
    memcpy(&v, line.bytes + offset, sizeof(T));
    return v;
}
template <class T, class V>
void store(T* p, V v) {
    *p = v;
    const char* at = reinterpret_cast<const char*>(p);
    const uintptr_t offset = reinterpret_cast<uintptr_t>(p) % kLine;
    const auto line = caches[blockIdx.x % kCaches].find(at - offset);
    if (line != caches[blockIdx.x % kCaches].end()) memcpy(line->second.bytes + offset, p, sizeof(T));
}
}  // namespace on_host
template <class T>
T atomicAdd(T* p, T v) { const T was = *p; *p = was + v; return was; }
template <class T>
T atomicMin(T* p, T v) { const T was = *p; *p = v < was ? v : was; return was; }
template <class T>
T atomicOr(T* p, T v) { const T was = *p; *p = was | v; return was; }
template <class T>
T atomicCAS(T* p, T want, T v) { const T was = *p; if (was == want) *p = v; return was; }
