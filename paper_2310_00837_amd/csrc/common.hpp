// Shared device-side helpers of the Helios HIP kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace helios {

constexpr int kBlock = 256;          // threads per workgroup in every kernel
constexpr int kWave = 64;            // CDNA wavefront
constexpr int kWavesPerBlock = kBlock / kWave;

// device-side error codes, same values as helios_status
constexpr int kErrCapacity = -2;
constexpr int kErrData = -5;
constexpr int kErrInternal = -6;

// A count that is known either on the host (dev == nullptr: the count is
// `host`) or only on the device (read from *dev by the kernel and clamped to
// `host`, the most the buffers behind it can hold).
struct Count {
    const int64_t* dev;
    int64_t host;
    __device__ __forceinline__ int64_t get() const {
        if (!dev) return host;
        const int64_t v = *dev;
        return v < host ? (v < 0 ? 0 : v) : host;
    }
};

// What changes from one mini-batch to the next.  Kernels of a recorded (graph) batch read it
// from device memory, so that one recording serves every batch; directly launched kernels get
// the same values as arguments and a null pointer here.
struct BatchVars {
    uint64_t rng_seed;
    const int32_t* seeds;
    uint32_t epoch_base;     // added to the per-launch epoch of the chained scans
    uint32_t io_round;       // round number of the miss queue the batch submits to (0 if none)
    uint32_t table;          // which of the rotating batch tables this batch uses
    uint32_t clear_slots;    // slots in use of the table that the batch's last launch empties (0: it is empty)
};

// How a recorded batch gets its BatchVars without a copy being part of the recording: the host writes
// them to the next slot of a ring in pinned memory before every launch; the workgroups of the batch's
// first kernel read the slot that the number of recorded batches run so far on the context selects (a
// device counter, advanced by the batch's second kernel) and the first of them leaves a copy in device
// memory for the kernels after it.
struct BatchFeed {
    const BatchVars* ring;        // pinned host memory, nullable (a directly launched batch)
    uint32_t ring_slots;
    const uint32_t* batches_run;  // device
    BatchVars* vars_out;          // device
};

// First error wins is not needed: any recorded error makes the call fail.
// err points to pinned, GPU-mapped host memory (int32[2]: code, detail).
__device__ __forceinline__ void raise(int32_t* err, int code) {
    *reinterpret_cast<volatile int32_t*>(err) = code;
}

// A role is a range of the workgroups of a launch that does one job; several roles share a launch
// when their jobs are independent and bound by different things (the host link, HBM, latency).
// Workgroup blockIdx.x belongs to the role with first <= blockIdx.x < first + blocks and is its
// workgroup number blockIdx.x - first.
struct Role {
    uint32_t first, blocks;
    __device__ __forceinline__ bool mine() const { return blockIdx.x - first < blocks; }   // unsigned wrap-around
    __device__ __forceinline__ uint32_t rb() const { return blockIdx.x - first; }
};
constexpr unsigned kMaxRoleBlocks = 32768;

// Optional timing of a role: workgroup rb of nrb stores its first and last tick of the constant-rate
// device clock at clock[rb] and clock[nrb + rb] (plain stores, no contention); a publish kernel
// reduces them to {earliest start, latest end} in pinned host memory.
struct Stamps {
    unsigned long long* clock;     // nullable
};
__device__ __forceinline__ void stamp_start(const Stamps& s, uint32_t rb) {
    if (s.clock && threadIdx.x == 0) s.clock[rb] = wall_clock64();
}
__device__ __forceinline__ void stamp_end(const Stamps& s, uint32_t rb, uint32_t nrb) {
    if (s.clock) {
        __syncthreads();
        if (threadIdx.x == 0) s.clock[nrb + rb] = wall_clock64();
    }
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

// Inclusive scan over the 64 lanes of a wave by DPP moves, without a trip through LDS per step: four shifts inside the
// rows of 16 lanes, then the last lane of a row is carried into the rows after it.
__device__ __forceinline__ uint32_t dpp_inclusive_scan(uint32_t v) {
    const auto add = [](uint32_t x, int moved) { return x + static_cast<uint32_t>(moved); };
    v = add(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xf, 0xf, false));      // row_shr:1
    v = add(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xf, 0xf, false));      // row_shr:2
    v = add(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xf, 0xf, false));      // row_shr:4
    v = add(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xf, 0xf, false));      // row_shr:8
    v = add(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xa, 0xf, false));      // row_bcast:15 into rows 1, 3
    v = add(v, __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xc, 0xf, false));      // row_bcast:31 into rows 2, 3
    return v;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) {      // lane: the same in all lanes
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), static_cast<int>(lane)));
}
__device__ __forceinline__ uint32_t dpp_sum(uint32_t v) { return lane_value(dpp_inclusive_scan(v), kWave - 1); }
// Lane LANE's value for all lanes of its group of G lanes (8 or 16), by DPP.
template <int G, int LANE>
__device__ __forceinline__ int32_t group_value(int32_t v) {
    static_assert((G == 8 || G == 16) && LANE < G, "a row has 16 lanes");
    if constexpr (G == 16) return __builtin_amdgcn_update_dpp(v, v, 0x150 + LANE, 0xf, 0xf, false);      // row_newbcast
    const int lower = __builtin_amdgcn_update_dpp(v, v, 0x150 + LANE, 0xf, 0x3, false);                  // into lanes 0-7 of a row
    return __builtin_amdgcn_update_dpp(lower, v, 0x158 + (LANE & 7), 0xf, 0xc, false);                   // and into lanes 8-15
}
// ... of 32 or 64 lanes, by the scalar unit; lane is the same in all lanes
template <int G>
__device__ __forceinline__ int32_t group_value(int32_t v, int lane) {
    static_assert(G == 32 || G == 64, "smaller groups use DPP");
    if constexpr (G == 64) return __builtin_amdgcn_readlane(v, lane);
    const int lower = __builtin_amdgcn_readlane(v, lane), upper = __builtin_amdgcn_readlane(v, 32 + lane);
    return (threadIdx.x & 32) ? upper : lower;
}
// how many lanes below this one are set in the mask
__device__ __forceinline__ uint32_t rank_in_mask(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// The bounds of a CSR row, read as one 16-byte access (the two words are adjacent, 8-byte aligned).
struct RowBounds {
    int64_t lo, hi;
};
__device__ __forceinline__ RowBounds row_bounds(const int64_t* offsets, uint32_t v) {
    typedef int64_t pair __attribute__((ext_vector_type(2), aligned(8)));
    const pair p = *reinterpret_cast<const pair*>(offsets + v);
    return RowBounds{p.x, p.y};
}

}  // namespace helios
