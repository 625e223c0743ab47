// Single-pass chained prefix sum across workgroups (decoupled look-back).
//
// A workgroup takes tiles in start order from a ticket counter.  A tile publishes
// its aggregate, then looks back over its predecessors, 256 at a time, until it
// meets one that has published a full inclusive prefix.  One 64-bit status word
// per tile and counter holds {epoch:30, flag:2, value:32}; the epoch changes on
// every launch, so a stale word reads as "not published" and the buffer never
// needs clearing between launches.
//
// Why tickets: a tile waits only for tiles with a smaller index, and with
// tickets those have all started already, whatever else runs on the GPU.  With
// tile = workgroup index that is not so once several scan kernels from
// different streams oversubscribe the chip: the waiting workgroups of one
// kernel can hold the slots of an XCD on which another kernel's lower tile is
// still to start, and the other way round (seen on this part with six streams:
// the bounded wait below fired).  The price is one device-scope atomic on one
// address per tile: 0.2 us, and about 10 ns more for each ticket beyond a few
// hundred that are drawn at the same time.
//
// The wait is bounded all the same: after kScanSpinBudget polls a tile gives up,
// records kErrInternal and carries on with a zero, so a launch always drains
// and the caller gets an error instead of a hang.
#pragma once
#include "common.hpp"

namespace helios {

struct ScanState {
    unsigned long long* status;   // [n_counters][stride]
    uint32_t* ticket;             // one counter, zero between launches
    uint32_t stride;              // tiles the status rows have room for
    uint32_t epoch;               // 1 .. 2^30-1, new for every launch
    const BatchVars* vars;        // nullable: if set, vars->epoch_base is added to epoch on the device
};

// the launch's epoch: the argument, plus the batch's base when the launch is part of a recorded batch
__device__ __forceinline__ ScanState scan_resolve(ScanState st) {
    if (st.vars) st.epoch += st.vars->epoch_base;
    return st;
}

constexpr uint32_t kFlagAggregate = 1u;
constexpr uint32_t kFlagPrefix = 2u;

__device__ __forceinline__ unsigned long long scan_pack(uint32_t epoch, uint32_t flag, uint32_t v) {
    return (static_cast<unsigned long long>(epoch) << 34) | (static_cast<unsigned long long>(flag) << 32) | v;
}

__device__ __forceinline__ void scan_store(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long scan_load(unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr uint32_t kScanSpinBudget = 1u << 20;     // polls of one status word before giving up (about a second)

// ---- the scan of one tile
//
// Tiles are K * kScanBlock items: item k of a thread is item k * kScanBlock + threadIdx.x of the tile, so reads are
// coalesced and the items of a wave are consecutive.  The waves put their totals into LDS; after one barrier wave c
// publishes counter c's tile total and looks back for it (all counters at the same time, each by a wave of its own, four
// words per lane in flight), while the others work out their place inside the tile; a second barrier ends it.
//
// Why one item per thread: a compaction is a chain of dependent steps on a nearly idle GPU, and what a wave spends on it
// is instructions one after the other (4 to 16 cycles each), not memory bandwidth.  With one item per thread the chain is a
// quarter as long as with four, and the waves of a SIMD fill each other's gaps.  Measured, second compaction of a batch of
// 40 k IDs: 8.1 us with 512 threads, 8.5 with 256, 9.0 with 1024 (four items on each of 256 threads: 13.6).  Beyond 256 tiles
// the tickets (about 10 ns each) and the look-back become the longest part, so a longer list takes four items per thread, and in the
// compactions of a batch two up to 262 144, where four would leave half of the CUs without a tile (three hops of 1024 seeds, all rows in HBM,
// 54.2 -> 52.2 us a batch; the lookup of a gather, with three counters and nothing beside it, 115 -> 117 us with two: left at four);
// which it is, the device decides by the actual length.
constexpr int kScanBlock = 512;
constexpr int kScanWaves = kScanBlock / kWave;
constexpr int kScanMaxItems = 4;
constexpr uint32_t kScanOneItemMax = 256 * kScanBlock;       // longest list with one item per thread
static_assert(kScanMaxItems * kScanWaves <= kWave, "a wave scans the totals of a tile's waves in one step");
// Workgroups of a scan over a list of at most n_max items.  They take tiles until none is left, so a grid need not cover the
// worst case: an idle workgroup costs about 2 ns of the launch, and the bound of a batch's lists is several times their
// length (two compactions of four batches, 82 tiles in each: 13.0 us with 128 workgroups per batch, 15.6 with 500).
inline unsigned scan_workgroups(int64_t n_max, unsigned limit) {
    const int64_t tiles = (n_max + kScanBlock - 1) / kScanBlock;
    return static_cast<unsigned>(tiles < 1 ? 1 : tiles > limit ? limit : tiles);
}
constexpr unsigned kScanMaxWorkgroups = 512;
// status words a row needs for lists of up to n_max items
inline uint32_t scan_row_stride(int64_t n_max) { return static_cast<uint32_t>(n_max / kScanBlock + 2); }

// One counter of the chained scan, by one whole wave: publishes the tile's total, sums the totals of the tiles before it
// back to the nearest published prefix, publishes this tile's prefix.  Returns the sum over all earlier tiles.
__device__ __forceinline__ uint32_t scan_lookback(const ScanState& st, uint32_t counter, uint32_t tile, uint32_t total, int32_t* err) {
    unsigned long long* row = st.status + static_cast<size_t>(counter) * st.stride;
    const uint32_t lane = static_cast<uint32_t>(lane_id());
    if (lane == 0) scan_store(row + tile, scan_pack(st.epoch, tile == 0 ? kFlagPrefix : kFlagAggregate, total));
    if (tile == 0) return 0;
    constexpr int kAhead = 4;
    uint32_t excl = 0;
    int32_t nearest = static_cast<int32_t>(tile) - 1 - static_cast<int32_t>(lane);      // lane l looks at the l-th predecessor
    for (bool done = false; !done; nearest -= kAhead * kWave) {
        unsigned long long w[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int32_t idx = nearest - q * kWave;
            w[q] = scan_load(row + (idx < 0 ? 0 : idx));
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            if (done) break;                                       // uniform: the nearest prefix was in an earlier window
            const int32_t idx = nearest - q * kWave;
            uint32_t budget = kScanSpinBudget;
            uint64_t ready, prefix;
            while (true) {
                // places before tile 0 act as an empty prefix; a word of an older epoch is not published yet
                const uint32_t flag = idx < 0 ? kFlagPrefix
                                      : static_cast<uint32_t>(w[q] >> 34) == st.epoch ? static_cast<uint32_t>(w[q] >> 32) & 3u : 0u;
                ready = __ballot(flag != 0);
                prefix = __ballot(flag == kFlagPrefix);
                // enough: every place up to the nearest prefix has been published
                if (prefix ? (ready | ~(((prefix & (~prefix + 1)) << 1) - 1)) == ~0ull : ready == ~0ull) break;
                if (--budget == 0) {                               // gave up: report, and let the launch drain
                    if (lane == 0) raise(err, kErrInternal);
                    prefix = 1;
                    w[q] = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                w[q] = scan_load(row + (idx < 0 ? 0 : idx));
            }
            const uint32_t value = idx < 0 ? 0u : static_cast<uint32_t>(w[q]);
            const uint64_t upto = prefix ? ((prefix & (~prefix + 1)) << 1) - 1 : ~0ull;   // lanes up to the nearest prefix
            excl += dpp_sum((upto >> lane) & 1u ? value : 0u);
            done = prefix != 0;
        }
    }
    if (lane == 0) scan_store(row + tile, scan_pack(st.epoch, kFlagPrefix, excl + total));
    return excl;
}

// NP rows of per-wave totals feed NC counters: counter c is row c, except that with NC == NP + 1 the last row holds two
// counters of 16 bits.
template <int NP, int NC, int K>
struct TileScan {
    static_assert(NC == NP || NC == NP + 1, "one row may be a pair");
    static_assert(NC == NP || K * kScanBlock < 65536, "a tile's items can be counted in half a word");
    struct Lds {
        uint32_t total[NP][K * kScanWaves];
        uint32_t excl[NC], agg[NC];
        uint32_t ticket;
    };
    static __device__ __forceinline__ uint32_t pick(uint32_t row_value, int c) {
        if (NC == NP || c < NP - 1) return row_value;
        return c == NP - 1 ? row_value & 0xffffu : row_value >> 16;
    }
    // The next tile of this workgroup, in the start order of all tiles (head of this file); >= n_tiles: none is left.
    // The caller lets the workgroups 0 .. n_wgs-1 take part (n_wgs <= n_tiles) and calls again until none is left; with as many
    // workgroups as tiles one call is enough.  Every draw is counted, so the last one puts the counter back to zero.
    static __device__ __forceinline__ uint32_t take_ticket(const ScanState& st, uint32_t n_tiles, uint32_t n_wgs, Lds& lds) {
        if (n_tiles == 1) return 0;
        if (threadIdx.x == 0) {
            const uint32_t t = atomicAdd(st.ticket, 1u);
            const uint32_t draws = n_wgs < n_tiles ? n_tiles + n_wgs : n_tiles;
            if (t == draws - 1) __hip_atomic_store(st.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            lds.ticket = t;
        }
        __syncthreads();
        return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(lds.ticket)));
    }
    // totals[p][k]: what this wave's k-th run of 64 items adds to row p (the same in all lanes).  before[p][k] = the sum
    // of row p over the tile's items before that run; lds.excl[c] / lds.agg[c] = counter c over the tiles before, and in
    // this tile.  st is resolved (its epoch is the launch's).
    static __device__ __forceinline__ void run(const ScanState& st, uint32_t tile, const uint32_t (&totals)[NP][K], uint32_t (&before)[NP][K],
                                               Lds& lds, int32_t* err) {
        const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave_id()));
        const uint32_t lane = static_cast<uint32_t>(lane_id());
        if (lane == 0) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int k = 0; k < K; ++k) lds.total[p][k * kScanWaves + wave] = totals[p][k];
        }
        __syncthreads();
        if (wave < NC) {
            const int c = static_cast<int>(wave);
            const int p = c < NP ? c : NP - 1;
            const uint32_t mine = lane < K * kScanWaves ? pick(lds.total[p][lane], c) : 0u;
            const uint32_t agg = dpp_sum(mine);
            const uint32_t excl = scan_lookback(st, wave, tile, agg, err);
            if (lane == 0) {
                lds.excl[c] = excl;
                lds.agg[c] = agg;
            }
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t mine = lane < K * kScanWaves ? lds.total[p][lane] : 0u;
            const uint32_t inc = dpp_inclusive_scan(mine);
#pragma unroll
            for (int k = 0; k < K; ++k) before[p][k] = lane_value(inc, k * kScanWaves + wave) - totals[p][k];
        }
        __syncthreads();
    }
};

}  // namespace helios
