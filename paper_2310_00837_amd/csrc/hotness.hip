// Pre-sampling hotness: per-node counters and the hotness order.
//
// hotness_add: one batch's de-duplicated ID list adds one to each of its nodes'
// counters.  The IDs of a call are distinct, so the atomic adds of one call
// never meet on an address; calls on different streams may.
//
// hotness_order: nodes sorted by counter, descending, ties by ascending ID: a
// stable least-significant-digit radix sort of (count, id) pairs whose ids
// start out ascending.  A digit is 11 bits, so three passes cover 32 bits, and
// a pass whose digit is the same in all counts is left out: the first reading
// of the counts finds out which bits vary, and every kernel of the later passes
// looks there.  Counters of a pre-sampling epoch are at most its number of
// batches, so that one pass is the rule up to 2048 batches.  A pass has three phases:
//   count    every group of consecutive tiles of 8192 pairs counts its digits (LDS);
//   scan     per digit, a prefix sum over the groups, 16 digits to a workgroup;
//   scatter  a group goes through its tiles: a tile ranks its pairs (wave ballots find
//            the lanes with the same digit, a counter per wave and digit in LDS carries
//            the rank along), puts their places into order in LDS and writes them out as runs.
// Bins are numbered from the highest digit down, so each pass goes out in
// descending digit order.  The first pass takes three launches, each of the others one, in which the workgroups draw
// the jobs of all phases (sort_pass_kernel), because an idle launch costs 2 us and there would be six of them.
//
// What bounds it: the chain of steps of the scatter's two tiles per workgroup, its ballots and its LDS traffic; memory second.
// Measured at 8 M nodes with counts up to 512: count 10 us, scan 8, scatter 29
// (its 64 MB would take 11 us); 52 us in all, 111 M nodes 520.  With three launches for each of the other passes, too, and a scatter
// that looked at all bits (35 us) it took 63 and 563 us, 20 000 nodes 33 (now 26); where two passes run, 20 000 nodes 49.7 (now 45.7),
// 1 M 56.7 (53.9), 4 M 94.8 (91.8), 8 M 145 (138), 111 M 1815 (1709); three, which takes counts of 4.2 M and more, 20 000 nodes 68.0 (69.5), 1 M 79.8
// (82.4), 2 M 94.4 (92.4), 4 M 138 (131), 8 M 224 (221), 111 M 3010 (2942).  The launches between the phases cost about what the
// waits do; what the one launch gains where the pass runs is the ranking of every workgroup's first tile before the sums are there
// (8 M, two passes 141 without, three 233).
// With a row of counters per tile, one copy of the count's counters and a scatter of one workgroup per CU it took
// 82 (17, 9.6 and 45) at 8 M and 858 us.
//
// Why groups of tiles: one row of counters per group, of which there are at most 512, keeps the table at 4 MB whatever the
// length of the list, and a scan thread has its rows in registers.
// Why 512 threads with 16 pairs each in the scatter: its counters then take 32 KB (16 waves of 8 pairs: 64 KB), and with the
// order kept as {digit, place in the tile}, 4 bytes a pair, two workgroups fit a CU (74 KB and 128 registers each), so that one has
// its memory traffic while the other ranks.  A digit's bit costs the ranking four instructions of a wave for 64 pairs, and the five
// higher bits are left out where a wave's 64 agree on them: 35 -> 29 us (a branch for every bit 52; the
// lower bits four or five in number 94.4 and 93.2 us for the cache set-up, six 92.4).  The next tile's keys asked for ahead, or a full tile
// without its bounds checks: no difference.  1024 groups, or tiles of 4096, made no difference or 5 us more.
#include "kernels.hpp"

#include <algorithm>

namespace helios {

namespace {

constexpr int kSortBlock = 1024;                          // count and scan of the first pass
constexpr int kSortTile = 8192;                           // pairs
constexpr int kPlaceBlock = 512;                          // scatter, and all phases of the other passes
constexpr int kPlaceWaves = kPlaceBlock / kWave;
constexpr int kPlaceItems = kSortTile / kPlaceBlock;
constexpr int kPlaceBits = 13;                            // a place in the tile
constexpr int kDigitBits = 11;
constexpr int kBins = 1 << kDigitBits;
constexpr int kSortPasses = 3;
constexpr int kScanBins = 16;                             // bins per workgroup of the scan
constexpr int kLowBits = 6;                               // of a digit, that are always looked at
constexpr uint32_t kSortMaxGroups = 512;
constexpr int kCopies = 4;                                // of the count's counters: lanes that meet on a digit spread over them
constexpr uint32_t kScanSlices = kBins / kScanBins;       // workgroups (or jobs) of a scan
constexpr int kControlStride = 32;                        // words: what is counted or waited for lies 128 bytes apart
constexpr int kGoLines = 32;                              // copies of the word that is waited for
constexpr int kCountTickets = 8;                         // counters that the groups to count are drawn from
constexpr int kControlLate = kCountTickets, kControlDone = kControlLate + 1, kControlGo = kControlDone + 2;       // lines of a pass
constexpr int kControlPass = (kControlGo + 2 * kGoLines) * kControlStride;
constexpr int kControlWords = (kSortPasses - 1) * kControlPass;
static_assert(kCopies == 4, "a bin is read as one word of 16 bytes");
static_assert(kSortTile == 1 << kPlaceBits && kBins == 4 * kPlaceBlock, "a thread of the scatter has four bins");

__global__ __launch_bounds__(kBlock) void hotness_add_kernel(const int32_t* __restrict__ ids, Count n_in, int64_t n_nodes,
                                                             int32_t* counts, int32_t* err) {
    const int64_t n = n_in.get();
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; j < n;
         j += static_cast<int64_t>(gridDim.x) * kBlock) {
        const int32_t id = ids[j];
        if (id < 0 || static_cast<int64_t>(id) >= n_nodes) raise(err, kErrData);
        else atomicAdd(counts + id, 1);
    }
}

struct SortArgs {
    const int32_t* counts;
    int32_t *keys[2];            // scratch, by parity of the running pass
    int32_t *vals1, *order;
    uint32_t n, n_tiles;
    uint32_t group_tiles, n_groups;   // group g: the tiles [g * group_tiles, (g + 1) * group_tiles) below n_tiles
    uint32_t* group_counts;      // [n_groups][kBins]; after the scan: pairs of the bin in the groups before
    uint32_t* totals;            // [kBins]
    uint32_t* group_bits;        // [n_groups][2]: bits set in some count, bits clear in some count
    uint32_t* varying;           // bits that are not the same in all counts (from the first pass's scan on)
    uint32_t* control;           // [kControlWords], of the passes after the first
    int32_t* err;
};

// What a pass does: passes whose digit does not vary are left out (the first always runs), and the buffers alternate
// so that the last one that runs leaves its values in `order`.
struct SortStep {
    bool active, last;
    int before;                  // passes that run before this one
    bool to_order;
    __device__ __forceinline__ SortStep(int pass, uint32_t varying) {
        int total = 0;
        before = 0;
        active = false;
#pragma unroll
        for (int p = 0; p < kSortPasses; ++p) {
            const bool runs = p == 0 || ((varying >> (p * kDigitBits)) & (kBins - 1)) != 0;
            if (p < pass && runs) ++before;
            if (p == pass) active = runs;
            if (runs) ++total;
        }
        last = before == total - 1;
        to_order = ((total - 1 - before) & 1) == 0;
    }
};
__device__ __forceinline__ uint32_t bin_of(int32_t key, int pass) {
    return kBins - 1 - ((static_cast<uint32_t>(key) >> (pass * kDigitBits)) & (kBins - 1));
}

// Words that one job of a launch writes for later ones of the same launch (SHARED) go past the L2s of the XCDs, both ways.
template <bool SHARED>
__device__ __forceinline__ uint32_t get_word(const uint32_t* p) {
    return SHARED ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
template <bool SHARED>
__device__ __forceinline__ void put_word(uint32_t* p, uint32_t v) {
    if (SHARED) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// threadIdx.x; in a loop over jobs, what is worked out from it is to be forgotten after the job (kept, it would fill the registers)
template <bool SHARED>
__device__ __forceinline__ uint32_t thread_now() {
    uint32_t t = threadIdx.x;
    if (SHARED) asm volatile("" : "+v"(t));
    return t;
}

// Bound by the LDS atomics: most counts are one of a few small numbers, and lanes that add to one word take their turns.
// Four copies of the counters, by lane, cut the queues to a quarter: 17.3 -> 10.2 us for 8 M counts (eight copies: no difference).
struct CountLds {
    alignas(16) uint32_t hist[kBins * kCopies];
    uint32_t set, clear;
};
template <int B, bool SHARED>
__device__ __forceinline__ void count_group(const SortArgs& a, int pass, const int32_t* keys, uint32_t group, CountLds& s) {
    const uint32_t t = thread_now<SHARED>();
    constexpr int kItems = kSortTile / B;
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    words4* bins = reinterpret_cast<words4*>(s.hist);
    uint32_t zero = 0;
    if (SHARED) asm volatile("" : "+v"(zero));            // (as in thread_now)
    for (uint32_t q = t; q < kBins; q += B) bins[q] = words4{zero, zero, zero, zero};
    if (t == 0) s.set = s.clear = 0;
    __syncthreads();
    const uint32_t tile1 = min((group + 1) * a.group_tiles, a.n_tiles);
    uint32_t set = 0, clear = 0;
    for (uint32_t tile = group * a.group_tiles; tile < tile1; ++tile) {
        const uint32_t i0 = tile * kSortTile + t;
        int32_t key[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) key[k] = keys[i0 + k * B < a.n ? i0 + k * B : a.n - 1];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            set |= static_cast<uint32_t>(key[k]);
            clear |= ~static_cast<uint32_t>(key[k]);
            if (i0 + k * B < a.n) atomicAdd(s.hist + bin_of(key[k], pass) * kCopies + t % kCopies, 1u);
        }
    }
    if (pass == 0) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            set |= __shfl_xor(set, d, kWave);
            clear |= __shfl_xor(clear, d, kWave);
        }
        if (lane_id() == 0) {
            atomicOr(&s.set, set);
            atomicOr(&s.clear, clear);
        }
    }
    __syncthreads();
    for (uint32_t q = t; q < kBins; q += B) {
        const words4 c = bins[q];
        const uint32_t sum = c.x + c.y + c.z + c.w;
        put_word<SHARED>(a.group_counts + static_cast<size_t>(group) * kBins + q, sum);
    }
    if (pass == 0 && t == 0) {
        a.group_bits[2 * group] = s.set;
        a.group_bits[2 * group + 1] = s.clear;
    }
}

__global__ __launch_bounds__(kSortBlock) void sort_count_kernel(SortArgs a) {
    __shared__ CountLds s;
    if (blockIdx.x == 0)
        for (uint32_t w = threadIdx.x; w < kControlWords; w += kSortBlock) a.control[w] = 0;
    count_group<kSortBlock, false>(a, 0, a.counts, blockIdx.x, s);
}

// Slice b: the bins [16 b, 16 b + 16) over all groups, by walkers that take consecutive groups each.
template <int B>
struct ScanLds {
    uint32_t sum[B / kScanBins][kScanBins + 1];
};
template <int B, bool SHARED>
__device__ __forceinline__ void scan_slice(const SortArgs& a, uint32_t slice, ScanLds<B>& s) {
    const uint32_t t = thread_now<SHARED>();
    constexpr uint32_t kWalkers = B / kScanBins, kPer = kSortMaxGroups / kWalkers;
    static_assert(kWalkers <= kWave, "one wave scans the walkers of one bin");
    const uint32_t walker = t / kScanBins, bin = t % kScanBins;
    uint32_t* column = a.group_counts + slice * kScanBins + bin;
    uint32_t v[kPer], sum = 0;
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {            // (unguarded: all in flight together)
        const uint32_t g = walker * kPer + q;
        v[q] = get_word<SHARED>(column + static_cast<size_t>(g < a.n_groups ? g : 0) * kBins);
    }
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        if (walker * kPer + q >= a.n_groups) v[q] = 0;
        sum += v[q];
    }
    s.sum[walker][bin] = sum;
    __syncthreads();
    for (uint32_t b = t / kWave; b < kScanBins; b += B / kWave) {                             // one wave per bin
        const uint32_t w = t % kWave;
        const uint32_t mine = w < kWalkers ? s.sum[w][b] : 0u, inc = dpp_inclusive_scan(mine);
        if (w < kWalkers) s.sum[w][b] = inc - mine;
        if (w == kWave - 1) put_word<SHARED>(a.totals + slice * kScanBins + b, inc);
    }
    __syncthreads();
    uint32_t run = s.sum[walker][bin];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        const uint32_t g = walker * kPer + q;
        if (g < a.n_groups) put_word<SHARED>(column + static_cast<size_t>(g) * kBins, run);
        run += v[q];
    }
}

// One workgroup more than slices: it gathers which bits vary.
__global__ __launch_bounds__(kSortBlock) void sort_scan_kernel(SortArgs a) {
    __shared__ ScanLds<kSortBlock> s;
    __shared__ uint32_t s_set, s_clear;
    if (blockIdx.x < kScanSlices) {
        scan_slice<kSortBlock, false>(a, blockIdx.x, s);
        return;
    }
    if (threadIdx.x == 0) s_set = s_clear = 0;
    __syncthreads();
    uint32_t set = 0, clear = 0;
    for (uint32_t t = threadIdx.x; t < a.n_groups; t += kSortBlock) {
        set |= a.group_bits[2 * t];
        clear |= a.group_bits[2 * t + 1];
    }
    atomicOr(&s_set, set);
    atomicOr(&s_clear, clear);
    __syncthreads();
    if (threadIdx.x == 0) *a.varying = s_set & s_clear;
}

// The lanes of a wave that hold the same bin as this one.
struct Peers {
    uint32_t lo, hi;
    template <int FROM, int TO>
    __device__ __forceinline__ void agree(uint32_t bin) {          // those that agree on the bits too; four instructions for each
#pragma unroll
        for (int b = FROM; b < TO; ++b) {
            uint32_t mine = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(bin), b, 1));
            asm("" : "+v"(mine));                                  // (or the comparison gets a shift of its own)
            const uint64_t ones = __ballot(mine != 0);
            lo = __builtin_amdgcn_bitop3_b32(lo, static_cast<uint32_t>(ones), mine, 0x90);      // x & ~(y ^ z)
            hi = __builtin_amdgcn_bitop3_b32(hi, static_cast<uint32_t>(ones >> 32), mine, 0x90);
        }
    }
    __device__ __forceinline__ uint32_t rank() const { return __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)); }
    __device__ __forceinline__ uint32_t count() const { return static_cast<uint32_t>(__popc(lo) + __popc(hi)); }
};

struct PlaceLds {
    // the ranks' counters (one per wave and bin) and, once the ranks are known, the tile in order share their memory
    union {
        uint16_t count[kPlaceWaves][kBins];
        uint32_t two[kPlaceWaves][kBins / 2];
        unsigned long long four[kPlaceWaves][kBins / 4];      // a thread's bins
        uint32_t out[kSortTile];                              // {bin : 11 | place in the tile : 13}
    };
    uint32_t to[kBins];                                       // where a bin goes in the output, minus where it begins in the tile
    int32_t word[kSortTile];
    uint32_t wave[kPlaceWaves];
};
// ready: waits until the sums of the counts are there.  The first tile is ranked before that, beside the phases that make them.
template <bool SHARED, class Ready>
__device__ __forceinline__ void scatter_group(const SortArgs& a, int pass, const SortStep& step, uint32_t group, PlaceLds& s, const Ready& ready) {
    const uint32_t t = thread_now<SHARED>();
    // (pointers by condition and no a.keys[i], or the arguments end up in scratch memory)
    const int32_t* keys_in = step.before == 0 ? a.counts : step.before == 1 ? a.keys[0] : a.keys[1];
    const int32_t* vals_in = step.before == 0 ? nullptr : step.to_order ? a.vals1 : a.order;
    int32_t* keys_out = step.last ? nullptr : step.before == 0 ? a.keys[0] : a.keys[1];
    int32_t* vals_out = step.to_order ? a.order : a.vals1;
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(t / kWave))), lane = t % kWave;
    constexpr int kPer = kBins / kPlaceBlock;    // bins per thread: consecutive ones
    // exclusive sums over the bins of the whole list
    const auto scan_bins = [&](const uint32_t (&v)[kPer], uint32_t (&before)[kPer]) {
        uint32_t mine = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) mine += v[q];
        const uint32_t inc = dpp_inclusive_scan(mine);
        if (lane == kWave - 1) s.wave[wave] = inc;
        __syncthreads();
        const uint32_t w = lane < kPlaceWaves ? s.wave[lane] : 0u;
        const uint32_t upto = dpp_inclusive_scan(w);
        uint32_t at = lane_value(upto, wave) - lane_value(w, wave) + inc - mine;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            before[q] = at;
            at += v[q];
        }
        __syncthreads();
    };
    const uint32_t n = a.n;
    uint32_t next[kPer];                         // where the tile's pairs of the bin go in the output
    const auto first_places = [&] {
        uint32_t total[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) total[q] = get_word<SHARED>(a.totals + t * kPer + q);
        scan_bins(total, next);
#pragma unroll
        for (int q = 0; q < kPer; ++q) next[q] += get_word<SHARED>(a.group_counts + static_cast<size_t>(group) * kBins + t * kPer + q);
    };
    if (!SHARED) first_places();
    const uint32_t tile1 = min((group + 1) * a.group_tiles, a.n_tiles);
    for (uint32_t tile = group * a.group_tiles; tile < tile1; ++tile) {
        // a wave owns 1024 consecutive pairs, 64 per round
        const uint32_t base = tile * kSortTile, here = min(n - base, static_cast<uint32_t>(kSortTile));
        const uint32_t at0 = wave * (kPlaceItems * kWave) + lane;
        uint32_t item[kPlaceItems];              // the bin, then {bin : 11 | rank : 13}
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) item[k] = bin_of(keys_in[base + (at0 + k * kWave < here ? at0 + k * kWave : 0)], pass);
#pragma unroll
        for (int w = 0; w < kPlaceWaves; ++w) s.four[w][t] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) {
            const uint32_t bin = item[k];
            const uint64_t there = __ballot(at0 + k * kWave < here);
            Peers peers{static_cast<uint32_t>(there), static_cast<uint32_t>(there >> 32)};
            peers.agree<0, kLowBits>(bin);
            // (most counts are small)
            if (__ballot((bin ^ static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(bin)))) >> kLowBits != 0) != 0) peers.agree<kLowBits, kDigitBits>(bin);
            const uint32_t among = peers.rank();
            // The wave's counter of the bin is read and then added to, two of them to a word; LDS works a wave's requests off in order,
            // so that nothing has to wait in between.
            item[k] = (bin << kPlaceBits) | (s.count[wave][bin] + among);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (among == 0 && at0 + k * kWave < here) __hip_atomic_fetch_add(&s.two[wave][bin / 2], peers.count() << (16 * (bin % 2)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        if (SHARED && tile == group * a.group_tiles) {
            ready();
            first_places();
        }
        // four counters of 16 bits at a time: their sums over the waves, and where the bins begin, stay below 2^16
        unsigned long long sum = 0, before[kPlaceWaves];
#pragma unroll
        for (int w = 0; w < kPlaceWaves; ++w) {
            before[w] = sum;
            sum += s.four[w][t];
        }
        uint32_t in_tile[kPer], start[kPer];
        unsigned long long begins = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) in_tile[q] = static_cast<uint32_t>(sum >> (16 * q)) & 0xffffu;
        scan_bins(in_tile, start);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            begins |= static_cast<unsigned long long>(start[q]) << (16 * q);
            s.to[t * kPer + q] = next[q] - start[q];
            next[q] += in_tile[q];
        }
#pragma unroll
        for (int w = 0; w < kPlaceWaves; ++w) s.four[w][t] = before[w] + begins;
        __syncthreads();
        uint32_t place[kPlaceItems];
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) place[k] = s.count[wave][item[k] >> kPlaceBits] + (item[k] & (kSortTile - 1));
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k)
            if (at0 + k * kWave < here && place[k] < kSortTile) s.out[place[k]] = (item[k] & ~(kSortTile - 1u)) | (at0 + k * kWave);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) {
            const uint32_t p = t + k * kPlaceBlock, e = s.out[p < here ? p : 0], to = s.to[e >> kPlaceBits] + p;
            if (p < here && to >= n) raise(a.err, kErrInternal);         // never, unless the counts changed between the kernels
            if (p < here && to < n && !vals_in) vals_out[to] = static_cast<int32_t>(base + (e & (kSortTile - 1)));
        }
        // The other words of the pairs, where there are any: read in order, picked from LDS.
        const auto move = [&](const int32_t* in, int32_t* out) {
#pragma unroll
            for (int k = 0; k < kPlaceItems; ++k) {
                const uint32_t p = t + k * kPlaceBlock;
                s.word[p] = in[base + (p < here ? p : 0)];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kPlaceItems; ++k) {
                const uint32_t p = t + k * kPlaceBlock, e = s.out[p < here ? p : 0], to = s.to[e >> kPlaceBits] + p;
                if (p < here && to < n) out[to] = s.word[e & (kSortTile - 1)];
            }
            __syncthreads();
        };
        if (vals_in) move(vals_in, vals_out);
        if (keys_out) move(keys_in, keys_out);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kPlaceBlock) void sort_scatter_kernel(SortArgs a) {
    __shared__ PlaceLds s;
    scatter_group<false>(a, 0, SortStep(0, *a.varying), blockIdx.x, s, [] {});
}

// A pass after the first, if it runs.  The jobs (a group to count, a slice to scan, a group to scatter) are done phase by phase, and
// a workgroup draws one after the other until there is none.  The groups to count are drawn from eight counters, a workgroup's own
// first (489 draws from one took 4 us), all other jobs, in order, from one more, and only once every group is seen to be drawn.
// A job waits until all jobs of the phase before it are done; workgroups that run already hold those, and the lowest job that is
// not done waits for nothing: however few workgroups the GPU has room for, the launch ends.  Between the phases only the counts
// and their sums change hands, as words that go past the L2s (put_word): a wave waits until its own are there before its job counts
// as done.  Whoever finishes a phase says so in 32 places, as hundreds that look at one word keep those away that add to it (10 ns
// each; 8 M nodes, a second pass: 120 us when they did).
__device__ __forceinline__ uint32_t draw(uint32_t* counter) {                  // (by the first wave)
    uint32_t t = 0;
    if (thread_now<true>() == 0) t = atomicAdd(counter, 1u);
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(t)));
}
__device__ __forceinline__ uint32_t draw_job(uint32_t* control, uint32_t n_groups, uint64_t look) {      // look: counters to draw from at once
    while (true) {
        for (; look != 0; look &= look - 1) {
            const uint32_t c = static_cast<uint32_t>(__ffsll(static_cast<long long>(look)) - 1), group = draw(control + c * kControlStride) * kCountTickets + c;
            if (group < n_groups) return group;
        }
        const uint32_t c = thread_now<true>() % kCountTickets;
        look = __ballot(get_word<true>(control + c * kControlStride) * kCountTickets + c < n_groups) & ((1u << kCountTickets) - 1);
        if (look == 0) return n_groups + draw(control + kControlLate * kControlStride);
    }
}

template <int PASS>
__global__ __launch_bounds__(kPlaceBlock, 4) void sort_pass_kernel(SortArgs a) {
    __shared__ union {
        CountLds count;
        ScanLds<kPlaceBlock> scan;
        PlaceLds place;
    } s;
    __shared__ uint32_t s_job;
    const SortStep step(PASS, *a.varying);
    if (!step.active) return;
    const uint32_t n_jobs = 2 * a.n_groups + kScanSlices;
    uint32_t* control = a.control + (PASS - 1) * kControlPass;
    if (threadIdx.x < kWave) s_job = draw_job(control, a.n_groups, 1u << blockIdx.x % kCountTickets);
    __syncthreads();
    for (uint32_t job; (job = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(s_job)))) < n_jobs;) {
        const uint32_t phase = job < a.n_groups ? 0u : job < a.n_groups + kScanSlices ? 1u : 2u;
        const auto wait = [&] {                  // for the phase before this one
            if (threadIdx.x == 0) {
                const uint32_t* go = control + (kControlGo + (phase - 1) * kGoLines + job % kGoLines) * kControlStride;
                uint32_t budget = kScanSpinBudget;
                while (__hip_atomic_load(go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0 && --budget > 0) __builtin_amdgcn_s_sleep(4);
                if (budget == 0) raise(a.err, kErrInternal);       // gave up: report, and let the launch drain
            }
            __syncthreads();
        };
        if (phase == 1) wait();
        if (phase == 0) count_group<kPlaceBlock, true>(a, PASS, step.before == 1 ? a.keys[0] : a.keys[1], job, s.count);
        else if (phase == 1) scan_slice<kPlaceBlock, true>(a, job - a.n_groups, s.scan);
        else scatter_group<true>(a, PASS, step, job - a.n_groups - kScanSlices, s.place, wait);
        if (phase < 2) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x < kWave) {
            if (phase < 2 && draw(control + (kControlDone + phase) * kControlStride) + 1 == (phase == 0 ? a.n_groups : kScanSlices)) {
                const uint32_t q = thread_now<true>();
                if (q < kGoLines) put_word<true>(control + (kControlGo + phase * kGoLines + q) * kControlStride, 1u);
            }
            s_job = phase == 0 ? draw_job(control, a.n_groups, 0) : a.n_groups + draw(control + kControlLate * kControlStride);
        }
        // (The loop has to end with a barrier: with that `if` as its end the compiler makes two loops of it, and the lanes beside lane 0
        // go round without it.)
        __syncthreads();
    }
}

unsigned grid_for(int64_t n, unsigned cap_blocks) {
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > cap_blocks) b = cap_blocks;
    return static_cast<unsigned>(b);
}

}  // namespace

hipError_t launch_hotness_add(hipStream_t stream, const int32_t* ids, Count n, int64_t n_max, int64_t n_nodes,
                              int32_t* counts, int32_t* err) {
    hipLaunchKernelGGL(hotness_add_kernel, dim3(grid_for(n_max, 4096)), dim3(kBlock), 0, stream, ids, n, n_nodes, counts, err);
    return hipGetLastError();
}

namespace {
struct SortLayout {              // scratch of the hotness order, in bytes
    size_t tiles, group_tiles, groups, totals, varying, control, bits, counts, keys1, keys2, vals1, bytes;
    explicit SortLayout(int64_t n) {
        const auto up = [](size_t b) { return (b + 255) / 256 * 256; };
        tiles = static_cast<size_t>((n + kSortTile - 1) / kSortTile);
        if (tiles < 1) tiles = 1;
        group_tiles = (tiles + kSortMaxGroups - 1) / kSortMaxGroups;
        groups = (tiles + group_tiles - 1) / group_tiles;
        const size_t ints = up(sizeof(int32_t) * static_cast<size_t>(n));
        totals = 0;
        varying = totals + up(sizeof(uint32_t) * kBins);
        control = varying + 256;
        bits = control + up(sizeof(uint32_t) * kControlWords);
        counts = bits + up(sizeof(uint32_t) * 2 * groups);
        keys1 = counts + up(sizeof(uint32_t) * kBins * groups);
        keys2 = keys1 + ints;
        vals1 = keys2 + ints;
        bytes = vals1 + ints;
    }
};
}  // namespace

size_t hotness_order_scratch_bytes(int64_t n_nodes) { return SortLayout(n_nodes).bytes; }

hipError_t launch_hotness_order(hipStream_t stream, const int32_t* counts, int64_t n_nodes, int32_t* order, void* scratch,
                                int32_t* err) {
    if (n_nodes < 1) return hipSuccess;
    const SortLayout at(n_nodes);
    unsigned char* p = static_cast<unsigned char*>(scratch);
    SortArgs a{};
    a.counts = counts;
    a.keys[0] = reinterpret_cast<int32_t*>(p + at.keys1);
    a.keys[1] = reinterpret_cast<int32_t*>(p + at.keys2);
    a.vals1 = reinterpret_cast<int32_t*>(p + at.vals1);
    a.order = order;
    a.n = static_cast<uint32_t>(n_nodes);
    a.n_tiles = static_cast<uint32_t>(at.tiles);
    a.group_tiles = static_cast<uint32_t>(at.group_tiles);
    a.n_groups = static_cast<uint32_t>(at.groups);
    a.group_counts = reinterpret_cast<uint32_t*>(p + at.counts);
    a.totals = reinterpret_cast<uint32_t*>(p + at.totals);
    a.group_bits = reinterpret_cast<uint32_t*>(p + at.bits);
    a.varying = reinterpret_cast<uint32_t*>(p + at.varying);
    a.control = reinterpret_cast<uint32_t*>(p + at.control);
    a.err = err;
    // With one pass or three the first one already writes to `order`.  If that is (part of) the counters' own memory, the pass
    // reads a copy, in the buffer that no pass writes before the second has begun.
    const uintptr_t c0 = reinterpret_cast<uintptr_t>(counts), o0 = reinterpret_cast<uintptr_t>(order), len = sizeof(int32_t) * a.n;
    if (c0 < o0 + len && o0 < c0 + len) {
        const hipError_t e = hipMemcpyAsync(a.keys[1], counts, len, hipMemcpyDefault, stream);
        if (e != hipSuccess) return e;
        a.counts = a.keys[1];
    }
    const dim3 groups(a.n_groups), block(kSortBlock);
    hipLaunchKernelGGL(sort_count_kernel, groups, block, 0, stream, a);
    hipLaunchKernelGGL(sort_scan_kernel, dim3(kScanSlices + 1), block, 0, stream, a);
    hipLaunchKernelGGL(sort_scatter_kernel, groups, dim3(kPlaceBlock), 0, stream, a);
    const dim3 workers(std::max(a.n_groups, kScanSlices));
    hipLaunchKernelGGL(sort_pass_kernel<1>, workers, dim3(kPlaceBlock), 0, stream, a);
    hipLaunchKernelGGL(sort_pass_kernel<2>, workers, dim3(kPlaceBlock), 0, stream, a);
    return hipGetLastError();
}

}  // namespace helios
