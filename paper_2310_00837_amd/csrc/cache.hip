// Cache map and cache lookup.
//
// rank_build: rank[order[r]] = r, with a check that order is a permutation: by scattered stores, or, where there is scratch
// memory for it, by way of buckets of neighbouring IDs.
//
// lookup_partition: one thread per ID reads rank[id] (one random 4-byte read),
// classifies it into the HBM tier, the host tier or a miss by two compares, and
// the three classes are compacted *stably* in one pass: wave ballots and a scan of
// the waves' totals give the ranks inside a tile and a three-counter
// chained scan (TileScan in scan.hpp) the ranks across workgroups.  The two hit lists (position, slot)
// feed the row-copy kernels (where it is quicker, helios_gather copies the HBM tier's rows
// without one, in the same launch); the miss list (position, id, slot) is the request
// list of the storage tier and comes out ascending in position.
#include "kernels.hpp"

namespace helios {

namespace {

__global__ __launch_bounds__(kBlock) void rank_fill_kernel(int32_t* rank, int64_t n, int64_t* holes) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *holes = 0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * kBlock)
        rank[i] = -1;
}

__global__ __launch_bounds__(kBlock) void rank_scatter_kernel(const int32_t* __restrict__ order, int64_t n, int32_t* rank,
                                                              int32_t* err) {
    for (int64_t r = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; r < n;
         r += static_cast<int64_t>(gridDim.x) * kBlock) {
        const int32_t v = order[r];
        if (v < 0 || static_cast<int64_t>(v) >= n) raise(err, kErrData);
        else rank[v] = static_cast<int32_t>(r);
    }
}

// a node that no rank points to means `order` repeated another node
__global__ __launch_bounds__(kBlock) void rank_check_kernel(const int32_t* __restrict__ rank, int64_t n, int64_t* holes, int32_t* err) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * kBlock)
        if (rank[i] < 0) {
            *holes = 1;
            raise(err, kErrData);
        }
}

// ---- the map by buckets
//
// The scattered stores are bound by the parts of lines that they write: a hotness order has the nodes of one count in a row, ascending, so
// every line of the map is written in parts once per count, by whichever XCD, and the memory takes some 60 such requests a ns.  By
// buckets every line is written once:
//   split   every tile of 4096 ranks hands its nodes to the buckets of 2^shift neighbouring nodes that they belong to; what a bucket
//           gets lies where its nodes' ranks will (a permutation fills it exactly).  64 nodes of one wave that all go to one bucket,
//           the rule in a hotness order, are a run: their ranks are consecutive, so the first rank and the 64 places in the bucket,
//           of 2 bytes, say it all.  Other nodes go as pairs {node, rank} of 8 bytes;
//   place   a workgroup per bucket puts the ranks in order in LDS and writes them out.
// Where an order goes through neighbouring nodes (all of one count, as those that no batch has met; nodes numbered by locality) its stores are
// whole lines to begin with: the split then stores them itself, and place only looks whether the order has the node there.
// Measured, us by scattered stores / by buckets with pairs only / with runs: the hotness order of a power law
//   1 M nodes 13.2/14.2/-   2 M 25/19.7/15.3 (the line)   3 M 34/23.6/19.0   8 M 78/38.0/29.1   16 M 142/66.2/52.4
// (a random order 8 M 114/83/80, 3 M 48/41/39), of counts that are 0 for 99 of 100 nodes (and for 9 of 10; and all the same)
//   2 M 14.5/15.1/13.4 (15.2/17.3/16.2; 12.0/11.6/10.0)   3 M 17.2/17.5/15.5 (19.6/20.6/19.0; 13.2/17.3/15.5)
//   8 M 28/30/27.1 (39/35.9/33.9; 27/28/25.2)   16 M 49/53/49 (64/64.5/62.5; 46/51/47)
// and the nodes in random blocks of 64: 8 M 27/28/25.4.  (With runs there is a launch less, too: 2 us.)  8 M of a power law by kernels: split 20.8 with pairs, 16.7 with runs, place 16.3 and 12.1.
// The buckets take 8 bytes of scratch per node, so they are used where the context has that from making a hotness order; and above 16.7 M
// nodes a bucket would not fit LDS.  (Four ranks per thread in the split: with 512 or 256 threads, or eight ranks, 0 to 4 us slower, random orders
// up to 50; workgroups that go through several tiles, the next one asked for ahead, 2 us slower.)
constexpr int kInvertBlock = 1024;
constexpr int kInvertItems = 4;
constexpr uint32_t kInvertTile = kInvertBlock * kInvertItems;
constexpr int kHandBlock = 1024;                       // split
constexpr int kHandItems = 4;
constexpr uint32_t kHandTile = kHandBlock * kHandItems;
constexpr uint32_t kInvertBuckets = 512;
constexpr uint32_t kInvertMaxShift = 15;               // 32768 ranks: 128 KB of LDS
constexpr int kPlaceItems = 8;                         // one at a time: 16 M by pairs 33.5 us in place, with eight 31
constexpr uint32_t kNear = 96;                         // three lines of ranks (every other node of a row, 128, is as quick by pairs)
constexpr int64_t kInvertMin = 2000000;
constexpr int64_t kInvertMax = static_cast<int64_t>(kInvertBuckets) << kInvertMaxShift;

// What a bucket is handed lies where its nodes are among all nodes, 8 bytes for each: the places of its runs (64 nodes of one wave, so 64
// consecutive ranks) from the front, 2 bytes a node, and its pairs from the back.  Of a permutation a bucket gets as many nodes as it
// has, so the two do not meet.
struct InvertScratch {
    uint32_t* cursors;           // [2][kInvertBuckets]: pairs and runs that a bucket has been handed so far; zero between calls
    unsigned long long* pairs;   // [n] {node : 32 | rank : 32}
    uint32_t* run_rank;          // [n / 64] rank of a run's first node
    __device__ __forceinline__ uint16_t* places(uint32_t first) const { return reinterpret_cast<uint16_t*>(pairs + first); }
};
constexpr int kRunsAhead = 4;
static_assert(2 * kInvertBuckets == kMapCursors, "the context's counters");

__global__ __launch_bounds__(kHandBlock) void rank_split_kernel(const int32_t* __restrict__ order, uint32_t n, uint32_t shift, InvertScratch s,
                                                                  int32_t* rank, int64_t* holes, int32_t* err) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *holes = 0;
    // of pairs [0, 512) and of runs [512, 1024): how many this tile has for a bucket, and where they go
    __shared__ uint32_t s_count[2 * kInvertBuckets], s_base[2 * kInvertBuckets], s_unused[kWave];
    const uint32_t r0 = blockIdx.x * kHandTile + threadIdx.x, lane = static_cast<uint32_t>(lane_id());
    uint32_t v[kHandItems];
#pragma unroll
    for (int k = 0; k < kHandItems; ++k) v[k] = static_cast<uint32_t>(order[min(r0 + k * kHandBlock, n - 1)]);
    for (uint32_t c = threadIdx.x; c < 2 * kInvertBuckets; c += kHandBlock) s_count[c] = 0;
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kHandItems; ++k) {
        const bool here = r0 + k * kHandBlock < n, node = v[k] < n;
        bad = bad || (here && !node);
        v[k] = here && node ? v[k] : ~0u;
    }
    if (bad) raise(err, kErrData);
    // A wave whose nodes ascend or descend by little: the first and the last one of its first 64 lie close together.  They are
    // stored at once, and are no pairs from here on.  (If the others don't, it only takes longer.  Asked of all 256, an order without
    // such waves took 1 us longer.)
    const uint32_t v0 = lane_value(v[0], 0), v1 = lane_value(v[0], kWave - 1);
    if ((v0 < v1 ? v1 - v0 : v0 - v1) < kNear && v1 != ~0u) {
#pragma unroll
        for (int k = 0; k < kHandItems; ++k) {
            if (v[k] != ~0u) rank[v[k]] = static_cast<int32_t>(r0 + k * kHandBlock);
            v[k] = ~0u;
        }
    }
    // In a hotness order the nodes of a wave are mostly of one bucket, and then a run.  Lane k has the bucket of the wave's k-th run and
    // its number, so that one addition counts them all.
    bool run[kHandItems], all_runs = true;
    uint32_t run_bucket = ~0u, nth = 0;
#pragma unroll
    for (int k = 0; k < kHandItems; ++k) {
        const uint32_t head = lane_value(v[k], 0);
        run[k] = __ballot(v[k] >> shift == head >> shift) == ~0ull && head != ~0u;
        all_runs = all_runs && (run[k] || __ballot(v[k] != ~0u) == 0);
        if (lane == static_cast<uint32_t>(k) && run[k]) run_bucket = head >> shift;
    }
    if (run_bucket != ~0u) nth = atomicAdd(s_count + kInvertBuckets + run_bucket, 1u);
    uint32_t at[kHandItems];
    if (!all_runs) {
        uint32_t lead[kHandItems];
        uint64_t same[kHandItems];
#pragma unroll
        for (int k = 0; k < kHandItems; ++k) {
            const uint32_t bucket = v[k] >> shift;
            // Those that go where the first goes are counted at once, by the first.  (Every lane adds somewhere, so that the additions of
            // all items are on their way together.)
            const uint64_t there = run[k] ? 0 : __ballot(v[k] != ~0u);
            lead[k] = there ? static_cast<uint32_t>(__ffsll(static_cast<long long>(there)) - 1) : 0u;
            same[k] = __ballot(bucket == lane_value(bucket, lead[k])) & there;
            const bool leads = lane == lead[k], counts = ((there >> lane) & 1u) && (leads || !((same[k] >> lane) & 1u));
            at[k] = atomicAdd(counts ? s_count + bucket : s_unused + lane, leads ? static_cast<uint32_t>(__popcll(same[k])) : 1u);
        }
#pragma unroll
        for (int k = 0; k < kHandItems; ++k) {
            const uint32_t from = lane_value(at[k], lead[k]);
            if ((same[k] >> lane) & 1u) at[k] = from + rank_in_mask(same[k]);
        }
    }
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < 2 * kInvertBuckets; c += kHandBlock)
        if (s_count[c] != 0) s_base[c] = atomicAdd(s.cursors + c, s_count[c]);
    __syncthreads();
    // (More than the bucket has nodes: some node is there twice.  What does not fit is left out, and the bucket's workgroup goes by the
    // order itself.)
    if (run_bucket != ~0u) {
        const uint32_t first = run_bucket << shift, nodes = min(n - first, 1u << shift);
        nth += s_base[kInvertBuckets + run_bucket];
        if ((nth + 1) * kWave > nodes) nth = ~0u;
        else s.run_rank[first / kWave + nth] = r0 - lane + lane * kHandBlock;
    }
#pragma unroll
    for (int k = 0; k < kHandItems; ++k) {
        if (run[k]) {
            const uint32_t first = lane_value(run_bucket, k) << shift, to = lane_value(nth, k);
            if (to != ~0u) s.places(first)[to * kWave + lane] = static_cast<uint16_t>(v[k] - first);
        } else if (!all_runs && v[k] != ~0u) {
            const uint32_t bucket = v[k] >> shift, first = bucket << shift, nodes = min(n - first, 1u << shift), place = s_base[bucket] + at[k];
            if (place < nodes) s.pairs[first + nodes - 1 - place] = (static_cast<unsigned long long>(v[k]) << 32) | (r0 + k * kHandBlock);
        }
    }
}

template <uint32_t MOST>
__global__ __launch_bounds__(kInvertBlock) void rank_place_kernel(const int32_t* __restrict__ order, uint32_t n, uint32_t shift,
                                                                  InvertScratch s, int32_t* rank, int64_t* holes, int32_t* err) {
    __shared__ int32_t s_rank[1u << MOST];               // (shift <= MOST)
    const uint32_t first = blockIdx.x << shift, nodes = min(n - first, 1u << shift);
    const uint32_t n_pairs = s.cursors[blockIdx.x], n_runs = s.cursors[kInvertBuckets + blockIdx.x];
    for (uint32_t i = threadIdx.x; i < nodes; i += kInvertBlock) s_rank[i] = -1;
    __syncthreads();
    if (threadIdx.x < 2) s.cursors[threadIdx.x * kInvertBuckets + blockIdx.x] = 0;
    if (n_pairs <= nodes && n_runs <= nodes / kWave && n_pairs + n_runs * kWave <= nodes) {
        const uint32_t lane = static_cast<uint32_t>(lane_id()), wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave_id()));
        for (uint32_t w0 = wave; w0 < n_runs; w0 += kRunsAhead * (kInvertBlock / kWave)) {
            uint32_t r[kRunsAhead], place[kRunsAhead];
#pragma unroll
            for (int k = 0; k < kRunsAhead; ++k) {
                const uint32_t w = min(w0 + k * (kInvertBlock / kWave), n_runs - 1);
                r[k] = s.run_rank[first / kWave + w] + lane;
                place[k] = s.places(first)[w * kWave + lane];
            }
#pragma unroll
            for (int k = 0; k < kRunsAhead; ++k)         // (a run that is there already once more)
                if (place[k] < nodes) s_rank[place[k]] = static_cast<int32_t>(r[k]);
        }
        for (uint32_t i0 = threadIdx.x; i0 < n_pairs; i0 += kInvertTile) {
            unsigned long long pair[kInvertItems];
#pragma unroll
            for (int k = 0; k < kInvertItems; ++k) pair[k] = s.pairs[first + nodes - 1 - (i0 + k * kInvertBlock < n_pairs ? i0 + k * kInvertBlock : 0)];
#pragma unroll
            for (int k = 0; k < kInvertItems; ++k) {
                const uint32_t place = static_cast<uint32_t>(pair[k] >> 32) - first;
                if (i0 + k * kInvertBlock < n_pairs && place < nodes) s_rank[place] = static_cast<int32_t>(static_cast<uint32_t>(pair[k]));
            }
        }
    } else {                                             // (an order that is no permutation)
        for (uint32_t r = threadIdx.x; r < n; r += kInvertBlock) {
            const uint32_t place = static_cast<uint32_t>(order[r]) - first;
            if (place < nodes) s_rank[place] = static_cast<int32_t>(r);
        }
    }
    __syncthreads();
    bool missing = false;
    for (uint32_t i0 = threadIdx.x; i0 < nodes; i0 += kPlaceItems * kInvertBlock) {
        int32_t r[kPlaceItems];
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) r[k] = s_rank[min(i0 + k * kInvertBlock, nodes - 1)];
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) {
            if (r[k] >= 0) rank[first + min(i0 + k * kInvertBlock, nodes - 1)] = r[k];
            missing = missing || r[k] < 0;
        }
    }
    if (!missing) return;
    // What the split has stored itself has no pair.  Such a node's word is right if the order has the node at that rank, whatever
    // the word held before; else the node has no rank.
    for (uint32_t i0 = threadIdx.x; i0 < nodes; i0 += kPlaceItems * kInvertBlock) {
        uint32_t stored[kPlaceItems], there[kPlaceItems];
        bool none[kPlaceItems];
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) {                    // (unguarded: all in flight together)
            const uint32_t i = min(i0 + k * kInvertBlock, nodes - 1);
            none[k] = s_rank[i] < 0;
            stored[k] = static_cast<uint32_t>(rank[first + (none[k] ? i : 0)]);
        }
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) there[k] = static_cast<uint32_t>(order[none[k] && stored[k] < n ? stored[k] : 0]);
#pragma unroll
        for (int k = 0; k < kPlaceItems; ++k) {
            const uint32_t i = min(i0 + k * kInvertBlock, nodes - 1);
            if (!none[k] || (stored[k] < n && there[k] == first + i)) continue;
            rank[first + i] = -1;
            *holes = 1;
            raise(err, kErrData);
        }
    }
}

struct PartitionArgs {
    const int32_t* ids;
    Count n;
    const int32_t* rank;
    int64_t n_nodes, n_hbm, n_host;
    TierLists lists;
    int32_t *miss_pos, *miss_id, *miss_slot;
    int64_t miss_cap;
    int64_t* stats_out;          // device-accessible int64[4], nullable
    int64_t* learn;              // pinned int64[4], nullable: a copy of the stats for the host's grid sizing
    bool hbm_direct;             // no list is wanted for the HBM tier
    ScanState scan;
    int32_t* err;
};

// Bound like a stage of the compaction (compact_dev.hpp) by its chain of dependent steps, and built like it.
template <int K>
__device__ __forceinline__ void partition_role(const PartitionArgs& a, uint32_t rb, uint32_t nrb) {
    using Scan = TileScan<2, 3, K>;
    __shared__ typename Scan::Lds lds;
    const ScanState scan = scan_resolve(a.scan);
    const uint32_t n = static_cast<uint32_t>(a.n.get());
    const uint32_t n_tiles = (n + K * kScanBlock - 1) / (K * kScanBlock);
    if (n == 0 && rb == 0 && threadIdx.x == 0) {
        a.lists.count[0] = a.lists.count[1] = a.lists.count[2] = 0;
        if (a.stats_out) { a.stats_out[0] = 0; a.stats_out[1] = 0; a.stats_out[2] = 0; a.stats_out[3] = 0; }
    }
    if (rb >= n_tiles) return;
    const uint32_t n_wgs = nrb < n_tiles ? nrb : n_tiles;
    for (uint32_t tile = Scan::take_ticket(scan, n_tiles, n_wgs, lds); tile < n_tiles;
         tile = n_wgs < n_tiles ? Scan::take_ticket(scan, n_tiles, n_wgs, lds) : n_tiles) {
        const uint32_t j0 = tile * (K * kScanBlock) + threadIdx.x;
        int32_t id[K], r[K];
#pragma unroll
        for (int k = 0; k < K; ++k) id[k] = a.ids[j0 + k * kScanBlock < n ? j0 + k * kScanBlock : 0];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool here = j0 + k * kScanBlock < n, ok = here && id[k] >= 0 && static_cast<int64_t>(id[k]) < a.n_nodes;
            if (here && !ok) raise(a.err, kErrData);
            const int32_t got = a.rank[ok ? id[k] : 0];          // all reads in flight together
            r[k] = ok ? got : -1;                                // -1: no ID here, a bad ID, or a node that the order left out
        }
        const uint32_t n_hbm = static_cast<uint32_t>(a.n_hbm), n_cached = static_cast<uint32_t>(a.n_hbm + a.n_host);
        uint32_t totals[2][K], before[2][K], in_class[K], in_hits[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t ur = static_cast<uint32_t>(r[k]);     // -1 is in none of the three classes
            const uint64_t hbm = __ballot(ur < n_hbm), host = __ballot(ur >= n_hbm && ur < n_cached), miss = __ballot(r[k] >= 0 && ur >= n_cached);
            totals[0][k] = static_cast<uint32_t>(__popcll(miss));
            totals[1][k] = static_cast<uint32_t>(__popcll(hbm)) | (static_cast<uint32_t>(__popcll(host)) << 16);
            in_class[k] = rank_in_mask(miss);
            in_hits[k] = rank_in_mask(hbm) | (rank_in_mask(host) << 16);
        }
        Scan::run(scan, tile, totals, before, lds, a.err);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (r[k] < 0) continue;
            const uint32_t ur = static_cast<uint32_t>(r[k]);
            const int32_t j = static_cast<int32_t>(j0 + k * kScanBlock);
            const uint32_t hits = before[1][k] + in_hits[k];
            if (ur < n_cached) {
                if (ur >= n_hbm) {
                    const uint32_t w = lds.excl[2] + (hits >> 16);
                    a.lists.pos[1][w] = j;
                    a.lists.slot[1][w] = static_cast<int32_t>(ur - n_hbm);
                } else if (!a.hbm_direct) {                  // (else copied without a list)
                    const uint32_t w = lds.excl[1] + (hits & 0xffffu);
                    a.lists.pos[0][w] = j;
                    a.lists.slot[0][w] = static_cast<int32_t>(ur);
                }
            } else {
                const int64_t w = static_cast<int64_t>(lds.excl[0]) + before[0][k] + in_class[k];
                if (w < a.miss_cap) {
                    a.miss_pos[w] = j;
                    a.miss_id[w] = id[k];
                    a.miss_slot[w] = static_cast<int32_t>(ur - n_cached);
                }
            }
        }
        if (tile == n_tiles - 1 && threadIdx.x == 0) {
            const int64_t c0 = static_cast<int64_t>(lds.excl[1]) + lds.agg[1];
            const int64_t c1 = static_cast<int64_t>(lds.excl[2]) + lds.agg[2];
            const int64_t c2 = static_cast<int64_t>(lds.excl[0]) + lds.agg[0];
            a.lists.count[0] = c0; a.lists.count[1] = c1; a.lists.count[2] = c2;
            if (a.stats_out) { a.stats_out[0] = n; a.stats_out[1] = c0; a.stats_out[2] = c1; a.stats_out[3] = c2; }
            if (a.learn) { a.learn[0] = n; a.learn[1] = c0; a.learn[2] = c1; a.learn[3] = c2; }
            if (c2 > a.miss_cap) raise(a.err, kErrCapacity);
        }
    }
}

// With all nodes in HBM nothing can be listed (no ID has a host row, none can miss), and of the partition only the counts are
// left: no order, so no tickets and no look-back.  Bound by the chain ID, rank, sums, one atomic per workgroup; the last
// workgroup to add its count writes the stats and leaves the word at zero.  Where every node has a rank, which the build of the
// map has found out, the ranks need not be read for it.  Call on 100 k rows of 64 bytes, copied beside it: 12.0 us with the partition,
// 10.1 with a count that reads the ranks, 7.5 with this; 243 k rows of 2 KB 174.3 -> 167.2.
constexpr unsigned kCountWorkgroups = 64;              // (a word that all add to takes about 10 ns for each)
struct CountCopyArgs {
    const int32_t* ids;
    const int32_t* rank;
    const chunk16* table;
    chunk16* out;
    int64_t *count, *stats_out, *learn;
    const int64_t* holes;
    unsigned long long* word;    // zero between launches (the scan's ticket)
    int32_t* err;
    uint32_t n, n_nodes;         // (all nodes are in HBM)
    int32_t chunks;
    uint32_t count_blocks;       // the workgroups before those that copy
};
// (a launch with 128 bytes of arguments or more costs the host 0.5 us more)
static_assert(sizeof(CountCopyArgs) <= 112, "arguments of a cheap launch");
__device__ __forceinline__ void count_role(const CountCopyArgs& a) {
    __shared__ uint32_t s_hits[kScanWaves];
    constexpr int kAhead = 4;
    const uint32_t n = a.n, nrb = a.count_blocks, step = nrb * kScanBlock;
    const bool whole = *a.holes == 0;
    uint32_t hits = 0;
    for (uint64_t j0 = blockIdx.x * kScanBlock + threadIdx.x; j0 < n; j0 += static_cast<uint64_t>(kAhead) * step) {
        int32_t id[kAhead], r[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) id[k] = a.ids[j0 + static_cast<uint64_t>(k) * step < n ? j0 + static_cast<uint64_t>(k) * step : j0];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const bool ok = static_cast<uint32_t>(id[k]) < a.n_nodes;
            if (!ok) raise(a.err, kErrData);
            r[k] = ok ? 0 : -1;
            if (!whole && ok) r[k] = a.rank[id[k]];
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) hits += j0 + static_cast<uint64_t>(k) * step < n && static_cast<uint32_t>(r[k]) < a.n_nodes ? 1u : 0u;
    }
    const uint32_t sum = dpp_sum(hits);
    if (lane_id() == 0) s_hits[wave_id()] = sum;
    __syncthreads();
    if (threadIdx.x != 0) return;
    unsigned long long mine = 1ull << 40;              // {workgroups done : 24 | hits : 40}
#pragma unroll
    for (int w = 0; w < kScanWaves; ++w) mine += s_hits[w];
    const unsigned long long all = atomicAdd(a.word, mine) + mine;
    if (all >> 40 != nrb) return;
    __hip_atomic_store(a.word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t c0 = static_cast<int64_t>(all & ((1ull << 40) - 1));
    a.count[0] = c0; a.count[1] = a.count[2] = 0;
    if (a.stats_out) { a.stats_out[0] = n; a.stats_out[1] = c0; a.stats_out[2] = 0; a.stats_out[3] = 0; }
    if (a.learn) { a.learn[0] = n; a.learn[1] = c0; a.learn[2] = 0; a.learn[3] = 0; }
}

// The HBM tier's rows without a list: out[j, :] = table[rank[ids[j]], :] for the IDs whose rank is in the tier.  A group of L
// lanes owns a row, as in copy_rows (gather_dev.hpp); it reads the ID and its rank by itself, so the copy need not wait for the
// partition, which makes the other lists in the same launch.
struct DirectArgs {
    const int32_t* ids;
    const int32_t* rank;
    uint32_t n, n_nodes, n_hbm;
    const chunk16* table;
    chunk16* out;
    int32_t chunks;
};
template <int L, int CPL>
__device__ __forceinline__ void direct_rows(const DirectArgs& a, uint32_t rb, uint32_t nrb) {
    constexpr int kLanes = L == 0 ? kWave : L, kGroups = kScanBlock / kLanes;
    const int l = threadIdx.x % kLanes;
    for (uint32_t j = rb * kGroups + threadIdx.x / kLanes; j < a.n; j += nrb * kGroups) {
        const uint32_t id = static_cast<uint32_t>(a.ids[j]);
        if (id >= a.n_nodes) continue;                           // reported by the partition
        const uint32_t r = static_cast<uint32_t>(a.rank[id]);
        if (r >= a.n_hbm) continue;
        const chunk16* src = a.table + static_cast<int64_t>(r) * a.chunks;
        chunk16* o = a.out + static_cast<int64_t>(j) * a.chunks;
        if constexpr (L == 0) {
            for (int c = l; c < a.chunks; c += kWave) store16(o + c, load16(src + c));
        } else {
            chunk16 v[CPL == 0 ? 1 : CPL];
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                if (l + c * L < a.chunks) v[c] = load16(src + l + c * L);
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                if (l + c * L < a.chunks) store16(o + l + c * L, v[c]);
        }
    }
}

// Lookup and partition, and beside it, if r_copy has workgroups, the copy of the HBM tier's rows.  As two launches the copy
// waited 8 to 13 us for lists it does not need: 243 k rows of 2 KB 179.1 -> 174.5 us for the call, 100 k rows of 64 bytes
// 15.0 -> 12.0.  (One row per group and step: with two 177.0 and 13.4 us, with four 184.2 and 13.7.)  When it does not pay:
// copy_beside_lookup below.
template <int K, int L, int CPL>
__global__ __launch_bounds__(kScanBlock) void lookup_copy_kernel(PartitionArgs a, DirectArgs d, Role r_part, Role r_copy) {
    if (r_part.mine()) {
        partition_role<K>(a, r_part.rb(), r_part.blocks);
        return;
    }
    direct_rows<L, CPL>(d, r_copy.rb(), r_copy.blocks);
}

// The same with all nodes in HBM: the count, and beside it the copy.
template <int L, int CPL>
__global__ __launch_bounds__(kScanBlock) void count_copy_kernel(CountCopyArgs a) {
    if (blockIdx.x < a.count_blocks) {
        count_role(a);
        return;
    }
    direct_rows<L, CPL>(DirectArgs{a.ids, a.rank, a.n, a.n_nodes, a.n_nodes, a.table, a.out, a.chunks}, blockIdx.x - a.count_blocks, gridDim.x - a.count_blocks);
}

unsigned grid_for(int64_t n, unsigned cap_blocks) {
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > cap_blocks) b = cap_blocks;
    return static_cast<unsigned>(b);
}

}  // namespace

hipError_t launch_rank_build(hipStream_t stream, const int32_t* order, int64_t n_nodes, int32_t* rank, int64_t* holes, uint32_t* cursors, void* scratch,
                             size_t scratch_bytes, int32_t* err) {
    const size_t nodes = static_cast<size_t>(n_nodes), runs_at = sizeof(unsigned long long) * nodes, bytes = runs_at + sizeof(uint32_t) * (nodes / kWave);
    if (scratch && n_nodes >= kInvertMin && n_nodes <= kInvertMax && scratch_bytes >= bytes) {
        uint32_t shift = kInvertMaxShift;                // 256 buckets or more, so that every CU has one or two
        while (shift > 10 && (n_nodes >> shift) < 256) --shift;
        const uint32_t n = static_cast<uint32_t>(n_nodes);
        unsigned char* p = static_cast<unsigned char*>(scratch);
        const InvertScratch s{cursors, reinterpret_cast<unsigned long long*>(p), reinterpret_cast<uint32_t*>(p + runs_at)};
        const dim3 block(kInvertBlock);
        hipLaunchKernelGGL(rank_split_kernel, dim3((n + kHandTile - 1) / kHandTile), dim3(kHandBlock), 0, stream, order, n, shift, s, rank, holes, err);
        const dim3 buckets((n + (1u << shift) - 1) >> shift);
        if (shift == kInvertMaxShift) hipLaunchKernelGGL(rank_place_kernel<kInvertMaxShift>, buckets, block, 0, stream, order, n, shift, s, rank, holes, err);
        else hipLaunchKernelGGL(rank_place_kernel<kInvertMaxShift - 1>, buckets, block, 0, stream, order, n, shift, s, rank, holes, err);
        return hipGetLastError();
    }
    const dim3 grid(grid_for(n_nodes, 8192)), block(kBlock);
    hipLaunchKernelGGL(rank_fill_kernel, grid, block, 0, stream, rank, n_nodes, holes);
    hipLaunchKernelGGL(rank_scatter_kernel, grid, block, 0, stream, order, n_nodes, rank, err);
    hipLaunchKernelGGL(rank_check_kernel, grid, block, 0, stream, rank, n_nodes, holes, err);
    return hipGetLastError();
}

// The copy beside the lookup takes a step for every ID, hit or not, while the one by list takes steps for hits only and knows
// their rows already.  So it pays as long as the steps are few enough to be over while the partition runs, or nearly all of
// them are hits.  What share of the IDs hits is known once they have been looked up; the tier's share of the nodes, below
// which a tier of the hottest nodes does not fall, stands in for it.  Measured, us for the call by list / beside the lookup, IDs
// drawn uniformly, rows of 64 / 512 / 2048 bytes:
//   1/100 of the nodes in HBM   4096 steps 18.8/22.2 (524 k IDs)  10.5/8.3  9.9/7.9     8192 steps 33.2/43.5  13.6/17.2  11.2/11.8
//   7 tenths                    4096 steps 31.4/29.6              19.4/16.7 25.7/20.7   8192 steps 58.0/57.1  31.2/33.5  42.7/38.2
//   9 tenths                    8192 steps 64.0/60.8  36.3/35.2  51.7/46.3    16384 steps -  59.4/60.1  95.0/93.5   32768 -  104/120  177/172
//   3 tenths                    8192 steps of 2048 / 4096 bytes: 25.3/25.7  40.7/36.8 (7 tenths 42.7/38.2  77.3/70.8)
// With four pieces per lane (rows of 2 to 4 KB) it stops paying earlier: 4096 bytes, 9 tenths in HBM, 16384 steps 195.3/199.4.
// With all nodes in HBM the lookup beside the copy only counts (count_role), and that way is the quicker one for all rows of up to 2 KB
// and above 4 KB: us for the call by list or beside a partition, whichever the partition leaves quicker / beside the count,
//   rows of 64     131 k IDs 14.5/7.9   524 k 35.5/24.4  2.1 M 131/86.6
//   512            65 k 18.6/14.6       262 k 62.6/51.6  1.0 M 220/194
//   2048           65 k 50.2/47.0       262 k 188/181    524 k 380/362
//   4096           65 k 97.6/93.7       131 k 193/190    262 k 376/385   (the line)
//   8192           33 k 95.9/93.9       131 k 375/364
bool copy_beside_lookup(int64_t n, int64_t n_nodes, int64_t n_hbm, int32_t chunks) {
    int64_t lanes = 4;
    while (lanes < chunks && lanes < kWave) lanes <<= 1;
    const int64_t steps = (n * lanes + kScanBlock - 1) / kScanBlock;
    if (n_hbm == n_nodes) return chunks <= 128 || chunks > 256 || steps <= 16384;
    if (10 * n_hbm < 9 * n_nodes) return n <= 262144 && steps <= (chunks >= 128 && 10 * n_hbm >= 3 * n_nodes ? 8192 : 4096);
    if (chunks > 128 && chunks <= 256) return steps <= 8192;
    return chunks >= 128 || steps <= 8192;
}

hipError_t launch_lookup_partition(hipStream_t stream, const int32_t* ids, int64_t n,
                                   const int32_t* rank, int64_t n_nodes, int64_t n_hbm, int64_t n_host,
                                   const TierLists& lists, int32_t* miss_pos, int32_t* miss_id,
                                   int32_t* miss_slot, int64_t miss_cap, int64_t* stats_out, int64_t* learn,
                                   const ScanState& scan, const int64_t* holes, int32_t* err, const chunk16* copy_table, chunk16* copy_out,
                                   int32_t chunks) {
    const bool copy = copy_table && n > 0 && n_hbm > 0;
    const PartitionArgs a{ids, Count{nullptr, n}, rank, n_nodes, n_hbm, n_host, lists, miss_pos, miss_id, miss_slot, miss_cap,
                          stats_out, learn, copy, scan, err};
    const DirectArgs d{ids, rank, static_cast<uint32_t>(n), static_cast<uint32_t>(n_nodes), static_cast<uint32_t>(n_hbm), copy_table, copy_out, chunks};
    const bool count_only = copy && n_hbm == n_nodes;
    const Role r_part{0, scan_workgroups(n, count_only ? kCountWorkgroups : kScanMaxWorkgroups)};
    const CountCopyArgs counting{ids, rank, copy_table, copy_out, lists.count, stats_out, learn, holes, reinterpret_cast<unsigned long long*>(scan.ticket), err,
                                 static_cast<uint32_t>(n), static_cast<uint32_t>(n_nodes), chunks, r_part.blocks};
    const dim3 block(kScanBlock);
    // One row per group and step, and as many workgroups as the list has steps: short-lived workgroups on consecutive rows copy
    // fastest (gather_dev.hpp).
#define HELIOS_CALL_(L, CPL, R)                                                                                              \
    do {                                                                                                                     \
        constexpr int64_t step = kScanBlock / ((L) == 0 ? kWave : (L));                                                     \
        int64_t nb = copy ? (n + step - 1) / step : 0;                                                                       \
        if (nb > kMaxRoleBlocks) nb = kMaxRoleBlocks;                                                                        \
        const Role r_copy{r_part.blocks, static_cast<uint32_t>(nb)};                                                         \
        const dim3 grid(r_part.blocks + r_copy.blocks);                                                                      \
        if (count_only) hipLaunchKernelGGL((count_copy_kernel<L, CPL>), grid, block, 0, stream, counting);                   \
        else if (n <= kScanOneItemMax) hipLaunchKernelGGL((lookup_copy_kernel<1, L, CPL>), grid, block, 0, stream, a, d, r_part, r_copy); \
        else hipLaunchKernelGGL((lookup_copy_kernel<kScanMaxItems, L, CPL>), grid, block, 0, stream, a, d, r_part, r_copy);  \
    } while (0)
    HELIOS_COPY_NEAR_SHAPE(copy ? chunks : 1, HELIOS_CALL_);
#undef HELIOS_CALL_
    return hipGetLastError();
}

}  // namespace helios
