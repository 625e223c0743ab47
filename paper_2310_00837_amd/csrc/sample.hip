// Hop 0 of seed lists that are too long for the count that the sampling pass folds in (sample_dev.hpp).
//
// Up to 16 384 seeds with fan-outs up to 8, and up to 32 768 with fan-outs of 9 to 64, are counted and sampled in one launch
// (sample_counted_kernel), unless the samples go where the seeds are.  Longer lists, and fan-outs above 64, get a count pass as a kernel of its own first: every
// thread reads the row bounds of its frontier nodes, the sample counts min(deg, fanout) are scanned in the workgroup
// and chained across workgroups (TileScan in scan.hpp) into indptr, each node's place in `flat`.
#include "kernels.hpp"

#include <algorithm>

namespace helios {

namespace {

struct CountArgs {
    const int64_t* offsets;
    int64_t n_nodes;
    const int32_t* frontier;
    BatchFeed feed;               // recorded batch: the batch's variables come from the host's ring, and the frontier is their seeds
    int32_t* frontier_out;        // nullable: receives a copy of the frontier
    Count n;
    int32_t fanout;
    int64_t* indptr;
    int64_t flat_cap;
    int64_t* n_flat_dev;
    int64_t* size_out;            // nullable: [0] = frontier size, [1] = sample-list size
    ScanState scan;
    int32_t* err;
};

// Bound by its chain of dependent reads, as a compaction is (compact_dev.hpp), and built like it.  The batch's variables are read
// through a pointer: a copy of the struct per thread ends up in LDS, addressed by way of the dispatch packet, which is in host
// memory, and 196 workgroups then take 13 us to begin.  Measured, count and sampling of 100 k seeds with fan-out 5: 18.4 us (27.0
// with the copy and two guarded 8-byte reads per node).
template <int K>
__global__ __launch_bounds__(kScanBlock) void frontier_count_kernel(CountArgs a) {
    using Scan = TileScan<1, 1, K>;
    __shared__ typename Scan::Lds lds;
    // A recorded batch starts here: every workgroup reads the batch's variables from the slot of the host's ring
    // that the count of batches run so far selects, and the first workgroup leaves them in device memory for the
    // kernels that follow (the batch's first compaction advances the count).
    const int32_t* frontier = a.frontier;
    ScanState scan = a.scan;
    if (a.feed.ring) {
        const BatchVars* bv = a.feed.ring + *a.feed.batches_run % a.feed.ring_slots;
        frontier = bv->seeds;
        scan.vars = nullptr;
        scan.epoch += bv->epoch_base;
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.feed.vars_out = *bv;
    }
    const uint32_t n = static_cast<uint32_t>(a.n.get());
    const uint32_t n_tiles = (n + K * kScanBlock - 1) / (K * kScanBlock);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (a.size_out) a.size_out[0] = n;
        if (n == 0) {                            // empty frontier: empty hop
            a.indptr[0] = 0;
            *a.n_flat_dev = 0;
            if (a.size_out) a.size_out[1] = 0;
        }
    }
    if (blockIdx.x >= n_tiles) return;
    const uint32_t n_wgs = gridDim.x < n_tiles ? gridDim.x : n_tiles;
    for (uint32_t tile = Scan::take_ticket(scan, n_tiles, n_wgs, lds); tile < n_tiles;
         tile = n_wgs < n_tiles ? Scan::take_ticket(scan, n_tiles, n_wgs, lds) : n_tiles) {
        const uint32_t j0 = tile * (K * kScanBlock) + threadIdx.x;
        int32_t v[K];
        uint32_t totals[1][K], before[1][K], local[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = frontier[j0 + k * kScanBlock < n ? j0 + k * kScanBlock : 0];
        // (all row bounds are asked for before the first is used, unguarded: a node that is none reads row 0)
        RowBounds row[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool ok = v[k] >= 0 && static_cast<int64_t>(v[k]) < a.n_nodes;
            row[k] = RowBounds{0, 0};
            if (a.n_nodes > 0) row[k] = row_bounds(a.offsets, ok ? static_cast<uint32_t>(v[k]) : 0u);      // (uniform guard)
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t j = j0 + k * kScanBlock;
            const bool ok = v[k] >= 0 && static_cast<int64_t>(v[k]) < a.n_nodes;
            const int64_t d = ok ? row[k].hi - row[k].lo : 0;
            const bool bad = d < 0 || d > 0x7fffffffLL;
            if (j < n && a.frontier_out && a.frontier_out != frontier) a.frontier_out[j] = v[k];
            if (j < n && (!ok || bad)) raise(a.err, kErrData);
            const int64_t f = a.fanout > 0 ? a.fanout : 0;
            const uint32_t cnt = j >= n || bad ? 0u : static_cast<uint32_t>(d < f ? d : f);
            const uint32_t inc = dpp_inclusive_scan(cnt);
            totals[0][k] = lane_value(inc, kWave - 1);
            local[k] = inc - cnt;
        }
        Scan::run(scan, tile, totals, before, lds, a.err);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (j0 + k * kScanBlock < n) a.indptr[j0 + k * kScanBlock] = static_cast<int64_t>(lds.excl[0]) + before[0][k] + local[k];
        if (tile == n_tiles - 1 && threadIdx.x == 0) {
            const int64_t total = static_cast<int64_t>(lds.excl[0]) + lds.agg[0];
            a.indptr[n] = total;
            *a.n_flat_dev = total;
            if (a.size_out) a.size_out[1] = total;
            if (total > a.flat_cap) raise(a.err, kErrCapacity);
        }
    }
}

// Count and sampling of hop 0 in one launch: a tile of at most 64 seeds per workgroup, a group of G lanes for each, in R rounds.  The
// first wave counts the tile's samples and publishes their sum; every group draws, and reads the neighbours it has drawn, which takes no place in `flat`;
// then the first wave sums up the totals of the tiles before (512 at most, eight words per lane), and the samples go where they
// belong.  Tiles are handed out by tickets (scan.hpp), so one waits only for tiles that have started.
// Bound by its chain of dependent reads: ticket, seed, row bounds, neighbour, tables.  10 000 seeds with fan-out 25: 12.1 us,
// as two launches 5.6 and 9.5.
constexpr uint32_t kCountedTiles = 512;
template <int G, int B, int R>
__global__ __launch_bounds__(B) void sample_counted_kernel(HopArgs a, ScanState scan, uint32_t per_tile) {
    constexpr uint32_t kGroups = B / G;
    static_assert(R * kGroups <= kWave && kCountedTiles % kWave == 0, "one wave counts a tile");
    __shared__ OwnNodesOf<R * kGroups> own;
    __shared__ uint32_t s_ticket, s_excl;
    const uint32_t n = static_cast<uint32_t>(a.n_frontier.host), n_tiles = (n + per_tile - 1) / per_tile;
    stamp_start(a.stamps, blockIdx.x);
    if (threadIdx.x == 0) {
        const uint32_t t = atomicAdd(scan.ticket, 1u);
        if (t == n_tiles - 1) __hip_atomic_store(scan.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_ticket = t;
    }
    // (a recorded batch starts here, as in frontier_count_kernel)
    const int32_t* frontier = a.frontier;
    uint64_t rng_seed = a.rng_seed;
    uint32_t which = a.batch.which;
    if (a.feed.ring) {
        const BatchVars* bv = a.feed.ring + *a.feed.batches_run % a.feed.ring_slots;
        frontier = bv->seeds;
        rng_seed = bv->rng_seed;
        which = bv->table % kBatchTables;
        scan.epoch += bv->epoch_base;
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.feed.vars_out = *bv;
    }
    __syncthreads();
    const uint32_t tile = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(s_ticket))), first = tile * per_tile;
    const bool counts = threadIdx.x < kWave;
    const uint32_t lane = static_cast<uint32_t>(lane_id()), i = first + lane;
    const bool mine = counts && lane < per_tile && i < n;
    const int f = a.fanout > 0 ? a.fanout : 0;
    uint32_t local = 0, total = 0;
    if (counts) {
        const int32_t v = frontier[mine ? i : n - 1];
        const bool ok = v >= 0 && static_cast<int64_t>(v) < a.n_nodes;
        RowBounds row{0, 0};
        if (a.n_nodes > 0) row = row_bounds(a.offsets, ok ? static_cast<uint32_t>(v) : 0u);      // (uniform guard)
        const int64_t d = ok ? row.hi - row.lo : 0;
        const bool bad = d < 0 || d > 0x7fffffffLL;
        if (mine && (!ok || bad)) raise(a.err, kErrData);
        const int32_t deg = bad ? 0 : static_cast<int32_t>(d);
        const uint32_t cnt = mine ? static_cast<uint32_t>(deg < f ? deg : f) : 0u, inc = dpp_inclusive_scan(cnt);
        local = inc - cnt;
        total = lane_value(inc, kWave - 1);
        if (lane == 0) scan_store(scan.status + tile, scan_pack(scan.epoch, kFlagAggregate, total));
        if (lane < R * kGroups) {
            own.v[lane] = v;
            own.base[lane] = row.lo;
            own.deg[lane] = mine ? deg : 0;
            own.out[lane] = local;
        }
        if (mine && a.frontier_out && a.frontier_out != frontier) a.frontier_out[i] = v;
    }
    __syncthreads();
    const uint32_t g = threadIdx.x / G;
    const int l = threadIdx.x % G;
    int32_t id[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t q = r * kGroups + g;
        const int32_t deg = own.deg[q], s = pick<G>(rng_seed, own.v[q], a.hop, deg, f, l);
        id[r] = -1;
        if (l < (deg < f ? deg : f)) id[r] = a.indices[own.base[q] + s];
    }
    if (counts) {
        uint32_t before = 0;
        unsigned long long w[kCountedTiles / kWave];
#pragma unroll
        for (uint32_t q = 0; q < kCountedTiles / kWave; ++q)
            if (q * kWave < tile) w[q] = scan_load(scan.status + min(q * kWave + lane, tile - 1));
#pragma unroll
        for (uint32_t q = 0; q < kCountedTiles / kWave; ++q) {
            if (q * kWave >= tile) continue;
            for (uint32_t budget = kScanSpinBudget; __ballot(w[q] >> 34 != scan.epoch) != 0;) {
                if (--budget == 0) {                               // gave up: report, and let the launch drain
                    raise(a.err, kErrInternal);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                w[q] = scan_load(scan.status + min(q * kWave + lane, tile - 1));
            }
            before += q * kWave + lane < tile ? static_cast<uint32_t>(w[q]) : 0u;
        }
        const uint32_t excl = dpp_sum(before);
        if (lane == 0) s_excl = excl;
        if (mine) a.indptr_out[i] = static_cast<int64_t>(excl) + local;
        if (tile == n_tiles - 1 && lane == 0) {
            const int64_t all = static_cast<int64_t>(excl) + total;
            a.indptr_out[n] = all;
            *a.n_flat_dev = all;
            if (a.size_out) { a.size_out[0] = n; a.size_out[1] = all; }
            if (all > a.flat_cap) raise(a.err, kErrCapacity);
        }
    }
    __syncthreads();
    SampleTables tabs{a.hop_table, nullptr, 0, nullptr, a.cat_out, 0, 0};
    if (a.batch.table0) {
        tabs.batch_table = a.batch.table(which);
        tabs.batch_mask = a.batch.n_slots - 1;
        tabs.batch_slot_of = a.batch.slot_of(which);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t q = r * kGroups + g, place = first + q;
        if (q >= per_tile || place >= n) continue;
        const int32_t v = own.v[q], deg = own.deg[q];
        const uint32_t at = s_excl + own.out[q] + static_cast<uint32_t>(l);
        const bool sample = l < (deg < f ? deg : f) && static_cast<int64_t>(at) < a.flat_cap, seed = tabs.batch_table && f < G && l == f;
        if (sample || seed) put_id(tabs, a.n_nodes, a.err, a.flat, sample ? id[r] : v, sample, at, sample ? static_cast<uint32_t>(a.n_seeds) + at : place);
        if (tabs.batch_table && f == G && l == 0) put_id(tabs, a.n_nodes, a.err, a.flat, v, false, 0, place);
    }
    if (a.batch.table0) {
        const uint32_t sum = dpp_sum(tabs.batch_claims);
        if (lane == 0) a.claims[blockIdx.x * (B / kWave) + wave_id()] = sum;
    }
    stamp_end(a.stamps, blockIdx.x, gridDim.x);
}

}  // namespace

// Seeds of a tile: a tile for each CU, or two, but 32 seeds or more, and no more tiles than there are status words.  (10 000 seeds with
// fan-outs 25 and 10: 250 tiles of 40 34.5 us, 313 of 32 35.8; 2 049 seeds: 65 tiles of 32 21.9, 129 of 16 23.3, 33 of 64 24.8.)
static int64_t counted_per_tile(int64_t n, uint32_t stride) {
    const int64_t tiles = n <= 256 * kWave ? 256 : kCountedTiles;
    return std::max<int64_t>({(n + tiles - 1) / tiles, (n + stride - 1) / stride, 32});
}

// Measured, us for helios_sample as two launches / as one: fan-outs 25 and 10, 2 049 seeds 25.2/21.9, 8 192 34.0/31.0, 16 384 45.7/42, 32 768 65.5/63;
// 10 alone, 2 049 10.8/7.8, 16 384 10.9/7.6, 32 768 13.7/11.8; 60 alone, 10 000 13.8/11.4, 32 768 22.2/19.6; 8 alone, 16 384 11.0/7.5, 32 768 (two
// tiles for each CU) 11.3/11.6, so that is left out.  Four streams at the same time, us for four calls: 9 000 seeds with 10 47/31, with 25 and 10
// 80/71.  Recorded batches, rows of 32 bytes in HBM, one after the other (alone; three streams at the same time, for three): 2 049 seeds with 25
// and 10 60.5/56.6 (69.0/65.0; 85.7/83.3), 9 000 99.4/96.2 (108/105; 195/193), 9 000 with 10 alone 39.7/35.0 (48.2/42.6; 60/56), 16 384 with 8
// 47.2/42.0 (55.8/50.9; 67.6/64.3), 32 768 with 10 61.3/56.2 (69.5/64.4; 100/101), 9 000 with 60 47.9/42.0 (56.6/51.4; 70/66).
unsigned sample_counted_blocks(int32_t fanout, int64_t n, uint32_t stride, unsigned* waves) {
    const int64_t per_tile = counted_per_tile(n, stride), lanes = group_lanes(fanout);
    *waves = lanes == 8 ? 8 : 16;
    if (fanout > 64 || per_tile > kWave || (lanes == 8 && n > 256 * kWave)) return 0;
    return static_cast<unsigned>((n + per_tile - 1) / per_tile);
}

hipError_t launch_sample_counted(hipStream_t stream, const HopArgs& a, const ScanState& scan) {
    unsigned waves;
    const dim3 blocks(sample_counted_blocks(a.fanout, a.n_frontier.host, scan.stride, &waves)), block(waves * kWave);
    if (blocks.x < 2) return hipErrorInvalidValue;
    const uint32_t per_tile = static_cast<uint32_t>(counted_per_tile(a.n_frontier.host, scan.stride));
    const int lanes = group_lanes(a.fanout);
    if (lanes == 8) hipLaunchKernelGGL((sample_counted_kernel<8, 512, 1>), blocks, block, 0, stream, a, scan, per_tile);
    else if (lanes == 16) hipLaunchKernelGGL((sample_counted_kernel<16, 1024, 1>), blocks, block, 0, stream, a, scan, per_tile);
    else if (lanes == 32 && per_tile <= 32) hipLaunchKernelGGL((sample_counted_kernel<32, 1024, 1>), blocks, block, 0, stream, a, scan, per_tile);
    else if (lanes == 32) hipLaunchKernelGGL((sample_counted_kernel<32, 1024, 2>), blocks, block, 0, stream, a, scan, per_tile);
    else if (per_tile <= 32) hipLaunchKernelGGL((sample_counted_kernel<64, 1024, 2>), blocks, block, 0, stream, a, scan, per_tile);
    else hipLaunchKernelGGL((sample_counted_kernel<64, 1024, 4>), blocks, block, 0, stream, a, scan, per_tile);
    return hipGetLastError();
}

hipError_t launch_frontier_count(hipStream_t stream, const CsrView& g, const int32_t* frontier, const BatchFeed& feed,
                                 int32_t* frontier_out, Count n, int64_t n_max, int32_t fanout, int64_t* indptr,
                                 int64_t flat_cap, int64_t* n_flat_dev, int64_t* size_out, const ScanState& scan, int32_t* err) {
    CountArgs a{g.offsets, g.n_nodes, frontier, feed, frontier_out, n, fanout, indptr, flat_cap, n_flat_dev, size_out, scan, err};
    const dim3 grid(scan_workgroups(n_max, kScanMaxWorkgroups)), block(kScanBlock);      // (the first workgroup also writes the sizes of an empty hop)
    if (n_max <= kScanOneItemMax) hipLaunchKernelGGL(frontier_count_kernel<1>, grid, block, 0, stream, a);
    else hipLaunchKernelGGL(frontier_count_kernel<kScanMaxItems>, grid, block, 0, stream, a);
    return hipGetLastError();
}

}  // namespace helios
