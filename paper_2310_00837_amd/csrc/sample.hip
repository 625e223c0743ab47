// Count pass of hop 0 as a kernel of its own, for seed lists too long for the count that the
// sampling pass folds in (sample_dev.hpp): every thread reads the row bounds of its frontier nodes,
// the sample counts min(deg, fanout) are scanned in the workgroup and chained across workgroups
// (TileScan in scan.hpp) into indptr, each node's place in `flat`.
#include "kernels.hpp"

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

}  // namespace

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
