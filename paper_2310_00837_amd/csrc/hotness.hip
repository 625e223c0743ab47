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
// batches, so that one pass is the rule up to 2048 batches.  A pass is three launches:
//   count    every tile of 8192 pairs counts its digits (LDS);
//   scan     per digit, a prefix sum over the tiles, 16 digits to a workgroup;
//   scatter  a tile ranks its pairs (wave ballots find the lanes with the same
//            digit, a counter per wave and digit in LDS carries the rank along),
//            puts them into order in LDS and writes them out as runs.
// Bins are numbered from the highest digit down, so each pass goes out in
// descending digit order.  Nothing waits for another workgroup.
//
// What bounds it: the scatter's ballots and LDS traffic first, memory second.
// Measured at 8 M nodes with counts up to 512: count 17 us, scan 9, scatter 45
// (its 64 MB would take 11 us), and 2-4 us for each launch of a pass that is left
// out; 96 us in all.  Sixteen two-bit splits by chained scan, which this
// replaces, took 2 300 us (138 each: 3 900 tickets on one address).
//
// One workgroup of the scatter runs per CU: it takes 81 984 bytes of LDS, 64 more than half of what a CU has, and 87 registers
// where two workgroups of 16 waves would have to do with 64.  So of a grid of 512 half start when the others end.
#include "kernels.hpp"

namespace helios {

namespace {

constexpr int kSortBlock = 1024;
constexpr int kSortWaves = kSortBlock / kWave;
constexpr int kSortItems = 8;                             // pairs per thread
constexpr int kSortTile = kSortBlock * kSortItems;        // 8192
constexpr int kDigitBits = 11;
constexpr int kBins = 1 << kDigitBits;
constexpr int kSortPasses = 3;
constexpr int kScanBins = 16;                             // bins per workgroup of the scan
constexpr int kWalkers = kSortBlock / kScanBins;          // each takes a share of the tiles
constexpr unsigned kSortMaxWorkgroups = 512;              // they loop over the tiles (see the end of the head comment)
static_assert(kWalkers == kWave && kSortWaves == kScanBins, "one wave scans the walkers of one bin");

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
    uint32_t* tile_counts;       // [n_tiles][kBins]; after the scan: pairs of the bin in the tiles before
    uint32_t* totals;            // [kBins]
    uint32_t* tile_bits;         // [n_tiles][2]: bits set in some count, bits clear in some count
    uint32_t* varying;           // bits that are not the same in all counts (from the first pass's scan on)
    int pass;
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

__global__ __launch_bounds__(kSortBlock) void sort_count_kernel(SortArgs a) {
    __shared__ uint32_t s_hist[kBins];
    __shared__ uint32_t s_set, s_clear;
    const SortStep step(a.pass, a.pass == 0 ? 0u : *a.varying);
    if (!step.active) return;
    const int32_t* keys = step.before == 0 ? a.counts : a.keys[(step.before - 1) & 1];
    for (uint32_t tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
        for (int q = threadIdx.x; q < kBins; q += kSortBlock) s_hist[q] = 0;
        if (threadIdx.x == 0) s_set = s_clear = 0;
        __syncthreads();
        const uint32_t i0 = tile * kSortTile + threadIdx.x;
        int32_t key[kSortItems];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) key[k] = keys[i0 + k * kSortBlock < a.n ? i0 + k * kSortBlock : a.n - 1];
        uint32_t set = 0, clear = 0;
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            set |= static_cast<uint32_t>(key[k]);
            clear |= ~static_cast<uint32_t>(key[k]);
            const uint32_t bin = bin_of(key[k], a.pass);
            uint64_t rest = __ballot(i0 + k * kSortBlock < a.n);
            // Most counts are one of a few small numbers: the bins of the first lanes left are counted for the whole
            // wave at once, so that the lanes do not queue up at one LDS word.
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                if (rest == 0) break;
                const uint32_t lead = static_cast<uint32_t>(__ffsll(static_cast<long long>(rest)) - 1);
                const uint32_t lead_bin = lane_value(bin, lead);
                const uint64_t same = __ballot(bin == lead_bin) & rest;
                if (static_cast<uint32_t>(lane_id()) == lead) atomicAdd(s_hist + bin, static_cast<uint32_t>(__popcll(same)));
                rest &= ~same;
            }
            if ((rest >> lane_id()) & 1u) atomicAdd(s_hist + bin, 1u);
        }
        if (a.pass == 0) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                set |= __shfl_xor(set, d, kWave);
                clear |= __shfl_xor(clear, d, kWave);
            }
            if (lane_id() == 0) {
                atomicOr(&s_set, set);
                atomicOr(&s_clear, clear);
            }
        }
        __syncthreads();
        for (int q = threadIdx.x; q < kBins; q += kSortBlock) a.tile_counts[static_cast<size_t>(tile) * kBins + q] = s_hist[q];
        if (a.pass == 0 && threadIdx.x == 0) {
            a.tile_bits[2 * tile] = s_set;
            a.tile_bits[2 * tile + 1] = s_clear;
        }
        __syncthreads();
    }
}

// Workgroup b: the bins [16 b, 16 b + 16) over all tiles, by 64 walkers that take consecutive tiles each.  In the first
// pass one workgroup more gathers which bits vary.
__global__ __launch_bounds__(kSortBlock) void sort_scan_kernel(SortArgs a) {
    __shared__ uint32_t s_sum[kWalkers][kScanBins + 1];
    __shared__ uint32_t s_set, s_clear;
    if (blockIdx.x == kBins / kScanBins) {
        if (threadIdx.x == 0) s_set = s_clear = 0;
        __syncthreads();
        uint32_t set = 0, clear = 0;
        for (uint32_t t = threadIdx.x; t < a.n_tiles; t += kSortBlock) {
            set |= a.tile_bits[2 * t];
            clear |= a.tile_bits[2 * t + 1];
        }
        atomicOr(&s_set, set);
        atomicOr(&s_clear, clear);
        __syncthreads();
        if (threadIdx.x == 0) *a.varying = s_set & s_clear;
        return;
    }
    if (a.pass > 0 && !SortStep(a.pass, *a.varying).active) return;
    const uint32_t walker = threadIdx.x / kScanBins, bin = threadIdx.x % kScanBins;
    const uint32_t per = (a.n_tiles + kWalkers - 1) / kWalkers;
    const uint32_t t0 = walker * per < a.n_tiles ? walker * per : a.n_tiles, t1 = t0 + per < a.n_tiles ? t0 + per : a.n_tiles;
    uint32_t* column = a.tile_counts + blockIdx.x * kScanBins + bin;
    uint32_t sum = 0;
#pragma unroll 8
    for (uint32_t t = t0; t < t1; ++t) sum += column[static_cast<size_t>(t) * kBins];
    s_sum[walker][bin] = sum;
    __syncthreads();
    {
        const uint32_t b = static_cast<uint32_t>(wave_id()), w = static_cast<uint32_t>(lane_id());      // one wave per bin
        const uint32_t v = s_sum[w][b], inc = dpp_inclusive_scan(v);
        s_sum[w][b] = inc - v;
        if (w == kWalkers - 1) a.totals[blockIdx.x * kScanBins + b] = inc;
    }
    __syncthreads();
    uint32_t run = s_sum[walker][bin];
#pragma unroll 8
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t v = column[static_cast<size_t>(t) * kBins];
        column[static_cast<size_t>(t) * kBins] = run;
        run += v;
    }
}

__global__ __launch_bounds__(kSortBlock) void sort_scatter_kernel(SortArgs a) {
    // the ranks' counters (one per wave and bin) and, once the ranks are known, the tile in order share their memory
    __shared__ union {
        uint16_t count[kSortWaves][kBins];
        struct { int32_t key[kSortTile], val[kSortTile]; } out;
    } s;
    __shared__ uint32_t s_start[kBins];          // where a bin begins in the tile in order
    __shared__ uint32_t s_to[kBins];             // ... and in the output, minus that
    __shared__ uint32_t s_wave[kSortWaves];
    const SortStep step(a.pass, *a.varying);
    if (!step.active) return;
    const int32_t* keys_in = step.before == 0 ? a.counts : a.keys[(step.before - 1) & 1];
    const int32_t* vals_in = step.before == 0 ? nullptr : step.to_order ? a.vals1 : a.order;
    int32_t* keys_out = step.last ? nullptr : a.keys[step.before & 1];
    int32_t* vals_out = step.to_order ? a.order : a.vals1;
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave_id())), lane = static_cast<uint32_t>(lane_id());
    constexpr int kPer = kBins / kSortBlock;     // bins per thread: consecutive ones
    // exclusive sums over the bins of the whole list
    const auto scan_bins = [&](const uint32_t (&v)[kPer], uint32_t (&before)[kPer]) {
        uint32_t mine = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) mine += v[q];
        const uint32_t inc = dpp_inclusive_scan(mine);
        if (lane == kWave - 1) s_wave[wave] = inc;
        __syncthreads();
        const uint32_t w = lane < kSortWaves ? s_wave[lane] : 0u;
        const uint32_t upto = dpp_inclusive_scan(w);
        uint32_t at = lane_value(upto, wave) - lane_value(w, wave) + inc - mine;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            before[q] = at;
            at += v[q];
        }
        __syncthreads();
    };
    uint32_t total[kPer], base[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) total[q] = a.totals[threadIdx.x * kPer + q];
    scan_bins(total, base);
    for (uint32_t tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
        uint32_t earlier[kPer];                  // pairs of the bin in the tiles before
#pragma unroll
        for (int q = 0; q < kPer; ++q) earlier[q] = a.tile_counts[static_cast<size_t>(tile) * kBins + threadIdx.x * kPer + q];
        // a wave owns 512 consecutive pairs, 64 per round
        const uint32_t i0 = tile * kSortTile + wave * (kSortItems * kWave) + lane;
        int32_t key[kSortItems], val[kSortItems];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const uint32_t i = i0 + k * kWave < a.n ? i0 + k * kWave : a.n - 1;
            key[k] = keys_in[i];
            val[k] = vals_in ? vals_in[i] : static_cast<int32_t>(i);
        }
        for (uint32_t q = threadIdx.x; q < kSortWaves * kBins / 2; q += kSortBlock) reinterpret_cast<uint32_t*>(s.count)[q] = 0;
        __syncthreads();
        uint32_t rank[kSortItems];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const uint32_t bin = bin_of(key[k], a.pass);
            uint64_t peers = __ballot(i0 + k * kWave < a.n);
#pragma unroll
            for (int b = 0; b < kDigitBits; ++b) {
                const uint64_t ones = __ballot((bin >> b) & 1u);
                peers &= (bin >> b) & 1u ? ones : ~ones;
            }
            const uint32_t among = rank_in_mask(peers);
            const uint32_t seen = s.count[wave][bin];
            rank[k] = seen + among;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (among == 0 && i0 + k * kWave < a.n) s.count[wave][bin] = static_cast<uint16_t>(seen + __popcll(peers));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        uint32_t in_tile[kPer], start[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t bin = threadIdx.x * kPer + q;
            uint32_t sum = 0;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t c = s.count[w][bin];
                s.count[w][bin] = static_cast<uint16_t>(sum);
                sum += c;
            }
            in_tile[q] = sum;
        }
        scan_bins(in_tile, start);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t bin = threadIdx.x * kPer + q;
            s_start[bin] = start[q];
            s_to[bin] = base[q] + earlier[q] - start[q];
        }
        __syncthreads();
        uint32_t place[kSortItems];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const uint32_t bin = bin_of(key[k], a.pass);
            place[k] = s_start[bin] + s.count[wave][bin] + rank[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            if (i0 + k * kWave < a.n && place[k] < kSortTile) {
                s.out.key[place[k]] = key[k];
                s.out.val[place[k]] = val[k];
            }
        }
        __syncthreads();
        const uint32_t here = a.n - tile * kSortTile < kSortTile ? a.n - tile * kSortTile : kSortTile;
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const uint32_t p = threadIdx.x + k * kSortBlock;
            if (p >= here) continue;
            const int32_t kk = s.out.key[p], vv = s.out.val[p];
            const uint32_t to = s_to[bin_of(kk, a.pass)] + p;
            if (to < a.n) {                              // always, unless the counts changed between the kernels
                vals_out[to] = vv;
                if (keys_out) keys_out[to] = kk;
            } else {
                raise(a.err, kErrInternal);
            }
        }
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
    size_t tiles, totals, varying, bits, counts, keys1, keys2, vals1, bytes;
    explicit SortLayout(int64_t n) {
        const auto up = [](size_t b) { return (b + 255) / 256 * 256; };
        tiles = static_cast<size_t>((n + kSortTile - 1) / kSortTile);
        if (tiles < 1) tiles = 1;
        const size_t ints = up(sizeof(int32_t) * static_cast<size_t>(n));
        totals = 0;
        varying = totals + up(sizeof(uint32_t) * kBins);
        bits = varying + 256;
        counts = bits + up(sizeof(uint32_t) * 2 * tiles);
        keys1 = counts + up(sizeof(uint32_t) * kBins * tiles);
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
    a.tile_counts = reinterpret_cast<uint32_t*>(p + at.counts);
    a.totals = reinterpret_cast<uint32_t*>(p + at.totals);
    a.tile_bits = reinterpret_cast<uint32_t*>(p + at.bits);
    a.varying = reinterpret_cast<uint32_t*>(p + at.varying);
    a.err = err;
    // With one pass or three the first one already writes to `order`.  If that is (part of) the counters' own memory, the pass
    // reads a copy, in the buffer that no pass writes before the second has begun.
    const uintptr_t c0 = reinterpret_cast<uintptr_t>(counts), o0 = reinterpret_cast<uintptr_t>(order), len = sizeof(int32_t) * a.n;
    if (c0 < o0 + len && o0 < c0 + len) {
        const hipError_t e = hipMemcpyAsync(a.keys[1], counts, len, hipMemcpyDefault, stream);
        if (e != hipSuccess) return e;
        a.counts = a.keys[1];
    }
    const dim3 tiles(a.n_tiles < kSortMaxWorkgroups ? a.n_tiles : kSortMaxWorkgroups), block(kSortBlock);
    for (int pass = 0; pass < kSortPasses; ++pass) {
        a.pass = pass;
        hipLaunchKernelGGL(sort_count_kernel, tiles, block, 0, stream, a);
        hipLaunchKernelGGL(sort_scan_kernel, dim3(kBins / kScanBins + (pass == 0 ? 1 : 0)), block, 0, stream, a);
        hipLaunchKernelGGL(sort_scatter_kernel, tiles, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace helios
