// Order-preserving de-duplication of an ID list.
//
// unique = the distinct IDs in order of first occurrence.  The order is made
// independent of thread scheduling by keeping, per distinct ID, the smallest
// input position that holds it:
//   1. insert: an open-addressing hash table of 64-bit words {id:32 | pos:32}
//      (hashtable.hpp).  The slot of every input is remembered.  For IDs that
//      the sampling kernel produces, that kernel does the inserting as it writes
//      them (sample_dev.hpp); the insert kernel here serves helios_dedup.
//   2. compact (compact_dev.hpp): input j is a first occurrence iff its slot's
//      position is j; the flags are scanned in-workgroup and chained across
//      workgroups, so the unique list comes out in input order in the same pass.
//   3. inverse (optional): the compaction writes it for first occurrences and
//      marks a repeat with the place of its first occurrence; a last pass over
//      the list turns the marks into unique indices.  It reads neither slots nor
//      table, so its launch empties the table for the next call as well.
// The table has at least twice as many slots as inputs and is empty before the
// first insert; at the sizes of one mini-batch (at most 32 MB) it stays in L2 /
// MALL.  The inserts of the sampling kernel are not staged through LDS.
// Measured on the power-law workloads (dedup_probe.py): 15-21 % of a batch's
// list entries repeat an earlier entry, but only 0.5-4.4 % repeat one within
// the same 4096 entries (0.1-1.2 % within 1024), because the hubs that repeat
// are spread over the whole list.  A per-workgroup LDS table would take that
// little off the global table, while every entry paid an LDS probe and a
// barrier more.  A long stand-alone list is another matter: there a workgroup
// goes through many steps of the list and remembers what it has met
// (dedup_insert_long_kernel), or the list is taken apart by hash first
// (dedup_split_kernel).
#include "kernels.hpp"

namespace helios {

namespace {

__global__ __launch_bounds__(kBlock) void dedup_insert_kernel(const int32_t* __restrict__ ids, Count n_in, int64_t n_nodes,
                                                              DedupScratch s, unsigned long long* zero, uint32_t n_zero, int32_t* err) {
    // The first ID is fetched before the device-side count has arrived (the buffer holds n_in.host
    // entries, so the read is in bounds whatever the count turns out to be).
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    int32_t early = 0;
    if (j0 < n_in.host) early = ids[j0];
    const int64_t n = n_in.get();
    const uint32_t mask = s.n_slots - 1;
    uint32_t claims = 0;
    for (uint32_t w = static_cast<uint32_t>(j0); w < n_zero; w += gridDim.x * kBlock) zero[w] = 0ull;
    for (int64_t j = j0; j < n; j += static_cast<int64_t>(gridDim.x) * kBlock) {
        const int32_t id = j == j0 ? early : ids[j];
        if (id < 0 || static_cast<int64_t>(id) >= n_nodes) {
            raise(err, kErrData);
            s.slot_of[j] = -1;
            continue;
        }
        s.slot_of[j] = static_cast<int32_t>(table_insert(s.table, mask, static_cast<uint32_t>(id), static_cast<uint32_t>(j), claims));
    }
}

// The same for a list that is too long to be taken apart (below): few workgroups go through it in steps, and each remembers the slots
// of recent IDs in LDS, one per cell; an ID that an earlier step of the workgroup has inserted needs no insertion of its own (the
// steps go through the list in order, so that occurrence lies before).  Bound by the atomics: 25 random ones per ns, and about 10 ns
// each for those that meet on one address, as the repeats of a hub do.  Measured, 1.1 M IDs of a power law: 67.6 us with one step for
// every ID, 54.6 with 512 workgroups, 57.7 with 1024, 62.4 with 2048.
constexpr int kRecent = 2048;
constexpr unsigned kInsertLongWorkgroups = 512;
__global__ __launch_bounds__(kBlock) void dedup_insert_long_kernel(const int32_t* __restrict__ ids, Count n_in, int64_t n_nodes, DedupScratch s,
                                                                   int32_t* err) {
    __shared__ unsigned long long recent[kRecent];        // {id : 32 | slot : 32}
    for (int w = threadIdx.x; w < kRecent; w += kBlock) recent[w] = kEmptySlot;
    const uint32_t n = static_cast<uint32_t>(n_in.get()), mask = s.n_slots - 1, step = gridDim.x * kBlock;
    uint32_t claims = 0;
    __syncthreads();
    for (uint32_t j0 = blockIdx.x * kBlock; j0 < n; j0 += step) {
        const uint32_t j = j0 + threadIdx.x;
        const int32_t id = j < n ? ids[j] : -1;
        const bool node = id >= 0 && static_cast<int64_t>(id) < n_nodes;
        const uint32_t home = hash_id(static_cast<uint32_t>(id), 0xffffffffu);
        // (a cell is read and written whole: two IDs that meet in one must not leave the slot of the other behind)
        unsigned long long* cell = recent + (home >> 16) % kRecent;
        const unsigned long long seen = __hip_atomic_load(cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        if (j < n) {
            int32_t slot = -1;
            if (!node) {
                raise(err, kErrData);
            } else if (static_cast<uint32_t>(seen >> 32) == static_cast<uint32_t>(id)) {
                slot = static_cast<int32_t>(static_cast<uint32_t>(seen));
            } else {
                slot = static_cast<int32_t>(table_insert(s.table, mask, static_cast<uint32_t>(id), j, claims));
                const unsigned long long met = (static_cast<unsigned long long>(static_cast<uint32_t>(id)) << 32) | static_cast<uint32_t>(slot);
                __hip_atomic_store(cell, met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            s.slot_of[j] = slot;
        }
        __syncthreads();
    }
}

// ---- a long list by parts, without the table
//
// The inserts of a long list are bound by the atomics of the memory (25 a ns) and its compaction by as many random reads.  So a
// list is taken apart by hash instead, until a part fits a table in LDS:
//   split     a tile (see PartShape) drops its repeats (LDS table), and the rest is put into order of 512 buckets and written out so,
//             with where the buckets begin;
//   buckets   a workgroup per bucket gathers its pieces of all tiles, finds the first position of every ID in an LDS table, and
//             leaves it where it has read the ID;
//   compact   a tile's first positions go back into input order (LDS), and from there on it is a compaction that also writes the
//             inverse map.
// All of it is streams, the buckets' reads in pieces of about 32 bytes (IDs, first positions) and 16 (places), shorter where the list is
// short or the tiles have dropped repeats.  They drop them so that no bucket is much longer than the others: of an ID that fills the list
// a bucket gets one entry per tile.
// What bounds it is a workgroup's chain of steps, LDS searches above all, so the tiles are as small as 256 workgroups allow: 1.1 M IDs
// 253 tiles of 4352 38.1 us (split 13.5, buckets 12, compact 12), 269 of 4096, so that 13 CUs have two, 41.0, 506 of 2176 43.8;
// 98 k 96 tiles of 1024 18.2, 24 of 4096 22.2.  Each number of rounds has an instance of its own: with guards in one for
// all 1.1 M took 40.2, with six rounds always 38.7.  256 buckets of 1024 threads with eight entries each, 64-bit words and
// a second search for the answers: buckets 44 us at 1.1 M; linear probing and 512 threads in the split: 15.
// When it pays against the table: dedup_by_parts.
constexpr int kPartTile = kMaxPartTile;
constexpr int kPartBits = 9;
constexpr int kParts = 1 << kPartBits;
constexpr int kSplitBlock = 1024;
constexpr int kMergeBlock = 1024;                      // compaction
constexpr int kMergeWaves = kMergeBlock / kWave;
constexpr int kBucketBlock = 1024;
constexpr int kBucketItems = 4;                        // entries per thread that stay in registers
constexpr uint32_t kPartSlots = 8192;                  // of an LDS table: keys, and the lowest position that holds the key
constexpr uint32_t kPartProbes = 128;                  // more than that at one ID: a bucket's table counts as full
constexpr uint16_t kNoPlace = 0xffff;
constexpr uint32_t kForeign = 2;                       // (of s_full) a stretch of the table full of another call's words: no search goes on
static_assert((kPartSlots & (kPartSlots - 1)) == 0 && kPartProbes <= kPartSlots, "odd steps come by every slot once");
static_assert(kPartsMax == kMaxPartTiles * 4096 && kMaxPartTiles <= kBucketBlock && kMaxPartTiles <= kMergeBlock, "a thread per tile");
static_assert(kParts <= kSplitBlock && kPartTile / kMergeBlock * kMergeWaves <= 2 * kWave, "a thread per bucket; two steps scan a tile");
static_assert(kSplitBlock == kMergeBlock && kPartTile == 6 * kMergeBlock && kPartTile < kPartSlots, "one to six rounds of all threads; the split's table never fills");

struct alignas(16) PartTable {                         // (part_clear stores 16 bytes at a time)
    uint32_t key[kPartSlots], low[kPartSlots];         // ~0: empty (IDs are below 2^31)
};
__device__ __forceinline__ void part_clear(PartTable& t, uint32_t from, uint32_t slots, uint32_t threads) {
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    words4 *keys = reinterpret_cast<words4*>(t.key), *lows = reinterpret_cast<words4*>(t.low);
    for (uint32_t q = from / 4 + threadIdx.x; q < slots / 4; q += threads) keys[q] = lows[q] = words4{~0u, ~0u, ~0u, ~0u};
}
// the whole hash: the highest bits are the bucket, the next the place in the table, the lowest the step
__device__ __forceinline__ uint32_t part_hash(uint32_t id) { return hash_id(id, 0xffffffffu); }
// The split's table is at most three quarters full (6144 IDs), a bucket's about half in the longest lists, and a wave waits for the longest of its 64
// searches: steps of the ID's own, odd ones, which come by every slot, keep those short.
__device__ __forceinline__ uint32_t part_step(uint32_t h) { return (h << 1) | 1u; }
// The ID's slot, claimed if need be; kNoSlot after probes_max others.  (A plain read before the atomic: the entries of a hub would
// take their turns at its word.)
__device__ __forceinline__ uint32_t part_slot(PartTable& t, uint32_t slots, uint32_t id, uint32_t h, uint32_t probes_max) {
    uint32_t slot = (h >> 10) & (slots - 1);
    for (uint32_t probes = 0; probes < probes_max; ++probes) {
        uint32_t cur = __hip_atomic_load(t.key + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == ~0u) cur = atomicCAS(t.key + slot, ~0u, id);
        if (cur == ~0u || cur == id) return slot;
        slot = (slot + part_step(h)) & (slots - 1);
    }
    return kNoSlot;
}
__device__ __forceinline__ uint32_t part_low(const PartTable& t, uint32_t slot) {
    return __hip_atomic_load(t.low + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ITEMS: rounds of all threads that go through a tile
template <int ITEMS>
__global__ __launch_bounds__(kSplitBlock) void dedup_split_kernel(const int32_t* __restrict__ ids, PartShape shape, int64_t n_nodes,
                                                                  PartScratch s, int32_t* err) {
    __shared__ union {
        PartTable table;
        struct { int32_t id[ITEMS * kSplitBlock]; uint16_t pos[ITEMS * kSplitBlock]; } out;
    } m;
    __shared__ uint32_t s_count[kParts], s_wave[kParts / kWave];
    const uint32_t tile = blockIdx.x, base = tile * shape.tile, entries = min(shape.n - base, shape.tile);
    int32_t id[ITEMS];
    uint32_t slot[ITEMS], rank[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) id[k] = ids[base + min(k * kSplitBlock + threadIdx.x, entries - 1)];
    if (s.clear && tile == 0)
        for (uint32_t w = threadIdx.x; w < s.n_clear; w += kSplitBlock) s.clear[w] = 0ull;
    part_clear(m.table, 0, shape.split_slots, kSplitBlock);
    if (threadIdx.x < kParts) s_count[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t p = k * kSplitBlock + threadIdx.x;
        const bool here = p < entries, node = id[k] >= 0 && static_cast<int64_t>(id[k]) < n_nodes;
        if (here && !node) raise(err, kErrData);
        slot[k] = kNoSlot;
        if (!here || !node) continue;
        const uint32_t at = part_slot(m.table, shape.split_slots, static_cast<uint32_t>(id[k]), part_hash(static_cast<uint32_t>(id[k])), shape.split_slots);
        slot[k] = at;                                  // (there is one: the tile has fewer IDs than the table slots)
        if (part_low(m.table, at) > p) atomicMin(m.table.low + at, p);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t p = k * kSplitBlock + threadIdx.x;
        const uint32_t low = slot[k] != kNoSlot ? part_low(m.table, slot[k]) : kNoPlace;
        if (p < entries) s.local[base + p] = static_cast<uint16_t>(low);
        slot[k] = low == p ? part_hash(static_cast<uint32_t>(id[k])) >> (32 - kPartBits) : kNoSlot;      // from here on the bucket
        rank[k] = low == p ? atomicAdd(s_count + slot[k], 1u) : 0u;
    }
    __syncthreads();
    const uint32_t mine = threadIdx.x < kParts ? s_count[threadIdx.x] : 0u, inc = dpp_inclusive_scan(mine);
    if (threadIdx.x < kParts && lane_id() == kWave - 1) s_wave[wave_id()] = inc;
    __syncthreads();
    uint32_t at = inc - mine, there = 0;
#pragma unroll
    for (int w = 0; w < kParts / kWave; ++w) {
        at += w < wave_id() ? s_wave[w] : 0u;
        there += s_wave[w];
    }
    if (threadIdx.x < kParts) {
        s_count[threadIdx.x] = at;
        uint16_t* starts = s.starts + static_cast<size_t>(tile) * (kParts + 1);
        starts[threadIdx.x] = static_cast<uint16_t>(at);
        if (threadIdx.x == kParts - 1) starts[kParts] = static_cast<uint16_t>(there);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        if (slot[k] == kNoSlot) continue;
        const uint32_t to = s_count[slot[k]] + rank[k];
        m.out.id[to] = id[k];
        m.out.pos[to] = static_cast<uint16_t>(k * kSplitBlock + threadIdx.x);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t p = k * kSplitBlock + threadIdx.x;
        if (p >= there) continue;
        s.id[base + p] = m.out.id[p];
        s.pos[base + p] = m.out.pos[p];
    }
}

// A bucket whose distinct IDs don't fit the table in LDS goes by a stretch of the call's table in memory, which no other bucket
// uses: two slots for each of its entries, behind two for each entry of the buckets before it.  The stretch is emptied first, and
// left empty.  Only lists made against the hash get there (of IDs in strides, in blocks and in a row a bucket gets at most 1.25
// times its share of lists this long): 1 M IDs of one bucket, 78 k of them distinct, take 3.4 ms, all of it one workgroup's, where the
// inserts into a table for all take 0.1; with one LDS table after the other, class by class of the hash, it was 606.  32 k of one bucket
// take 410 us, 98 k 768, 32 k of four buckets 178, 98 k of 14 buckets 47 (by the table altogether 21, 23, 21 and 26).
__device__ __forceinline__ uint32_t stretch_slot(uint32_t id, uint32_t size) { return __umulhi(part_hash(~id), size); }

__global__ __launch_bounds__(kBucketBlock) void dedup_bucket_kernel(PartScratch s, PartShape shape, unsigned long long* table_in_memory,
                                                                    uint32_t n_slots, int32_t* err) {
    __shared__ PartTable table;
    __shared__ uint32_t s_before[kMaxPartTiles], s_from[kMaxPartTiles];     // of a tile's piece: entries before it, where it begins
    __shared__ uint32_t s_wave[kMaxPartTiles / kWave];
    __shared__ uint32_t s_full, s_lower;                                    // s_lower: entries of the buckets before this one
    const uint32_t t = threadIdx.x, n_tiles = shape.n_tiles;
    uint32_t len = 0, from = 0;
    if (t < n_tiles) {
        // (Calls that overlap on the static array of helios_dedup_noalloc may each have written one of the two words.  What lies
        // within a tile is taken, so every place below is one of the tile's own.)
        const uint16_t* starts = s.starts + static_cast<size_t>(t) * (kParts + 1) + blockIdx.x;
        const uint32_t begin = starts[0], end = starts[1];
        const bool piece = begin <= end && end <= min(shape.n - t * shape.tile, shape.tile);
        if (!piece) raise(err, kErrInternal);
        from = piece ? begin : 0u;
        len = piece ? end - begin : 0u;
    }
    const uint32_t inc = dpp_inclusive_scan(len);
    if (t < kMaxPartTiles && lane_id() == kWave - 1) s_wave[wave_id()] = inc;
    if (t == 0) s_full = s_lower = 0;
    part_clear(table, 0, shape.bucket_slots, kBucketBlock);
    __syncthreads();
    uint32_t at = inc - len, total = 0;
#pragma unroll
    for (int w = 0; w < static_cast<int>(kMaxPartTiles) / kWave; ++w) {
        at += w < wave_id() ? s_wave[w] : 0u;
        total += s_wave[w];
    }
    if (t < kMaxPartTiles) {
        s_before[t] = t < n_tiles ? at : ~0u;
        s_from[t] = t * shape.tile + from;
    }
    // A bucket of more than twice its share gets a larger table than the others (all entries of 131 k IDs in 16 buckets 163 us without, 29.4; in
    // 65 buckets 102 and 20.9).
    uint32_t slots = shape.bucket_slots;
    while (slots < kPartSlots && slots < 2 * total) slots *= 2;
    if (slots > shape.bucket_slots) part_clear(table, shape.bucket_slots, slots, kBucketBlock);
    __syncthreads();
    uint32_t place[kBucketItems], pos[kBucketItems], id[kBucketItems], slot[kBucketItems];
    const uint32_t chunks = (total + kBucketBlock * kBucketItems - 1) / (kBucketBlock * kBucketItems);
    const auto entries = [&](uint32_t chunk) {                              // where they are (~0: there is none), and what
#pragma unroll
        for (int k = 0; k < kBucketItems; ++k) {
            const uint32_t e = (chunk * kBucketItems + k) * kBucketBlock + t;
            uint32_t lo = 0;                                                // the last tile with at most e entries before its piece
#pragma unroll
            for (uint32_t half = kMaxPartTiles / 2; half > 0; half /= 2)
                if (s_before[lo + half] <= e) lo += half;
            place[k] = e < total ? s_from[lo] + (e - s_before[lo]) : ~0u;
            pos[k] = lo * shape.tile;
        }
#pragma unroll
        for (int k = 0; k < kBucketItems; ++k) {
            const uint32_t p = place[k] != ~0u ? place[k] : 0u;
            id[k] = static_cast<uint32_t>(s.id[p]);
            pos[k] += s.pos[p];
        }
    };
    for (uint32_t chunk = 0; chunk < chunks; ++chunk) {
        if (__hip_atomic_load(&s_full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0) break;
        entries(chunk);
#pragma unroll
        for (int k = 0; k < kBucketItems; ++k) {
            if (place[k] == ~0u) continue;
            slot[k] = part_slot(table, slots, id[k], part_hash(id[k]), kPartProbes);
            if (slot[k] == kNoSlot) s_full = 1;
            else if (part_low(table, slot[k]) > pos[k]) atomicMin(table.low + slot[k], pos[k]);
        }
    }
    __syncthreads();
    if (s_full == 0) {
        for (uint32_t chunk = 0; chunk < chunks; ++chunk) {
            if (chunks > 1) {                                               // (one chunk is still in registers)
                entries(chunk);
#pragma unroll
                for (int k = 0; k < kBucketItems; ++k)
                    if (place[k] != ~0u) slot[k] = part_slot(table, slots, id[k], part_hash(id[k]), kPartProbes);
            }
#pragma unroll
            for (int k = 0; k < kBucketItems; ++k)
                if (place[k] != ~0u) s.first[place[k]] = slot[k] != kNoSlot ? part_low(table, slot[k]) : ~0u;
        }
        return;
    }
    if (t < n_tiles) atomicAdd(&s_lower, from);
    __syncthreads();
    const uint32_t size = 2 * total;
    if (2 * s_lower + size > n_slots) {                                     // (only if another call writes to the same memory)
        if (t == 0) raise(err, kErrInternal);
        return;
    }
    unsigned long long* stretch = table_in_memory + 2 * s_lower;
    for (uint32_t w = t; w < size; w += kBucketBlock) scan_store(stretch + w, kEmptySlot);
    __syncthreads();
    for (uint32_t chunk = 0; chunk < chunks; ++chunk) {
        if (__hip_atomic_load(&s_full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == kForeign) break;
        entries(chunk);
#pragma unroll
        for (int k = 0; k < kBucketItems; ++k) {
            if (place[k] == ~0u) continue;
            const unsigned long long mine = (static_cast<unsigned long long>(id[k]) << 32) | pos[k];
            uint32_t q = stretch_slot(id[k], size), left = size;
            for (; left > 0; --left, q = q + 1 < size ? q + 1 : 0) {
                unsigned long long cur = scan_load(stretch + q);            // (a plain read first, as in part_slot)
                if (cur == kEmptySlot) cur = atomicCAS(stretch + q, kEmptySlot, mine);
                if (cur != kEmptySlot && cur >> 32 != id[k]) continue;
                if (mine < cur && cur != kEmptySlot) atomicMin(stretch + q, mine);
                break;
            }
            if (left == 0) {                                                // (as above)
                s_full = kForeign;
                raise(err, kErrInternal);
            }
        }
    }
    __syncthreads();
    for (uint32_t chunk = 0; chunk < chunks; ++chunk) {
        if (__hip_atomic_load(&s_full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == kForeign) break;
        entries(chunk);
#pragma unroll
        for (int k = 0; k < kBucketItems; ++k) {
            if (place[k] == ~0u) continue;
            uint32_t q = stretch_slot(id[k], size), left = size;
            unsigned long long cur = kEmptySlot;
            for (; left > 0; --left, q = q + 1 < size ? q + 1 : 0) {
                cur = scan_load(stretch + q);
                if (cur == kEmptySlot || cur >> 32 == id[k]) break;
            }
            if (left == 0) s_full = kForeign;
            s.first[place[k]] = static_cast<uint32_t>(cur);                 // (it is there, unless another call wrote)
        }
    }
    __syncthreads();
    for (uint32_t w = t; w < size; w += kBucketBlock) scan_store(stretch + w, kEmptySlot);
}

// The compaction of a list that came by parts: like compact_tiles, but the first positions come from the split tile, and it writes the
// whole inverse map.  Which of a tile's entries are first occurrences goes out, 16 to a word with how many of the tile come before them (a
// tile's words begin a line, see PartShape), before the tile's total does.  A workgroup waits for the totals of all tiles before its own and sums them up, which gives it the place of
// its own first occurrences and of everybody's before; a repeat then finds its index as what the tiles before its first occurrence's
// have, what the word says, and the bits below.  With marks in the inverse map and a launch more that
// looks them up, the totals chained from tile to tile and 512 threads: 400 k IDs 30.7 us, now 27.5, 1.1 M 43.2 and 41.0.  (The sum up to a
// repeat's tile read from the chain's words, at memory, by every repeat: 48.9.)
__device__ __forceinline__ uint32_t first_word(uint32_t before, uint32_t mask) { return (before << 16) | (mask & 0xffffu); }

template <int ITEMS>
__global__ __launch_bounds__(kMergeBlock) void dedup_compact_parts_kernel(CompactArgs a, PartScratch s, PartShape shape) {
    __shared__ uint32_t s_first[ITEMS * kMergeBlock], s_total[ITEMS * kMergeWaves], s_upto[kMaxPartTiles], s_wave[kMaxPartTiles / kWave], s_ticket;
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave_id())), lane = static_cast<uint32_t>(lane_id());
    const ScanState scan = scan_resolve(a.scan);
    const uint32_t n = shape.n, n_tiles = shape.n_tiles;
    uint32_t* words = reinterpret_cast<uint32_t*>(a.s.index_of_first);
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.n_total_dev) *a.n_total_dev = n;
    if (threadIdx.x == 0) {
        s_ticket = 0;
        if (n_tiles > 1) {                       // (a workgroup per tile; the last draw puts the counter back)
            const uint32_t t = atomicAdd(scan.ticket, 1u);
            if (t == n_tiles - 1) __hip_atomic_store(scan.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_ticket = t;
        }
    }
    __syncthreads();
    const uint32_t tile = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(s_ticket)));
    if (tile >= n_tiles) {                       // (calls that overlap on the static array of helios_dedup_noalloc draw from one counter)
        if (threadIdx.x == 0) raise(a.err, kErrInternal);
        return;
    }
    const uint32_t base = tile * shape.tile, entries = min(n - base, shape.tile);
    const uint32_t there = min(static_cast<uint32_t>(s.starts[static_cast<size_t>(tile) * (kParts + 1) + kParts]), entries);
    uint32_t first_of[ITEMS], pos[ITEMS], in_tile[ITEMS];
    int32_t id[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t p = k * kMergeBlock + threadIdx.x, at = base + (p < there ? p : 0);
        first_of[k] = s.first[at];
        pos[k] = s.pos[at];
        in_tile[k] = s.local[base + min(p, entries - 1)];
        id[k] = a.ids[base + min(p, entries - 1)];
        asm volatile("" : "+v"(id[k]));          // (read before the tile's total goes out: `unique` may lie over the IDs)
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        if (k * kMergeBlock + threadIdx.x < there) s_first[pos[k] % (ITEMS * kMergeBlock)] = first_of[k];
    __syncthreads();
    uint32_t before[ITEMS], local[ITEMS], total[ITEMS];
    uint64_t firsts[ITEMS];
    bool first[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t p = k * kMergeBlock + threadIdx.x, j = base + p;
        first_of[k] = in_tile[k] != kNoPlace ? s_first[in_tile[k] % (ITEMS * kMergeBlock)] : ~0u;        // (~0: no node)
        first[k] = p < entries && first_of[k] == j;
        firsts[k] = __ballot(first[k]);
        local[k] = rank_in_mask(firsts[k]);
        total[k] = static_cast<uint32_t>(__popcll(firsts[k]));
        if (lane == 0) s_total[k * kMergeWaves + wave] = total[k];
    }
    __syncthreads();
    constexpr uint32_t kRuns = ITEMS * kMergeWaves, kFirstItems = kWave / kMergeWaves;
    const uint32_t inc = dpp_inclusive_scan(lane < kRuns ? s_total[lane] : 0u);
    const uint32_t more = kRuns > kWave ? dpp_inclusive_scan(kWave + lane < kRuns ? s_total[kWave + lane] : 0u) : 0u;
    const uint32_t in_first = lane_value(inc, kWave - 1), in_all = in_first + lane_value(more, kWave - 1);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        before[k] = (k < kFirstItems ? lane_value(inc, k * kMergeWaves + wave) : in_first + lane_value(more, (k - kFirstItems) * kMergeWaves + wave)) - total[k];
        const uint32_t mask = static_cast<uint32_t>(firsts[k] >> (lane % 4 * 16)), p = k * kMergeBlock + wave * kWave + lane * 16;
        const uint32_t below = static_cast<uint32_t>(__popcll(firsts[k] & ((1ull << (lane % 4 * 16)) - 1)));
        if (a.inverse && lane < 4 && p < entries) __hip_atomic_store(words + tile * shape.row + p / 16, first_word(before[k] + below, mask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (they go past the L2: now they are there for all)
    __syncthreads();
    if (threadIdx.x == 0) scan_store(scan.status + tile, scan_pack(scan.epoch, kFlagAggregate, in_all));
    // (512 tiles at most: a lane for each.  The wait is bounded: a wave that gives up says so, and the launch drains.)
    uint32_t mine = 0, sums = 0;
    if (threadIdx.x < kMaxPartTiles) {
        const bool wanted = threadIdx.x < tile;
        unsigned long long w = 0;
        for (uint32_t budget = kScanSpinBudget; budget > 0; --budget) {
            if (wanted) w = scan_load(scan.status + threadIdx.x);
            if (__ballot(wanted && w >> 34 != scan.epoch) == 0) break;
            if (budget == 1) raise(a.err, kErrInternal);
            __builtin_amdgcn_s_sleep(1);
        }
        mine = static_cast<uint32_t>(w);
        sums = dpp_inclusive_scan(mine);
        if (lane == kWave - 1) s_wave[wave] = sums;
    }
    __syncthreads();
    uint32_t excl = 0;
#pragma unroll
    for (uint32_t w = 0; w < kMaxPartTiles / kWave; ++w) {
        if (w < wave) sums += s_wave[w];
        excl += s_wave[w];
    }
    if (threadIdx.x < kMaxPartTiles) s_upto[threadIdx.x] = sums - mine;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint32_t p = k * kMergeBlock + threadIdx.x, j = base + p;
        if (p >= entries) continue;
        const uint32_t at = excl + before[k] + local[k], of = first_of[k];
        if (a.inverse && of < j) {
            uint32_t in = __umulhi(of, shape.per_tile);         // the tile, or one more
            if (in * shape.tile > of) --in;
            // (A tile's words are on lines of their own, and the tile is this one or one whose total has been waited for: the whole line
            // is complete, and the same for the rest of the launch, so it may come from the L2.  A line with words of a later tile could be
            // fetched before they are there, and stay so for whoever waits for that tile.)
            const uint32_t word = __hip_atomic_load(words + in * shape.row + (of - in * shape.tile) / 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            a.inverse[j] = static_cast<int32_t>(s_upto[in] + (word >> 16) + static_cast<uint32_t>(__popc(word & ((1u << (of % 16)) - 1))));
        } else if (a.inverse) {
            a.inverse[j] = first[k] ? static_cast<int32_t>(at) : -1;
        }
        if (first[k] && at < a.unique_cap) a.unique[at] = id[k];
    }
    if (tile == n_tiles - 1 && threadIdx.x == 0) {
        const int64_t sum = static_cast<int64_t>(excl) + in_all;
        *a.n_unique_dev = sum;
        if (a.n_unique_out) *a.n_unique_out = sum;
        if (sum > a.unique_cap) raise(a.err, kErrCapacity);
    }
}

__global__ __launch_bounds__(kScanBlock) void dedup_compact_kernel(CompactArgs a) {
    compact_role<kCompactPlain>(a, blockIdx.x, gridDim.x);
}

// The end of a stand-alone de-duplication: the inverse map, and beside it the emptying of what the call has used.
struct EndArgs {
    InverseArgs inv;
    ClearJob clear;
    Role r_inv, r_clear;
};
__global__ __launch_bounds__(kBlock) void dedup_end_kernel(EndArgs a) {
    if (a.r_inv.mine()) {
        inverse_role(a.inv, a.r_inv.rb(), a.r_inv.blocks);
        return;
    }
    const uint32_t step = a.r_clear.blocks * kBlock, first = a.r_clear.rb() * kBlock + threadIdx.x;
    for (uint32_t w = first; a.clear.table && w < a.clear.n_slots; w += step) a.clear.table[w] = kEmptySlot;
}

unsigned grid_for(int64_t n_max, unsigned cap_blocks) {
    int64_t b = (n_max + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > cap_blocks) b = cap_blocks;
    return static_cast<unsigned>(b);
}

}  // namespace

hipError_t launch_dedup_insert(hipStream_t stream, const int32_t* ids, Count n, int64_t n_max, int64_t n_nodes,
                               const DedupScratch& s, unsigned long long* zero, uint32_t n_zero, int32_t* err) {
    if (n_max > kPartsMax && n_zero > 0) return hipErrorInvalidValue;
    if (n_max > kPartsMax)
        hipLaunchKernelGGL(dedup_insert_long_kernel, dim3(kInsertLongWorkgroups), dim3(kBlock), 0, stream, ids, n, n_nodes, s, err);
    else hipLaunchKernelGGL(dedup_insert_kernel, dim3(grid_for(n_max, 4096)), dim3(kBlock), 0, stream, ids, n, n_nodes, s, zero, n_zero, err);
    return hipGetLastError();
}

hipError_t launch_dedup_by_parts(hipStream_t stream, const CompactArgs& a, int64_t n, int64_t n_nodes, const PartScratch& s) {
    if (n < 1 || n > kPartsMax || !a.s.table || a.s.n_slots < 2 * n) return hipErrorInvalidValue;
    if (reinterpret_cast<uintptr_t>(a.s.index_of_first) % (sizeof(uint32_t) * kLineWords) != 0) return hipErrorInvalidValue;
    const PartShape shape(n);
#define HELIOS_CALL_(ITEMS)                                                                                                          \
    do {                                                                                                                             \
        hipLaunchKernelGGL(dedup_split_kernel<ITEMS>, dim3(shape.n_tiles), dim3(kSplitBlock), 0, stream, a.ids, shape, n_nodes, s, a.err); \
        hipLaunchKernelGGL(dedup_bucket_kernel, dim3(kParts), dim3(kBucketBlock), 0, stream, s, shape, a.s.table, a.s.n_slots, a.err); \
        hipLaunchKernelGGL(dedup_compact_parts_kernel<ITEMS>, dim3(shape.n_tiles), dim3(kMergeBlock), 0, stream, a, s, shape);       \
    } while (0)
    switch ((shape.tile + kMergeBlock - 1) / kMergeBlock) {
        case 1: HELIOS_CALL_(1); break;
        case 2: HELIOS_CALL_(2); break;
        case 3: HELIOS_CALL_(3); break;
        case 4: HELIOS_CALL_(4); break;
        case 5: HELIOS_CALL_(5); break;
        case 6: HELIOS_CALL_(6); break;
        default: return hipErrorInvalidValue;
    }
#undef HELIOS_CALL_
    return hipGetLastError();
}

hipError_t launch_dedup_compact_plain(hipStream_t stream, const CompactArgs& a, int64_t n_max) {
    hipLaunchKernelGGL(dedup_compact_kernel, dim3(scan_workgroups(n_max, kScanMaxWorkgroups)), dim3(kScanBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_dedup_end(hipStream_t stream, const InverseArgs& inv, int64_t n_max, const ClearJob& clear) {
    EndArgs a{inv, clear, Role{0, 0}, Role{0, 0}};
    a.r_inv.blocks = inv.inverse ? grid_for(n_max, 2048) : 0u;
    a.r_clear.first = a.r_inv.blocks;
    // eight slots per thread up to a grid that fills the chip
    a.r_clear.blocks = clear.table ? grid_for((static_cast<int64_t>(clear.n_slots) + 7) / 8, 1024) : 0u;
    const unsigned blocks = a.r_inv.blocks + a.r_clear.blocks;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(dedup_end_kernel, dim3(blocks), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
}

}  // namespace helios
