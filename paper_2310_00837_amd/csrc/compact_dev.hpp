// Device code of the second pass of the order-preserving de-duplication (see dedup.hip for the
// whole scheme): the inputs have been inserted into a hash table that keeps, per distinct ID, the
// smallest input position holding it, and the slot of every input is remembered.  Input j is a
// first occurrence iff its slot's position is j.  The flags are counted by wave ballots, summed in the
// workgroup and chained across workgroups (TileScan in scan.hpp), so `unique` comes out in
// input order.  The pass has the new unique IDs in registers, so two things that need them ride on
// it instead of being kernels of their own:
//   kCompactNextHop  the unique list is the frontier of the next hop: read every new frontier node's
//                    row bounds and scan the sample counts min(deg, fanout) as a second counter,
//                    which gives that hop its indptr;
//   kCompactLookup   the unique list is (a stage of) the batch's ID list: read rank[id], classify into
//                    HBM tier, host tier or miss, and scan the two hit classes as further counters
//                    (the miss rank is what is left), which gives the stable per-tier lists and the
//                    miss list that cache.hip's stand-alone lookup kernel would produce from `unique`.
//
// Stages.  The list may be compacted piece by piece: a stage handles the inputs [begin, begin + n)
// and continues the numbering where the stage before it stopped (its totals are read from device
// memory; this stage leaves its own for the next).  Because `unique` is in order of first occurrence,
// the unique IDs of a prefix of the list are a prefix of the final unique list, so a stage's part of
// `unique`, of the tier lists and of the miss list is final as soon as the inputs of that stage are
// in the table: the whole-path call compacts [seeds | flat_0] right after hop 0, flat_1 after hop 1,
// and so on, and the row copies of a stage run while the next hop is being sampled.
#pragma once
#include "common.hpp"
#include "hashtable.hpp"
#include "scan.hpp"

namespace helios {

enum CompactMode { kCompactPlain = 0, kCompactNextHop = 1, kCompactLookup = 2 };

struct DedupScratch {
    unsigned long long* table;   // n_slots entries {id:32, first position:32}; all ones = empty
    uint32_t n_slots;            // power of two
    int32_t* slot_of;            // [n] table slot of every input position
    int32_t* index_of_first;     // [n] index in `unique` of a first occurrence (nullable: not wanted)
};

// The rotating tables of the batch de-duplication: batch b of a context uses table b mod kBatchTables,
// so that the table of a finished batch stays readable (helios_make_blocks) while the next batch
// runs, and a table is emptied, off the critical path, by the batch before the one that uses it.
constexpr uint32_t kBatchTables = 3;
struct BatchTables {
    unsigned long long* table0;  // nullable: no batch de-duplication; table t starts at table0 + t * table_stride
    uint64_t table_stride;       // in slots
    int32_t* iof0;               // index_of_first of table t starts at iof0 + t * iof_stride
    uint64_t iof_stride;
    int32_t* slot0;              // slot of every position in the batch's ID list, for table t at slot0 + t * iof_stride
    int64_t* list_n;             // device [kBatchTables]: length of the ID list that the table's last batch inserted, or kListIncomplete
    uint32_t n_slots;            // slots in use (power of two)
    uint32_t which;              // the batch's table, unless BatchVars say otherwise
    __device__ __forceinline__ uint32_t pick(const BatchVars* vars) const { return vars ? vars->table % kBatchTables : which; }
    __device__ __forceinline__ unsigned long long* table(uint32_t t) const { return table0 + t * table_stride; }
    __device__ __forceinline__ int32_t* iof(uint32_t t) const { return iof0 + t * iof_stride; }
    __device__ __forceinline__ int32_t* slot_of(uint32_t t) const { return slot0 + t * iof_stride; }
};

// Empties the table of the context's next batch, of which `slots` slots are in use: the batch before the last used it,
// and the slot of every ID that it inserted stands at the ID's place in the list, if the batch's own last launch has found
// so (check_table_list).  The table is sized for the worst case of a
// batch, which is several times what batches bring, so emptying the slots of the list is far less memory traffic than
// emptying the table: 0.25 MB of list against 8 MB per batch with fan-outs 25 and 10.  A scattered 8-byte store takes
// about 14 ps of the whole chip's time and a streamed one 1.6, so a list longer than an eighth of the table streams.
__device__ __forceinline__ void empty_next_table(const BatchTables& b, const BatchVars* vars, uint32_t slots, uint32_t rb, uint32_t nrb) {
    const uint32_t t = (b.pick(vars) + 1) % kBatchTables;
    if (vars) slots = vars->clear_slots;
    const uint64_t n = static_cast<uint64_t>(b.list_n[t]);
    unsigned long long* table = b.table(t);
    const uint32_t step = nrb * kBlock;
    if (n > b.iof_stride || n * 8 > slots) {                   // (kListIncomplete is more than any list)
        for (uint32_t w = rb * kBlock + threadIdx.x; w < slots; w += step) table[w] = ~0ull;
        return;
    }
    const int32_t* slot_of = b.slot_of(t);
    for (uint32_t j = rb * kBlock + threadIdx.x; j < n; j += step) {
        const uint32_t slot = static_cast<uint32_t>(slot_of[j]);
        if (slot < slots) table[slot] = ~0ull;                 // (-1: the entry was no node)
    }
}

// Whether the list of a batch names every word of its table, by one workgroup once the batch is compacted.  A word counts as a
// first occurrence at the one place that is its position, and only if the list holds the word's slot there; so if the
// first occurrences (n_firsts) are as many as the words that the sampling passes have added (the sum of claims), every
// word is named.  It is not so if what the batch reads has changed while it ran (a caller that refills the seeds too
// early, buffers that overlap): two samples may then have met at one place, of which the list holds one.  The batch is
// reported, and its table will be emptied in full whatever is queued behind it.
constexpr int64_t kListIncomplete = INT64_MAX;
__device__ __forceinline__ void check_table_list(const BatchTables& b, const BatchVars* vars, const uint32_t* claims, uint32_t n_claims,
                                                 const int64_t* n_firsts, int32_t* err) {
    // one wave without LDS, which every workgroup of the launch would be given (0.3 us); eight reads in flight, unguarded (a
    // place past the end reads the first)
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    static_assert(kWavesPerBlock == 4, "a workgroup's words are read at once");
    if (threadIdx.x >= kWave) return;
    const words4* per_block = reinterpret_cast<const words4*>(claims);
    const uint32_t n_blocks = n_claims / kWavesPerBlock;
    const uint64_t firsts = static_cast<uint64_t>(*n_firsts);
    uint32_t sum = 0;
    for (uint32_t w0 = threadIdx.x; w0 < n_blocks + threadIdx.x; w0 += 8 * kWave) {
        words4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = per_block[w0 + k * kWave < n_blocks ? w0 + k * kWave : 0];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (w0 + k * kWave < n_blocks) sum += v[k].x + v[k].y + v[k].z + v[k].w;
    }
    if (dpp_sum(sum) == firsts || threadIdx.x != 0) return;
    b.list_n[b.pick(vars)] = kListIncomplete;
    raise(err, kErrData);
}

// What the de-duplication between two hops also computes for the hop that follows: the sample
// counts min(deg, fanout) of the new frontier, scanned into indptr (indptr[n_unique] = total, also
// to *n_flat_dev); size_out (nullable, device-accessible) gets {n_unique, total}.
struct NextHopCount {
    const int64_t* offsets;
    int64_t n_nodes;
    int32_t fanout;
    int64_t* indptr;
    int64_t flat_cap;
    int64_t* n_flat_dev;
    int64_t* size_out;
};
struct TierLists {
    int32_t* pos[2];    // positions in the ID list, per cached tier (0 = HBM, 1 = host)
    int32_t* slot[2];   // row in the tier table
    int64_t* count;     // device int64[3]: entries to copy from tier 0 and tier 1, misses to serve
};
// What the batch's de-duplication also computes: the cache lookup of the unique IDs (see
// launch_lookup_partition, whose outputs these are, with positions = indices into `unique`).
struct LookupOut {
    const int32_t* rank;
    int64_t n_hbm, n_host;
    TierLists lists;
    int32_t *miss_pos, *miss_id, *miss_slot;
    int64_t miss_cap;
    int64_t* stats_out;          // device-accessible int64[4], nullable; written by the last stage
    int64_t* learn;              // pinned int64[4], nullable: the library's own copy of the stats, from which the host
                                 // sizes the grids of the batches that follow
};
// Totals a stage leaves behind in device memory (int64[kStageWords]).
constexpr int kStageUnique = 0, kStageHbm = 1, kStageHost = 2;      // unique IDs, HBM hits, host hits so far
constexpr int kStageHbmCopy = 3, kStageHostCopy = 4;                // list entries that may be copied (none of a stage
                                                                    // whose part of `unique` did not fit its capacity)
constexpr int kStageEnd = 5;                                        // inputs compacted so far: where the next stage begins
constexpr int kStageWords = 8;

struct CompactArgs {
    const int32_t* ids;
    uint32_t n_nodes;            // IDs from here on are never used as an index
    Count len;                   // inputs of this stage: len + fixed
    uint32_t fixed;
    uint32_t n_max;              // bound on them
    int64_t* n_total_dev;        // receives begin + n: the inputs compacted so far (nullable)
    DedupScratch s;              // table / index_of_first are overridden by `batch` when that is set
    BatchTables batch;
    const BatchVars* vars;
    int32_t* unique;
    int64_t unique_cap;
    int32_t* inverse;            // nullable; see InverseArgs
    const int64_t* prev;         // totals of the stage before (nullable: this is the first)
    int64_t* mine;               // totals after this stage (nullable)
    bool last;                   // the last stage writes the outputs below
    int64_t* n_unique_dev;
    int64_t* n_unique_out;       // device-accessible, nullable
    union {                      // a pass is either the batch's (look) or the one between two hops (next), or neither
        LookupOut look;
        NextHopCount next;
    };
    uint32_t* batches_run;       // nullable: the first compaction of a recorded batch counts the batch
    ScanState scan;
    int32_t* err;
    Stamps stamps;
};

// K items per thread (see scan.hpp).  What bounds a stage: nothing but the chain itself -- counts of the stages before,
// ticket, slot and ID, table word and rank / row bounds, tile scan, look-back, stores.  Every load of a step is issued for
// all items before the first is used, and unconditionally (an item that is not there reads entry 0), because a guarded load
// makes the compiler wait for it at the end of its branch.
// How the compaction marks a repeat in `inverse` until the inverse pass has looked its index up: -2 - the place of the ID's
// first occurrence (-1 is an entry that is no node).
__device__ __forceinline__ int32_t repeat_of(uint32_t first) { return -2 - static_cast<int32_t>(first); }

template <int MODE, int K>
__device__ __forceinline__ void compact_tiles(const CompactArgs& a, const DedupScratch& s, const ScanState& scan, const int64_t (&prev)[kStageWords],
                                              uint32_t begin, uint32_t n, uint32_t rb, uint32_t nrb) {
    constexpr int NP = MODE == kCompactPlain ? 1 : 2;
    constexpr int NC = MODE == kCompactNextHop ? 2 : MODE == kCompactLookup ? 3 : 1;
    using Scan = TileScan<NP, NC, K>;
    __shared__ typename Scan::Lds lds;
    const uint32_t end = begin + n;
    const int64_t base[3] = {prev[kStageUnique], prev[kStageHbm], prev[kStageHost]};
    const uint32_t n_tiles = (n + K * kScanBlock - 1) / (K * kScanBlock);
    if (rb >= n_tiles) return;
    const uint32_t n_wgs = nrb < n_tiles ? nrb : n_tiles;
    for (uint32_t tile = Scan::take_ticket(scan, n_tiles, n_wgs, lds); tile < n_tiles;
         tile = n_wgs < n_tiles ? Scan::take_ticket(scan, n_tiles, n_wgs, lds) : n_tiles) {
        const uint32_t j0 = begin + tile * (K * kScanBlock) + threadIdx.x;
        int32_t slot[K], id[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t j = j0 + k * kScanBlock;
            const uint32_t at = j < end ? j : begin;
            slot[k] = s.slot_of[at];
            id[k] = a.ids[at];
        }
        // The table word and the row bounds / the rank are fetched together: those of a repeated ID are
        // read for nothing, but they are in cache and nobody waits for the flag first.  (A slot >= 0
        // means the insert pass found the ID to be a node ID.)
        unsigned long long word[K];
        int64_t lo[K], hi[K];
        int32_t r[K];
        bool live[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            // (both checked: an input that changes while the batch runs leaves places of the list unwritten, and what they
            // hold then must not become an address)
            const bool real = j0 + k * kScanBlock < end && static_cast<uint32_t>(id[k]) < a.n_nodes;
            live[k] = real && static_cast<uint32_t>(slot[k]) < s.n_slots;
            if (real && !live[k]) raise(a.err, kErrInternal);      // kNoSlot: its table was full
            const uint32_t at = live[k] ? static_cast<uint32_t>(slot[k]) : 0u, node = live[k] ? static_cast<uint32_t>(id[k]) : 0u;
            word[k] = s.table[at];
            if (MODE == kCompactNextHop) { lo[k] = a.next.offsets[node]; hi[k] = a.next.offsets[node + 1]; }
            if (MODE == kCompactLookup) r[k] = a.look.rank[node];
        }
        uint32_t totals[NP][K], before[NP][K], local[K], local2[K], cnt[K];
        bool first[K];
        int tier[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            first[k] = live[k] && static_cast<uint32_t>(word[k]) == j0 + k * kScanBlock;
            const uint64_t firsts = __ballot(first[k]);
            totals[0][k] = static_cast<uint32_t>(__popcll(firsts));
            local[k] = rank_in_mask(firsts);
            if (MODE == kCompactNextHop) {
                const int64_t d = hi[k] - lo[k];
                const bool bad = d < 0 || d > 0x7fffffffLL;
                if (live[k] && bad) raise(a.err, kErrData);
                const int64_t f = a.next.fanout > 0 ? a.next.fanout : 0;
                cnt[k] = !first[k] || bad ? 0u : static_cast<uint32_t>(d < f ? d : f);
                const uint32_t inc = dpp_inclusive_scan(cnt[k]);
                totals[NP - 1][k] = lane_value(inc, kWave - 1);
                local2[k] = inc - cnt[k];
            }
            if (MODE == kCompactLookup) {
                // a negative rank (the hotness order was no permutation; reported when the map was built, and
                // here) counts as a miss whose slot no table has
                if (first[k] && r[k] < 0) raise(a.err, kErrData);
                const uint32_t ur = static_cast<uint32_t>(r[k]);
                tier[k] = ur < static_cast<uint32_t>(a.look.n_hbm) ? 0 : ur < static_cast<uint32_t>(a.look.n_hbm + a.look.n_host) ? 1 : 2;
                const uint64_t hbm = __ballot(first[k] && tier[k] == 0), host = __ballot(first[k] && tier[k] == 1);
                totals[NP - 1][k] = static_cast<uint32_t>(__popcll(hbm)) | (static_cast<uint32_t>(__popcll(host)) << 16);
                local2[k] = rank_in_mask(hbm) | (rank_in_mask(host) << 16);
            }
        }
        Scan::run(scan, tile, totals, before, lds, a.err);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t j = j0 + k * kScanBlock;
            if (a.inverse && j < end && !first[k]) {
                // a repeat leaves the place of its first occurrence, whose index another tile may still be working out
                const uint32_t of = static_cast<uint32_t>(word[k]);
                a.inverse[j] = live[k] && of < j ? repeat_of(of) : -1;
            }
            if (!first[k]) continue;
            const int64_t at = base[0] + lds.excl[0] + before[0][k] + local[k];
            if (s.index_of_first) s.index_of_first[j] = static_cast<int32_t>(at);
            if (a.inverse) a.inverse[j] = static_cast<int32_t>(at);
            if (MODE == kCompactNextHop) {
                const int64_t at_cnt = static_cast<int64_t>(lds.excl[NC - 1]) + before[NP - 1][k] + local2[k];
                if (at <= a.unique_cap) a.next.indptr[at] = at_cnt;
                // the frontier is cut off here: the next hop samples the nodes that fit, and its sample list
                // ends where this node's samples would have begun
                if (at == a.unique_cap) *a.next.n_flat_dev = at_cnt;
            }
            if (at >= a.unique_cap) continue;
            a.unique[at] = id[k];
            if (MODE == kCompactLookup) {
                const uint32_t in_tile = before[NP - 1][k] + local2[k];          // no carry between the halves: a tile has at most 2048 items
                const int64_t at_hbm = base[1] + lds.excl[NC - 2] + (in_tile & 0xffffu);
                const int64_t at_host = base[2] + lds.excl[NC - 1] + (in_tile >> 16);
                if (tier[k] < 2) {
                    const int64_t w = tier[k] == 0 ? at_hbm : at_host;
                    (tier[k] == 0 ? a.look.lists.pos[0] : a.look.lists.pos[1])[w] = static_cast<int32_t>(at);
                    (tier[k] == 0 ? a.look.lists.slot[0] : a.look.lists.slot[1])[w] =
                        r[k] - (tier[k] == 0 ? 0 : static_cast<int32_t>(a.look.n_hbm));
                } else {
                    const int64_t w = at - at_hbm - at_host;                     // every unique ID is in exactly one class
                    if (w < a.look.miss_cap) {
                        a.look.miss_pos[w] = static_cast<int32_t>(at);
                        a.look.miss_id[w] = id[k];
                        a.look.miss_slot[w] = r[k] < 0 ? -1 : r[k] - static_cast<int32_t>(a.look.n_hbm + a.look.n_host);
                    }
                }
            }
        }
        if (tile == n_tiles - 1 && threadIdx.x == 0) {
            const int64_t total = base[0] + lds.excl[0] + lds.agg[0];
            const bool fits = total <= a.unique_cap;
            if (a.last) {
                *a.n_unique_dev = total;
                if (a.n_unique_out) *a.n_unique_out = total;
            }
            if (!fits) raise(a.err, kErrCapacity);
            if (a.mine) a.mine[kStageUnique] = total;
            if (MODE == kCompactNextHop) {
                const int64_t total_cnt = static_cast<int64_t>(lds.excl[NC - 1]) + lds.agg[NC - 1];
                if (fits) {                          // else the thread at the cut has written both
                    a.next.indptr[total] = total_cnt;
                    *a.next.n_flat_dev = total_cnt;
                }
                if (a.next.size_out) { a.next.size_out[0] = total; a.next.size_out[1] = total_cnt; }
                if (total_cnt > a.next.flat_cap) raise(a.err, kErrCapacity);
            }
            if (MODE == kCompactLookup) {
                const int64_t c0 = base[1] + lds.excl[NC - 2] + lds.agg[NC - 2];
                const int64_t c1 = base[2] + lds.excl[NC - 1] + lds.agg[NC - 1];
                const int64_t c2 = total - c0 - c1;
                // if `unique` overflowed, list entries past its capacity were not written: this stage's are not copied
                const int64_t copy0 = fits ? c0 : prev[kStageHbmCopy];
                const int64_t copy1 = fits ? c1 : prev[kStageHostCopy];
                if (a.mine) {
                    a.mine[kStageHbm] = c0; a.mine[kStageHost] = c1;
                    a.mine[kStageHbmCopy] = copy0; a.mine[kStageHostCopy] = copy1;
                }
                if (a.last) {
                    a.look.lists.count[0] = copy0; a.look.lists.count[1] = copy1; a.look.lists.count[2] = fits ? c2 : 0;
                    if (a.look.stats_out) { a.look.stats_out[0] = total; a.look.stats_out[1] = c0; a.look.stats_out[2] = c1; a.look.stats_out[3] = c2; }
                    if (a.look.learn) { a.look.learn[0] = total; a.look.learn[1] = c0; a.look.learn[2] = c1; a.look.learn[3] = c2; }
                    if (c2 > a.look.miss_cap) raise(a.err, kErrCapacity);
                }
            }
        }
    }
}

template <int MODE>
__device__ __forceinline__ void compact_role(const CompactArgs& a, uint32_t rb, uint32_t nrb) {
    stamp_start(a.stamps, rb);
    const ScanState scan = scan_resolve(a.scan);
    const uint32_t which = a.batch.pick(a.vars);
    const uint32_t n_raw = a.fixed + static_cast<uint32_t>(a.len.get());
    int64_t prev[kStageWords] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (a.prev) {
#pragma unroll
        for (int q = 0; q < kStageWords; ++q) prev[q] = a.prev[q];
    }
    if (a.batches_run && rb == 0 && threadIdx.x == 0) *a.batches_run += 1;   // every workgroup of the batch's first kernel has read its slot
    DedupScratch s = a.s;
    if (a.batch.table0) s = DedupScratch{a.batch.table(which), a.batch.n_slots, a.batch.slot_of(which), a.batch.iof(which)};
    const uint32_t n = n_raw < a.n_max ? n_raw : a.n_max;
    const uint32_t begin = static_cast<uint32_t>(prev[kStageEnd]), end = begin + n;
    const int64_t base[3] = {prev[kStageUnique], prev[kStageHbm], prev[kStageHost]};
    if (rb == 0 && threadIdx.x == 0) {
        if (a.n_total_dev) *a.n_total_dev = end;
        if (a.mine) a.mine[kStageEnd] = end;
        if (a.batch.table0) a.batch.list_n[which] = end;
        if (n == 0) {                              // an empty stage: the totals pass through
            if (a.mine) {
                a.mine[kStageUnique] = base[0]; a.mine[kStageHbm] = base[1]; a.mine[kStageHost] = base[2];
                a.mine[kStageHbmCopy] = prev[kStageHbmCopy];
                a.mine[kStageHostCopy] = prev[kStageHostCopy];
            }
            if (a.last) {
                *a.n_unique_dev = base[0];
                if (a.n_unique_out) *a.n_unique_out = base[0];
            }
            if (MODE == kCompactNextHop) {
                a.next.indptr[0] = 0;
                *a.next.n_flat_dev = 0;
                if (a.next.size_out) { a.next.size_out[0] = 0; a.next.size_out[1] = 0; }
            }
            if (MODE == kCompactLookup && a.last) {
                const int64_t c2 = base[0] - base[1] - base[2];
                const bool fits = base[0] <= a.unique_cap;
                a.look.lists.count[0] = prev[kStageHbmCopy];
                a.look.lists.count[1] = prev[kStageHostCopy];
                a.look.lists.count[2] = fits ? c2 : 0;
                if (a.look.stats_out) { a.look.stats_out[0] = base[0]; a.look.stats_out[1] = base[1]; a.look.stats_out[2] = base[2]; a.look.stats_out[3] = c2; }
            }
        }
    }
    if (static_cast<uint64_t>(rb) * kScanBlock < n) {
        if (n <= kScanOneItemMax) compact_tiles<MODE, 1>(a, s, scan, prev, begin, n, rb, nrb);
        else if (n <= 2 * kScanOneItemMax) compact_tiles<MODE, 2>(a, s, scan, prev, begin, n, rb, nrb);
        else compact_tiles<MODE, kScanMaxItems>(a, s, scan, prev, begin, n, rb, nrb);
    }
    stamp_end(a.stamps, rb, nrb);
}

struct InverseArgs {
    Count n;                     // inputs of the list (a device count written by the compaction)
    const int32_t* iof;          // index in unique of a first occurrence; overridden by `batch` when that is set
    BatchTables batch;
    const BatchVars* vars;
    int32_t* inverse;
    bool by_table;               // batch only: the compaction has not been given `inverse`, so there are no marks
    Stamps stamps;
};

// Third pass (optional): inverse[j] = index in unique of input j.  The compaction has written it for every first occurrence,
// which most inputs are, and marked the repeats, so the pass streams over the list and looks up only those; it needs
// neither the slots nor the table (which may be emptied beside it).  1.1 M IDs, a third of them distinct: 11.3 us with the emptying of a 33 MB table beside it, 17.6 + 10.0 us when
// every input looked its slot, its table word and its index up (by_table: the way for an inverse in the memory of a buffer that
// the batch still needs after its compactions have begun).
__device__ __forceinline__ void inverse_role(const InverseArgs& a, uint32_t rb, uint32_t nrb) {
    stamp_start(a.stamps, rb);
    const uint32_t which = a.batch.pick(a.vars);
    const int32_t* iof = a.batch.table0 ? a.batch.iof(which) : a.iof;
    const uint32_t n = static_cast<uint32_t>(a.n.get());
    if (a.by_table) {
        const unsigned long long* table = a.batch.table(which);
        const int32_t* slot_of = a.batch.slot_of(which);
        for (uint32_t j = rb * kBlock + threadIdx.x; j < n; j += nrb * kBlock) {
            const uint32_t slot = static_cast<uint32_t>(slot_of[j]);
            const uint32_t of = slot < a.batch.n_slots ? static_cast<uint32_t>(table[slot]) : ~0u;
            a.inverse[j] = of < n ? iof[of] : -1;
        }
    }
    for (uint32_t j = rb * kBlock + threadIdx.x; j < n && !a.by_table; j += nrb * kBlock) {
        const int32_t mark = a.inverse[j];
        const uint32_t of = static_cast<uint32_t>(-2 - mark);
        if (mark < -1 && of < n) a.inverse[j] = iof[of];       // (the marks stand in a buffer of the caller's: never an address unchecked)
    }
    stamp_end(a.stamps, rb, nrb);
}

}  // namespace helios
