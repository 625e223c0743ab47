// Host-side launchers of the Helios kernels.
// Every launcher enqueues on `stream` and returns the hipError_t of the launch.
#pragma once
#include "common.hpp"
#include "compact_dev.hpp"
#include "gather_dev.hpp"
#include "hashtable.hpp"
#include "sample_dev.hpp"
#include "scan.hpp"

namespace helios {

struct CsrView {
    const int64_t* offsets;
    const int32_t* indices;
    int64_t n_nodes;
};

// ---- sample.hip
// Count pass of hop 0 as a kernel of its own, for seed lists too long for the folded count of the
// sampling pass: indptr[i] = start of frontier[i]'s samples in flat, indptr[n] = total (also to
// *n_flat_dev); size_out (nullable, device-accessible) gets {n, total}.  frontier_out (nullable, may
// equal frontier) receives a copy of the frontier; feed.ring (nullable): a recorded batch, whose
// variables this kernel takes from the host's ring (the frontier is their seeds).
hipError_t launch_frontier_count(hipStream_t stream, const CsrView& g, const int32_t* frontier, const BatchFeed& feed,
                                 int32_t* frontier_out, Count n, int64_t n_max, int32_t fanout, int64_t* indptr,
                                 int64_t flat_cap, int64_t* n_flat_dev, int64_t* size_out, const ScanState& scan, int32_t* err);

// Count and sampling of hop 0 in one launch: sample_counted_blocks workgroups of `waves` waves (0: the list is too long, or the fan-out too
// large); stride: the scan's status words.  a as for a folded hop; scan.vars is not used.
unsigned sample_counted_blocks(int32_t fanout, int64_t n, uint32_t stride, unsigned* waves);
hipError_t launch_sample_counted(hipStream_t stream, const HopArgs& a, const ScanState& scan);

// ---- pipeline.hip: the launches of the sampling / whole-path pipeline; each carries one or more roles
// Every launch takes the jobs of n mini-batches (1 <= n <= kMaxGang), one per member of a gang; the
// members' roles share the launch.
constexpr int kMaxGang = 4;
// Sampling pass of one hop (see sample_dev.hpp), and beside it, if link_blocks > 0, a row copy from a
// source behind the host link (the cached rows that the stage before has just listed).  The fan-outs
// of all members select the same group width.
struct SampleJob {
    HopArgs hop;
    unsigned hop_blocks;
    GatherArgs link;
    unsigned link_blocks;
};
hipError_t launch_sample(hipStream_t stream, const SampleJob* jobs, int n);
// Compaction pass(es) after a hop: the hop's samples into the next frontier (hop_blocks > 0) and the
// stage of the batch's ID list that the hop has completed, with its cache lookup (look_blocks > 0).
struct CompactJob {
    CompactArgs hop;
    unsigned hop_blocks;
    CompactArgs look;
    unsigned look_blocks;
};
hipError_t launch_compact(hipStream_t stream, const CompactJob* jobs, int n);
// The end of a batch in one launch: host-tier copy of the last stage, the rows of the miss list from the
// storage stand-in (if the batch serves its own misses), HBM-tier copy of all stages, the inverse map,
// and the emptying of the table that the next batch of the context uses, any of which may be absent (0 workgroups); and the
// check of the batch's own list.  The table to empty is the one after the batch's own among bt's; clear_slots of its slots are in use (with
// vars, a recorded batch, the variables say how many).  The rows of all members have one size.
struct FinishJob {
    GatherArgs hbm;
    unsigned hbm_blocks;
    GatherArgs link;
    unsigned link_blocks;
    GatherArgs miss;
    unsigned miss_blocks;
    InverseArgs inv;
    unsigned inv_blocks;
    uint32_t clear_slots;
    unsigned clear_blocks;
    const uint32_t* claims;      // for the check of the batch's own list (check_table_list)
    uint32_t n_claims;
    const int64_t* n_firsts;
    int32_t* err;
    BatchTables bt;
    const BatchVars* vars;
};
hipError_t launch_finish(hipStream_t stream, const FinishJob* jobs, int n);
// what the kernels receive: the members' arguments and workgroup ranges side by side
struct SampleMember {
    HopArgs hop;
    GatherArgs link;
    Role r_hop, r_link;
};
struct SampleGang {
    SampleMember m[kMaxGang];
    int n;
};
struct CompactMember {
    CompactArgs hop, look;
    Role r_hop, r_look;
};
struct CompactGang {
    CompactMember m[kMaxGang];
    int n;
};
struct FinishMember {
    GatherArgs hbm, link, miss;
    InverseArgs inv;
    BatchTables bt;
    const BatchVars* vars;
    const uint32_t* claims;
    const int64_t* n_firsts;
    int32_t* err;
    uint32_t clear_slots, n_claims;
    Role r_hbm, r_link, r_miss, r_inv, r_clear;
};
struct FinishGang {
    FinishMember m[kMaxGang];
    int n;
};
static_assert(sizeof(SampleGang) <= 4096 && sizeof(CompactGang) <= 4096 && sizeof(FinishGang) <= 4096,
              "kernel arguments are limited to 4 KB");
hipError_t launch_clear(hipStream_t stream, const ClearJob& job);
// reduces the stamps of n_roles roles (role q: workgroups[q] workgroups, stamps at clock + offset[q]) to
// {earliest start, latest end} pairs in pinned host memory
constexpr int kMaxStampRoles = 48;
struct StampTable {
    uint32_t offset[kMaxStampRoles];
    uint32_t workgroups[kMaxStampRoles];
};
hipError_t launch_clock_publish(hipStream_t stream, const uint64_t* clock, const StampTable& table, int n_roles,
                                uint64_t* host_out);

// ---- dedup.hip (the stand-alone de-duplication)
constexpr int64_t kPartsMax = 2097152;
// Slots of the table for a list of n IDs, if there are `most`: eight for each, so that a wave, which waits for the longest of its 64
// searches, rarely looks at more than two (each a round trip to memory).  Two or more slots / eight, us: 8 192 IDs 15.7/13.1, 16 384
// drawn evenly 23.4/14.4, 41 237 17.9/17.4 (19.7/16.2).  Emptying them costs less: 4 MB 0.7 us.  Lists that are too long to be taken apart
// (below) are bound by the memory's atomics and by the emptying instead, so two for each are enough: 2.2 M IDs drawn evenly 229 us with eight,
// 188 with two, 3 M 291 and 254.
inline uint32_t list_slots(int64_t n, uint32_t most) {
    const int64_t want = n <= kPartsMax ? 8 * n : 2 * n;
    uint32_t slots = 1024;
    while (slots < most && static_cast<int64_t>(slots) < want) slots <<= 1;
    return slots;
}
// First pass as a kernel of its own (for IDs that no kernel of this library produced): inserts ids[0, n)
// into s.table, which must be empty.  Beside it zero[0, n_zero) (nullable) is set to zero.
hipError_t launch_dedup_insert(hipStream_t stream, const int32_t* ids, Count n, int64_t n_max, int64_t n_nodes,
                               const DedupScratch& s, unsigned long long* zero, uint32_t n_zero, int32_t* err);
// Second pass over the whole list.
hipError_t launch_dedup_compact_plain(hipStream_t stream, const CompactArgs& a, int64_t n_max);
// Both passes for a list of up to kPartsMax IDs (see dedup.hip), and whether that is the quicker way.  a.len is n, known on the host.  The table may hold anything and
// is not used but by lists that hash unevenly; what they use of it is left empty.
// Measured, us for the call with a table of eight slots an ID / by parts, IDs by a power law (drawn evenly; one ID throughout):
//   4 k 12.9/17 (12.5/17)   8 k 12.9/15.7 (13/15.6; 145/15.3)   16 k 13.5/15.7 (14/16.5)   25 k 14.7/15.8 (14.8/16)   32 k 16.0/16.1 (16.6/16.2; 510/16)
//   41 k 17.2/16.3 (16.1/16.7)   50 k 18.3/16.6 (17.5/16.7)   65 k 20.5/17 (19.7/17; 1050/15); with two slots an ID 98 k 24.5/18.2   262 k 41/23
//   1.1 M 102/38   2 M 165/57.  Above 2 M a bucket would have more IDs than half its table.
// Of few distinct IDs without a hub the table is the quicker way a little longer: 3 000 distinct ones, 32 k 15.4/16.9, 50 k 17.0/17.7, 65 k 18.9/18.
// All IDs of one bucket of the hash: see dedup.hip.
// With two to four slots an ID the table takes 20 k 16.3 (17.6), 25 k 16.3 (18.5), 32 k 19.5 (25.5), so there the line lies lower.
inline bool dedup_by_parts(int64_t n, uint32_t slots) { return n >= (slots >= 4 * n ? 32768 : 20000) && n <= kPartsMax; }
// The list is cut into tiles, one to a workgroup: 256 of them, so that every CU has one, but of 1024 entries or more; and 512 if 256
// would have more than 6144 each.
constexpr uint32_t kMinPartTile = 1024, kMaxPartTile = 6144, kLineWords = 32;
struct PartShape {
    uint32_t n, tile, n_tiles;   // entries, entries of a tile (a multiple of 64), tiles
    uint32_t per_tile;           // 2^32 / tile, rounded up
    uint32_t row;                // words from one tile's flags to the next one's (dedup_compact_parts_kernel): whole lines of 128 bytes
    uint32_t split_slots, bucket_slots;      // of the tables in LDS: 8192, or twice the entries of a tile and four times those of a bucket
    explicit PartShape(int64_t ids) : n(static_cast<uint32_t>(ids)) {
        const uint32_t most = ids <= 256 * kMaxPartTile ? 256 : 512;
        tile = (n + most * 64 - 1) / (most * 64) * 64;
        if (tile < kMinPartTile) tile = kMinPartTile;
        n_tiles = (n + tile - 1) / tile;
        per_tile = 0xffffffffu / tile + 1;
        row = (tile / 16 + kLineWords - 1) / kLineWords * kLineWords;      // (no more words in all than the list has entries)
        for (split_slots = 1024; split_slots < 8192 && split_slots < 2 * tile;) split_slots *= 2;
        for (bucket_slots = 1024; bucket_slots < 8192 && bucket_slots < n / 128;) bucket_slots *= 2;
    }
};
constexpr int64_t kMaxPartTiles = 512;
struct PartScratch {             // all of n entries, but starts: split_starts_bytes(PartShape(n).n_tiles)
    int32_t* id;                 // the distinct IDs of every tile in order of bucket
    uint16_t* pos;               // their places in the tile
    uint32_t* first;             // the first positions of those IDs in the list
    uint16_t* local;             // for every input, the place in its tile where its ID is first, or 0xffff
    uint16_t* starts;            // [tile][513]: where a bucket begins in the tile
    unsigned long long* clear;   // n_clear words that the first launch sets to zero (nullable)
    uint32_t n_clear;
};
constexpr int64_t split_starts_bytes(int64_t n_tiles) { return n_tiles * 513 * 2; }
hipError_t launch_dedup_by_parts(hipStream_t stream, const CompactArgs& a, int64_t n, int64_t n_nodes, const PartScratch& s);
// The optional third pass (inv.inverse nullable), and in the same launch the emptying of a table, which that pass does not read.
hipError_t launch_dedup_end(hipStream_t stream, const InverseArgs& inv, int64_t n_max, const ClearJob& clear);

// ---- cache.hip
// rank[order[r]] = r; *holes (device) = 1 if that leaves a node without a rank, else 0.  scratch (nullable): device memory
// that may be used, 8 1/16 bytes per node.  cursors: kMapCursors device words, zero before and after.
constexpr uint32_t kMapCursors = 1024;
hipError_t launch_rank_build(hipStream_t stream, const int32_t* order, int64_t n_nodes, int32_t* rank, int64_t* holes, uint32_t* cursors,
                             void* scratch, size_t scratch_bytes, int32_t* err);

// Lookup of ids[0, n) and partition into the per-tier lists and the miss list.  With copy_table, the rows of the HBM tier are copied
// in the same launch (out[j] = copy_table[rank[ids[j]]], rows of `chunks` 16-byte pieces), and that tier gets no list; its count
// is written all the same.  copy_beside_lookup says whether that is the quicker way.
bool copy_beside_lookup(int64_t n, int64_t n_nodes, int64_t n_hbm, int32_t chunks);
hipError_t launch_lookup_partition(hipStream_t stream, const int32_t* ids, int64_t n,
                                   const int32_t* rank, int64_t n_nodes, int64_t n_hbm, int64_t n_host,
                                   const TierLists& lists, int32_t* miss_pos, int32_t* miss_id,
                                   int32_t* miss_slot, int64_t miss_cap, int64_t* stats_out, int64_t* learn,
                                   const ScanState& scan, const int64_t* holes, int32_t* err, const chunk16* copy_table, chunk16* copy_out,
                                   int32_t chunks);

// ---- gather.hip
// The row copy as a kernel of its own.  far_source selects the launch shape for a source behind the host
// link (few workgroups, one per CU).  With t_start / t_stop (nullable) the launch carries HIP events that
// take the kernel's own begin and end, as a kernel trace reports them.  expected: the probable length of the
// list (0 = unknown; see copy_role_blocks).  *blocks_out = workgroups launched.
hipError_t launch_gather_rows(hipStream_t stream, const GatherArgs& a, int64_t n_max, bool far_source, bool standin,
                              unsigned blocks_limit /* 0 = default */, int64_t expected, hipEvent_t t_start, hipEvent_t t_stop,
                              unsigned* blocks_out);

// ---- blocks.hip
// For every list: out[j] = index in a de-duplication's unique list of ids[j] (s = the scratch that de-duplication used,
// untouched since); an ID that is not in the list raises kErrData.  n_max[k] bounds list k.
struct LocalIdsList {
    const int32_t* ids;
    Count n;
    int32_t* out;
};
constexpr int kMaxLocalIdsLists = 16;        // frontier and samples of up to eight hops
hipError_t launch_local_ids(hipStream_t stream, const LocalIdsList* lists, const int64_t* n_max, int n_lists, const DedupScratch& s,
                            int32_t* err);

// ---- hotness.hip
hipError_t launch_hotness_add(hipStream_t stream, const int32_t* ids, Count n, int64_t n_max, int64_t n_nodes,
                              int32_t* counts, int32_t* err);
size_t hotness_order_scratch_bytes(int64_t n_nodes);
// order = nodes by counts descending, ties by ascending ID; scratch: hotness_order_scratch_bytes(n_nodes) of device memory
hipError_t launch_hotness_order(hipStream_t stream, const int32_t* counts, int64_t n_nodes, int32_t* order, void* scratch,
                                int32_t* err);

// dst[0, bytes) = src[0, bytes) with the same 16-byte non-temporal accesses as the row copy
hipError_t launch_calibration_copy(hipStream_t stream, const void* src, void* dst, int64_t bytes);

}  // namespace helios
