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
// (dedup_insert_long_kernel).
#include "kernels.hpp"

namespace helios {

namespace {

__global__ __launch_bounds__(kBlock) void dedup_insert_kernel(const int32_t* __restrict__ ids, Count n_in, int64_t n_nodes,
                                                              DedupScratch s, int32_t* err) {
    // The first ID is fetched before the device-side count has arrived (the buffer holds n_in.host
    // entries, so the read is in bounds whatever the count turns out to be).
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    int32_t early = 0;
    if (j0 < n_in.host) early = ids[j0];
    const int64_t n = n_in.get();
    const uint32_t mask = s.n_slots - 1;
    uint32_t claims = 0;
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

// The same for a long list: few workgroups go through it in steps, and each remembers the slots of recent IDs in LDS, one per
// cell; an ID that an earlier step of the workgroup has inserted needs no insertion of its own (the steps go through the list
// in order, so that occurrence lies before).  Bound by the atomics: 25 random ones per ns, and about 10 ns each for those that
// meet on one address, as the repeats of a hub do.  Measured, 1.1 M IDs: of a power law 67.6 us with one step for every ID, 54.6
// with 512 workgroups, 57.7 with 1024, 62.4 with 2048; uniform over 50 M nodes the whole call 103.6 -> 105.4 us; 300 k IDs 50.7
// -> 45.7 us.  At 140 k IDs (31.9 against 30.4 us) it does not pay any more.
constexpr int kRecent = 2048;
constexpr int64_t kInsertLong = 262144;
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

__global__ __launch_bounds__(kScanBlock) void dedup_compact_kernel(CompactArgs a) {
    compact_role<kCompactPlain>(a, blockIdx.x, gridDim.x);
}

// The end of a stand-alone de-duplication: the inverse map, and beside it the emptying of what the call has used.
struct EndArgs {
    InverseArgs inv;
    ClearJob clear;
    unsigned long long* zero;
    uint32_t n_zero;
    Role r_inv, r_clear;
};
__global__ __launch_bounds__(kBlock) void dedup_end_kernel(EndArgs a) {
    if (a.r_inv.mine()) {
        inverse_role(a.inv, a.r_inv.rb(), a.r_inv.blocks);
        return;
    }
    const uint32_t step = a.r_clear.blocks * kBlock, first = a.r_clear.rb() * kBlock + threadIdx.x;
    for (uint32_t w = first; a.clear.table && w < a.clear.n_slots; w += step) a.clear.table[w] = kEmptySlot;
    for (uint32_t w = first; w < a.n_zero; w += step) a.zero[w] = 0ull;
}

unsigned grid_for(int64_t n_max, unsigned cap_blocks) {
    int64_t b = (n_max + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > cap_blocks) b = cap_blocks;
    return static_cast<unsigned>(b);
}

}  // namespace

hipError_t launch_dedup_insert(hipStream_t stream, const int32_t* ids, Count n, int64_t n_max, int64_t n_nodes,
                               const DedupScratch& s, int32_t* err) {
    if (n_max > kInsertLong)
        hipLaunchKernelGGL(dedup_insert_long_kernel, dim3(kInsertLongWorkgroups), dim3(kBlock), 0, stream, ids, n, n_nodes, s, err);
    else hipLaunchKernelGGL(dedup_insert_kernel, dim3(grid_for(n_max, 4096)), dim3(kBlock), 0, stream, ids, n, n_nodes, s, err);
    return hipGetLastError();
}

hipError_t launch_dedup_compact_plain(hipStream_t stream, const CompactArgs& a, int64_t n_max) {
    hipLaunchKernelGGL(dedup_compact_kernel, dim3(scan_workgroups(n_max, kScanMaxWorkgroups)), dim3(kScanBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_dedup_end(hipStream_t stream, const InverseArgs& inv, int64_t n_max, const ClearJob& clear, unsigned long long* zero,
                            uint32_t n_zero) {
    EndArgs a{inv, clear, zero, n_zero, Role{0, 0}, Role{0, 0}};
    a.r_inv.blocks = inv.inverse ? grid_for(n_max, 2048) : 0u;
    a.r_clear.first = a.r_inv.blocks;
    // eight slots per thread up to a grid that fills the chip
    a.r_clear.blocks = clear.table || n_zero ? grid_for((static_cast<int64_t>(clear.n_slots) + 7) / 8, 1024) : 0u;
    const unsigned blocks = a.r_inv.blocks + a.r_clear.blocks;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(dedup_end_kernel, dim3(blocks), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
}

}  // namespace helios
