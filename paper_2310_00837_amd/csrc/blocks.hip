// Batch generation: node IDs -> their index in the batch's unique list.
//
// The hash table of the batch's de-duplication still maps every ID of the batch
// to the input position of its first occurrence, and index_of_first maps that
// position to the index in `unique`; so relabelling an ID is one probe of a
// table that sits in L2, with no second table to build.
#include "kernels.hpp"

namespace helios {

namespace {

struct LocalIdsArgs {
    LocalIdsList list[kMaxLocalIdsLists];
    int n_lists;
    DedupScratch s;
    int32_t* err;
};

// All lists of a batch (every hop's frontier and samples) in one launch: they are cut into pieces of kBlock IDs, and the
// workgroups take the pieces in turn.  Bound by the chain of a piece (length, ID, table word, index), so one launch of a
// three-hop batch takes little longer than the longest list did alone: 6.8 us in place of six launches of 4.0 to 6.0 us (blocks of a three-hop batch of 777 seeds),
// each with 4 us of the host's time.
__global__ __launch_bounds__(kBlock) void local_ids_kernel(LocalIdsArgs a) {
    uint32_t n[kMaxLocalIdsLists];
#pragma unroll
    for (int k = 0; k < kMaxLocalIdsLists; ++k) n[k] = k < a.n_lists ? static_cast<uint32_t>(a.list[k].n.get()) : 0u;
    uint32_t pieces = 0;
#pragma unroll
    for (int k = 0; k < kMaxLocalIdsLists; ++k) pieces += (n[k] + kBlock - 1) / kBlock;
    const uint32_t mask = a.s.n_slots - 1;
    for (uint32_t piece = blockIdx.x; piece < pieces; piece += gridDim.x) {
        uint32_t in_list = piece, list = 0, len = 0;
        bool found = false;
#pragma unroll
        for (int k = 0; k < kMaxLocalIdsLists; ++k) {
            const uint32_t mine = (n[k] + kBlock - 1) / kBlock;
            if (!found && in_list < mine) {
                found = true;
                list = k;
                len = n[k];
            }
            if (!found) in_list -= mine;
        }
        const uint32_t j = in_list * kBlock + threadIdx.x;
        if (j >= len) continue;
        const int32_t id = a.list[list].ids[j];
        int32_t local = -1;
        if (id >= 0) {
            uint32_t slot = hash_id(static_cast<uint32_t>(id), mask);
            for (uint32_t probes = 0; probes <= mask; ++probes) {          // the table is never full
                const unsigned long long cur = a.s.table[slot];
                if (cur == kEmptySlot) break;                              // not in the batch
                if (static_cast<uint32_t>(cur >> 32) == static_cast<uint32_t>(id)) {
                    local = a.s.index_of_first[static_cast<uint32_t>(cur)];
                    break;
                }
                slot = (slot + 1) & mask;
            }
        }
        if (local < 0) raise(a.err, kErrData);
        a.list[list].out[j] = local;
    }
}

}  // namespace

hipError_t launch_local_ids(hipStream_t stream, const LocalIdsList* lists, const int64_t* n_max, int n_lists, const DedupScratch& s,
                            int32_t* err) {
    if (n_lists < 1 || n_lists > kMaxLocalIdsLists) return hipErrorInvalidValue;
    LocalIdsArgs a{};
    int64_t pieces = 0;
    for (int k = 0; k < n_lists; ++k) {
        a.list[k] = lists[k];
        pieces += (n_max[k] + kBlock - 1) / kBlock;
    }
    a.n_lists = n_lists;
    a.s = s;
    a.err = err;
    pieces = pieces < 1 ? 1 : pieces > 2048 ? 2048 : pieces;
    hipLaunchKernelGGL(local_ids_kernel, dim3(static_cast<unsigned>(pieces)), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
}

}  // namespace helios
