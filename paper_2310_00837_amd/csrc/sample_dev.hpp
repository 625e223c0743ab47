// Device code of one hop of uniform neighbour sampling without replacement over a CSR graph.
//
// The work per node is two dependent random reads (the row bounds, then up to `fanout` entries of
// the row), so a hop is bound by memory latency, not bandwidth.  It has two parts:
//
//   count   row bounds -> sample count min(deg, fanout) per frontier node, scanned into indptr, each
//           node's place in `flat`.  For hop 0 of a batch of at most kFoldMaxSeeds seeds every
//           workgroup of the sampling pass redoes this scan for the whole seed list (a thousand
//           cached 16-byte reads cost less than a kernel launch) and keeps its own nodes' bounds in
//           LDS; larger seed lists get frontier_count_kernel (sample.hip) first; for the later hops
//           the de-duplication that produces the frontier does it in the same pass (compact_dev.hpp).
//   sample  a group of G lanes owns one node (G = the smallest of 8, 16, 32, 64 that covers the
//           fan-out): lane k computes the k-th Philox draw and Floyd candidate, the group settles
//           collisions lane by lane, and lane k reads the k-th chosen neighbour and writes it to
//           flat[indptr[i] + k].  All reads of a node are issued together; any number of
//           workgroups can run, in any order.
// Fan-outs above 64 use one wave per node, loop over the picks in chunks of 64 and keep the chosen
// positions in LDS.
//
// The sampled IDs are de-duplicated right afterwards (into the next hop's frontier, and, in the
// whole-path call, into the batch's ID list), so the lane that writes a sample also inserts it into
// the hash tables of those de-duplications: they then start at their second pass.  The tables must
// be empty before the first insert; who empties which table when is the host runtime's business.
#pragma once
#include "compact_dev.hpp"
#include "philox.hpp"

namespace helios {

constexpr int kMaxFanout = 1024;
constexpr int kFoldItems = 8;                          // seeds per thread in the folded count pass
constexpr int kFoldMaxSeeds = kBlock * kFoldItems;     // 2048

struct HopArgs {
    const int64_t* offsets;
    const int32_t* indices;
    int64_t n_nodes;
    const int32_t* frontier;      // with fold and a recorded batch: unused, the frontier is the batch's seeds
    const int64_t* indptr;        // without fold: [n + 1], read
    Count n_frontier;
    int32_t fanout;
    int32_t hop;
    uint64_t rng_seed;
    const BatchVars* vars;        // nullable: rng_seed and the batch table come from here (recorded batch, not folded)
    int32_t* flat;
    int64_t flat_cap;
    ClearJob clear;               // a table emptied on the way (one that no kernel of this launch touches)
    InsertInto hop_table;         // de-duplication of this hop's samples; position = place in flat
    BatchTables batch;            // de-duplication of [seeds | flat_0 | ...]; position = place in that list
    int32_t* cat_out;             // with batch: receives [seeds | flat_0 | ...]
    int64_t n_seeds;
    uint32_t* claims;             // with batch: [workgroups of the role][waves] words that each wave has added to the batch's table
    const int64_t* cat_begin;     // device word: where flat_hop starts in that list (nullable: hop 0, right after the seeds)
    int32_t* err;
    // folded count pass (hop 0): the outputs that frontier_count_kernel would write
    bool fold;
    BatchFeed feed;               // feed.ring set: a recorded batch starts here
    int32_t* frontier_out;        // nullable: receives a copy of the frontier
    int64_t* indptr_out;          // [n + 1]
    int64_t* n_flat_dev;
    int64_t* size_out;            // nullable: [0] = frontier size, [1] = sample-list size
    Stamps stamps;
};

struct SampleTables {
    InsertInto hop;
    unsigned long long* batch_table;   // nullable
    uint32_t batch_mask;
    int32_t* batch_slot_of;
    int32_t* cat_out;
    uint32_t hop_claims, batch_claims;   // words this lane has added to the two tables
};

// id goes to place `at` of flat, if it is a sample and not a seed, to place cat_at of [seeds | flat_0 | ...], and
// into the tables of the de-duplications that follow.  (One table after the other: with both first tries in flight together, and
// with a plain read before each, the passes took 0.5 to 2 us longer.)
__device__ __forceinline__ void put_id(SampleTables& t, int64_t n_nodes, int32_t* err, int32_t* flat, int32_t id, bool sample, uint32_t at,
                                       uint32_t cat_at) {
    const uint32_t uid = static_cast<uint32_t>(id);
    const bool node = uid < static_cast<uint32_t>(n_nodes);
    if (sample) {
        flat[at] = id;
        if (!node) raise(err, kErrData);                 // (a seed that is no node has been reported by the count pass)
        if (t.hop.table) t.hop.slot_of[at] = node ? static_cast<int32_t>(table_insert(t.hop.table, t.hop.n_slots - 1, uid, at, t.hop_claims)) : -1;
    }
    if (t.batch_table) {
        t.cat_out[cat_at] = id;
        t.batch_slot_of[cat_at] = node ? static_cast<int32_t>(table_insert(t.batch_table, t.batch_mask, uid, cat_at, t.batch_claims)) : -1;
    }
}

// What the count pass, where the sampling kernel does it, leaves in LDS for the nodes that this workgroup samples.
template <int N>
struct OwnNodesOf {
    int64_t base[N];
    int32_t v[N], deg[N];
    uint32_t out[N];
};
using OwnNodes = OwnNodesOf<kBlock / 8>;

// The count pass of a frontier of at most K * kBlock nodes, redone by every workgroup: item k of a thread is node
// k * kBlock + threadIdx.x.  All loads of a step are issued before the first is used.
template <int K>
__device__ __forceinline__ void fold_count(const HopArgs& a, const int32_t* frontier, uint32_t n, uint32_t own0, uint32_t n_own, bool first_wg,
                                           OwnNodes& own, uint32_t* s_tot /* 4 K words */) {
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave_id())), lane = static_cast<uint32_t>(lane_id());
    int32_t v[K];
    RowBounds row[K];
    uint32_t cnt[K], inc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t j = threadIdx.x + k * kBlock;
        v[k] = n > 0 ? frontier[j < n ? j : n - 1] : -1;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool ok = v[k] >= 0 && static_cast<int64_t>(v[k]) < a.n_nodes;
        row[k] = RowBounds{0, 0};
        if (a.n_nodes > 0) row[k] = row_bounds(a.offsets, ok ? static_cast<uint32_t>(v[k]) : 0u);      // (uniform guard)
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool here = threadIdx.x + k * kBlock < n;
        const bool ok = v[k] >= 0 && static_cast<int64_t>(v[k]) < a.n_nodes;
        const int64_t d = ok ? row[k].hi - row[k].lo : 0;
        const bool bad = d < 0 || d > 0x7fffffffLL;
        if (here && (!ok || bad)) raise(a.err, kErrData);
        const int64_t f = a.fanout > 0 ? a.fanout : 0;
        cnt[k] = here && !bad ? static_cast<uint32_t>(d < f ? d : f) : 0u;
        inc[k] = dpp_inclusive_scan(cnt[k]);
        if (lane == kWave - 1) s_tot[k * kWavesPerBlock + wave] = inc[k];
        row[k].hi = bad ? 0 : d;
    }
    __syncthreads();
    const uint32_t mine = lane < K * kWavesPerBlock ? s_tot[lane] : 0u;
    const uint32_t upto = dpp_inclusive_scan(mine);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t j = threadIdx.x + k * kBlock, run = k * kWavesPerBlock + wave;
        const uint32_t at = lane_value(upto, run) - lane_value(mine, run) + inc[k] - cnt[k];
        if (j < n && j - own0 < n_own) {                  // unsigned: not below own0 either
            own.base[j - own0] = row[k].lo;
            own.v[j - own0] = v[k];
            own.deg[j - own0] = static_cast<int32_t>(row[k].hi);
            own.out[j - own0] = at;
        }
        if (first_wg && j < n) {
            a.indptr_out[j] = at;
            if (a.frontier_out && a.frontier_out != frontier) a.frontier_out[j] = v[k];
        }
    }
    if (first_wg && threadIdx.x == 0) {
        const uint32_t total = lane_value(upto, kWave - 1);
        a.indptr_out[n] = total;
        *a.n_flat_dev = total;
        if (a.size_out) { a.size_out[0] = n; a.size_out[1] = total; }
        if (static_cast<int64_t>(total) > a.flat_cap) raise(a.err, kErrCapacity);
    }
    __syncthreads();
}

// Floyd: step k takes t_k unless an earlier step already holds it, then it takes j_k.  Step i's pick is final once
// the steps before it have been applied to it.  Lane l has step l.
template <int G, int I = 0>
__device__ __forceinline__ void floyd_settle(int f, bool floyd, int l, int32_t t, int32_t j, int32_t& s) {
    if constexpr (G <= 16) {
        if constexpr (I + 1 < G) {
            if (I + 1 >= f) return;                               // uniform
            const int32_t si = group_value<G, I>(s);
            if (floyd && l > I && si == t) s = j;
            floyd_settle<G, I + 1>(f, floyd, l, t, j, s);
        }
    } else {
        for (int i = 0; i + 1 < f; ++i) {
            const int32_t si = group_value<G>(s, i);
            if (floyd && l > i && si == t) s = j;
        }
    }
}

// The position in v's row of the l-th sample, of a group of G lanes for one node; f <= G.
template <int G>
__device__ __forceinline__ int32_t pick(uint64_t rng_seed, int32_t v, int32_t hop, int32_t deg, int f, int l) {
    int32_t pos = l;                                  // deg <= f: the whole row, CSR order
    const bool floyd = deg > f && l < f;
    const int32_t j = deg - f + l;                    // position looked at in step l
    int32_t s = pos;
    if (__ballot(floyd) != 0) {                       // about half the nodes have no more neighbours than the fan-out
        if (floyd) pos = static_cast<int32_t>(bounded(node_draw(rng_seed, v, hop, static_cast<uint32_t>(l)), static_cast<uint32_t>(j) + 1u));
        s = pos;
        floyd_settle<G>(f, floyd, l, pos, j, s);
    }
    return s;
}

// What bounds the role: for a short frontier the chain of dependent reads and instructions (batch variables, seeds, row bounds,
// draw, picks, neighbour, tables), for a long one the table inserts (the part does about 25 random atomics per ns).
// Measured, hop 0 of 1024 seeds: 12.1 us in a recorded batch (14.9 with guarded loads in the folded count, the row bounds read
// twice and the seed's insert before its samples'), 15.7 us in a gang of four (18.3), 7.7 us for 128 seeds (10.3).
template <int G>
__device__ __forceinline__ void sample_role(const HopArgs& a, uint32_t rb, uint32_t nrb) {
    constexpr int kGroups = kBlock / G;          // nodes per workgroup and step
    __shared__ int32_t s_chosen[(G == kWave) ? kWavesPerBlock * kMaxFanout : 1];
    __shared__ OwnNodes own;
    __shared__ uint32_t s_tot[kFoldItems * kWavesPerBlock];

    stamp_start(a.stamps, rb);
    const int f = a.fanout;
    const int group = threadIdx.x / G;
    const int l = threadIdx.x % G;
    const uint32_t step = nrb * kGroups;
    // The first node of the group is fetched before the actual length of the frontier is known (the buffers hold
    // n_frontier.host entries, so the read is in bounds).
    uint32_t i = rb * kGroups + group;
    int32_t v = -1;
    int64_t out = -1;
    if (!a.fold && i < a.n_frontier.host) {
        v = a.frontier[i];
        out = a.indptr[i];
    }
    const uint32_t n = static_cast<uint32_t>(a.n_frontier.get());
    const uint32_t cat_base = static_cast<uint32_t>(a.cat_begin ? *a.cat_begin : a.n_seeds);      // where flat_hop starts in [seeds | flat_0 | ...]
    // A recorded batch starts at its folded hop 0: every workgroup reads the batch's variables from the slot of
    // the host's ring that the count of batches run so far selects, and the first leaves them in device memory
    // for the kernels that follow (the next kernel advances the count).
    uint64_t rng_seed = a.rng_seed;
    uint32_t which = a.batch.which;
    if (a.fold) {
        const int32_t* frontier = a.frontier;
        if (a.feed.ring) {
            const BatchVars bv = a.feed.ring[*a.feed.batches_run % a.feed.ring_slots];
            if (rb == 0 && threadIdx.x == 0) *a.feed.vars_out = bv;
            frontier = bv.seeds;
            rng_seed = bv.rng_seed;
            which = bv.table % kBatchTables;
        }
        // (a folded frontier is sampled in one step: the grid covers it)
        if (n <= kBlock) fold_count<1>(a, frontier, n, rb * kGroups, kGroups, rb == 0, own, s_tot);
        else if (n <= 4 * kBlock) fold_count<4>(a, frontier, n, rb * kGroups, kGroups, rb == 0, own, s_tot);
        else fold_count<kFoldItems>(a, frontier, n, rb * kGroups, kGroups, rb == 0, own, s_tot);
    } else if (a.vars) {
        rng_seed = a.vars->rng_seed;
        which = a.vars->table % kBatchTables;
    }
    for (uint32_t w = rb * kBlock + threadIdx.x; a.clear.table && w < a.clear.n_slots; w += nrb * kBlock)
        a.clear.table[w] = kEmptySlot;                    // side job of the role (at its end it would be a tail of its own)
    SampleTables tabs{a.hop_table, nullptr, 0, nullptr, a.cat_out, 0, 0};
    uint32_t* claims = nullptr;
    if (a.batch.table0) {
        // (fetched with the arguments here: at the end of the role, where it is used, the read would be waited for by itself, 0.3 us)
        claims = a.claims;
        asm volatile("" : "+s"(claims));
        tabs.batch_table = a.batch.table(which);
        tabs.batch_mask = a.batch.n_slots - 1;
        tabs.batch_slot_of = a.batch.slot_of(which);
    }
    const bool seeds_too = tabs.batch_table && a.hop == 0;   // the frontier of hop 0 is the head of the batch's list
    if (f > 0 || seeds_too) {
        for (bool again = false; i < n; i += step, again = true) {
            // the lanes of a group read the same words
            int64_t base;
            int32_t deg;
            if (a.fold) {
                v = own.v[group];
                base = own.base[group];
                deg = own.deg[group];
                out = own.out[group];
            } else {
                if (again) {
                    v = a.frontier[i];
                    out = a.indptr[i];
                }
                // a value that is no node ID, or a row that is none, has been reported by the count pass
                const bool ok = v >= 0 && static_cast<int64_t>(v) < a.n_nodes;
                RowBounds row{0, 0};
                if (a.n_nodes > 0) row = row_bounds(a.offsets, ok ? static_cast<uint32_t>(v) : 0u);
                const int64_t d = ok ? row.hi - row.lo : 0;
                base = row.lo;
                deg = d > 0 && d <= 0x7fffffffLL ? static_cast<int32_t>(d) : 0;
            }
            const int cnt = deg < f ? deg : f;
            // `out` can only be off if an earlier output overflowed its capacity; never write outside flat, but
            // write every place below the capacity: the de-duplications read all of them
            const bool out_ok = out >= 0;
            const int64_t room = a.flat_cap - out;   // samples of this node that fit

            if (f <= G) {
                const int32_t s = pick<G>(rng_seed, v, a.hop, deg, f, l);
                const bool sample = l < cnt && out_ok && l < room;
                const uint32_t at = static_cast<uint32_t>(out) + l;
                if (!seeds_too) {
                    if (sample) put_id(tabs, a.n_nodes, a.err, a.flat, a.indices[base + s], true, at, cat_base + at);
                    continue;
                }
                // the seed itself goes into the batch's list by a lane that has no sample (or by lane 0 afterwards)
                const bool seed = f < G && l == f;
                if (sample || seed) {
                    int32_t id = v;
                    if (sample) id = a.indices[base + s];
                    put_id(tabs, a.n_nodes, a.err, a.flat, id, sample, at, sample ? cat_base + at : i);
                }
                if (f == G && l == 0) put_id(tabs, a.n_nodes, a.err, a.flat, v, false, 0, i);
                continue;
            }
            if constexpr (G == kWave) {                           // fan-out above 64: one wave per node
                const uint32_t at = static_cast<uint32_t>(out);
                if (seeds_too && l == 0) put_id(tabs, a.n_nodes, a.err, a.flat, v, false, 0, i);
                if (deg <= f) {
                    for (int k = l; k < deg; k += kWave)
                        if (out_ok && k < room) put_id(tabs, a.n_nodes, a.err, a.flat, a.indices[base + k], true, at + k, cat_base + at + k);
                    continue;
                }
                int32_t* chosen = s_chosen + wave_id() * kMaxFanout;
                for (int c0 = 0; c0 < f; c0 += kWave) {
                    const int k = c0 + l;
                    const bool active = k < f;
                    const int32_t j = deg - f + k;
                    int32_t t = -1, s = -1;
                    if (active) {
                        t = static_cast<int32_t>(bounded(node_draw(rng_seed, v, a.hop, static_cast<uint32_t>(k)), static_cast<uint32_t>(j) + 1u));
                        s = t;
                        for (int p = 0; p < c0; ++p)
                            if (chosen[p] == t) s = j;            // taken in an earlier chunk
                    }
                    const int in_chunk = f - c0 < kWave ? f - c0 : kWave;
                    for (int i2 = 0; i2 + 1 < in_chunk; ++i2) {
                        const int32_t si = group_value<kWave>(s, i2);
                        if (active && l > i2 && si == t) s = j;
                    }
                    if (active) {
                        chosen[k] = s;
                        if (out_ok && k < room) put_id(tabs, a.n_nodes, a.err, a.flat, a.indices[base + s], true, at + k, cat_base + at + k);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
            }
        }
    }
    if (claims) {
        const uint32_t sum = dpp_sum(tabs.batch_claims);
        if (lane_id() == 0) claims[rb * kWavesPerBlock + wave_id()] = sum;
    }
    stamp_end(a.stamps, rb, nrb);
}

inline int group_lanes(int32_t fanout) { return fanout <= 8 ? 8 : fanout <= 16 ? 16 : fanout <= 32 ? 32 : 64; }

// Workgroups of a sampling role over a frontier of at most n_max nodes.  The bound is usually several times the
// frontier's length, and a workgroup costs about 1 ns of the launch whether it has work or not, so a launch gets no more
// than the chip holds at once (eight per CU) and they loop.  Measured: second hop of four batches of 41 k samples 14.8 us with
// one step per workgroup (6400), 11.0 with 2048, 12.6 with 1024; second hop of 10 k seeds, fan-outs 25 and 10, 17.3 us with
// 15625, 11.8 with 2048, 17.4 with 512.
constexpr int64_t kSampleMaxWorkgroups = 2048;
static_assert(kFoldMaxSeeds / (kBlock / kWave) <= kSampleMaxWorkgroups / 4, "a folded frontier is sampled in one step, in a gang of four too");
inline unsigned sample_role_blocks(int32_t fanout, int64_t n_max, int share /* roles that run in the same launch */) {
    const int64_t per_block = kBlock / group_lanes(fanout);
    int64_t blocks = (n_max + per_block - 1) / per_block;
    if (blocks < 1) blocks = 1;
    if (blocks > kSampleMaxWorkgroups / share) blocks = kSampleMaxWorkgroups / share;
    return static_cast<unsigned>(blocks);
}

}  // namespace helios
