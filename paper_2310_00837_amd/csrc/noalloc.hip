// helios_dedup_noalloc: the de-duplication of helios_dedup for callers that cannot allocate
// (code under HIP graph capture, tight serving loops, harnesses that forbid hipMalloc).
//
// helios_dedup takes its scratch (hash table, slot of every input, unique index of every first
// occurrence, scan status words, counters) from memory the context allocates and grows.  Here all
// of it lives in one file-scope device array of fixed size, so the call enqueues kernels and
// nothing else.  The array exists once per GPU the library runs on.  It is filled once, when the
// first context of that GPU is created.  The first launch of every call zeroes the scan status and the ticket, and the
// last one leaves the table empty, beside work that uses none of them (a launch of its own at the start of every call
// took 3 us).  So a captured call can be replayed.
// Only a call that a launch error has cut short leaves the table in use; the next call fills the array first.
// All calls on one GPU share the array, so calls that overlap on one GPU (two streams, two
// contexts, two host threads) race; callers serialise them.  Calls that did overlap spoil each other and no
// later one: what a call has put into the table, also while another was at work in it, its own last launch,
// which is behind its own writes on its stream, takes out again, and status and ticket a call never takes over from
// another (two scans that draw from the ticket at the same time may both miss the draw that puts it back to zero).
#include "context.hpp"
#include "noalloc.hpp"

#include <mutex>

using namespace helios;

namespace {

constexpr int64_t kMaxIds = HELIOS_DEDUP_NOALLOC_MAX_IDS;
constexpr uint32_t kSlots = 2u * static_cast<uint32_t>(kMaxIds);              // power of two, twice the inputs
constexpr uint32_t kStride = static_cast<uint32_t>(kMaxIds / kScanBlock + 2);   // tiles the status rows hold
static_assert((kSlots & (kSlots - 1)) == 0, "the table size must be a power of two");

// layout of the scratch array, in bytes (every part 256-byte aligned)
constexpr size_t kOffTable = 0;
constexpr size_t kOffSlotOf = kOffTable + sizeof(unsigned long long) * kSlots;
constexpr size_t kOffIndexOfFirst = kOffSlotOf + sizeof(int32_t) * kMaxIds;
constexpr size_t kOffStatus = kOffIndexOfFirst + sizeof(int32_t) * kMaxIds;
constexpr size_t kStatusBytes = (sizeof(unsigned long long) * 3 * kStride + 255) / 256 * 256;
constexpr size_t kOffSmall = kOffStatus + kStatusBytes;     // ticket (uint32) at +0, counters (int64[2]) at +64
constexpr size_t kSmallBytes = 256;
constexpr size_t kOffTicket = kOffSmall, kOffCounters = kOffSmall + 64;
// what the first launch of a call zeroes: the scan status and the ticket right behind it
constexpr uint32_t kZeroWords = static_cast<uint32_t>((kOffTicket + sizeof(unsigned long long) - kOffStatus) / sizeof(unsigned long long));
static_assert(kOffStatus + kZeroWords * sizeof(unsigned long long) >= kOffTicket + sizeof(uint32_t) &&
              kOffStatus + kZeroWords * sizeof(unsigned long long) <= kOffCounters, "the ticket is in, the counters are not");
// A long list is taken apart by hash in memory of its own (and uses the table, if at all, as other calls do: it leaves it empty).
// Of the index of every first occurrence it uses 1/16, and where its buckets begin stands behind that.
constexpr size_t kOffPartId = kOffSmall + kSmallBytes;
constexpr size_t kOffPartFirst = kOffPartId + sizeof(int32_t) * kMaxIds;
constexpr size_t kOffPartPos = kOffPartFirst + sizeof(uint32_t) * kMaxIds;
constexpr size_t kOffPartLocal = kOffPartPos + sizeof(uint16_t) * kMaxIds;
constexpr size_t kScratchBytes = kOffPartLocal + sizeof(uint16_t) * kMaxIds;
constexpr size_t kOffPartStarts = kOffIndexOfFirst + sizeof(uint32_t) * (kMaxIds / 16);
static_assert(kMaxIds <= kPartsMax && kMaxIds <= 256 * kMinPartTile && kMinPartTile / 16 % kLineWords == 0 && kOffPartStarts + static_cast<size_t>(split_starts_bytes(256)) <= kOffStatus,
              "the longest list can be taken apart, into 256 tiles at most, whose words leave no room between them");
static_assert(kScratchBytes < (9u << 20) + (256u << 10), "include/helios.h says how large the array is");

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_mu;
unsigned char* g_ptr[kMaxDevices] = {nullptr};     // device address of `scratch` on every GPU seen so far
bool g_in_use[kMaxDevices] = {false};              // a call has been cut short: the array has to be filled

// empties the table, zeroes the scan status words and the small block
__global__ __launch_bounds__(kBlock) void noalloc_reset_kernel(unsigned long long* table, uint32_t n_slots,
                                                               unsigned long long* zero_from, uint32_t n_zero_words) {
    const uint32_t step = gridDim.x * kBlock;
    for (uint32_t w = blockIdx.x * kBlock + threadIdx.x; w < n_slots; w += step) table[w] = kEmptySlot;
    for (uint32_t w = blockIdx.x * kBlock + threadIdx.x; w < n_zero_words; w += step) zero_from[w] = 0ull;
}

hipError_t launch_reset(hipStream_t stream, unsigned char* base, uint32_t slots) {
    const uint32_t zero_words = static_cast<uint32_t>((kStatusBytes + kSmallBytes) / sizeof(unsigned long long));
    unsigned blocks = (slots + kBlock * 16 - 1) / (kBlock * 16);
    blocks = blocks < 1 ? 1 : blocks > 1024 ? 1024 : blocks;
    hipLaunchKernelGGL(noalloc_reset_kernel, dim3(blocks), dim3(kBlock), 0, stream, reinterpret_cast<unsigned long long*>(base + kOffTable),
                       slots, reinterpret_cast<unsigned long long*>(base + kOffStatus), zero_words);
    return hipGetLastError();
}

}  // namespace

namespace helios {

int noalloc_init(int device, hipStream_t stream) {
    if (device < 0 || device >= kMaxDevices) return HELIOS_EINVAL;
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_ptr[device]) return HELIOS_OK;
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {     // the current device's copy of the array
        (void)hipGetLastError();
        return HELIOS_EHIP;
    }
    if (launch_reset(stream, static_cast<unsigned char*>(p), kSlots) != hipSuccess || hipStreamSynchronize(stream) != hipSuccess) {
        (void)hipGetLastError();
        return HELIOS_EHIP;
    }
    g_ptr[device] = static_cast<unsigned char*>(p);
    return HELIOS_OK;
}

}  // namespace helios

extern "C" int helios_dedup_noalloc(helios_ctx* c, const int32_t* ids, int64_t n_ids, int32_t* unique, int64_t unique_cap,
                                    int32_t* inverse, int64_t* n_unique) {
    if (!c) return HELIOS_EINVAL;
    if (!c->has_graph) return fail(c, HELIOS_ESTATE, "helios_dedup_noalloc before helios_csr_load");
    if (n_ids < 0 || unique_cap < 0) return fail(c, HELIOS_EINVAL, "negative size");
    if (n_ids > kMaxIds)
        return fail(c, HELIOS_EINVAL, "helios_dedup_noalloc handles at most %lld IDs per call (got %lld); use helios_dedup",
                    (long long)kMaxIds, (long long)n_ids);
    if ((n_ids > 0 && !ids) || (unique_cap > 0 && !unique)) return fail(c, HELIOS_EINVAL, "NULL pointer");
    unsigned char* base = nullptr;
    bool fill = false;
    if (c->device >= 0 && c->device < kMaxDevices) {
        std::lock_guard<std::mutex> lk(g_mu);
        base = g_ptr[c->device];
        fill = g_in_use[c->device];
        g_in_use[c->device] = true;              // until the last launch has gone out
    }
    if (!base) return fail(c, HELIOS_ESTATE, "the static scratch of device %d was not set up by helios_create", c->device);
    DeviceGuard guard(c->device);
    unsigned long long* table = reinterpret_cast<unsigned long long*>(base + kOffTable);
    unsigned long long* status = reinterpret_cast<unsigned long long*>(base + kOffStatus);
    uint32_t* ticket = reinterpret_cast<uint32_t*>(base + kOffTicket);
    int64_t* counters = reinterpret_cast<int64_t*>(base + kOffCounters);
    const uint32_t slots = list_slots(n_ids, kSlots);
    const DedupScratch s{table, slots, reinterpret_cast<int32_t*>(base + kOffSlotOf),
                         reinterpret_cast<int32_t*>(base + kOffIndexOfFirst)};
    if (fill) HIP_TRY(c, launch_reset(c->stream, base, kSlots));
    // the first launch zeroes the status words, so any epoch but zero reads them as unpublished; the same value every
    // call keeps a captured call replayable
    const ScanState scan{status, ticket, kStride, 1u, nullptr};
    const Count n{nullptr, n_ids};
    CompactArgs a{};
    a.ids = ids;
    a.n_nodes = static_cast<uint32_t>(c->g.n_nodes);
    a.len = n;
    a.n_max = static_cast<uint32_t>(n_ids);
    a.n_total_dev = counters + 0;
    a.s = s;
    a.unique = unique;
    a.unique_cap = unique_cap;
    a.last = true;
    a.n_unique_dev = counters + 1;
    a.n_unique_out = n_unique;
    a.inverse = inverse;
    a.scan = scan;
    a.err = c->err;
    const bool by_parts = dedup_by_parts(n_ids, slots);
    if (by_parts) {
        const PartScratch parts{reinterpret_cast<int32_t*>(base + kOffPartId), reinterpret_cast<uint16_t*>(base + kOffPartPos),
                                reinterpret_cast<uint32_t*>(base + kOffPartFirst), reinterpret_cast<uint16_t*>(base + kOffPartLocal),
                                reinterpret_cast<uint16_t*>(base + kOffPartStarts), status, kZeroWords};
        HIP_TRY(c, launch_dedup_by_parts(c->stream, a, n_ids, c->g.n_nodes, parts));
    } else {
        HIP_TRY(c, launch_dedup_insert(c->stream, ids, n, n_ids, c->g.n_nodes, s, status, kZeroWords, c->err));
        HIP_TRY(c, launch_dedup_compact_plain(c->stream, a, n_ids));
        const InverseArgs inv{Count{counters + 0, n_ids}, s.index_of_first, BatchTables{}, nullptr, inverse, false, Stamps{nullptr}};
        HIP_TRY(c, launch_dedup_end(c->stream, inv, n_ids, ClearJob{table, slots}));
    }
    // A call that is being captured has not run.  It found the array clean, and leaves it so, unless the filling was
    // captured with it: then the next call still has to do that.
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (fill && hipStreamIsCapturing(c->stream, &capture) != hipSuccess) (void)hipGetLastError();
    std::lock_guard<std::mutex> lk(g_mu);
    g_in_use[c->device] = capture != hipStreamCaptureStatusNone;
    return HELIOS_OK;
}
