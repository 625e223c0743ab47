"""The kernels that take a long list apart by hash, compiled for the host: their results, and what they do with scratch memory that
another call has written into (calls of helios_dedup_noalloc that overlap on one GPU share it, and may only spoil each other's
results).  Every buffer lies between pages that cannot be touched, so an access out of bounds ends the program."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2310_00837_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
PROGRAM = r"""
#include "dedup.hip"
#include <sys/mman.h>
#include <string.h>
#include <algorithm>
#include <string>
#include <unordered_map>
using namespace helios;

static_assert(alignof(PartTable) >= 16, "it is cleared 16 bytes at a time");

// n elements that end where a page that cannot be touched begins, with 32 GiB of such pages on either side
template <class T>
T* guarded(size_t n) {
    const size_t guard = size_t{32} << 30, bytes = (n * sizeof(T) + 4095) / 4096 * 4096;
    char* p = static_cast<char*>(mmap(nullptr, guard + bytes + guard, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
    if (p == MAP_FAILED || mprotect(p + guard, bytes, PROT_READ | PROT_WRITE) != 0) abort();
    memset(p + guard, 0x5a, bytes);
    return reinterpret_cast<T*>(p + guard + bytes - n * sizeof(T));
}

constexpr int64_t kNodes = 0x7fffffff;
struct Call {
    PartShape shape;
    int64_t n, tiles;
    int32_t *ids, *unique, *inverse, *iof;
    PartScratch s;
    uint32_t n_slots;
    unsigned long long *table, *status;
    unsigned long long* ticket;
    int64_t* counters;
    int32_t* err;
    CompactArgs a{};
    explicit Call(const std::vector<int32_t>& list, int64_t cap, bool in_place = false) : shape(list.size()), n(list.size()), tiles(shape.n_tiles) {
        ids = guarded<int32_t>(n);
        unique = in_place ? ids : guarded<int32_t>(cap);
        inverse = guarded<int32_t>(n);
        const int64_t words = (n + 31) / 32 * 32;          // (whole lines, so that it begins one)
        iof = guarded<int32_t>(words);
        on_host::cached.begin = reinterpret_cast<const char*>(iof);
        on_host::cached.end = reinterpret_cast<const char*>(iof + words);
        s = PartScratch{guarded<int32_t>(n), guarded<uint16_t>(n), guarded<uint32_t>(n), guarded<uint16_t>(n),
                        guarded<uint16_t>(split_starts_bytes(tiles) / 2), nullptr, 0};
        for (n_slots = 1024; n_slots < 2 * n;) n_slots *= 2;
        table = guarded<unsigned long long>(n_slots);
        status = guarded<unsigned long long>(tiles);
        ticket = guarded<unsigned long long>(1);
        counters = guarded<int64_t>(2);
        err = guarded<int32_t>(2);
        memcpy(ids, list.data(), 4 * n);
        memset(table, 0xff, 8 * size_t{n_slots});
        memset(status, 0, 8 * tiles);
        *ticket = 0;
        err[0] = 0;
        a.ids = ids;
        a.n_nodes = kNodes;
        a.len = Count{nullptr, n};
        a.n_total_dev = counters;
        a.s = DedupScratch{table, n_slots, nullptr, iof};
        a.unique = unique;
        a.unique_cap = cap;
        a.last = true;
        a.n_unique_dev = counters + 1;
        a.inverse = inverse;
        a.scan = ScanState{status, reinterpret_cast<uint32_t*>(ticket), static_cast<uint32_t>(tiles), 1, nullptr};
        a.err = err;
    }
    void split() const {
        hipLaunchKernelGGL(dedup_split_kernel<6>, dim3(tiles), dim3(kSplitBlock), 0, nullptr, a.ids, shape, kNodes, s, err);
    }
    void buckets() const { hipLaunchKernelGGL(dedup_bucket_kernel, dim3(kParts), dim3(kBucketBlock), 0, nullptr, s, shape, table, n_slots, err); }
    bool table_empty() const { return std::all_of(table, table + n_slots, [](unsigned long long w) { return w == kEmptySlot; }); }
    void compact() const { hipLaunchKernelGGL(dedup_compact_parts_kernel<6>, dim3(tiles), dim3(kMergeBlock), 0, nullptr, a, s, shape); }
};

void check(bool ok, const char* what) {
    if (ok) return;
    printf("wrong: %s\n", what);
    exit(1);
}

void results(const std::vector<int32_t>& list, int64_t cap, bool in_place) {
    Call c(list, cap, in_place);
    launch_dedup_by_parts(nullptr, c.a, c.n, kNodes, c.s);
    std::unordered_map<int32_t, int32_t> at;
    std::vector<int32_t> want;
    bool bad = false;
    for (int64_t j = 0; j < c.n; ++j) {
        if (list[j] < 0 || list[j] >= kNodes) {
            bad = true;
            check(c.inverse[j] == -1, "inverse of an entry that is no node");
            continue;
        }
        if (at.emplace(list[j], static_cast<int32_t>(want.size())).second) want.push_back(list[j]);
        check(c.inverse[j] == at[list[j]], "inverse");
    }
    const int64_t u = want.size();
    check(c.counters[1] == u, "n_unique");
    check(std::equal(want.begin(), want.begin() + std::min(u, cap), c.unique), "unique");
    check(c.err[0] == (u > cap ? kErrCapacity : bad ? kErrData : 0), "error");
    check(*c.ticket == 0 && c.table_empty(), "left as found");
}

uint32_t next_random() {
    static uint64_t x = 88172645463325252ull;
    x ^= x << 13, x ^= x >> 7, x ^= x << 17;
    return static_cast<uint32_t>(x >> 16);
}
std::vector<int32_t> hashing_to(size_t n, uint32_t mask, uint32_t value) {
    std::vector<int32_t> v;
    for (int32_t id = 0; v.size() < n; ++id)
        if ((part_hash(static_cast<uint32_t>(id)) & mask) == value) v.push_back(id);
    return v;
}

int main(int argc, char** argv) {
    const std::string what = argv[1];
    if (what == "results") {
        for (int64_t n : {1, 4096, 8195}) {
            std::vector<int32_t> few(n);
            for (int64_t j = 0; j < n; ++j) few[j] = next_random() % (n / 3 + 1);
            if (n > 1) results(few, n, true);            // `unique` in the memory of the IDs
            if (n != 4096) results(few, n / 5, false);
            if (n == 4096) continue;
            few[0] = -1, few[n / 2] = kNodes, few[n - 1] = INT32_MIN;
            results(few, n, n % 2);
        }
    } else if (what == "uneven") {                       // more in two buckets than fits their tables, repeats among them
        std::vector<int32_t> v = hashing_to(18000, 0xff800000u, 5u << 23);
        const std::vector<int32_t> w = hashing_to(9000, 0xff800000u, 200u << 23);
        v.insert(v.end(), w.begin(), w.end());
        for (int j = 0; j < 3000; ++j) v.push_back(v[next_random() % v.size()]);
        for (int j = 0; j < 3000; ++j) v.push_back(static_cast<int32_t>(next_random() >> 1));
        for (size_t j = v.size() - 1; j > 0; --j) std::swap(v[j], v[next_random() % (j + 1)]);
        results(v, v.size(), false);
    } else if (what == "slots") {                        // of a list's table: two or more for each ID, eight up to the longest list by parts, never more than there are
        for (int64_t n : {int64_t{1}, int64_t{1000}, int64_t{8192}, int64_t{19999}, kPartsMax, kPartsMax + 1, int64_t{3000000}, int64_t{16000000}})
            for (uint32_t most = 1024; most >= 1024 && most <= 1u << 28; most *= 2) {
                if (most < 2 * n) continue;
                const uint32_t slots = list_slots(n, most);
                check(slots <= most && slots >= 2 * n && slots >= 1024 && (slots & (slots - 1)) == 0, "a table for the list");
                check(slots <= std::max<int64_t>(1024, (n <= kPartsMax ? 16 : 4) * n), "no larger than needed");
                check(n > kPartsMax || slots >= 8 * n || slots == most, "eight for each");
            }
    } else if (what == "lines") {                        // tiles that are no whole lines of flags; repeats of first occurrences of the same tile and of all before
        for (int64_t n : {263000, 300000}) {
            const uint32_t tile = PartShape(n).tile;
            check(tile > kMinPartTile && tile % 512 != 0, "such tiles");
            std::vector<int32_t> v(n);
            for (int64_t j = 0; j < n; ++j) {
                const int64_t in = j % tile, begin = j - in;
                v[j] = static_cast<int32_t>(j);
                if (in >= tile - 4) v[j] = v[j - 40];                                                   // their first occurrences in the tile's last words
                else if (in >= tile / 2 && in < tile / 2 + 100 && j >= tile) v[j] = v[next_random() % (begin / tile) * tile + next_random() % 60];      // in a tile's first words
            }
            results(v, n, false);
        }
    } else if (what == "crowded") {                      // a bucket of many times its share, that a table in LDS takes: nothing goes by memory
        std::vector<int32_t> v = hashing_to(5000, 0xff800000u, 5u << 23);
        for (int j = 0; j < 16000; ++j) v.push_back(static_cast<int32_t>(next_random() >> 1));
        for (size_t j = v.size() - 1; j > 0; --j) std::swap(v[j], v[next_random() % (j + 1)]);
        results(v, v.size(), false);
        Call c(v, v.size());
        c.n_slots = 0;                                   // (what would use the memory raises an error)
        c.split();
        c.buckets();
        check(c.err[0] == 0, "by LDS");
    } else if (what == "pieces") {                       // the words of two calls side by side, as their waves write them, and any words
        const int n = 32 * kPartTile;
        std::vector<int32_t> one(n, 77), distinct(n);
        for (int j = 0; j < n; ++j) distinct[j] = j;
        Call a(distinct, n), b(one, n);
        a.split();
        b.split();
        for (int64_t t = 0; t < a.tiles; ++t)
            for (int w = 64; w <= kParts; ++w)
                if ((w / 64) % 2) a.s.starts[t * (kParts + 1) + w] = b.s.starts[t * (kParts + 1) + w];
        a.buckets();
        check(a.err[0] == kErrInternal, "the call has to notice");
        for (int64_t q = 0; q < split_starts_bytes(a.tiles) / 2; ++q) a.s.starts[q] = static_cast<uint16_t>(next_random());
        a.buckets();
        a.compact();                                     // (the bound of a tile's entries is such a word too)
    } else if (what == "tickets") {                      // two calls draw tickets from one counter
        std::vector<int32_t> v(3 * kPartTile - 5);
        for (size_t j = 0; j < v.size(); ++j) v[j] = static_cast<int32_t>(j / 2);
        for (unsigned drawn : {0u, 1u, 40u}) {
            Call c(v, v.size());
            c.split();
            c.buckets();
            for (int64_t t = 0; t < c.tiles; ++t) c.status[t] = scan_pack(1, kFlagPrefix, 0);     // (what the other call has published)
            *c.ticket = c.tiles + drawn;
            c.compact();
            check(c.err[0] == kErrInternal, "the call has to notice");
        }
    } else if (what == "foreign") {                      // a bucket's piece holds another call's IDs, all of one class of the hash
        const int n = 16 * kPartTile;
        std::vector<int32_t> v(n, 77);
        Call c(v, n);
        c.split();
        const std::vector<int32_t> same = hashing_to(n, 1023, 3);
        memcpy(c.s.id, same.data(), 4 * n);
        for (int j = 0; j < n; ++j) c.s.pos[j] = j % c.shape.tile;
        for (int64_t t = 0; t < c.tiles; ++t)
            for (int w = 0; w <= kParts; ++w) c.s.starts[t * (kParts + 1) + w] = w > 9 ? std::min<int64_t>(c.shape.tile, n - t * c.shape.tile) : 0;      // all in bucket 9
        c.buckets();
        check(c.table_empty(), "left as found");
        for (int j = 0; j < n; ++j) check(c.s.first[j] == static_cast<uint32_t>(j), "first position");
    } else {
        return 3;
    }
    printf("ok\n");
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run([CLANG, "-std=c++17", "-O0", "-w", "-U_FORTIFY_SOURCE", "-I", os.path.join(HERE, "hip_on_the_host"), "-I", CSRC,
                    str(d / "main.cpp"), "-o", str(d / "main")], check=True, timeout=100)
    return str(d / "main")


@pytest.mark.parametrize("what", ["results", "uneven", "slots", "lines", "crowded", "pieces", "tickets", "foreign"])
def test_list_by_parts(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout)
