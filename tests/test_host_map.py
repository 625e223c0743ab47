"""The kernels that make the cache map by buckets, compiled for the host: the map of orders of every kind, permutations and others, at a
small size.  Every buffer lies between pages that cannot be touched, so an access out of bounds ends the program."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2310_00837_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
PROGRAM = r"""
#include "cache.hip"
#include <sys/mman.h>
#include <string.h>
#include <algorithm>
#include <string>
using namespace helios;

// n elements that end where a page that cannot be touched begins, with 32 GiB of such pages on either side
template <class T>
T* guarded(size_t n) {
    const size_t guard = size_t{32} << 30, bytes = (n * sizeof(T) + 4095) / 4096 * 4096;
    char* p = static_cast<char*>(mmap(nullptr, guard + bytes + guard, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
    if (p == MAP_FAILED || mprotect(p + guard, bytes, PROT_READ | PROT_WRITE) != 0) abort();
    memset(p + guard, 0x5a, bytes);
    return reinterpret_cast<T*>(p + guard + bytes - n * sizeof(T));
}

void check(bool ok, const char* what) {
    if (ok) return;
    printf("wrong: %s\n", what);
    exit(1);
}

void map_of(const std::vector<int32_t>& list, uint32_t shift) {
    const uint32_t n = list.size();
    int32_t *order = guarded<int32_t>(n), *rank = guarded<int32_t>(n), *err = guarded<int32_t>(2);
    int64_t* holes = guarded<int64_t>(1);
    memcpy(order, list.data(), 4 * n);
    err[0] = 0;
    const InvertScratch s{guarded<uint32_t>(2 * kInvertBuckets), guarded<unsigned long long>(n), guarded<uint32_t>(n / kWave)};
    const dim3 block(kInvertBlock), tiles((n + kHandTile - 1) / kHandTile), buckets((n + (1u << shift) - 1) >> shift);
    std::fill(s.cursors, s.cursors + kMapCursors, 0u);
    hipLaunchKernelGGL(rank_split_kernel, tiles, dim3(kHandBlock), 0, nullptr, order, n, shift, s, rank, holes, err);
    hipLaunchKernelGGL(rank_place_kernel<kInvertMaxShift>, buckets, block, 0, nullptr, order, n, shift, s, rank, holes, err);
    check(std::all_of(s.cursors, s.cursors + kMapCursors, [](uint32_t w) { return w == 0; }), "left as found");
    std::vector<int> times(n, 0);
    bool bad = false;
    for (uint32_t r = 0; r < n; ++r) {
        if (list[r] < 0 || list[r] >= static_cast<int32_t>(n)) bad = true;
        else times[list[r]] += 1;
    }
    for (uint32_t v = 0; v < n; ++v) {
        bad = bad || times[v] != 1;
        if (times[v]) check(rank[v] >= 0 && rank[v] < static_cast<int32_t>(n) && list[rank[v]] == static_cast<int32_t>(v), "rank");
        else check(rank[v] == -1, "hole");
    }
    check((*holes != 0) == std::any_of(times.begin(), times.end(), [](int t) { return t == 0; }), "holes");
    check(err[0] == (bad ? kErrData : 0), "error");
}

uint32_t next_random() {
    static uint64_t x = 88172645463325252ull;
    x ^= x << 13, x ^= x >> 7, x ^= x << 17;
    return static_cast<uint32_t>(x >> 16);
}

int main(int argc, char** argv) {
    const std::string what = argv[1];
    const uint32_t n = std::stoul(argv[2]), shift = std::stoul(argv[3]);
    std::vector<int32_t> v(n);
    for (uint32_t j = 0; j < n; ++j) v[j] = j;
    if (what == "descending") std::reverse(v.begin(), v.end());
    if (what == "random") for (uint32_t j = n - 1; j > 0; --j) std::swap(v[j], v[next_random() % (j + 1)]);
    if (what == "hot" || what == "repeats" || what == "too full") {          // classes of equal counts, each ascending: runs, and pairs between them
        std::vector<uint32_t> count(n);
        for (uint32_t j = 0; j < n; ++j) count[j] = next_random() % 100 < 3 ? next_random() % 500 : next_random() % 4;
        std::stable_sort(v.begin(), v.end(), [&](int32_t a, int32_t b) { return count[a] > count[b]; });
    }
    if (what == "repeats") {
        for (uint32_t j = 5; j < n; j += 997) v[j] = v[j - 1];
        v[n / 2] = -3;
        v[n / 3] = n;
    }
    if (what == "too full") for (uint32_t j = n / 4; j < n / 2; ++j) v[j] = n / 5;      // pairs, then runs of one node
    map_of(v, shift);
    printf("ok\n");
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("map")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run([CLANG, "-std=c++17", "-O0", "-w", "-U_FORTIFY_SOURCE", "-I", os.path.join(HERE, "hip_on_the_host"), "-I", CSRC,
                    str(d / "main.cpp"), "-o", str(d / "main")], check=True, timeout=100)
    return str(d / "main")


@pytest.mark.parametrize("n,shift", [(30_001, 10), (65_536, 15), (9_000, 12)])
@pytest.mark.parametrize("what", ["ascending", "descending", "random", "hot", "repeats", "too full"])
def test_map_by_buckets(program, what, n, shift):
    r = subprocess.run([program, what, str(n), str(shift)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout)
