"""The hotness order compiled for the host, where the workgroups of a launch run one after the other: the first one is alone with the jobs
of a pass after the first, and has to end (a launch may find room for few of its workgroups)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2310_00837_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
PROGRAM = r"""
#include <hip/hip_runtime.h>
#undef __builtin_amdgcn_readfirstlane
#define __builtin_amdgcn_readfirstlane(v) on_host_readlane(v, 0)
#include "sort.hip"
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

uint32_t next_random() {
    static uint64_t x = 88172645463325252ull;
    x ^= x << 13, x ^= x >> 7, x ^= x << 17;
    return static_cast<uint32_t>(x >> 16);
}

int main(int argc, char** argv) {
    const int64_t n = std::stol(argv[1]);
    const uint32_t below = static_cast<uint32_t>(std::stoul(argv[2]));
    const bool in_place = std::string(argv[3]) == "in place";
    const size_t bytes = hotness_order_scratch_bytes(n);
    unsigned char* scratch = guarded<unsigned char>((bytes + 255) / 256 * 256);
    int32_t *counts = guarded<int32_t>(n), *order = in_place ? counts : guarded<int32_t>(n), *err = guarded<int32_t>(2);
    for (int call = 0; call < 2; ++call) {               // (the second finds the scratch as the first has left it)
        err[0] = 0;
        std::vector<int32_t> count(n), want(n);
        for (int64_t v = 0; v < n; ++v) {
            count[v] = static_cast<int32_t>(next_random() % 3 ? next_random() % 5 : next_random() % below);
            counts[v] = count[v];
            want[v] = static_cast<int32_t>(v);
        }
        std::stable_sort(want.begin(), want.end(), [&](int32_t a, int32_t b) { return count[a] > count[b]; });
        if (launch_hotness_order(nullptr, counts, n, order, scratch, err) != hipSuccess) return 2;
        if (err[0] != 0 || memcmp(want.data(), order, 4 * n) != 0) {
            printf("wrong: error %d\n", err[0]);
            return 1;
        }
    }
    printf("ok\n");
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("sort")
    (d / "main.cpp").write_text(PROGRAM)
    with open(os.path.join(CSRC, "hotness.hip")) as f:
        (d / "sort.hip").write_text(f.read().replace('asm("" : "+v"(mine));', ""))       # (a hint to the optimiser, in a form the header has no word for)
    subprocess.run([CLANG, "-std=c++17", "-O0", "-w", "-U_FORTIFY_SOURCE", "-I", os.path.join(HERE, "hip_on_the_host"), "-I", CSRC,
                    str(d / "main.cpp"), "-o", str(d / "main")], check=True, timeout=100)
    return str(d / "main")


@pytest.mark.parametrize("where", ["apart", "in place"])
@pytest.mark.parametrize("n,below", [(1, 2**31 - 1), (8_193, 100_000), (80_000, 2**31 - 1), (140_001, 5_000_000), (20_000, 2_000)])
def test_hotness_order(program, n, below, where):
    r = subprocess.run([program, str(n), str(below), where], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout)
