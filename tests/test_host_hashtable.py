"""The insert of the de-duplication's hash table, compiled for the host: its probe sequence on tables that are nearly full, full,
and full of other IDs (a device-side insert that found no end would hold the GPU)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_00837_amd", "csrc")
HIP_FOR_THE_HOST = """
#pragma once
#define __device__
#define __forceinline__ inline
struct Index { unsigned x; };
static Index blockIdx{0}, threadIdx{0}, blockDim{1}, gridDim{1};
static inline unsigned long long atomicCAS(unsigned long long* p, unsigned long long want, unsigned long long v) {
    const unsigned long long was = *p;
    if (was == want) *p = v;
    return was;
}
static inline unsigned long long atomicMin(unsigned long long* p, unsigned long long v) {
    const unsigned long long was = *p;
    if (v < was) *p = v;
    return was;
}
"""
PROGRAM = """
#include "hashtable.hpp"
#include <cstdio>
#include <vector>
using namespace helios;
int main() {
    for (uint32_t slots : {1u, 8u, 1024u}) {
        std::vector<unsigned long long> t(slots, kEmptySlot);
        std::vector<bool> taken(slots, false);
        uint32_t claims = 0;
        for (uint32_t k = 0; k < slots; ++k) {                 // fills up: every ID gets a slot of its own
            const uint32_t s = table_insert(t.data(), slots - 1, 1000 + 7 * k, 2 * k + 5, claims);
            if (s >= slots || taken[s] || claims != k + 1) return 1;
            taken[s] = true;
        }
        for (uint32_t k = 0; k < slots; ++k) {                 // IDs that are there: the same slot, the smaller position
            const uint32_t a = table_insert(t.data(), slots - 1, 1000 + 7 * k, 2 * k + 9, claims);
            if (t[a] != ((1000ull + 7 * k) << 32 | (2 * k + 5))) return 2;
            if (table_insert(t.data(), slots - 1, 1000 + 7 * k, 2 * k + 1, claims) != a) return 3;
            if (t[a] != ((1000ull + 7 * k) << 32 | (2 * k + 1))) return 4;
        }
        const std::vector<unsigned long long> before = t;
        for (uint32_t k = 0; k < 64; ++k)                      // no room and not there: ends, and changes nothing
            if (table_insert(t.data(), slots - 1, 5 + k, 0, claims) < slots) return 5;
        if (t != before || claims != slots) return 6;
    }
    std::puts("ok");
    return 0;
}
"""


def test_insert_ends_on_a_full_table(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_FOR_THE_HOST)
    (tmp_path / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", str(tmp_path), "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")],
                   check=True, timeout=100)
    r = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True, timeout=10)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout)
