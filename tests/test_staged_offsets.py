"""Offsets into the list of staged entries, on the host: the rule of
csrc/staged.hpp at numbers of tiles around those where a 32-bit product or
counter would wrap.  No two chunks may meet, and an entry that has no 32-bit
place below the list's size goes nowhere."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "staged.hpp"
using namespace mgs;

// A workgroup's chunks as the forward compositing takes them: the first by the
// index, then one of the counter for every batch that does not fit.
static int check(uint64_t groups, uint64_t cap, uint64_t counter) {
    const uint64_t first = staged_first(groups);
    // at most 2 KB per tile below, an entry per pixel of 8x8 tiles above the line
    if (first == 0 || first > (groups <= STG_MANY ? 256u : 64u) || staged_room(groups, 64 * groups) > 256 * groups + 64 * groups)
        return 1;
    if (groups > STG_MANY && staged_room(groups, 64 * groups) > 64 * groups) return 1;
    const uint64_t probes[] = {0, groups / 3, groups / 2, groups - 1};
    uint64_t end = 0;  // the highest entry in use by an earlier chunk
    for (const uint64_t g : probes) {
        const uint64_t base = g * first;
        const uint32_t off = staged_offset(base, (uint32_t)first, cap);
        if (off != STG_NOWHERE && (off != base || off + first > cap)) return 2;
        if (off == STG_NOWHERE && base + first <= cap && base + first <= STG_NOWHERE) return 3;
        if (off != STG_NOWHERE && base + first > end) end = base + first;
    }
    for (int k = 0; k < 5; ++k) {  // chunks of the counter, which starts anywhere
        const uint64_t base = groups * first + counter + (uint64_t)k * STG_CHUNK;
        const uint32_t off = staged_offset(base, STG_CHUNK, cap);
        if (off != STG_NOWHERE && (off != base || off < end || (uint64_t)off + STG_CHUNK > cap)) return 4;
        if (off == STG_NOWHERE && base + STG_CHUNK <= cap && base + STG_CHUNK <= STG_NOWHERE) return 5;
        if (off != STG_NOWHERE) end = (uint64_t)off + STG_CHUNK;
    }
    return 0;
}

int main() {
    const uint64_t groups[] = {1, 2, 131072, 524287, 524288, 524289, (1u << 24) - 1, 1u << 24, (1u << 24) + 1, 20971520, 67108864};
    const uint64_t caps[] = {0, 255, 256, 4096, 1u << 25, 0x7fffffffull, 0xfffffffeull, 0xffffffffull, 0x100000000ull,
                             0x200000000ull};
    const uint64_t counters[] = {0, 512, 0xfffff000ull, 0xfffffe00ull, 0x100000000ull, 0x300000200ull};
    for (const uint64_t g : groups)
        for (const uint64_t c : caps)
            for (const uint64_t n : counters)
                if (const int e = check(g, c, n)) {
                    std::printf("rule %d at %llu workgroups, room for %llu, counter at %llu\n", e,
                                (unsigned long long)g, (unsigned long long)c, (unsigned long long)n);
                    return 1;
                }
    return 0;
}
"""


def test_staged_offsets_never_wrap(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "staged.cpp", tmp_path / "staged"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2412_20522_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
