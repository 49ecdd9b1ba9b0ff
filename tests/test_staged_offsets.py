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
static int check(uint64_t groups, uint64_t list, uint32_t taken) {
    const uint32_t cap = (uint32_t)(list < STG_NOWHERE ? list : STG_NOWHERE);
    const uint64_t first = staged_first(groups);
    // at most 2 KB per tile below, an entry per pixel of 8x8 tiles above the line
    if (first != (groups <= STG_MANY ? 256u : 64u)) return 1;
    if (staged_room(groups, 64 * groups) > (groups <= STG_MANY ? 320 : 64) * groups + STG_CHUNK) return 1;
    const uint64_t probes[] = {0, groups / 3, groups / 2, groups - 1};
    uint64_t end = 0;  // behind the entries in use by earlier chunks
    for (const uint64_t g : probes) {
        uint32_t base = staged_first_base((uint32_t)g, (uint32_t)first);
        if (base != g * first) return 2;
        for (uint32_t left = (uint32_t)first, m = 50; left >= m; left -= m) {  // batches of it
            const uint32_t off = staged_offset(base, m, cap);
            if (off != STG_NOWHERE && (off != base || (uint64_t)off + m > list)) return 3;
            if (off == STG_NOWHERE && base != STG_NOWHERE && (uint64_t)base + m <= cap) return 4;
            if (off != STG_NOWHERE) end = (uint64_t)off + m;
            base = staged_next(off, m);
        }
    }
    for (uint32_t k = 0; k < 5; ++k) {  // chunks of the counter, which starts behind the first ones
        const uint32_t unit = staged_first_units(groups) + taken + k;
        const uint64_t want = (uint64_t)unit * STG_CHUNK;
        const uint32_t off = staged_offset(staged_base(unit), STG_CHUNK, cap);
        if (off != STG_NOWHERE && (off != want || off < end || want < groups * first || want + STG_CHUNK > list)) return 5;
        if (off == STG_NOWHERE && want + STG_CHUNK <= cap && want + STG_CHUNK < STG_NOWHERE) return 6;
        if (off != STG_NOWHERE) end = want + STG_CHUNK;
    }
    return 0;
}

int main() {
    const uint64_t groups[] = {1, 2, 3, 131072, 524287, 524288, 524289, (1u << 24) - 1, 1u << 24, (1u << 24) + 1, 20971520, 67108864};
    const uint64_t lists[] = {0, 255, 256, 4096, 1u << 25, 0x7fffffffull, 0xfffffffeull, 0xffffffffull, 0x100000000ull,
                              0x200000000ull};
    const uint32_t taken[] = {0, 1, 0x7ffff0u, 0x7ffffdu, 0x7fffffu, 0x800000u, 0x12345678u, 0xf0000000u};
    for (const uint64_t g : groups)
        for (const uint64_t c : lists)
            for (const uint32_t n : taken)
                if (const int e = check(g, c, n)) {
                    std::printf("rule %d at %llu workgroups, room for %llu, %u chunks taken\n", e,
                                (unsigned long long)g, (unsigned long long)c, n);
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
