// Where the forward compositing puts the entries it staged, for the backward
// to read again: offsets into one list that all workgroups share.
#pragma once

#include <cstdint>

namespace mgs {

// A workgroup's first chunk is its own by its index, further ones come from a
// global counter (with every workgroup of a launch at that counter at its
// start, forward compositing waits).
constexpr uint32_t STG_FIRST = 256;
constexpr uint32_t STG_CHUNK = 512;
// First chunks take 2 KB per tile whether or not the tile has entries; beyond
// this many entries for all of them (256 MB), every chunk comes from the
// counter.
constexpr uint64_t STG_FIRST_MAX = 1ull << 25;
constexpr uint32_t STG_NOWHERE = 0xffffffffu;

// Entries of each workgroup's first chunk in a launch of so many workgroups.
constexpr uint32_t staged_first(uint64_t workgroups) {
    return workgroups <= STG_FIRST_MAX / STG_FIRST ? STG_FIRST : 0u;
}

// The 32-bit offset of m entries from `base` on in a list of `cap` entries, or
// STG_NOWHERE if they do not fit (the backward then forms the batch again).
// The base is 64-bit: neither a workgroup's index times its chunk nor the
// counter may wrap into entries of another workgroup.
constexpr uint32_t staged_offset(uint64_t base, uint32_t m, uint64_t cap) {
    return base + m <= cap && base + m <= STG_NOWHERE ? (uint32_t)base : STG_NOWHERE;
}

}  // namespace mgs
