// Where the forward compositing puts the entries it staged, for the backward
// to read again: offsets into one list that all workgroups share.
#pragma once

#include <cstdint>

namespace mgs {

// A workgroup's first chunk is its own by its index, further ones come from a
// global counter, where forward compositing waits: with every workgroup of a
// launch there at its start, and later at 6.5 ns for each of them.
constexpr uint32_t STG_FIRST = 256;
constexpr uint32_t STG_CHUNK = 512;
// First chunks take their room (8 bytes an entry) whether or not the tile has
// entries: 2 KB per tile, and in launches of more than STG_MANY workgroups (1
// GB) 512 bytes, which is an entry per pixel of the smallest tiles.  16 views
// of 1920x1080 in 8x8 tiles (518,400), forward with first chunks of 256, 64 and
// no entries: 256 splats 584, 582 and 1,705 us, 4096 splats 641, 637 and 3,381
// us, 20,000 splats, whose lists are longer than 64, 1,065, 1,684 and 3,631 us.
constexpr uint64_t STG_MANY = 524288;
constexpr uint32_t STG_FIRST_MANY = 64;
constexpr uint32_t STG_NOWHERE = 0xffffffffu;

// Entries of each workgroup's first chunk in a launch of so many workgroups.
constexpr uint32_t staged_first(uint64_t workgroups) {
    return workgroups <= STG_MANY ? STG_FIRST : STG_FIRST_MANY;
}

// The list in units of STG_CHUNK, in which the counter runs, that the first
// chunks take.
constexpr uint32_t staged_first_units(uint64_t workgroups) {
    return (uint32_t)((workgroups * staged_first(workgroups) + STG_CHUNK - 1) / STG_CHUNK);
}

// Entries of the list for a first forward over so many tiles and pixels: the
// first chunks, and an entry per pixel, beside them or, with many tiles, among
// them.
constexpr uint64_t staged_room(uint64_t tiles, uint64_t pixels) {
    const uint64_t first = (uint64_t)staged_first_units(tiles) * STG_CHUNK;
    return tiles <= STG_MANY ? pixels + first : (pixels > first ? pixels : first);
}

// The first entry of a workgroup's first chunk.  (At most 16 views of 2,048 x
// 2,048 tiles: below 2^32.)
constexpr uint32_t staged_first_base(uint32_t workgroup, uint32_t first) { return workgroup * first; }

// The first entry of the counter's chunk `unit`, or STG_NOWHERE: a product of
// 2^32 or more must not wrap into entries of another workgroup.
constexpr uint32_t staged_base(uint32_t unit) {
    return unit < STG_NOWHERE / STG_CHUNK ? unit * STG_CHUNK : STG_NOWHERE;
}

// The offset of the next m entries of a chunk with `base` next in a list of
// `cap` entries, or STG_NOWHERE if they have no place (the backward then forms
// the batch again).
constexpr uint32_t staged_offset(uint32_t base, uint32_t m, uint32_t cap) {
    return m <= cap && base <= cap - m ? base : STG_NOWHERE;
}
// ... and the entry after them.
constexpr uint32_t staged_next(uint32_t offset, uint32_t m) {
    return offset == STG_NOWHERE ? STG_NOWHERE : offset + m;
}

}  // namespace mgs
