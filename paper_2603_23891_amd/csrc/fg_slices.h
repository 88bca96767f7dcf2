// Places in the bounded list of emission slices (fg_sort.hip), told apart from
// the kernel so that the rule can also be run on the host.
//
// The list's counter only grows: a block adds the number of slices that it wants
// and never takes any back, so the ranges that blocks get are disjoint in every
// order of their additions. A block whose whole range lies below the capacity
// lists its slices there. Any other block emits all of its pairs itself, and
// where its range begins below the capacity it writes empty entries there, so
// that every entry below min(counter, capacity) is written by its owner. (A
// refused block that subtracted its request again would let a block in between
// take places past the counter's final value and leave others unwritten.)
#pragma once

#include <cstdint>

namespace fgs {

struct Claim {
    bool listed;           // the block's slices go to entries [first, last); else they become empty
    uint64_t first, last;
};

// at: the counter before the block added `more` to it.
constexpr Claim claim(uint64_t at, uint64_t more, uint64_t cap)
{
    const bool listed = at <= cap && more <= cap - at;
    const uint64_t first = at < cap ? at : cap;
    return Claim{listed, first, listed ? at + more : cap};
}

// Entries to read once every block has made its claim.
constexpr uint64_t entries(uint64_t counter, uint64_t cap) { return counter < cap ? counter : cap; }

}  // namespace fgs
