// Segments of a long list: the arithmetic that the pre-filter kernels and the kernels that read
// their output share.  Plain C++ (constexpr functions are usable on both sides).  A list holds at most
// 2^31 - 2^17 entries and a segment up to 2^25, so a segment's nominal end can lie past the
// largest int: ends and counts are formed by subtraction.
#pragma once

namespace cb {

// Tile of the pre-filter kernels: eight entries per thread of 1,024, so that two workgroups share a CU.
constexpr int SEG_TILE = 8192;
constexpr int SEG_MAX = 64;                        // segments of a long list

// entries per segment of a list of count >= 1: whole tiles, so that a segment's bound comes from a
// full tile whenever there is one
constexpr int seg_len(int count) {
    const int tiles = (count - 1) / SEG_TILE + 1;
    return ((tiles - 1) / SEG_MAX + 1) * SEG_TILE;
}
constexpr int seg_count(int count) { return (count - 1) / seg_len(count) + 1; }
// end of the segment that begins at lo < count
constexpr int seg_end(int lo, int len, int count) { return count - lo > len ? lo + len : count; }

}  // namespace cb
