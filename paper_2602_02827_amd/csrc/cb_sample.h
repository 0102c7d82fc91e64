// Where the quantiser's sample of a long segment is taken.  Plain C++ (constexpr functions are
// usable on both sides).
#pragma once
#include <stdint.h>

namespace cb {

// Piece of 16 bytes that sample i takes: one of the i-th run of `step` pieces, at a place mixed from i.
// At the start of every run a step that shares a factor with the pieces of a row (any multiple of 4
// at d = 128) would see the same few columns of every row, and an encoder's columns differ in
// scale: 1,000,000 rows of 128 with scales from 1 to 0.01 took 485 us, because the bound missed, and take 181.
constexpr int64_t sample_piece(uint32_t i, int64_t step) {
    uint32_t h = i * 0x9E3779B1u;
    h = (h ^ (h >> 15)) * 0x85EBCA77u;
    h ^= h >> 13;
    return (int64_t)i * step + (int64_t)(((uint64_t)h * (uint64_t)step) >> 32);
}

}  // namespace cb
