// Stream compaction by keep bits: a first kernel writes one bit per row and the
// number of kept rows per block, a second one writes the kept rows out (see
// filter.hip and semijoin.hip).
#pragma once
#include "tqp_internal.hpp"

namespace tqp {

constexpr int kFilterNT = 256;
constexpr int kFilterIPT = 8;                            // rows per thread and step: a byte of keep bits
constexpr int kFilterTile = kFilterNT * kFilterIPT;      // rows per workgroup and step
constexpr int kFilterMaxSteps = 8;                       // steps (tiles) per block

// keep[row / 8] bit row % 8, and bcnt[block] kept rows; a block is `steps` tiles, and
// every byte of it is there (rows past n have their bits clear).
struct KeepLayout {
    int steps;
    int64_t nblocks;
    uint8_t *keep;
    int32_t *bcnt;
    size_t bytes;
};
KeepLayout keep_layout(void *ws, int64_t n);

// The keep bits of 8 * steps rows as one word.
__device__ __forceinline__ uint64_t keep_word(const uint8_t *keep, int64_t unit, int steps) {
    if (steps == 8) return reinterpret_cast<const uint64_t *>(keep)[unit];
    if (steps == 4) return reinterpret_cast<const uint32_t *>(keep)[unit];
    if (steps == 2) return reinterpret_cast<const uint16_t *>(keep)[unit];
    return keep[unit];
}

}  // namespace tqp
