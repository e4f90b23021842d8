// Which rows of a table (or of a part of one) the semi-join's mask kernel loads.
// Plain arithmetic without device code, so that a host program can walk it.
#pragma once
#include <stdint.h>

namespace tqp {

constexpr int kSjIPT = 8;                        // rows per lane and chunk
constexpr int kSjChunk = 64 * kSjIPT;            // rows per wave and chunk
constexpr int64_t kSjPartRows = int64_t(1) << 25;       // rows per part of tqp_semijoin_noalloc

// The rows of the part that begins at row0 of a table of n, taken `most` at a time.
constexpr int64_t sj_part_rows(int64_t n, int64_t row0, int64_t most) { return n - row0 < most ? n - row0 : most; }

// Whether a part of `rows` rows, its key columns 16-byte aligned or not, takes the form
// that loads whole chunks.  It has to hold one: see sj_chunk_row.
constexpr bool sj_whole_chunks(bool aligned, int64_t rows) { return aligned && rows >= kSjChunk; }

// That form's loads for the chunk at row0 of n rows begin at this row: the first chunk
// stands in for one that is not whole (its keys are loaded again one by one).  All of
// them are inside the table only if n >= kSjChunk, or the first chunk is not whole
// either.
constexpr int64_t sj_chunk_row(int64_t row0, int64_t n) { return row0 + kSjChunk > n ? 0 : row0; }

// Lane's load k of V keys begins this many keys later.
template <int V> constexpr uint32_t sj_lane_key(uint32_t lane, int k) { return (lane * (kSjIPT / V) + k) * V; }

// The other form: row r of a lane of the chunk at row0 < n, the last row standing in
// for those past the end.
constexpr int64_t sj_any_row(int64_t row0, int64_t n, uint32_t lane, int r) {
    const uint32_t left = uint32_t(n - 1 - row0 < kSjChunk ? n - 1 - row0 : kSjChunk - 1);
    const uint32_t i = lane * kSjIPT + r;
    return i < left ? i : left;
}

}  // namespace tqp
