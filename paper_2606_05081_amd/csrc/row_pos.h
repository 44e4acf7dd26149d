// Positions in the column array of a CSR, host and device.
//
// A graph may have up to 2^31 - 1 arcs, and a wave that walks a row forms
// positions past the row's end before it compares them with it: by its lanes,
// the columns it loads ahead and its last step, kRowAhead in all at most. In
// signed 32 bits those of the last rows of such a graph wrap to negative
// numbers, which are below the end; in unsigned 32 bits none wraps (nor does a
// position plus the length of a part of a row, which is below 2^28).
#pragma once

#include <cstdint>

namespace blest {

using row_pos = uint32_t;
constexpr uint32_t kMaxArcs = 0x7fffffffu;
constexpr uint32_t kRowAhead = 2048;
static_assert(kMaxArcs + kRowAhead > kMaxArcs, "positions past the last row do not wrap");

// Whether the column `ahead` past p lies in a row that ends at `end`.
constexpr bool row_has(row_pos p, uint32_t ahead, row_pos end) { return p + ahead < end; }

// The end of the part of at most len columns that starts at p.
constexpr row_pos row_part_end(row_pos p, uint32_t len, row_pos end) { return p + len < end ? p + len : end; }

// Piece `i` of a row cut into `pieces` of whole steps of 64 columns: its first
// column, possibly past the end, and its length before the end cuts it.
constexpr uint32_t row_piece_len(row_pos p, row_pos end, uint32_t pieces) {
  return ((end - p + pieces - 1) / pieces + 63u) & ~63u;
}

}  // namespace blest
