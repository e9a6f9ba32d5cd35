// Which rows of an operand a load of the direct-to-LDS products names: plain arithmetic, shared by the kernels of gemm.hip and
// the CPU tests (include/areal_host.h).
//
// A load moves a group of 8 tile rows, 128 bytes of each, by a buffer load: base + lane offset + scalar offset.  Whether the
// resource's range is held against the lane offset alone or also against the scalar one, and what it is held against where
// the scalar offset alone exceeds the range, is not relied on: the scalar offset is the K slab's, which stays inside a row;
// where the group begins is part of the base, and the range ends with the operand's last row.  So a lane passes the check
// exactly if its row exists.  Groups wholly outside name the last row, which exists: no range is empty.
#pragma once
#include <stdint.h>

#if defined(__HIP__)
#define AREAL_HD __attribute__((host)) __attribute__((device)) __attribute__((always_inline)) inline
#else
#define AREAL_HD inline
#endif

namespace areal {

struct RowRange { uint32_t first, bytes; };       // byte offset of the resource's base, and its size
// The group that begins at row `row` of an operand of `bytes` > 0 bytes of rows, up to the operand's end.
AREAL_HD RowRange row_range(int row, uint32_t row_bytes, uint32_t bytes) {
  const uint32_t at = (uint32_t)row * row_bytes, last = bytes - row_bytes, first = at < last ? at : last;
  return {first, bytes - first};
}
// Row of the group that a lane moves a chunk of.  `spread`: the group's halves lie four rows apart.
AREAL_HD int group_row(int lane, bool spread) {
  const int r = lane >> 3;
  return spread ? 8 * (r >> 2) + (r & 3) : r;
}
// Byte offset of a lane's chunk (chunks of 16 bytes, swizzled by the lane's place in the group) from the group's first row.
AREAL_HD int group_lane_offset(int lane, bool spread, int row_bytes) {
  return group_row(lane, spread) * row_bytes + ((lane & 7) ^ (lane >> 3)) * 16;
}
// The same from the operand's first row, for a group that begins at row `row`: rows behind the last name the last.
AREAL_HD int tile_lane_offset(int lane, int row, int rows, int row_bytes) {
  const int r = row + (lane >> 3);
  return (r < rows ? r : rows - 1) * row_bytes + ((lane & 7) ^ (lane >> 3)) * 16;
}

}  // namespace areal
