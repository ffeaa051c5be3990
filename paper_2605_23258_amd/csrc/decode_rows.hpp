// Index arithmetic of the decode kernels that needs no device: constexpr, so that it runs on the host as well.
#pragma once

namespace vec {

// Paged retained segments: which entry of its (sequence, head)'s block table a lane keeps for the rows row_begin ..
// row_end - 1 of a workgroup (row_begin < row_end): entry (row_begin >> block_shift) + lane, the last one of the range in the
// lanes beyond.  cap: rows the table has blocks for, at least 1.  A step's own token is row cap where the block
// is full; it has no entry (its row comes from the caller's buffers), so the range ends with the capacity for this.
constexpr int block_entry(int row_begin, int row_end, int cap, int block_shift, int lane) {
  const int last = ((row_end < cap ? row_end : cap) - 1) >> block_shift, mine = (row_begin >> block_shift) + lane;
  return mine < last ? mine : last;
}

}  // namespace vec
