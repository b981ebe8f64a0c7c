// Addresses of the LM-head tile kernel's loads: plain constant-expression C++, shared by the kernel
// and by the host test that walks every load of every tile height.
#pragma once

#include <cstdint>

namespace eb {

// An operand tile (up to 256 rows of W or of h, `rows` of them inside the operand) reaches LDS by
// load instructions of 8 rows x 128 bytes.  Instruction q covers rows 8 q .. 8 q + 7; lane L reads
// one 16-byte chunk of row 8 q + L / 8.  Its address is
//   resource base + vector offset + scalar offset,
// where the resource starts at row tile_load_row0(q, rows) of the tile and ends with the operand's
// last row, the vector offset holds the lane's row within the 16-row group and its chunk, and the
// scalar offset holds the stage's columns only.  The bounds check is thus right whether the scalar
// offset counts in it (then it is compared with the range less that offset, which stays positive,
// as the offset is less than a row) or not (then a lane past the operand's last row is out of range
// by its vector offset alone).  Loads out of range return zeros.

// First row of the resource of instruction q: the 16-row group of its rows, or for a group that
// lies past the operand the last one that does not (those rows' logits are used by nobody).
constexpr int tile_load_row0(int q, int rows) {
  const int group = (q & ~1) * 8, last = (rows - 1) & ~15;
  return group < last ? group : last;
}

// Range in bytes of that resource.
constexpr uint32_t tile_load_range(int row0, int rows, uint32_t row_bytes) {
  return static_cast<uint32_t>(rows - row0) * row_bytes;
}

// 16-byte chunk c of row r sits at place c ^ tile_swizzle(r) of the LDS row of eight places.  LDS
// has 16 places of 16 bytes across its banks and serves 32 lanes of a fragment read in two parts
// (lanes 0-3, 12-15 and 20-27, then the others): with this order every read is a 2-way conflict
// (SQ_LDS_BANK_CONFLICT 6.5e8 in a launch with 1.6e8 reads of 4 cycles each).  It hides behind the
// MFMAs.  With row bit 1 in the place of bit 0 no read has a conflict (1.4e6 counted), and 1024
// positions of a 126464 x 4096 head take 768 us both ways, 9626 of 152064 x 3584 7323 and 7340 us,
// 512 of 126464 x 2048 218 and 222 us.
constexpr int tile_swizzle(int r) { return ((r >> 2) & 3) | ((r & 1) << 2); }

// Vector offset of lane `lane` of the instructions of parity q & 1.
constexpr uint32_t tile_load_voff(int parity, int lane, uint32_t row_bytes) {
  const int row = 8 * parity + (lane >> 3);
  return static_cast<uint32_t>(row) * row_bytes +
         16u * static_cast<uint32_t>((lane & 7) ^ tile_swizzle(row));
}

}  // namespace eb
