// How a launch's tiles are spread over the chip's eight XCDs (internal; host rules, no device
// code).
#pragma once
#include <cstddef>

namespace wf {

constexpr int kXcds = 8;
constexpr size_t kXcdRowBytes = (size_t)5 << 19;  // operand bytes one XCD's blocks share at most (L2: 4 MB)

// nmb x nnb tiles: XCD x takes row part x % rs of rs and column part x / rs of 8 / rs, row
// blocks fastest.  Blocks of the fullest XCD (the one with part 0 of both):
inline int xcd_most_blocks(int nmb, int nnb, int rs) { return ((nmb + rs - 1) / rs) * ((nnb * rs + kXcds - 1) / kXcds); }
// and the launch's, those past the tiles of a smaller part among them.
inline unsigned xcd_blocks(int nmb, int nnb, int rs) { return (unsigned)kXcds * xcd_most_blocks(nmb, nnb, rs); }

// Row parts so that the operand rows of one XCD's blocks (block_bytes per row block) stay in
// its L2 while the weights pass by: 1776 two-plane rows, K = 1280, 5120 columns 90 us with all
// rows per XCD, 65, 60 and 68 with half, a quarter and an eighth; 864 rows 37, 33, 34 and 35.
// Not where the parts come out so uneven that the fullest XCD gets over an eighth more
// blocks: K = 6400, 20 column blocks, 9 row blocks 35 us in 2 parts, 62 in 8 (two to each of
// four XCDs, one, and three XCDs idle), 14 row blocks 53 in 2, 58 in 4, 59 in 8; K = 2560, 26
// row blocks 60 in 2, 56 in 4, 61 in 8.
inline int xcd_row_parts(int nmb, int nnb, size_t block_bytes) {
  int rs = 1;
  while (rs < kXcds && (size_t)((nmb + rs - 1) / rs) * block_bytes > kXcdRowBytes &&
         8 * xcd_most_blocks(nmb, nnb, 2 * rs) <= 9 * xcd_most_blocks(nmb, nnb, rs))
    rs *= 2;
  return rs;
}

}  // namespace wf
