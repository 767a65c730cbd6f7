// How a launch's tiles are spread over the chip's eight XCDs, and which tile a request-time
// product takes (internal; host rules, no device code).
#pragma once
#include <cstddef>

namespace wf {

constexpr int kXcds = 8;
constexpr int kXcdCus = 32;  // compute units of one XCD
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

// Request-time products: the split with the fewest rounds of blocks per XCD (32 CUs of `occ`
// blocks), then the one whose blocks share the fewest rows and columns: 6144 rows, K = 5120,
// N = 1280 on 256 x 128 tiles 148, 137 and 76 us with 1, 2 and 4 row parts (48, 36 and 30
// blocks per XCD).
struct XcdSplit {
  int nmb, nnb, rs;
  long long rounds;
};
inline XcdSplit xcd_split(int rows, int cols, int bm, int bn, int occ, int batch) {
  XcdSplit best{(rows + bm - 1) / bm, (cols + bn - 1) / bn, 1, 0};
  long long least = 0;
  for (int rs = 1; rs <= kXcds; rs *= 2) {
    const long long nrh = (best.nmb + rs - 1) / rs, ncq = (best.nnb * rs + kXcds - 1) / kXcds;
    const long long rounds = (nrh * ncq * batch + kXcdCus * occ - 1) / (kXcdCus * occ), share = nrh * bm + ncq * bn;
    if (rs == 1 || rounds < best.rounds || (rounds == best.rounds && share < least)) {
      best.rounds = rounds;
      best.rs = rs;
      least = share;
    }
  }
  return best;
}

// The tile with the least time: rounds of blocks times what a round of 1280 columns of
// k takes (256 x 128 tiles, one block per CU, 27 us; 128 x 128 in two stages, two per
// CU, 29; 64 x 128 in four stages, one per CU, 12).  1500 rows: 5120 columns 27, 29
// and 54 us, 3840 columns 21, 27 and 37, 1280 columns 22, 21 and 10.  For short rows
// and half-filled rounds the three lie closer than that: over the request-time products of
// widths 512, 768 and 1280 for one to four requests the tile taken is the fastest of the
// three or within 10% of it in five of six, and 31% behind at most (1500 rows, 1024
// columns, K = 512, two matrices 15.5 us, 11.9 on 256 x 128 tiles).
struct MmTile {
  int rows;  // 256, 128 or 64
  XcdSplit split;
};
inline MmTile mm_tile(int rows, int cols, int bn, int batch) {
  const XcdSplit w = xcd_split(rows, cols, 256, bn, 1, batch), m = xcd_split(rows, cols, 128, bn, 2, batch),
                 n = xcd_split(rows, cols, 64, bn, 1, batch);
  const long long tw = 27 * w.rounds, tm = 29 * m.rounds, tn = 12 * n.rounds;
  return tw <= tm && tw <= tn ? MmTile{256, w} : tm <= tn ? MmTile{128, m} : MmTile{64, n};
}

}  // namespace wf
