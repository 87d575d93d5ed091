// The row chunks of the block process's passes over the basis (host side; a CPU
// test includes it too).
#pragma once

#include <algorithm>

// The block process's dot pass: rows per wavefront, and its row chunks of four
// wavefronts.  By N alone (never by the slots, so that a source's sums are the
// same alone and in a batch): 128 rows, so that the partial sums stay at 3 per
// cent of the basis, and 64 on lattices whose chunks of 512 rows are too few to
// fill the chip; at most 128 chunks.  Whole lines of 128 bytes (8 rows), and no
// coarser, so that 128 chunks of a large lattice stay 128, the same number on
// every XCD: 12^4 x 4, s = 4, 240 columns, chunks of 1952 / 2048 rows (128 and
// 122 of them): 51.5 / 53.4 ms of dot passes.  132000 rows x 4, s = 8, chunks of
// 1056 / 1040 rows (no whole lines): 15.9 / 16.9 ms.
constexpr int kSmallRows = 12288;  // below: the shorter chunks
inline int row_chunks(int N, int& rpw) {
  const int want = (N + 4 * 128 - 1) / (4 * 128);
  rpw = std::max(N < kSmallRows ? 64 : 128, (want + 7) & ~7);
  return (N + 4 * rpw - 1) / (4 * rpw);
}
// rows of a chunk of the update pass, whose workgroups take 16 to 128 of them
inline int update_chunk(int rpw) { return (4 * rpw + 127) & ~127; }
