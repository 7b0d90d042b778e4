// Which order the second launch of a row-wise kernel on long rows takes (rowwise_kernel.h has the two launches).  Host arithmetic only.
#pragma once

#include <stdint.h>

#include <numeric>

namespace swz {

// Layer normalisation also reads gamma and beta, 4 N bytes a row.  In dispatch order chunk c of every row is on XCD c mod X where X divides the chunks, and an XCD needs 4 N / X of
// those bytes for all rows, which its L2 keeps up to N = 2^23 (at 2^24 the two orders are level, 64 rows 1860 us, 1873); with a row's chunks back to back on one XCD all of them cross the
// fabric again for every row once they outgrow the 4 MB.  64 x 1048576 95 us with the rows of an XCD together, 67 in dispatch order (60 x 1000000 77, 66; 128 x 524288 69, 66;
// 16 x 131072 8.2, 7.9); where X does not divide the chunks and gamma and beta fit, 100 x 600000 (37 chunks) 63 and 65, 90 x 700008 (43) 67 and 69: the caller's mode.
// Each chunk of every row on X / gcd(chunks, X) XCDs: where that is all of them nothing is saved (64 rows of 790000, 800000 and 900000 elements, 49 and 55 chunks, 56.5, 57.0 and 67.0 us
// in the caller's order, 58.2, 58.8 and 68.6 in dispatch order; but 52, 58 and 62 chunks, 850000, 950000 and 1000000 elements, 61.3, 74.4, 82.4 and 58.9, 66.4, 69.7).
// Chunks that end inside a 128-byte line: the two parts of the line are then written on two XCDs.  As long as the matrix is small the reuse is worth more (16 and 64 rows of 114696 elements
// 9.5 and 13.1 us, 9.3 and 12.6; 64 x 393208 32.4, 31.0), from 2^25 elements on it is not unless gamma and beta exceed 3 MiB (256 x 250000 65.5, 67.7; 256 x 390000 97.3, 101.7;
// 1024 x 114696 110.7, 118.4; 1024 x 130000 129.7, 134.9).
// named: the caller named group_m or num_xcd, and gets the mapping that the mode and these say.
inline bool emit_in_dispatch_order(int64_t M, int64_t N, int chunks, int num_xcd, bool named) {
  if (named || std::gcd(chunks, num_xcd) == 1) return false;
  if (N * 4 > ((int64_t)3 << 20)) return true;
  return chunks % num_xcd == 0 && (N % ((int64_t)64 * chunks) == 0 || M * N < ((int64_t)1 << 25));
}

}  // namespace swz
