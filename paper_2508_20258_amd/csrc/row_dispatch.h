// Which order the second launch of a row-wise kernel on long rows takes (rowwise_kernel.h has the two launches).  Host arithmetic only.
#pragma once

#include <stdint.h>

namespace swz {

// Layer normalisation also reads gamma and beta, 4 N bytes a row.  In dispatch order chunk c of every row is on XCD c mod X where X divides the chunks, and an XCD needs 4 N / X of
// those bytes for all rows, which its L2 keeps up to N = 2^23 (at 2^24 the two orders are level, 64 rows 1860 us, 1873); with a row's chunks back to back on one XCD all of them cross the
// fabric again for every row once they outgrow the 4 MB.  64 x 1048576 95 us with the rows of an XCD together, 67 in dispatch order (60 x 1000000 77, 66; 128 x 524288 69, 66;
// 16 x 131072 8.2, 7.9); where X does not divide the chunks and gamma and beta fit, 100 x 600000 (37 chunks) 63 and 65, 90 x 700008 (43) 67 and 69: the caller's mode.
// named: the caller named group_m or num_xcd, and gets the mapping that the mode and these say.
inline bool emit_in_dispatch_order(int64_t N, int chunks, int num_xcd, bool named) {
  return !named && (chunks % num_xcd == 0 || N * 4 > ((int64_t)3 << 20));
}

}  // namespace swz
