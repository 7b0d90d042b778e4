// How a transpose is launched: which order its tiles are taken in, how many bytes are asked for at a time, which blocks a transpose into part lines takes.
// Host arithmetic only.
#pragma once

#include <stdint.h>

#include "pid_decode.h"

namespace swz {

// A launch has fewer than 2^32 threads: the grid is handed to the device in threads, as a 32-bit number, and a larger one
// comes back as "ok" with only the remainder modulo 2^32 run (2^24 + 1 workgroups of 256: one of them).
constexpr int64_t kLaunchThreads = ((int64_t)1 << 32) - 1;

// Rows and threads of a block of a transpose into part lines (transpose_lines_kernel)
constexpr int lines_rows(int elem_bytes, bool tall) { return !tall ? 64 : elem_bytes == 2 ? 256 : 128; }
constexpr int lines_threads(int rows) { return rows == 64 ? 256 : 512; }

// Rows of n two-byte elements that are 8 KiB, or a power of two of them
inline bool power_of_two_pitch(int64_t n) { return n >= 4096 && (n & (n - 1)) == 0; }

// How many bytes the workgroups of a two-byte transpose have on their way at a time: both loads of a thread or one (paced), and LDS on top of the tile's 8 KB, which
// holds five workgroups to a compute unit instead of eight.  us under the default mode, paced / both / both and five.  Up to 32 MiB latency counts: both, eight (2176 x 2968 7.7 / 7.5;
// 3200 x 1440 6.0 / 5.2), but round robin from 20 MiB on paced (2176 x 2968 8.6 / 9.1).  Above, the HBM serves more
// bytes a second the fewer are asked for, 32 to 40 KB a compute unit: 3712 x 17656 57.6 / 61.9 / 58.4; 20416 x 1912 31.7 / 34.4 / 33.2; 12416 x 2704 26.3 / 29.6 / 28.7.
//   Rows of `out` in whole multiples of 8 KiB: fewer workgroups are better than paced ones, 8192 x 8192 49.2 / 50.8 / 47.1; 16384 x 16384 179.4 / 186.3 / 176.3 (under the bands without
//   the skew not in odd multiples of 16 KiB, 8192 x 8192 49.7 / 51.5 / 52.0, and round robin below 56 MiB, 4096 x 2560 10.8 / 11.7 / 11.3).
//   Rows of `out` in such multiples and of `in` in whole tiles, or of `in` 8 KiB or a power of two of them, under the bands and below 68 MiB: both, eight, 4096 x 4096 15.4 / 13.8 / 14.3; 2048 x 4096 9.3 / 9.0 / 8.5; 4160 x 4096 16.6 / 15.6 / 16.2;
//   4096 x 4160 16.2 / 15.4 / 16.5; 8192 x 2048 15.6 / 14.8 / 15.4; 24576 x 640 14.9 / 14.5 both five, eight; but part tiles 24576 x 672 15.8 both five, 16.3 eight, other rows of `in`
//   320 x 36864 11.4 / 11.8, and above 320 x 57344 15.5 / 16.2; 1600 x 12288 16.5 / 17.2.
// Tiles of 128, whose threads have eight loads each: all together, 1024 x 1024 4.0 us, paced 7.1 (out of the memory-side cache 3.2, 3.8), 8192 x 16384 97.5, 114, but paced without the skew
// where both pitches alias: rows of `out` in multiples of 32 KiB and of `in` in 8, from 256 MiB on, 16384 x 16384 219, 267 together (16384 x 8192 123, 138; 16384 x 4096 62, 64; but
// 16384 x 2048 31.9, 25.7 and 32768 x 2048 60, 56), and without the bands in multiples of 8 and 16 KiB, from 64 MiB on (4096 x 8192 29.7, 34.2; 8192 x 8192 58.9, 61.2; but 8192 x 4096
// 29.5, 25.8).
struct LoadPace { int paced, lds; };
inline LoadPace load_pace(int tile, int64_t M, int64_t N, int mode) {
  if (tile == 128) {
    const bool far = M * 2 % 32768 == 0 && N * 2 % 8192 == 0 && M * N * 4 >= ((int64_t)256 << 20);
    const bool unbanded = (mode & 3) == kModeXcd && M * 2 % 8192 == 0 && N * 2 % 16384 == 0 && M * N * 4 >= ((int64_t)64 << 20);
    return {!swz_mode_skewed(mode) && (far || unbanded) ? 1 : 0, 0};
  }
  const bool banded = swz_mode_grouped(mode), rr = (mode & 3) == kModeRR, out_8k = M * 2 % 8192 == 0;
  const int64_t moved = M * N * 4;
  if (tile != 64 || moved < (int64_t)(rr ? 20 : 32) << 20) return {0, 0};
  if (banded && ((out_8k && N % 64 == 0) || power_of_two_pitch(N)) && moved < ((int64_t)68 << 20)) return {0, 0};
  const bool few = out_8k && !(rr && moved < ((int64_t)56 << 20)) && !(banded && !swz_mode_skewed(mode) && M * 2 % 32768 == 16384);
  return {few ? 0 : 1, few ? 24576 : 0};
}

// Four-byte tiles: all four loads of a thread on their way, and LDS for five workgroups to a compute unit: level with eight up to 64 MiB (1024 x 1024 3.9 us, 3.8; 2048 x 2048 7.8, 7.9;
// 2048 x 4096 14.6, 14.4), ahead from there to 256 MiB (1024 x 16384 27.9, 30.1; 4128 x 4200 29.1, 29.9; 5600 x 5600 51.0, 50.5), then three: 3648 x 9272 50.1, five 51.0, eight 51.5, paced
// 54.1; 8192 x 8192 87.9, 90.7, 92.4, 90.0.  But from 36 to 63 MiB one load at a time and as many workgroups as fit, paced / together and five, operands out of HBM and out of the memory-side
// cache: 2048 x 3072 9.8 / 11.1 and 10.0 / 10.7; 2144 x 2300 8.6 / 9.3 and 8.2 / 8.8; 4096 x 1500 9.9 / 11.2 and 10.0 / 10.8; 2720 x 3000 13.6 / 14.8 and 13.2 / 13.8; below and above
// not, 2048 x 2048 8.4 / 7.8; 4096 x 2048 14.5 / 14.6 and 15.1 / 13.7.
inline bool paced_tiles32(int64_t M, int64_t N) { return M * N * 8 >= ((int64_t)36 << 20) && M * N * 8 < ((int64_t)63 << 20); }

// Which transposes under the default mode, with the band height left to the library, take the sweep of tile_sweep.h.  Time of the sweep over that of the skewed raster, loads and
// occupancy as they are now.  Tiles: no pitch a power of two 0.84 to 1.00, on average 0.92 (40 sizes).  Both pitches multiples of 16 KiB: 8192 x 8192 x 4 B 0.99, 12288 x 8192
// x 4 B 0.98, 16384 x 8192 x 2 B 0.94, but with one of 64 KiB 32768 x 8192 x 2 B 1.14, 16384 x 8192 x 4 B 1.13, 8192 x 16384 x 4 B 1.08, 16384 x 4096 x 4 B 1.01; 16384 x 16384
// x 2 B (32 KiB) level.  Two bytes, rows of `in` 8 KiB or a power of two of them, sweep and skew: 1792 x 8192 13.9, 13.0; 2048 x 4096 8.8, 8.2; 1024 x 16384 14.9, 13.9; 4160 x 4096
// 14.5, 14.4; but 512 x 8192 4.66, 4.81, other multiples of 8 KiB 64 x 184320 11.6, 12.0; 320 x 36864 11.4, 11.8, and from 68 MiB on level, 1216 x 16384 16.5, 16.3; 2048 x 12288 20.1, 20.7.  Blocks into part lines, four bytes: 0.91 to 0.99, pitch of `in` a multiple of 8 KiB 0.98 to 1.04.
inline bool sweep_tiles(int64_t M, int64_t N, int elem_bytes) {
  const int64_t moved = 2 * M * N * elem_bytes;
  if (elem_bytes == 2 && power_of_two_pitch(N) && moved >= ((int64_t)24 << 20) && moved < ((int64_t)68 << 20)) return false;
  return (M | N) * elem_bytes % 16384 != 0 || (M * elem_bytes % 65536 != 0 && N * elem_bytes % 65536 != 0);
}
inline bool sweep_part_lines(int64_t N, int elem_bytes) { return elem_bytes == 4 && N * elem_bytes % 8192 != 0; }

// Blocks of 256 (two bytes) or 128 rows in 512 threads for a transpose into part lines (tall), rather than 64 rows in 256 threads, and whether a thread's loads are on their way one at a time
// (paced) or together.  us, tall / 64 rows, operands out of HBM and, where it says otherwise, out of the memory-side cache (three sets of buffers in turn):
//   Few rows, one block either way, most of a tall one empty: two bytes 56 rows 8.4 / 6.8 (17 MiB moved), 72 rows 7.5 / 7.7, 136 rows 51 / 54 (200 MiB); four bytes 44 rows 0.89 to 1.14
//   of the time, 52 rows 9.9 / 10.6 (47 MiB).
//   Just above one block, the second nearly empty: two bytes 264 rows 8.4 / 7.1, 280 rows 7.2 / 7.4 and 5.2 / 6.1 out of the cache, but from 128 MiB on 280 x 187240 59.7 / 54.3, 304 x 172456
//   54.9 / 51.9; four bytes 132 rows 7.5 / 6.3, 164 x 16780 8.4 / 7.3, 180 x 16748 8.6 / 7.8, 196 x 14040 6.5 / 8.0.
//   Few blocks for the compute units, two bytes above 1024 rows, below 22 MiB: 1032 x 4312 7.6 / 7.4 and 5.8 / 5.5, 8200 x 536 7.4 / 7.1 and 5.5 / 4.9; up to 1024 rows 520 x 8568 7.4 / 7.4
//   and 4.9 / 5.8, 776 x 8104 8.1 / 9.1 and 5.7 / 7.1; four bytes 516 x 4316 6.6 / 6.5 and 4.4 / 5.5, 1028 x 2164 6.6 / 6.5 and 4.7 / 4.9.
//   Tall and paced / together (64 rows for two bytes below 40 MiB, else tall): two bytes 4104 x 1656 7.7 / 9.3 and 7.0 / 6.6, 2056 x 4840 10.7 / 11.8 and 9.1 / 9.3, 8200 x 1400
//   10.7 / 12.6 and 9.6 / 9.7, but 1032 x 13208 15.8 / 15.0 and 14.0 / 12.1; four bytes 1028 x 4204 8.7 / 10.1 and 7.7 / 8.1, 2052 x 2424 8.9 / 10.5 and 8.0 / 8.0, 516 x 8380 8.6 / 10.1 and
//   7.4 / 7.3, but 516 x 13208 14.3 / 13.8 and 11.9 / 10.1.  Outside the sizes below loads together are up to 20 % ahead of one at a time out of the cache and level on average out of HBM, but
//   two bytes 8200 x 664 8.2 / 7.2, 776 x 8776 10.2 / 8.6, 392 x 22064 10.5 / 9.1 there.
// A launch has to hold its threads too: with one row of blocks, or two instead of three, half and three quarters as many columns fit.
enum LineBlocks : int { kLines = 0, kLinesTall = 1, kLinesTallPaced = 2 };
inline LineBlocks line_blocks(int64_t M, int64_t N, int elem_bytes) {
  const int rows = lines_rows(elem_bytes, true);
  const int64_t blocks_m = (M + rows - 1) / rows, gn = (N + 63) / 64, mib = (2 * M * N * elem_bytes) >> 20;
  if (blocks_m * gn * lines_threads(rows) > kLaunchThreads) return kLines;
  if (elem_bytes == 2) {
    if (M <= 64 || (M > 256 && M < (mib < 128 ? 280 : 320)) || (M > 1024 && mib < 22)) return kLines;
    return M > 1024 && mib < (M > 3072 ? 50 : 40) ? kLinesTallPaced : kLinesTall;
  }
  if (M <= 48 || (M > 128 && M < 188)) return kLines;
  return M > 256 && mib >= 31 && mib < (M > 1000 ? 56 : 40) ? kLinesTallPaced : kLinesTall;
}

}  // namespace swz
