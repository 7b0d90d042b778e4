// The order in which a transpose visits its tiles where no power-of-two pitch asks for the skewed raster: the whole chip sweeps the columns of a
// window of tile rows together, every XCD in tile rows of its own.
//
// XCD x = w mod X owns `rows` neighbouring tile rows of a window of X * rows and walks them column by column.  What is written at a time then is
// whole stretches of neighbouring rows of the output (X * rows tiles of 64 elements), what is read a band of whole rows of the input, and tiles
// beside and below each other, which share lines of the input where rows start inside one, are on one XCD.  Under the XCD renumbering the XCDs
// work in eight places far apart, and the HBM serves 4 to 14 % fewer bytes a second (transpose_kernel.h has the times).
//
// Windows are whole: F = grid_m div (X * rows) of them take the first F * X * rows * grid_n ids, a multiple of X, so that id w of a window, w = i * X + x
// with i in [0, rows * grid_n), is tile row x * rows + i mod rows, column i div rows: every tile of the window once.  The R < X * rows rows left are one
// more raster, column by column, of which XCD x gets the run that the renumbering of pid_decode.h gives it.
#pragma once

#include "pid_decode.h"

// Requires 1 <= rows, num_xcd; grid_m * grid_n < 2^31; 0 <= w < grid_m * grid_n.
SWZ_HD void swz_sweep_tile(int w, int grid_m, int grid_n, int num_xcd, int rows, int* pm, int* pn) {
  const int64_t height = (int64_t)num_xcd * rows;                // may be larger than the grid: no window then
  const int windows = (int)(grid_m / height), first = (int)(windows * height), whole = first * grid_n;
  if (w < whole) {
    const int size = (int)height * grid_n, win = w / size, k = w - win * size;
    const int i = k / num_xcd, x = k - i * num_xcd, c = i / rows;
    *pm = win * (int)height + x * rows + (i - c * rows);
    *pn = c;
  } else {
    const int left = grid_m - first, l = swz_xcd_renumber(w - whole, left * grid_n, num_xcd), c = l / left;
    *pm = first + (l - c * left);
    *pn = c;
  }
}

// Tile rows of an XCD in a window: four.  Where the grid has no window of that height, two-byte elements take one (1600 x 16776 23.8 us, with three 25.3;
// 640 x 30000 16.2, 17.5), four-byte ones as many as fit (800 x 16000 18.6 us, with one 20.2).
SWZ_HD int swz_sweep_rows(int grid_m, int num_xcd, int elem_bytes) {
  if (grid_m >= (int64_t)4 * num_xcd) return 4;
  return elem_bytes == 4 && grid_m >= num_xcd ? grid_m / num_xcd : 1;
}
