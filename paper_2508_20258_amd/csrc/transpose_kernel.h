// Tiled 16-bit matrix transpose with a remapped program id:  out (N x M) = in (M x N)^T, both
// row-major (SwizzlePerf, Results and Appendix "Case Study: Other Swizzling Pattern Examples":
// the transpose kernel is the paper's largest win from XCD swizzling).
//
// One workgroup (256 threads) moves one TILE x TILE block: rows of `in` are read as 16-byte
// chunks into LDS, and read back with the transposing LDS read of gfx950 (ds_read_b64_tr_b16:
// inside a 16-lane group, lane s supplies 4 consecutive elements of row s/4 and lane i receives
// rows 0..3 of column i), so a lane ends up with 8 consecutive elements of one row of `out` and
// stores them as 16 bytes.  The kernel is bound by HBM: 4*M*N bytes per launch.
//
// TILE = 128: row segments of 256 bytes on both sides.
// TILE = 64: every row segment read or written is one whole 128-byte line, so tiles share no
//            lines and the mapping of tiles to XCDs cannot change the L2 hit rate.
// TILE = 32: row segments are half lines; horizontally adjacent tiles share the lines they read
//            and vertically adjacent tiles the lines they write.  This is the situation in which
//            co-locating neighbouring tiles on one XCD pays, and it is kept to show exactly that.
// With whole-line tiles what the order of the tiles decides is not the L2 but the memory channels:
// all tiles of one tile row write into the same TILE*2-byte wide column stripe of `out`, and when
// the row pitch of `out` is a power of two that stripe lives in a few channels only.  The skewed
// raster (pid_decode.h) makes tiles that run at the same time differ in their tile row as well as
// in their tile column; measured at 16384 x 16384, with a band height named, it takes the 64-wide tile from 4.4 to 5.9 TB/s
// (the 128-wide one from 4.8 to 5.8).  Under the default order most sizes are swept instead (tile_sweep.h; sweep_tiles has those that are not): us under the skewed raster -> swept, loads and
// occupancy as they are now: two bytes 16384 x 16384 183 -> 177 (6.1 TB/s), 8192 x 8192 55 -> 47.5, 10048 x 7040 60 -> 52.7, 3712 x 17656 64 -> 58, 16384 x 8192 93 -> 87, 4096 x 32768 98 -> 87; four bytes 5824 x 5824
// 54 -> 48.8, 5800 x 5804 55 -> 51.3.  What is left to a copy (5824 x 5824 x 4 43 us) is the memory's: workgroups that copy the same blocks to the same places without
// transposing them take 48 to 54 us by the order of the blocks, 47 to 52 with both sides of a block in one piece of 16 KiB.
// How many loads are on their way at a time, and in how many workgroups, follows from size, pitches and order (load_pace, paced_tiles32 and line_blocks in transpose_dispatch.h).
//
// LDS layout: row r at byte r*(TILE*2), 16-byte chunk c in slot c ^ key(r) (same idea as the
// GEMM's B panel; TILE*2/16 slots per row).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pid_decode.h"
#include "tile_sweep.h"
#include "transpose_dispatch.h"

namespace swz {

typedef __attribute__((ext_vector_type(4))) short t_s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t t_u32x4;

// Block (pm, pn) of this workgroup: by the mode, or, where sweep is not 0, in the sweep with so many tile rows to an XCD.
__device__ __forceinline__ void tr_block(int grid_m, int grid_n, int num_xcd, int group_m, int mode, int sweep, int* pm, int* pn) {
  if (sweep != 0) swz_sweep_tile((int)blockIdx.x, grid_m, grid_n, num_xcd, sweep, pm, pn);       // uniform
  else swz_decode_tile((int)blockIdx.x, grid_m, grid_n, num_xcd, group_m, mode, pm, pn);
}

// Where the 16 bytes at row m, column n of `in` are, m and n brought inside it: no branch around a load.  With one, the compiler waits for every load
// before it issues the next, and a block's two to five loads a thread took as many trips to memory (us one at a time -> together: 1024 x 1024 x 4 B 4.0 -> 2.7,
// 2048 x 2048 x 2 B 5.4 -> 4.6, 300 x 600 x 4 B 2.6 -> 2.2).  Lanes beyond the edge read the edge again, out of a cache: with 8 to 24 rows of two bytes in blocks of 64 rows 2 % more time
// than a branch takes (8 x 1441800 37.4, 38.2 us); four-byte tiles of up to 32 rows leave those loads out (LOADS below).
template <class T>
__device__ __forceinline__ const t_u32x4* tr_source(const T* in, int m, int n, int M, int N) {
  m = m < 0 ? 0 : m < M ? m : M - 1;
  n = n < N ? n : N - 16 / (int)sizeof(T);
  return reinterpret_cast<const t_u32x4*>(in + (size_t)m * N + n);
}

template <int TILE>
__device__ __forceinline__ int tr_key(int row) {
  // the 16 lanes of a transposing read take 4 consecutive rows x 32 bytes (a chunk pair): give
  // those rows different chunk pairs where the row has room for it
  return TILE >= 64 ? (row & 3) << 1 : (row & 1) << 1;
}

// STREAM: the whole-line stores are streaming (non-temporal) stores.  That is the faster choice when the
// matrices are larger than the memory-side cache (6.1 against 5.4 TB/s at 16384 x 16384 with the skewed
// raster) and the slower one when `out` would have stayed in that cache (5.5 against 6.2 TB/s at
// 8192 x 8192), so the host decides.
template <int TILE, int MODE, bool STREAM>
__global__ __launch_bounds__(256) void transpose16_kernel(const uint16_t* __restrict__ in, uint16_t* __restrict__ out,
                                                          int M, int N, int grid_m, int grid_n, int num_xcd,
                                                          int group_m, int skew, int sweep, int paced) {
  constexpr int ROW_BYTES = TILE * 2;
  constexpr int SLOTS = ROW_BYTES / 16;                  // 16-byte chunks per tile row
  constexpr int CHUNKS = TILE * SLOTS;                   // chunks per tile
  constexpr int PER_THREAD = CHUNKS / 256 > 0 ? CHUNKS / 256 : 1;
  __shared__ __attribute__((aligned(16))) unsigned char tile[TILE * ROW_BYTES];

  int pm, pn;
  tr_block(grid_m, grid_n, num_xcd, group_m, MODE | (skew ? kModeSkew : 0), sweep, &pm, &pn);
  const int m0 = pm * TILE, n0 = pn * TILE;
  const int tid = threadIdx.x;

  // ---- in -> LDS: row-contiguous 16-byte chunks (columns are whole chunks: N % 8 == 0) ----
  // Rows and columns outside `in` come from its edge (tr_source), their part of the tile is never stored.
  t_u32x4 v[PER_THREAD];
#pragma unroll
  for (int i = 0; i < PER_THREAD; ++i) {
    const int q = tid + 256 * i;
    if (CHUNKS % 256 != 0 && q >= CHUNKS) continue;
    const t_u32x4* src = tr_source(in, m0 + q / SLOTS, n0 + q % SLOTS * 8, M, N);
    // whole-line tiles read every line exactly once: streaming loads; half-line tiles rely on the L2 keeping
    // the line for the neighbouring tile
    if constexpr (TILE >= 64) v[i] = __builtin_nontemporal_load(src);
    else v[i] = *src;
    if (PER_THREAD > 1 && paced != 0) asm volatile("s_waitcnt vmcnt(0)" : : : "memory");        // uniform
  }
#pragma unroll
  for (int i = 0; i < PER_THREAD; ++i) {
    const int q = tid + 256 * i, r = q / SLOTS, c = q % SLOTS;
    if (CHUNKS % 256 == 0 || q < CHUNKS) *reinterpret_cast<t_u32x4*>(tile + r * ROW_BYTES + ((c ^ tr_key<TILE>(r)) << 4)) = v[i];
  }
  __syncthreads();

  // ---- LDS -> out: a unit of work for a wave is 16 columns (rows of out) x 32 rows of the tile ----
  // lane: i = lane%16 -> column, g = lane/16 -> 8-row block; two transposing reads give rows 8g..8g+7
  const int lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, g = lane >> 4;
  constexpr int COL_BLOCKS = TILE / 16;                  // 16-column blocks
  constexpr int ROW_BLOCKS = TILE / 32;                  // 32-row blocks
  constexpr int UNITS = COL_BLOCKS * ROW_BLOCKS;         // wave-level units of work: 8 (TILE 64) or 2 (TILE 32)
  // what a lane holds after the two transposing reads of 32-row block rb of column block cb:
  // in[m0 + 32rb + 8g .. +7][n0 + 16cb + i]  =  out[n0 + 16cb + i][m0 + 32rb + 8g .. +7], 16 bytes
  auto read_unit = [&](int cb, int rb) __attribute__((always_inline)) {
    const int row = 32 * rb + 8 * g + (i >> 2);          // the row whose 4 elements this lane supplies (+4 for the second read)
    const int col = 16 * cb + 4 * (i & 3);
    const unsigned char* p0 = tile + row * ROW_BYTES + (((col >> 3) ^ tr_key<TILE>(row)) << 4) + (col & 7) * 2;
    const unsigned char* p1 = tile + (row + 4) * ROW_BYTES + (((col >> 3) ^ tr_key<TILE>(row + 4)) << 4) + (col & 7) * 2;
    const t_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) t_s16x4*)p0);
    const t_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) t_s16x4*)p1);
    t_u32x4 v;
    v[0] = (uint32_t)(uint16_t)lo[0] | ((uint32_t)(uint16_t)lo[1] << 16);
    v[1] = (uint32_t)(uint16_t)lo[2] | ((uint32_t)(uint16_t)lo[3] << 16);
    v[2] = (uint32_t)(uint16_t)hi[0] | ((uint32_t)(uint16_t)hi[1] << 16);
    v[3] = (uint32_t)(uint16_t)hi[2] | ((uint32_t)(uint16_t)hi[3] << 16);
    return v;
  };
  if constexpr (ROW_BLOCKS >= 2) {
    // Two 32-row blocks give the two 64-byte halves of 16 lines of `out`.  Lanes i and i + 8 trade one
    // half (a rotation by 8 inside the 16-lane row), after which one store instruction writes 8 whole
    // 128-byte lines (lanes i < 8 their left halves, lanes i >= 8 the right halves) and the next one the other 8.
    constexpr int PAIRS = COL_BLOCKS * (ROW_BLOCKS / 2);
#pragma unroll
    for (int u = wave; u < PAIRS; u += 4) {
      const int cb = u % COL_BLOCKS, rp = u / COL_BLOCKS;
      const t_u32x4 h0 = read_unit(cb, 2 * rp), h1 = read_unit(cb, 2 * rp + 1);
      const bool low = i < 8;
      t_u32x4 got, s0, s1;
#pragma unroll
      for (int e = 0; e < 4; ++e) got[e] = __builtin_amdgcn_mov_dpp(low ? h1[e] : h0[e], 0x128 /* row_ror:8 */, 0xf, 0xf, false);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0[e] = low ? h0[e] : got[e];
        s1[e] = low ? got[e] : h1[e];
      }
      const int on = n0 + 16 * cb + (i & 7);
      const int om = m0 + 64 * rp + (low ? 0 : 32) + 8 * g;
      if (om < M) {                                        // M % 8 == 0: the 8 elements are in or out together
        t_u32x4* d0 = reinterpret_cast<t_u32x4*>(out + (size_t)on * M + om);
        t_u32x4* d1 = reinterpret_cast<t_u32x4*>(out + (size_t)(on + 8) * M + om);
        if constexpr (STREAM) {
          if (on < N) __builtin_nontemporal_store(s0, d0);
          if (on + 8 < N) __builtin_nontemporal_store(s1, d1);
        } else {
          if (on < N) *d0 = s0;
          if (on + 8 < N) *d1 = s1;
        }
      }
    }
  } else {
#pragma unroll
    for (int u = wave; u < UNITS; u += 4) {
      const int cb = u % COL_BLOCKS, rb = u / COL_BLOCKS;
      const t_u32x4 v = read_unit(cb, rb);
      const int on = n0 + 16 * cb + i;
      const int om = m0 + 32 * rb + 8 * g;
      if (on < N && om < M) *reinterpret_cast<t_u32x4*>(out + (size_t)on * M + om) = v;
    }
  }
}

// Four-byte elements: out (N x M) = in (M x N)^T, one 256-thread workgroup per 64 x 64 block (16 KiB of LDS).
// There is no transposing LDS read for 32-bit elements, so a lane gathers its four consecutive elements of a row
// of `out` with four 4-byte LDS reads from four consecutive tile rows.  A wave instruction covers 8 rows of
// `out` x 32 elements = 8 whole 128-byte lines: lane l takes column 8 jb + l/8 of the tile and tile rows
// 32 h + 4 (l%8) .. +3.  LDS layout: row r at byte r*256, 16-byte chunk c (4 columns) in slot
// c ^ (((r >> 2) & 7) << 1): the 64 lanes of one read (8 row groups x 8 columns = 2 chunks) then hit 64
// different banks.  Same mapping arguments, same streaming-store rule as the 16-bit kernel.
// LOADS of the four that a thread has for a tile, 16 rows each: fewer where `in` has no more rows (one tile row).
template <int MODE, bool STREAM, bool PACED, int LOADS>
__global__ __launch_bounds__(256) void transpose32_kernel(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                          int M, int N, int grid_m, int grid_n, int num_xcd,
                                                          int group_m, int skew, int sweep) {
  constexpr int TILE = 64, SLOTS = TILE / 4, CHUNKS = TILE * SLOTS, ROW_BYTES = TILE * 4;
  __shared__ __attribute__((aligned(16))) unsigned char tile[TILE * ROW_BYTES];
  int pm, pn;
  tr_block(grid_m, grid_n, num_xcd, group_m, MODE | (skew ? kModeSkew : 0), sweep, &pm, &pn);
  const int m0 = pm * TILE, n0 = pn * TILE;
  const int tid = threadIdx.x;
  auto key = [](int r) { return ((r >> 2) & 7) << 1; };
  static_assert(LOADS * 256 <= CHUNKS, "a tile");
  t_u32x4 in_v[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int q = tid + 256 * i;
    in_v[i] = __builtin_nontemporal_load(tr_source(in, m0 + q / SLOTS, n0 + q % SLOTS * 4, M, N));
    if constexpr (PACED) asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
  }
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int q = tid + 256 * i, r = q / SLOTS, c = q % SLOTS;
    *reinterpret_cast<t_u32x4*>(tile + r * ROW_BYTES + ((c ^ key(r)) << 4)) = in_v[i];
  }
  __syncthreads();
  const int lane = tid & 63, wave = tid >> 6;
  const int jj = lane >> 3, rg = lane & 7;
#pragma unroll
  for (int u = wave; u < 16; u += 4) {                 // 8 column blocks x 2 halves of the tile's rows
    const int jb = u >> 1, h = u & 1;
    const int col = 8 * jb + jj;                       // tile column = row of out
    const int row = 32 * h + 4 * rg;                   // first of this lane's 4 tile rows = column of out
    t_u32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      v[k] = *reinterpret_cast<const uint32_t*>(tile + (row + k) * ROW_BYTES + (((col >> 2) ^ key(row + k)) << 4) + (col & 3) * 4);
    const int on = n0 + col, om = m0 + row;
    if (on < N && om < M) {                            // M % 4 == 0
      t_u32x4* dst = reinterpret_cast<t_u32x4*>(out + (size_t)on * M + om);
      if constexpr (STREAM) __builtin_nontemporal_store(v, dst);
      else *dst = v;
    }
  }
}

// The same transpose where rows of `out` do not start on 128-byte lines (M * sizeof(T) no multiple of 128, or `out` itself
// off a line).  A 64-wide tile of the other kernels then writes two part lines per row, which reach memory in two
// pieces.  Here a workgroup takes BM rows of `in` x 64 columns, and the BM elements it
// writes of row n of `out` are shifted left by s(n), the elements by which the row overhangs a line, so that it writes whole lines: row n
// gets columns [BM pm - s(n), BM pm - s(n) + BM), the last block of the row everything up to M (one line more at
// most).  Its block of `in` grows by the E - 1 rows above it (E elements fill a line), which the block above reads too.  BM is 64 with 256
// threads: 31 rows more of four bytes, 63 of two, half and all of the input once more; or 128 of four bytes and 256 of two with 512 threads, a
// quarter more.  Part of that the L2 serves.  line_blocks (transpose_dispatch.h) says which: the tall blocks lose where M leaves most of one empty and where
// there are too few of them.  PACED: a thread's loads one at a time.  s(n) differs from row
// to row, so a lane gathers its 16 bytes element by element, four rows or eight rows of the tile at a column: the
// transposing LDS read takes the same rows for 4 columns.
// A wave instruction stores 8 rows x 8 chunks = 8 whole lines: lane l takes row l / 8, chunk l % 8.
// LDS: 16-byte chunk c of tile row r in slot c ^ key(r); key steps with the chunk of rows a lane gathers, so that the 8
// chunks of one column lie in different banks whatever their shift.  The stores are streaming ones at every size: nothing
// is left to merge in the L2.
// Bound by HBM and the rows read twice.  Measured, matrices not in cache, 64 rows and 256 threads -> tall (us; GB/s of the matrix read and written):
//     two bytes   10000 x 7000  75 -> 60 (4670)    8200 x 8208  67 -> 57 (4720)    30000 x 1544   49 -> 41 (4560)    3000 x 3000  10.7 -> 9.0
//     four bytes   5800 x 5804  60 -> 56 (4810)    200 x 20000  9.5 -> 8.6         15764 x 8092  214 -> 204 (5000)
// and with a block's loads on their way together, four-byte blocks swept: 10000 x 7000 60.5 -> 58, 5800 x 5804 56 -> 52 (5170), 15764 x 8092 209 -> 200, 5288 x 3128 x 2 B 15.1 -> 13.3.
// Two-byte blocks are not swept: 10000 x 7000 57.5 -> 58.1, 8200 x 8200 up to 9 % slower, 5288 x 3128 13.3 -> 12.3; they keep the skewed raster, which is level with the plain one out of HBM
// and slower in a cache (one set of buffers, 10000 x 7000 47.5 against 43.7 us, 173 MiB fetched against 143).
// (tiles on line-blind boundaries 102, 110 and 82, 363 us; 60 us where both pitches are whole lines, 10048 x 7040.)  256 rows of four bytes leave a
// compute unit two workgroups: 58 us at 5800 x 5804; with 256 threads 77.  128 columns: 60 us there, 61 at 10000 x 7000.

template <class T, int BM_, bool PACED>
__global__ __launch_bounds__(lines_threads(BM_)) void transpose_lines_kernel(const T* __restrict__ in, T* __restrict__ out, int M, int N, int grid_m,
                                                                                  int grid_n, int num_xcd, int group_m, int mode, int sweep) {
  constexpr int TILE = 64, BM = BM_, NT = lines_threads(BM_);
  constexpr int CH = 16 / (int)sizeof(T), E = 128 / (int)sizeof(T);                  // elements per chunk, per line
  constexpr int SLOTS = TILE / CH, ROWS = BM + E, ROW_BYTES = TILE * (int)sizeof(T), LINES = BM / E;
  __shared__ __attribute__((aligned(16))) unsigned char tile[ROWS * ROW_BYTES];
  int pm, pn;
  tr_block(grid_m, grid_n, num_xcd, group_m, mode, sweep, &pm, &pn);
  const int m0 = pm * BM - E, n0 = pn * TILE;                    // first row of `in` in the tile, first column
  const int tid = threadIdx.x;
  auto key = [](int r) { return sizeof(T) == 2 ? (r >> 3) & 7 : ((r >> 2) & 7) << 1; };
  static_assert(ROWS * SLOTS % NT == 0, "whole loads");
  constexpr int LOADS = ROWS * SLOTS / NT;
  t_u32x4 in_v[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int q = tid + NT * i;
    in_v[i] = *tr_source(in, m0 + q / SLOTS, n0 + q % SLOTS * CH, M, N);
    if constexpr (PACED) asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
  }
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int q = tid + NT * i, r = q / SLOTS, c = q % SLOTS;
    *reinterpret_cast<t_u32x4*>(tile + r * ROW_BYTES + ((c ^ key(r)) << 4)) = in_v[i];
  }
  __syncthreads();
  const int lane = tid & 63, wave = tid >> 6;
  const int jj = lane >> 3, rg = lane & 7;
  const uint32_t base = (uint32_t)(reinterpret_cast<uintptr_t>(out) / sizeof(T));
  const int lines = pm == grid_m - 1 ? LINES + 1 : LINES;        // uniform
#pragma unroll
  for (int jb = wave; jb < TILE / 8; jb += NT / 64) {
    const int col = 8 * jb + jj, n = n0 + col;                   // tile column = row of out
    const int shift = (int)((base + (uint32_t)n * (uint32_t)M) % (uint32_t)E);       // E divides 2^32
    for (int h = 0; h < lines; ++h) {
      const int row = E - shift + h * E + CH * rg;               // tile row of this lane's first element
      const int m = m0 + row;
      if (n < N && m >= 0 && m < M) {                            // M % CH == 0: the chunk is in or out as a whole
        T e[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          e[k] = *reinterpret_cast<const T*>(tile + (row + k) * ROW_BYTES + (((col / CH) ^ key(row + k)) << 4) + (col % CH) * (int)sizeof(T));
        t_u32x4 v;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          if constexpr (sizeof(T) == 2) v[w] = (uint32_t)e[2 * w] | ((uint32_t)e[2 * w + 1] << 16);
          else v[w] = (uint32_t)e[w];
        }
        __builtin_nontemporal_store(v, reinterpret_cast<t_u32x4*>(out + (size_t)n * M + m));
      }
    }
  }
}

}  // namespace swz
