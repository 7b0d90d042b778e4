// Which kernel a GEMM launch takes, over which grid, and which block of C each of its workgroups computes: host logic only,
// shared by the launch (swz_gemm_ex) and by the entry point that reports it (swz_gemm_launch_map).
#pragma once

#include <stdint.h>

#include "../../include/swz.h"
#include "pid_decode.h"

namespace swz {

constexpr int kStageK = 64;    // K extent of a ring stage of the sub-tile kernel: two MFMA steps, whole 128-byte lines of A

// The sub-tile shapes: rows and columns of C, waves along each, ring stages, and what a stage of one workgroup costs in ns on a
// chip whose every CU has one (measured: the slope of kernel time over K).  The fixed part of a round (launch or hand-over, the
// first operands, the stores) is about kRoundNs whatever the shape; a whole tile of gemm_kernel.h takes kWholeRoundNs, as it
// also runs its look-ahead past the end of K.
struct SubTile { int bm, bn, wm, wn, stages, stage_ns; };
constexpr int kSubTileCount = 7;
constexpr SubTile kSubTiles[kSubTileCount] = {{32, 32, 2, 2, 8, 140},   {32, 64, 2, 2, 6, 160},   {64, 64, 2, 2, 5, 195},  {128, 64, 4, 2, 6, 310},
                                              {64, 128, 2, 4, 6, 310},  {128, 128, 2, 4, 5, 520}, {128, 256, 2, 4, 3, 950}};
constexpr int kQuarterPiece = 5, kHalfPiece = 6;       // of a 256x256 tile
constexpr int64_t kRoundNs = 2500, kWholeRoundNs = 4000;

// Which sub-tile shape (index into kSubTiles) computes this product fastest, or -1 where the plan's tile as one
// workgroup does.  The estimate is  rounds x (kRoundNs + stages x cost), rounds = workgroups that touch C over CUs.  One
// 128x128, 128x256 and 256x256 tile of gemm_kernel.h costs 600, 840 and 1350 ns a stage (two 128x128 ones share a CU: 920 the
// pair; a partial last round of 256x256 tiles costs what its pieces make of it, see gemm_launch).  Ties go to the larger
// tile: it moves fewer bytes.  A sub-tile has to be 5 % better than the tile, the spread of the estimate near a tie.
// Fitted on 60 products.  On 140 others, every shape timed (log-uniform sizes, N and K from 64 to 16384): 60 with M from 1 to
// 16384 are on average as fast as with their best shape (worst 3.6 % behind), 80 with M from 128 to 16384 0.5 % behind (worst 13 %:
// 1528x4880x536, 16.2 us in whole 128x256 tiles and 14.3 in sub-tiles of that size).
inline int choose_subtile(int64_t M, int64_t N, int64_t K, const swz_params& r, int cus) {
  const int64_t stages = (K + kStageK - 1) / kStageK;
  auto rounds = [&](int64_t bm, int64_t bn, int64_t per_round) {
    return (((M + bm - 1) / bm) * ((N + bn - 1) / bn) + per_round - 1) / per_round;
  };
  auto estimate = [&](int64_t n, int64_t ns) { return n * (kRoundNs + stages * ns); };
  auto whole = [&](int64_t n, int64_t ns) { return n * (kWholeRoundNs + stages * ns); };
  int64_t best;
  if (r.bm == 128 && r.bn == 128) {
    best = rounds(128, 128, cus) == 1 ? whole(1, 600) : whole(rounds(128, 128, 2 * cus), 920);
  } else if (r.bm != r.bn) {
    best = whole(rounds(r.bm, r.bn, cus), 840);
  } else {
    const int64_t tiles = rounds(256, 256, 1), tail = tiles % cus;
    best = whole(tiles / cus, 1350) + (tail == 0 ? 0 : whole(1, tiles < cus ? 1350 : 4 * tail <= cus ? 520 : 2 * tail <= cus ? 840 : 1350));
  }
  best -= best / 20;
  int choice = -1;
  for (int s = kSubTileCount - 1; s >= 0; --s) {
    if (kSubTiles[s].bm > r.bm || kSubTiles[s].bn > r.bn) continue;         // a sub-tile is no larger than the plan's tile
    const int64_t e = estimate(rounds(kSubTiles[s].bm, kSubTiles[s].bn, cus), kSubTiles[s].stage_ns);
    if (e < best) {
      best = e;
      choice = s;
    }
  }
  return choice;
}

// A launch with one workgroup per tile or sub-tile.
struct GemmLaunch {
  int sub;                            // -1: the plan's tiles, whole.  Else an index into kSubTiles: the shape of all workgroups
  bool pieces;                        //   or, where `pieces` is set, of those behind the first `whole`, which compute 256x256 tiles
  int bm, bn, grid_m, grid_n, group_m;   // the grid the map is evaluated on (with `pieces` that of the 256x256 tiles)
  int whole, deal;                    // see swz_tail_piece
  int64_t blocks;                     // workgroups launched
};

// r: the resolved plan; cus: compute units.  `free_tile`: the caller left the tile to the library, otherwise a tile is one workgroup.
// Bounds for anything else: 32-bit source offsets over 64 rows of B, and a grid well inside the 32-bit range whatever the shape.
inline GemmLaunch gemm_launch(int64_t M, int64_t N, int64_t K, const swz_params& r, int grid_m, int grid_n, int group_m, bool free_tile, int cus) {
  GemmLaunch l = {-1, false, r.bm, r.bn, grid_m, grid_n, group_m, 0, 1, (int64_t)grid_m * grid_n};
  if (!free_tile || N >= ((int64_t)1 << 24) || l.blocks >= ((int64_t)1 << 16)) return l;
  l.sub = choose_subtile(M, N, K, r, cus);
  if (l.sub >= 0) {
    const SubTile& s = kSubTiles[l.sub];
    l.bm = s.bm;
    l.bn = s.bn;
    l.grid_m = (int)((M + s.bm - 1) / s.bm);
    l.grid_n = (int)((N + s.bn - 1) / s.bn);
    l.blocks = (int64_t)l.grid_m * l.grid_n;
    const int64_t band = (int64_t)group_m * (r.bm / s.bm);       // rows of sub-tiles as high as a band of tiles
    l.group_m = (int)(band < l.grid_m ? band : l.grid_m);
    return l;
  }
  // A last round that fills at most half of the compute units is cut into halves or quarters of tiles, which then fit it:
  // 1350 -> 840 or 520 ns a stage.  Measured, start -> here: 4352x4096x4096 (16 tiles left over) 154 -> 117 us, 6000x3000x3000 (32) 124 -> 101,
  // 5120x4608x4096 (104) 162 -> 146, 10000x7000x4096 (96, fifth round) 442 -> 427.  Above half a round the pieces need a second
  // round of their own: 5120x5120x5120 (144) stays at 198 us whole.
  const int total = grid_m * grid_n, whole = total / cus * cus, tail = total - whole;
  if (r.bm == 256 && r.bn == 256 && whole > 0 && tail > 0 && 2 * tail <= cus) {
    l.sub = 4 * tail <= cus ? kQuarterPiece : kHalfPiece;
    l.pieces = true;
    l.whole = whole;
    l.deal = r.num_xcd < tail ? r.num_xcd : tail;
    const int subs = (256 / kSubTiles[l.sub].bm) * (256 / kSubTiles[l.sub].bn);
    l.blocks = whole + ((int64_t)tail + l.deal - 1) / l.deal * l.deal * subs;
  }
  return l;
}

// The block of C hardware workgroup w of the launch computes: first row, first column, rows, columns (all 0: it leaves at once).
struct GemmBlock { int32_t row, col, rows, cols; };
inline GemmBlock gemm_block(const GemmLaunch& l, int num_xcd, int mode, int64_t M, int64_t N, int w) {
  int pm, pn;
  int64_t row, col, rows = l.bm, cols = l.bn;
  if (!l.pieces || w < l.whole) {
    swz_decode_tile(w, l.grid_m, l.grid_n, num_xcd, l.group_m, mode, &pm, &pn);
    row = (int64_t)pm * l.bm;
    col = (int64_t)pn * l.bn;
  } else {
    rows = kSubTiles[l.sub].bm;
    cols = kSubTiles[l.sub].bn;
    const int sub_m = l.bm / (int)rows;
    int v, sub;
    if (!swz_tail_piece(w, l.whole, l.deal, sub_m * (l.bn / (int)cols), l.grid_m * l.grid_n, &v, &sub)) return {0, 0, 0, 0};
    swz_decode_tile(v, l.grid_m, l.grid_n, num_xcd, l.group_m, mode, &pm, &pn);
    row = (int64_t)pm * l.bm + (sub % sub_m) * rows;
    col = (int64_t)pn * l.bn + (sub / sub_m) * cols;
    if (row >= M || col >= N) return {0, 0, 0, 0};
  }
  return {(int32_t)row, (int32_t)col, (int32_t)(M - row < rows ? M - row : rows), (int32_t)(N - col < cols ? N - col : cols)};
}

}  // namespace swz
