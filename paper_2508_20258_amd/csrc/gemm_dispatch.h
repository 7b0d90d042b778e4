// Which kernel a GEMM launch takes, over which grid, and which block of C each of its workgroups computes: host logic only,
// shared by the launch (swz_gemm_ex) and by the entry point that reports it (swz_gemm_launch_map).
#pragma once

#include <math.h>
#include <stdint.h>

#include "../../include/swz.h"
#include "pid_decode.h"

namespace swz {

constexpr int kStageK = 64;    // K extent of a ring stage of the sub-tile kernel: two MFMA steps, whole 128-byte lines of A

// The sub-tile shapes: rows and columns of C, waves along each, ring stages, and what a stage of one workgroup costs in ns on a
// chip whose every CU has one (measured: the slope of kernel time over K).  The fixed part of a round (launch or hand-over, the
// first operands, the stores) is about kRoundNs whatever the shape; a whole tile of gemm_kernel.h takes kWholeRoundNs, as it
// also runs its look-ahead past the end of K.
// stage_ns 0: only with feeders.  fed_ns: what a stage costs where other workgroups fetch ahead (see feed_launch; 0: never).
struct SubTile { int bm, bn, wm, wn, stages, stage_ns, fed_ns; };
constexpr int kSubTileCount = 10;
constexpr SubTile kSubTiles[kSubTileCount] = {{32, 32, 2, 2, 8, 140, 90},    {32, 64, 2, 2, 6, 160, 120},  {64, 64, 2, 2, 5, 195, 150},
                                              {128, 64, 4, 2, 6, 310, 0},    {64, 128, 2, 4, 6, 310, 0}, {128, 128, 2, 4, 5, 520, 0},
                                              {128, 256, 2, 4, 3, 950, 0},   {64, 32, 2, 2, 8, 0, 130},    {96, 128, 2, 2, 5, 440, 0},
                                              {192, 128, 4, 2, 4, 715, 0}};
constexpr int kQuarterPiece = 5, kHalfPiece = 6;       // of a 256x256 tile
// Bytes of B per XCD that are fetched ahead: an eighth of the L2 (32 x 2048 x 16384: 1/32 and 1/8 24 us, 1/4 27, 1/2 42)
constexpr int kFeedLead = 1 << 19;
constexpr int64_t kRoundNs = 2500, kWholeRoundNs = 4000;

// Which sub-tile shape (index into kSubTiles) computes this product fastest, or -1 where the plan's tile as one
// workgroup does.  The estimate is  rounds x (kRoundNs + stages x cost), rounds = workgroups that touch C over CUs.  One
// 128x128, 128x256 and 256x256 tile of gemm_kernel.h costs 600, 840 and 1350 ns a stage (two 128x128 ones share a CU: 920 the
// pair; a partial last round of 256x256 tiles costs what its pieces make of it, see gemm_launch).  Ties go to the later
// shape of the table.  A sub-tile has to be 5 % better than the tile, the spread of the estimate near a tie.
// 96 and 192 rows fill a round that the powers of two leave half empty or just outgrow: 9516x544x1056 20.2 -> 16.3 us (128x256 -> 192x128), 542x4128x14888 147 -> 123
// (128x128 -> 96x128), 11034x368x2048 29.3 -> 22.9; over the 120 products drawn for which the choice changed 0.93 of the time (see rows96_pay for those where it was more), over 150 more with K from 704 0.92 with operands out of HBM
// and 0.91 out of the memory-side cache, where 11 and 6 of them are more than 3 % slower (7554x560x3248 45.0, 52.1 and 39.4, 37.1; 9505x592x3944 without bands 60, 69 and 55, 61).  Not kept:
// 96x64 and 192x64, 0.95 to 1.32 of the time, as stripes of B half as wide come out of HBM at half the pace (13429x136x4744 55 -> 72); 160x128, no faster than 192x128.
// Fitted on 60 products.  On 140 others, every shape timed (log-uniform sizes, N and K from 64 to 16384): 60 with M from 1 to
// 16384 are on average as fast as with their best shape (worst 3.6 % behind), 80 with M from 128 to 16384 0.5 % behind (worst 13 %:
// 1528x4880x536, 16.2 us in whole 128x256 tiles and 14.3 in sub-tiles of that size).

// Where 96 rows to a sub-tile may take the place of 128.  They have the fabric carry B once more for every further row of sub-tiles, half and a third as often again where 128 rows make two
// and three of them.  us with 128x128 and with 96x128, first with operands out of HBM, then out of the memory-side cache:
//   One stage of K, one round: nothing to gain.  203 x 9576 x 8 4.7, 5.0 and 3.8, 4.0; 289 x 6792 x 32 4.9, 5.1 and 3.9, 4.0; 440 x 5200 x 8 4.6, 4.9 and 4.0, 3.9.
//   193 to 256 rows, where the third row of sub-tiles is less than half full or K short: 193 x 10400 x 520 9.9, 9.2 and 8.2, 8.5, x 2056 25.1, 23.3 and 18.9, 21.5, x 4104 46, 42 and
//   33, 39; 224 x 10400 x 4104 46, 41 and 34, 37; 256 x 8200 x 264 8.2, 7.6 and 5.9, 6.2.  But 240 x 9000 x 520 11.2, 9.9 and 8.4, 8.2; 256 x 9000 x 2056 29.8, 24.8 and 20.5, 19.1.
//   289 to 384 rows: 289 x 6792 x 168 6.4, 6.3 and 4.8, 5.0; 300 x 7504 x 264 7.9, 7.6 and 6.1, 6.3; from K = 328 on 300 x 6792 8.4, 8.0 and 6.7, 6.7, x 520 10.3, 9.6 and 8.4, 8.1.
//   More rows, two stages: 480 x 4504 x 104 5.8, 5.5 and 4.4, 4.3.
inline bool rows96_pay(int64_t M, int64_t K, bool one_round) {
  if (one_round && K <= kStageK) return false;
  if (M > 192 && M <= 256) return M >= 240 && K >= 512;
  return M <= 288 || M > 384 || K >= 328;
}

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
    if (kSubTiles[s].stage_ns == 0 || kSubTiles[s].bn > r.bn || kSubTiles[s].bm > r.bm * 3 / 2) continue;      // those with feeders only; larger than the plan's tile
    if (kSubTiles[s].bm > r.bm && K >= (1 << 23)) continue;                    // the 32-bit source offsets of bm rows are checked for the plan's tile
    const int64_t n = rounds(kSubTiles[s].bm, kSubTiles[s].bn, cus), e = estimate(n, kSubTiles[s].stage_ns);
    if (e < best) {
      if (kSubTiles[s].bm == 96 && !rows96_pay(M, K, n == 1)) continue;
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
  bool pair;                          // tiles of 128x256, two workgroups to a compute unit (gemm_pair_kernel.h)
  int a_feeders, b_feeders, feed_ticks;   // workgroups per XCD that fetch A and B ahead, ticks of 10 ns per 1024 of K; 0: none fetches ahead
};

// Few rows and a long K: sub-tiles on at most 9/16 of the compute units, and others fetch their operands ahead of them into the
// L2 of their XCD (fetch_ahead in gemm_subtile_kernel.h says why).  false: not this product.
//   K from 2048 on, M up to 128; from 4096 on up to 192 (229 x 792 x 16312 60.5 us without, 62.6 with).  Below, what is gained with B in HBM (32 x 8192 x 1024
//   7.1, 6.5) is lost where it is in a cache already (4.3, 5.3; 192 x 1000 x 2048 6.3, 6.8; but 32 x 8192 x 8192 25.9, 25.1).
//   More than 9/16 of the compute units with a sub-tile leave too few to fetch: 11008 columns in 172 sub-tiles 21.1 us without, 22.4 with.  The
//   columns of an XCD's sub-tiles have to be a run, or every row of sub-tiles would fetch them again: one row, or bands that hold all rows.
// Shape: the smallest ns a stage, the larger of the sub-tile's own cost, of B at 6.2 TB/s and of what the feeders of one XCD need at 2.4 ns a line.
// A takes feeders of its own, so many that a line costs each 4 ns (with K = 8192 every row of A is in the same sets: 128 x 1024 x 8192 with one
// 49 us, two 26, four 14).  Pace: where the sub-tiles are expected, a little slower, as lines that leave the L2 before
// their use cost a sub-tile the 4 ns this is for (32 x 2048 x 16384 without a pace 44 us, with it 25).
// How many: half as many again for B as that pace needs at 2.4 ns a line; the other workgroups leave at once.  The launch ends when the last of these ends, and one
// that starts late, on a compute unit that another stream held, still takes its time.  With all of them at it: 16 x 2048 x 8192 13.5 us, 13.2 with as many as
// needed; with 32, 64 and 224 compute units held by another kernel 19.7, 22.4, 82, now 13.5, 13.7, 64 (without feeders 33, 33, 50); 192 x 64 x 8192 13.5 and, 32
// held, 19.6, now 12.7 and 12.8 (16); 160 x 1000 x 16384 45, now 34.5 (60).  With twice the need as with one and a half, with the need itself 15.0 at 16 x 2048 x 8192.
// Held half of the chip: 32 x 8192 x 8192 68 us without feeders, 55 with; 64 x 4096 x 8192 55, 39; 8 x 4096 x 4096 17.4, 18.8; 32 x 4096 x 16384 73, 82; held 192
// and more 0.66 to 1.28 times the time without, 192 x 64 x 8192 1.9.
// Measured on 62 products the rule takes out of 77 with M up to 192 and K from 2048 (4096 above 128 rows), log-uniform, kernel time with over without: 0.32 to 0.99, on
// average 0.63, with the operands out of HBM, as a program's weights come; repeated on operands that stay in a cache 0.62 to 1.25, on average 0.93 (the worst of 320
// products with K from 2048: 1 x 8192 x 2048 5.2 us without, 6.8 with, 10.4 and 8.8 out of HBM; 128 x 2048 x 4096 8.5, 9.5, out of HBM 18.5 and 10.8).
inline bool feed_launch(int64_t M, int64_t N, int64_t K, const swz_params& r, int mode, int cus, GemmLaunch* l) {
  if (M > 192 || K < (M <= 128 ? 2048 : 4096) || r.bm != 128 || r.num_xcd > cus) return false;
  int64_t best = 0;
  l->sub = -1;
  for (int s = 0; s < kSubTileCount; ++s) {
    const SubTile& t = kSubTiles[s];
    const int64_t gm = (M + t.bm - 1) / t.bm, gn = (N + t.bn - 1) / t.bn;
    const bool runs = gm == 1 || (swz_mode_renumbers(mode) && swz_mode_grouped(mode) && (int64_t)r.group_m * (r.bm / t.bm) >= gm);
    if (t.fed_ns == 0 || !runs || 16 * gm * gn > 9 * cus || (t.bm == 64 && M <= 32)) continue;
    const int64_t stage = N * 2 % 128 == 0 ? t.fed_ns : t.fed_ns * 23 / 20;        // columns that start inside a line: more lines
    const int64_t memory = kStageK * N * 2 / 6200, own = stage > memory ? stage : memory;
    if (stage != t.fed_ns && memory > stage) continue;                             // 3 x 7824 x 3424 13.3 us without, 13.8 with
    const int64_t a_feeders = (4 * M + own - 1) / own, idle = cus / r.num_xcd - (gm * gn + r.num_xcd - 1) / r.num_xcd;        // of one XCD
    if (idle < 2 * a_feeders) continue;
    const int64_t lines = (gn + r.num_xcd - 1) / r.num_xcd * t.bn / 64, feed = kStageK * lines * 12 / 5 / (idle - a_feeders);
    const int64_t e = feed > own ? feed : own;
    if (l->sub >= 0 && (e > best || (e == best && t.fed_ns > kSubTiles[l->sub].fed_ns))) continue;
    const double both = (double)memory / (double)stage, pace = (double)stage * sqrt(sqrt(1.0 + both * both * both * both));
    best = e;
    l->sub = s;
    l->bm = t.bm;
    l->bn = t.bn;
    l->grid_m = l->group_m = (int)gm;
    l->grid_n = (int)gn;
    l->blocks = cus;
    l->a_feeders = (int)a_feeders;
    // whole lines: two sub-tiles of 32 columns share one
    const int64_t need = (kStageK * ((gn + r.num_xcd - 1) / r.num_xcd * t.bn + 63) / 64 * 18 / 5 + own - 1) / own;
    l->b_feeders = (int)(need < idle - a_feeders ? need : idle - a_feeders);
    l->feed_ticks = (int)((pace > (double)e ? pace : (double)e) * 1.6);
  }
  return l->sub >= 0;
}

// Whether tiles of 128x256, two to a compute unit (gemm_pair_kernel.h), compute it instead of 256x256 ones and what choose_subtile puts in their place.  Time of the
// pair over that without, 640 products of K from 64 to 2048, log-uniform; where there are two figures, operands and C out of HBM, then out of the memory-side cache:
//   More than half a round of 256x256 tiles: K up to 160 0.70 to 0.97 and 0.66 to 0.97, up to 352 where rows of C end on 64 bytes 0.71 to 1.00 and 0.72 to 0.98 (3976 x 2744 x 336 16.1 us,
//   14.9); then level and worse, as the tiles move half as many bytes again into LDS: 384 1.06, 504 to 576 1.00 to 1.13, 1024 1.05 to 1.12, 2048 1.20.
//   K from 168 to 352, rows of C that end inside 64 bytes: 0.82 to 1.17, on average 0.96, and 0.78 to 1.13, on average 0.90.  Out of HBM wide C (5 M <= 2 N) loses where 256x256 tiles fill
//   their rounds: 1117 x 12176 x 296 18.9 us, 22.2 (out of the cache 14.9, 13.8), 2660 x 14000 x 192 33.4, 36.9 (30.1, 25.2), 3215 x 15064 x 240 47.9, 51.8 (44.3, 42.4); of 53 such
//   products 1.01 on average there and 0.90 out of the cache (the worst of both 4327 x 14440 x 248, 1.02 and 1.13), so they stay.
//   One and a quarter to one and a half rounds, which the finer tiles fill better: K = 400 0.87 to 0.97, 448 0.94 to 1.00, 512 0.94 to 1.02, 640 0.99 to 1.09 (up to one and
//   a quarter, whose last tiles go in quarters: K = 400 0.97 to 1.01, 512 1.03 to 1.08); 1620 x 11600 x 432 1.10 and 0.94.
//   Renumbered without bands, where B comes from the memory-side cache again and again: K up to 304 0.71 to 1.07, on average 0.92 (4789 x 16256 x 192 61 us, 65), 8192 x 8192 x 344 1.03;
//   round robin 0.63 to 1.12, on average 0.89 (9099 x 15104 x 216 121 us, 136).
//   Half a round of tiles or less, where smaller sub-tiles are at work: 0.98 to 2.4.
//   Fewer columns than half a tile: 100000 x 64 x 64 12.9 us, 8.8, x 304 18.3, 22.7; 65537 x 136 x 304 21.6, 19.2; few rows: 64 x 100000 x 304 16.3, 14.4.
inline bool pair_wins(int64_t N, int64_t K, const swz_params& r, int64_t tiles, int mode, int cus) {
  if (r.bm != 256 || r.bn != 256 || 2 * tiles <= cus || (N < 128 && K > 128)) return false;
  if (4 * tiles > 5 * cus && 2 * tiles <= 3 * cus) return K <= 448;
  return K <= (swz_mode_renumbers(mode) && !swz_mode_grouped(mode) ? 304 : 352);
}

// r: the resolved plan; cus: compute units.  `free_tile`: the caller left the tile to the library, otherwise a tile is one workgroup.
// Bounds for anything else: 32-bit source offsets over 64 rows of B, and a grid well inside the 32-bit range whatever the shape.
inline GemmLaunch gemm_launch(int64_t M, int64_t N, int64_t K, const swz_params& r, int grid_m, int grid_n, int group_m, int mode, bool free_tile, int cus) {
  GemmLaunch l = {-1, false, r.bm, r.bn, grid_m, grid_n, group_m, 0, 1, (int64_t)grid_m * grid_n, false, 0, 0, 0};
  if (!free_tile || N >= ((int64_t)1 << 24) || l.blocks >= ((int64_t)1 << 16)) return l;
  if (feed_launch(M, N, K, r, mode, cus, &l)) return l;
  if (pair_wins(N, K, r, l.blocks, mode, cus)) {
    l.pair = true;
    l.bm = 128;
    l.bn = 256;
    l.grid_m = (int)((M + l.bm - 1) / l.bm);
    l.grid_n = (int)((N + l.bn - 1) / l.bn);
    l.blocks = (int64_t)l.grid_m * l.grid_n;
    const int64_t band = (int64_t)group_m * (r.bm / l.bm);         // as high as a band of the plan's tiles
    l.group_m = (int)(band < l.grid_m ? band : l.grid_m);
    return l;
  }
  l.sub = choose_subtile(M, N, K, r, cus);
  if (l.sub >= 0) {
    const SubTile& s = kSubTiles[l.sub];
    l.bm = s.bm;
    l.bn = s.bn;
    l.grid_m = (int)((M + s.bm - 1) / s.bm);
    l.grid_n = (int)((N + s.bn - 1) / s.bn);
    l.blocks = (int64_t)l.grid_m * l.grid_n;
    const int64_t band = r.bm < s.bm ? group_m : (int64_t)group_m * (r.bm / s.bm);   // rows of sub-tiles, as high as a band of tiles
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
  if (!l.pieces && w >= l.grid_m * l.grid_n) return {0, 0, 0, 0};             // fetches ahead
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
