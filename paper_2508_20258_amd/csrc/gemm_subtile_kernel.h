// Tiled bf16 GEMM for gfx950 for products that the large tiles of gemm_kernel.h leave the chip idle or
// waiting on: few rows, few columns, small grids.  Same operands, layouts, fragments and K order as there (one chain
// of v_mfma_f32_16x16x32_bf16 per element, k ascending), hence the same bits; what differs is how much of C a
// workgroup owns and how the K loop is fed.
//
// Whole tiles are bound by latency here: a 256 x 256 or 128 x 128 tile leaves 64 to 250 of 256 CUs without work, and with
// three K steps of look-ahead (0.3 us) a tile that has its CU to itself waits for most of its operands.  Hence
//   * sub-tiles: workgroups of 32x32 to 128x256 elements of C, in a raster as fine as they are;
//   * a ring of 3 to 8 stages, 64 of K each, fetched global -> LDS as far ahead as the LDS allows (12 and 16 stages of the
//     small shapes were no faster than 6 and 8, which leave room for a second workgroup on the CU);
//   * one barrier per stage, and two sets of fragments: the reads of one half of a stage (32 of K) are issued
//     between the MFMAs of the other half, the barrier falls between the two.  Measured against reading a whole
//     stage, then multiplying it: 128x128 at 2048^3 21.7 -> 18.8 us, 64x64 at 1024^3 6.3 -> 6.2 us;
//   * every slot address a compile-time constant (the loop is unrolled over the ring, base pointers advance by additions):
//     with slots computed at run time the scalar instructions of a stage alone took 200 ns, a third more than the whole of a
//     32x32 stage now (512^3 4.6 -> 3.9 us).
// What bounds them now is the loads.  In working copies, us a launch with the operands out of HBM and out of a cache: 2048^3 (128x128) 23.2 and 19.2; loads alone, without
// MFMAs and fragment reads, 22.1 and 15.3; without MFMAs 22.2, 15.8; without fragment reads 22.3, 16.0; without loads 15.1, 14.9.  1024x1024x4096 (64x64) 22.6 and 15.2,
// loads alone 22.3 and 14.4, without loads 9.8 and 9.3.  A stage of 128x128 takes 560 ns out of HBM and 454 out of a cache (the slope from K = 2048 to 8192 at
// 2048 x 2048), loads alone 540 and 349: a full chip moves 15 and 19 TB/s, alone 15.5 and 24, from the L2s to LDS.  The LDS is not the bound out of HBM
// (4 % without the fragment reads; 22 % of the clocks at 2048^3 by its counter).  A product of few rows waits for its column stripes out of HBM, unless other workgroups fetch them ahead (fetch_ahead).  One barrier per two stages instead of one was no faster (32x8192x8192 28.9 -> 35.9 us).
// Measured (kernel time, operands not in cache; 128x128, 128x256 or 256x256 tiles of gemm_kernel.h -> sub-tiles, the
// shape the rule in gemm_dispatch.h takes; fed: with feeders):
//   512^3            8.1 ->  4.0 us (32x32)      1024^3          12.6 ->  6.2 us (64x64)
//   1536^3          17.0 -> 13.2 us (128x128)    2048^3          21.9 -> 19.0 us (128x128)
//   8x4096x4096     32.2 -> 17 -> 9.0 us (32x32, fed)          32x8192x8192    66.5 -> 40.4 -> 26 us (32x64, fed; reading B takes 21 at 6.3 TB/s)
//   256x2048x2048   19.0 ->  9.0 us (32x64)      1024x2048x4096  33.2 -> 23.1 us (128x64)
//   128x32768x2048  40.6 -> 29.4 us (128x128)    64x65536x4096  118.3 -> 96.8 us (64x128)
//   4575x1112x576   13.1 -> 10.7 us (192x128)    940x2816x12696   136 -> 116 us (96x128)   [against the sub-tiles without these two shapes]
//
// LDS of a stage: A, BM rows x 64 of K (128 bytes, chunk c of row r in slot c ^ ((r >> 1) & 7)), then B, 64 rows x
// BN columns (chunk c of row k in slot c ^ sub_b_key(k)); both conflict-free for the fragment reads.
// Rows >= M and columns >= N are fetched from clamped addresses, chunks with k >= K from a block of zeros.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_dispatch.h"
#include "gemm_kernel.h"
#include "pid_decode.h"

namespace swz {

template <int BM_, int BN_, int WM_, int WN_, int STAGES_>
struct SubShape {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, STAGES = STAGES_;
  static constexpr int NW = WM * WN, NT = NW * 64;
  static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  static constexpr int A_BYTES = BM * kStageK * 2, B_BYTES = kStageK * BN * 2;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int B_ROW_CHUNKS = BN / 8;
  static constexpr int A_LOADS = A_BYTES / (NT * 16), B_LOADS = B_BYTES / (NT * 16);
  static constexpr int LOADS = A_LOADS + B_LOADS;               // per thread and stage
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
  static_assert(BM % (WM * 16) == 0 && BN % (WN * 16) == 0, "wave tiling");
  static_assert(A_BYTES % (NT * 16) == 0 && B_BYTES % (NT * 16) == 0, "load tiling");
  static_assert((STAGES - 1) * LOADS < 64, "loads in flight per wave: the counter has six bits");
  static_assert(LDS_BYTES <= 160 * 1024 && STAGES >= 3, "LDS per workgroup");
};

// XOR key of row k of a B stage (applied to 16-byte chunk indices, whole 32-byte pairs): the 8 rows a half-wave
// of transposing reads touches (k mod 16 in 0..3 and 8..11) land in 8 different 32-byte bank groups.
template <int BN>
__device__ __forceinline__ int sub_b_key(int k) {
  if constexpr (BN >= 128) return b_key(k);
  else if constexpr (BN == 64) return (((k >> 1) & 1) | (((k >> 3) & 1) << 1)) << 1;
  else return ((k >> 3) & 1) << 1;
}

template <class S>
__device__ __forceinline__ void gemm_subtile(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                             uint16_t* __restrict__ C, int M, int N, int K, int m0, int n0,
                                             unsigned char* smem) {
  constexpr int BM = S::BM, BN = S::BN, TM = S::TM, TN = S::TN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave / S::WN, wn = wave % S::WN;

  uint32_t a_off[S::A_LOADS], b_off[S::B_LOADS];
#pragma unroll
  for (int i = 0; i < S::A_LOADS; ++i) {
    const int q = (wave * S::A_LOADS + i) * 64 + lane;
    const int row = q >> 3, c = a_slot(row, q & 7);
    const int r = (m0 + row < M) ? row : (M - 1 - m0);
    a_off[i] = (uint32_t)r * (uint32_t)K * 2u + (uint32_t)c * 16u;
  }
#pragma unroll
  for (int i = 0; i < S::B_LOADS; ++i) {
    const int q = (wave * S::B_LOADS + i) * 64 + lane;
    const int krow = q / S::B_ROW_CHUNKS, c = (q % S::B_ROW_CHUNKS) ^ sub_b_key<BN>(krow);
    const int col = (n0 + c * 8 < N) ? c * 8 : (N - 8 - n0);
    b_off[i] = (uint32_t)krow * (uint32_t)N * 2u + (uint32_t)(col * 2);
  }
  const unsigned char* a_tile = reinterpret_cast<const unsigned char*>(A + (size_t)m0 * K);
  const unsigned char* b_tile = reinterpret_cast<const unsigned char*>(B + n0);
  const unsigned char* zero = reinterpret_cast<const unsigned char*>(&kZeroChunk);
  const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const size_t b_stage = (size_t)kStageK * N * 2;

  const uint32_t a_dst = smem_addr + (uint32_t)wave * (S::A_LOADS * 1024);
  const uint32_t b_dst = smem_addr + S::A_BYTES + (uint32_t)wave * (S::B_LOADS * 1024);
  const unsigned char *a_next = a_tile, *b_next = b_tile;      // where the next stage to fetch starts
  auto load_full = [&](uint32_t slot_off) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < S::B_LOADS; ++i) load_to_lds_base_off(b_next, b_off[i], b_dst + slot_off + i * 1024);
#pragma unroll
    for (int i = 0; i < S::A_LOADS; ++i) load_to_lds_base_off(a_next, a_off[i], a_dst + slot_off + i * 1024);
    a_next += kStageK * 2;
    b_next += b_stage;
  };
  auto load_tail = [&](int k_left, uint32_t slot_off) __attribute__((always_inline)) {     // k_left < kStageK of K are left
#pragma unroll
    for (int i = 0; i < S::B_LOADS; ++i) {
      const int krow = ((wave * S::B_LOADS + i) * 64 + lane) / S::B_ROW_CHUNKS;
      load_to_lds(krow < k_left ? b_next + b_off[i] : zero, b_dst + slot_off + i * 1024);
    }
#pragma unroll
    for (int i = 0; i < S::A_LOADS; ++i) {
      const int q = (wave * S::A_LOADS + i) * 64 + lane;
      load_to_lds(a_slot(q >> 3, q & 7) * 8 < k_left ? a_next + a_off[i] : zero, a_dst + slot_off + i * 1024);
    }
  };
  auto load_any = [&](int t, uint32_t slot_off) __attribute__((always_inline)) {
    if ((t + 1) * kStageK <= K) load_full(slot_off);
    else load_tail(K - t * kStageK, slot_off);
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  typedef __attribute__((address_space(3))) const bf16x8* lds_a_ptr;
  typedef __attribute__((address_space(3))) s16x4* lds_b_ptr;
  const int a_row0 = wm * (TM * 16) + (lane & 15);
  const int b_krow0 = 8 * (lane >> 4) + ((lane & 15) >> 2);
  uint32_t a_rd[2], b_rd[TN];
#pragma unroll
  for (int h = 0; h < 2; ++h) a_rd[h] = smem_addr + (uint32_t)a_lds_off(a_row0, (lane >> 4) + 4 * h);
#pragma unroll
  for (int bj = 0; bj < TN; ++bj) {
    const int col = wn * (TN * 16) + 4 * (lane & 3) + 16 * bj;
    b_rd[bj] = smem_addr + (uint32_t)(S::A_BYTES + b_krow0 * (BN * 2) + (((col >> 3) ^ sub_b_key<BN>(b_krow0)) << 4) + (col & 7) * 2);
  }
  // Two sets of fragments, one per half of a stage: while the MFMAs of one half run, the other half's fragments
  // are on their way.
  bf16x8 af[2][TM];
  s16x4 bq[2][TN][2];
  auto read_half = [&](auto half, uint32_t base) __attribute__((always_inline)) {          // base: byte offset of the stage's slot
    constexpr int H = decltype(half)::value;
#pragma unroll
    for (int bj = 0; bj < TN; ++bj)
#pragma unroll
      for (int hi = 0; hi < 2; ++hi)
        bq[H][bj][hi] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_b_ptr)(uintptr_t)(b_rd[bj] + base + (uint32_t)((32 * H + 4 * hi) * BN * 2)));
#pragma unroll
    for (int bi = 0; bi < TM; ++bi) af[H][bi] = *(lds_a_ptr)(uintptr_t)(a_rd[H] + base + (uint32_t)bi * 2048u);
  };
  auto multiply_half = [&](auto half) __attribute__((always_inline)) {
    constexpr int H = decltype(half)::value;
#pragma unroll
    for (int bi = 0; bi < TM; ++bi)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int bj = (bi & 1) ? TN - 1 - j : j;
        const bf16x8 b = __builtin_bit_cast(bf16x8, __builtin_shufflevector(bq[H][bj][0], bq[H][bj][1], 0, 1, 2, 3, 4, 5, 6, 7));
        acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, af[H][bi], acc[bi][bj], 0, 0, 0);
      }
  };
  auto interleave = [&]() __attribute__((always_inline)) {
    constexpr int NM = TM * TN, NR = TM + 2 * TN, PER = (NR + NM - 1) / NM;
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);        // one MFMA
      if (i * PER < NR) __builtin_amdgcn_sched_group_barrier(0x100, PER, 0);   // then the reads that go with it
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::integral_constant<int, 0> kLow{};
  constexpr std::integral_constant<int, 1> kHigh{};

  const int T = (K + kStageK - 1) / kStageK, full = K / kStageK;
  constexpr int AHEAD = S::STAGES - 1;                           // stages fetched ahead of the one being multiplied
  for_each_index([&](auto i) __attribute__((always_inline)) {
    if (decltype(i)::value < T) load_any(decltype(i)::value, decltype(i)::value * S::STAGE_BYTES);
  }, std::make_integer_sequence<int, AHEAD>{});
  auto publish = [&](auto newer) __attribute__((always_inline)) {          // newer: stages issued after the one waited for
    wait_vmcnt<decltype(newer)::value * S::LOADS>();
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  for_each_index([&](auto i) __attribute__((always_inline)) {    // stage 0 has landed; min(T, AHEAD) were issued
    constexpr int NEWER = AHEAD - 1 - decltype(i)::value;
    if (NEWER == 0 ? T == 1 : NEWER == AHEAD - 1 ? T > NEWER : T == NEWER + 1) wait_vmcnt<NEWER * S::LOADS>();
  }, std::make_integer_sequence<int, AHEAD>{});
  __builtin_amdgcn_sched_barrier(0);
  block_barrier();
  __builtin_amdgcn_sched_barrier(0);
  read_half(kLow, 0);
  int t = 0;
  // whole turns of the ring: every slot is a compile-time constant
  for (; t + S::STAGES + AHEAD <= full; t += S::STAGES)
    for_each_index([&](auto pos) __attribute__((always_inline)) {
      constexpr int P = decltype(pos)::value;
      read_half(kHigh, P * S::STAGE_BYTES);
      multiply_half(kLow);
      interleave();
      publish(std::integral_constant<int, AHEAD - 2>{});
      load_full(((P + AHEAD) % S::STAGES) * S::STAGE_BYTES);
      __builtin_amdgcn_sched_barrier(0);
      read_half(kLow, ((P + 1) % S::STAGES) * S::STAGE_BYTES);
      multiply_half(kHigh);
      interleave();
    }, std::make_integer_sequence<int, S::STAGES>{});
  uint32_t off = 0, off_ld = AHEAD * S::STAGE_BYTES;
  auto next_slot = [](uint32_t o) __attribute__((always_inline)) { return o == AHEAD * S::STAGE_BYTES ? 0u : o + S::STAGE_BYTES; };
  for (; t + AHEAD < T; ++t) {
    read_half(kHigh, off);
    multiply_half(kLow);
    interleave();
    publish(std::integral_constant<int, AHEAD - 2>{});
    load_any(t + AHEAD, off_ld);
    __builtin_amdgcn_sched_barrier(0);
    off = next_slot(off);
    off_ld = next_slot(off_ld);
    read_half(kLow, off);
    multiply_half(kHigh);
    interleave();
  }
  // the last stages: nothing left to fetch, one stage fewer in flight each time
  for_each_index([&](auto i) __attribute__((always_inline)) {
    constexpr int LEFT = AHEAD - 1 - decltype(i)::value;         // stages after this one
    if (LEFT < T) {
      read_half(kHigh, off);
      multiply_half(kLow);
      interleave();
      if constexpr (LEFT > 0) {
        publish(std::integral_constant<int, LEFT - 1>{});
        off = next_slot(off);
        read_half(kLow, off);
      }
      multiply_half(kHigh);
      if constexpr (LEFT > 0) interleave();
    }
  }, std::make_integer_sequence<int, AHEAD>{});
  store_wave_tile<TM, TN>(acc, C, M, N, m0 + wm * (TM * 16), n0 + wn * (TN * 16), lane);
}

// What a workgroup without a sub-tile does: it reads B, or A, in the order of K ahead of the workgroups of its XCD, into LDS that nobody
// reads, so that their loads find the lines in the L2.  No result depends on it, but the launch ends when the last of these ends: they keep to the pace at which the
// sub-tiles are expected from when they start, and no more of them run than that pace needs (feed_launch says what it costs where they start late).
// A CU that reads a column stripe gets one line of it from HBM every 3 to 4 ns, whatever the stripe's width, the loads in flight, their
// order or the number of CUs that do so (plain reads of 8192 rows: 24.5 us, 33 where the pitch is a power of two), and a
// sub-tile needs all K of them: a product of few rows took K x 4 ns however narrow B is.  From the L2 a line takes about 1 ns, and
// the CUs without a sub-tile read rows in pieces as wide as their XCD's columns, at 2.3 ns a line each and 6 TB/s together.
// K can not be cut instead: the order of the sums is part of the contract.  Measured (kernel time, operands not in cache, without -> with):
//   32x8192x8192   40 -> 26 us (HBM: 21)     32x4096x16384  76 -> 29     64x4096x8192   36 -> 18.7    8x4096x4096  17 -> 9.0
//   128x1024x8192  31 -> 13.4                16x2048x8192   33 -> 13.2   160x1000x16384 60 -> 34.5    192x64x8192  16 -> 12.8
// In LDS of 90 KB a workgroup, one to a CU by force, the times are the same.
template <class S>
__device__ __forceinline__ void fetch_ahead(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, int M, int N, int K, int grid_m,
                                            int grid_n, int num_xcd, int mode, int a_feeders, int b_feeders, int feed_ticks, unsigned char* smem) {
  constexpr int CHUNKS = S::BN / 8;                               // 16-byte chunks of a row of B per sub-tile
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int total = grid_m * grid_n, x = (int)blockIdx.x % num_xcd;
  const int workers = x < total ? (total - 1 - x) / num_xcd + 1 : 0;      // of this XCD, like the feeders
  const int mine = (int)blockIdx.x / num_xcd - workers, left = ((int)gridDim.x - 1 - x) / num_xcd + 1 - workers;
  const int feeders = left < a_feeders + b_feeders ? left : a_feeders + b_feeders;
  if (workers == 0 || mine >= feeders) return;
  // the columns of sub-tiles on this XCD: first, first + stride, ...
  const bool run = swz_mode_renumbers(mode);
  const int s0 = run ? swz_xcd_renumber(x, total, num_xcd) : x;
  const int first = run ? s0 / grid_m : x, stride = run ? 1 : num_xcd;
  const int cols = run ? (s0 + workers - 1) / grid_m - first + 1 : workers;
  const uint32_t dst = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + (uint32_t)wave * 1024u;
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  const int lead = kFeedLead / (cols * S::BN * 2);
  int loads = 0;
  auto pace = [&](int k) __attribute__((always_inline)) {
    wait_vmcnt<15>();
    if ((loads++ & 7) != 0) return;
    const uint64_t due = k > lead ? t0 + (uint64_t)(uint32_t)(k - lead) * (uint32_t)feed_ticks / 1024u : t0;
    while (__builtin_amdgcn_s_memrealtime() < due) __builtin_amdgcn_s_sleep(4);
  };
  if (mine >= feeders - a_feeders) {                              // A: 256 of K of two rows a load
    const int pairs = (M + 1) / 2, spans = (K + 255) / 256;
    for (int f = (mine - (feeders - a_feeders)) * S::NW + wave; f < pairs * spans; f += a_feeders * S::NW) {
      const int span = f / pairs;
      int row = 2 * (f - span * pairs) + (lane >> 5), k = span * 256 + (lane & 31) * 8;
      if (row >= M) row = M - 1;
      if (k >= K) k = K - 8;
      pace(span * 256);
      load_to_lds(A + (size_t)row * K + k, dst);
    }
  } else {
    // B: 64 chunks a load, row by row of the XCD's columns.  The loads of all waves together are whole rows, so that a wave's lanes keep their columns
    // and a load is one addition: with the columns found anew for each the feeders brought 3.5 TB/s.
    const int row_chunks = cols * CHUNKS;
    int unit = cols;
    for (int n = 64 / CHUNKS; n > 1 && unit % 2 == 0; n /= 2) unit /= 2;
    const int waves = (feeders - a_feeders) * S::NW, team = waves - waves % unit, q = mine * S::NW + wave;
    if (q >= team) return;
    int k = q * 64 / row_chunks;
    const int c0 = q * 64 - k * row_chunks, e = c0 + lane, lrow = e / row_chunks, c = e - lrow * row_chunks;
    const int col = (first + c / CHUNKS * stride) * S::BN + c % CHUNKS * 8;
    const uint32_t off = (uint32_t)lrow * (uint32_t)N * 2u + (uint32_t)(col < N ? col : N - 8) * 2u;
    const int rows = (c0 + 63) / row_chunks + 1, step = team * 64 / row_chunks;
    const unsigned char* src = reinterpret_cast<const unsigned char*>(B) + (size_t)k * N * 2;
    const size_t src_step = (size_t)step * N * 2;
    for (; k + rows <= K; k += step) {
      pace(k);
      load_to_lds_base_off(src, off, dst);
      src += src_step;
    }
  }
  wait_vmcnt<0>();
}

// One workgroup per sub-tile.  The raster and the renumbering are those of a tile grid, over the grid of sub-tiles
// (bands of as many rows of C): every XCD gets its share of them to within one.  Dealing whole tiles of the plan instead, with their
// sub-tiles on one XCD, left some XCDs with more than 32 for their 32 CUs, and sub-tiles beyond C that leave at once
// do not free the place they were dealt: 4352x416x6272 in 128x64 sub-tiles took 74 us that way.
template <class S>
__global__ __launch_bounds__(S::NT) void gemm_bf16_subtile_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                                  uint16_t* __restrict__ C, int M, int N, int K, int grid_m,
                                                                  int grid_n, int num_xcd, int group_m, int mode, int a_feeders,
                                                                  int b_feeders, int feed_ticks) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if ((int)blockIdx.x >= grid_m * grid_n) {                       // uniform
    fetch_ahead<S>(A, B, M, N, K, grid_m, grid_n, num_xcd, mode, a_feeders, b_feeders, feed_ticks, smem);
    return;
  }
  int pm, pn;
  swz_decode_tile((int)blockIdx.x, grid_m, grid_n, num_xcd, group_m, mode, &pm, &pn);
  gemm_subtile<S>(A, B, C, M, N, K, pm * S::BM, pn * S::BN, smem);
}

// Whole tiles (S) for hardware ids below `whole`, a multiple of the compute units; the tiles of the last, partial round
// in sub-tiles (P) behind them, so that the round lasts as long as a sub-tile and not as long as a tile.  One launch: the first
// sub-tiles start where the first whole tiles end.  Which id gets which piece: swz_tail_piece.  From as many left-over tiles as XCDs
// on, a tile's pieces run on the XCD the map gives the tile and share its operand panels in its L2; fewer tiles are
// spread (on one XCD each, with ids that leave at once between them: 2 x 131 tiles of K = 4096 120.9 us against 119.8, 7 x 37 114.3
// against 114.6).  At most half a round of tiles is left over, in halves, or a quarter, in quarters, so no XCD gets more
// than it has CUs.  Ids past the last tile and sub-tiles outside C leave at once.
template <class S, class P>
__global__ __launch_bounds__(S::NT) void gemm_bf16_tail_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                               uint16_t* __restrict__ C, int M, int N, int K, int grid_m, int grid_n,
                                                               int num_xcd, int group_m, int mode, int whole, int deal) {
  static_assert(S::NT == P::NT && S::BM % P::BM == 0 && S::BN % P::BN == 0, "one block size, pieces that fill a tile");
  constexpr int SUB_M = S::BM / P::BM, SUBS = SUB_M * (S::BN / P::BN);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int w = (int)blockIdx.x;
  int pm, pn;
  if (w < whole) {
    swz_decode_tile(w, grid_m, grid_n, num_xcd, group_m, mode, &pm, &pn);
    gemm_tile<S>(A, B, C, M, N, K, pm, pn, false, false, 0, 0, smem);
  } else {
    int v, sub;
    if (!swz_tail_piece(w, whole, deal, SUBS, grid_m * grid_n, &v, &sub)) return;       // uniform, like the exit below
    swz_decode_tile(v, grid_m, grid_n, num_xcd, group_m, mode, &pm, &pn);
    const int m0 = pm * S::BM + (sub % SUB_M) * P::BM, n0 = pn * S::BN + (sub / SUB_M) * P::BN;
    if (m0 >= M || n0 >= N) return;
    gemm_subtile<P>(A, B, C, M, N, K, m0, n0, smem);
  }
}

}  // namespace swz
