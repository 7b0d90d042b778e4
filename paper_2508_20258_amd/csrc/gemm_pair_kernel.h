// Tiled bf16 GEMM for gfx950 for large products of a short K: tiles of 128 x 256, two workgroups to a compute unit.
//
// Writing C takes as long as multiplying here (K = 256: 0.32 ps an element at 6.3 TB/s, 0.33 at 1.55 PFLOP/s), and a 256 x 256 tile alone on its compute unit
// does the two, and the wait for its first operands, one after the other.  Its persistent form does not lay them over each other either: loads and
// stores share one counter, and the loads of the next tile that follow the stores are waited for with them (8192 x 8192 x 128 43 us).  Two workgroups that share
// nothing run out of step by themselves: one's stores and first loads under the other's products.  Eight waves of 64 x 64 take 105 registers, so that sixteen
// fit, and a ring of three stages of 32 of K is 72 KB of the 160.  Each element is the same chain of v_mfma_f32_16x16x32_bf16 over ascending k as
// in gemm_kernel.h, hence the same bits.
// Measured (us, operands not in cache; 256x256 tiles of gemm_kernel.h -> here; fill_ of C alone):
//   8192x8192x128   46.5 -> 35.6 (21.2)    16384x16384x64  146 -> 111 (78)    10347x3752x240  36.1 -> 29.8 (12.9)
//   8192x8192x256   57.7 -> 48.0           16384x8192x256  107 -> 89 (40)     13383x6792x272   100 -> 87
// What bounds it: the loads into LDS and the stores still add up, 16 TB/s (the slope over K) and the time C alone takes (the intercept, 24 us at 8192 x 8192).
// Other shapes, us at 8192x8192x128, 8192x8192x256, 10347x3752x240: four waves of 128x64 35.9, 49.3, 31.8; 256x128 in such waves 37.6, 52.2, 33.0; 128x128 in four
// waves of 64x64, three to a compute unit, 34.2, 49.5, 35.9 (a third more bytes into LDS).
//
// LDS of a stage: A, 128 rows x 32 of K (64 bytes, chunk c of row r in slot c ^ ((r >> 2) & 3)), then B, 32 rows x 256 columns as in gemm_kernel.h.  Reads of B are free of
// conflicts.  Of A two of every eight lanes meet in a bank, a third of the clocks the LDS is in use by its counter; it is not what bounds the kernel: the key that avoids
// it, (r >> 1) & 3, was 1 % faster to 3 % slower over 13 products (8192x8192x128 36.2 us, 37.0).
// Rows >= M and columns >= N are fetched from clamped addresses, chunks with k >= K from a block of zeros.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_kernel.h"
#include "pid_decode.h"

namespace swz {

struct PairShape {
  static constexpr int BM = 128, BN = 256, WM = 2, WN = 4, NW = WM * WN, NT = NW * 64, STAGES = 3;
  static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  static constexpr int A_BYTES = BM * kStepK * 2, B_BYTES = kStepK * BN * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int A_LOADS = A_BYTES / (NT * 16), B_LOADS = B_BYTES / (NT * 16), LOADS = A_LOADS + B_LOADS;   // per thread and stage
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
  static_assert(A_BYTES % (NT * 16) == 0 && B_BYTES % (NT * 16) == 0, "load tiling");
  static_assert(2 * LDS_BYTES <= 160 * 1024, "two workgroups to a compute unit");
};

__device__ __forceinline__ int pair_a_slot(int row, int chunk) { return chunk ^ ((row >> 2) & 3); }

__global__ __launch_bounds__(PairShape::NT, 4) void gemm_bf16_pair_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                                          uint16_t* __restrict__ C, int M, int N, int K, int grid_m, int grid_n,
                                                                          int num_xcd, int group_m, int mode) {
  using S = PairShape;
  constexpr int TM = S::TM, TN = S::TN, ROW_CHUNKS = S::BN / 8;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  int pm, pn;
  swz_decode_tile((int)blockIdx.x, grid_m, grid_n, num_xcd, group_m, mode, &pm, &pn);
  const int m0 = pm * S::BM, n0 = pn * S::BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave / S::WN, wn = wave % S::WN;

  uint32_t a_off[S::A_LOADS], b_off[S::B_LOADS];
  int a_k[S::A_LOADS], b_k[S::B_LOADS];                          // of K, from the start of the stage
#pragma unroll
  for (int i = 0; i < S::A_LOADS; ++i) {
    const int q = (wave * S::A_LOADS + i) * 64 + lane, row = q >> 2, c = pair_a_slot(row, q & 3);
    const int r = m0 + row < M ? row : M - 1 - m0;
    a_k[i] = c * 8;
    a_off[i] = (uint32_t)r * (uint32_t)K * 2u + (uint32_t)c * 16u;
  }
#pragma unroll
  for (int i = 0; i < S::B_LOADS; ++i) {
    const int q = (wave * S::B_LOADS + i) * 64 + lane, krow = q / ROW_CHUNKS, c = (q % ROW_CHUNKS) ^ b_key(krow);
    const int col = n0 + c * 8 < N ? c * 8 : N - 8 - n0;
    b_k[i] = krow;
    b_off[i] = (uint32_t)krow * (uint32_t)N * 2u + (uint32_t)(col * 2);
  }
  const unsigned char* a_next = reinterpret_cast<const unsigned char*>(A + (size_t)m0 * K);        // where the next stage to fetch starts
  const unsigned char* b_next = reinterpret_cast<const unsigned char*>(B + n0);
  const unsigned char* zero = reinterpret_cast<const unsigned char*>(&kZeroChunk);
  const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t a_dst = smem_addr + (uint32_t)wave * (S::A_LOADS * 1024), b_dst = smem_addr + S::A_BYTES + (uint32_t)wave * (S::B_LOADS * 1024);
  const size_t b_stage = (size_t)kStepK * N * 2;
  auto load = [&](int k_left, uint32_t slot) __attribute__((always_inline)) {       // k_left: of K, from this stage on
    if (k_left >= kStepK) {
#pragma unroll
      for (int i = 0; i < S::B_LOADS; ++i) load_to_lds_base_off(b_next, b_off[i], b_dst + slot + i * 1024);
#pragma unroll
      for (int i = 0; i < S::A_LOADS; ++i) load_to_lds_base_off(a_next, a_off[i], a_dst + slot + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < S::B_LOADS; ++i) load_to_lds(b_k[i] < k_left ? b_next + b_off[i] : zero, b_dst + slot + i * 1024);
#pragma unroll
      for (int i = 0; i < S::A_LOADS; ++i) load_to_lds(a_k[i] < k_left ? a_next + a_off[i] : zero, a_dst + slot + i * 1024);
    }
    a_next += kStepK * 2;
    b_next += b_stage;
  };

  typedef __attribute__((address_space(3))) const bf16x8* lds_a_ptr;
  typedef __attribute__((address_space(3))) s16x4* lds_b_ptr;
  const int a_row = wm * (TM * 16) + (lane & 15), b_krow = 8 * (lane >> 4) + ((lane & 15) >> 2);
  const uint32_t a_rd = smem_addr + (uint32_t)(a_row * (kStepK * 2) + (pair_a_slot(a_row, lane >> 4) << 4));
  uint32_t b_rd[TN];
#pragma unroll
  for (int bj = 0; bj < TN; ++bj) {
    const int col = wn * (TN * 16) + 4 * (lane & 3) + 16 * bj;
    b_rd[bj] = smem_addr + (uint32_t)(S::A_BYTES + b_krow * (S::BN * 2) + (((col >> 3) ^ b_key(b_krow)) << 4) + (col & 7) * 2);
  }
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int T = (K + kStepK - 1) / kStepK;
  load(K, 0);
  if (T > 1) load(K - kStepK, S::STAGE_BYTES);
  uint32_t slot = 0, slot_ld = 2 * S::STAGE_BYTES;
  auto next_slot = [](uint32_t s) __attribute__((always_inline)) { return s == (S::STAGES - 1) * S::STAGE_BYTES ? 0u : s + S::STAGE_BYTES; };
  for (int t = 0; t < T; ++t) {
    if (t + 1 < T) wait_vmcnt<S::LOADS>();                       // stage t has landed, t + 1 may be on its way
    else wait_vmcnt<0>();
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();                                             // and every wave is done with the slot that stage t + 2 goes to
    __builtin_amdgcn_sched_barrier(0);
    if (t + 2 < T) load(K - (t + 2) * kStepK, slot_ld);
    bf16x8 af[TM], bf[TN];
#pragma unroll
    for (int bj = 0; bj < TN; ++bj) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_b_ptr)(uintptr_t)(b_rd[bj] + slot));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_b_ptr)(uintptr_t)(b_rd[bj] + slot + (uint32_t)(4 * S::BN * 2)));
      bf[bj] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
#pragma unroll
    for (int bi = 0; bi < TM; ++bi) af[bi] = *(lds_a_ptr)(uintptr_t)(a_rd + slot + (uint32_t)(bi * 16 * kStepK * 2));
#pragma unroll
    for (int bi = 0; bi < TM; ++bi)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int bj = (bi & 1) ? TN - 1 - j : j;
        acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[bj], af[bi], acc[bi][bj], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
    slot = next_slot(slot);
    slot_ld = next_slot(slot_ld);
  }
  store_wave_tile<TM, TN>(acc, C, M, N, m0 + wm * (TM * 16), n0 + wn * (TN * 16), lane);
}

}  // namespace swz
