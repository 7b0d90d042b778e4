// Row softmax and layer normalisation over bf16 rows with a remapped program id (SwizzlePerf,
// Results and Appendix "Case Study: Other Swizzling Pattern Examples": the swizzle found for
// both kernels puts all column chunks of one row on one XCD).
//
// Both are bound by HBM: 4*M*N bytes, x read once and y written once, which needs the row to stay on the
// chip between its statistics and its stores.
//
//   Rows of up to 98304 elements.  TPR threads hold a row in KEEP 16-byte vectors each, in registers: 16 to 64 lanes of a
//   wave for short rows (up to 16 rows per 256-thread workgroup, no LDS, no barrier), a workgroup of 256, 512 or 1024
//   threads for longer ones.  The grid is one-dimensional over groups of consecutive rows, taken in dispatch order.  Where there are more rows
//   than compute units, two forms of the same sums take over for some lengths: two rows beside each other on a compute unit (the *_wide_rows
//   kernels) and, for layer normalisation, a workgroup that takes row after row (layernorm_loop_rows_kernel).
//   Longer rows.  A row is cut into segments of 32768 elements; row_stats_kernel computes the statistics of one segment
//   per workgroup, row_emit_kernel merges them and produces one column chunk per workgroup, reading x a second
//   time.  Between the launches a segment's statistics (8 bytes) wait in `out` itself: every chunk gets its own copy of all of
//   them at its start, so that a workgroup reads only what it overwrites, after its own barrier.  No scratch memory, nothing
//   exchanged inside a launch.  Grids rows x segments and rows x chunks, both decoded by swz_decode_tile: under the
//   XCD renumbering a row's workgroups run back to back on one XCD.  The second launch of a layer normalisation may take its
//   chunks in dispatch order instead (row_dispatch.h).
//
// The decomposition of the paper, in which the workgroup of every column chunk reads the whole row for its statistics, is bound
// by those reads and the arithmetic on them even where the remap has the L2 serve 82 % of them: 8 chunks of
// 1024 x 65536 took 125 us (softmax) and 118 us (layer normalisation), the row in the registers of one workgroup takes 47 and 55.
//
// At 6 TB/s a CU has about 11 vector instructions per element, and a row's latencies stand in series: load, maximum or mean, sum, store.
// So the maximum is taken first, on the raw values, and each exponential computed once and kept (an online maximum costs a
// second one and a rescale); mean and deviations are two passes over registers (a merge of (count, mean, M2) per vector costs a
// division); lanes are reduced with DPP and permlane exchanges (a shuffle through LDS takes about 60 ns a step); gamma and
// beta are requested ahead of the statistics where there are registers for them.  Measured, operands not in cache, online and merging
// kernels with late gamma and beta -> these (us; copy16_kernel on 128 MiB in and out: 43):
//     layernorm 8192 x 8192    66 -> 45      softmax 8192 x 8192    55 -> 44      layernorm 32768 x 16384  388 -> 368
//     softmax 32768 x 16384   382 -> 354     softmax 131072 x 128   49 -> 13      layernorm 300 x 2048     4.9 -> 3.0
//     softmax 64 x 1048576    300 -> 70      softmax 1 x 1048576   220 -> 9       softmax 16 x 131072       29 -> 9
//
// All arithmetic is fp32 on values widened exactly from bf16; results are rounded once to bf16 (nearest even).  How a row is
// accumulated follows from N alone: the bits depend neither on M, nor on the mode, nor on `chunks`.
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pid_decode.h"

namespace swz {

typedef __attribute__((ext_vector_type(4))) uint32_t rw_u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t rw_u32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 rw_bf16x2;

constexpr int kSegThreads = 512;               // threads that share a segment (32768 elements) of a row of more than 98304
constexpr int kSegKeep = 8;                    // 16-byte vectors each of them takes, at most
constexpr int kSegVecs = kSegThreads * kSegKeep;
constexpr int kMaxSegs = (1 << 24) / (kSegVecs * 8);
constexpr int kEmitThreads = 256;              // a column chunk of a longer row: at most 8 vectors a thread, at least half
constexpr int kEmitKeep = 8;                   // of that, so its first 4096 bytes can hold the statistics of all 512 segments
constexpr int kMaxWaves = 16;
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ void rw_unpack(const rw_u32x4& v, float (&x)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[2 * e] = __uint_as_float(v[e] << 16);
    x[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u);
  }
}

__device__ __forceinline__ rw_u32x4 rw_pack(const float (&y)[8]) {
  rw_u32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    rw_bf16x2 h;
    h[0] = (__bf16)y[2 * e];
    h[1] = (__bf16)y[2 * e + 1];
    v[e] = __builtin_bit_cast(uint32_t, h);
  }
  return v;
}

__device__ __forceinline__ float rw_sum8(const float (&x)[8]) {
  return ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
}

__device__ __forceinline__ float rw_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

struct RwMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct RwSum { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };

// op over groups of LANES (16, 32 or 64) lanes; every lane gets the result.  After the two quad steps the
// lanes of a quad agree, so mirroring 8 (then 16) lanes pairs every quad (every 8) with the other one.
template <int LANES, class Op>
__device__ __forceinline__ float rw_reduce_lanes(float x, Op op) {
  auto dpp = [](float v, auto ctrl) __attribute__((always_inline)) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  x = op(x, dpp(x, std::integral_constant<int, 0xB1>{}));        // quad_perm [1,0,3,2]
  x = op(x, dpp(x, std::integral_constant<int, 0x4E>{}));        // quad_perm [2,3,0,1]
  x = op(x, dpp(x, std::integral_constant<int, 0x141>{}));       // row_half_mirror
  x = op(x, dpp(x, std::integral_constant<int, 0x140>{}));       // row_mirror
  if constexpr (LANES >= 32) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(s[0]), __uint_as_float(s[1]));
  }
  if constexpr (LANES >= 64) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(s[0]), __uint_as_float(s[1]));
  }
  return x;
}

// op over the threads that share a row or segment: LANES <= 64 lanes of a wave, or this thread's group of LANES / 64
// waves; `slots` is LDS for one float per wave of the workgroup, not written again before the next barrier.
template <int LANES, class Op>
__device__ __forceinline__ float rw_reduce_group(float x, Op op, float* slots) {
  if constexpr (LANES <= 64) {
    return rw_reduce_lanes<LANES>(x, op);
  } else {
    constexpr int W = LANES / 64;
    x = rw_reduce_lanes<64>(x, op);
    const int wave = (int)threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) slots[wave] = x;
    __syncthreads();
    float g[W];
#pragma unroll
    for (int w = 0; w < W; ++w) g[w] = slots[(wave & ~(W - 1)) + w];
#pragma unroll
    for (int n = W; n > 1; n /= 2)
#pragma unroll
      for (int w = 0; w < n / 2; ++w) g[w] = op(g[2 * w], g[2 * w + 1]);
    return g[0];
  }
}

// exp(x - m), m the largest entry of the row or segment, is computed as exp2(x * scale - shift).  As a rule scale = log2(e) and
// shift = m * log2(e), rounded: one fused multiply-add, and what the rounding of shift takes from every exponent, at most
// 2^-4, leaves with the sum.  That rounding grows with |m| (m = 1e10: 2^328, and the sum is inf).  From 2^20 on the
// bfloat16 numbers next to m are at least 2^12 away, so that only entries equal to m count, and scale = 1, shift = m has
// them at exactly 0 and the others below every exponent, whatever m (-FLT_MAX, of entries that are all -inf, among them).
constexpr float kSoftLarge = 1048576.f;
__device__ __forceinline__ bool soft_large(float m) { return fabsf(m) >= kSoftLarge; }
struct SoftScale {
  float scale, shift;
  __device__ __forceinline__ explicit SoftScale(float m) : scale(soft_large(m) ? 1.f : kLog2e), shift(soft_large(m) ? m : m * kLog2e) {}
};

// What the exponentials of a segment of maximum ms, summed against its own SoftScale, are worth in a row of maximum m >= ms.  Where m
// is small and ms is not, the segment is 2^12 or more below m; its shift, kept from being fused into the difference
// by the fmaxf, is then beside the point.
__device__ __forceinline__ float soft_weight(float ms, float m) {
  return rw_exp2(soft_large(m) ? ms - m : fmaxf(ms * kLog2e, -FLT_MAX) - SoftScale(m).shift);
}

// Of KEEP vectors a thread holds: maximum, sum of exponentials, sum, sum of squared deviations.
template <int KEEP>
__device__ __forceinline__ float held_max(const rw_u32x4* held) {
  float m = -FLT_MAX;
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    float x[8];
    rw_unpack(held[i], x);                                       // vectors past the row's end hold -inf
    m = fmaxf(m, fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7]))));
  }
  return m;
}

__device__ __forceinline__ void soft_exps(const rw_u32x4& v, const SoftScale& base, float (&p)[8]) {
  rw_unpack(v, p);
#pragma unroll
  for (int e = 0; e < 8; ++e) p[e] = rw_exp2(__builtin_fmaf(p[e], base.scale, -base.shift));
}

template <int KEEP>
__device__ __forceinline__ float held_exp_sum(const rw_u32x4* held, const SoftScale& base) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    float p[8];
    soft_exps(held[i], base, p);
    s += rw_sum8(p);
  }
  return s;
}

// Sums of a row are kept in units of 2^17, more than its 98304 elements: a sum of eight that fp32 holds then never grows out of
// it, and powers of two leave every rounding where it was.
constexpr float kSumUnit = 131072.f;
__device__ __forceinline__ float mean_of(float sum, int n) { return sum / ((float)n * (1.f / kSumUnit)); }

// vectors first, first + stride, ... below nv are real, the others hold -inf
template <int KEEP>
__device__ __forceinline__ float held_sum(const rw_u32x4* held, int first, int stride, int nv) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if (first + i * stride < nv) {
      float x[8];
      rw_unpack(held[i], x);
      s = __builtin_fmaf(rw_sum8(x), 1.f / kSumUnit, s);
    }
  return s;
}

__device__ __forceinline__ float dev8(const rw_u32x4& v, float mean) {
  float x[8];
  rw_unpack(v, x);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = (x[e] - mean) * (x[e] - mean);
  return rw_sum8(x);
}

template <int KEEP>
__device__ __forceinline__ float held_dev(const rw_u32x4* held, int first, int stride, int nv, float mean) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if (first + i * stride < nv) s += dev8(held[i], mean);
  return s;
}

constexpr uint32_t kNegInfPair = 0xFF80FF80u;  // two bfloat16 -inf

template <int KEEP, bool STREAM = true>
__device__ __forceinline__ void load_vectors(const rw_u32x4* __restrict__ p, int first, int stride, int nv, rw_u32x4* held) {
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    held[i] = rw_u32x4{kNegInfPair, kNegInfPair, kNegInfPair, kNegInfPair};
    if (first + i * stride < nv) {
      if constexpr (STREAM) held[i] = __builtin_nontemporal_load(p + first + i * stride);
      else held[i] = p[first + i * stride];
    }
  }
}

// Elements of segment s of a row of N.
__device__ __forceinline__ int seg_elems(int s, int N) {
  const int left = N - s * (kSegVecs * 8);
  return left < 0 ? 0 : left < kSegVecs * 8 ? left : kSegVecs * 8;
}

constexpr int row_block(int tpr) { return tpr < 256 ? 256 : tpr; }

// Which row a workgroup of TPR-thread groups works on: TPR <= 64, groups of lanes; above, the whole workgroup.
// Rows held whole share nothing, so no mapping helps the L2, and rows that run at the same time are best neighbours in memory: in
// dispatch order 8192 x 8192 takes 44 us (softmax; layer normalisation in this form 50), with every XCD on a run of rows of its own
// 50 and 56; 65536 x 1024 44 and 45 against 48 and 51, 4000 x 30000 84 and 88 against 88 and 92.  The softmax shape of 1024 threads
// with two vectors each is MAPPED: the host hands it the caller's mode where runs are not slower (soft_rows_mapped in swz.hip).
template <int TPR, bool MAPPED>
struct RowJob {
  static constexpr int THREADS = row_block(TPR);
  int row, tid;
  bool live;                                   // uniform per group of TPR threads; TPR >= 256: per workgroup
  __device__ __forceinline__ RowJob(int M, int num_xcd, int group_m, int mode) {
    constexpr int ROWS = THREADS / TPR;
    int group = (int)blockIdx.x, chunk;
    if constexpr (MAPPED) swz_decode_tile((int)blockIdx.x, (M + ROWS - 1) / ROWS, 1, num_xcd, group_m, mode, &group, &chunk);
    row = group * ROWS + (int)threadIdx.x / TPR;
    tid = (int)threadIdx.x % TPR;
    live = row < M;
  }
};

template <int KEEP, int TPR>
__global__ __launch_bounds__(row_block(TPR)) void softmax_rows_kernel(const uint16_t* __restrict__ in, uint16_t* __restrict__ out,
                                                                           int M, int N, int num_xcd, int group_m, int mode) {
  __shared__ float slots[2][kMaxWaves];
  const RowJob<TPR, TPR == 1024 && KEEP == 2> job(M, num_xcd, group_m, mode);
  if (!job.live) return;
  const int nv = N >> 3, tid = job.tid;
  rw_u32x4 held[KEEP];
  load_vectors<KEEP>(reinterpret_cast<const rw_u32x4*>(in + (size_t)job.row * N), tid, TPR, nv, held);
  const SoftScale base(rw_reduce_group<TPR>(held_max<KEEP>(held), RwMax{}, slots[0]));
  constexpr bool KEEP_EXPS = KEEP <= 8;                          // the exponentials stay in registers where there is room
  float p[KEEP_EXPS ? KEEP : 1][8], s = 0.f;
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    float(&q)[8] = p[KEEP_EXPS ? i : 0];
    soft_exps(held[i], base, q);
    s += rw_sum8(q);
  }
  const float inv = 1.0f / rw_reduce_group<TPR>(s, RwSum{}, slots[1]);
  rw_u32x4* outp = reinterpret_cast<rw_u32x4*>(out + (size_t)job.row * N);
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if (tid + i * TPR < nv) {
      float(&q)[8] = p[KEEP_EXPS ? i : 0];
      if constexpr (!KEEP_EXPS) soft_exps(held[i], base, q);
#pragma unroll
      for (int e = 0; e < 8; ++e) q[e] *= inv;
      __builtin_nontemporal_store(rw_pack(q), outp + tid + i * TPR);
    }
}

__device__ __forceinline__ rw_u32x4 ln_vector(const rw_u32x4& xv, const rw_u32x4& gv, const rw_u32x4& bv, float mean, float rstd) {
  float x[8], g[8], b[8];
  rw_unpack(xv, x);
  rw_unpack(gv, g);
  rw_unpack(bv, b);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = (x[e] - mean) * rstd * g[e] + b[e];
  return rw_pack(x);
}

template <int KEEP, int TPR>
__global__ __launch_bounds__(row_block(TPR)) void layernorm_rows_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ gamma,
                                                                             const uint16_t* __restrict__ beta, uint16_t* __restrict__ out,
                                                                             int M, int N, float eps) {
  __shared__ float slots[2][kMaxWaves];
  const RowJob<TPR, false> job(M, 0, 0, 0);
  if (!job.live) return;
  const int nv = N >> 3, tid = job.tid;
  const rw_u32x4 *gp = reinterpret_cast<const rw_u32x4*>(gamma), *bp = reinterpret_cast<const rw_u32x4*>(beta);
  constexpr bool EARLY = KEEP <= 8 && TPR <= 256;               // 4000 x 30000 with 512 threads: early 116 us, late 93
  rw_u32x4 held[KEEP], gv[EARLY ? KEEP : 1], bv[EARLY ? KEEP : 1];
  load_vectors<KEEP>(reinterpret_cast<const rw_u32x4*>(in + (size_t)job.row * N), tid, TPR, nv, held);
  if constexpr (EARLY) {                                         // behind the row, ahead of its statistics
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
      if (tid + i * TPR < nv) {
        gv[i] = gp[tid + i * TPR];
        bv[i] = bp[tid + i * TPR];
      }
  }
  const float mean = mean_of(rw_reduce_group<TPR>(held_sum<KEEP>(held, tid, TPR, nv), RwSum{}, slots[0]), N);
  const float dev = rw_reduce_group<TPR>(held_dev<KEEP>(held, tid, TPR, nv, mean), RwSum{}, slots[1]);
  const float rstd = 1.0f / sqrtf(dev / (float)N + eps);
  rw_u32x4* outp = reinterpret_cast<rw_u32x4*>(out + (size_t)job.row * N);
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if (tid + i * TPR < nv) {
      const int v = tid + i * TPR;
      if constexpr (EARLY) __builtin_nontemporal_store(ln_vector(held[i], gv[i], bv[i], mean, rstd), outp + v);
      else __builtin_nontemporal_store(ln_vector(held[i], gp[v], bp[v], mean, rstd), outp + v);
    }
}

// ---- the same rows, bit for bit, where there are more of them than compute units ----

// A row as a buffer: what is loaded past its end is 0, what is stored there is dropped, and no access needs a branch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_view(const uint16_t* p, int N, bool there = true) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, there ? N * 2 : 0, 0x00027000);
}
constexpr int kNonTemporal = 2;
template <int STRIDE, int AUX>
__device__ __forceinline__ rw_u32x4 view_load(__amdgpu_buffer_rsrc_t r, int i) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, threadIdx.x * 16u + (uint32_t)i * (STRIDE * 16u), 0, AUX);
}
template <int STRIDE>
__device__ __forceinline__ void view_store(const rw_u32x4& v, __amdgpu_buffer_rsrc_t r, int i) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, threadIdx.x * 16u + (uint32_t)i * (STRIDE * 16u), 0, kNonTemporal);
}
// The next pass over v widens it again: its eight floats kept from the last pass would take twice its registers.
__device__ __forceinline__ void anew(rw_u32x4& v) { asm volatile("" : "+v"(v)); }

// Rows of more than 32768 elements.  With 1024 threads a row fills the registers of a compute unit and its load, its arithmetic and its stores
// follow each other; 512 threads with twice the vectors, kept as they came, leave room for a second row beside it (128 registers a thread).  Thread
// t holds the vectors of threads t and t + 512 of the other form and sums them apart, which gives the same sums.  Scheduling
// barriers keep the compiler from widening several vectors at once.
//     softmax    1024 x 65536  54 -> 47 us    300 x 65536  20 -> 15.7   1024 x 49152  42 -> 37    2048 x 65536  99.5 -> 93
//     layernorm  4096 x 36000 122 -> 111      8000 x 32776 219 -> 198   1024 x 49152  43 -> 40.5
// Not kept: the next row fetched into LDS meanwhile (55 us at 1024 x 65536: the waves wait to issue the loads and stores), 64 registers and 1024
// threads (spills).
constexpr int kWideThreads = 512;
template <class Op>
__device__ __forceinline__ float wide_reduce(float even, float odd, Op op, float* slots) {
  even = rw_reduce_lanes<64>(even, op);
  odd = rw_reduce_lanes<64>(odd, op);
  const int wave = (int)threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    slots[wave] = even;
    slots[wave + 8] = odd;
  }
  __syncthreads();
  float g[kMaxWaves];
#pragma unroll
  for (int w = 0; w < kMaxWaves; ++w) g[w] = slots[w];
#pragma unroll
  for (int n = kMaxWaves; n > 1; n /= 2)
#pragma unroll
    for (int w = 0; w < n / 2; ++w) g[w] = op(g[2 * w], g[2 * w + 1]);
  return g[0];
}

// KEEP vectors a thread, the first SURE of which are real in every row of this length.
template <int KEEP, int SURE>
__global__ __launch_bounds__(kWideThreads, 4) void softmax_wide_rows_kernel(const uint16_t* __restrict__ in, uint16_t* __restrict__ out, int N) {
  __shared__ float slots[2][kMaxWaves];
  const int nv = N >> 3;
  const auto src = row_view(in + (size_t)blockIdx.x * N, N), dst = row_view(out + (size_t)blockIdx.x * N, N);
  rw_u32x4 held[KEEP];
#pragma unroll
  for (int i = 0; i < KEEP; ++i) held[i] = view_load<kWideThreads, kNonTemporal>(src, i);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = SURE; i < KEEP; ++i)
    if ((int)threadIdx.x + i * kWideThreads >= nv) held[i] = rw_u32x4{kNegInfPair, kNegInfPair, kNegInfPair, kNegInfPair};
  float m = -FLT_MAX;
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    m = fmaxf(m, held_max<1>(held + i));
    anew(held[i]);
    __builtin_amdgcn_sched_barrier(0);
  }
  const SoftScale base(rw_reduce_group<kWideThreads>(m, RwMax{}, slots[0]));
  constexpr int KEPT = KEEP <= 12 ? KEEP : (88 - 4 * KEEP) / 4;      // exponentials there are registers for; the others are computed twice
  static_assert(KEPT > 0, "16 vectors at most");
  float p[KEPT][8], s[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    float q[8];
    soft_exps(held[i], base, q);
    s[i & 1] += rw_sum8(q);
    if (i < KEPT) {
#pragma unroll
      for (int e = 0; e < 8; ++e) p[i < KEPT ? i : 0][e] = q[e];
    } else {
      anew(held[i]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  const float inv = 1.0f / wide_reduce(s[0], s[1], RwSum{}, slots[1]);
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    float q[8];
    if (i >= KEPT) soft_exps(held[i], base, q);
#pragma unroll
    for (int e = 0; e < 8; ++e) q[e] = (i < KEPT ? p[i < KEPT ? i : 0][e] : q[e]) * inv;
    view_store<kWideThreads>(rw_pack(q), dst, i);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int KEEP, int SURE>
__global__ __launch_bounds__(kWideThreads, 4) void layernorm_wide_rows_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ gamma,
                                                                              const uint16_t* __restrict__ beta, uint16_t* __restrict__ out, int N, float eps) {
  __shared__ float slots[2][kMaxWaves];
  const int nv = N >> 3;
  const auto src = row_view(in + (size_t)blockIdx.x * N, N), dst = row_view(out + (size_t)blockIdx.x * N, N);
  const auto gsrc = row_view(gamma, N), bsrc = row_view(beta, N);
  rw_u32x4 held[KEEP];
#pragma unroll
  for (int i = 0; i < KEEP; ++i) held[i] = view_load<kWideThreads, kNonTemporal>(src, i);
  __builtin_amdgcn_sched_barrier(0);
  float s[2] = {0.f, 0.f}, d[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {                               // zeros past the row's end
    float x[8];
    rw_unpack(held[i], x);
    s[i & 1] = __builtin_fmaf(rw_sum8(x), 1.f / kSumUnit, s[i & 1]);
    anew(held[i]);
    __builtin_amdgcn_sched_barrier(0);
  }
  const float mean = mean_of(wide_reduce(s[0], s[1], RwSum{}, slots[0]), N);
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    const float q = dev8(held[i], mean);
    d[i & 1] += i < SURE || (int)threadIdx.x + i * kWideThreads < nv ? q : 0.f;
    anew(held[i]);
    __builtin_amdgcn_sched_barrier(0);
  }
  constexpr int AHEAD = KEEP <= 10 ? 6 : 5;                      // gamma and beta there are registers for
  static_assert(KEEP <= 12, "registers");
  rw_u32x4 gv[AHEAD], bv[AHEAD];
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) {
    gv[i] = view_load<kWideThreads, 0>(gsrc, i);
    bv[i] = view_load<kWideThreads, 0>(bsrc, i);
  }
  __builtin_amdgcn_sched_barrier(0);
  const float rstd = 1.0f / sqrtf(wide_reduce(d[0], d[1], RwSum{}, slots[1]) / (float)N + eps);
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    const rw_u32x4 y = ln_vector(held[i], gv[i % AHEAD], bv[i % AHEAD], mean, rstd);
    if (i + AHEAD < KEEP) {
      gv[i % AHEAD] = view_load<kWideThreads, 0>(gsrc, i + AHEAD);
      bv[i % AHEAD] = view_load<kWideThreads, 0>(bsrc, i + AHEAD);
    }
    view_store<kWideThreads>(y, dst, i);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Layer normalisation of rows of 3400 to 4096 and 6000 to 8192 elements, many of them: a workgroup takes row after row, gamma and beta stay in its registers (they were two thirds of
// what came out of the L2) and the next row is on its way while one is normalised.  One or two workgroups a compute unit are enough.
//     8192 x 8192  50 -> 45 us    12000 x 7200  70 -> 60    2100 x 8192  16.7 -> 14.9    60000 x 4096  175 -> 163    1100 x 8192  11.1 -> 9.0
constexpr int kLoopThreads = 256;
template <int KEEP>
__global__ __launch_bounds__(kLoopThreads, 4) void layernorm_loop_rows_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ gamma,
                                                                         const uint16_t* __restrict__ beta, uint16_t* __restrict__ out, int M, int N, float eps) {
  __shared__ float slots[2][kMaxWaves];
  const int nv = N >> 3, tid = (int)threadIdx.x, step = (int)gridDim.x;
  rw_u32x4 next[KEEP], gv[KEEP], bv[KEEP];
  auto load = [&](int row) __attribute__((always_inline)) {      // no traffic past the last row
    const auto r = row_view(in + (size_t)(row < M ? row : 0) * N, N, row < M);
#pragma unroll
    for (int i = 0; i < KEEP; ++i) next[i] = view_load<kLoopThreads, kNonTemporal>(r, i);
  };
  int row = (int)blockIdx.x;
  load(row);
  const auto gsrc = row_view(gamma, N), bsrc = row_view(beta, N);
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    gv[i] = view_load<kLoopThreads, 0>(gsrc, i);
    bv[i] = view_load<kLoopThreads, 0>(bsrc, i);
  }
  // all of it waited for here: a wait at the top of the loop would count as if no stores were behind the loads
#pragma unroll
  for (int i = 0; i < KEEP; ++i) asm volatile("" : "+v"(gv[i]), "+v"(bv[i]), "+v"(next[i]));
  for (; row < M; row += step) {
    rw_u32x4 held[KEEP];
#pragma unroll
    for (int i = 0; i < KEEP; ++i) held[i] = next[i];
    load(row + step);
    const float mean = mean_of(rw_reduce_group<kLoopThreads>(held_sum<KEEP>(held, 0, 0, 1), RwSum{}, slots[0]), N);
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
      const float q = dev8(held[i], mean);
      d += tid + i * kLoopThreads < nv ? q : 0.f;
    }
    const float rstd = 1.0f / sqrtf(rw_reduce_group<kLoopThreads>(d, RwSum{}, slots[1]) / (float)N + eps);
    const auto dst = row_view(out + (size_t)row * N, N);
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
      anew(gv[i]);                                               // widened ahead of the loop they would take twice the registers
      anew(bv[i]);
      view_store<kLoopThreads>(ln_vector(held[i], gv[i], bv[i], mean, rstd), dst, i);
    }
  }
}

// ---- rows longer than a workgroup holds: two launches ----

// First vector of chunk c of a row of nv vectors cut into `chunks` chunks (chunk c ends where c + 1 begins).
__host__ __device__ __forceinline__ int chunk_first(int c, int chunks, int nv) { return (int)((int64_t)c * nv / chunks); }

// Statistics of segment `seg` of row `row`, written into slot seg of every chunk of that row of `out`.
template <bool SOFTMAX>
__global__ __launch_bounds__(kSegThreads) void row_stats_kernel(const uint16_t* __restrict__ in, uint16_t* out, int M, int N, int segs,
                                                                int chunks, int num_xcd, int group_m, int mode) {
  __shared__ float slots[2][kMaxWaves];
  int row, seg;
  swz_decode_tile((int)blockIdx.x, M, segs, num_xcd, group_m, mode, &row, &seg);
  const int nv = N >> 3, first = seg * kSegVecs + (int)threadIdx.x;
  rw_u32x4 held[kSegKeep];
  load_vectors<kSegKeep, false>(reinterpret_cast<const rw_u32x4*>(in + (size_t)row * N), first, kSegThreads, nv, held);
  float a, b;
  if constexpr (SOFTMAX) {
    a = rw_reduce_group<kSegThreads>(held_max<kSegKeep>(held), RwMax{}, slots[0]);
    b = rw_reduce_group<kSegThreads>(held_exp_sum<kSegKeep>(held, SoftScale(a)), RwSum{}, slots[1]);
  } else {
    a = mean_of(rw_reduce_group<kSegThreads>(held_sum<kSegKeep>(held, first, kSegThreads, nv), RwSum{}, slots[0]), seg_elems(seg, N));
    b = rw_reduce_group<kSegThreads>(held_dev<kSegKeep>(held, first, kSegThreads, nv, a), RwSum{}, slots[1]);
  }
  for (int c = (int)threadIdx.x; c < chunks; c += kSegThreads) {
    rw_u32x4* chunk = reinterpret_cast<rw_u32x4*>(out + (size_t)row * N) + chunk_first(c, chunks, nv);
    reinterpret_cast<rw_u32x2*>(chunk)[seg] = rw_u32x2{__float_as_uint(a), __float_as_uint(b)};
  }
}

template <bool SOFTMAX>
__global__ __launch_bounds__(kEmitThreads) void row_emit_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ gamma,
                                                                const uint16_t* __restrict__ beta, uint16_t* out, int M, int N, float eps,
                                                                int segs, int chunks, int num_xcd, int group_m, int mode) {
  __shared__ float slots[2][kMaxWaves];
  int row, chunk;
  // from the last row backwards: what the other kernel read last is the likeliest to be in a cache still
  swz_decode_tile((int)(gridDim.x - 1 - blockIdx.x), M, chunks, num_xcd, group_m, mode, &row, &chunk);
  const int nv = N >> 3, v0 = chunk_first(chunk, chunks, nv), v1 = chunk_first(chunk + 1, chunks, nv);
  const int first = v0 + (int)threadIdx.x;
  rw_u32x4* outp = reinterpret_cast<rw_u32x4*>(out + (size_t)row * N);
  rw_u32x4 held[kEmitKeep];
  load_vectors<kEmitKeep>(reinterpret_cast<const rw_u32x4*>(in + (size_t)row * N), first, kEmitThreads, v1, held);
  const rw_u32x4 *gp = reinterpret_cast<const rw_u32x4*>(gamma), *bp = reinterpret_cast<const rw_u32x4*>(beta);
  rw_u32x4 gv[SOFTMAX ? 1 : kEmitKeep], bv[SOFTMAX ? 1 : kEmitKeep];
  const rw_u32x2* stats = reinterpret_cast<const rw_u32x2*>(outp + v0);
  constexpr int PER = kMaxSegs / kEmitThreads;
  float sa[PER], sb[PER], a, b = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int s = (int)threadIdx.x + i * kEmitThreads;
    sa[i] = SOFTMAX ? -FLT_MAX : 0.f;
    sb[i] = 0.f;
    if (s < segs) {
      const rw_u32x2 w = stats[s];
      sa[i] = __uint_as_float(w[0]);
      sb[i] = __uint_as_float(w[1]);
    }
  }
  if constexpr (!SOFTMAX) {
#pragma unroll
    for (int i = 0; i < kEmitKeep; ++i)
      if (first + i * kEmitThreads < v1) {
        gv[i] = gp[first + i * kEmitThreads];
        bv[i] = bp[first + i * kEmitThreads];
      }
  }
  // The barriers inside the reductions separate these reads from the stores below: every thread has read the
  // statistics before any of the chunk is overwritten.
  if constexpr (SOFTMAX) {
    a = -FLT_MAX;
#pragma unroll
    for (int i = 0; i < PER; ++i) a = fmaxf(a, sa[i]);
    a = rw_reduce_group<kEmitThreads>(a, RwMax{}, slots[0]);
#pragma unroll
    for (int i = 0; i < PER; ++i) b += sb[i] * soft_weight(sa[i], a);
  } else {
    auto count = [&](int i) __attribute__((always_inline)) { return seg_elems((int)threadIdx.x + i * kEmitThreads, N); };
    // around the first segment's mean, so that equal means give that mean: the weights count / N are rounded and need not sum to 1
    const float pivot = __uint_as_float(stats[0][0]);
    a = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) a += count(i) > 0 ? (sa[i] - pivot) * ((float)count(i) / (float)N) : 0.f;
    a = pivot + rw_reduce_group<kEmitThreads>(a, RwSum{}, slots[0]);
#pragma unroll
    for (int i = 0; i < PER; ++i) b += count(i) > 0 ? sb[i] + (sa[i] - a) * (sa[i] - a) * (float)count(i) : 0.f;
  }
  b = rw_reduce_group<kEmitThreads>(b, RwSum{}, slots[1]);
  const float scale = SOFTMAX ? 1.0f / b : 1.0f / sqrtf(b / (float)N + eps);
  const SoftScale base(a);
#pragma unroll
  for (int i = 0; i < kEmitKeep; ++i) {
    const int v = first + i * kEmitThreads;
    if (v < v1) {
      if constexpr (SOFTMAX) {
        float y[8];
        soft_exps(held[i], base, y);
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] *= scale;
        __builtin_nontemporal_store(rw_pack(y), outp + v);
      } else {
        __builtin_nontemporal_store(ln_vector(held[i], gv[i], bv[i], a, scale), outp + v);
      }
    }
  }
}

}  // namespace swz
