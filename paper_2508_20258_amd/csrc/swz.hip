// libswz: C-ABI entry points (declared in include/swz.h).  Host side: argument checks,
// tile choice, launches.  Nothing here allocates device memory or synchronises.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <stdlib.h>

#include <atomic>
#include <mutex>
#include <tuple>
#include <utility>

#include "../../include/swz.h"
#include "aux_kernels.h"
#include "gemm_dispatch.h"
#include "gemm_kernel.h"
#include "gemm_pair_kernel.h"
#include "gemm_subtile_kernel.h"
#include "mfma_peak_kernel.h"
#include "pid_decode.h"
#include "row_dispatch.h"
#include "rowwise_kernel.h"
#include "transpose_dispatch.h"
#include "transpose_kernel.h"

namespace {

constexpr int kCusPerXcd = 32;   // gfx950: 8 XCDs x 32 CUs
constexpr int kMaxDevices = 64;
constexpr int kWholeCus = 256;   // compute units assumed where no device can be asked (a whole MI355X)
constexpr int kDefaultBK = 64;  // K panel of a tile step; the kernel moves it as two 32-wide halves (ring of 4)

struct DeviceFacts {
  bool known = false;
  int num_xcd = 0, cus = 0, l2_bytes = 0, lds_bytes = 0;   // num_xcd 0: could not be derived
};
DeviceFacts g_facts[kMaxDevices];
std::atomic<bool> g_attr_set[kMaxDevices][4][4][2];
std::atomic<bool> g_sub_attr_set[kMaxDevices][2 * swz::kSubTileCount + 1];   // sub-tiles, then pieces of the last round, then the pair kernel
std::mutex g_mu;

// SWZ_NUM_XCD in the environment (read once per process): the XCD count to assume instead of the
// one derived from the CU count, for partitioned devices.  0 = not set or not a number in 1..1024.
int env_num_xcd() {
  static const int value = [] {
    const char* e = getenv("SWZ_NUM_XCD");
    if (e == nullptr || *e == 0) return 0;
    char* end = nullptr;
    const long v = strtol(e, &end, 10);
    return (end != nullptr && *end == 0 && v >= 1 && v <= 1024) ? (int)v : 0;
  }();
  return value;
}

int query_device(DeviceFacts* out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SWZ_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_mu);
  DeviceFacts& f = g_facts[dev];
  if (!f.known) {
    int cus = 0, l2 = 0, lds = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return SWZ_ERR_HIP;
    if (hipDeviceGetAttribute(&l2, hipDeviceAttributeL2CacheSize, dev) != hipSuccess) return SWZ_ERR_HIP;
    if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return SWZ_ERR_HIP;
    f.cus = cus;
    f.l2_bytes = l2;
    f.lds_bytes = lds;
    // XCDs come in whole units of 32 CUs (a partitioned device exposes fewer of them); any other
    // CU count is not guessed at: the caller then has to name the XCD count.
    if (env_num_xcd() > 0) f.num_xcd = env_num_xcd();
    else f.num_xcd = (cus >= kCusPerXcd && cus % kCusPerXcd == 0) ? cus / kCusPerXcd : 0;
    f.known = true;
  }
  *out = f;
  return SWZ_OK;
}

using swz::kLaunchThreads;

// Launch through the call that returns the launch's own status: hipGetLastError() after a launch
// would also report (and clear) an error some earlier, unrelated HIP call left behind.
template <class... KArgs, size_t... Is>
int launch_impl(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                std::tuple<KArgs...>& vals, std::index_sequence<Is...>) {
  void* ptrs[] = {static_cast<void*>(&std::get<Is>(vals))...};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, stream) == hipSuccess ? SWZ_OK
                                                                                                             : SWZ_ERR_HIP;
}
template <class... KArgs, class... Args>
int launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, Args... args) {
  static_assert(sizeof...(KArgs) == sizeof...(Args), "argument count");
  if ((int64_t)grid.x * block.x > kLaunchThreads) return SWZ_ERR_OVERFLOW;
  std::tuple<KArgs...> vals{static_cast<KArgs>(args)...};
  return launch_impl(kernel, grid, block, lds, stream, vals, std::index_sequence_for<KArgs...>{});
}

bool valid_mode(int mode) { return mode >= 0 && mode < kModeCount; }

// Shared checks of the two PID-map entry points.  Clamps group_m to grid_m (same raster).
int check_map_args(int grid_m, int grid_n, int num_xcd, int* group_m, int mode) {
  if (grid_m < 1 || grid_n < 1 || num_xcd < 1 || *group_m < 1 || !valid_mode(mode)) return SWZ_ERR_INVALID_ARG;
  if ((int64_t)grid_m * (int64_t)grid_n >= (int64_t)1 << 31) return SWZ_ERR_OVERFLOW;
  if (*group_m > grid_m) *group_m = grid_m;
  return SWZ_OK;
}

// num_wg == 0: one workgroup per tile; otherwise the persistent kernel with num_wg workgroups.
template <class S, int MODE>
int launch_gemm_mode(const void* A, const void* B, void* C, int M, int N, int K, int grid_m, int grid_n,
                     int num_xcd, int group_m, int skew, int num_wg, hipStream_t stream, int slot) {
  auto kernel = num_wg > 0 ? swz::gemm_bf16_persistent_kernel<S, MODE> : swz::gemm_bf16_kernel<S, MODE>;
  const int style = num_wg > 0 ? 1 : 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SWZ_ERR_HIP;
  std::atomic<bool>& ready = g_attr_set[dev][slot][MODE][style];
  if (!ready.load(std::memory_order_acquire)) {       // first launch of this kernel on this device only
    std::lock_guard<std::mutex> lock(g_mu);
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            S::LDS_BYTES) != hipSuccess)
      return SWZ_ERR_HIP;
    ready.store(true, std::memory_order_release);
  }
  const unsigned blocks = (unsigned)(num_wg > 0 ? num_wg : grid_m * grid_n);
  return launch(kernel, dim3(blocks), dim3(S::NT), S::LDS_BYTES, stream, static_cast<const uint16_t*>(A),
                static_cast<const uint16_t*>(B), static_cast<uint16_t*>(C), M, N, K, grid_m, grid_n, num_xcd, group_m, skew);
}

template <class S>
int launch_gemm(const void* A, const void* B, void* C, int M, int N, int K, int grid_m, int grid_n,
                int num_xcd, int group_m, int mode, int num_wg, hipStream_t stream, int slot) {
  const int skew = swz_mode_skewed(mode) ? 1 : 0;
  switch (mode & 3) {
    case SWZ_MODE_RR: return launch_gemm_mode<S, kModeRR>(A, B, C, M, N, K, grid_m, grid_n, num_xcd, group_m, skew, num_wg, stream, slot);
    case SWZ_MODE_XCD: return launch_gemm_mode<S, kModeXcd>(A, B, C, M, N, K, grid_m, grid_n, num_xcd, group_m, skew, num_wg, stream, slot);
    case SWZ_MODE_XCD_GROUPM: return launch_gemm_mode<S, kModeXcdGroupM>(A, B, C, M, N, K, grid_m, grid_n, num_xcd, group_m, skew, num_wg, stream, slot);
    default: return launch_gemm_mode<S, kModeGroupM>(A, B, C, M, N, K, grid_m, grid_n, num_xcd, group_m, skew, num_wg, stream, slot);
  }
}

template <class S>
int launch_gemm_probe(const void* A, const void* B, void* C, int M, int N, int K, int grid_m, int grid_n, int num_xcd,
                      int group_m, int mode, uint64_t* probe, hipStream_t stream) {
  auto go = [&](auto kernel) {
    // set on every call: this is a measurement aid, not a hot path
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            S::LDS_BYTES) != hipSuccess)
      return (int)SWZ_ERR_HIP;
    return launch(kernel, dim3((unsigned)(grid_m * grid_n)), dim3(S::NT), S::LDS_BYTES, stream,
                  static_cast<const uint16_t*>(A), static_cast<const uint16_t*>(B), static_cast<uint16_t*>(C), M, N, K,
                  grid_m, grid_n, num_xcd, group_m, swz_mode_skewed(mode) ? 1 : 0, probe);
  };
  switch (mode & 3) {
    case SWZ_MODE_RR: return go(swz::gemm_bf16_probe_kernel<S, kModeRR>);
    case SWZ_MODE_XCD: return go(swz::gemm_bf16_probe_kernel<S, kModeXcd>);
    case SWZ_MODE_XCD_GROUPM: return go(swz::gemm_bf16_probe_kernel<S, kModeXcdGroupM>);
    default: return go(swz::gemm_bf16_probe_kernel<S, kModeGroupM>);
  }
}

// Once per kernel and device: a kernel that asks for more LDS than the default has to say so.
int allow_lds(const void* kernel, int bytes, int slot) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SWZ_ERR_HIP;
  std::atomic<bool>& ready = g_sub_attr_set[dev][slot];
  if (!ready.load(std::memory_order_acquire)) {
    std::lock_guard<std::mutex> lock(g_mu);
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return SWZ_ERR_HIP;
    ready.store(true, std::memory_order_release);
  }
  return SWZ_OK;
}

template <int I>
using SubOf = swz::SubShape<swz::kSubTiles[I].bm, swz::kSubTiles[I].bn, swz::kSubTiles[I].wm, swz::kSubTiles[I].wn, swz::kSubTiles[I].stages>;

// All of C in sub-tiles of shape I, or only the last, partial round of a grid of 256x256 tiles (pieces).
template <int I>
int launch_subtile(const void* A, const void* B, void* C, int M, int N, int K, const swz::GemmLaunch& l, int num_xcd, int mode, hipStream_t stream) {
  using S = SubOf<I>;
  auto kernel = swz::gemm_bf16_subtile_kernel<S>;
  const int st = allow_lds(reinterpret_cast<const void*>(kernel), S::LDS_BYTES, I);
  if (st != SWZ_OK) return st;
  return launch(kernel, dim3((unsigned)l.blocks), dim3(S::NT), S::LDS_BYTES, stream, static_cast<const uint16_t*>(A),
                static_cast<const uint16_t*>(B), static_cast<uint16_t*>(C), M, N, K, l.grid_m, l.grid_n, num_xcd, l.group_m, mode,
                l.a_feeders, l.b_feeders, l.feed_ticks);
}

template <int I>
int launch_pieces(const void* A, const void* B, void* C, int M, int N, int K, const swz::GemmLaunch& l, int num_xcd, int mode, hipStream_t stream) {
  using Whole = swz::GemmShape<256, 256, 2, 4>;
  using P = SubOf<I>;
  auto kernel = swz::gemm_bf16_tail_kernel<Whole, P>;
  const int lds = Whole::LDS_BYTES > P::LDS_BYTES ? Whole::LDS_BYTES : P::LDS_BYTES;
  const int st = allow_lds(reinterpret_cast<const void*>(kernel), lds, swz::kSubTileCount + I);
  if (st != SWZ_OK) return st;
  return launch(kernel, dim3((unsigned)l.blocks), dim3(Whole::NT), lds, stream, static_cast<const uint16_t*>(A), static_cast<const uint16_t*>(B),
                static_cast<uint16_t*>(C), M, N, K, l.grid_m, l.grid_n, num_xcd, l.group_m, mode, l.whole, l.deal);
}

int launch_pair(const void* A, const void* B, void* C, int M, int N, int K, const swz::GemmLaunch& l, int num_xcd, int mode, hipStream_t stream) {
  using S = swz::PairShape;
  const int st = allow_lds(reinterpret_cast<const void*>(swz::gemm_bf16_pair_kernel), S::LDS_BYTES, 2 * swz::kSubTileCount);
  if (st != SWZ_OK) return st;
  return launch(swz::gemm_bf16_pair_kernel, dim3((unsigned)l.blocks), dim3(S::NT), S::LDS_BYTES, stream, static_cast<const uint16_t*>(A),
                static_cast<const uint16_t*>(B), static_cast<uint16_t*>(C), M, N, K, l.grid_m, l.grid_n, num_xcd, l.group_m, mode);
}

int resolve_plan(int64_t M, int64_t N, int64_t K, const swz_params* p, swz_params* r, int* grid_m, int* grid_n) {
  if (M < 1 || N < 1 || K < 1) return SWZ_ERR_INVALID_ARG;
  const int64_t lim = (int64_t)1 << 31;
  if (M >= lim || N >= lim || K >= lim) return SWZ_ERR_OVERFLOW;
  swz_params q = {0, 0, 0, 0, 0, 0, 0};
  if (p != nullptr) q = *p;
  if (q.bm < 0 || q.bn < 0 || q.bk < 0 || q.group_m < 0 || q.num_xcd < 0 || q.num_wg < 0 ||
      (q.persistent != 0 && q.persistent != 1))
    return SWZ_ERR_INVALID_ARG;
  if (q.bm == 0 && q.bn == 0) {
    // 256x256 tiles are the faster kernel once they fill the chip; below that, more and smaller tiles are.
    // Measured (tiles of the 256x256 grid against compute units): up to a quarter, 128x128 tiles are 1.6-2.0x
    // faster; between a quarter and a half, 128x256 tiles are 1.25-1.3x faster (and 3-14 % ahead of 128x128);
    // above a half, 256x256 tiles win by 1.2-1.3x.  The device is only asked where its CU count decides.
    const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256);
    int cus = kWholeCus;
    if (t256 > 8 && t256 <= 152) {
      DeviceFacts f;
      if (query_device(&f) == SWZ_OK && f.cus > 0) cus = f.cus;
    }
    q.bm = 2 * t256 <= cus ? 128 : 256;
    q.bn = 4 * t256 <= cus ? 128 : 256;
  }
  if (q.bm == 0) q.bm = q.bn;
  if (q.bn == 0) q.bn = q.bm;
  if (q.bk == 0) q.bk = kDefaultBK;
  if (q.group_m == 0) q.group_m = 4;
  if (!((q.bm == 128 || q.bm == 256) && (q.bn == 128 || q.bn == 256)) || q.bk != kDefaultBK) return SWZ_ERR_UNSUPPORTED;
  const int64_t gm = (M + q.bm - 1) / q.bm, gn = (N + q.bn - 1) / q.bn;
  if (gm * gn >= lim) return SWZ_ERR_OVERFLOW;
  if (q.num_xcd == 0 || (q.persistent && q.num_wg == 0)) {
    DeviceFacts f;
    const int st = query_device(&f);
    if (st != SWZ_OK) return st;
    if (q.num_xcd == 0) q.num_xcd = f.num_xcd;
    if (q.num_xcd == 0) return SWZ_ERR_UNSUPPORTED;   // CU count is not a whole number of XCDs: the caller must name it
    if (q.persistent && q.num_wg == 0) q.num_wg = f.cus;
  }
  if (!q.persistent) q.num_wg = 0;
  else if (q.num_wg > gm * gn) q.num_wg = (int32_t)(gm * gn);   // never more workgroups than tiles
  if (r != nullptr) *r = q;
  if (grid_m != nullptr) *grid_m = (int)gm;
  if (grid_n != nullptr) *grid_n = (int)gn;
  return SWZ_OK;
}

constexpr int64_t kMemorySideCacheBytes = (int64_t)256 << 20;   // gfx950: 256 MB behind the L2s, in front of HBM

template <int TILE, bool STREAM>
int launch_transpose_s(const void* in, void* out, int M, int N, int gm, int gn, int num_xcd, int group_m, int mode, int sweep,
                       hipStream_t stream) {
  const dim3 grid((unsigned)(gm * gn)), block(256);
  auto* i = static_cast<const uint16_t*>(in);
  auto* o = static_cast<uint16_t*>(out);
  const swz::LoadPace pace = swz::load_pace(TILE, M, N, mode);
  const int skew = swz_mode_skewed(mode) ? 1 : 0;
  switch (mode & 3) {
    case SWZ_MODE_RR: return launch(swz::transpose16_kernel<TILE, kModeRR, STREAM>, grid, block, pace.lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep, pace.paced);
    case SWZ_MODE_XCD: return launch(swz::transpose16_kernel<TILE, kModeXcd, STREAM>, grid, block, pace.lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep, pace.paced);
    case SWZ_MODE_XCD_GROUPM: return launch(swz::transpose16_kernel<TILE, kModeXcdGroupM, STREAM>, grid, block, pace.lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep, pace.paced);
    default: return launch(swz::transpose16_kernel<TILE, kModeGroupM, STREAM>, grid, block, pace.lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep, pace.paced);
  }
}

template <bool STREAM, bool PACED, int LOADS>
int launch_transpose32(const void* in, void* out, int M, int N, int gm, int gn, int num_xcd, int group_m, int mode, int sweep,
                       hipStream_t stream) {
  const dim3 grid((unsigned)(gm * gn)), block(256);
  auto* i = static_cast<const uint32_t*>(in);
  auto* o = static_cast<uint32_t*>(out);
  const size_t lds = PACED || LOADS < 4 ? 0 : STREAM ? 32768 : 12288;       // on top of the tile's 16 KB: eight, three or five workgroups to a compute unit
  const int skew = swz_mode_skewed(mode) ? 1 : 0;
  switch (mode & 3) {
    case SWZ_MODE_RR: return launch(swz::transpose32_kernel<kModeRR, STREAM, PACED, LOADS>, grid, block, lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep);
    case SWZ_MODE_XCD: return launch(swz::transpose32_kernel<kModeXcd, STREAM, PACED, LOADS>, grid, block, lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep);
    case SWZ_MODE_XCD_GROUPM: return launch(swz::transpose32_kernel<kModeXcdGroupM, STREAM, PACED, LOADS>, grid, block, lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep);
    default: return launch(swz::transpose32_kernel<kModeGroupM, STREAM, PACED, LOADS>, grid, block, lds, stream, i, o, M, N, gm, gn, num_xcd, group_m, skew, sweep);
  }
}

template <int TILE>
int launch_transpose(const void* in, void* out, int M, int N, int gm, int gn, int num_xcd, int group_m, int mode, int sweep,
                     hipStream_t stream) {
  // streaming stores once input plus output no longer fit the memory-side cache (and only where a store
  // instruction covers whole lines: tiles of 64 and 128)
  if (TILE >= 64 && (int64_t)M * N * 4 > kMemorySideCacheBytes)
    return launch_transpose_s<TILE, true>(in, out, M, N, gm, gn, num_xcd, group_m, mode, sweep, stream);
  return launch_transpose_s<TILE, false>(in, out, M, N, gm, gn, num_xcd, group_m, mode, sweep, stream);
}

template <class T, bool TALL, bool PACED>
int launch_transpose_lines(const void* in, void* out, int M, int N, int gn, int num_xcd, int group_m, int mode, bool sweep, hipStream_t stream) {
  constexpr int ROWS = swz::lines_rows((int)sizeof(T), TALL);
  const int blocks_m = (M + ROWS - 1) / ROWS;
  return launch(swz::transpose_lines_kernel<T, ROWS, PACED>, dim3((unsigned)(blocks_m * gn)), dim3(swz::lines_threads(ROWS)), 0, stream, static_cast<const T*>(in),
                static_cast<T*>(out), M, N, blocks_m, gn, num_xcd, group_m < blocks_m ? group_m : blocks_m, mode,
                sweep ? swz_sweep_rows(blocks_m, num_xcd, (int)sizeof(T)) : 0);
}

// Threads per row and 16-byte vectors each of them holds, for rows of up to max_vecs vectors: the fastest of the pairs
// measured (16 to 1024 threads x 1 to 16 vectors, M from 1 to 131072).  Few lanes for short rows (131072 x 128: 14 us with 16
// lanes, 35 with 64), enough threads to leave each one 2 to 8 vectors for longer ones.  The two kernels part between 4096 and 16384
// elements: softmax is faster with more threads (8192 x 8192: 50 us with 512, 52 with 256; 32768 x 16384: 356 us with 1024, 377
// with 256), layer normalisation, which also holds gamma and beta, with fewer (32768 x 16384: 370 us with 256, 394 with 512).
struct RowShape { int max_vecs, keep, tpr; };
constexpr int kRowShapes = 16;
constexpr RowShape kSoftmaxShapes[kRowShapes] = {
    {16, 1, 16},    {32, 1, 32},    {64, 1, 64},    {128, 2, 64},   {224, 4, 64},   {256, 1, 256},  {512, 2, 256},   {1024, 2, 512},
    {1536, 4, 512}, {2048, 2, 1024}, {4096, 8, 512}, {5120, 5, 1024}, {6144, 6, 1024}, {8192, 8, 1024}, {10240, 10, 1024}, {12288, 12, 1024}};
constexpr RowShape kLayernormShapes[kRowShapes] = {
    {16, 1, 16},    {32, 1, 32},    {64, 1, 64},    {128, 2, 64},   {224, 4, 64},   {256, 1, 256},  {512, 2, 256},   {1024, 4, 256},
    {1536, 8, 256}, {2048, 8, 256}, {4096, 8, 512}, {5120, 5, 1024}, {6144, 6, 1024}, {8192, 8, 1024}, {10240, 10, 1024}, {12288, 12, 1024}};

// How the two row-wise entry points launch: index into the kernel's table of shapes (-1: longer than a
// workgroup holds, two launches, segs x chunks per row), mapping parameters.
struct RowPlan {
  int shape, grid_m, num_xcd, group_m, segs, chunks, cus;
  bool named;                         // the caller named num_xcd or group_m
};

int resolve_rows(int64_t M, int64_t N, int chunks, int mode, const swz_params* params, const RowShape* shapes, RowPlan* plan) {
  if (M < 1 || N < 1 || chunks < 1 || !valid_mode(mode)) return SWZ_ERR_INVALID_ARG;
  if (swz_mode_skewed(mode)) return SWZ_ERR_UNSUPPORTED;   // a skew would pull the chunks of a row apart again
  const int64_t lim = (int64_t)1 << 31;
  if (M >= lim || N >= lim || M * chunks >= lim) return SWZ_ERR_OVERFLOW;
  if ((N % 8) != 0 || N > ((int64_t)1 << 24)) return SWZ_ERR_UNSUPPORTED;   // 16-byte vectors; fp32 element counts stay exact
  const int64_t nv = N / 8;
  if (chunks > nv) return SWZ_ERR_INVALID_ARG;
  plan->group_m = 4;
  plan->num_xcd = 0;
  if (params != nullptr) {
    if (params->group_m < 0 || params->num_xcd < 0) return SWZ_ERR_INVALID_ARG;
    if (params->group_m > 0) plan->group_m = params->group_m;
    plan->num_xcd = params->num_xcd;
  }
  plan->named = params != nullptr && (params->group_m > 0 || params->num_xcd > 0);
  DeviceFacts f;
  const int known = query_device(&f);
  plan->cus = known == SWZ_OK && f.cus > 0 ? f.cus : kWholeCus;
  if (plan->num_xcd == 0) {
    if (known != SWZ_OK) return known;
    plan->num_xcd = f.num_xcd;
    if (plan->num_xcd == 0) return SWZ_ERR_UNSUPPORTED;
  }
  plan->segs = plan->chunks = 1;
  plan->grid_m = (int)M;
  plan->shape = 0;
  while (plan->shape < kRowShapes && nv > shapes[plan->shape].max_vecs) ++plan->shape;
  if (plan->shape == kRowShapes) {
    plan->shape = -1;
    plan->segs = (int)((nv + swz::kSegVecs - 1) / swz::kSegVecs);
    plan->chunks = (int)((nv + swz::kEmitThreads * swz::kEmitKeep - 1) / (swz::kEmitThreads * swz::kEmitKeep));
  } else {
    const int rows_per_wg = swz::row_block(shapes[plan->shape].tpr) / shapes[plan->shape].tpr;
    plan->grid_m = (int)((M + rows_per_wg - 1) / rows_per_wg);
  }
  return check_map_args(plan->grid_m, plan->chunks, plan->num_xcd, &plan->group_m, mode);
}

// launch(first row, rows, workgroups) over all rows: once, or in as few parts as a launch's threads allow.
template <class F>
int for_row_parts(const RowPlan& plan, int tpr, int64_t M, F&& launch_part) {
  const int block = swz::row_block(tpr), rows_per_wg = block / tpr;
  const int64_t part = kLaunchThreads / block;
  for (int64_t g = 0; g < plan.grid_m; g += part) {
    const int64_t groups = plan.grid_m - g < part ? plan.grid_m - g : part, row = g * rows_per_wg;
    const int st = launch_part(row, (int)(M - row < groups * rows_per_wg ? M - row : groups * rows_per_wg), (int)groups);
    if (st != SWZ_OK) return st;
  }
  return SWZ_OK;
}

// Whether softmax rows follow the caller's mode: from 16128 elements a row (to 16384, the end of the one shape that can) and 2^29
// elements in all.  Time under the XCD renumbering over that in dispatch order, for 16128, 16376 and 16384 elements: 32768 rows 1.006, 0.979,
// 0.994 (0.975 with three sets of buffers in turn), 40000 rows 1.007, 0.982, 0.989, 65536 rows 0.986, 0.980, 1.006.  Outside, dispatch order is
// ahead: fewer rows (16384 elements x 24000, 16384, 4096 rows 1.007, 1.020, 1.126), shorter ones (12544 elements 1.10 to 1.28, 13312
// 1.05 to 1.13, 15360 1.02 to 1.10, 16000 1.00 to 1.06; 14336 alone is at 0.96 to 0.99 from 32768 rows on).
bool soft_rows_mapped(int64_t M, int64_t N) { return N >= 16128 && M * N >= ((int64_t)1 << 29); }

template <int KEEP, int TPR>
int launch_softmax_rows(const uint16_t* in, uint16_t* out, int64_t M, int N, const RowPlan& plan, int mode, hipStream_t stream) {
  // Rows of 40968 to 65536 elements: two to a compute unit.  With many rows the one-row form drifts into overlap by itself: 4096 x 65528 202 us with
  // 1024 threads, 205 with 512 (2048 x 65536 101, 95; 4096 x 41000 132, 120); shorter rows fit twice in either form (4096 x 36000 100 us, 104).
  if constexpr (TPR == 1024 && (KEEP == 6 || KEEP == 8)) {
    if (M > plan.cus && M <= (KEEP == 6 ? 16 : 8) * plan.cus)
      return launch(swz::softmax_wide_rows_kernel<2 * KEEP, KEEP == 6 ? 10 : 12>, dim3((unsigned)M), dim3(swz::kWideThreads), 0, stream, in, out, N);
  }
  if (!soft_rows_mapped(M, N)) mode = SWZ_MODE_RR;
  return for_row_parts(plan, TPR, M, [&](int64_t row, int rows, int groups) {
    const int group_m = plan.group_m < groups ? plan.group_m : groups;
    return launch(swz::softmax_rows_kernel<KEEP, TPR>, dim3((unsigned)groups), dim3(swz::row_block(TPR)), 0, stream, in + row * N,
                  out + row * N, rows, N, plan.num_xcd, group_m, mode);
  });
}

template <int KEEP, int TPR>
int launch_layernorm_rows(const uint16_t* in, const uint16_t* gamma, const uint16_t* beta, uint16_t* out, int64_t M, int N, float eps,
                          const RowPlan& plan, hipStream_t stream) {
  // Rows of 32776 to 49152 elements: two to a compute unit (from there to 65536 elements it is level: 1024 x 65536 55 us either way)
  if constexpr (TPR == 1024 && (KEEP == 5 || KEEP == 6)) {
    if (M > plan.cus)
      return for_row_parts(plan, swz::kWideThreads, M, [&](int64_t row, int rows, int groups) {
        return launch(swz::layernorm_wide_rows_kernel<2 * KEEP, 2 * KEEP - 2>, dim3((unsigned)groups), dim3(swz::kWideThreads), 0, stream, in + row * N,
                      gamma, beta, out + row * N, N, eps);
      });
  }
  // Row after row where most of the KEEP x 256 vectors are real and the workgroups have enough rows.  Time of the loop over that of a workgroup a row, operands
  // not in cache: four vectors, from 2 rows a compute unit on 513 rows 0.90 to 0.99, 800 rows 0.83 to 0.97, 1540 rows 0.83 to 0.86 (of 6000 to 8192 elements;
  // 4800 and less 1.06 at 1100 rows).  Two vectors: 4 to 5 rows a compute unit 0.94 to 1.02; from 5 on some workgroups have a third row and the others wait for
  // them, 1290 rows 1.04 to 1.09; 1500 rows of 3400 and 3480 elements 1.05 to 1.08, of 3600 and more 0.93 to 0.98; 1600 rows 0.90 to 0.97, 2060 rows 0.88 to 0.96.
  // One against two workgroups a compute unit: 5000 x 7200 27.2 us, 27.7; 12000 x 8192 64.9, 67.2; but 2100 x 8192 15.3, 14.9 and 12000 x 6400 55.5, 54.0.
  if constexpr (TPR == swz::kLoopThreads && (KEEP == 2 || KEEP == 4)) {
    if (KEEP == 4 ? N >= 6000 && M > 2 * plan.cus : N >= 3400 && 2 * M > (N >= 3600 ? 11 : 12) * plan.cus) {
      const int64_t per_cu = N >= 7000 && M * N >= ((int64_t)1 << 25) ? 1 : 2;
      return launch(swz::layernorm_loop_rows_kernel<KEEP>, dim3((unsigned)(per_cu * plan.cus)), dim3(swz::kLoopThreads), 0, stream, in, gamma, beta, out, (int)M,
                    N, eps);
    }
  }
  return for_row_parts(plan, TPR, M, [&](int64_t row, int rows, int groups) {
    return launch(swz::layernorm_rows_kernel<KEEP, TPR>, dim3((unsigned)groups), dim3(swz::row_block(TPR)), 0, stream, in + row * N,
                  gamma, beta, out + row * N, rows, N, eps);
  });
}

// FN<KEEP, TPR> of the chosen shape.
#define SWZ_ROWS_CASE(S, FN, SHAPES, ...) \
  case S: return FN<SHAPES[S].keep, SHAPES[S].tpr>(__VA_ARGS__);
#define SWZ_ROWS_CASES(A, B, C, D, ...) \
  SWZ_ROWS_CASE(A, __VA_ARGS__) SWZ_ROWS_CASE(B, __VA_ARGS__) SWZ_ROWS_CASE(C, __VA_ARGS__) SWZ_ROWS_CASE(D, __VA_ARGS__)
#define SWZ_LAUNCH_ROWS(...)                                                                                                 \
  switch (plan.shape) {                                                                                                      \
    SWZ_ROWS_CASES(0, 1, 2, 3, __VA_ARGS__) SWZ_ROWS_CASES(4, 5, 6, 7, __VA_ARGS__) SWZ_ROWS_CASES(8, 9, 10, 11, __VA_ARGS__) \
    SWZ_ROWS_CASES(12, 13, 14, 15, __VA_ARGS__)                                                                              \
    default: break;                                                                                                          \
  }
static_assert(kRowShapes == 16, "the cases above");

template <bool SOFTMAX>
int launch_long_rows(const uint16_t* in, const uint16_t* gamma, const uint16_t* beta, uint16_t* out, int M, int N, float eps,
                     const RowPlan& plan, int mode, hipStream_t stream) {
  // `out` holds the statistics while `in` is read a second time
  const uintptr_t i = reinterpret_cast<uintptr_t>(in), o = reinterpret_cast<uintptr_t>(out), bytes = (uintptr_t)M * (uintptr_t)N * 2;
  if (i < o + bytes && o < i + bytes) return SWZ_ERR_INVALID_ARG;
  const int st = launch(swz::row_stats_kernel<SOFTMAX>, dim3((unsigned)((int64_t)M * plan.segs)), dim3(swz::kSegThreads), 0, stream, in, out, M,
                        N, plan.segs, plan.chunks, plan.num_xcd, plan.group_m, mode);
  if (st != SWZ_OK) return st;
  const int order = !SOFTMAX && swz::emit_in_dispatch_order(M, N, plan.chunks, plan.num_xcd, plan.named) ? (int)SWZ_MODE_RR : mode;
  return launch(swz::row_emit_kernel<SOFTMAX>, dim3((unsigned)((int64_t)M * plan.chunks)), dim3(swz::kEmitThreads), 0, stream, in, gamma, beta,
                out, M, N, eps, plan.segs, plan.chunks, plan.num_xcd, plan.group_m, order);
}
}  // namespace

extern "C" {

const char* swz_status_string(int status) {
  switch (status) {
    case SWZ_OK: return "ok";
    case SWZ_ERR_INVALID_ARG: return "invalid argument";
    case SWZ_ERR_UNSUPPORTED: return "unsupported dtype, alignment or tile shape";
    case SWZ_ERR_OVERFLOW: return "size does not fit 32-bit tile arithmetic";
    case SWZ_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

int swz_device_info(int* num_xcd, int* compute_units, int* l2_bytes, int* lds_bytes) {
  DeviceFacts f;
  const int st = query_device(&f);
  if (st != SWZ_OK) return st;
  if (num_xcd) *num_xcd = f.num_xcd;
  if (compute_units) *compute_units = f.cus;
  if (l2_bytes) *l2_bytes = f.l2_bytes;
  if (lds_bytes) *lds_bytes = f.lds_bytes;
  return SWZ_OK;
}

int swz_pid_map(int grid_m, int grid_n, int num_xcd, int group_m, int mode, int32_t* out) {
  if (out == nullptr) return SWZ_ERR_INVALID_ARG;
  const int st = check_map_args(grid_m, grid_n, num_xcd, &group_m, mode);
  if (st != SWZ_OK) return st;
  const int total = grid_m * grid_n;
  for (int w = 0; w < total; ++w) {
    int pm, pn;
    swz_decode_tile(w, grid_m, grid_n, num_xcd, group_m, mode, &pm, &pn);
    out[w] = pm * grid_n + pn;
  }
  return SWZ_OK;
}

int swz_pid_map_device(int grid_m, int grid_n, int num_xcd, int group_m, int mode, int32_t* d_tile,
                       int32_t* d_xcc, hipStream_t stream) {
  if (d_tile == nullptr) return SWZ_ERR_INVALID_ARG;
  const int st = check_map_args(grid_m, grid_n, num_xcd, &group_m, mode);
  if (st != SWZ_OK) return st;
  return launch(swz::pid_map_kernel, dim3((unsigned)(grid_m * grid_n)), dim3(64), 0, stream, grid_m, grid_n, num_xcd,
                group_m, mode, d_tile, d_xcc);
}

int swz_pid_map_persistent(int grid_m, int grid_n, int num_xcd, int group_m, int mode, int num_wg, int32_t* out) {
  if (out == nullptr || num_wg < 1) return SWZ_ERR_INVALID_ARG;
  const int st = check_map_args(grid_m, grid_n, num_xcd, &group_m, mode);
  if (st != SWZ_OK) return st;
  const int total = grid_m * grid_n;
  const int64_t rounds = ((int64_t)total + num_wg - 1) / num_wg;
  if (rounds * num_wg >= (int64_t)1 << 31) return SWZ_ERR_OVERFLOW;
  for (int round = 0; round < (int)rounds; ++round) {
    for (int w = 0; w < num_wg; ++w) {
      const int l = swz_persistent_logical(w, round, num_wg, total, num_xcd, mode);
      int t = -1;
      if (l >= 0) {
        int pm, pn;
        swz_tile_at(l, grid_m, grid_n, group_m, mode, &pm, &pn);
        t = pm * grid_n + pn;
      }
      out[(size_t)round * num_wg + w] = t;
    }
  }
  return SWZ_OK;
}

int swz_pid_map_persistent_device(int grid_m, int grid_n, int num_xcd, int group_m, int mode, int num_wg,
                                  int32_t* d_tile, int32_t* d_xcc, hipStream_t stream) {
  if (d_tile == nullptr || num_wg < 1) return SWZ_ERR_INVALID_ARG;
  const int st = check_map_args(grid_m, grid_n, num_xcd, &group_m, mode);
  if (st != SWZ_OK) return st;
  const int64_t rounds = ((int64_t)grid_m * grid_n + num_wg - 1) / num_wg;
  if (rounds * num_wg >= (int64_t)1 << 31) return SWZ_ERR_OVERFLOW;
  return launch(swz::pid_map_persistent_kernel, dim3((unsigned)num_wg), dim3(64), 0, stream, grid_m, grid_n, num_xcd,
                group_m, mode, (int)rounds, d_tile, d_xcc);
}

int swz_transpose(const void* in, void* out, int64_t M, int64_t N, int elem_bytes, int tile, int mode,
                  const swz_params* params, hipStream_t stream) {
  if (in == nullptr || out == nullptr || M < 1 || N < 1 || !valid_mode(mode)) return SWZ_ERR_INVALID_ARG;
  const int64_t lim = (int64_t)1 << 31;
  if (M >= lim || N >= lim) return SWZ_ERR_OVERFLOW;
  if (elem_bytes == 4) {
    if (tile != 64 || (M % 4) != 0 || (N % 4) != 0) return SWZ_ERR_UNSUPPORTED;
  } else if (elem_bytes != 2 || (tile != 32 && tile != 64 && tile != 128) || (M % 8) != 0 || (N % 8) != 0) {
    return SWZ_ERR_UNSUPPORTED;
  }
  if ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) return SWZ_ERR_UNSUPPORTED;
  int group_m = 4, num_xcd = 0;
  if (params != nullptr) {
    if (params->group_m < 0 || params->num_xcd < 0) return SWZ_ERR_INVALID_ARG;
    if (params->group_m > 0) group_m = params->group_m;
    num_xcd = params->num_xcd;
  }
  if (num_xcd == 0) {
    DeviceFacts f;
    const int st = query_device(&f);
    if (st != SWZ_OK) return st;
    num_xcd = f.num_xcd;
    if (num_xcd == 0) return SWZ_ERR_UNSUPPORTED;
  }
  const int64_t gm = (M + tile - 1) / tile, gn = (N + tile - 1) / tile;
  if (gm * gn >= lim) return SWZ_ERR_OVERFLOW;
  const int st = check_map_args((int)gm, (int)gn, num_xcd, &group_m, mode);
  if (st != SWZ_OK) return st;
  // Rows of `out` that start inside a 128-byte line, and enough of them that the memory decides: below 16 MiB moved the extra
  // rows a block reads cost more than its part lines (blocks of 64 rows: 1000 x 1004 x 4 B 5.4 us against 5.6, 1000 x 1000 x 2 B 3.7 against 4.2; 3000 x
  // 3000 x 2 B, 34 MiB moved, 11.5 against 9.9).
  const bool part_lines = ((M * elem_bytes) & 127) != 0 || (reinterpret_cast<uintptr_t>(out) & 127) != 0;
  const bool ours = tile == 64 && mode == (SWZ_MODE_XCD_GROUPM | SWZ_MODE_SKEW) && (params == nullptr || params->group_m == 0);
  if (tile == 64 && part_lines && M < ((int64_t)1 << 30) && 2 * M * N * elem_bytes >= ((int64_t)16 << 20)) {
    const bool sweep = ours && swz::sweep_part_lines(N, elem_bytes);
    const int m = (int)M, n = (int)N, g = (int)gn;
    auto go = [&](auto elem) {
      using T = decltype(elem);
      switch (swz::line_blocks(M, N, elem_bytes)) {
        case swz::kLinesTallPaced: return launch_transpose_lines<T, true, true>(in, out, m, n, g, num_xcd, group_m, mode, sweep, stream);
        case swz::kLinesTall: return launch_transpose_lines<T, true, false>(in, out, m, n, g, num_xcd, group_m, mode, sweep, stream);
        default: return launch_transpose_lines<T, false, false>(in, out, m, n, g, num_xcd, group_m, mode, sweep, stream);
      }
    };
    return elem_bytes == 2 ? go(uint16_t{}) : go(uint32_t{});
  }
  const int sweep = ours && swz::sweep_tiles(M, N, elem_bytes) ? swz_sweep_rows((int)gm, num_xcd, elem_bytes) : 0;
  if (elem_bytes == 4) {
    const int m = (int)M, n = (int)N, tm = (int)gm, tn = (int)gn;
    // one row of tiles, a quarter or half of it real: no loads for the rest, and eight workgroups to a compute unit, as each has little on its way (us, all loads and five workgroups, three
    // above 256 MiB -> these: 4 x 521008 13.6 -> 10.0, 16 x 98304 4.6 -> 4.1, 24 x 86832 5.5 -> 4.7, 32 x 1228800 61.2 -> 57.8, 32 x 3686400 176 -> 168)
    const bool beyond = M * N * 8 > kMemorySideCacheBytes;
    if (M <= 16 && !beyond) return launch_transpose32<false, false, 1>(in, out, m, n, tm, tn, num_xcd, group_m, mode, sweep, stream);
    if (M <= 32) return (beyond ? launch_transpose32<true, false, 2> : launch_transpose32<false, false, 2>)(in, out, m, n, tm, tn, num_xcd, group_m, mode, sweep, stream);
    if (beyond) return launch_transpose32<true, false, 4>(in, out, m, n, tm, tn, num_xcd, group_m, mode, sweep, stream);
    if (swz::paced_tiles32(M, N)) return launch_transpose32<false, true, 4>(in, out, m, n, tm, tn, num_xcd, group_m, mode, sweep, stream);
    return launch_transpose32<false, false, 4>(in, out, m, n, tm, tn, num_xcd, group_m, mode, sweep, stream);
  }
  if (tile == 128) return launch_transpose<128>(in, out, (int)M, (int)N, (int)gm, (int)gn, num_xcd, group_m, mode, sweep, stream);
  return tile == 64 ? launch_transpose<64>(in, out, (int)M, (int)N, (int)gm, (int)gn, num_xcd, group_m, mode, sweep, stream)
                    : launch_transpose<32>(in, out, (int)M, (int)N, (int)gm, (int)gn, num_xcd, group_m, mode, sweep, stream);
}

int swz_softmax(const void* in, void* out, int64_t M, int64_t N, int chunks, int mode, const swz_params* params,
                hipStream_t stream) {
  if (in == nullptr || out == nullptr) return SWZ_ERR_INVALID_ARG;
  RowPlan plan;
  const int st = resolve_rows(M, N, chunks, mode, params, kSoftmaxShapes, &plan);
  if (st != SWZ_OK) return st;
  if ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) return SWZ_ERR_UNSUPPORTED;
  auto* x = static_cast<const uint16_t*>(in);
  auto* y = static_cast<uint16_t*>(out);
  SWZ_LAUNCH_ROWS(launch_softmax_rows, kSoftmaxShapes, x, y, M, (int)N, plan, mode, stream)
  return launch_long_rows<true>(x, nullptr, nullptr, y, (int)M, (int)N, 0.f, plan, mode, stream);
}

int swz_layernorm(const void* in, const void* gamma, const void* beta, void* out, int64_t M, int64_t N, float eps,
                  int chunks, int mode, const swz_params* params, hipStream_t stream) {
  if (in == nullptr || gamma == nullptr || beta == nullptr || out == nullptr || !(eps >= 0.f)) return SWZ_ERR_INVALID_ARG;
  RowPlan plan;
  const int st = resolve_rows(M, N, chunks, mode, params, kLayernormShapes, &plan);
  if (st != SWZ_OK) return st;
  if ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(gamma) |
       reinterpret_cast<uintptr_t>(beta)) & 15)
    return SWZ_ERR_UNSUPPORTED;
  auto* x = static_cast<const uint16_t*>(in);
  auto* g = static_cast<const uint16_t*>(gamma);
  auto* b = static_cast<const uint16_t*>(beta);
  auto* y = static_cast<uint16_t*>(out);
  SWZ_LAUNCH_ROWS(launch_layernorm_rows, kLayernormShapes, x, g, b, y, M, (int)N, eps, plan, stream)
  return launch_long_rows<false>(x, g, b, y, (int)M, (int)N, eps, plan, mode, stream);
}

int swz_mfma_peak(float* out, int64_t out_floats, int iters, int random_operands, int* workgroups, hipStream_t stream) {
  if (out == nullptr || iters < 1) return SWZ_ERR_INVALID_ARG;
  DeviceFacts f;
  const int st = query_device(&f);
  if (st != SWZ_OK) return st;
  if (out_floats < (int64_t)f.cus * 512) return SWZ_ERR_INVALID_ARG;
  if (workgroups != nullptr) *workgroups = f.cus;
  return launch(swz::mfma_peak_kernel, dim3((unsigned)f.cus), dim3(512), 0, stream, out, iters, random_operands ? 1 : 0);
}

int swz_copy_bytes(const void* src, void* dst, int64_t bytes, hipStream_t stream) {
  if (src == nullptr || dst == nullptr || bytes < 16) return SWZ_ERR_INVALID_ARG;
  if ((bytes & 15) || ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15)) return SWZ_ERR_UNSUPPORTED;
  const int64_t n = bytes / 16;
  const int64_t want = (n + 1023) / 1024;                       // a workgroup moves 1024 words per round
  const unsigned blocks = (unsigned)(want < 8192 ? want : 8192);
  return launch(swz::copy16_kernel, dim3(blocks), dim3(256), 0, stream, static_cast<const swz::aux_u32x4*>(src),
                static_cast<swz::aux_u32x4*>(dst), n);
}

int swz_gemm_plan(int64_t M, int64_t N, int64_t K, const swz_params* params, swz_params* resolved, int* grid_m,
                  int* grid_n) {
  return resolve_plan(M, N, K, params, resolved, grid_m, grid_n);
}

// The four tile shapes: 8 waves each; 256x256 -> wave tile 128x64, the other three -> wave tile 64x64 or 64x32.
using Shape128 = swz::GemmShape<128, 128, 2, 4>;
using Shape256 = swz::GemmShape<256, 256, 2, 4>;
using Shape128x256 = swz::GemmShape<128, 256, 2, 4>;
using Shape256x128 = swz::GemmShape<256, 128, 4, 2>;

// The sizes and parameters that the GEMM entry points take; on success r, grid_m, grid_n and group_m describe the plan's tiles.
static int check_gemm_sizes(int64_t M, int64_t N, int64_t K, int dtype, int mode, const swz_params* params, swz_params* r, int* grid_m,
                            int* grid_n, int* group_m) {
  int st = resolve_plan(M, N, K, params, r, grid_m, grid_n);
  if (st != SWZ_OK) return st;
  if (dtype != SWZ_DTYPE_BF16) return SWZ_ERR_UNSUPPORTED;
  if ((K % 8) != 0 || (N % 8) != 0) return SWZ_ERR_UNSUPPORTED;   // 16-byte vector loads along k and n
  // per-lane source offsets inside a tile step are 32-bit: (bm-1) rows of A, 31 rows of B
  if ((int64_t)r->bm * K * 2 >= ((int64_t)1 << 32) || (int64_t)32 * N * 2 >= ((int64_t)1 << 32)) return SWZ_ERR_OVERFLOW;
  *group_m = r->group_m;
  return check_map_args(*grid_m, *grid_n, r->num_xcd, group_m, mode);
}

static int check_gemm(const void* A, const void* B, const void* C, int64_t M, int64_t N, int64_t K, int dtype, int mode,
                      const swz_params* params, swz_params* r, int* grid_m, int* grid_n, int* group_m) {
  if (A == nullptr || B == nullptr || C == nullptr || !valid_mode(mode)) return SWZ_ERR_INVALID_ARG;
  const int st = check_gemm_sizes(M, N, K, dtype, mode, params, r, grid_m, grid_n, group_m);
  if (st != SWZ_OK) return st;
  if ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B) | reinterpret_cast<uintptr_t>(C)) & 15)
    return SWZ_ERR_UNSUPPORTED;
  return SWZ_OK;
}

static bool tile_is_free(const swz_params* params) { return params == nullptr || (params->bm == 0 && params->bn == 0); }

int swz_gemm_launch_map(int64_t M, int64_t N, int64_t K, int mode, const swz_params* params, int32_t* out, int64_t out_words, int64_t* workgroups) {
  if (workgroups == nullptr || !valid_mode(mode)) return SWZ_ERR_INVALID_ARG;
  swz_params r;
  int grid_m = 0, grid_n = 0, group_m = 0;
  const int st = check_gemm_sizes(M, N, K, SWZ_DTYPE_BF16, mode, params, &r, &grid_m, &grid_n, &group_m);
  if (st != SWZ_OK) return st;
  if (r.persistent) return SWZ_ERR_UNSUPPORTED;
  DeviceFacts f;
  const int cus = tile_is_free(params) && query_device(&f) == SWZ_OK && f.cus > 0 ? f.cus : kWholeCus;
  const swz::GemmLaunch l = swz::gemm_launch(M, N, K, r, grid_m, grid_n, group_m, mode, tile_is_free(params), cus);
  if (out != nullptr && out_words < 4 * l.blocks) return SWZ_ERR_INVALID_ARG;
  *workgroups = l.blocks;
  for (int64_t w = 0; out != nullptr && w < l.blocks; ++w) {
    const swz::GemmBlock b = swz::gemm_block(l, r.num_xcd, mode, M, N, (int)w);
    out[4 * w] = b.row;
    out[4 * w + 1] = b.col;
    out[4 * w + 2] = b.rows;
    out[4 * w + 3] = b.cols;
  }
  return SWZ_OK;
}

int swz_gemm_ex(const void* A, const void* B, void* C, int64_t M, int64_t N, int64_t K, int dtype, int mode,
                const swz_params* params, hipStream_t stream) {
  swz_params r;
  int grid_m = 0, grid_n = 0, group_m = 0;
  const int st = check_gemm(A, B, C, M, N, K, dtype, mode, params, &r, &grid_m, &grid_n, &group_m);
  if (st != SWZ_OK) return st;
  if (tile_is_free(params) && !r.persistent) {
    DeviceFacts f;
    const int qs = query_device(&f);
    if (qs != SWZ_OK) return qs;
    const int m = (int)M, n = (int)N, k = (int)K;
    const swz::GemmLaunch l = swz::gemm_launch(M, N, K, r, grid_m, grid_n, group_m, mode, true, f.cus > 0 ? f.cus : kWholeCus);
    if (l.pair) return launch_pair(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
    if (l.pieces)
      return l.sub == swz::kQuarterPiece ? launch_pieces<swz::kQuarterPiece>(A, B, C, m, n, k, l, r.num_xcd, mode, stream)
                                         : launch_pieces<swz::kHalfPiece>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
    switch (l.sub) {
      case 0: return launch_subtile<0>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 1: return launch_subtile<1>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 2: return launch_subtile<2>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 3: return launch_subtile<3>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 4: return launch_subtile<4>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 5: return launch_subtile<5>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 6: return launch_subtile<6>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 7: return launch_subtile<7>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 8: return launch_subtile<8>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      case 9: return launch_subtile<9>(A, B, C, m, n, k, l, r.num_xcd, mode, stream);
      default: break;                                   // whole tiles
    }
  }
  if (r.bm == 128 && r.bn == 128)
    return launch_gemm<Shape128>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, r.num_wg, stream, 0);
  if (r.bm == 128)
    return launch_gemm<Shape128x256>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, r.num_wg, stream, 2);
  if (r.bn == 128)
    return launch_gemm<Shape256x128>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, r.num_wg, stream, 3);
  return launch_gemm<Shape256>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, r.num_wg, stream, 1);
}

int swz_gemm_probe(const void* A, const void* B, void* C, int64_t M, int64_t N, int64_t K, int dtype, int mode,
                   const swz_params* params, uint64_t* probe, int64_t probe_words, hipStream_t stream) {
  if (probe == nullptr) return SWZ_ERR_INVALID_ARG;
  swz_params r;
  int grid_m = 0, grid_n = 0, group_m = 0;
  const int st = check_gemm(A, B, C, M, N, K, dtype, mode, params, &r, &grid_m, &grid_n, &group_m);
  if (st != SWZ_OK) return st;
  if (r.persistent) return SWZ_ERR_UNSUPPORTED;
  if (probe_words < (int64_t)grid_m * grid_n * swz::kProbeWords) return SWZ_ERR_INVALID_ARG;
  if (reinterpret_cast<uintptr_t>(probe) & 7) return SWZ_ERR_UNSUPPORTED;
  if (r.bm == 128 && r.bn == 128)
    return launch_gemm_probe<Shape128>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, probe, stream);
  if (r.bm == 128)
    return launch_gemm_probe<Shape128x256>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, probe, stream);
  if (r.bn == 128)
    return launch_gemm_probe<Shape256x128>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, probe, stream);
  return launch_gemm_probe<Shape256>(A, B, C, (int)M, (int)N, (int)K, grid_m, grid_n, r.num_xcd, group_m, mode, probe, stream);
}

int swz_gemm(const void* A, const void* B, void* C, int64_t M, int64_t N, int64_t K, int dtype, int mode,
             hipStream_t stream) {
  return swz_gemm_ex(A, B, C, M, N, K, dtype, mode, nullptr, stream);
}

}  // extern "C"
