// Shared host-side helpers of libjz (argument checks, launch error mapping).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "jz.h"

namespace jz {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// [a, a+na) and [b, b+nb) share a byte
inline bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  if (!a || !b || na == 0 || nb == 0) return false;
  uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
  return pa < pb + nb && pb < pa + na;
}

// Forward convolution for the fused convolution + batch normalization entry point.  conv_fwd_stats_plan: the workspace
// the convolution needs and, when its kernel (or its split reduction) can leave column sums of y and y^2 over groups of
// rows (its row tiles, or slabs of the reduction), the number of groups (else 0).  conv_fwd_run with stats != nullptr (only after a plan that said so) writes them as [tiles_m][2][K] floats; it
// returns JZ_ERR_UNSUPPORTED, before anything is launched, if the plan no longer has stats_tiles_m row tiles.
// BnTail: the normalization itself, for a split reduction that can do it all; `done` says that it did.
struct BnTail {
  const float* gamma;
  const float* beta = nullptr;         // forward
  float eps = 0.f;
  int relu = 0;
  const void* residual16 = nullptr;
  void* y16 = nullptr;
  float *save_mean = nullptr, *save_invstd = nullptr;
  void *dx16 = nullptr, *dgamma16 = nullptr, *dbeta16 = nullptr;  // backward
  bool done = false;
};
int conv_fwd_stats_plan(const jz_conv_desc* d, size_t* conv_ws_bytes, int* tiles_m);
int conv_fwd_run(const jz_conv_desc* d, const void* x, const void* w, void* y, void* ws, size_t ws_bytes, float* stats,
                 int stats_tiles_m, BnTail* tail, void* stream);

// Backward-data convolution for the fused "backward-data + batch-norm backward" entry point (jz_bn.hip): the layer whose
// output (after batch normalization + ReLU) was this convolution's input.  conv_bwd_data_stats_plan: the convolution's
// workspace and, when its kernel or split reduction can leave sums of g and g x^ (g = dx where y > 0) over groups of rows, their number (else 0);
// conv_bwd_data_run with stats != nullptr (only after a plan that said so) writes them as [tiles_m][2][C] floats.
struct BnBwdOperands {
  const void* x16;      // the normalization's input  [N,H,W,C] of the convolution's input shape
  const void* y16;      // its output after the ReLU = the convolution's forward input
  const float* mean;    // [C]
  const float* invstd;  // [C]
  // block end: y16 = relu(bn(x16) + shortcut) is a residual block's output and the convolution's result is one
  // contribution to its gradient; what the convolution stores (and sums) is g = RNE16(result [+ add16]) where y16 > 0
  bool block_end = false;
  const void* add16 = nullptr;  // the other contribution, optional
};
int conv_bwd_data_stats_plan(const jz_conv_desc* d, size_t* conv_ws_bytes, int* tiles_m);
int conv_bwd_data_run(const jz_conv_desc* d, const void* dy, const void* w, void* dx, void* ws, size_t ws_bytes, float* stats,
                      int stats_tiles_m, const BnBwdOperands* bn, BnTail* tail, void* stream);

// Splitting a reduction is a matter of speed.  A plan's partial sums take at most kPartialSumLimit bytes, the size of the
// last-level cache: more of them would be written to memory and read back, and lie outside what the cost models were fitted to
// (5x5 and 7x7 layers of 3e12 to 1e13 operations that had taken 300-480 MB: 2-4 % slower with the bound, repeats differ by 5 %).
// A caller with less workspace than the plan asks for gets fewer splits: a forward or backward-data layer always runs, without
// any if need be; a weight gradient, whose reduction runs over all pixels, if 64 x 64 tiles times the splits that fit still are
// kFewSplitsGrid workgroups, one per compute unit (else it is refused, JZ_ERR_WORKSPACE).
constexpr size_t kPartialSumLimit = size_t(256) << 20;
constexpr long long kFewSplitsGrid = 256;
inline bool runs_with_fewer_splits(int op, int M, int N, int splits) {
  return op != JZ_BWD_WEIGHT || (long long)((M + 63) / 64) * ((N + 63) / 64) * splits >= kFewSplitsGrid;
}

// Lets a kernel use `bytes` of dynamic LDS, at its first launch.  done: one per kernel, shared by all threads (setting the
// attribute twice is harmless).
inline bool allow_lds(const void* kernel, size_t bytes, std::atomic<bool>& done) {
  if (done.load(std::memory_order_relaxed)) return true;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
  done.store(true, std::memory_order_relaxed);
  return true;
}

inline int launch_status() { return hipGetLastError() == hipSuccess ? JZ_OK : JZ_ERR_LAUNCH; }

}  // namespace jz
