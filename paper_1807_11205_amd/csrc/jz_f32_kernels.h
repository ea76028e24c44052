// The FP32 kernels for channel counts that are multiples of 4 and their launchers, included by one translation unit per operation.
#pragma once
#include <type_traits>

#include "jz_f32_plan.h"
#include "jz_internal.h"

namespace {
using namespace jz;

typedef float f32x16 __attribute__((ext_vector_type(16)));

#include "jz_lds_dma.h"
#include "jz_f32_dma.h"
#include "jz_f32_split.h"
#include "jz_f32_window.h"

template <int BM, int BN, bool PARTS>
constexpr size_t lds_bytes_f32 = PARTS ? F32Split<BM, BN>::LDS_BYTES : (size_t)FD_NST * (BM + BN) * FD_BK * 4;

template <int OP, int BM, int BN, int FORM, bool PARTS>
int launch_f32_tile(const F32Args& a, hipStream_t st) {
  constexpr size_t smem = lds_bytes_f32<BM, BN, PARTS>;
  static std::atomic<bool> lds_set{false};
  if (!allow_lds(reinterpret_cast<const void*>(&f32_kernel<OP, BM, BN, FORM, PARTS>), smem, lds_set)) return JZ_ERR_LAUNCH;
  hipLaunchKernelGGL((f32_kernel<OP, BM, BN, FORM, PARTS>), dim3((unsigned)(a.full_rows + (a.tiles_m - a.full_rows) * a.splits) * (unsigned)a.tiles_n),
                     dim3(256), smem, st, a);
  return jz::launch_status();
}
template <int BM, int BN, int FORM, bool PARTS>
int launch_f32_set_tile(const F32Set& set, hipStream_t st) {
  constexpr size_t smem = lds_bytes_f32<BM, BN, PARTS>;
  static std::atomic<bool> lds_set{false};
  if (!allow_lds(reinterpret_cast<const void*>(&f32_set_kernel<BM, BN, FORM, PARTS>), smem, lds_set)) return JZ_ERR_LAUNCH;
  hipLaunchKernelGGL((f32_set_kernel<BM, BN, FORM, PARTS>), dim3(set.first[FD_MAX_SET]), dim3(256), smem, st, set);
  return jz::launch_status();
}

template <int OP, int BN, int LP>
int launch_f32_window_tile(const F32Args& a, hipStream_t st) {
  constexpr size_t smem = F32Window<BN, LP>::LDS_BYTES;
  static std::atomic<bool> lds_set{false};
  if (!allow_lds(reinterpret_cast<const void*>(&f32_window_kernel<OP, BN, LP>), smem, lds_set)) return JZ_ERR_LAUNCH;
  hipLaunchKernelGGL((f32_window_kernel<OP, BN, LP>), dim3((unsigned)(a.full_rows + (a.tiles_m - a.full_rows) * a.splits) * (unsigned)a.tiles_n),
                     dim3(256), smem, st, a);
  return jz::launch_status();
}
// what the kernel takes for granted; narrow images need fewer rows of window
template <int OP>
int launch_f32_window(const PlanF32& pl, hipStream_t st) {
  const F32Args& a = pl.args;
  if (a.g.R != 3 || a.g.S != 3 || a.g.ph != 1 || a.g.pw != 1 || a.g.sh != 1 || a.g.sw != 1 || a.g.IH != a.g.OH || a.g.IW != a.g.OW || a.sc_on || pl.BM != 128 ||
      a.g.IW > 63 || a.g.IC % (2 * FD_BK) != 0 || a.kt_per_split % 18 != 0 || a.nkt % 18 != 0)
    return JZ_ERR_UNSUPPORTED;
  const bool narrow = f32_window_rows(a.g) == 192;
  if (pl.BN == 128) return narrow ? launch_f32_window_tile<OP, 128, 3>(a, st) : launch_f32_window_tile<OP, 128, 4>(a, st);
  return narrow ? launch_f32_window_tile<OP, 64, 3>(a, st) : launch_f32_window_tile<OP, 64, 4>(a, st);
}

template <int OP, int FORM, bool PARTS>
int launch_f32_tiles(const PlanF32& pl, hipStream_t st) {
  if (pl.BM == 128 && pl.BN == 128) return launch_f32_tile<OP, 128, 128, FORM, PARTS>(pl.args, st);
  if (pl.BM == 128) return launch_f32_tile<OP, 128, 64, FORM, PARTS>(pl.args, st);
  if (pl.BN == 128) return launch_f32_tile<OP, 64, 128, FORM, PARTS>(pl.args, st);
  return launch_f32_tile<OP, 64, 64, FORM, PARTS>(pl.args, st);
}
template <int OP, int FORM>
int launch_f32_form(const PlanF32& pl, hipStream_t st) {
  return pl.parts ? launch_f32_tiles<OP, FORM, true>(pl, st) : launch_f32_tiles<OP, FORM, false>(pl, st);
}
template <int FORM, bool PARTS>
int launch_f32_set(const PlanF32& pl, const F32Set& set, hipStream_t st) {
  if (pl.BM == 128 && pl.BN == 128) return launch_f32_set_tile<128, 128, FORM, PARTS>(set, st);
  if (pl.BM == 128) return launch_f32_set_tile<128, 64, FORM, PARTS>(set, st);
  if (pl.BN == 128) return launch_f32_set_tile<64, 128, FORM, PARTS>(set, st);
  return launch_f32_set_tile<64, 64, FORM, PARTS>(set, st);
}

}  // namespace
