// FP32 gradients of the input: kernels and variant dispatch.
#include "jz_f32_kernels.h"

int jz::launch_f32_bwd_data(const PlanF32& pl, hipStream_t st, const F32Set* set) {
  if (!set && pl.window) return launch_f32_window<OP_BWD_DATA>(pl, st);
  if (!set) return pl.gen ? launch_f32_form<OP_BWD_DATA, F32_TAPS>(pl, st) : launch_f32_form<OP_BWD_DATA, F32_MASKS>(pl, st);
  if (pl.gen) return pl.parts ? launch_f32_set<F32_TAPS, true>(pl, *set, st) : launch_f32_set<F32_TAPS, false>(pl, *set, st);
  return pl.parts ? launch_f32_set<F32_MASKS, true>(pl, *set, st) : launch_f32_set<F32_MASKS, false>(pl, *set, st);
}
