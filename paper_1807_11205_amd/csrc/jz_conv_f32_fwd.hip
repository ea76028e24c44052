// FP32 forward convolutions: kernels and variant dispatch.
#include "jz_f32_kernels.h"

int jz::launch_f32_fwd(const PlanF32& pl, hipStream_t st) {
  if (pl.window) return launch_f32_window<OP_FWD>(pl, st);
  return pl.gen ? launch_f32_form<OP_FWD, F32_TAPS>(pl, st) : launch_f32_form<OP_FWD, F32_MASKS>(pl, st);
}
