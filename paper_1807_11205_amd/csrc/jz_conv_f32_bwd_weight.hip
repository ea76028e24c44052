// FP32 gradients of the filter: kernels and variant dispatch.
#include "jz_f32_kernels.h"

int jz::launch_f32_bwd_weight(const PlanF32& pl, hipStream_t st) {
  if (pl.args.bw_linear) return launch_f32_form<OP_BWD_WEIGHT, F32_MATRIX>(pl, st);
  return pl.args.bw_same ? launch_f32_form<OP_BWD_WEIGHT, F32_SAME>(pl, st) : launch_f32_form<OP_BWD_WEIGHT, F32_GATHER>(pl, st);
}
