// The window kernel (jz_window.h), forward: see jz_conv_plan.h
#include "jz_igemm_kernels.h"
#include "jz_window.h"

int jz::launch_window_fwd(const Plan& pl, hipStream_t st) { return launch_window<OP_FWD>(pl, st); }
int jz::launch_window_fwd_stats(const Plan& pl, hipStream_t st) { return launch_window<OP_FWD_STATS>(pl, st); }
