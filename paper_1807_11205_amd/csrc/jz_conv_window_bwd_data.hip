// The window kernel (jz_window.h), backward-data: see jz_conv_plan.h
#include "jz_igemm_kernels.h"
#include "jz_window.h"

int jz::launch_window_bwd_data(const Plan& pl, hipStream_t st) { return launch_window<OP_BWD_DATA>(pl, st); }
int jz::launch_window_bwd_data_stats(const Plan& pl, hipStream_t st) { return launch_window<OP_BWD_DATA_STATS>(pl, st); }
int jz::launch_window_bwd_data_block_end(const Plan& pl, hipStream_t st) { return launch_window<OP_BWD_DATA_BLOCK_END>(pl, st); }
