// Kernel instantiations and variant dispatch of one implicit-GEMM operation (a translation unit of its own so that
// the operations compile in parallel).
#include "jz_igemm_kernels.h"

int jz::launch_bwd_data(const Plan& pl, hipStream_t st, const GemmSet* set) { return launch_op<OP_BWD_DATA>(pl, st, set); }
