// Weight gradients of several layers in one launch (jz_conv2d_bwd_weight_set): kernels and variant dispatch.
//
// A layer's weight gradient alone has few output tiles and a long reduction, so it fills the chip only with its reduction split,
// at the price of partial sums, a second launch that adds them and two launches' start-up for microseconds of work; in a
// backward pass nothing waits for it.  Here the workgroups of up to kWgradSet layers follow one another, those with the longest
// reductions first, so that together they fill the chip with few splits or none.  Measured in a training step (ResNet-50, one
// stream, all but the stem's in sets): 8 images of 64 x 64 pixels 53 launches of 5.0 us and 13 reductions -> 5 launches of 7-15
// us and 2 reductions, the step 1618 -> 1414 us; 22 x 96 x 96 2053 -> 1727 us; 55 x 224 x 224 6.23 -> 6.02 ms.
#include "jz_igemm_kernels.h"

namespace {
template <int BM, int BN, int TBK, int NST, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void igemm_wgrad_set_kernel(WgradSet s) {
  int k = 0;
#pragma unroll
  for (int j = 1; j < kWgradSet; ++j) k += blockIdx.x >= s.first[j] ? 1 : 0;  // behind the last member: first[j] is the grid size
  const unsigned block = blockIdx.x - s.first[k], blocks = s.first[k + 1] - s.first[k];
  if (s.g[k].bw_x == BW_MATRIX) igemm_dma_body<OP_BWD_WEIGHT, BM, BN, TBK, NST, false, WGM, WGN, false, false, BW_MATRIX>(s.g[k], block, blocks);
  else if (s.g[k].bw_x == BW_SAME) igemm_dma_body<OP_BWD_WEIGHT, BM, BN, TBK, NST, false, WGM, WGN, false, false, BW_SAME>(s.g[k], block, blocks);
  else igemm_dma_body<OP_BWD_WEIGHT, BM, BN, TBK, NST, false, WGM, WGN, false, false, BW_GATHER>(s.g[k], block, blocks);
}

template <int BM, int BN, int TBK, int NST, int WGM, int WGN>
int launch(const WgradSet& set, hipStream_t st) {
  constexpr size_t ring_bytes = (size_t)NST * (BM + BN) * 2 * TBK;
  constexpr size_t epi_bytes = (size_t)BM / dma_epass(BM, BN) * (BN + 8) * sizeof(unsigned short);
  constexpr size_t smem = ring_bytes > epi_bytes ? ring_bytes : epi_bytes;
  static std::atomic<bool> lds_set{false};
  if (!jz::allow_lds(reinterpret_cast<const void*>(&igemm_wgrad_set_kernel<BM, BN, TBK, NST, WGM, WGN>), smem, lds_set)) return JZ_ERR_LAUNCH;
  hipLaunchKernelGGL((igemm_wgrad_set_kernel<BM, BN, TBK, NST, WGM, WGN>), dim3(set.first[kWgradSet]), dim3(64 * WGM * WGN), smem, st, set);
  return jz::launch_status();
}
}  // namespace

int jz::launch_bwd_weight_set(const Plan& v, const WgradSet& set, hipStream_t st) {
  if (v.BM == 128 && v.BN == 128 && v.bk == 32 && v.waves == 8 && v.nst == 4) return launch<128, 128, 32, 4, 4, 2>(set, st);
  if (v.BM == 64 && v.BN == 64 && v.bk == 64 && v.waves == 4) return launch<64, 64, 64, 4, 2, 2>(set, st);
  if (v.BM == 64 && v.BN == 64 && v.bk == 32 && v.waves == 4 && v.nst == 4) return launch<64, 64, 32, 4, 2, 2>(set, st);
  return JZ_ERR_UNSUPPORTED;
}
