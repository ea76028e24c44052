// What the FP32 planner (jz_conv_f32.hip) hands to the kernels of jz_f32_split.h and jz_f32_dma.h and to their launchers, which live in
// one translation unit per operation (jz_conv_f32_fwd.hip, jz_conv_f32_bwd_data.hip, jz_conv_f32_bwd_weight.hip) so that they compile
// in parallel.
#pragma once
#include <hip/hip_runtime.h>

#include "jz.h"
#include "jz_igemm.h"

namespace jz {

struct F32Args {
  const float* A;
  const float* B;
  float* D;      // [M][N], written where the reduction is not split
  float* Dpart;  // [splits][rows][N], the rows whose reduction is split
  int M, N, Kred;
  int nkt, kt_per_split, splits, tiles_m, tiles_n;
  ConvGeom g;
  // those kernels': descriptor bounds, tile decomposition, where tap (r, s) of the launch sits among the w_taps taps
  // of a filter (backward-data), and the scatter of strided backward-data as in GemmArgs
  unsigned bytesA, bytesB;
  int full_rows;  // rows of tiles whose reduction is not split (all of them: splits == 1)
  FastDiv d_tiles_mn, d_tiles_n;  // d_tiles_mn: the tiles of the other rows
  int w_taps, w_tap0, w_tap_r, w_tap_s;
  int bw_same;    // backward-weight, unit stride, output grid = input grid: x is read at a constant pixel distance per tap
  int bw_linear;  // backward-weight of a 1x1 unit-stride unpadded layer: x is a plain [Kred][IC] matrix
  int sc_on, sc_H, sc_W, sc_sh, sc_sw, sc_oh, sc_ow, sc_fill;
};

constexpr int FD_BK = 16;   // floats per k tile: a KC row is 64 bytes
constexpr int FD_NST = 4;   // ring stages

// how an operand is gathered: x and dy per pixel in forward and backward-data, x in backward-weight
enum { F32_MASKS = 0, F32_TAPS = 1, F32_MATRIX = 0, F32_SAME = 1, F32_GATHER = 2 };

struct PlanF32 {
  int op = 0;
  bool vec = false;
  bool dma = false;      // a kernel of jz_f32_split.h or jz_f32_dma.h
  bool gen = false;      // ... with per-lane tap arithmetic
  bool parts = false;    // ... its operands taken apart for the bfloat16 matrix instructions (jz_f32_split.h)
  bool window = false;   // ... and the pixels under a tile once for all taps (jz_f32_window.h)
  bool classes = false;  // strided multi-tap backward-data: one launch per residue of the stride (class_args_f32)
  bool widen = false;    // channels rounded up to 4 on copies: `wide` is the layer that runs
  int BM = 128, BN = 128;
  int rounded = 0, may_round = 0;  // roundings of the large sums (roundings_f32): of this plan, and of the one without a window
  F32Args args{};
  size_t ws_bytes = 0, bytesA = 0, bytesB = 0, bytesD = 0;
  jz_conv_desc wide{};
  size_t wide_a = 0, wide_b = 0, wide_d = 0;  // bytes of the copies (0: that operand is used where it is)
  size_t plain_ws_bytes = 0;                  // what the same layer needs without them
};

// Several launches in one: the residues of the stride of a strided backward-data layer, each of which alone fills a part of
// the chip (ResNet-50 v1.5 at batch 20, 3x3 512 -> 512 on 14x14: 128 workgroups each).
constexpr int FD_MAX_SET = 4;
struct F32Set {
  F32Args c[FD_MAX_SET];
  unsigned first[FD_MAX_SET + 1];  // workgroup numbers of member k: first[k] .. first[k + 1] - 1
};

// k tiles that a workgroup of jz_f32_window.h with 64-wide tiles adds up before it starts a new sum, of the k_tiles that it works through: one
// window or two, whichever makes for fewer roundings (a run's, and one per run).
__host__ __device__ inline int window_run_f32(int k_tiles) { return 9 + k_tiles / 9 <= 18 + k_tiles / 18 ? 9 : 18; }
// rows of window that a tile of a layer on jz_f32_window.h gets: its 128 pixels and what their taps reach
inline int f32_window_rows(const ConvGeom& g) { return 128 + 2 * g.IW + 2 <= 192 ? 192 : 256; }

int launch_f32_fwd(const PlanF32& pl, hipStream_t st);
int launch_f32_bwd_data(const PlanF32& pl, hipStream_t st, const F32Set* set = nullptr);  // set: these problems instead of the plan's own
int launch_f32_bwd_weight(const PlanF32& pl, hipStream_t st);

}  // namespace jz
