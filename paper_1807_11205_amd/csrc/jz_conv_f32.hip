// FP32-storage / FP32-accumulate convolution forward, backward-data, backward-weight and fully connected GEMMs for
// gfx950: the single-precision side of the paper's FP32-versus-mixed-precision throughput comparison (Jia et al. 2018,
// Section 5.4, Table 9).  Same operations, layouts and GEMM view as the FP16 path (jz_igemm.h):
//
//   D[m][n] = sum_k A(m,k) * B(n,k), 24-bit operands, sums in FP32.
//
// Channel counts that are multiples of 4 run on the kernels of jz_f32_split.h (products of bfloat16 parts with the accuracy of FP32)
// and jz_f32_dma.h (FP32 matrix instructions), whichever choose_tiling_f32 expects to be faster (strided multi-tap backward-data as
// one unit-stride launch per residue of the stride, strided 1x1 backward-data with a scattering epilogue); other counts run on them
// through copies with the channels rounded up to 4, where that adds at most half to the work (3-channel stems).
//
// What is left (a filter smaller than its stride in backward-data; 1 or 2 channels; callers without room for the copies) runs on
// igemm_f32_kernel below: a workgroup of 4 wavefronts (2 x 2) owns a BM x BN output tile, walks the reduction in
// tiles of 16 with v_mfma_f32_32x32x2_f32, and stages operands global -> registers -> LDS, double buffered.  Both tiles sit in
// LDS as [k][row] (row contiguous), so an MFMA operand (lane l: row l % 32, k l / 32) is one conflict-free 4-byte read per
// lane.  Operands that are contiguous along the reduction in memory (x / dy gathered per pixel, the forward filter) are
// fetched as 4 consecutive k of one row and written to LDS as 4 scalars; operands contiguous along their own row index
// (the filter in backward-data, dy and x in backward-weight) as 4 consecutive rows of one k, one 16-byte write.  With
// channel counts that are not multiples of 4 the same kernel fetches element by element (VEC = false).  Addressing is the
// plain index definition of each operation, bounds-checked per fetched vector.
//
// Split reductions (any operation with too few output tiles for the chip) leave FP32 partial sums in the workspace, added in a
// fixed order by splitk_reduce_f32: deterministic.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <type_traits>

#include "jz_f32_plan.h"
#include "jz_internal.h"
#include "jz_plan_cache.h"

namespace {
using namespace jz;

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int F_THREADS = 256;
constexpr int F_BK = 16;  // reduction elements per tile

#include "jz_lds_dma.h"

// Address of the gathered tensor's element for pixel `pix` of the (n, OH, OW) grid at filter tap `tap`, channel c, or
// nullptr when the tap falls outside the image (or, backward-data, when no output pixel reads the input pixel through it).
template <int OP>
__device__ __forceinline__ const float* gather_addr(const ConvGeom& g, const float* T, unsigned pix, unsigned tap, unsigned c) {
  const unsigned n = fd_div(pix, g.d_ohow);
  const unsigned rem = pix - n * (unsigned)(g.OH * g.OW);
  const unsigned oh = fd_div(rem, g.d_ow);
  const unsigned ow = rem - oh * (unsigned)g.OW;
  const unsigned r = fd_div(tap, g.d_s);
  const unsigned s = tap - r * (unsigned)g.S;
  int ih, iw;
  if (OP == OP_BWD_DATA) {
    const int th = (int)oh + g.ph - (int)r, tw = (int)ow + g.pw - (int)s;
    if (th < 0 || tw < 0) return nullptr;
    ih = (int)fd_div((unsigned)th, g.d_sh);
    iw = (int)fd_div((unsigned)tw, g.d_sw);
    if (ih * g.sh != th || iw * g.sw != tw) return nullptr;
  } else {
    ih = (int)oh * g.sh - g.ph + (int)r;
    iw = (int)ow * g.sw - g.pw + (int)s;
  }
  if ((unsigned)ih >= (unsigned)g.IH || (unsigned)iw >= (unsigned)g.IW) return nullptr;
  return T + ((size_t)(n * g.IH + ih) * g.IW + iw) * g.IC + c;
}

// A(m, k) and B(n, k) of the three operations (table in jz_igemm.h): address or nullptr (= zero)
template <int OP>
__device__ __forceinline__ const float* addrA(const F32Args& a, int m, int k) {
  if (m >= a.M || k >= a.Kred) return nullptr;
  if (OP == OP_BWD_WEIGHT) return a.A + (size_t)k * a.M + m;  // dy[(n,p,q)][k_out]
  const unsigned tap = fd_div((unsigned)k, a.g.d_ic);
  return gather_addr<OP>(a.g, a.A, (unsigned)m, tap, (unsigned)k - tap * (unsigned)a.g.IC);
}
template <int OP>
__device__ __forceinline__ const float* addrB(const F32Args& a, int n, int k) {
  if (n >= a.N || k >= a.Kred) return nullptr;
  if (OP == OP_FWD) return a.B + (size_t)n * a.Kred + k;  // w[k_out][(r,s,c)]
  if (OP == OP_BWD_DATA) {                                  // w[k_out][r][s][c] read as B(c, (r,s,k_out))
    const unsigned tap = fd_div((unsigned)k, a.g.d_ic);
    const unsigned ko = (unsigned)k - tap * (unsigned)a.g.IC;
    return a.B + ((size_t)ko * (a.g.R * a.g.S) + tap) * a.N + n;
  }
  const unsigned tap = fd_div((unsigned)n, a.g.d_ic);  // backward-weight: n = (r,s,c), k = (n,p,q)
  return gather_addr<OP_FWD>(a.g, a.B, (unsigned)k, tap, (unsigned)n - tap * (unsigned)a.g.IC);
}

// Four operand values: along k (KC = true: row fixed, k .. k+3) or along the row index (row .. row+3, k fixed).  VEC:
// the four lie in one aligned 16-byte piece of memory and share their validity (the host checked the divisibility that
// guarantees it).
template <int OP, bool IS_A, bool KC, bool VEC>
__device__ __forceinline__ float4 fetch4(const F32Args& a, int row, int k) {
  auto at = [&](int r, int kk) { return IS_A ? addrA<OP>(a, r, kk) : addrB<OP>(a, r, kk); };
  if (VEC) {
    const float* p = at(row, k);
    return p ? *reinterpret_cast<const float4*>(p) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float* p = KC ? at(row, k + j) : at(row + j, k);
    v[j] = p ? *p : 0.0f;
  }
  return make_float4(v[0], v[1], v[2], v[3]);
}

template <int OP, bool VEC, int BM, int BN>
__global__ __launch_bounds__(F_THREADS) void igemm_f32_kernel(F32Args a) {
  constexpr bool A_KC = OP != OP_BWD_WEIGHT, B_KC = OP == OP_FWD;
  constexpr int TM = BM / 64, TN = BN / 64;      // 32x32 MFMA tiles per wavefront (2 x 2 wavefronts)
  constexpr int PA = BM + 32, PB = BN + 32;      // LDS row pitch: k and k+1 land in different halves of the banks
  constexpr int QA = BM * F_BK / 4 / F_THREADS;  // 4-element fetches per thread and tile
  constexpr int QB = BN * F_BK / 4 / F_THREADS;
  static_assert(QA >= 1 && QB >= 1, "tile too small for 256 loaders");
  __shared__ __align__(16) float sA[2][F_BK][PA];
  __shared__ __align__(16) float sB[2][F_BK][PB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  unsigned L = blockIdx.x;
  const int tiles_mn = a.tiles_m * a.tiles_n;
  const int split = (int)(L / (unsigned)tiles_mn);
  L -= (unsigned)split * (unsigned)tiles_mn;
  const int m0 = (int)(L / (unsigned)a.tiles_n) * BM;
  const int n0 = (int)(L % (unsigned)a.tiles_n) * BN;
  const int kt_begin = split * a.kt_per_split;
  const int kt_end = kt_begin + a.kt_per_split < a.nkt ? kt_begin + a.kt_per_split : a.nkt;

  // fetch q of this thread: KC operand: row = f % ROWS, k quad = f / ROWS; row-contiguous operand: row quad = f % (ROWS/4),
  // k = f / (ROWS/4); f = q * 256 + tid.  Consecutive lanes: consecutive rows (KC: conflict-free scalar LDS writes) or
  // consecutive row quads (coalesced 16-byte accesses).
  float4 ra[QA], rb[QB];
  auto fetch = [&](int kt) {
    const int k0 = kt * F_BK;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int f = q * F_THREADS + tid;
      ra[q] = A_KC ? fetch4<OP, true, true, VEC>(a, m0 + f % BM, k0 + 4 * (f / BM))
                   : fetch4<OP, true, false, VEC>(a, m0 + 4 * (f % (BM / 4)), k0 + f / (BM / 4));
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int f = q * F_THREADS + tid;
      rb[q] = B_KC ? fetch4<OP, false, true, VEC>(a, n0 + f % BN, k0 + 4 * (f / BN))
                   : fetch4<OP, false, false, VEC>(a, n0 + 4 * (f % (BN / 4)), k0 + f / (BN / 4));
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int f = q * F_THREADS + tid;
      if (A_KC) {
        const int row = f % BM, kq = 4 * (f / BM);
        sA[buf][kq][row] = ra[q].x; sA[buf][kq + 1][row] = ra[q].y; sA[buf][kq + 2][row] = ra[q].z; sA[buf][kq + 3][row] = ra[q].w;
      } else {
        *reinterpret_cast<float4*>(&sA[buf][f / (BM / 4)][4 * (f % (BM / 4))]) = ra[q];
      }
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int f = q * F_THREADS + tid;
      if (B_KC) {
        const int row = f % BN, kq = 4 * (f / BN);
        sB[buf][kq][row] = rb[q].x; sB[buf][kq + 1][row] = rb[q].y; sB[buf][kq + 2][row] = rb[q].z; sB[buf][kq + 3][row] = rb[q].w;
      } else {
        *reinterpret_cast<float4*>(&sB[buf][f / (BN / 4)][4 * (f % (BN / 4))]) = rb[q];
      }
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  if (kt_begin < kt_end) {
    fetch(kt_begin);
    stash(0);
  }
  __syncthreads();
  int buf = 0;
  const int arow = wm * (BM / 2) + (lane & 31), brow = wn * (BN / 2) + (lane & 31), kh = lane >> 5;
  for (int kt = kt_begin; kt < kt_end; ++kt) {
    const bool more = kt + 1 < kt_end;
    if (more) fetch(kt + 1);  // in flight while this tile is multiplied
#pragma unroll
    for (int ks = 0; ks < F_BK / 2; ++ks) {
      float fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = sA[buf][2 * ks + kh][arow + 32 * i];
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = sB[buf][2 * ks + kh][brow + 32 * j];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          // n operand in the first slot: each lane then owns 4 consecutive n for one m (row = lane % 32)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    if (more) stash(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }

  // accumulator register r of tile (i,j): m = wrow + 32 i + lane % 32, n = wcol + 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4
  float* out = a.splits > 1 ? a.Dpart + (size_t)split * a.M * a.N : a.D;
  const bool vec = (a.N & 3) == 0;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm * (BM / 2) + 32 * i + (lane & 31);
    if (m >= a.M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int n = n0 + wn * (BN / 2) + 32 * j + 8 * q4 + 4 * (lane >> 5);
        float* dst = out + (size_t)m * a.N + n;
        if (vec && n + 3 < a.N) {
          *reinterpret_cast<float4*>(dst) = make_float4(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < a.N) dst[e] = acc[i][j][4 * q4 + e];
        }
      }
  }
}

// D[i] = sum_s part[s][i].  A workgroup owns 256 / G groups of four consecutive outputs and G = 2^lg lanes per group: lane g
// adds splits g, g + G, ... in that order, four loads in flight, then the lane sums are added in lane order (deterministic:
// the order depends on splits and G only).  One thread per output that walked through all splits one load at a time took
// 11 us per launch of the ResNet-50 step.
__global__ __launch_bounds__(256) void splitk_reduce_f32(const float* __restrict__ part, float* __restrict__ out, long long MN, int splits, int lg) {
  __shared__ float4 red[256];
  const int G = 1 << lg, Q = 256 >> lg;
  const int q = threadIdx.x & (Q - 1), lane = threadIdx.x >> (8 - lg);
  const long long i = ((long long)blockIdx.x * Q + q) * 4;
  const bool full = i + 3 < MN && (MN & 3) == 0;  // every split's slab starts on a 16-byte boundary
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (full) {
    int k = lane;
    for (; k + 3 * G < splits; k += 4 * G) {
      float4 t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = *reinterpret_cast<const float4*>(part + (size_t)(k + u * G) * MN + i);
#pragma unroll
      for (int u = 0; u < 4; ++u) { s.x += t[u].x; s.y += t[u].y; s.z += t[u].z; s.w += t[u].w; }
    }
    for (; k < splits; k += G) {
      const float4 t = *reinterpret_cast<const float4*>(part + (size_t)k * MN + i);
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
  } else if (i < MN) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = lane; k < splits; k += G)
      for (int e = 0; e < 4 && i + e < MN; ++e) v[e] += part[(size_t)k * MN + i + e];
    s = make_float4(v[0], v[1], v[2], v[3]);
  }
  if (G > 1) {
    red[threadIdx.x] = s;
    __syncthreads();
    if (lane != 0) return;
    for (int l = 1; l < G; ++l) {
      const float4 t = red[l * Q + q];
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
  }
  if (full) {
    *reinterpret_cast<float4*>(out + i) = s;
  } else {
    const float v[4] = {s.x, s.y, s.z, s.w};
    for (int e = 0; e < 4 && i + e < MN; ++e) out[i + e] = v[e];
  }
}

// Channel counts that are not multiples of 4: rows of C floats copied to rows of C4 (zeros behind), `real` of the rows
// present in the source; two tensors per launch (blockIdx.y), one 16-byte chunk per thread and pass.  And the way back.
struct WidenF32 {
  const float* src[2];
  float* dst[2];
  long long chunks[2], real_rows[2];
  int C[2];
  FastDiv d_cpr[2];
};
__global__ __launch_bounds__(256) void widen_channels_f32(WidenF32 a) {
  const int t = blockIdx.y, C = a.C[t];
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < a.chunks[t]; i += (long long)gridDim.x * 256) {
    const unsigned row = fd_div((unsigned)i, a.d_cpr[t]);
    const int c0 = (int)((unsigned)i - row * a.d_cpr[t].d) * 4;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = row < a.real_rows[t] && c0 + e < C ? a.src[t][(size_t)row * C + c0 + e] : 0.f;
    *reinterpret_cast<float4*>(a.dst[t] + i * 4) = make_float4(v[0], v[1], v[2], v[3]);
  }
}
__global__ __launch_bounds__(256) void narrow_channels_f32(const float* __restrict__ src, float* __restrict__ dst, long long n, FastDiv d_c, int C4) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
    const unsigned row = fd_div((unsigned)i, d_c);
    dst[i] = src[(size_t)row * C4 + ((unsigned)i - row * d_c.d)];
  }
}

size_t up256f(size_t x) { return (x + 255) & ~size_t(255); }

void finish_geometry_f32(ConvGeom& g) {
  g.tap_rep = 0;
  if (g.R * g.S <= 32)
    for (int r = 0; r < g.R; ++r) g.tap_rep |= 1u << (r * g.S);
  g.row_pitch = g.IW * g.IC; g.pix_step = g.IC; g.s_step = g.IC;
  g.d_ohow = make_fastdiv((unsigned)(g.OH * g.OW));
  g.d_ow = make_fastdiv((unsigned)g.OW);
  g.d_ic = make_fastdiv((unsigned)g.IC);
  g.d_s = make_fastdiv((unsigned)g.S);
  g.d_sh = make_fastdiv((unsigned)g.sh);
  g.d_sw = make_fastdiv((unsigned)g.sw);
}

// whether the gathered operand needs the kernel's per-lane tap arithmetic: a k tile must lie inside one tap, the masks hold 32
// taps, and descriptor plus padding margin must stay below the out-of-range mark
bool needs_gen_f32(const PlanF32& pl) {
  const ConvGeom& g = pl.args.g;
  if (pl.op == JZ_BWD_WEIGHT) return false;
  const long long margin = 4ll * g.IC * ((long long)(pl.op == JZ_FWD ? g.ph : g.R - 1) * g.IW + (pl.op == JZ_FWD ? g.pw : g.S - 1));
  return g.IC % FD_BK != 0 || g.R * g.S > 32 || (long long)pl.bytesA + margin >= 0xfffffff0ll;
}

// How often the large sums of a result are rounded: once per k tile of a run that is added up in the accumulators, once per such run where
// there are several (window_run_f32), once per part of a split reduction.  A sum of n terms added one by one is off by sqrt(n / 2) roundings
// of its final size, so is a sum of such sums, and variances add: plans compare by this number.  18x22x22 pixels, 128 -> 64, backward-data, 36
// k tiles: three splits of 12 without a window 15 and a relative error of 8.46e-8; with one, whole, in runs of 18 20 and 9.66e-8, of 9 13 and
// 7.85e-8.
int roundings_f32(bool window, int bn, int k_tiles, int parts) {
  const int run = window && bn == 64 ? window_run_f32(k_tiles) : k_tiles;
  return run + (run < k_tiles ? k_tiles / run : 0) + (parts > 1 ? parts : 0);
}

// Form, tile and split of a launch, by a cost model in microseconds.  Forms: operands in three bfloat16 parts (jz_f32_split.h), or
// the FP32 matrix instructions (jz_f32_dma.h), which are ahead in launches of a few microseconds and for reductions of one k tile
// only.  A compute unit works through its share of the workgroups, `resident` of them at a time; its vector or matrix pipes bound it
// at `thr` a k tile, a workgroup whose waits nothing covers takes `lat`, and the operands have to come from memory once: the launch
// takes the fourth-power norm of the three.  A split adds a second launch and re-reading the partial sums.
// Which part of the reduction is split: all of it, or only the rows of tiles that would start the last, unfilled round of
// workgroups (full_rows rows of tiles are then computed whole).  Batch 64 makes 98 * 2^n tiles, 784 for most layers of
// ResNet-50: four rounds of 256 instead of 3.06 (14 x 14, 256 -> 256, 3x3 with FP32 instructions: 135 -> 118 us forward, 139 -> 124
// backward-data).
// The constants (forward, backward-data, backward-weight with plain and with gathered x) are least-squares fits to timings of
// both forms, every tile and up to six splits of each on 3100 operations: ResNet-50 of both kinds and AlexNet at batch sizes from 2
// to 128, random layers.  On a quarter of them left out of the fit the choices were 0.8-1.2 % slower than the best.  parts_ahead:
// by how much the first form has to be faster to be taken, about what the model is wrong by on launches of 6-8 us, where it gains
// nothing and its choices were up to 0.6 us slower without.  limit: bytes of partial sums.
// 3x3 layers on their own grid have a third form, the pixels of a tile taken apart once for all taps (jz_f32_window.h, with timings); its constants
// are fits to ten layers in up to eleven splits each: ResNet-50's four at batch 64 and 24, 13x13x384 at 128, 28x28x512 at 16.  They are on the
// safe side: over 4343 forced plans of 270 random layers the model says 6 ... 10 % too much in the mean.  Over 500 random layers on a plan with a window the
// choices take 0.87 of the time of the plan without in the geometric mean, 1.03 at worst.
// Its 128-wide tiles are not offered parts of 18 k tiles, whose first window nothing covers: 1.06 of the time without in the mean of 42 layers (1.00 ...
// 1.12), where the model has them ahead.  Parts of 36 take 0.96 (107 layers; forward on no more workgroups than compute units 0.98, 0.93 ... 1.05
// of which 0.04 are the difference of two timings), longer ones 0.91 (111).
// 7x7x512 at batch 64 stays on the other forms (100 tiles, and splits only in steps of 18 k tiles).
void choose_tiling_f32(PlanF32* pl, bool may_split, bool fixed_tile = false, size_t limit = 0, bool may_parts = true) {
  struct Tile { bool parts, window; int bm, bn, resident; double lat[4], thr[4], prologue[4], own[4]; };
  static const Tile tiles[] = {
      {true, false, 128, 128, 2, {0.427, 0.537, 0.629, 0.756}, {0.572, 0.567, 0.533, 0.612}, {3.458, 2.504, 3.066, 2.014}, {0.883, 0.888, 2.248, 0.346}},
      {true, false, 128, 64, 3, {0.324, 0.382, 0.463, 0.489}, {0.323, 0.327, 0.340, 0.359}, {1.365, 1.111, 1.112, 0.101}, {0.622, 0.637, 0.989, 0.079}},
      {true, false, 64, 128, 3, {0.329, 0.395, 0.476, 0.560}, {0.328, 0.332, 0.349, 0.381}, {1.581, 1.099, 1.412, 1.033}, {0.456, 0.442, 1.133, 0.316}},
      {true, false, 64, 64, 5, {0.254, 0.303, 0.309, 0.333}, {0.188, 0.191, 0.206, 0.215}, {0.000, 0.000, 0.000, 0.000}, {0.303, 0.312, 0.439, 0.000}},
      {false, false, 128, 128, 2, {0.935, 1.023, 1.020, 1.181}, {0.889, 0.919, 0.907, 1.065}, {1.798, 1.665, 2.516, 2.486}, {2.607, 2.429, 2.484, 0.813}},
      {false, false, 128, 64, 3, {0.513, 0.615, 0.604, 0.685}, {0.461, 0.464, 0.488, 0.532}, {0.137, 0.147, 0.335, 0.128}, {1.206, 1.280, 0.974, 0.474}},
      {false, false, 64, 128, 3, {0.489, 0.579, 0.630, 0.800}, {0.456, 0.476, 0.494, 0.565}, {0.159, 0.239, 0.687, 0.228}, {1.199, 1.092, 0.988, 0.657}},
      {false, false, 64, 64, 5, {0.283, 0.342, 0.352, 0.421}, {0.235, 0.246, 0.255, 0.288}, {0.037, 0.039, 0.043, 0.030}, {0.512, 0.548, 0.429, 0.187}},
      {true, true, 128, 128, 2, {0.46, 0.48}, {0.50, 0.51}, {3.5, 3.5}, {1.5, 1.5}},
      {true, true, 128, 64, 2, {0.31, 0.32}, {0.265, 0.267}, {1.4, 1.4}, {2.0, 2.0}}};
  const double parts_ahead = 0.3;
  // FP32 instructions, parts; the last two per megabyte (2.3: anything from 2 to 3.1 fits as well)
  static const double fixed[2][4] = {{4.76, 4.82, 5.10, 5.64}, {4.347, 5.147, 4.159, 5.374}},
                      reduce_launch[2][4] = {{3.38, 3.81, 3.59, 4.01}, {2.3, 2.3, 3.543, 4.043}},
                      reduce_byte[2][4] = {{0.187, 0.169, 0.160, 0.208}, {0.244, 0.234, 0.218, 0.285}},
                      byte[2][4] = {{0.135, 0.127, 0.135, 0.230}, {0.120, 0.088, 0.120, 0.185}};
  F32Args& a = pl->args;
  a.nkt = (a.Kred + FD_BK - 1) / FD_BK;
  const int c = pl->op == JZ_FWD ? 0 : pl->op == JZ_BWD_DATA ? 1 : a.bw_linear ? 2 : 3;
  const ConvGeom& g = a.g;
  const bool may_window = pl->op != JZ_BWD_WEIGHT && !pl->gen && !a.sc_on && g.R == 3 && g.S == 3 && g.ph == 1 && g.pw == 1 && g.sh == 1 && g.sw == 1 &&
                          g.IH == g.OH && g.IW == g.OW && g.IW <= 63 && g.IC % (2 * FD_BK) == 0 &&
                          // offsets of the rows of a last tile's window that lie behind the tensor must not wrap into it
                          (long long)pl->bytesA + 4ll * g.IC * (128 + g.IW + 1) < 0xfffffff0ll;
  const double in = 1e-6 * ((double)std::min<long long>(pl->bytesA, 4ll * a.M * a.Kred) + (double)std::min<long long>(pl->bytesB, 4ll * a.N * a.Kred));
  // k tiles that a workgroup takes: two at a time in parts, nine taps of twice 16 channels out of a window
  auto even = [](const Tile& t, int k) { return t.window ? (k + 17) / 18 * 18 : t.parts ? k + (k & 1) : k; };
  auto p4 = [](double x) { return (x * x) * (x * x); };
  auto rounds = [](double w) { return w <= 4.0 ? ceil(w) : w + 0.5; };  // many small rounds even out
  double best = 1e30;
  double most_part = 0.0;  // bytes of partial sums of the plan without a window: the workspace that a layer asks for does not grow with one,
  int most_rounded = 0;    // and no sum is rounded more often
  int bsp = 1, bfull = 0, kt_step = 1;
  for (const Tile& t : tiles) {
    if (fixed_tile && (t.parts != pl->parts || t.bm != pl->BM || t.bn != pl->BN)) continue;
    if (t.window && !(may_window && may_split)) continue;
    if (t.parts && (!may_parts || a.nkt == 1)) continue;  // half of its work would be done on zeros
    const long long tm = (a.M + t.bm - 1) / t.bm, tn = (a.N + t.bn - 1) / t.bn, slots = 256 * t.resident;
    for (int sp = 1; sp <= 512; sp = sp < 8 ? sp + 1 : sp + sp / 4) {
      if (sp > 1 && (!may_split || a.nkt / sp < 8)) break;
      const int kps = even(t, (a.nkt + sp - 1) / sp), real = (a.nkt + kps - 1) / kps;
      // full rows of tiles: none (all of them without a split), or as many as fill whole rounds
      const long long round_rows = tm * tn / 256 * 256 / tn;
      for (int tail = 0; tail < 2; ++tail) {
        if (tail && (sp == 1 || round_rows == 0 || round_rows >= tm)) break;
        const long long full = sp == 1 ? tm : tail ? round_rows : 0, wf = full * tn, ws = (tm - full) * tn * real;
        const double n1 = tail ? ceil(wf / 256.0) : rounds(wf / 256.0), n2 = tail ? ceil(ws / 256.0) : rounds(ws / 256.0);
        const double t_thr = n1 * (t.own[c] + t.thr[c] * even(t, a.nkt)) + n2 * (t.own[c] + t.thr[c] * kps);
        const long long l1 = (wf + slots - 1) / slots, l2 = wf > 0 ? (wf + ws + slots - 1) / slots - l1 : (ws + slots - 1) / slots;
        const double t_lat = l1 * (t.prologue[c] + t.lat[c] * even(t, a.nkt)) + l2 * (t.prologue[c] + t.lat[c] * kps);
        const double out = 4e-6 * a.M * a.N, part = sp > 1 ? 4e-6 * real * (double)(a.M - full * t.bm) * a.N : 0.0;
        if (1e6 * part > (t.window ? most_part : (double)limit)) continue;
        // the rows that are rounded most often in a plan with a window, least often in one without
        int rounded = sp > 1 ? roundings_f32(t.window, t.bn, kps, real) : roundings_f32(t.window, t.bn, a.nkt, 1);
        if (sp > 1 && full > 0) {
          const int whole = roundings_f32(t.window, t.bn, a.nkt, 1);
          rounded = t.window ? std::max(rounded, whole) : std::min(rounded, whole);
        }
        if (t.window && rounded > most_rounded) continue;
        if (t.window && t.bn == 128 && sp > 1 && kps < 36) continue;
        const double t_mem = byte[t.parts][c] * (in + part + (full > 0 ? out : 0.0));
        double time = fixed[t.parts][c] + (t.parts ? parts_ahead : 0.0) + sqrt(sqrt(p4(t_thr) + p4(t_lat) + p4(t_mem)));
        if (sp > 1) time += reduce_launch[t.parts][c] + reduce_byte[t.parts][c] * part;
        if (time < best) {
          best = time;
          if (!t.window) { most_part = 1e6 * part; most_rounded = rounded; }
          pl->parts = t.parts; pl->window = t.window; pl->BM = t.bm; pl->BN = t.bn;
          pl->rounded = rounded; pl->may_round = most_rounded;
          kt_step = t.window ? 18 : t.parts ? 2 : 1;
          bsp = sp; bfull = (int)full;
        }
      }
    }
  }
  a.tiles_m = (a.M + pl->BM - 1) / pl->BM;
  a.tiles_n = (a.N + pl->BN - 1) / pl->BN;
  a.kt_per_split = ((a.nkt + bsp - 1) / bsp + kt_step - 1) / kt_step * kt_step;
  a.splits = (a.nkt + a.kt_per_split - 1) / a.kt_per_split;
  a.full_rows = a.splits > 1 ? bfull : a.tiles_m;
  const int tail_tiles = (a.tiles_m - a.full_rows) * a.tiles_n;
  a.d_tiles_mn = make_fastdiv((unsigned)(tail_tiles > 0 ? tail_tiles : 1));
  a.d_tiles_n = make_fastdiv((unsigned)a.tiles_n);
}

// One residue (ca, cb) of the stride of a strided multi-tap backward-data layer: the input pixels h = ca + sh i, w = cb + sw l
// meet the taps r = r0 + sh j, s = s0 + sw k only, at dy row i + (ca + ph) / sh - j: a unit-stride layer over those taps.
// false: no such pixel.
bool class_args_f32(const jz_conv_desc* d, const PlanF32& base, int ca, int cb, PlanF32* pl) {
  const int sh = d->stride_h, sw = d->stride_w;
  const int Ha = (d->H - ca + sh - 1) / sh, Wb = (d->W - cb + sw - 1) / sw;
  if (Ha <= 0 || Wb <= 0) return false;
  const int r0 = (ca + d->pad_h) % sh, s0 = (cb + d->pad_w) % sw;
  *pl = base;
  F32Args& a = pl->args;
  a.A = a.B = nullptr;
  a.D = a.Dpart = nullptr;
  ConvGeom& g = a.g;
  g.R = (d->R - r0 + sh - 1) / sh; g.S = (d->S - s0 + sw - 1) / sw;
  g.OH = Ha; g.OW = Wb; g.sh = g.sw = 1;
  g.ph = (ca + d->pad_h) / sh; g.pw = (cb + d->pad_w) / sw;
  finish_geometry_f32(g);
  a.M = d->N * Ha * Wb; a.Kred = g.R * g.S * d->K;
  a.w_tap0 = r0 * d->S + s0; a.w_tap_r = sh * d->S; a.w_tap_s = sw;
  a.sc_on = 1; a.sc_H = d->H; a.sc_W = d->W; a.sc_sh = sh; a.sc_sw = sw; a.sc_oh = ca; a.sc_ow = cb; a.sc_fill = 0;
  choose_tiling_f32(pl, false, true);  // one tile for all residues: the layer's
  return true;
}

int compute_plan_f32(int op, const jz_conv_desc* d, PlanF32* pl, size_t limit, bool may_parts = true);

// Channels rounded up to 4 on copies, when that adds at most half to the multiply-adds.
void plan_widened_f32(int op, const jz_conv_desc* d, PlanF32* pl) {
  jz_conv_desc w = *d;
  w.C = (d->C + 3) & ~3;
  if (op != JZ_FWD) w.K = (d->K + 3) & ~3;  // forward takes any number of output channels
  if ((w.C == d->C && w.K == d->K) || (double)w.C * w.K > 1.5 * d->C * d->K) return;
  PlanF32 in;
  if (compute_plan_f32(op, &w, &in, kPartialSumLimit) != JZ_OK || !in.dma) return;
  const bool x_wide = w.C != d->C, y_wide = w.K != d->K;
  const size_t nx = up256f((size_t)d->N * d->H * d->W * w.C * 4), nw = up256f((size_t)w.K * d->R * d->S * w.C * 4);
  const size_t ny = op == JZ_FWD ? 0 : up256f(pl->bytesA / d->K * w.K);
  if (op == JZ_FWD) { pl->wide_a = x_wide ? nx : 0; pl->wide_b = nw; }
  else if (op == JZ_BWD_DATA) { pl->wide_a = y_wide ? ny : 0; pl->wide_b = nw; pl->wide_d = x_wide ? nx : 0; }
  else { pl->wide_a = y_wide ? ny : 0; pl->wide_b = x_wide ? nx : 0; pl->wide_d = nw; }
  pl->widen = true;
  pl->wide = w;
  const size_t need = pl->wide_a + pl->wide_b + pl->wide_d + in.ws_bytes;
  if (need > pl->ws_bytes) pl->ws_bytes = need;
}

int out_dim(int in, int pad, int f, int st) { return (in + 2 * pad - f) / st + 1; }

int compute_plan_f32(int op, const jz_conv_desc* d, PlanF32* pl, size_t limit, bool may_parts) {
  if (!d) return JZ_ERR_NULL;
  if (op != JZ_FWD && op != JZ_BWD_DATA && op != JZ_BWD_WEIGHT) return JZ_ERR_UNSUPPORTED;
  if (d->N <= 0 || d->H <= 0 || d->W <= 0 || d->C <= 0 || d->K <= 0 || d->R <= 0 || d->S <= 0 || d->stride_h <= 0 ||
      d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0)
    return JZ_ERR_SHAPE;
  if (d->pad_h >= d->R || d->pad_w >= d->S) return JZ_ERR_SHAPE;
  if (d->H + 2 * d->pad_h < d->R || d->W + 2 * d->pad_w < d->S) return JZ_ERR_SHAPE;
  const int P = out_dim(d->H, d->pad_h, d->R, d->stride_h), Q = out_dim(d->W, d->pad_w, d->S, d->stride_w);
  if (P <= 0 || Q <= 0) return JZ_ERR_SHAPE;
  const long long lim = (1ll << 30) - 1;  // the same bound as the FP16 path: GEMM dimensions and pixel indices fit 32 bits
  const long long nx = (long long)d->N * d->H * d->W * d->C, ny = (long long)d->N * P * Q * d->K,
                  nw = (long long)d->K * d->R * d->S * d->C;
  if (nx > lim || ny > lim || nw > lim) return JZ_ERR_UNSUPPORTED;
  F32Args& a = pl->args;
  ConvGeom& g = a.g;
  pl->op = op;
  g.R = d->R; g.S = d->S; g.sh = d->stride_h; g.sw = d->stride_w; g.ph = d->pad_h; g.pw = d->pad_w;
  g.kvalid = 0; g.tap_rep = 0;
  if (op == JZ_FWD) {
    a.M = d->N * P * Q; a.N = d->K; a.Kred = d->R * d->S * d->C;
    g.IH = d->H; g.IW = d->W; g.IC = d->C; g.OH = P; g.OW = Q;
    pl->vec = d->C % 4 == 0;
    pl->bytesA = 4 * nx; pl->bytesB = 4 * nw; pl->bytesD = 4 * ny;
  } else if (op == JZ_BWD_DATA) {
    a.M = d->N * d->H * d->W; a.N = d->C; a.Kred = d->R * d->S * d->K;
    g.IH = P; g.IW = Q; g.IC = d->K; g.OH = d->H; g.OW = d->W;
    pl->vec = d->K % 4 == 0 && d->C % 4 == 0;
    pl->bytesA = 4 * ny; pl->bytesB = 4 * nw; pl->bytesD = 4 * nx;
  } else {
    a.M = d->K; a.N = d->R * d->S * d->C; a.Kred = d->N * P * Q;
    g.IH = d->H; g.IW = d->W; g.IC = d->C; g.OH = P; g.OW = Q;
    pl->vec = d->K % 4 == 0 && d->C % 4 == 0;
    pl->bytesA = 4 * ny; pl->bytesB = 4 * nx; pl->bytesD = 4 * nw;  // A = dy, B = x
  }
  // a grid of one row or column never steps: the kernels' sums of coordinates and strides then stay far below 2^31
  if (op != JZ_BWD_DATA && P == 1) g.sh = 1;
  if (op != JZ_BWD_DATA && Q == 1) g.sw = 1;
  const bool strided = d->stride_h > 1 || d->stride_w > 1;
  a.bytesA = (unsigned)pl->bytesA;
  a.bytesB = (unsigned)pl->bytesB;
  a.w_taps = d->R * d->S; a.w_tap0 = 0; a.w_tap_r = d->S; a.w_tap_s = 1;
  a.sc_on = 0; a.sc_H = a.sc_W = 0; a.sc_sh = a.sc_sw = 1; a.sc_oh = a.sc_ow = 0; a.sc_fill = 0;
  const bool single_tap = d->R == 1 && d->S == 1;
  pl->dma = pl->vec && (op != JZ_BWD_DATA || !strided || single_tap || (d->R >= d->stride_h && d->S >= d->stride_w));
  pl->classes = pl->dma && op == JZ_BWD_DATA && strided && !single_tap;
  if (pl->dma && op == JZ_BWD_DATA && strided && single_tap) {
    // only the input pixels (p sh, q sw) receive gradient: the GEMM runs over the output pixels, its epilogue scatters
    a.M = d->N * P * Q;
    g.OH = P; g.OW = Q; g.sh = g.sw = 1;
    a.sc_on = 1; a.sc_H = d->H; a.sc_W = d->W; a.sc_sh = d->stride_h; a.sc_sw = d->stride_w; a.sc_fill = 1;
  }
  finish_geometry_f32(g);
  a.bw_same = op == JZ_BWD_WEIGHT && !single_tap && !strided && P == d->H && Q == d->W &&
              (long long)pl->bytesB + 4ll * d->C * ((long long)d->pad_h * d->W + d->pad_w) < 0xfffffff0ll;
  a.bw_linear = op == JZ_BWD_WEIGHT && single_tap && !strided && d->pad_h == 0 && d->pad_w == 0;
  if (pl->dma) {
    pl->gen = needs_gen_f32(*pl);
    if (pl->classes) {  // every input pixel meets one residue's taps only
      const int all = a.Kred;
      a.Kred = all / (d->stride_h * d->stride_w) + 1;
      choose_tiling_f32(pl, false, false, 0, may_parts);
      a.Kred = all;
      a.splits = 1;
    } else {
      choose_tiling_f32(pl, !a.sc_on, false, limit, may_parts);
    }
    pl->ws_bytes = a.splits > 1 ? (size_t)a.splits * (a.M - a.full_rows * pl->BM) * a.N * sizeof(float) : 0;
    pl->plain_ws_bytes = pl->ws_bytes;
    return JZ_OK;
  }
  a.full_rows = 0;
  // Tile and split: 128 x 128 tiles where they give the chip (256 compute units, two workgroups each) enough
  // workgroups, else 64 x 64; then split the reduction until about 512 workgroups exist, never shorter than 8 k tiles.
  a.nkt = (a.Kred + F_BK - 1) / F_BK;
  auto tiles = [&](int t) { return (long long)((a.M + t - 1) / t) * ((a.N + t - 1) / t); };
  pl->BM = pl->BN = tiles(128) >= 384 ? 128 : 64;
  a.tiles_m = (a.M + pl->BM - 1) / pl->BM;
  a.tiles_n = (a.N + pl->BM - 1) / pl->BM;
  long long want = 512 / tiles(pl->BM);
  if (want > a.nkt / 8) want = a.nkt / 8;
  if (want > 256) want = 256;
  want = std::min(want, (long long)(limit / ((size_t)a.M * a.N * sizeof(float))));
  if (want < 1) want = 1;
  a.kt_per_split = (int)((a.nkt + want - 1) / want);
  a.splits = (a.nkt + a.kt_per_split - 1) / a.kt_per_split;
  pl->ws_bytes = a.splits > 1 ? (size_t)a.splits * a.M * a.N * sizeof(float) : 0;
  pl->plain_ws_bytes = pl->ws_bytes;
  plan_widened_f32(op, d, pl);
  return JZ_OK;
}

int make_plan_f32(int op, const jz_conv_desc* d, PlanF32* pl, size_t limit = kPartialSumLimit, bool may_parts = true) {
  if (!d) return JZ_ERR_NULL;
  constexpr int kNoParts = 16;
  return cached_plan(1, PlanKey{may_parts ? op : op + kNoParts, -1, -1, limit, *d}, pl,
                     [&](PlanF32* p) { return compute_plan_f32(op, d, p, limit, may_parts); });
}
// Whether a layer runs in less room than its plan asks for (runs_with_fewer_splits): as the plan of the FP32 instructions has it,
// so that which calls are taken does not depend on which form is faster.
bool runs_in_f32(int op, const jz_conv_desc* d, size_t room) {
  PlanF32 pl;
  if (make_plan_f32(op, d, &pl, kPartialSumLimit, false) != JZ_OK) return false;
  if (room >= pl.plain_ws_bytes) return true;
  return make_plan_f32(op, d, &pl, room, false) == JZ_OK && room >= pl.plain_ws_bytes &&
         runs_with_fewer_splits(op, pl.args.M, pl.args.N, pl.args.splits);
}
// residues of larger strides are planned anew by every call: they would fill the table
constexpr int kKeptResidues = 16;
bool make_class_plan_f32(const jz_conv_desc* d, const PlanF32& base, int ca, int cb, PlanF32* pl) {
  if ((long long)d->stride_h * d->stride_w > kKeptResidues) return class_args_f32(d, base, ca, cb, pl);
  return cached_plan(1, PlanKey{JZ_BWD_DATA, ca, cb, 0, *d}, pl, [&](PlanF32* p) { return class_args_f32(d, base, ca, cb, p) ? 1 : 0; }) != 0;
}

template <int OP>
int launch_f32(const PlanF32& pl, hipStream_t st) {
  const F32Args& a = pl.args;
  if (pl.dma) return OP == OP_FWD ? launch_f32_fwd(pl, st) : OP == OP_BWD_DATA ? launch_f32_bwd_data(pl, st) : launch_f32_bwd_weight(pl, st);
  const dim3 grid((unsigned)a.tiles_m * (unsigned)a.tiles_n * (unsigned)a.splits), block(F_THREADS);
  if constexpr (OP == OP_BWD_DATA)
    if (pl.vec) {  // a filter smaller than its stride
      if (pl.BM == 128) hipLaunchKernelGGL((igemm_f32_kernel<OP, true, 128, 128>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((igemm_f32_kernel<OP, true, 64, 64>), grid, block, 0, st, a);
      return jz::launch_status();
    }
  if (pl.BM == 128) hipLaunchKernelGGL((igemm_f32_kernel<OP, false, 128, 128>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((igemm_f32_kernel<OP, false, 64, 64>), grid, block, 0, st, a);
  return jz::launch_status();
}

int run_widened_f32(int op, const jz_conv_desc* d, const PlanF32& pl, const void* A, const void* B, void* D, void* ws, size_t ws_bytes, void* stream);

// A, B in the kernel's order: FWD (x, w), BWD_DATA (dy, w), BWD_WEIGHT (dy, x)
int run_f32(int op, const jz_conv_desc* d, const void* A, const void* B, void* D, void* ws, size_t ws_bytes, void* stream) {
  PlanF32 pl;
  int rc = make_plan_f32(op, d, &pl);
  if (rc != JZ_OK) return rc;
  if (!A || !B || !D) return JZ_ERR_NULL;
  if (!aligned16(A) || !aligned16(B) || !aligned16(D) || (ws && !aligned16(ws))) return JZ_ERR_ALIGN;
  if (overlaps(D, pl.bytesD, A, pl.bytesA) || overlaps(D, pl.bytesD, B, pl.bytesB)) return JZ_ERR_ALIAS;
  if (pl.widen && (!ws || ws_bytes < pl.ws_bytes)) {  // no room for the copies
    pl.widen = false;
    pl.ws_bytes = pl.plain_ws_bytes;
  }
  const size_t room = ws ? ws_bytes : 0;
  if (room < pl.ws_bytes) {  // fewer splits
    if ((rc = make_plan_f32(op, d, &pl, room)) != JZ_OK) return rc;
    if (pl.widen) {
      pl.widen = false;
      pl.ws_bytes = pl.plain_ws_bytes;
    }
    if (room < pl.ws_bytes || !runs_in_f32(op, d, room)) return JZ_ERR_WORKSPACE;
  }
  if (pl.ws_bytes > 0 && (overlaps(ws, pl.ws_bytes, A, pl.bytesA) || overlaps(ws, pl.ws_bytes, B, pl.bytesB) ||
                          overlaps(ws, pl.ws_bytes, D, pl.bytesD)))
    return JZ_ERR_ALIAS;
  if (pl.widen) return run_widened_f32(op, d, pl, A, B, D, ws, ws_bytes, stream);
  hipStream_t st = static_cast<hipStream_t>(stream);
  F32Args& a = pl.args;
  a.A = static_cast<const float*>(A);
  a.B = static_cast<const float*>(B);
  a.D = static_cast<float*>(D);
  a.Dpart = static_cast<float*>(ws);
  if (pl.classes) {
    // residues in launches of at most FD_MAX_SET, those with the most taps (the last ones to start would end last) first: along
    // an axis they have ceil(R / stride) taps or one less
    F32Set set{};
    int k = 0;
    auto flush = [&] {
      for (int j = k; j < FD_MAX_SET; ++j) {
        set.c[j] = set.c[0];
        set.first[j + 1] = set.first[j];
      }
      k = 0;
      return launch_f32_bwd_data(pl, st, &set);
    };
    const int Rm = (d->R + d->stride_h - 1) / d->stride_h, Sm = (d->S + d->stride_w - 1) / d->stride_w;
    const bool rows_first = (Rm - 1) * Sm >= Rm * (Sm - 1);
    const int taps[4][2] = {{Rm, Sm}, {rows_first ? Rm - 1 : Rm, rows_first ? Sm : Sm - 1}, {rows_first ? Rm : Rm - 1, rows_first ? Sm - 1 : Sm}, {Rm - 1, Sm - 1}};
    for (const auto& t : taps)
      for (int ca = 0; ca < d->stride_h; ++ca) {
        if ((d->R - (ca + d->pad_h) % d->stride_h + d->stride_h - 1) / d->stride_h != t[0]) continue;
        for (int cb = 0; cb < d->stride_w; ++cb) {
          PlanF32 cp;
          if ((d->S - (cb + d->pad_w) % d->stride_w + d->stride_w - 1) / d->stride_w != t[1] || !make_class_plan_f32(d, pl, ca, cb, &cp)) continue;
          F32Args& c = set.c[k];
          c = cp.args;
          c.A = a.A; c.B = a.B; c.D = a.D; c.Dpart = nullptr;
          set.first[k + 1] = set.first[k] + (unsigned)(c.tiles_m * c.tiles_n);
          if (++k == FD_MAX_SET && (rc = flush()) != JZ_OK) return rc;
        }
      }
    return k > 0 ? flush() : JZ_OK;
  }
  if (op == JZ_FWD) rc = launch_f32<OP_FWD>(pl, st);
  else if (op == JZ_BWD_DATA) rc = launch_f32<OP_BWD_DATA>(pl, st);
  else rc = launch_f32<OP_BWD_WEIGHT>(pl, st);
  if (rc != JZ_OK) return rc;
  if (a.splits > 1) {
    const long long first = (long long)a.full_rows * pl.BM * a.N, MN = (long long)a.M * a.N - first, groups = (MN + 3) / 4;
    int lg = 0;  // lanes per output group: enough workgroups to cover the chip first, then shorten each thread's chain
    while (lg < 5 && (2 << lg) <= a.splits && (groups + (256 >> lg) - 1) / (256 >> lg) < 1024) ++lg;
    hipLaunchKernelGGL(splitk_reduce_f32, dim3((unsigned)((groups + (256 >> lg) - 1) / (256 >> lg))), dim3(256), 0, st,
                       (const float*)a.Dpart, a.D + first, MN, a.splits, lg);
    rc = jz::launch_status();
  }
  return rc;
}

int run_widened_f32(int op, const jz_conv_desc* d, const PlanF32& pl, const void* A, const void* B, void* D, void* ws, size_t ws_bytes,
                    void* stream) {
  const jz_conv_desc& w = pl.wide;
  const long long RS = (long long)d->R * d->S, npix = (long long)d->N * d->H * d->W;
  const long long nout = (long long)d->N * out_dim(d->H, d->pad_h, d->R, d->stride_h) * out_dim(d->W, d->pad_w, d->S, d->stride_w);
  char* const base = static_cast<char*>(ws);
  hipStream_t st = static_cast<hipStream_t>(stream);
  WidenF32 wa{};
  int nt = 0;
  long long most = 0;
  auto copy = [&](const void* src, char* dst, long long rows, long long real_rows, int c, int c4) {
    wa.src[nt] = static_cast<const float*>(src);
    wa.dst[nt] = reinterpret_cast<float*>(dst);
    wa.chunks[nt] = rows * (c4 / 4);
    wa.real_rows[nt] = real_rows;
    wa.C[nt] = c;
    wa.d_cpr[nt] = make_fastdiv((unsigned)(c4 / 4));
    if (wa.chunks[nt] > most) most = wa.chunks[nt];
    ++nt;
  };
  const void* a2 = A;
  const void* b2 = B;
  if (pl.wide_a) {
    a2 = base;
    if (op == JZ_FWD) copy(A, base, npix, npix, d->C, w.C);
    else copy(A, base, nout, nout, d->K, w.K);
  }
  if (pl.wide_b) {
    b2 = base + pl.wide_a;
    if (op == JZ_BWD_WEIGHT) copy(B, base + pl.wide_a, npix, npix, d->C, w.C);
    else copy(B, base + pl.wide_a, w.K * RS, d->K * RS, d->C, w.C);
  }
  int rc = JZ_OK;
  if (nt > 0) {
    const long long blocks = (most + 255) / 256;
    hipLaunchKernelGGL(widen_channels_f32, dim3((unsigned)(blocks < 8192 ? blocks : 8192), (unsigned)nt), dim3(256), 0, st, wa);
    if ((rc = jz::launch_status()) != JZ_OK) return rc;
  }
  const size_t used = pl.wide_a + pl.wide_b + pl.wide_d;
  void* const d2 = pl.wide_d ? base + pl.wide_a + pl.wide_b : D;
  rc = run_f32(op, &w, a2, b2, d2, ws_bytes > used ? base + used : nullptr, ws_bytes - used, stream);
  if (rc != JZ_OK || !pl.wide_d) return rc;
  const long long n = op == JZ_BWD_DATA ? npix * d->C : (long long)d->K * RS * d->C;
  const long long blocks = (n + 255) / 256;
  hipLaunchKernelGGL(narrow_channels_f32, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, st, static_cast<const float*>(d2),
                     static_cast<float*>(D), n, make_fastdiv((unsigned)d->C), w.C);
  return jz::launch_status();
}

int fc_desc_f32(int mode, int batch, int in_features, int out_features, jz_conv_desc* d) {
  if (mode != JZ_FWD && mode != JZ_BWD_DATA && mode != JZ_BWD_WEIGHT) return JZ_ERR_UNSUPPORTED;
  if (batch <= 0 || in_features <= 0 || out_features <= 0) return JZ_ERR_SHAPE;
  *d = jz_conv_desc{batch, 1, 1, in_features, out_features, 1, 1, 1, 1, 0, 0};  // a 1x1 convolution over a 1x1 image
  return JZ_OK;
}

}  // namespace

extern "C" int jz_conv2d_f32_workspace_bytes(int op, const jz_conv_desc* desc, size_t* bytes) {
  if (!bytes) return JZ_ERR_NULL;
  PlanF32 pl;
  int rc = make_plan_f32(op, desc, &pl);
  if (rc != JZ_OK) return rc;
  *bytes = pl.ws_bytes;
  return JZ_OK;
}

extern "C" int jz_conv2d_f32_describe_plan(int op, const jz_conv_desc* desc, char* text, size_t text_bytes) {
  if (!text || text_bytes == 0) return JZ_ERR_NULL;
  PlanF32 pl;
  int rc = make_plan_f32(op, desc, &pl);
  if (rc != JZ_OK) return rc;
  const bool widen = pl.widen;
  if (widen) {
    const jz_conv_desc w = pl.wide;
    pl = PlanF32{};
    if ((rc = make_plan_f32(op, &w, &pl)) != JZ_OK) return rc;
  }
  const F32Args& a = pl.args;
  char form[80];
  if (pl.window) snprintf(form, sizeof form, "parts, window of %d rows, rounded %d times (%d without)", f32_window_rows(a.g), pl.rounded, pl.may_round);
  else snprintf(form, sizeof form, "%s%s", !pl.dma ? "operands through registers" : pl.parts ? "parts" : "FP32 instructions", pl.gen ? ", per-lane taps" : "");
  snprintf(text, text_bytes, "M %d N %d K %d: %s%s%s, tile %dx%d, %d x %d tiles, %d splits of %d k tiles, %d rows of tiles whole", a.M, a.N, a.Kred,
           widen ? "copies of 4 n channels, " : "", form, pl.classes ? ", residues of the stride" : "", pl.BM, pl.BN, a.tiles_m, a.tiles_n, a.splits,
           a.kt_per_split, a.full_rows);
  return JZ_OK;
}

extern "C" int jz_conv2d_fwd_f32(const jz_conv_desc* desc, const float* x32, const float* w32, float* y32, void* ws,
                                 size_t ws_bytes, void* hip_stream) {
  return run_f32(JZ_FWD, desc, x32, w32, y32, ws, ws_bytes, hip_stream);
}

extern "C" int jz_conv2d_bwd_data_f32(const jz_conv_desc* desc, const float* dy32, const float* w32, float* dx32, void* ws,
                                      size_t ws_bytes, void* hip_stream) {
  return run_f32(JZ_BWD_DATA, desc, dy32, w32, dx32, ws, ws_bytes, hip_stream);
}

extern "C" int jz_conv2d_bwd_weight_f32(const jz_conv_desc* desc, const float* x32, const float* dy32, float* dw32, void* ws,
                                        size_t ws_bytes, void* hip_stream) {
  return run_f32(JZ_BWD_WEIGHT, desc, dy32, x32, dw32, ws, ws_bytes, hip_stream);  // A = dy, B = x
}

extern "C" int jz_gemm_fc_f32_workspace_bytes(int mode, int batch, int in_features, int out_features, size_t* bytes) {
  jz_conv_desc d;
  int rc = fc_desc_f32(mode, batch, in_features, out_features, &d);
  if (rc != JZ_OK) return rc;
  return jz_conv2d_f32_workspace_bytes(mode, &d, bytes);
}

extern "C" int jz_gemm_fc_f32(int mode, int batch, int in_features, int out_features, const float* a32, const float* b32,
                              float* out32, void* ws, size_t ws_bytes, void* hip_stream) {
  jz_conv_desc d;
  int rc = fc_desc_f32(mode, batch, in_features, out_features, &d);
  if (rc != JZ_OK) return rc;
  // FWD: (x, w) ; BWD_DATA: (dy, w) ; BWD_WEIGHT: (dy, x) -- already the kernel's (A, B) order in every mode
  return run_f32(mode, &d, a32, b32, out32, ws, ws_bytes, hip_stream);
}
