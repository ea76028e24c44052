// FP16-storage / FP32-accumulate convolution forward, backward-data, backward-weight and the fully
// connected GEMMs (Jia et al. 2018, Section 4.1) as one implicit-GEMM kernel family for gfx950.
//
// This file holds the host side: the planner (tile shape, split of the reduction, which kernel), argument checks, the
// extern "C" entry points, and the small helper kernels (split-K reduction, the 4-channel padded copy for 3-channel
// stems).  The GEMM kernels and their epilogue are in jz_igemm_kernels.h / jz_igemm_dma.h, instantiated in one
// translation unit per operation (jz_conv_fwd.hip, ...).
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

#include "jz_conv_plan.h"
#include "jz_plan_cache.h"
#include "jz_sumsq.h"

namespace {
using namespace jz;

constexpr int BK = 64;  // k tile depth of the element-wise kernel

#include "jz_bn_math.h"

// ---------------------------------------------------------------------------------------------
// small-channel layers (C <= 4: the 3-channel stems of ResNet-50 and AlexNet)
// ---------------------------------------------------------------------------------------------
// With 3 channels a filter tap is 6 bytes: nothing to vectorise.  But in NHWC the S taps of one filter row are
// adjacent in memory, so the input is copied once into a zero-padded 4-channel image xp[N][H+2ph][Wp][4]; one filter
// row of an output pixel is then ONE contiguous, 16-byte aligned run of 4*S halves starting at pixel q*stride_w
// (needs an even stride_w), and the layer becomes an ordinary implicit GEMM whose "taps" are the R filter rows and
// whose "channels" are that run, rounded up to the k tile (32 or 64; backward-weight, where the runs are columns of the
// GEMM: to whole 16-byte chunks).  The filter is repacked to match
// (w'[k][r][4 s + c], zeros elsewhere); for backward-weight the GEMM produces dw' in that layout and the real
// entries are copied out.

// One launch does both copies.  A workgroup writes PAD_PAIRS consecutive pixel pairs of one image of xp (a pair is one
// 16-byte store; Wp is even).  Padding only adds pixels, so the image pixels among them are one contiguous run of x,
// which comes in through LDS in whole aligned 16-byte chunks whatever C and the row length are, all loads of a thread
// in flight together.  Bound by memory; 2-byte loads straight from x (a 3-channel row starts on any even byte) kept the
// load units busy instead: 227 x 227 x 3 x 128 (92 MB moved) took 26 us that way, 6.5 us more than this; 512 pairs
// measure the same.  The workgroups behind the images' (present when w != nullptr) repack the filter: w[K][R][S][C] ->
// wp[K][R][KT] with wp[k][r][4 s + c] = w[k][r][s][c], zero elsewhere.
constexpr int PAD_PAIRS = 1024, PAD_THREADS = 256;
struct PadArgs {
  const unsigned short *x, *w;
  unsigned short *xp, *wp;
  int N, H, W, C, Hp, Wp, ph, pw;
  int K, R, S, KT, chunk_major;
  unsigned pairs, groups;  // pixel pairs per image of xp, workgroups per image
  FastDiv d_row;           // Wp / 2
};
__global__ __launch_bounds__(PAD_THREADS) void pad_to_c4(PadArgs a) {
  const int z = blockIdx.x / a.groups, C = a.C;
  if (z >= a.N) {
    const int i = (blockIdx.x - a.N * a.groups) * PAD_THREADS + threadIdx.x;
    if (i >= a.K * a.R * a.KT) return;
    int j = i % a.KT, kr = i / a.KT;
    int s = j >> 2, c = j & 3;
    // chunk_major (the patch kernel's layout): wq[r][j / 8][k][j % 8], 16-byte chunks of one filter row side by side per k
    const int k = kr / a.R, r = kr - k * a.R;
    const int dst = a.chunk_major ? ((r * (a.KT / 8) + (j >> 3)) * a.K + k) * 8 + (j & 7) : i;
    a.wp[dst] = (s < a.S && c < C) ? a.w[((size_t)kr * a.S + s) * C + c] : (unsigned short)0;
    return;
  }
  constexpr int CHUNKS = PAD_PAIRS + 2;  // 2 PAD_PAIRS pixels of up to 4 halves, and a partial chunk at each end
  __shared__ __align__(16) unsigned short in[CHUNKS * 8];
  const unsigned q0 = (blockIdx.x - z * a.groups) * PAD_PAIRS, q1 = min(q0 + PAD_PAIRS, a.pairs);
  auto before = [&](unsigned q) {  // pixels of the image in front of padded pair q
    const int hp = (int)fd_div(q, a.d_row), wi = 2 * (int)(q - hp * a.d_row.d) - a.pw, h = hp - a.ph;
    return h < 0 ? 0 : h >= a.H ? a.H * a.W : h * a.W + min(max(wi, 0), a.W);
  };
  const size_t image = (size_t)z * a.H * a.W * C, total = (size_t)a.N * a.H * a.W * C;
  const int first = before(q0);
  const size_t g0 = image + (size_t)first * C, g1 = image + (size_t)before(q1) * C, a0 = g0 & ~(size_t)7;
  constexpr int ITERS = (CHUNKS + PAD_THREADS - 1) / PAD_THREADS;
  uint4 t[ITERS];
#pragma unroll
  for (int i = 0; i < ITERS; ++i) {
    const size_t g = a0 + 8 * (size_t)(i * PAD_THREADS + threadIdx.x);
    if (g + 8 <= total) {
      if (g < g1) t[i] = *reinterpret_cast<const uint4*>(a.x + g);
    } else if (g < g1) {  // the last chunk of x where x does not end on a 16-byte boundary
      unsigned short e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) e[k] = g + k < total ? a.x[g + k] : (unsigned short)0;
      t[i] = make_uint4((unsigned)e[0] | ((unsigned)e[1] << 16), (unsigned)e[2] | ((unsigned)e[3] << 16),
                        (unsigned)e[4] | ((unsigned)e[5] << 16), (unsigned)e[6] | ((unsigned)e[7] << 16));
    }
  }
#pragma unroll
  for (int i = 0; i < ITERS; ++i) {
    const int c = i * PAD_THREADS + threadIdx.x;
    if (a0 + 8 * (size_t)c < g1) *reinterpret_cast<uint4*>(&in[8 * c]) = t[i];
  }
  __syncthreads();
  const int lead = (int)(g0 - a0) - first * C;  // in[lead + C * pixel]: a pixel of the image
#pragma unroll
  for (int i = 0; i < PAD_PAIRS / PAD_THREADS; ++i) {
    const unsigned q = q0 + i * PAD_THREADS + threadIdx.x;
    if (q >= q1) break;
    const int hp = (int)fd_div(q, a.d_row), wi = 2 * (int)(q - hp * a.d_row.d) - a.pw, h = hp - a.ph;
    unsigned v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if ((unsigned)h < (unsigned)a.H) {
#pragma unroll
      for (int p = 0; p < 2; ++p)
        if ((unsigned)(wi + p) < (unsigned)a.W) {
          const unsigned short* px = &in[lead + C * (h * a.W + wi + p)];
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (c < C) v[4 * p + c] = px[c];
        }
    }
    *reinterpret_cast<uint4*>(a.xp + ((size_t)z * a.pairs + q) * 8) =
        make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
  }
}

// Channel counts that are not multiples of 8: rows of C halves copied to rows of C8 (zeros behind), `real` of `rows` rows
// present in the source (the others are all zero: a filter's missing output channels).  Two tensors per launch
// (blockIdx.y); one 16-byte chunk of the copy per thread and pass.  A pass over the operands, memory-bound.
struct WidenArgs {
  const unsigned short* src[2];
  unsigned short* dst[2];
  long long chunks[2], real_rows[2];
  int C[2];
  jz::FastDiv d_cpr[2];
};
__global__ __launch_bounds__(256) void widen_channels(WidenArgs a) {
  const int t = blockIdx.y;
  const unsigned cpr = a.d_cpr[t].d;
  const int C = a.C[t];
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < a.chunks[t]; i += (long long)gridDim.x * 256) {
    const unsigned row = jz::fd_div((unsigned)i, a.d_cpr[t]);  // at most 2^30 / 8 chunks
    const int c0 = (int)((unsigned)i - row * cpr) * 8;
    unsigned short v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = row < a.real_rows[t] && c0 + e < C ? a.src[t][(size_t)row * C + c0 + e] : (unsigned short)0;
    *reinterpret_cast<uint4*>(a.dst[t] + i * 8) = make_uint4((unsigned)v[0] | ((unsigned)v[1] << 16), (unsigned)v[2] | ((unsigned)v[3] << 16),
                                                             (unsigned)v[4] | ((unsigned)v[5] << 16), (unsigned)v[6] | ((unsigned)v[7] << 16));
  }
}
// the way back: dst[row][0..C) = src[row][0..C) of rows C8 long
__global__ __launch_bounds__(256) void narrow_channels(const unsigned short* __restrict__ src, unsigned short* __restrict__ dst,
                                                       long long n, jz::FastDiv d_c, int C8) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
    const unsigned row = jz::fd_div((unsigned)i, d_c);
    dst[i] = src[(size_t)row * C8 + ((unsigned)i - row * d_c.d)];
  }
}

// dwp[K][R][KT] -> dw[K][R][S][C]
__global__ __launch_bounds__(256) void unpack_filter_c4(const unsigned short* __restrict__ dwp, unsigned short* __restrict__ dw,
                                                        int K, int R, int S, int C, int KT) {
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= K * R * S * C) return;
  int c = i % C, t = i / C;
  int s = t % S, kr = t / S;
  dw[i] = dwp[(size_t)kr * KT + 4 * s + c];
}

// D16[i] = RNE16( sum_s part[s][i] ).  A workgroup owns 256 / G groups of four consecutive outputs and G = 2^lg
// "split lanes": lane g adds splits g, g + G, g + 2G, ... in that order, then the G lane sums are added in lane order.
// The order depends only on (splits, G), so the result is deterministic.  Splitting the reduction over lanes matters
// for the small outputs that need many splits: with one thread per output group those launches were latency-bound.
// KT4 > 0 (small-channel backward-weight): the sums are dw'[K][R][4 KT4] of the padded 4-channel problem; group
// (kr, s) of four goes to dw[kr][s][0..C) when s < S and nowhere otherwise, which saves the separate unpacking launch.
__device__ __forceinline__ void splitk_reduce_body(const float* __restrict__ part, unsigned short* __restrict__ out, long long MN, int splits,
                                                   int lg, int KT4, int S, int C, unsigned block) {
  __shared__ float4 red[256];
  const int G = 1 << lg, Q = 256 >> lg;
  const int q = threadIdx.x & (Q - 1), g = threadIdx.x >> (8 - lg);
  const long long i = ((long long)block * Q + q) * 4;
  // 16-byte loads need every split's slab to start on a 16-byte boundary: MN a multiple of 4
  const bool full = i + 3 < MN && (MN & 3) == 0;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < MN) {
    if (full) {
      int k = g;
      for (; k + 3 * G < splits; k += 4 * G) {  // four loads in flight per thread
        float4 t0 = *reinterpret_cast<const float4*>(part + (size_t)k * MN + i);
        float4 t1 = *reinterpret_cast<const float4*>(part + (size_t)(k + G) * MN + i);
        float4 t2 = *reinterpret_cast<const float4*>(part + (size_t)(k + 2 * G) * MN + i);
        float4 t3 = *reinterpret_cast<const float4*>(part + (size_t)(k + 3 * G) * MN + i);
        s.x += t0.x; s.y += t0.y; s.z += t0.z; s.w += t0.w;
        s.x += t1.x; s.y += t1.y; s.z += t1.z; s.w += t1.w;
        s.x += t2.x; s.y += t2.y; s.z += t2.z; s.w += t2.w;
        s.x += t3.x; s.y += t3.y; s.z += t3.z; s.w += t3.w;
      }
      for (; k < splits; k += G) {
        float4 t = *reinterpret_cast<const float4*>(part + (size_t)k * MN + i);
        s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
      }
    } else {  // ragged end of the matrix: element-wise
      float* sv = reinterpret_cast<float*>(&s);
      for (int k = g; k < splits; k += G)
        for (int e = 0; e < 4 && i + e < MN; ++e) sv[e] += part[(size_t)k * MN + i + e];
    }
  }
  if (G > 1) {
    red[threadIdx.x] = s;
    __syncthreads();
    if (g != 0) return;
    for (int gg = 1; gg < G; ++gg) {
      float4 t = red[gg * Q + q];
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
  }
  if (i >= MN) return;
  _Float16 h[4] = {(_Float16)s.x, (_Float16)s.y, (_Float16)s.z, (_Float16)s.w};
  if (KT4 > 0) {  // MN is a multiple of 4 here
    const long long grp = i >> 2, kr = grp / KT4;
    const int sx = (int)(grp - kr * KT4);
    if (sx < S) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c < C) {
          unsigned short bts;
          __builtin_memcpy(&bts, &h[c], 2);
          out[(kr * S + sx) * C + c] = bts;
        }
    }
    return;
  }
  if (full) {
    uint2 pk;
    __builtin_memcpy(&pk, h, 8);
    *reinterpret_cast<uint2*>(out + i) = pk;
  } else {
    for (int e = 0; e < 4 && i + e < MN; ++e) {
      unsigned short bts;
      __builtin_memcpy(&bts, &h[e], 2);
      out[i + e] = bts;
    }
  }
}

__global__ __launch_bounds__(256) void splitk_reduce(const float* __restrict__ part, unsigned short* __restrict__ out,
                                                     long long MN, int splits, int lg, int KT4, int S, int C) {
  splitk_reduce_body(part, out, MN, splits, lg, KT4, S, C, blockIdx.x);
}

// The same for several weight gradients in one launch.
struct ReduceSet {
  const float* part[kWgradSet];
  unsigned short* out[kWgradSet];
  long long MN[kWgradSet];
  int splits[kWgradSet], lg[kWgradSet];
  unsigned first[kWgradSet + 1];
};
__global__ __launch_bounds__(256) void splitk_reduce_set(ReduceSet s) {
  int k = 0;
#pragma unroll
  for (int j = 1; j < kWgradSet; ++j) k += blockIdx.x >= s.first[j] ? 1 : 0;
  splitk_reduce_body(s.part[k], s.out[k], s.MN[k], s.splits[k], s.lg[k], 0, 0, 0, blockIdx.x - s.first[k]);
}

// splitk_reduce that also leaves the sum of squares of the FP16 values it writes (and whether any of them is Inf / NaN)
// in a sink: the weight gradient's norm for Eq. 1, taken while the gradient is still in registers.  Same sums, same order,
// same bits in `out` as splitk_reduce.  A workgroup walks several slabs of outputs (grid stride) and contributes once, so
// that the number of atomic additions per tensor stays in the hundreds.
__global__ __launch_bounds__(256) void splitk_reduce_sumsq(const float* __restrict__ part, unsigned short* __restrict__ out,
                                                           long long MN, int splits, int lg, int KT4, int S, int C,
                                                           long long slabs, jz::SumsqSink sink) {
  __shared__ float4 red[256];
  __shared__ unsigned long long wsum[5];
  if (threadIdx.x < 5) wsum[threadIdx.x] = 0ull;
  __syncthreads();
  const int G = 1 << lg, Q = 256 >> lg;
  const int q = threadIdx.x & (Q - 1), g = threadIdx.x >> (8 - lg);
  jz::SumsqAcc sq;
  int bad = 0;
  for (long long slab = blockIdx.x; slab < slabs; slab += gridDim.x) {
    const long long i = (slab * Q + q) * 4;
    const bool full = i + 3 < MN && (MN & 3) == 0;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < MN) {
      if (full) {
        int k = g;
        for (; k + 3 * G < splits; k += 4 * G) {
          float4 t0 = *reinterpret_cast<const float4*>(part + (size_t)k * MN + i);
          float4 t1 = *reinterpret_cast<const float4*>(part + (size_t)(k + G) * MN + i);
          float4 t2 = *reinterpret_cast<const float4*>(part + (size_t)(k + 2 * G) * MN + i);
          float4 t3 = *reinterpret_cast<const float4*>(part + (size_t)(k + 3 * G) * MN + i);
          s.x += t0.x; s.y += t0.y; s.z += t0.z; s.w += t0.w;
          s.x += t1.x; s.y += t1.y; s.z += t1.z; s.w += t1.w;
          s.x += t2.x; s.y += t2.y; s.z += t2.z; s.w += t2.w;
          s.x += t3.x; s.y += t3.y; s.z += t3.z; s.w += t3.w;
        }
        for (; k < splits; k += G) {
          float4 t = *reinterpret_cast<const float4*>(part + (size_t)k * MN + i);
          s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
      } else {
        float* sv = reinterpret_cast<float*>(&s);
        for (int k = g; k < splits; k += G)
          for (int e = 0; e < 4 && i + e < MN; ++e) sv[e] += part[(size_t)k * MN + i + e];
      }
    }
    if (G > 1) {
      __syncthreads();  // the previous slab's sums have been read
      red[threadIdx.x] = s;
      __syncthreads();
      if (g == 0)
        for (int gg = 1; gg < G; ++gg) {
          float4 t = red[gg * Q + q];
          s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
    }
    if (g != 0 || i >= MN) continue;
    _Float16 h[4] = {(_Float16)s.x, (_Float16)s.y, (_Float16)s.z, (_Float16)s.w};
    unsigned short hb[4];
    __builtin_memcpy(hb, h, 8);
    int nst = 0;  // how many of the four are real outputs
    if (KT4 > 0) {
      const long long grp = i >> 2, kr = grp / KT4;
      const int sx = (int)(grp - kr * KT4);
      if (sx < S) {
        nst = C < 4 ? C : 4;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < C) out[(kr * S + sx) * C + c] = hb[c];
      }
    } else if (full) {
      nst = 4;
      uint2 pk;
      __builtin_memcpy(&pk, h, 8);
      *reinterpret_cast<uint2*>(out + i) = pk;
    } else {
      for (int e = 0; e < 4 && i + e < MN; ++e) {
        out[i + e] = hb[e];
        nst = e + 1;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < nst) bad |= jz::sumsq_acc_add(sq, hb[e]);
  }
  jz::sumsq_block_flush(sq, bad, sink, blockIdx.x, wsum);
}

// splitk_reduce for a convolution with a batch normalization behind it (MODE 0) or underneath it (MODE 1, 2): the kernel that
// adds the partial sums and rounds also takes the per-channel sums that the normalization's statistics pass would, over
// slabs of rows_per_slab rows, laid out as that pass's and the convolution epilogue's: stats[slab][2][N].
//   MODE 0: sums of the stored value and of its square.   MODE 1: of g and g x^, g = the stored value where y > 0, else 0,
//   x^ = (c - mean) invstd.   MODE 2: what is stored is g = RNE16(value [+ add]) where y > 0, else 0; sums of g and g x^.
// A reduction is split where a layer has too few output tiles, i.e. in short layers, for which a launch costs as much as
// the work: at 8 images of 64 x 64 the reduction (3.1 us) and the statistics pass behind it (3.8-5.7 us) were bound by
// their start-up and the latency of a few loads; together they take 3.4-3.9 us, and ResNet-50's step went from 1.85 to
// 1.66 ms (45 launches fewer).  A workgroup owns 64 columns; a thread 4 of them (one 16-byte load per split, eight in
// flight) in every 16th row.
constexpr int RS_COLS = 64, RS_ROWS = 16;
// four columns of a row: splitk_reduce's order, hence its bits: splits g, g + G, g + 2G, ... for lane g, then the lanes; eight loads in flight
__device__ __forceinline__ float4 split_sum(const float* __restrict__ p, size_t MN, int splits, int G) {
  float v[4] = {0.f, 0.f, 0.f, 0.f}, lane[4] = {0.f, 0.f, 0.f, 0.f};
  for (int k = 0, g = 0; g < G;) {
    float4 t[8];
    int ends = 0;  // bit u: load u is its lane's last
    int n8 = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      t[u] = *reinterpret_cast<const float4*>(p + (size_t)(g < G ? k : 0) * MN);
      if (g < G) {
        ++n8;
        k += G;
        if (k >= splits) { ends |= 1 << u; k = ++g; }
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < n8) {
        lane[0] += t[u].x; lane[1] += t[u].y; lane[2] += t[u].z; lane[3] += t[u].w;
        if (ends >> u & 1)
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[e] += lane[e]; lane[e] = 0.f; }
      }
  }
  return make_float4(v[0], v[1], v[2], v[3]);
}
template <int MODE>
__global__ __launch_bounds__(256) void splitk_reduce_stats(const float* __restrict__ part, unsigned short* __restrict__ out, int M, int N,
                                                           int splits, int G, int rows_per_slab, const unsigned short* __restrict__ y,
                                                           const unsigned short* __restrict__ c, const unsigned short* __restrict__ add,
                                                           const float* __restrict__ mean, const float* __restrict__ invstd,
                                                           float* __restrict__ stats) {
  __shared__ float4 red[2][RS_ROWS][RS_COLS / 4];
  const int q = threadIdx.x % (RS_COLS / 4), rsub = threadIdx.x / (RS_COLS / 4);
  const int n = blockIdx.x * RS_COLS + q * 4;
  const bool live = n < N;  // N is a multiple of 8
  const size_t MN = (size_t)M * N;
  const int r1 = (int)(blockIdx.y + 1) * rows_per_slab < M ? (int)(blockIdx.y + 1) * rows_per_slab : M;
  float s0[4] = {0.f, 0.f, 0.f, 0.f}, s1[4] = {0.f, 0.f, 0.f, 0.f};
  float4 mu = make_float4(0.f, 0.f, 0.f, 0.f), is = mu;
  if (MODE >= 1 && live) {
    mu = *reinterpret_cast<const float4*>(mean + n);
    is = *reinterpret_cast<const float4*>(invstd + n);
  }
  const float muv[4] = {mu.x, mu.y, mu.z, mu.w}, isv[4] = {is.x, is.y, is.z, is.w};
  auto half_at = [](const uint2& v, int e) {
    const unsigned short b = (unsigned short)((e < 2 ? v.x : v.y) >> ((e & 1) * 16));
    _Float16 h;
    __builtin_memcpy(&h, &b, 2);
    return (float)h;
  };
  for (int r = blockIdx.y * rows_per_slab + rsub; live && r < r1; r += RS_ROWS) {
    const size_t i = (size_t)r * N + n;
    uint2 yq = make_uint2(0u, 0u), cq = yq, aq = yq;
    if (MODE >= 1) {
      yq = *reinterpret_cast<const uint2*>(y + i);
      cq = *reinterpret_cast<const uint2*>(c + i);
      if (MODE == 2 && add) aq = *reinterpret_cast<const uint2*>(add + i);
    }
    const float4 v4 = split_sum(part + i, MN, splits, G);
    const float v[4] = {v4.x, v4.y, v4.z, v4.w};
    _Float16 h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[e] = (_Float16)v[e];
      if (MODE == 2) {
        h[e] = (_Float16)((float)h[e] + half_at(aq, e));  // exact in FP32, rounded once
        if (!(half_at(yq, e) > 0.f)) h[e] = (_Float16)0.f;
      }
      const float g = MODE == 1 && !(half_at(yq, e) > 0.f) ? 0.f : (float)h[e];
      s0[e] += g;
      s1[e] += MODE == 0 ? g * g : g * ((half_at(cq, e) - muv[e]) * isv[e]);
    }
    uint2 pk;
    __builtin_memcpy(&pk, h, 8);
    *reinterpret_cast<uint2*>(out + i) = pk;
  }
  red[0][rsub][q] = make_float4(s0[0], s0[1], s0[2], s0[3]);
  red[1][rsub][q] = make_float4(s1[0], s1[1], s1[2], s1[3]);
  __syncthreads();
  if (threadIdx.x < 2 * RS_COLS) {  // a thread per column and kind of sum, rows in order
    const int kind = threadIdx.x / RS_COLS, col = threadIdx.x % RS_COLS;
    const float* src = reinterpret_cast<const float*>(red[kind]) + col;
    float t = 0.f;
#pragma unroll
    for (int r = 0; r < RS_ROWS; ++r) t += src[r * RS_COLS];
    if (blockIdx.x * RS_COLS + col < (unsigned)N) stats[((size_t)blockIdx.y * 2 + kind) * N + blockIdx.x * RS_COLS + col] = t;
  }
}

// splitk_reduce_stats and the normalization behind it in one launch, for reductions of few rows: a workgroup owns 16 columns of all
// rows, so that their statistics need no other workgroup, and what it has summed is still in its registers when they are there.
// MODE as above; out2 is y (MODE 0: [relu](a c + b [+ add])) or the gradient of the normalization's input.
// What bounds it is a chain of latencies: the loads of the splits, two barriers' worth of sums, the coefficients.  5.1-5.7 us a launch where the
// two it replaces took 3.1-3.6 and 3.7; ResNet-50's step at 8 images of 64 x 64 (35 of them) 1.383 -> 1.342 ms.
constexpr int RN_THREADS = 512, RN_COLS = 16, RN_LANES = RN_COLS / 4, RN_ROWS = RN_THREADS / RN_LANES, RN_PASSES = 2;
constexpr int RN_MAX_ROWS = RN_ROWS * RN_PASSES;
// A workgroup reads rows x splits x 64 bytes, and the two launches share that among more of them the more rows there are.  Microseconds gained over the two
// (mean over 64 ... 1024 columns, both directions): 16 rows 2.0 (8 ... 116 splits); 64 rows, 8 ... 16 splits 1.3, 29 ... 47 1.5, 80 0.8, 96 -0.9; 98 rows, 8 1.0,
// 12 ... 16 0.6, 58 -0.3; 128 rows, 6 ... 8 0.5, 12 ... 16 -0.2, 58 -2.3; 144 rows, 4 ... 6 0.9, 8 -0.4, 24 -2.6; 196 rows, 4 ... 6 0, 8 -1.4, 48 -8.2.
// Those are captured calls.  Launched one by one a launch less is worth more: the step above, whose 3x3 layers at 128 rows have 12 and 15 splits, is 0.4 % faster
// with them merged.
bool reduce_normalizes(int rows, int splits) {
  return rows <= RN_MAX_ROWS && (long long)rows * rows * splits <= (rows <= RN_ROWS ? 250000 : 150000);
}
struct NormArgs {
  const float* part;
  unsigned short* out;
  int M, N, splits, G;
  const unsigned short *y, *c, *add;
  const float *mean, *invstd;
  const float *gamma, *beta;
  float eps;
  int relu;
  double inv_rows;
  unsigned short* out2;
  float *save_mean, *save_invstd;
  unsigned short *dgamma, *dbeta;
};
template <int MODE>
__global__ __launch_bounds__(RN_THREADS) void splitk_reduce_norm(NormArgs a) {
  __shared__ float red[2][RN_ROWS][RN_COLS];
  __shared__ double parts[RN_THREADS / (2 * RN_COLS)][2 * RN_COLS];
  __shared__ float coef[3][RN_COLS];
  const int tid = threadIdx.x, q = tid % RN_LANES, rsub = tid / RN_LANES;
  const int first = blockIdx.x * RN_COLS, n = first + q * 4;
  const bool live = n < a.N;  // N is a multiple of 8
  const size_t MN = (size_t)a.M * a.N;
  float mu[4] = {0.f, 0.f, 0.f, 0.f}, is[4] = {0.f, 0.f, 0.f, 0.f};
  if (MODE >= 1 && live) {
    const float4 m4 = *reinterpret_cast<const float4*>(a.mean + n), i4 = *reinterpret_cast<const float4*>(a.invstd + n);
    mu[0] = m4.x; mu[1] = m4.y; mu[2] = m4.z; mu[3] = m4.w;
    is[0] = i4.x; is[1] = i4.y; is[2] = i4.z; is[3] = i4.w;
  }
  auto half_at = [](const uint2& v, int e) {
    const unsigned short b = (unsigned short)((e < 2 ? v.x : v.y) >> ((e & 1) * 16));
    _Float16 h;
    __builtin_memcpy(&h, &b, 2);
    return (float)h;
  };
  uint2 cq[RN_PASSES], aq[RN_PASSES], kept[RN_PASSES];  // kept: what is normalized, or the gradient behind the ReLU
  float s0[4] = {0.f, 0.f, 0.f, 0.f}, s1[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < RN_PASSES; ++p) {
    const int r = p * RN_ROWS + rsub;
    cq[p] = aq[p] = kept[p] = make_uint2(0u, 0u);
    if (!live || r >= a.M) continue;
    const size_t i = (size_t)r * a.N + n;
    uint2 yq = make_uint2(0u, 0u);
    if (MODE >= 1) {
      yq = *reinterpret_cast<const uint2*>(a.y + i);
      cq[p] = *reinterpret_cast<const uint2*>(a.c + i);
    }
    if (MODE != 1 && a.add) aq[p] = *reinterpret_cast<const uint2*>(a.add + i);
    _Float16 h[4];
    const float4 v = split_sum(a.part + i, MN, a.splits, a.G);
    h[0] = (_Float16)v.x; h[1] = (_Float16)v.y; h[2] = (_Float16)v.z; h[3] = (_Float16)v.w;
    if (MODE == 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        h[e] = (_Float16)((float)h[e] + half_at(aq[p], e));  // exact in FP32, rounded once
        if (!(half_at(yq, e) > 0.f)) h[e] = (_Float16)0.f;
      }
    }
    uint2 pk;
    __builtin_memcpy(&pk, h, 8);
    *reinterpret_cast<uint2*>(a.out + i) = pk;
    if (MODE == 1) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!(half_at(yq, e) > 0.f)) h[e] = (_Float16)0.f;
      __builtin_memcpy(&pk, h, 8);
    }
    kept[p] = pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float g = (float)h[e];
      s0[e] += g;
      s1[e] = fmaf(g, MODE == 0 ? g : (half_at(cq[p], e) - mu[e]) * is[e], s1[e]);
    }
  }
  // at most RN_PASSES rows a thread in FP32, everything else in FP64
  *reinterpret_cast<float4*>(&red[0][rsub][q * 4]) = make_float4(s0[0], s0[1], s0[2], s0[3]);
  *reinterpret_cast<float4*>(&red[1][rsub][q * 4]) = make_float4(s1[0], s1[1], s1[2], s1[3]);
  __syncthreads();
  {
    constexpr int PARTS = RN_THREADS / (2 * RN_COLS), PER = RN_ROWS / PARTS;
    const int i = tid % (2 * RN_COLS), j = tid / (2 * RN_COLS);
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < PER; ++k) t += (double)red[i / RN_COLS][j + k * PARTS][i % RN_COLS];
    parts[j][i] = t;
    __syncthreads();
    if (tid < 2 * RN_COLS) {
      t = 0.0;
#pragma unroll
      for (int k = 0; k < PARTS; ++k) t += parts[k][tid];
      parts[0][tid] = t;
    }
    __syncthreads();
    if (tid < RN_COLS && first + tid < a.N) {
      const int c = first + tid;
      if (MODE == 0)
        bn_fwd_coef(parts[0][tid], parts[0][RN_COLS + tid], a.inv_rows, a.eps, a.gamma[c], a.beta[c], a.save_mean + c, a.save_invstd + c, &coef[0][tid], RN_COLS);
      else
        bn_bwd_coef(parts[0][tid], parts[0][RN_COLS + tid], a.inv_rows, a.gamma[c], a.mean[c], a.invstd[c], a.dgamma + c, a.dbeta + c, &coef[0][tid],
                    RN_COLS);
    }
    __syncthreads();
  }
  float ca[4], cb[4], cc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    ca[e] = coef[0][q * 4 + e];
    cb[e] = coef[1][q * 4 + e];
    cc[e] = MODE == 0 ? 0.f : coef[2][q * 4 + e];
  }
#pragma unroll
  for (int p = 0; p < RN_PASSES; ++p) {
    const int r = p * RN_ROWS + rsub;
    if (!live || r >= a.M) continue;
    _Float16 h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (MODE == 0) {
        float z = fmaf(half_at(kept[p], e), ca[e], cb[e]);
        if (a.add) z += half_at(aq[p], e);
        h[e] = (_Float16)(a.relu && !(z > 0.f) ? 0.f : z);
      } else {
        h[e] = (_Float16)bn_dx(ca[e], half_at(kept[p], e), cb[e], half_at(cq[p], e), cc[e]);
      }
    }
    uint2 pk;
    __builtin_memcpy(&pk, h, 8);
    *reinterpret_cast<uint2*>(a.out2 + (size_t)r * a.N + n) = pk;
  }
}

// sum of squares of n FP16 values into a sink (gradients whose producing kernel has no fused form)
__global__ __launch_bounds__(256) void sumsq_half(const unsigned short* __restrict__ g16, long long n, jz::SumsqSink sink) {
  __shared__ unsigned long long wsum[5];
  if (threadIdx.x < 5) wsum[threadIdx.x] = 0ull;
  __syncthreads();
  jz::SumsqAcc sq;
  int bad = 0;
  const long long groups = n >> 3;  // 16-byte groups; g16 is 16-byte aligned
  for (long long j = (long long)blockIdx.x * 256 + threadIdx.x; j < groups; j += (long long)gridDim.x * 256) {
    const uint4 v = *reinterpret_cast<const uint4*>(g16 + j * 8);
    const unsigned wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) bad |= jz::sumsq_acc_add(sq, (unsigned short)(wv[e >> 1] >> ((e & 1) * 16)));
  }
  if (blockIdx.x == 0) {  // the tail, at most 7 elements
    const long long i = (groups << 3) + threadIdx.x;
    if (i < n) bad |= jz::sumsq_acc_add(sq, g16[i]);
  }
  jz::sumsq_block_flush(sq, bad, sink, blockIdx.x, wsum);
}

// ---------------------------------------------------------------------------------------------
// host side: plan (tile shape, fast/generic, split-K) and launch
// ---------------------------------------------------------------------------------------------
int out_dim(int in, int pad, int f, int st) { return (in + 2 * pad - f) / st + 1; }
size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// Compute units that a launch's workgroups are counted against: the chip's, or half of them for a weight gradient beside other
// streams' work.  GEMMs of a ResNet-50 step, weight gradients on two side streams, none of the layers recorded: batch 48, 63 and
// 100 take 3.00, 3.53 and 4.85 ms planned for the whole chip, 2.92, 3.43 and 4.74 for half of it, 2.99, 3.55 and 5.06 where at
// most 128 workgroups are allowed instead.  (Batch 64, recorded choices: 3.40 ms against 3.53 planned alone.  With one side
// stream beside a chained step it makes no difference, 6.36 ms at batch 64: such a step keeps the plans of a single stream.)
constexpr int kUnits = 256, kUnitsBeside = 128;

// Pick the kernel variant (output tile, k tile depth, wavefronts per workgroup) and the split of the reduction with a
// cost model, in microseconds.  A compute unit works through n = ceil(workgroups / 256) workgroups, `resident` of them
// at a time, each over kps k tiles; what it can be bound by, and the time as their (fourth-power) norm:
//   latency     ceil(workgroups / (256 resident)) rounds of (prologue + kps * lat)
//   throughput  n * (own + kps * thr), whatever shares the unit
//   memory      operands read once and the result written once, at `byte` per megabyte
//   time = fixed + norm (+ reducing a split: second launch + reading its partial sums)
// The constants are least-squares fits (robust, logarithmic, weighted towards the fastest choices of a shape) to cold-
// operand timings of every variant and split on 1,060 layers: ResNet-50 of both kinds and AlexNet at batch sizes from 3
// to 128 and images from 64 to 224 pixels, fully connected layers, and random single layers.  On 320 of them left out
// of the fit the choices were 2-3 % slower than the best of all variants and splits, which is also what choosing by one
// timing costs; the model this replaces (rounds * kps * one constant per variant, fitted to batch 64, 11 of the 19
// variants offered) was 6, 10 and 5 % slower than the best (forward, backward-data, backward-weight), 71 % at worst.
constexpr int kMaxClasses = 16;  // parity classes of a stride (sh * sw) the backward-data decomposition handles

struct Variant {
  int BM, BN, bk, waves, nst;  // output tile, k tile, wavefronts, ring depth
  int resident;                // workgroups of it that share a compute unit (LDS)
  // per k tile and per workgroup, each for forward, backward-data, backward-weight
  double lat[3], thr[3], prologue[3], own[3];
};
const Variant kVariants[] = {
    {128, 128, 32, 4, 4, 2, {0.272, 0.302, 0.359}, {0.232, 0.193, 0.180}, {1.786, 1.815, 1.093}, {1.579, 1.602, 0.995}},
    {128, 64, 32, 4, 4, 3, {0.174, 0.200, 0.246}, {0.178, 0.149, 0.114}, {1.418, 1.269, 0.438}, {0.803, 0.797, 0.608}},
    {64, 128, 32, 4, 4, 3, {0.178, 0.226, 0.294}, {0.173, 0.144, 0.148}, {1.404, 1.103, 0.615}, {0.773, 0.782, 0.525}},
    {64, 64, 32, 4, 4, 5, {0.146, 0.170, 0.193}, {0.116, 0.110, 0.089}, {1.053, 0.956, 0.082}, {0.446, 0.460, 0.330}},
    {128, 128, 64, 8, 4, 1, {0.405, 0.439, 0.463}, {0.300, 0.296, 0.288}, {1.958, 1.968, 1.013}, {0.399, 0.401, 0.406}},
    {256, 128, 64, 8, 3, 1, {0.550, 0.628, 0.731}, {0.710, 0.626, 0.511}, {3.142, 3.096, 1.700}, {0.387, 0.396, 0.409}},
    {256, 128, 32, 8, 4, 1, {0.393, 0.380, 0.343}, {0.240, 0.278, 0.211}, {2.627, 2.648, 1.864}, {0.406, 0.400, 0.414}},
    {256, 256, 32, 8, 4, 1, {0.556, 0.471, 0.521}, {0.526, 0.600, 0.466}, {4.934, 5.079, 4.209}, {0.398, 0.394, 0.399}},
    {128, 128, 64, 4, 4, 1, {0.427, 0.493, 0.651}, {0.280, 0.301, 0.303}, {2.616, 2.459, 1.310}, {0.401, 0.400, 0.400}},
    {128, 64, 64, 4, 4, 1, {0.287, 0.317, 0.426}, {0.148, 0.146, 0.150}, {1.905, 1.762, 0.847}, {0.401, 0.404, 0.399}},
    {64, 128, 64, 4, 4, 1, {0.277, 0.359, 0.512}, {0.143, 0.150, 0.150}, {1.760, 1.676, 0.862}, {0.404, 0.401, 0.397}},
    {64, 64, 64, 4, 4, 2, {0.208, 0.242, 0.290}, {0.154, 0.171, 0.199}, {1.087, 1.062, 0.109}, {0.795, 0.764, 0.482}},
    {128, 128, 32, 4, 3, 3, {0.357, 0.418, 0.434}, {0.204, 0.185, 0.173}, {1.582, 1.392, 0.907}, {1.420, 1.366, 0.393}},
    {128, 64, 32, 4, 3, 4, {0.266, 0.329, 0.347}, {0.172, 0.153, 0.101}, {1.098, 0.772, 0.165}, {0.640, 0.646, 0.548}},
    {64, 128, 32, 4, 3, 4, {0.277, 0.337, 0.365}, {0.164, 0.140, 0.135}, {1.102, 0.762, 0.346}, {0.602, 0.635, 0.438}},
    {64, 64, 32, 4, 3, 6, {0.226, 0.308, 0.300}, {0.119, 0.108, 0.086}, {0.839, 0.435, 0.053}, {0.337, 0.380, 0.272}},
    {256, 128, 32, 8, 3, 2, {0.419, 0.441, 0.395}, {0.349, 0.325, 0.281}, {1.538, 1.534, 1.464}, {2.063, 2.100, 0.552}},
    {128, 128, 32, 8, 4, 2, {0.239, 0.287, 0.245}, {0.224, 0.213, 0.179}, {1.548, 1.417, 1.014}, {1.300, 1.311, 0.701}},
    {128, 128, 32, 8, 3, 3, {0.346, 0.420, 0.374}, {0.229, 0.214, 0.175}, {1.140, 1.008, 0.486}, {1.067, 1.117, 0.380}},
};
struct CostGlobals {
  double fixed, reduce_launch, reduce_byte, byte, taps;  // taps: factor on the loop of a multi-tap layer
};
const CostGlobals kCost[3] = {{3.11, 2.54, 0.343, 0.162, 1.01}, {3.11, 2.57, 0.344, 0.154, 1.05}, {3.61, 2.83, 0.339, 0.122, 1.19}};

// Measured choices for known GEMM shapes (written by `python -m paper_1807_11205_amd.tune --write`): the per-k-tile model
// below ranks variants that differ by a few percent poorly, a table of cold-cache timings does not.
struct Tuned {
  int op, M, N, K, taps, scatter, BM, BN, bk, waves, nst, splits;
};
const Tuned kTuned[] = {
#include "jz_tuned.inc"
#include "jz_tuned_alexnet.inc"
#include "jz_tuned_resnet50_n128.inc"
#include "jz_tuned_resnet50_n256.inc"
#include "jz_tuned_resnet50_n32.inc"
#include "jz_tuned_resnet50_v15.inc"
    // the 3-channel stem of ResNet-50 at batch 64 on its padded 4-channel copy ("taps" = the 7 filter rows), measured
    // the same way: forward 62.8 us (what the fused convolution + batch-norm call runs; the plain forward call takes the
    // patch kernel), backward-weight 67.0 us including the copy
    {0, 802816, 64, 224, 7, 0, 128, 64, 32, 4, 3, 1},
    {2, 64, 224, 802816, 7, 0, 64, 64, 32, 4, 4, 256},
    // backward-weight of the 11x11 stride-4 stem at batch 128, chosen inside the AlexNet step (tune.py --model alexnet --in-place)
    {2, 96, 528, 387200, 11, 0, 128, 128, 32, 4, 3, 128},
};

// Choices set at run time through jz_conv2d_tune_set: looked up before the table above (an in-place tuning run tries
// candidates this way without rebuilding the library).  g_use_table: whether the table above is consulted at all
// (jz_conv2d_tune_use_table; the cost model alone is what an unknown shape gets).
std::mutex g_tune_mutex;
std::vector<Tuned> g_tune_rt;
bool g_use_table = true;
std::atomic<unsigned> g_tune_generation{1};  // changes whenever one of the above does: plans made before are stale

bool same_key(const Tuned& x, const Tuned& y) {
  return x.op == y.op && x.M == y.M && x.N == y.N && x.K == y.K && x.taps == y.taps && x.scatter == y.scatter;
}

// bk64_ok: the 64-deep k tile is usable for this layer; forced_bk: the k tile depth is fixed (register path, packed mode)
void set_tiles(Plan* pl, int splits) {
  GemmArgs& a = pl->args;
  a.nkt = (a.Kred + pl->bk - 1) / pl->bk;
  a.tiles_m = (a.M + pl->BM - 1) / pl->BM;
  a.tiles_n = (a.N + pl->BN - 1) / pl->BN;
  a.kt_per_split = (a.nkt + splits - 1) / splits;
  if (pl->window) {  // whole blocks of channels
    const int taps = a.g.R * a.g.S, blocks = a.nkt / taps;
    a.kt_per_split = (blocks + splits - 1) / splits * taps;
  }
  a.splits = (a.nkt + a.kt_per_split - 1) / a.kt_per_split;  // drop empty splits
  a.d_tiles_mn = make_fastdiv((unsigned)(a.tiles_m * a.tiles_n));
  a.d_tiles_n = make_fastdiv((unsigned)a.tiles_n);
}

// Whether the window kernel's variant v takes this problem: unit stride, output grid = input grid, whole blocks of channels, a
// window that holds the tile's pixels and what their taps reach, and window offsets within 31 bits.
bool window_fits(const Plan& pl, const WindowVariant& v) {
  const GemmArgs& a = pl.args;
  const ConvGeom& g = a.g;
  return (pl.op == JZ_FWD || pl.op == JZ_BWD_DATA) && pl.fast && !pl.packed && !pl.gen && !pl.flat && !a.sc_on && g.sh == 1 && g.sw == 1 &&
         g.IH == g.OH && g.IW == g.OW && 2 * g.ph + 1 == g.R && 2 * g.pw + 1 == g.S && g.R * g.S >= 9 && g.R * g.S <= 32 && g.IC % v.ck == 0 &&
         (v.windows > 1 || g.IC == v.ck) && (long long)v.BM + (long long)(g.R - 1) * g.IW + g.S - 1 <= v.rows &&
         2ll * v.rows * g.IC < (1ll << 31);
}

// The entry (+ 1) that a recorded window variant names, 0 where it does not take this problem.  A key does not hold the image's width, the stride
// or the padding, which decide that: layers share keys that the variant takes and that it does not.
int recorded_window(const Plan& pl, const Tuned& t) {
  for (int i = 0; i < kNumWindows; ++i) {
    const WindowVariant& v = kWindows[i];
    if (v.BM == t.BM && v.BN == t.BN && v.ck == t.bk && v.waves == t.waves && v.nst + kWindowRing == t.nst && window_fits(pl, v)) return i + 1;
  }
  return 0;
}

// The window kernel's entry (+ 1) for a plan that the tables or the cost model have made for the ring kernels, or 0.  From 90 random layers (3x3 and
// 5x5, 64 ... 512 channels, images of 7 ... 63 pixels, 5 ... 3300 tiles), both directions, time against the ring kernel's:
//   more than 64 channels in, the plan is 256x128 tiles: 0.76 ... 1.006, median 0.95 (fewer bytes into LDS at the same tile);
//   ... is 128x128 tiles on 4 wavefronts: 0.83 ... 0.99 where 256x128 tiles leave at most 30 % of their last round of workgroups empty,
//   up to 1.11 where they leave more; eight wavefronts, 256x256 tiles or 64 columns: mostly slower, up to 1.1 and 1.4;
//   64 channels in and at most 64 out: 0.66 ... 0.96 from 155 tiles of 256x64 on, slower from 93 down (1.2); more columns bring the
//   window in several times: 0.76 ... 1.014, median 0.92, where the last round is 80 % full, up to 1.08 elsewhere.
int choose_window(const Plan& pl) {
  const GemmArgs& a = pl.args;
  auto tiles = [&](const WindowVariant& v) { return (long long)((a.M + v.BM - 1) / v.BM) * ((a.N + v.BN - 1) / v.BN); };
  auto full = [&](long long t) { return (double)t / (double)((t + kUnits - 1) / kUnits * kUnits); };
  if (window_fits(pl, kWindows[1])) {
    const long long t = tiles(kWindows[1]);
    return (a.N <= 64 ? t >= 150 : t >= kUnits && full(t) >= 0.8) ? 2 : 0;
  }
  if (!window_fits(pl, kWindows[0]) || a.g.IC <= 64 || a.N <= 64 || pl.BN != 128) return 0;
  return pl.BM == 256 || (pl.BM == 128 && pl.waves == 4 && pl.bk == 32 && full(tiles(kWindows[0])) >= 0.7) ? 1 : 0;
}

void choose_tiling(Plan* pl, bool bk64_ok, int forced_bk, bool tables = true) {
  GemmArgs& a = pl->args;
  static const int split_opts[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512};
  const int oi = pl->op == JZ_FWD ? 0 : pl->op == JZ_BWD_DATA ? 1 : 2;
  double best = 1e30;
  const Variant* bv = &kVariants[0];
  int bS = 1;
  if (!pl->fast) forced_bk = BK;  // the element-wise kernel: one shape (the first variant's), 64-deep tiles, ~8x slower
  const Tuned* hit = nullptr;
  Tuned rt_hit{};
  if (tables && pl->fast && (!forced_bk || pl->packed)) {
    const Tuned key{oi, a.M, a.N, a.Kred, a.g.R * a.g.S, a.sc_on, 0, 0, 0, 0, 0, 0};
    auto usable = [&](const Tuned& t) {
      if ((pl->gen || pl->flat) && (t.waves != 4 || t.bk != 32 || t.nst != 4 || t.BM > 128 || t.BN > 128)) return false;  // the only kernels of those modes
      if (t.nst > kWindowRing && recorded_window(*pl, t) == 0) return false;
      return same_key(t, key) && (forced_bk ? t.bk == forced_bk : (t.bk == 32 || bk64_ok));
    };
    bool use_table;
    {
      std::lock_guard<std::mutex> lock(g_tune_mutex);
      use_table = g_use_table;
      for (const Tuned& t : g_tune_rt)
        if (usable(t)) {
          rt_hit = t;
          hit = &rt_hit;
          pl->rt_forced = true;
          break;
        }
    }
    if (!hit && use_table && !pl->gen)
      for (const Tuned& t : kTuned)
        if (usable(t)) {
          hit = &t;
          break;
        }
  }
  const double megabytes_in = 1e-6 * ((double)std::min<long long>(pl->bytesA, 2ll * a.M * a.Kred) +
                                      (double)std::min<long long>(pl->bytesB, 2ll * a.N * a.Kred));
  const CostGlobals& cg = kCost[oi];
  const int units = pl->beside ? kUnitsBeside : kUnits;
  // variant v with sp splits (v.bk may differ from the k tile that runs: vbk)
  auto cost = [&](const Variant& v, int vbk, int sp) {
    const int nkt = (a.Kred + vbk - 1) / vbk, kps = (nkt + sp - 1) / sp;
    const long long tiles = (long long)((a.M + v.BM - 1) / v.BM) * ((a.N + v.BN - 1) / v.BN);
    const long long blocks = tiles * ((nkt + kps - 1) / kps);
    const double loop = kps * (vbk / (double)v.bk) * (a.g.R * a.g.S > 1 ? cg.taps : 1.0) * (pl->fast ? 1.0 : 8.0);
    const double out = 1e-6 * (double)a.M * a.N;
    const double t_lat = (double)((blocks + units * v.resident - 1) / (units * v.resident)) * (v.prologue[oi] + v.lat[oi] * loop);
    const double t_thr = (double)((blocks + units - 1) / units) * (v.own[oi] + v.thr[oi] * loop);
    const double t_mem = cg.byte * (megabytes_in + (sp > 1 ? 4.0 * sp : 2.0) * out);
    auto p4 = [](double x) { return (x * x) * (x * x); };
    return cg.fixed + std::sqrt(std::sqrt(p4(t_lat) + p4(t_thr) + p4(t_mem))) +
           (sp > 1 ? cg.reduce_launch + cg.reduce_byte * 4.0 * sp * out : 0.0);
  };
  // the best admissible split of it, kept if better than what is known so far
  auto try_variant = [&](const Variant& v, int vbk) {
    const int nkt = (a.Kred + vbk - 1) / vbk;
    for (int sp : split_opts) {
      if (sp > 1 && (nkt / sp < 4 || a.sc_on || 4.0 * sp * a.M * a.N > (double)pl->part_limit)) break;  // the scatter lives in the fp16 epilogue
      const double t = cost(v, vbk, sp);
      if (t < best) { best = t; bv = &v; bS = sp; }
    }
  };
  if (hit) {
    pl->BM = hit->BM; pl->BN = hit->BN; pl->bk = hit->bk; pl->waves = hit->waves;
    pl->nst = hit->nst;
    if (hit->nst > kWindowRing) {
      pl->nst -= kWindowRing;
      pl->window = recorded_window(*pl, *hit);
    }
    bS = hit->splits;
    const int nkt_h = (a.Kred + hit->bk - 1) / hit->bk;
    if (bS > 1 && (nkt_h / bS < 4 || a.sc_on)) bS = 1;  // the same admissibility rules as the search below
    const bool too_much = bS > 1 && !pl->rt_forced && 4.0 * bS * a.M * a.N > (double)pl->part_limit;
    if (too_much) bS = 1;
    // backward-weight: most of the table's split counts were chosen for launches that share the chip with two other streams
    // (fewer splits, hence fewer workgroups and partial sums) and stay for such launches; one of its own wants the chip filled.  The tile is kept,
    // and so is the split where the model does not see a twelfth in changing it: batch 64 (chosen in company) 1.78 -> 1.32 ms
    // for the 52 layers, batch 32 (measured alone) keeps its splits.
    if ((oi == 2 && !pl->rt_forced && !pl->packed && !pl->beside) || too_much)
      for (const Variant& v : kVariants)
        if (v.BM == hit->BM && v.BN == hit->BN && v.bk == hit->bk && v.waves == hit->waves && v.nst == hit->nst) {
          best = (too_much ? 1.0 : 11.0 / 12.0) * cost(v, v.bk, bS);
          try_variant(v, v.bk);
        }
  } else {
    for (const Variant& v : kVariants) {
      if (!pl->fast && &v != &kVariants[0]) break;
      if ((forced_bk || pl->gen || pl->flat) && (v.waves != 4 || v.bk != 32 || v.nst != 4)) continue;  // the only kernels of those modes
      if (!forced_bk && v.bk == 64 && !bk64_ok) continue;
      try_variant(v, forced_bk ? forced_bk : v.bk);
    }
    pl->BM = bv->BM; pl->BN = bv->BN;
    pl->bk = forced_bk ? forced_bk : bv->bk;
    pl->waves = bv->waves;
    pl->nst = bv->nst;
  }
  pl->tuned = hit != nullptr;
  set_tiles(pl, bS);
  if (!pl->rt_forced && a.splits == 1) {
    const int w = choose_window(*pl);
    if (w != 0) {
      const WindowVariant& v = kWindows[w - 1];
      pl->window = w;
      pl->replaced = {pl->BM, pl->BN, pl->bk, pl->waves, pl->nst, a.tiles_m, a.tiles_n, a.nkt};
      pl->BM = v.BM; pl->BN = v.BN; pl->bk = v.ck; pl->waves = v.waves; pl->nst = v.nst;
      set_tiles(pl, 1);
    }
  }
}

void finish_geometry(ConvGeom& g) {
  g.tap_rep = 0;
  if (g.R * g.S <= 32)
    for (int r = 0; r < g.R; ++r) g.tap_rep |= 1u << (r * g.S);
  g.d_ohow = make_fastdiv((unsigned)(g.OH * g.OW));
  g.d_ow = make_fastdiv((unsigned)g.OW);
  g.d_ic = make_fastdiv((unsigned)g.IC);
  g.d_s = make_fastdiv((unsigned)g.S);
  g.d_sh = make_fastdiv((unsigned)g.sh);
  g.d_sw = make_fastdiv((unsigned)g.sw);
}

// The patch kernel's view of a packed forward layer (jz_conv_stem.hip); false: the layer stays on the implicit-GEMM kernel
// (output channels not a multiple of 32 or more than 128, filter + patch larger than the LDS).
bool stem_fwd_setup(const Plan& pl, const jz_conv_desc* d, StemArgs* sa) {
  if (!pl.packed || pl.op != JZ_FWD || d->K % 32 != 0 || d->K > 128) return false;
  const int P = out_dim(d->H, d->pad_h, d->R, d->stride_h), Q = out_dim(d->W, d->pad_w, d->S, d->stride_w);
  StemArgs a;
  a.NT = d->K / 32;
  a.NKS = (4 * d->S + 15) / 16;
  const int TM = stem_fwd_tm(a.NT);
  if (TM == 0 || a.NKS < 1 || a.NKS > 4 || a.NKS * 16 > pl.KT) return false;
  const int MB = 4 * TM * 32;
  a.N = d->N; a.Hp = pl.Hp; a.Wp = pl.Wp; a.P = P; a.Q = Q; a.R = d->R; a.sh = d->stride_h; a.sw = d->stride_w;
  a.xp_bytes = (unsigned)((size_t)d->N * pl.Hp * pl.Wp * 8);
  a.wq_bytes = (unsigned)((size_t)d->R * a.NKS * 2 * d->K * 16);
  if (a.wq_bytes > pl.wp_bytes) return false;
  // output rows that MB consecutive pixels can touch, and the input rows under them
  long long rows = ((long long)MB + Q - 2) / Q + 1;
  if (rows > P) rows = P;
  const size_t patch = (size_t)((rows - 1) * d->stride_h + d->R) * pl.Wp * 8;
  const size_t staging = (size_t)4 * 32 * (d->K * 2 + 16);
  const size_t lds_p = ((patch > staging ? patch : staging) + 4095) & ~size_t(4095);
  const size_t lds_w = ((size_t)a.wq_bytes + 4095) & ~size_t(4095);
  if (lds_w + lds_p > 160 * 1024) return false;
  a.lds_w_bytes = (unsigned)lds_w;
  a.lds_p_bytes = (unsigned)lds_p;
  a.blocks_per_image = (P * Q + MB - 1) / MB;
  const long long total = (long long)d->N * a.blocks_per_image;
  if (total > 0x7fffffff) return false;
  a.total_blocks = (int)total;
  // workgroups per compute unit: what the LDS and the instance's register budget allow
  const long long fit = (long long)((160 * 1024) / (lds_w + lds_p));
  const long long slots = 256 * (fit < stem_fwd_wgs(a.NT) ? fit : (long long)stem_fwd_wgs(a.NT));
  a.grid = (int)(total < slots ? total : slots);
  *sa = a;
  return true;
}

void plan_text(const Plan& pl, char* buf, size_t n) {
  const GemmArgs& a = pl.args;
  if (pl.widen) {
    snprintf(buf, n, "op %d M %d N %d K %d: run as %d -> %d channels on zero-extended copies", pl.op, a.M, a.N, a.Kred, pl.wide.C, pl.wide.K);
    return;
  }
  if (pl.stem) {
    const int mb = 128 * stem_fwd_tm(a.N / 32);
    snprintf(buf, n, "op %d M %d N %d K %d: patch kernel, %d pixels x %d channels per block, %d blocks per image, filter resident in LDS, "
             "4 wavefronts, 4-channel padded copy", pl.op, a.M, a.N, a.Kred, mb, a.N, (a.g.OH * a.g.OW + mb - 1) / mb);
    return;
  }
  if (pl.window && !pl.rt_forced) {
    const auto& r = pl.replaced;
    snprintf(buf, n, "op %d M %d N %d K %d: vector tile %dx%dx%d, %d wavefronts, ring %d, %d x %d tiles, 1 splits of %d k tiles%s; "
             "replaced by window tile %dx%dx%d, %d wavefronts, ring %d, %d x %d tiles", pl.op, a.M, a.N, a.Kred, r.BM, r.BN, r.bk, r.waves, r.nst,
             r.tiles_m, r.tiles_n, r.nkt, pl.tuned ? ", recorded choice" : "", pl.BM, pl.BN, pl.bk, pl.waves, pl.nst + kWindowRing, a.tiles_m, a.tiles_n);
    return;
  }
  snprintf(buf, n, "op %d M %d N %d K %d: %s tile %dx%dx%d, %d wavefronts, ring %d, %d x %d tiles, %d splits of %d k tiles%s%s%s", pl.op, a.M,
           a.N, a.Kred, pl.window ? "window" : pl.fast ? "vector" : "element-wise", pl.BM, pl.BN, pl.bk, pl.fast ? pl.waves : 4,
           pl.window ? pl.nst + kWindowRing : pl.fast ? pl.nst : 2, a.tiles_m, a.tiles_n,
           a.splits, a.kt_per_split, pl.packed ? ", 4-channel padded copy" : "",
           pl.flat ? (pl.classes ? ", flattened taps, the residues of the stride in one launch" : ", flattened taps")
           : a.sc_on ? ", scatter epilogue" : pl.classes ? ", the parity classes of the stride in one launch" : pl.gen ? ", per-load tap arithmetic" : "",
           pl.tuned ? ", recorded choice" : "");
}

// whether strided multi-tap backward-data can run as one unit-stride launch per parity class: every class has a tap, and
// at most 32 of them (the masks)
bool has_classes(const jz_conv_desc* d) {
  return (d->stride_h > 1 || d->stride_w > 1) && d->R >= d->stride_h && d->S >= d->stride_w && d->stride_h * d->stride_w <= kMaxClasses &&
         ((d->R + d->stride_h - 1) / d->stride_h) * ((d->S + d->stride_w - 1) / d->stride_w) <= 32;
}

void plan_widened(int op, const jz_conv_desc* d, Plan* pl);

// limit: bytes that the partial sums of a split reduction may take
int compute_plan(int op, const jz_conv_desc* d, Plan* pl, size_t limit = kPartialSumLimit) {
  if (!d) return JZ_ERR_NULL;
  pl->beside = op == (JZ_BWD_WEIGHT | JZ_BESIDE);
  if (pl->beside) op = JZ_BWD_WEIGHT;
  if (op != JZ_FWD && op != JZ_BWD_DATA && op != JZ_BWD_WEIGHT) return JZ_ERR_UNSUPPORTED;
  if (d->N <= 0 || d->H <= 0 || d->W <= 0 || d->C <= 0 || d->K <= 0 || d->R <= 0 || d->S <= 0 || d->stride_h <= 0 ||
      d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0)
    return JZ_ERR_SHAPE;
  if (d->pad_h >= d->R || d->pad_w >= d->S) return JZ_ERR_SHAPE;
  if (d->H + 2 * d->pad_h < d->R || d->W + 2 * d->pad_w < d->S) return JZ_ERR_SHAPE;
  const int P = out_dim(d->H, d->pad_h, d->R, d->stride_h), Q = out_dim(d->W, d->pad_w, d->S, d->stride_w);
  if (P <= 0 || Q <= 0) return JZ_ERR_SHAPE;
  // Byte offsets are formed in unsigned 32-bit integers, 0xffffffff marks "out of range" and is OR-ed into live
  // offsets, and a gathered operand's descriptor is widened by a margin smaller than the tensor: with at most 2^30 - 1
  // elements (2^31 - 2 bytes) per tensor every live offset, and every descriptor size, stays below 2^32 - 1.
  const long long lim = (1ll << 30) - 1;
  const long long nx = (long long)d->N * d->H * d->W * d->C, ny = (long long)d->N * P * Q * d->K,
                  nw = (long long)d->K * d->R * d->S * d->C;
  if (nx > lim || ny > lim || nw > lim) return JZ_ERR_UNSUPPORTED;
  if ((long long)d->N * P * Q > lim / 2 || (long long)d->N * d->H * d->W > lim / 2) return JZ_ERR_UNSUPPORTED;

  GemmArgs& a = pl->args;
  ConvGeom& g = a.g;
  pl->op = op;
  pl->part_limit = limit;
  // k tile depth for the applicability checks: the LDS-direct kernels come 32 and 64 deep (chosen by the planner when
  // the layer allows both; 32 lets two workgroups share a compute unit)
  int bk = 32;
  bool bk64_ok = true;
  int forced_bk = 0;
  g.R = d->R; g.S = d->S; g.sh = d->stride_h; g.sw = d->stride_w; g.ph = d->pad_h; g.pw = d->pad_w;
  g.kvalid = 0;
  // a single filter tap: the reduction is one contiguous channel run, whose ragged last k tile the vector kernel can mask
  const bool one_tap = d->R == 1 && d->S == 1;
  if (op == JZ_FWD) {
    a.M = d->N * P * Q; a.N = d->K; a.Kred = d->R * d->S * d->C;
    g.IH = d->H; g.IW = d->W; g.IC = d->C; g.OH = P; g.OW = Q;
    pl->flat = d->C % bk != 0 && d->C % 8 == 0 && !one_tap && d->R * d->S <= 32;
    pl->fast = d->C % bk == 0 || (one_tap && d->C % 8 == 0) || pl->flat;
    bk64_ok = d->C % 64 == 0 || (one_tap && d->C % 8 == 0);
    pl->bytesA = 2 * nx; pl->bytesB = 2 * nw; pl->bytesD = 2 * ny;
  } else if (op == JZ_BWD_DATA) {
    a.M = d->N * d->H * d->W; a.N = d->C; a.Kred = d->R * d->S * d->K;
    g.IH = P; g.IW = Q; g.IC = d->K; g.OH = d->H; g.OW = d->W;
    // strided multi-tap layers only through their parity classes (each a unit-stride problem); the per-load variant for the
    // others walks whole k tiles inside one tap
    pl->flat = d->K % bk != 0 && d->K % 8 == 0 && d->C % 8 == 0 && !one_tap &&
               (d->stride_h > 1 || d->stride_w > 1 ? has_classes(d) : d->R * d->S <= 32);
    pl->fast = ((d->K % bk == 0 || (one_tap && d->K % 8 == 0)) && d->C % 8 == 0) || pl->flat;
    bk64_ok = d->K % 64 == 0 || (one_tap && d->K % 8 == 0);
    pl->bytesA = 2 * ny; pl->bytesB = 2 * nw; pl->bytesD = 2 * nx;
  } else {
    a.M = d->K; a.N = d->R * d->S * d->C; a.Kred = d->N * P * Q;
    g.IH = d->H; g.IW = d->W; g.IC = d->C; g.OH = P; g.OW = Q;
    pl->fast = d->K % 8 == 0 && d->C % 8 == 0;
    pl->bytesA = 2 * ny; pl->bytesB = 2 * nx; pl->bytesD = 2 * nw;  // A = dy, B = x
  }
  // a grid of one row or column never steps: the kernels' sums of coordinates and strides then stay far below 2^31
  if (op != JZ_BWD_DATA && P == 1) g.sh = 1;
  if (op != JZ_BWD_DATA && Q == 1) g.sw = 1;
  a.sc_on = 0; a.sc_H = a.sc_W = 0; a.sc_sh = a.sc_sw = 1; a.sc_oh = a.sc_ow = 0; a.sc_fill = 0;
  a.w_taps = d->R * d->S; a.w_tap0 = 0; a.w_tap_r = d->S; a.w_tap_s = 1;
  g.always_mask = 0;
  a.bw_x = BW_GATHER;
  if (op == JZ_BWD_WEIGHT && d->stride_h == 1 && d->stride_w == 1) {
    if (d->R == 1 && d->S == 1 && d->pad_h == 0 && d->pad_w == 0) a.bw_x = BW_MATRIX;
    else if (pl->fast && P == d->H && Q == d->W && (long long)d->R * d->W < (1ll << 30) &&
             (long long)pl->bytesB + 2ll * d->C * ((long long)d->pad_h * d->W + d->pad_w) < 0xfffffff0ll)
      a.bw_x = BW_SAME;
  }
  if (op == JZ_BWD_DATA && pl->fast && d->R == 1 && d->S == 1 && d->pad_h == 0 && d->pad_w == 0 &&
      (d->stride_h > 1 || d->stride_w > 1)) {
    // strided 1x1 layer (the ResNet downsampling convs): only input pixels (p*sh, q*sw) receive gradient, so the GEMM
    // runs over the N*P*Q output pixels as a stride-1 problem and the epilogue scatters its rows (and the zeros)
    a.M = d->N * P * Q;
    g.OH = P; g.OW = Q; g.sh = 1; g.sw = 1;
    a.sc_on = 1; a.sc_H = d->H; a.sc_W = d->W; a.sc_sh = d->stride_h; a.sc_sw = d->stride_w; a.sc_fill = 1;
  }
  g.row_pitch = g.IW * g.IC;
  g.pix_step = g.IC;
  g.s_step = g.IC;

  // small-channel layers: gather from a zero-padded 4-channel copy (see pad_to_c4)
  if (!pl->fast && op != JZ_BWD_DATA && d->C <= 4 && d->stride_w % 2 == 0 && 4 * d->S <= 64 &&
      d->R <= 32 && (op == JZ_FWD || d->K % 8 == 0)) {
    // forward: the run of a filter row is one k tile (32 or 64 halves); backward-weight: the runs are columns of the
    // GEMM, whole 16-byte chunks suffice (an 11-tap row: 48 columns instead of 64, a quarter fewer columns to compute)
    const int KT = op == JZ_BWD_WEIGHT ? (4 * d->S + 7) & ~7 : 4 * d->S <= 32 ? 32 : 64;
    int Hp = d->H + 2 * d->pad_h, Wp = d->W + 2 * d->pad_w;
    if (Wp < (Q - 1) * d->stride_w + KT / 4) Wp = (Q - 1) * d->stride_w + KT / 4;
    Wp = (Wp + 1) & ~1;  // rows stay 16-byte aligned
    const long long nxp = (long long)d->N * Hp * Wp * 4;
    if (nxp <= lim && Hp <= 65535 && d->N < 65535) {
      pl->packed = true;
      pl->fast = true;
      pl->Hp = Hp; pl->Wp = Wp; pl->KT = KT;
      pl->xp_bytes = up256((size_t)nxp * 2);
      pl->wp_bytes = up256((size_t)d->K * d->R * KT * 2);
      g.IH = Hp; g.IW = Wp; g.IC = KT; g.S = 1; g.ph = 0; g.pw = 0;
      g.row_pitch = Wp * 4; g.pix_step = 4; g.s_step = 0;
      if (op == JZ_FWD) {
        a.Kred = d->R * KT;
        g.kvalid = 4 * d->S;
        bk = KT;
        forced_bk = KT;
      } else {
        a.N = d->R * KT;
      }
    }
  }
  // the vector kernel marks padding taps with a 32-bit mask per row and, for backward-data, needs the source pixel to
  // be an affine function of the tap (unit stride); other shapes take its variant with per-load tap arithmetic
  pl->gen = pl->fast && !pl->packed && op != JZ_BWD_WEIGHT &&
            (g.R * g.S > 32 || (op == JZ_BWD_DATA && (g.sh != 1 || g.sw != 1)));
  finish_geometry(g);
  if (!pl->fast) bk = BK;  // the element-wise kernel walks 64-deep tiles
  pl->bk = bk;
  if (pl->packed && !forced_bk) forced_bk = 32;  // small-channel backward-weight: 4-wavefront 32-deep kernels
  choose_tiling(pl, bk64_ok, forced_bk);
  if (pl->packed && op == JZ_FWD && !pl->rt_forced) {
    StemArgs sa;
    pl->stem = stem_fwd_setup(*pl, d, &sa);
  }
  const size_t part = a.splits > 1 ? (size_t)a.splits * a.M * a.N * sizeof(float) : 0;
  pl->part_offset = pl->packed ? pl->xp_bytes + pl->wp_bytes : 0;
  pl->ws_bytes = pl->part_offset + part;
  // Strided multi-tap backward-data: input pixel (h, w) only meets the taps r = (h + ph) mod sh (+ sh, + 2 sh, ...) and
  // likewise along w, so the pixels of one parity class (h mod sh, w mod sw) form a unit-stride backward-data problem
  // on the dy grid with the filter's taps of that class.  Together they do the useful multiply-adds only (the per-load
  // variant fetches and masks every tap for every pixel: sh * sw times the work), and they run as one launch out of the
  // filter where it lies.  Packing each class's filter into the workspace and one launch per class took five launches:
  // 128, 256 and 512 channels at batch 24: 35, 43 and 68 us, now 17, 21 and 23.  Every class needs a tap (R >= sh, S >= sw).
  // Nothing is kept in a workspace.  Layers with whole k tiles per tap ask for the filter's size all the same, as they always
  // have; the flattened ones, which never did, do not.
  pl->classes = pl->gen && op == JZ_BWD_DATA && has_classes(d);
  if (pl->classes) pl->ws_bytes = pl->flat ? 0 : up256((size_t)nw * 2);
  pl->element_ws_bytes = pl->ws_bytes;
  if (!pl->fast) plan_widened(op, d, pl);
  return JZ_OK;
}

// Channel counts that are not multiples of 8 leave nothing to load 16 bytes at a time, and the element-wise kernel is 5-20
// times slower than the vector kernels.  Where rounding the counts up adds at most half to the multiply-adds, the layer
// runs on zero-extended copies instead (memory-bound passes over the operands and the result).  Below that (5 -> 3
// channels would become 8 -> 8) the element-wise kernel stays.
void plan_widened(int op, const jz_conv_desc* d, Plan* pl) {
  const int C8 = (d->C + 7) & ~7, K8 = (d->K + 7) & ~7;
  jz_conv_desc w = *d;
  w.C = C8;
  if (op != JZ_FWD) w.K = K8;  // forward takes any number of output channels
  if (w.C == d->C && w.K == d->K) return;
  if ((double)w.C * w.K > 1.5 * d->C * d->K) return;
  Plan in;
  if (compute_plan(pl->beside ? op | JZ_BESIDE : op, &w, &in) != JZ_OK || !in.fast) return;
  const size_t npix = (size_t)d->N * d->H * d->W, nout = pl->bytesD / 2;
  const size_t ny = op == JZ_FWD ? nout : (pl->bytesA / 2) / d->K * w.K, nx = npix * w.C, nw = (size_t)w.K * d->R * d->S * w.C;
  const bool x_wide = w.C != d->C, y_wide = w.K != d->K, w_wide = x_wide || y_wide;
  if (op == JZ_FWD) {
    pl->wide_a_bytes = x_wide ? up256(nx * 2) : 0;
    pl->wide_b_bytes = w_wide ? up256(nw * 2) : 0;
  } else if (op == JZ_BWD_DATA) {
    pl->wide_a_bytes = y_wide ? up256(ny * 2) : 0;
    pl->wide_b_bytes = w_wide ? up256(nw * 2) : 0;
    pl->wide_d_bytes = x_wide ? up256(nx * 2) : 0;
  } else {
    pl->wide_a_bytes = y_wide ? up256(ny * 2) : 0;
    pl->wide_b_bytes = x_wide ? up256(nx * 2) : 0;
    pl->wide_d_bytes = w_wide ? up256(nw * 2) : 0;
  }
  pl->widen = true;
  pl->wide = w;
  const size_t need = pl->wide_a_bytes + pl->wide_b_bytes + pl->wide_d_bytes + in.ws_bytes;
  if (need > pl->ws_bytes) pl->ws_bytes = need;
}

int make_plan(int op, const jz_conv_desc* d, Plan* pl, size_t limit = kPartialSumLimit) {
  if (!d) return JZ_ERR_NULL;
  return cached_plan(g_tune_generation.load(std::memory_order_acquire), PlanKey{op, -1, -1, limit, *d}, pl,
                     [&](Plan* p) { return compute_plan(op, d, p, limit); });
}

// One parity class (ca, cb) of a strided multi-tap backward-data layer as a plan of its own (see compute_plan).  base: the
// layer's plan; false: the class has no pixels.
bool compute_class_plan(const jz_conv_desc* d, const Plan& base, int ca, int cb, Plan* pl) {
  const int sh = d->stride_h, sw = d->stride_w;
  const int P = out_dim(d->H, d->pad_h, d->R, sh), Q = out_dim(d->W, d->pad_w, d->S, sw);
  const int Ha = (d->H - ca + sh - 1) / sh, Wb = (d->W - cb + sw - 1) / sw;     // pixels h = ca + sh i, w = cb + sw l
  const int r0 = (ca + d->pad_h) % sh, s0 = (cb + d->pad_w) % sw;               // first tap of the class
  const int Ra = (d->R - r0 + sh - 1) / sh, Sb = (d->S - s0 + sw - 1) / sw;     // taps r0 + sh j, s0 + sw i
  if (Ha <= 0 || Wb <= 0) return false;
  *pl = base;
  pl->gen = false;
  pl->classes = false;
  GemmArgs& a = pl->args;
  ConvGeom& g = a.g;
  a.M = d->N * Ha * Wb; a.N = d->C; a.Kred = Ra * Sb * d->K;
  g.IH = P; g.IW = Q; g.IC = d->K; g.OH = Ha; g.OW = Wb;
  g.R = Ra; g.S = Sb; g.sh = 1; g.sw = 1;
  g.ph = (ca + d->pad_h) / sh; g.pw = (cb + d->pad_w) / sw;   // dy row of tap j for pixel row i: i + ph - j
  g.row_pitch = Q * d->K; g.pix_step = d->K; g.s_step = d->K;
  g.kvalid = 0;
  g.always_mask = 1;   // the class grid and the dy grid are not tied by the usual size formula
  a.w_tap0 = r0 * d->S + s0; a.w_tap_r = sh * d->S; a.w_tap_s = sw;   // its taps among the filter's
  a.sc_on = 1; a.sc_H = d->H; a.sc_W = d->W; a.sc_sh = sh; a.sc_sw = sw; a.sc_oh = ca; a.sc_ow = cb; a.sc_fill = 0;
  a.bw_x = BW_GATHER;
  finish_geometry(g);
  pl->bk = 32;
  choose_tiling(pl, d->K % 64 == 0, 0);
  if (!pl->tuned) {  // the classes run in one launch: one variant, chosen for all pixels and a class's share of the taps
    Plan all = *pl;
    all.args.M = d->N * d->H * d->W;
    all.args.Kred = (d->R * d->S * d->K + sh * sw - 1) / (sh * sw);
    all.args.g.R = d->R; all.args.g.S = d->S;
    choose_tiling(&all, d->K % 64 == 0, 0, false);
    pl->BM = all.BM; pl->BN = all.BN; pl->bk = all.bk; pl->waves = all.waves; pl->nst = all.nst;
    set_tiles(pl, 1);
  }
  pl->part_offset = 0;
  pl->ws_bytes = 0;
  return true;
}

bool make_class_plan(const jz_conv_desc* d, const Plan& base, int ca, int cb, Plan* pl) {
  return cached_plan(g_tune_generation.load(std::memory_order_acquire), PlanKey{JZ_BWD_DATA, ca, cb, 0, *d}, pl,
                     [&](Plan* p) { return compute_class_plan(d, base, ca, cb, p) ? 1 : 0; }) != 0;
}

// slabs of rows whose sums a split reduction leaves (splitk_reduce_stats): at most 64, so that the normalization's apply pass
// can add them up itself, unless that would leave fewer than two workgroups per compute unit
int reduce_slab_rows(const GemmArgs& a) {
  const int passes = (a.M + RS_ROWS - 1) / RS_ROWS, cols = (a.N + RS_COLS - 1) / RS_COLS;
  const int slabs = cols < 8 ? 512 / cols : 64;
  return (passes + slabs - 1) / slabs * RS_ROWS;
}
int reduce_slabs(const GemmArgs& a) {
  const int rows = reduce_slab_rows(a);
  return (a.M + rows - 1) / rows;
}
// a split reduction that can leave the column sums: one over a whole [M][N] result, whole 16-byte pieces of its rows
bool split_leaves_stats(const Plan& pl) { return pl.args.splits > 1 && !pl.widen && !pl.packed && !pl.args.sc_on && (pl.args.N & 7) == 0; }

// a forward plan whose kernel can leave the per-tile column sums: the ring kernels (their LDS holds the sums), or the
// reduction behind a split one
bool plan_leaves_stats(const Plan& pl) {
  return pl.op == JZ_FWD && ((pl.fast && !pl.flat && pl.args.splits == 1) || split_leaves_stats(pl));
}
// a backward-data plan whose kernel can leave the sums of a batch-norm backward: the ring kernels with masks and
// no scatter epilogue, whole 16-byte pieces of a row, or the reduction behind a split one
bool plan_leaves_bwd_stats(const Plan& pl) {
  return pl.op == JZ_BWD_DATA && !pl.classes &&
         ((pl.fast && !pl.gen && !pl.flat && pl.args.splits == 1 && !pl.args.sc_on && (pl.args.N & 7) == 0) || split_leaves_stats(pl));
}
// row groups of those sums: row tiles, or slabs of the reduction
int stats_groups(const Plan& pl) { return pl.args.splits > 1 ? reduce_slabs(pl.args) : pl.args.tiles_m; }

// log2 of the split lanes per output group: enough workgroups to cover the chip first, then shorten each thread's chain
int reduce_lanes(long long MN, int splits) {
  int lg = 0;
  while (splits > 1 && lg < 5 && (2 << lg) <= splits && ((MN + 3) / 4 + (256 >> lg) - 1) / (256 >> lg) < 1024) ++lg;
  return lg;
}

int run_widened(int op, const jz_conv_desc* d, const Plan& pl, const void* A, const void* B, void* D, void* ws, size_t ws_bytes,
                void* stream, const jz::SumsqSink* sink);

// The plan that a call runs in the workspace it was given, or why it is refused; what run() checks before its first launch.
// A, B in the kernel's order: FWD (x, w), BWD_DATA (dy, w), BWD_WEIGHT (dy, x)
// plan_op may be JZ_BWD_WEIGHT | JZ_BESIDE
int admit(int plan_op, const jz_conv_desc* d, const void* A, const void* B, const void* D, const void* ws, size_t ws_bytes, Plan* out,
          bool stats = false, int stats_tiles_m = 0, const jz::BnBwdOperands* bn = nullptr) {
  Plan& pl = *out;
  int rc = make_plan(plan_op, d, &pl);
  if (rc != JZ_OK) return rc;
  const int op = pl.op;
  // the caller sized the buffer of the column sums from an earlier plan: it has to be this plan (the run-time tuning table
  // may have been changed in between)
  if (stats && !(op == JZ_BWD_DATA ? plan_leaves_bwd_stats(pl) && bn != nullptr : plan_leaves_stats(pl))) return JZ_ERR_UNSUPPORTED;
  if (stats && stats_groups(pl) != stats_tiles_m) return JZ_ERR_UNSUPPORTED;
  if (!A || !B || !D) return JZ_ERR_NULL;
  if (!aligned16(A) || !aligned16(B) || !aligned16(D) || (ws && !aligned16(ws))) return JZ_ERR_ALIGN;
  if (overlaps(D, pl.bytesD, A, pl.bytesA) || overlaps(D, pl.bytesD, B, pl.bytesB)) return JZ_ERR_ALIAS;
  if (pl.widen && (!ws || ws_bytes < pl.ws_bytes)) {  // no room for the copies: the element-wise kernel
    pl.widen = false;
    pl.ws_bytes = pl.element_ws_bytes;
  }
  const size_t room = ws ? ws_bytes : 0;
  if (room < pl.ws_bytes && !stats && !pl.rt_forced) {  // fewer splits (a choice made by hand runs as it was made, or not at all)
    if ((rc = make_plan(plan_op, d, &pl, room > pl.part_offset ? room - pl.part_offset : 0)) != JZ_OK) return rc;
    if (pl.widen) {
      pl.widen = false;
      pl.ws_bytes = pl.element_ws_bytes;
    }
    if (!runs_with_fewer_splits(op, pl.args.M, pl.args.N, pl.args.splits)) return JZ_ERR_WORKSPACE;
  }
  if (room < pl.ws_bytes) return JZ_ERR_WORKSPACE;
  if (pl.ws_bytes > 0 && (overlaps(ws, pl.ws_bytes, A, pl.bytesA) || overlaps(ws, pl.ws_bytes, B, pl.bytesB) ||
                          overlaps(ws, pl.ws_bytes, D, pl.bytesD)))
    return JZ_ERR_ALIAS;
  return JZ_OK;
}

int run(int op, const jz_conv_desc* d, const void* A, const void* B, void* D, void* ws, size_t ws_bytes, void* stream,
        float* stats = nullptr, int stats_tiles_m = 0, const jz::SumsqSink* sink = nullptr, const jz::BnBwdOperands* bn = nullptr,
        jz::BnTail* tail = nullptr) {
  Plan pl;
  int rc = admit(op, d, A, B, D, ws, ws_bytes, &pl, stats != nullptr, stats_tiles_m, bn);
  if (rc != JZ_OK) return rc;
  op = pl.op;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (pl.widen) return run_widened(op, d, pl, A, B, D, ws, ws_bytes, stream, sink);
  if (pl.classes) {
    // strided multi-tap backward-data: the classes of one variant in launches of up to kGemmSet, those with the most taps first
    // (the last workgroups to start are then the shortest)
    Plan cps[kMaxClasses];
    int n = 0;
    for (int ca = 0; ca < d->stride_h; ++ca)
      for (int cb = 0; cb < d->stride_w; ++cb)
        if (make_class_plan(d, pl, ca, cb, &cps[n])) {
          GemmArgs& c = cps[n++].args;
          c.A = static_cast<const unsigned short*>(A);
          c.B = static_cast<const unsigned short*>(B);
          c.D16 = static_cast<unsigned short*>(D);
          c.bytesA = (unsigned)pl.bytesA;
          c.bytesB = (unsigned)pl.bytesB;
          c.Dpart = nullptr;
          c.stats = nullptr;
          c.st_y = c.st_c = c.st_add = nullptr;
          c.st_mean = c.st_invstd = nullptr;
        }
    int order[kMaxClasses];
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order, order + n, [&](int x, int y) { return cps[x].args.Kred > cps[y].args.Kred; });
    bool done[kMaxClasses] = {};
    for (int i = 0; i < n; ++i) {
      if (done[i]) continue;
      const Plan& first = cps[order[i]];
      GemmSet set;
      int k = 0;
      set.first[0] = 0;
      for (int j = i; j < n && k < kGemmSet; ++j) {
        const Plan& c = cps[order[j]];
        if (done[j] || c.BM != first.BM || c.BN != first.BN || c.bk != first.bk || c.waves != first.waves || c.nst != first.nst) continue;
        done[j] = true;
        set.g[k] = c.args;
        set.first[k + 1] = set.first[k] + (unsigned)c.args.tiles_m * (unsigned)c.args.tiles_n;
        ++k;
      }
      for (; k < kGemmSet; ++k) {
        set.g[k] = set.g[0];
        set.first[k + 1] = set.first[k];
      }
      if ((rc = launch_bwd_data(first, st, &set)) != JZ_OK) return rc;
    }
    return JZ_OK;
  }
  GemmArgs& a = pl.args;
  a.A = static_cast<const unsigned short*>(A);
  a.B = static_cast<const unsigned short*>(B);
  a.D16 = static_cast<unsigned short*>(D);
  a.bytesA = (unsigned)pl.bytesA;
  a.bytesB = (unsigned)pl.bytesB;
  a.Dpart = reinterpret_cast<float*>(static_cast<char*>(ws) + pl.part_offset);
  a.stats = stats;
  a.st_y = a.st_c = a.st_add = nullptr;
  a.st_mean = a.st_invstd = nullptr;
  if (stats && op == JZ_BWD_DATA) {
    a.st_add = static_cast<const unsigned short*>(bn->add16);
    a.st_y = static_cast<const unsigned short*>(bn->y16);
    a.st_c = static_cast<const unsigned short*>(bn->x16);
    a.st_mean = bn->mean;
    a.st_invstd = bn->invstd;
  }
  unsigned short* dwp = nullptr;
  if (pl.packed) {
    unsigned short* xp = static_cast<unsigned short*>(ws);
    unsigned short* wp = reinterpret_cast<unsigned short*>(static_cast<char*>(ws) + pl.xp_bytes);
    const unsigned short* x = static_cast<const unsigned short*>(op == JZ_FWD ? A : B);
    const unsigned short* wsrc = op == JZ_FWD ? static_cast<const unsigned short*>(B) : nullptr;
    StemArgs sa;
    const bool stem = pl.stem && !stats && stem_fwd_setup(pl, d, &sa);
    PadArgs pa{x, wsrc, xp, wp, d->N, d->H, d->W, d->C, pl.Hp, pl.Wp, d->pad_h, d->pad_w, d->K, d->R, d->S,
               stem ? sa.NKS * 16 : pl.KT, stem ? 1 : 0, (unsigned)pl.Hp * (pl.Wp / 2), 0, make_fastdiv(pl.Wp / 2)};
    pa.groups = (pa.pairs + PAD_PAIRS - 1) / PAD_PAIRS;
    const unsigned wgroups = wsrc ? ((unsigned)(pa.K * pa.R * pa.KT) + PAD_THREADS - 1) / PAD_THREADS : 0;
    hipLaunchKernelGGL(pad_to_c4, dim3(pa.groups * (unsigned)d->N + wgroups), dim3(PAD_THREADS), 0, st, pa);
    if (stem) {
      if ((rc = jz::launch_status()) != JZ_OK) return rc;
      sa.xp = xp;
      sa.wq = wp;
      sa.y = static_cast<unsigned short*>(D);
      return launch_stem_fwd(sa, st);
    }
    if (op == JZ_FWD) {
      a.A = xp; a.bytesA = (unsigned)pl.xp_bytes;
      a.B = wp; a.bytesB = (unsigned)pl.wp_bytes;
    } else {
      a.B = xp; a.bytesB = (unsigned)pl.xp_bytes;
      dwp = wp;
      a.D16 = dwp;
    }
    if ((rc = jz::launch_status()) != JZ_OK) return rc;
  }
  const bool epilogue_stats = stats && a.splits == 1;
  if (pl.window) {
    if (op == JZ_FWD) rc = epilogue_stats ? launch_window_fwd_stats(pl, st) : launch_window_fwd(pl, st);
    else rc = !epilogue_stats ? launch_window_bwd_data(pl, st) : bn->block_end ? launch_window_bwd_data_block_end(pl, st) : launch_window_bwd_data_stats(pl, st);
  } else if (op == JZ_FWD) rc = epilogue_stats ? launch_fwd_stats(pl, st) : launch_fwd(pl, st);
  else if (op == JZ_BWD_DATA) rc = !epilogue_stats ? launch_bwd_data(pl, st) : bn->block_end ? launch_bwd_data_block_end(pl, st) : launch_bwd_data_stats(pl, st);
  else rc = launch_bwd_weight(pl, st);
  if (rc != JZ_OK) return rc;
  const int lg = reduce_lanes((long long)a.M * a.N, a.splits);
  if (a.splits > 1 && stats && tail && reduce_normalizes(a.M, a.splits)) {
    NormArgs n{a.Dpart, a.D16, a.M, a.N, a.splits, 1 << lg, a.st_y, a.st_c, op == JZ_FWD ? static_cast<const unsigned short*>(tail->residual16) : a.st_add,
               a.st_mean, a.st_invstd, tail->gamma, tail->beta, tail->eps, tail->relu, 1.0 / (double)a.M,
               static_cast<unsigned short*>(op == JZ_FWD ? tail->y16 : tail->dx16), tail->save_mean, tail->save_invstd,
               static_cast<unsigned short*>(tail->dgamma16), static_cast<unsigned short*>(tail->dbeta16)};
    const dim3 grid((unsigned)((a.N + RN_COLS - 1) / RN_COLS));
    if (op == JZ_FWD) hipLaunchKernelGGL(splitk_reduce_norm<0>, grid, dim3(RN_THREADS), 0, st, n);
    else if (!bn->block_end) hipLaunchKernelGGL(splitk_reduce_norm<1>, grid, dim3(RN_THREADS), 0, st, n);
    else hipLaunchKernelGGL(splitk_reduce_norm<2>, grid, dim3(RN_THREADS), 0, st, n);
    tail->done = true;
    return jz::launch_status();
  }
  if (a.splits > 1 && stats) {
    const dim3 grid((unsigned)((a.N + RS_COLS - 1) / RS_COLS), (unsigned)reduce_slabs(a));
    const int mode = op == JZ_FWD ? 0 : bn->block_end ? 2 : 1;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, a.Dpart, a.D16, a.M, a.N, a.splits, 1 << lg, reduce_slab_rows(a), a.st_y, a.st_c, a.st_add,
                         a.st_mean, a.st_invstd, stats);
    };
    if (mode == 0) go(splitk_reduce_stats<0>);
    else if (mode == 1) go(splitk_reduce_stats<1>);
    else go(splitk_reduce_stats<2>);
    return jz::launch_status();
  }
  if (a.splits > 1) {
    long long MN = (long long)a.M * a.N;
    const long long per_block = 256 >> lg;
    unsigned blocks = (unsigned)(((MN + 3) / 4 + per_block - 1) / per_block);
    // small-channel backward-weight: the reduction writes the real filter entries straight into dw
    if (sink) {
      const unsigned grid = blocks < 2048u ? blocks : 2048u;  // at most 32 workgroups per counter quadruple of the sink
      hipLaunchKernelGGL(splitk_reduce_sumsq, dim3(grid), dim3(256), 0, st, a.Dpart, dwp ? static_cast<unsigned short*>(D) : a.D16,
                         MN, a.splits, lg, dwp ? pl.KT / 4 : 0, d->S, d->C, (long long)blocks, *sink);
      sink = nullptr;  // taken
    } else {
      hipLaunchKernelGGL(splitk_reduce, dim3(blocks), dim3(256), 0, st, a.Dpart, dwp ? static_cast<unsigned short*>(D) : a.D16,
                         MN, a.splits, lg, dwp ? pl.KT / 4 : 0, d->S, d->C);
    }
    if ((rc = jz::launch_status()) != JZ_OK) return rc;
    dwp = nullptr;
  }
  if (dwp) {
    int ndw = d->K * d->R * d->S * d->C;
    hipLaunchKernelGGL(unpack_filter_c4, dim3((unsigned)((ndw + 255) / 256)), dim3(256), 0, st, dwp,
                       static_cast<unsigned short*>(D), d->K, d->R, d->S, d->C, pl.KT);
    if ((rc = jz::launch_status()) != JZ_OK) return rc;
  }
  // no split reduction to take the sum of squares in: one pass over the gradient just written (still in cache)
  if (sink) rc = jz::sumsq_half_launch(static_cast<const unsigned short*>(D), (long long)d->K * d->R * d->S * d->C, *sink, st);
  return rc;
}

// a layer with channel counts that are not multiples of 8 on zero-extended copies (plan_widened)
int run_widened(int op, const jz_conv_desc* d, const Plan& pl, const void* A, const void* B, void* D, void* ws, size_t ws_bytes,
                void* stream, const jz::SumsqSink* sink) {
  const jz_conv_desc& w = pl.wide;
  const int RS = d->R * d->S;
  char* base = static_cast<char*>(ws);
  char* const inner_ws = base + pl.wide_a_bytes + pl.wide_b_bytes + pl.wide_d_bytes;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const long long npix = (long long)d->N * d->H * d->W;
  const long long nout = (long long)d->N * out_dim(d->H, d->pad_h, d->R, d->stride_h) * out_dim(d->W, d->pad_w, d->S, d->stride_w);
  WidenArgs wa{};
  int nt = 0;
  long long most = 0;
  auto copy = [&](const void* src, char* dst, long long rows, long long real_rows, int c, int c8) {
    wa.src[nt] = static_cast<const unsigned short*>(src);
    wa.dst[nt] = reinterpret_cast<unsigned short*>(dst);
    wa.chunks[nt] = rows * (c8 / 8);
    wa.real_rows[nt] = real_rows;
    wa.C[nt] = c;
    wa.d_cpr[nt] = make_fastdiv((unsigned)(c8 / 8));
    if (wa.chunks[nt] > most) most = wa.chunks[nt];
    ++nt;
  };
  const void* a2 = A;
  const void* b2 = B;
  if (pl.wide_a_bytes) {
    a2 = base;
    if (op == JZ_FWD) copy(A, base, npix, npix, d->C, w.C);
    else copy(A, base, nout, nout, d->K, w.K);
  }
  if (pl.wide_b_bytes) {
    char* const p = base + pl.wide_a_bytes;
    b2 = p;
    if (op == JZ_BWD_WEIGHT) copy(B, p, npix, npix, d->C, w.C);
    else copy(B, p, (long long)w.K * RS, (long long)d->K * RS, d->C, w.C);
  }
  void* d2 = pl.wide_d_bytes ? base + pl.wide_a_bytes + pl.wide_b_bytes : static_cast<char*>(D);
  int rc = JZ_OK;
  if (nt > 0) {
    const long long blocks = (most + 255) / 256;
    hipLaunchKernelGGL(widen_channels, dim3((unsigned)(blocks < 4096 ? blocks : 4096), (unsigned)nt), dim3(256), 0, st, wa);
    if ((rc = jz::launch_status()) != JZ_OK) return rc;
  }
  const size_t used = (size_t)(inner_ws - base);
  rc = run(pl.beside ? op | JZ_BESIDE : op, &w, a2, b2, d2, ws_bytes > used ? inner_ws : nullptr, ws_bytes - used, stream, nullptr, 0, pl.wide_d_bytes ? nullptr : sink);
  if (rc != JZ_OK || !pl.wide_d_bytes) return rc;
  const long long n = op == JZ_BWD_DATA ? npix * d->C : (long long)d->K * RS * d->C;
  const long long blocks = (n + 255) / 256;
  hipLaunchKernelGGL(narrow_channels, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, st, static_cast<const unsigned short*>(d2),
                     static_cast<unsigned short*>(D), n, make_fastdiv((unsigned)d->C), w.C);
  if ((rc = jz::launch_status()) != JZ_OK) return rc;
  return sink ? jz::sumsq_half_launch(static_cast<const unsigned short*>(D), n, *sink, st) : JZ_OK;
}

int fc_desc(int mode, int batch, int in_features, int out_features, jz_conv_desc* d) {
  if (mode != JZ_FWD && mode != JZ_BWD_DATA && mode != JZ_BWD_WEIGHT) return JZ_ERR_UNSUPPORTED;
  if (batch <= 0 || in_features <= 0 || out_features <= 0) return JZ_ERR_SHAPE;
  // a fully connected layer is a 1x1 convolution over a 1x1 image
  *d = jz_conv_desc{batch, 1, 1, in_features, out_features, 1, 1, 1, 1, 0, 0};
  return JZ_OK;
}

}  // namespace

// for the fused convolution + batch normalization entry point (jz_bn.hip)
int jz::conv_fwd_stats_plan(const jz_conv_desc* d, size_t* conv_ws_bytes, int* tiles_m) {
  Plan pl;
  int rc = make_plan(JZ_FWD, d, &pl);
  if (rc != JZ_OK) return rc;
  *conv_ws_bytes = pl.ws_bytes;
  *tiles_m = plan_leaves_stats(pl) ? stats_groups(pl) : 0;
  return JZ_OK;
}
int jz::conv_fwd_run(const jz_conv_desc* d, const void* x, const void* w, void* y, void* ws, size_t ws_bytes, float* stats,
                     int stats_tiles_m, BnTail* tail, void* stream) {
  return run(JZ_FWD, d, x, w, y, ws, ws_bytes, stream, stats, stats_tiles_m, nullptr, nullptr, tail);
}
int jz::conv_bwd_data_stats_plan(const jz_conv_desc* d, size_t* conv_ws_bytes, int* tiles_m) {
  Plan pl;
  int rc = make_plan(JZ_BWD_DATA, d, &pl);
  if (rc != JZ_OK) return rc;
  *conv_ws_bytes = pl.ws_bytes;
  *tiles_m = plan_leaves_bwd_stats(pl) ? stats_groups(pl) : 0;
  return JZ_OK;
}
int jz::conv_bwd_data_run(const jz_conv_desc* d, const void* dy, const void* w, void* dx, void* ws, size_t ws_bytes, float* stats,
                          int stats_tiles_m, const BnBwdOperands* bn, BnTail* tail, void* stream) {
  return run(JZ_BWD_DATA, d, dy, w, dx, ws, ws_bytes, stream, stats, stats_tiles_m, nullptr, bn, tail);
}

extern "C" int jz_conv2d_workspace_bytes(int op, const jz_conv_desc* desc, size_t* bytes) {
  if (!bytes) return JZ_ERR_NULL;
  Plan pl;
  int rc = make_plan(op, desc, &pl);
  if (rc != JZ_OK) return rc;
  *bytes = pl.ws_bytes;
  return JZ_OK;
}

extern "C" int jz_conv2d_describe_plan(int op, const jz_conv_desc* desc, char* text, size_t text_bytes) {
  if (!text || text_bytes == 0) return JZ_ERR_NULL;
  Plan pl;
  int rc = make_plan(op, desc, &pl);
  if (rc != JZ_OK) return rc;
  if (pl.classes) {  // the launches of the parity classes: the first class stands for all (same filter shape up to a tap row / column)
    Plan cp;
    if (make_class_plan(desc, pl, 0, 0, &cp)) {
      cp.classes = true;
      cp.args.sc_on = 0;
      plan_text(cp, text, text_bytes);
      return JZ_OK;
    }
  }
  plan_text(pl, text, text_bytes);
  return JZ_OK;
}

extern "C" int jz_conv2d_tune_set(int op, const jz_conv_desc* desc, int tile_m, int tile_n, int k_tile, int wavefronts,
                                  int ring, int splits) {
  Plan pl;
  int rc = make_plan(op, desc, &pl);
  if (rc != JZ_OK) return rc;
  if (pl.beside) return JZ_ERR_UNSUPPORTED;  // a recorded choice is for both kinds of call
  if (!pl.fast || splits < 1) return JZ_ERR_UNSUPPORTED;  // the element-wise path has one kernel shape
  const Variant* v = nullptr;
  for (const Variant& c : kVariants)
    if (c.BM == tile_m && c.BN == tile_n && c.bk == k_tile && c.waves == wavefronts && c.nst == ring) v = &c;
  Variant window{};
  for (const WindowVariant& c : kWindows)
    if (c.BM == tile_m && c.BN == tile_n && c.ck == k_tile && c.waves == wavefronts && c.nst + kWindowRing == ring && window_fits(pl, c)) {
      window.BM = c.BM; window.BN = c.BN; window.bk = c.ck; window.waves = c.waves; window.nst = ring;
      v = &window;
    }
  if (!v) return JZ_ERR_UNSUPPORTED;
  if (pl.classes) {  // the variant goes to every parity class's launch (their reductions are never split)
    std::vector<Tuned> keys;
    for (int ca = 0; ca < desc->stride_h; ++ca)
      for (int cb = 0; cb < desc->stride_w; ++cb) {
        Plan cp;
        if (!make_class_plan(desc, pl, ca, cb, &cp)) continue;
        const GemmArgs& a = cp.args;
        keys.push_back(Tuned{1, a.M, a.N, a.Kred, a.g.R * a.g.S, a.sc_on, tile_m, tile_n, k_tile, wavefronts, ring, 1});
      }
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    g_tune_generation.fetch_add(1);
    for (const Tuned& t : keys) {
      bool found = false;
      for (Tuned& e : g_tune_rt)
        if (same_key(e, t)) { e = t; found = true; }
      if (!found) g_tune_rt.push_back(t);
    }
    return JZ_OK;
  }
  // per-load tap arithmetic exists for the four basic 4-wavefront tiles, 32 deep, four-stage ring
  if ((pl.gen || pl.flat) && (v->waves != 4 || v->bk != 32 || v->nst != 4 || v->BM > 128 || v->BN > 128)) return JZ_ERR_UNSUPPORTED;
  // the small-channel path runs the 4-wavefront kernels of the four basic tiles at its own k tile depth only
  if (pl.packed && (v->waves != 4 || v->BM > 128 || v->BN > 128 || k_tile != pl.bk || (ring == 3 && k_tile != 32)))
    return JZ_ERR_UNSUPPORTED;
  const GemmArgs& a = pl.args;
  const Tuned t{op == JZ_FWD ? 0 : op == JZ_BWD_DATA ? 1 : 2, a.M, a.N, a.Kred, a.g.R * a.g.S, a.sc_on,
                tile_m, tile_n, k_tile, wavefronts, ring, splits};
  std::lock_guard<std::mutex> lock(g_tune_mutex);
  g_tune_generation.fetch_add(1);
  for (Tuned& e : g_tune_rt)
    if (same_key(e, t)) {
      e = t;
      return JZ_OK;
    }
  g_tune_rt.push_back(t);
  return JZ_OK;
}

extern "C" int jz_conv2d_tune_clear(void) {
  std::lock_guard<std::mutex> lock(g_tune_mutex);
  g_tune_generation.fetch_add(1);
  g_tune_rt.clear();
  g_use_table = true;
  return JZ_OK;
}

extern "C" int jz_conv2d_tune_use_table(int on) {
  std::lock_guard<std::mutex> lock(g_tune_mutex);
  g_tune_generation.fetch_add(1);
  g_use_table = on != 0;
  return JZ_OK;
}

extern "C" int jz_conv2d_fwd(const jz_conv_desc* desc, const void* x16, const void* w16, void* y16, void* ws,
                             size_t ws_bytes, void* hip_stream) {
  return run(JZ_FWD, desc, x16, w16, y16, ws, ws_bytes, hip_stream);
}

extern "C" int jz_conv2d_bwd_data(const jz_conv_desc* desc, const void* dy16, const void* w16, void* dx16, void* ws,
                                  size_t ws_bytes, void* hip_stream) {
  return run(JZ_BWD_DATA, desc, dy16, w16, dx16, ws, ws_bytes, hip_stream);
}

extern "C" int jz_conv2d_bwd_weight(const jz_conv_desc* desc, const void* x16, const void* dy16, void* dw16, void* ws,
                                    size_t ws_bytes, void* hip_stream) {
  return run(JZ_BWD_WEIGHT, desc, dy16, x16, dw16, ws, ws_bytes, hip_stream);  // A = dy, B = x
}

// ---- backward-weight that also hands the gradient's sum of squares to the optimiser ---------------------------------
namespace {
int check_sink(const jz_sumsq_sink* sink, const void* dw, size_t dw_bytes, const void* ws, size_t ws_bytes, jz::SumsqSink* out) {
  if (!sink || !sink->sums || !sink->nonfinite) return JZ_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(sink->sums) & 127u) || (reinterpret_cast<uintptr_t>(sink->nonfinite) & 3u)) return JZ_ERR_ALIGN;
  if (overlaps(sink->sums, JZ_SUMSQ_SINK_BYTES, dw, dw_bytes) || overlaps(sink->nonfinite, sizeof(int), dw, dw_bytes) ||
      overlaps(sink->sums, JZ_SUMSQ_SINK_BYTES, ws, ws_bytes) || overlaps(sink->nonfinite, sizeof(int), ws, ws_bytes) ||
      overlaps(sink->sums, JZ_SUMSQ_SINK_BYTES, sink->nonfinite, sizeof(int)))
    return JZ_ERR_ALIAS;
  *out = jz::SumsqSink{static_cast<unsigned long long*>(sink->sums), sink->nonfinite};
  return JZ_OK;
}
}  // namespace

int jz::sumsq_half_launch(const unsigned short* g16, long long n, const jz::SumsqSink& sink, hipStream_t st) {
  if (n <= 0) return JZ_OK;
  long long want = (n / 8 + 255) / 256;  // one 16-byte group per thread and pass; at most 2^20 elements per workgroup
  const unsigned grid = (unsigned)(want < 1 ? 1 : (want > 1024 ? 1024 : want));
  hipLaunchKernelGGL(sumsq_half, dim3(grid), dim3(256), 0, st, g16, n, sink);
  return jz::launch_status();
}

extern "C" int jz_conv2d_bwd_weight_sumsq(const jz_conv_desc* desc, const void* x16, const void* dy16, void* dw16, void* ws,
                                          size_t ws_bytes, const jz_sumsq_sink* sink, void* hip_stream) {
  Plan pl;
  int rc = make_plan(JZ_BWD_WEIGHT, desc, &pl);
  if (rc != JZ_OK) return rc;
  jz::SumsqSink sk;
  if ((rc = check_sink(sink, dw16, pl.bytesD, ws, ws_bytes < pl.ws_bytes ? ws_bytes : pl.ws_bytes, &sk)) != JZ_OK) return rc;
  return run(JZ_BWD_WEIGHT, desc, dy16, x16, dw16, ws, ws_bytes, hip_stream, nullptr, 0, &sk);
}

extern "C" int jz_conv2d_bwd_weight_beside(const jz_conv_desc* desc, const void* x16, const void* dy16, void* dw16, void* ws,
                                           size_t ws_bytes, const jz_sumsq_sink* sink, void* hip_stream) {
  const int op = JZ_BWD_WEIGHT | JZ_BESIDE;
  if (!sink) return run(op, desc, dy16, x16, dw16, ws, ws_bytes, hip_stream);
  Plan pl;
  int rc = make_plan(op, desc, &pl);
  if (rc != JZ_OK) return rc;
  jz::SumsqSink sk;
  if ((rc = check_sink(sink, dw16, pl.bytesD, ws, ws_bytes < pl.ws_bytes ? ws_bytes : pl.ws_bytes, &sk)) != JZ_OK) return rc;
  return run(op, desc, dy16, x16, dw16, ws, ws_bytes, hip_stream, nullptr, 0, &sk);
}

// ---- weight gradients of several layers -----------------------------------------------------------------------------------------
namespace {

bool joins_set(const Plan& pl) { return pl.fast && !pl.packed && !pl.widen; }

struct SetPlan {
  Plan m[kWgradSet];  // the members, longest reductions first, all of one variant
  int index[kWgradSet];
  int n = 0;
  size_t part_bytes = 0;
};

// One variant for all members and the most k tiles a workgroup walks through (longer reductions are split), by the cost model
// of choose_tiling with all members' workgroups together.  `in`: the members' own plans.
void choose_set(const Plan* in, int n, size_t limit, SetPlan* sp) {
  // offered: what the model chooses for sets of ResNet-50's layers, 8 to 64 images of 64 to 224 pixels; sets of other networks are held
  // to these (a variant is a kernel of three forms of reading x)
  static const int offered[][5] = {{128, 128, 32, 8, 4}, {64, 64, 64, 4, 4}, {64, 64, 32, 4, 4}};
  static const int caps[] = {4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 512, 1 << 30};
  const CostGlobals& cg = kCost[2];
  auto p4 = [](double x) { return (x * x) * (x * x); };
  double best = 1e30;
  const Variant* bv = nullptr;
  int bcap = 1 << 30;
  for (const Variant& v : kVariants) {
    bool ok = false;
    for (const auto& o : offered) ok |= v.BM == o[0] && v.BN == o[1] && v.bk == o[2] && v.waves == o[3] && v.nst == o[4];
    if (!ok) continue;
    for (int cap : caps) {
      double lat = 0, thr = 0, longest = 0, mem = 0;
      size_t part_bytes = 0;
      for (int i = 0; i < n; ++i) {
        const GemmArgs& a = in[i].args;
        const int nkt = (a.Kred + v.bk - 1) / v.bk, s = (nkt - 1) / cap + 1, kps = (nkt + s - 1) / s, real = (nkt + kps - 1) / kps;
        const double blocks = (double)((a.M + v.BM - 1) / v.BM) * ((a.N + v.BN - 1) / v.BN) * real;
        const double loop = kps * (a.g.R * a.g.S > 1 ? cg.taps : 1.0), out = 1e-6 * (double)a.M * a.N;
        lat += blocks * (v.prologue[2] + v.lat[2] * loop);
        thr += blocks * (v.own[2] + v.thr[2] * loop);
        longest = std::max(longest, v.prologue[2] + v.lat[2] * loop);
        mem += 1e-6 * ((double)std::min<long long>(in[i].bytesA, 2ll * a.M * a.Kred) + (double)std::min<long long>(in[i].bytesB, 2ll * a.N * a.Kred)) + 2.0 * out;
        if (real > 1) part_bytes += up256((size_t)real * a.M * a.N * sizeof(float));
      }
      // whole bytes, as below: the workspace that the query reports has to hold what it was reported for
      if (part_bytes > limit) continue;
      const double part = 1e-6 * (double)part_bytes;
      const double t_lat = std::max(longest, lat / (kUnits * v.resident) + 0.5 * longest);
      double t = cg.fixed + std::sqrt(std::sqrt(p4(t_lat) + p4(thr / kUnits) + p4(cg.byte * (mem + part))));
      if (part > 0) t += cg.reduce_launch + cg.reduce_byte * part;
      if (t < best) { best = t; bv = &v; bcap = cap; }
    }
  }
  sp->n = n;
  for (int i = 0; i < n; ++i) sp->index[i] = i;
  std::stable_sort(sp->index, sp->index + n, [&](int x, int y) {
    auto kps = [&](int i) { const int nkt = (in[i].args.Kred + bv->bk - 1) / bv->bk, s = (nkt - 1) / bcap + 1; return (nkt + s - 1) / s; };
    return kps(x) > kps(y);
  });
  sp->part_bytes = 0;
  for (int i = 0; i < n; ++i) {
    Plan& m = sp->m[i];
    m = in[sp->index[i]];
    m.BM = bv->BM; m.BN = bv->BN; m.bk = bv->bk; m.waves = bv->waves; m.nst = bv->nst;
    set_tiles(&m, ((m.args.Kred + m.bk - 1) / m.bk - 1) / bcap + 1);
    m.part_offset = sp->part_bytes;
    if (m.args.splits > 1) sp->part_bytes += up256((size_t)m.args.splits * m.args.M * m.args.N * sizeof(float));
  }
}

int run_set(const SetPlan& sp, const void* const* x16, const void* const* dy16, void* const* dw16, void* ws, hipStream_t st) {
  WgradSet set;
  ReduceSet red{};
  int r = 0;
  set.first[0] = 0;
  for (int i = 0; i < kWgradSet; ++i) {
    if (i >= sp.n) {
      set.first[i + 1] = set.first[i];
      continue;
    }
    const Plan& m = sp.m[i];
    GemmArgs& a = set.g[i];
    a = m.args;
    a.A = static_cast<const unsigned short*>(dy16[sp.index[i]]);
    a.B = static_cast<const unsigned short*>(x16[sp.index[i]]);
    a.D16 = static_cast<unsigned short*>(dw16[sp.index[i]]);
    a.bytesA = (unsigned)m.bytesA;
    a.bytesB = (unsigned)m.bytesB;
    a.Dpart = reinterpret_cast<float*>(static_cast<char*>(ws) + m.part_offset);
    a.stats = nullptr;
    a.st_y = a.st_c = a.st_add = nullptr;
    a.st_mean = a.st_invstd = nullptr;
    set.first[i + 1] = set.first[i] + (unsigned)a.tiles_m * (unsigned)a.tiles_n * (unsigned)a.splits;
    if (a.splits > 1) {
      const long long MN = (long long)a.M * a.N;
      red.part[r] = a.Dpart;
      red.out[r] = a.D16;
      red.MN[r] = MN;
      red.splits[r] = a.splits;
      red.lg[r] = reduce_lanes(MN, a.splits);
      const long long per_block = 256 >> red.lg[r];
      red.first[r + 1] = red.first[r] + (unsigned)(((MN + 3) / 4 + per_block - 1) / per_block);
      ++r;
    }
  }
  int rc = launch_bwd_weight_set(sp.m[0], set, st);
  if (rc != JZ_OK || r == 0) return rc;
  for (int i = r; i < kWgradSet; ++i) red.first[i + 1] = red.first[i];
  hipLaunchKernelGGL(splitk_reduce_set, dim3(red.first[kWgradSet]), dim3(256), 0, st, red);
  return jz::launch_status();
}

}  // namespace

extern "C" int jz_conv2d_bwd_weight_set_workspace_bytes(int n, const jz_conv_desc* descs, size_t* bytes) {
  if (!descs || !bytes) return JZ_ERR_NULL;
  if (n < 1 || n > JZ_SET_MAX) return JZ_ERR_SHAPE;
  Plan set[JZ_SET_MAX];
  int k = 0;
  size_t need = 0;
  for (int i = 0; i < n; ++i) {
    const int rc = make_plan(JZ_BWD_WEIGHT, descs + i, &set[k]);
    if (rc != JZ_OK) return rc;
    if (joins_set(set[k])) ++k;
    else need = std::max(need, set[k].ws_bytes);
  }
  if (k > 0) {
    SetPlan sp;
    choose_set(set, k, kPartialSumLimit, &sp);
    need = std::max(need, sp.part_bytes);
  }
  *bytes = need;
  return JZ_OK;
}

extern "C" int jz_conv2d_bwd_weight_set(int n, const jz_conv_desc* descs, const void* const* x16, const void* const* dy16, void* const* dw16,
                                        void* ws, size_t ws_bytes, void* hip_stream) {
  if (!descs || !x16 || !dy16 || !dw16) return JZ_ERR_NULL;
  if (n < 1 || n > JZ_SET_MAX) return JZ_ERR_SHAPE;
  if (ws && !aligned16(ws)) return JZ_ERR_ALIGN;
  // Everything is settled before the first launch: a call that is refused has written nothing.
  Plan set[JZ_SET_MAX], own;
  const void *x[JZ_SET_MAX], *dy[JZ_SET_MAX];
  void* dw[JZ_SET_MAX];
  struct { size_t x, dy, dw; } bytes[JZ_SET_MAX];
  int alone[JZ_SET_MAX], k = 0, m = 0;
  size_t ws_used = 0;
  for (int i = 0; i < n; ++i) {
    int rc = make_plan(JZ_BWD_WEIGHT, descs + i, &own);
    if (rc != JZ_OK) return rc;
    if (!x16[i] || !dy16[i] || !dw16[i]) return JZ_ERR_NULL;
    if (!aligned16(x16[i]) || !aligned16(dy16[i]) || !aligned16(dw16[i])) return JZ_ERR_ALIGN;
    bytes[i] = {(size_t)own.bytesB, (size_t)own.bytesA, (size_t)own.bytesD};
    if (!joins_set(own)) {
      if ((rc = admit(JZ_BWD_WEIGHT, descs + i, dy16[i], x16[i], dw16[i], ws, ws_bytes, &own)) != JZ_OK) return rc;
      ws_used = std::max(ws_used, own.ws_bytes);
      alone[m++] = i;
      continue;
    }
    set[k] = own;
    x[k] = x16[i];
    dy[k] = dy16[i];
    dw[k++] = dw16[i];
  }
  SetPlan sp;
  if (k > 0) choose_set(set, k, std::min(kPartialSumLimit, ws ? ws_bytes : 0), &sp);
  ws_used = std::max(ws_used, sp.part_bytes);
  // a result overlaps no operand and no other result of the call, the workspace that it uses none of them
  for (int i = 0; i < n; ++i) {
    for (int j = 0; j < n; ++j)
      if (overlaps(dw16[i], bytes[i].dw, dy16[j], bytes[j].dy) || overlaps(dw16[i], bytes[i].dw, x16[j], bytes[j].x) ||
          (i < j && overlaps(dw16[i], bytes[i].dw, dw16[j], bytes[j].dw)))
        return JZ_ERR_ALIAS;
    if (ws_used > 0 && (overlaps(ws, ws_used, dy16[i], bytes[i].dy) || overlaps(ws, ws_used, x16[i], bytes[i].x) ||
                        overlaps(ws, ws_used, dw16[i], bytes[i].dw)))
      return JZ_ERR_ALIAS;
  }
  int rc = k > 0 ? run_set(sp, x, dy, dw, ws, static_cast<hipStream_t>(hip_stream)) : JZ_OK;
  for (int i = 0; i < m && rc == JZ_OK; ++i)
    rc = run(JZ_BWD_WEIGHT, descs + alone[i], dy16[alone[i]], x16[alone[i]], dw16[alone[i]], ws, ws_bytes, hip_stream);
  return rc;
}

// ---- backward-weight without a caller workspace ---------------------------------------------------------------
// For callers that cannot allocate device memory (code under HIP graph capture, tight serving loops): the same
// kernels, with the split-K partial sums (and the padded copy of a small-channel layer) in a fixed array that lives
// in the library's code object.  Every GPU the library runs on holds its own copy of the array at its own address for
// the life of the process; host code must not use the array's name as an address, so the address is looked up once
// per device and kept.
#define JZ_SCRATCH_LEN ((size_t)JZ_STATIC_SCRATCH_BYTES)
constexpr size_t kStaticScratchBytes = JZ_SCRATCH_LEN;
static __device__ __align__(256) unsigned char scratch[JZ_SCRATCH_LEN];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return JZ_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return JZ_ERR_LAUNCH;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return JZ_OK;
}

extern "C" int jz_conv2d_bwd_weight_static(const jz_conv_desc* desc, const void* x16, const void* dy16, void* dw16,
                                           void* hip_stream) {
  Plan pl;
  int rc = make_plan(JZ_BWD_WEIGHT, desc, &pl);
  if (rc != JZ_OK) return rc;
  void* ws = nullptr;
  if (pl.ws_bytes > 0 && (rc = static_scratch(&ws)) != JZ_OK) return rc;
  return run(JZ_BWD_WEIGHT, desc, dy16, x16, dw16, ws, ws ? kStaticScratchBytes : 0, hip_stream);  // A = dy, B = x
}

extern "C" int jz_gemm_fc_workspace_bytes(int mode, int batch, int in_features, int out_features, size_t* bytes) {
  jz_conv_desc d;
  int rc = fc_desc(mode, batch, in_features, out_features, &d);
  if (rc != JZ_OK) return rc;
  return jz_conv2d_workspace_bytes(mode, &d, bytes);
}

extern "C" int jz_gemm_fc(int mode, int batch, int in_features, int out_features, const void* a16, const void* b16,
                          void* out16, void* ws, size_t ws_bytes, void* hip_stream) {
  jz_conv_desc d;
  int rc = fc_desc(mode, batch, in_features, out_features, &d);
  if (rc != JZ_OK) return rc;
  // FWD: (x, w) ; BWD_DATA: (dy, w) ; BWD_WEIGHT: (dy, x) -- already the kernel's (A, B) order in every mode
  return run(mode, &d, a16, b16, out16, ws, ws_bytes, hip_stream);
}

extern "C" int jz_gemm_fc_bwd_weight_sumsq(int batch, int in_features, int out_features, const void* dy16, const void* x16,
                                           void* dw16, void* ws, size_t ws_bytes, const jz_sumsq_sink* sink, void* hip_stream) {
  jz_conv_desc d;
  int rc = fc_desc(JZ_BWD_WEIGHT, batch, in_features, out_features, &d);
  if (rc != JZ_OK) return rc;
  return jz_conv2d_bwd_weight_sumsq(&d, x16, dy16, dw16, ws, ws_bytes, sink, hip_stream);
}
