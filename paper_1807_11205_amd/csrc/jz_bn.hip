// Training-mode batch normalization with an optional ReLU, forward and backward, for gfx950 (Jia et al. 2018,
// Section 4.2: x^ = (x - mean_B) / sqrt(var_B + eps), y = gamma x^ + beta, statistics per channel over the mini-batch).
//
// Activations are FP16 [rows][C] (NHWC with rows = N*H*W), gamma / beta / the saved statistics FP32, sums FP32 per
// workgroup slab (FP64 for bn_whole's slabs, which are longer) and FP64 across slabs.  Every pass is bound by HBM, so each direction is three stream-ordered launches:
//
//   forward   bn_stats      a workgroup owns a slab of rows: per channel sum(x) and sum(x^2) of the slab (no atomics)
//             bn_fwd_final  per channel: the slabs' sums added in a fixed order in FP64 -> mean, 1/sqrt(var + eps), and the
//                           affine form y = a x + b (a = gamma invstd, b = beta - mean a) for the next pass
//             bn_apply      y = [max(., 0)](a x + b), 16 bytes per lane in and out
//   backward  bn_bwd_stats  per slab and channel: sum(g) and sum(g x^), g = dy masked by (y > 0) when the ReLU is on
//             bn_bwd_final  dbeta = sum g, dgamma = sum g x^ (FP16 copies for the optimizer's gradient buffer)
//             bn_bwd_apply  dx = gamma invstd (g - dbeta/M - x^ dgamma/M), evaluated as a g + P x + Q per channel
//
// Channel counts that are multiples of 64 go through one launch a direction instead, which reads every tensor once (jz_bn_whole.h,
// and launch_whole below for where it may run); the passes above are for the others, and with its slabs for what it may not take.
//
// Where there is room in the workspace the backward statistics leave the ReLU's mask as bits for the apply pass, which then
// reads x, dy and 1/16 of y's bytes instead of y (bn_bwd_apply_masked).  Where the partial sums are few the apply pass adds them
// up itself (*_merged).
//
// A lane always handles 8 consecutive channels (one 16-byte access); the C/8 lanes of a row sit side by side, so a
// wavefront reads whole rows contiguously.  Results are deterministic: the order of every sum depends only on
// (rows, C).
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <initializer_list>
#include <type_traits>
#include <utility>

#include "jz_internal.h"

namespace {

#include "jz_bn_math.h"

constexpr int BN_THREADS = 256;
constexpr int BN_BWD_ROWS = 4;         // rows of a lane whose loads are in flight together in the backward passes
constexpr int BN_MAX_C = 2048;       // C / 8 lanes of a row have to fit one workgroup
constexpr int BN_TARGET_SLABS = 512;   // two per compute unit
constexpr int BN_MERGE_SLABS = 64;     // most partial sums per channel that an apply pass adds up itself (ResNet-50 at batch 64: 64 is
                                       // even with none, 128 costs 1 %, 512 costs 4 %; small steps have fewer anyway)
// Forward tensors between these sizes: slabs shared by workgroups of 64 channels and up, so that at most 128 partial sums per
// channel are left, and an apply pass of about 512 workgroups of 512 threads that adds them up (12544 x 256: 14.4 us in three
// launches, 10.9 in two; x 1024: 21.6 and 18.2; 50176 x 512, 51 MB: 33.6 and 31-34).  Above (100 MB) the 128-byte pieces of rows cost
// the statistics what the launch costs (57.2 and 57-60 us); below, 2048 workgroups of 256 threads are better (8 x 64 x 64
// training step 1.62 and 1.65 ms).  Backward it does not pay: its statistics read three tensors (3136 x 512: 13.6 us in three
// launches, 16.1 in two).
constexpr int BN_MERGE_SLABS_WIDE = 128;
constexpr int64_t BN_WIDE_BYTES = 4 << 20, BN_FEW_SLABS_BYTES = 64 << 20;
constexpr int BN_FIN_C = 8;            // channels a finalize workgroup handles (32 contiguous bytes of every slab's sums);
constexpr int BN_FIN_LANES = BN_THREADS / BN_FIN_C;  // its 32 lanes per channel share the slabs

// bn_whole (jz_bn_whole.h)
constexpr int BW_THREADS = 512;                  // one workgroup per compute unit: 2 wavefronts per SIMD, 256 registers a lane
constexpr int BW_CH = 64;                        // channels of a workgroup: one 128-byte line of every row
constexpr int BW_ROWS = BW_THREADS / (BW_CH / 8);  // rows one pass of a workgroup covers

size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

struct BnPlan {
  int64_t rows = 0;
  int C = 0, cpr = 0;        // 16-byte chunks per row
  int csplit = 1;            // workgroups that share a slab of rows, each with cpr / csplit of the chunks (wide, short tensors)
  int threads = BN_THREADS;  // of the statistics pass
  int rpp = 0;               // rows one pass of a workgroup covers (threads / (cpr / csplit); lanes beyond that idle)
  int64_t rows_per_slab = 0; // a multiple of rpp
  int slabs = 0;
  size_t off_part = 0, off_coef = 0, total = 0;  // workspace: [slabs][2][C] partial sums, [4][C] float coefficients (bn_whole: its flags, a word a workgroup)
  int mask_iters = 0;        // words of it a lane of the statistics pass has
  size_t mask_bytes = 0;     // behind them, if there is room: one bit per element, the backward pass's ReLU mask
};

int make_bn_plan(int64_t rows, int channels, bool forward, BnPlan* p) {
  if (rows <= 0 || channels <= 0) return JZ_ERR_SHAPE;
  if (channels % 8 != 0 || channels > BN_MAX_C) return JZ_ERR_UNSUPPORTED;
  if (rows * (int64_t)channels >= (int64_t(1) << 40)) return JZ_ERR_UNSUPPORTED;
  p->rows = rows;
  p->C = channels;
  p->cpr = channels / 8;
  // at most BN_TARGET_SLABS slabs, and at least 16 passes of the workgroup and 64 rows per slab: small tensors get fewer
  // slabs, so that the partial sums stay small beside the tensor.  A wide tensor with few rows would then leave most of
  // the chip idle (2048 channels x 3136 rows: 49 slabs), so its slabs are shared by csplit workgroups that take a range
  // of at least 32 chunks (512 contiguous bytes of a row) each: more workgroups, the same number of partial sums.
  const bool merge = forward && rows * channels * 2 <= BN_FEW_SLABS_BYTES && rows * channels * 2 >= BN_WIDE_BYTES;
  for (int cs = 1;; cs *= 2) {
    const int cpr_l = p->cpr / cs;
    p->csplit = cs;
    p->rpp = BN_THREADS / cpr_l;
    const int target = merge ? BN_TARGET_SLABS / cs : BN_TARGET_SLABS;
    // fewer passes per workgroup (16, 8, 4) until at least 256 workgroups exist
    for (int min_passes = 16; min_passes >= (merge ? 2 : 4); min_passes /= 2) {
      int64_t per = (rows + target - 1) / target;
      if (per < min_passes * (int64_t)p->rpp) per = min_passes * (int64_t)p->rpp;
      if (per < 32) per = 32;
      per = (per + p->rpp - 1) / p->rpp * p->rpp;
      p->rows_per_slab = per;
      p->slabs = (int)((rows + per - 1) / per);
      if ((int64_t)p->slabs * cs >= 256) break;
    }
    const bool full = (int64_t)p->slabs * cs >= 256;
    if (merge) {
      if ((full && p->slabs <= BN_MERGE_SLABS_WIDE) || cpr_l % 2 != 0 || cpr_l / 2 < 8) break;
    } else if (full || cs == 8 || cpr_l % 2 != 0 || cpr_l / 2 < 32) {
      break;
    }
  }
  p->off_part = 0;
  p->off_coef = up256((size_t)p->slabs * 2 * channels * sizeof(float));
  p->total = p->off_coef + up256((size_t)4 * channels * sizeof(float));
  p->mask_iters = (int)((p->rows_per_slab + BN_BWD_ROWS * (int64_t)p->rpp - 1) / (BN_BWD_ROWS * (int64_t)p->rpp));
  if (p->slabs > BN_MERGE_SLABS)  // an apply pass that finishes the statistics itself reads y
    p->mask_bytes = (size_t)p->slabs * p->csplit * p->mask_iters * BN_THREADS * 4;
  return JZ_OK;
}

__device__ __forceinline__ void unpack8(const uint4& v, float (&f)[8]) {
  const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    _Float16 lo, hi;
    unsigned short a = (unsigned short)(w[i] & 0xffffu), b = (unsigned short)(w[i] >> 16);
    __builtin_memcpy(&lo, &a, 2);
    __builtin_memcpy(&hi, &b, 2);
    f[2 * i] = (float)lo;
    f[2 * i + 1] = (float)hi;
  }
}

__device__ __forceinline__ void load8(const float* p, float (&f)[8]) {
  const float4 t0 = reinterpret_cast<const float4*>(p)[0], t1 = reinterpret_cast<const float4*>(p)[1];
  f[0] = t0.x; f[1] = t0.y; f[2] = t0.z; f[3] = t0.w; f[4] = t1.x; f[5] = t1.y; f[6] = t1.z; f[7] = t1.w;
}

__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  unsigned w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    _Float16 lo = (_Float16)f[2 * i], hi = (_Float16)f[2 * i + 1];  // round to nearest even
    unsigned short a, b;
    __builtin_memcpy(&a, &lo, 2);
    __builtin_memcpy(&b, &hi, 2);
    w[i] = (unsigned)a | ((unsigned)b << 16);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// A result of the passes over large tensors goes out with the non-temporal hint: written back while the pass that makes it
// reads out of the last-level cache and memory is idle, instead of during the next pass, which does read from memory and
// slowed down to 3.3-4.3 TB/s beside the write-back.  ResNet-50's 53 layers forward and backward, batch 64: 3.52 -> 3.17 ms
// (statistics passes 1.66 -> 1.35 ms, the apply passes the same); the training step, where a convolution reads the result
// next, is neither faster nor slower.
__device__ __forceinline__ void store_streaming(uint4* p, const uint4& v) {
  typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
  const u32x4_t t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t*>(p));
}

// Sums over a slab of rows, for the 8 channels of each lane: s0 and s1 are whatever the mode produces per element.
// The rpp lanes that share a channel chunk (one per row of a pass) are then added through LDS, and the
// slab's 2 x C sums are stored.  ST_SUM: (x, x^2).  ST_GRAD: (g, g x^) with g = dy.  ST_RELU: ... with g = dy where y > 0, else 0.
// ST_MASK: the same, and the bits y > 0 are left for the apply pass.  ST_END: the end of a
// residual block: g = RNE16(dy [+ dy2]) where y > 0, else 0, is formed here, written to g_out for the other consumers of
// that gradient, and summed (the sums see the rounded g, as a pass over g_out would).
enum { ST_SUM, ST_GRAD, ST_RELU, ST_MASK, ST_END };
struct BnStatsArgs {
  const uint4 *x, *y, *dy, *dy2;
  uint4* g_out;
  unsigned* mask;
  const float *mean, *invstd;
  void* part;  // BnSum
  int64_t rows, rows_per_slab;
  int C, cpr, rpp, csplit, mask_iters;
};
// What a slab's sums are stored as.  bn_whole's slabs are up to 16 times as long as the others: in FP32 they would be less exact
// (mean over 12544 x 1024, deviations from FP64 in standard deviations: 3.2e-10, in FP64 2.4e-10, FP32 and the other slabs 2.5e-10).
template <bool WHOLE>
using BnSum = std::conditional_t<WHOLE, double, float>;
template <int MODE, int T>
__global__ __launch_bounds__(T) void bn_stats(BnStatsArgs a) {
  __shared__ __align__(16) float red[2][T][8];
  constexpr bool GRAD = MODE != ST_SUM, NEEDS_Y = MODE == ST_RELU || MODE == ST_MASK || MODE == ST_END;
  constexpr bool WHOLE_PLAN = T != BN_THREADS;  // bn_whole's, for calls that may not take it: what is known is constant
  const int tid = threadIdx.x, cpr = a.cpr, rpp = WHOLE_PLAN ? BW_ROWS : a.rpp, C = a.C;
  const int cpr_l = WHOLE_PLAN ? BW_CH / 8 : cpr / a.csplit;  // chunks of a row this workgroup handles: [cfirst, cfirst + cpr_l)
  const int slab = blockIdx.x / a.csplit, cfirst = (blockIdx.x % a.csplit) * cpr_l;
  const int chunk_l = tid % cpr_l, rsub = tid / cpr_l;
  const int chunk = cfirst + chunk_l;
  const int64_t r0 = (int64_t)slab * a.rows_per_slab;
  const int64_t r1 = r0 + a.rows_per_slab < a.rows ? r0 + a.rows_per_slab : a.rows;
  float s0[8], s1[8], mu[8], is[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    s0[e] = 0.f; s1[e] = 0.f; mu[e] = 0.f; is[e] = 0.f;
  }
  if (GRAD && rsub < rpp) {
    load8(a.mean + chunk * 8, mu);
    load8(a.invstd + chunk * 8, is);
  }
  unsigned held = 0, *word = nullptr;  // ST_MASK: the bits of the rows before, and where they go
  unsigned* next_word = MODE == ST_MASK ? a.mask + (size_t)blockIdx.x * a.mask_iters * T + tid : nullptr;
  // U rows of a lane are requested together (the loop is bound by memory latency otherwise); rows beyond the slab add nothing
  // (x = 0 and g = 0 contribute zero to every sum)
  constexpr int U = MODE == ST_SUM ? 8 : BN_BWD_ROWS;
  auto group = [&](int64_t r, auto whole_tag) {
    constexpr bool WHOLE = decltype(whole_tag)::value;
    uint4 qx[U], qd[U], qy[U], qe[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t ru = r + (int64_t)u * rpp;
      const size_t idx = (size_t)ru * cpr + chunk;
      if constexpr (!WHOLE) qx[u] = qd[u] = qy[u] = qe[u] = make_uint4(0u, 0u, 0u, 0u);
      if (WHOLE || ru < r1) {
        qx[u] = a.x[idx];
        if constexpr (GRAD) qd[u] = a.dy[idx];
        if constexpr (NEEDS_Y) qy[u] = a.y[idx];
        if constexpr (MODE == ST_END)
          if (a.dy2) qe[u] = a.dy2[idx];
      }
    }
    if constexpr (MODE == ST_MASK) {
      // the word of the group before goes out behind this group's loads: a wait for loads behind it would wait for the store too
      if (word) __builtin_nontemporal_store(held, word);
      word = next_word;
      next_word += T;
      held = 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xv[8];
      unpack8(qx[u], xv);
      if constexpr (MODE == ST_SUM) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          s0[e] += xv[e];
          s1[e] = fmaf(xv[e], xv[e], s1[e]);
        }
        continue;
      }
      float gv[8], yv[8];
      unpack8(qd[u], gv);
      if constexpr (NEEDS_Y) unpack8(qy[u], yv);
      if constexpr (MODE == ST_END) {  // form g and store it
        if (a.dy2) {
          float ev[8];
          unpack8(qe[u], ev);
#pragma unroll
          for (int e = 0; e < 8; ++e) gv[e] += ev[e];  // exact in FP32; pack8 rounds once
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) gv[e] = yv[e] > 0.f ? gv[e] : 0.f;
        const uint4 g = pack8(gv);
        unpack8(g, gv);
        const int64_t ru = r + (int64_t)u * rpp;
        if (WHOLE || ru < r1) a.g_out[(size_t)ru * cpr + chunk] = g;
      } else if constexpr (NEEDS_Y) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool on = yv[e] > 0.f;
          gv[e] = on ? gv[e] : 0.f;
          if constexpr (MODE == ST_MASK) held |= on ? 1u << (8 * u + e) : 0u;
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        s0[e] += gv[e];
        s1[e] = fmaf(gv[e], (xv[e] - mu[e]) * is[e], s1[e]);
      }
    }
  };
  if (rsub < rpp) {
    int64_t r = r0 + rsub;
    for (; r + (int64_t)(U - 1) * rpp < r1; r += (int64_t)U * rpp) group(r, std::true_type{});
    if (r < r1) group(r, std::false_type{});
  }
  if (MODE == ST_MASK && word) __builtin_nontemporal_store(held, word);
  // the rows' sums are added by all threads: each takes a channel's sum, of a part of the rows where there are fewer sums than
  // threads (the lanes of one row adding up the others': 8.7 instead of 7.5 us for 200704 x 64).  The forward sums in FP64: where
  // rows are shared by workgroups a slab has four times as many, and FP32 would make the variance of channels far from zero less exact
  // than with small slabs (12544 x 256, mean 10 std: relative error 5.3e-7, in FP64 3.2e-7; FP32 and slabs of 32 rows: 3.2e-7).
  // The gradients' too where bn_whole's slabs are summed.
  using Part = BnSum<WHOLE_PLAN>;
  using Acc = std::conditional_t<GRAD, Part, double>;
  const int ch = 8 * cpr_l, sums = 2 * ch;  // red[0] and red[1] are [rows of a pass][ch]
  const float* const r0s = &red[0][0][0];
  const float* const r1s = &red[1][0][0];
#pragma unroll
  for (int e = 0; e < 8; e += 4) {
    *reinterpret_cast<float4*>(&red[0][tid][e]) = make_float4(s0[e], s0[e + 1], s0[e + 2], s0[e + 3]);
    *reinterpret_cast<float4*>(&red[1][tid][e]) = make_float4(s1[e], s1[e + 1], s1[e + 2], s1[e + 3]);
  }
  __syncthreads();
  Part* const out = static_cast<Part*>(a.part) + (size_t)slab * 2 * C + cfirst * 8;
  if (sums >= T) {
    for (int i = tid; i < sums; i += T) {
      const float* p = i < ch ? r0s + i : r1s + (i - ch);
      Acc t = 0;
      for (int j = 0; j < rpp; ++j) t += p[j * ch];
      out[i < ch ? i : C + i - ch] = (Part)t;
    }
    return;
  }
  const int parts = T / sums, i = tid % sums, first = tid / sums;
  Acc t = 0;
  if (first < parts) {
    const float* p = i < ch ? r0s + i : r1s + (i - ch);
    for (int j = first; j < rpp; j += parts) t += p[j * ch];
  }
  __syncthreads();
  Acc* const part_sums = reinterpret_cast<Acc*>(&red[0][0][0]);
  if (first < parts) part_sums[first * sums + i] = t;
  __syncthreads();
  if (tid < sums) {
    t = 0;
    for (int k = 0; k < parts; ++k) t += part_sums[k * sums + tid];
    out[tid < ch ? tid : C + tid - ch] = (Part)t;
  }
}

// lanes of a channel that have a slab to add
__device__ __forceinline__ int bn_lanes(int slabs) { return slabs < BN_FIN_LANES ? slabs : BN_FIN_LANES; }

// The two sums of channel c over all slabs, FP64: lane js of the channel's 32 lanes adds slabs js, js + 32, ... in that order,
// then lane 0 adds the 32 lane sums in lane order (deterministic).  Returns true on the lane that holds the totals.
template <class P>
__device__ __forceinline__ bool bn_slab_totals(const P* __restrict__ part, int slabs, int C, int c, double& s, double& q) {
  __shared__ double red[2][BN_THREADS];
  constexpr int LANES = BN_FIN_LANES;
  const int js = threadIdx.x / BN_FIN_C;
  s = 0.0;
  q = 0.0;
  if (c < C)
    for (int k = js; k < slabs; k += 8 * LANES) {  // eight slabs' sums requested together, added in slab order
      P a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {  // all sixteen loads first (clamped index), the selection afterwards
        const int ku = k + u * LANES;
        const int kc = ku < slabs ? ku : k;
        a[u] = part[((size_t)kc * 2) * C + c];
        b[u] = part[((size_t)kc * 2 + 1) * C + c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k + u * LANES >= slabs) {
          a[u] = 0;
          b[u] = 0;
        }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s += (double)a[u];
        q += (double)b[u];
      }
    }
  red[0][threadIdx.x] = s;
  red[1][threadIdx.x] = q;
  __syncthreads();
  if (js != 0 || c >= C) return false;
  for (int l = 1; l < LANES; ++l) {
    s += red[0][l * BN_FIN_C + threadIdx.x];
    q += red[1][l * BN_FIN_C + threadIdx.x];
  }
  return true;
}

template <class P>
__global__ __launch_bounds__(BN_THREADS) void bn_fwd_final(const P* __restrict__ part, int slabs, int C, double inv_rows,
                                                          float eps, const float* __restrict__ gamma,
                                                          const float* __restrict__ beta, float* __restrict__ save_mean,
                                                          float* __restrict__ save_invstd, float* __restrict__ coef) {
  const int c = blockIdx.x * BN_FIN_C + threadIdx.x % BN_FIN_C;
  double s, q;
  if (!bn_slab_totals(part, slabs, C, c, s, q)) return;
  bn_fwd_coef(s, q, inv_rows, eps, gamma[c], beta[c], save_mean + c, save_invstd + c, coef + c, C);
}

// RES: a residual tensor is added in front of the ReLU (the end of a bottleneck block)
template <int RES>
__global__ __launch_bounds__(BN_THREADS) void bn_apply(const uint4* __restrict__ x, const uint4* __restrict__ res,
                                                      uint4* __restrict__ y, const float* __restrict__ coef, int64_t n_chunks, int C,
                                                      int cpr, int relu) {
  const int64_t stride = (int64_t)gridDim.x * BN_THREADS;
  for (int64_t i = (int64_t)blockIdx.x * BN_THREADS + threadIdx.x; i < n_chunks; i += stride) {
    const int chunk = (int)(i % cpr);
    float a[8], b[8], v[8];
    const float4* ca = reinterpret_cast<const float4*>(coef + chunk * 8);
    const float4* cb = reinterpret_cast<const float4*>(coef + C + chunk * 8);
    float4 t0 = ca[0], t1 = ca[1], u0 = cb[0], u1 = cb[1];
    a[0] = t0.x; a[1] = t0.y; a[2] = t0.z; a[3] = t0.w; a[4] = t1.x; a[5] = t1.y; a[6] = t1.z; a[7] = t1.w;
    b[0] = u0.x; b[1] = u0.y; b[2] = u0.z; b[3] = u0.w; b[4] = u1.x; b[5] = u1.y; b[6] = u1.z; b[7] = u1.w;
    unpack8(x[i], v);
    float rv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (RES) unpack8(res[i], rv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float z = fmaf(v[e], a[e], b[e]);
      if (RES) z += rv[e];
      v[e] = (relu && !(z > 0.f)) ? 0.f : z;
    }
    store_streaming(y + i, pack8(v));
  }
}

template <class P>
__global__ __launch_bounds__(BN_THREADS) void bn_bwd_final(const P* __restrict__ part, int slabs, int C, double inv_rows,
                                                          const float* __restrict__ gamma, const float* __restrict__ mean,
                                                          const float* __restrict__ invstd, unsigned short* __restrict__ dgamma16,
                                                          unsigned short* __restrict__ dbeta16, float* __restrict__ coef) {
  const int c = blockIdx.x * BN_FIN_C + threadIdx.x % BN_FIN_C;
  double sb, sg;
  if (!bn_slab_totals(part, slabs, C, c, sb, sg)) return;
  bn_bwd_coef(sb, sg, inv_rows, gamma[c], mean[c], invstd[c], dgamma16 + c, dbeta16 + c, coef + c, C);
}

__global__ __launch_bounds__(BN_THREADS) void bn_bwd_apply(const uint4* __restrict__ x, const uint4* __restrict__ y,
                                                          const uint4* __restrict__ dy, uint4* __restrict__ dx,
                                                          const float* __restrict__ coef, int64_t n_chunks, int C, int cpr, int relu) {
  const int64_t stride = (int64_t)gridDim.x * BN_THREADS;
  for (int64_t i = (int64_t)blockIdx.x * BN_THREADS + threadIdx.x; i < n_chunks; i += stride) {
    const int c0 = (int)(i % cpr) * 8;
    const uint4 qx = x[i], qd = dy[i];
    const uint4 qy = relu ? y[i] : make_uint4(0u, 0u, 0u, 0u);
    float a[8], pc[8], qc[8], xv[8], gv[8], out[8];
    load8(coef + c0, a);
    load8(coef + C + c0, pc);
    load8(coef + 2 * C + c0, qc);
    unpack8(qx, xv);
    unpack8(qd, gv);
    if (relu) {
      float yv[8];
      unpack8(qy, yv);
#pragma unroll
      for (int e = 0; e < 8; ++e) gv[e] = yv[e] > 0.f ? gv[e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = bn_dx(a[e], gv[e], pc[e], xv[e], qc[e]);
    store_streaming(dx + i, pack8(out));
  }
}

// The same with the ReLU's mask out of the words that the statistics pass left, by the workgroups, lanes and rows of that pass:
// a quarter of the reads less.  802816 x 64 (103 MB a tensor): statistics 56 -> 63 us for writing the words, apply pass 63 -> 52;
// ResNet-50's 53 layers at batch 64: 920 -> 970 and 888 -> 710 us.  A byte per 16 bytes of y at its place in the tensor, which any
// mapping could read, cost the statistics 145 us; the words with the non-temporal hint cost the apply passes 50.
template <int T>
__global__ __launch_bounds__(T) void bn_bwd_apply_masked(const uint4* __restrict__ x, const uint4* __restrict__ dy, uint4* __restrict__ dx,
                                                                 const float* __restrict__ coef, const unsigned* __restrict__ mask,
                                                                 int64_t rows, int C, int cpr, int rpp, int64_t rows_per_slab, int csplit) {
  constexpr int U = BN_BWD_ROWS;
  const int cpr_l = cpr / csplit, slab = blockIdx.x / csplit, rsub = threadIdx.x / cpr_l;
  const int chunk = (blockIdx.x % csplit) * cpr_l + threadIdx.x % cpr_l;
  const int64_t r0 = (int64_t)slab * rows_per_slab, r1 = r0 + rows_per_slab < rows ? r0 + rows_per_slab : rows;
  if (rsub >= rpp) return;
  mask += (size_t)blockIdx.x * ((rows_per_slab + U * rpp - 1) / (U * rpp)) * T + threadIdx.x;
  float a[8], pc[8], qc[8];
  load8(coef + chunk * 8, a);
  load8(coef + C + chunk * 8, pc);
  load8(coef + 2 * C + chunk * 8, qc);
  uint4 qx[U], qd[U];
  unsigned w = 0;
  auto fetch = [&](int64_t r) {
    if (r < r1) {
      w = *mask;
      mask += T;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t ru = r + (int64_t)u * rpp;
      if (ru < r1) {
        qx[u] = x[(size_t)ru * cpr + chunk];
        qd[u] = dy[(size_t)ru * cpr + chunk];
      }
    }
  };
  fetch(r0 + rsub);
  for (int64_t r = r0 + rsub; r < r1; r += (int64_t)U * rpp) {
    uint4 o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xv[8], gv[8], out[8];
      unpack8(qx[u], xv);
      unpack8(qd[u], gv);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float g = (w >> (8 * u + e)) & 1u ? gv[e] : 0.f;
        out[e] = bn_dx(a[e], g, pc[e], xv[e], qc[e]);
      }
      o[u] = pack8(out);
    }
    fetch(r + (int64_t)U * rpp);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t ru = r + (int64_t)u * rpp;
      if (ru < r1) store_streaming(dx + (size_t)ru * cpr + chunk, o[u]);
    }
  }
}

// ---- apply passes that finish the statistics themselves ----------------------------------------------------------------------
// With few partial sums per channel (BN_MERGE_SLABS) the launch between the statistics and the apply pass does nothing but cost
// its 4-5 us: here a workgroup owns 64 channels and a range of rows, adds up the partial sums of its channels (a few tens of KB
// out of L2, while its first rows are on their way) and goes on.  The first workgroup of a channel range also writes what the
// finalize kernel would.
constexpr int BM_CH = 64;    // channels of a workgroup: one 128-byte line of every row
constexpr int BM_ROWS = BN_THREADS / (BM_CH / 8);  // rows one pass of a workgroup covers
constexpr int BM_U = 4;      // passes whose loads are in flight together

// the two sums of channel first + tid (tid < 64), FP64: T / 64 lanes per channel take every (T / 64)-th slab, then added in lane
// order
template <int T>
__device__ __forceinline__ bool bn_merged_totals(const float* __restrict__ part, int slabs, int C, int first, double& s, double& q) {
  constexpr int LANES = T / BM_CH;
  __shared__ double red[2][T];
  const int c = first + (threadIdx.x & (BM_CH - 1)), j = threadIdx.x / BM_CH;
  s = q = 0.0;
  if (c < C)
    for (int k = j; k < slabs; k += 8 * LANES) {  // eight slabs' sums requested together, added in slab order
      float a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int ku = k + LANES * u < slabs ? k + LANES * u : k;
        a[u] = part[((size_t)ku * 2) * C + c];
        b[u] = part[((size_t)ku * 2 + 1) * C + c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k + LANES * u < slabs) {
          s += (double)a[u];
          q += (double)b[u];
        }
    }
  red[0][threadIdx.x] = s;
  red[1][threadIdx.x] = q;
  __syncthreads();
  if (j != 0 || c >= C) return false;
  for (int l = 1; l < LANES; ++l) {
    s += red[0][l * BM_CH + threadIdx.x];
    q += red[1][l * BM_CH + threadIdx.x];
  }
  return true;
}

// The same in bn_slab_totals' order, which is bn_whole's: for tensors that it takes where it may run.  A thread stands for 32 / (T / 64) of
// the channel's 32 lanes.  (For all tensors it made the 8 x 64 x 64 training step 1.6 % slower.)
template <int T>
__device__ __forceinline__ bool bn_merged_totals_32(const double* __restrict__ part, int slabs, int C, int first, double& s, double& q) {
  constexpr int THREADS = T / BM_CH, OWN = BN_FIN_LANES / THREADS;
  __shared__ double red[2][BN_FIN_LANES][BM_CH];
  const int cl = threadIdx.x & (BM_CH - 1), c = first + cl, j = __builtin_amdgcn_readfirstlane(threadIdx.x / BM_CH);
  if (slabs <= BN_FIN_LANES) {  // a lane has one slab at most: one thread adds them, without the detour through LDS
    if (j != 0 || c >= C) return false;
    constexpr int U = 16;
    s = q = 0.0;
    for (int k = 0; k < slabs; k += U) {
      double a[U], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        a[u] = b[u] = 0.0;
        if (k + u < slabs) {
          a[u] = part[((size_t)(k + u) * 2) * C + c];
          b[u] = part[((size_t)(k + u) * 2 + 1) * C + c];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        s += a[u];
        q += b[u];
      }
    }
    return true;
  }
  double ts[OWN], tq[OWN];
#pragma unroll
  for (int o = 0; o < OWN; ++o) ts[o] = tq[o] = 0.0;
  if (c < C)
    for (int k = j; k < slabs; k += BN_FIN_LANES) {  // OWN slabs' sums requested together
      double a[OWN], b[OWN];
#pragma unroll
      for (int o = 0; o < OWN; ++o) {
        a[o] = b[o] = 0.0;
        if (k + THREADS * o < slabs) {
          a[o] = part[((size_t)(k + THREADS * o) * 2) * C + c];
          b[o] = part[((size_t)(k + THREADS * o) * 2 + 1) * C + c];
        }
      }
#pragma unroll
      for (int o = 0; o < OWN; ++o) {
        ts[o] += a[o];
        tq[o] += b[o];
      }
    }
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    red[0][j + THREADS * o][cl] = ts[o];
    red[1][j + THREADS * o][cl] = tq[o];
  }
  __syncthreads();
  if (j < 2) {  // the first 64 threads add the lanes' first sums, the next 64 their second ones
    double t = 0.0;
    for (int l0 = 0; l0 < bn_lanes(slabs); l0 += 8) {  // eight read together; lanes beyond the slabs hold zeros
      double v[8];
#pragma unroll
      for (int l = 0; l < 8; ++l) v[l] = red[j][l0 + l][cl];
#pragma unroll
      for (int l = 0; l < 8; ++l) t += v[l];
    }
    red[j][0][cl] = t;
  }
  __syncthreads();
  if (j != 0 || c >= C) return false;
  s = red[0][0][cl];
  q = red[1][0][cl];
  return true;
}

template <int RES, int T, bool WHOLE = false>
__global__ __launch_bounds__(T) void bn_apply_merged(const uint4* __restrict__ x, const uint4* __restrict__ res, uint4* __restrict__ y,
                                                             int64_t rows, int rows_per_wg, int C, const BnSum<WHOLE>* __restrict__ part, int slabs,
                                                             double inv_rows, float eps, int relu, const float* __restrict__ gamma,
                                                             const float* __restrict__ beta, float* __restrict__ save_mean,
                                                             float* __restrict__ save_invstd) {
  constexpr int ROWS = T / (BM_CH / 8);  // rows one pass covers
  __shared__ __align__(16) float coef[2][BM_CH];
  const int cpr = C / 8, first = blockIdx.x * BM_CH;
  const int chunk = blockIdx.x * (BM_CH / 8) + (threadIdx.x & 7), rsub = threadIdx.x / 8;
  const bool live = chunk < cpr;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_wg, r1 = r0 + rows_per_wg < rows ? r0 + rows_per_wg : rows;
  uint4 q[BM_U], e[BM_U];
  auto fetch = [&](int64_t r) {
#pragma unroll
    for (int u = 0; u < BM_U; ++u) {
      const int64_t ru = r + u * ROWS;
      if (live && ru < r1) {
        q[u] = x[(size_t)ru * cpr + chunk];
        if (RES) e[u] = res[(size_t)ru * cpr + chunk];
      }
    }
  };
  fetch(r0 + rsub);
  double s, sq;
  bool has;
  if constexpr (WHOLE) has = bn_merged_totals_32<T>(part, slabs, C, first, s, sq);
  else has = bn_merged_totals<T>(part, slabs, C, first, s, sq);
  if (has) {
    const int c = first + threadIdx.x;
    const bool writer = blockIdx.y == 0;
    bn_fwd_coef(s, sq, inv_rows, eps, gamma[c], beta[c], writer ? save_mean + c : nullptr, writer ? save_invstd + c : nullptr,
                &coef[0][threadIdx.x], BM_CH);
  }
  __syncthreads();
  float a[8], b[8];
  load8(&coef[0][(threadIdx.x & 7) * 8], a);
  load8(&coef[1][(threadIdx.x & 7) * 8], b);
  for (int64_t r = r0 + rsub; r < r1; r += BM_U * ROWS) {
    uint4 o[BM_U];
#pragma unroll
    for (int u = 0; u < BM_U; ++u) {
      float v[8], rv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      unpack8(q[u], v);
      if (RES) unpack8(e[u], rv);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        float z = fmaf(v[k], a[k], b[k]);
        if (RES) z += rv[k];
        v[k] = (relu && !(z > 0.f)) ? 0.f : z;
      }
      o[u] = pack8(v);
    }
    fetch(r + BM_U * ROWS);
#pragma unroll
    for (int u = 0; u < BM_U; ++u) {
      const int64_t ru = r + u * ROWS;
      if (!live || ru >= r1) continue;
      if (T == BN_THREADS) y[(size_t)ru * cpr + chunk] = o[u];
      else store_streaming(y + (size_t)ru * cpr + chunk, o[u]);
    }
  }
}

template <bool WHOLE>
__global__ __launch_bounds__(BN_THREADS) void bn_bwd_apply_merged(const uint4* __restrict__ x, const uint4* __restrict__ y,
                                                                 const uint4* __restrict__ dy, uint4* __restrict__ dx, int64_t rows,
                                                                 int rows_per_wg, int C, const BnSum<WHOLE>* __restrict__ part, int slabs,
                                                                 double inv_rows, int relu, const float* __restrict__ gamma,
                                                                 const float* __restrict__ mean, const float* __restrict__ invstd,
                                                                 unsigned short* __restrict__ dgamma16, unsigned short* __restrict__ dbeta16) {
  __shared__ __align__(16) float coef[3][BM_CH];
  const int cpr = C / 8, first = blockIdx.x * BM_CH;
  const int chunk = blockIdx.x * (BM_CH / 8) + (threadIdx.x & 7), rsub = threadIdx.x / 8;
  const bool live = chunk < cpr;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_wg, r1 = r0 + rows_per_wg < rows ? r0 + rows_per_wg : rows;
  uint4 qx[BM_U], qd[BM_U], qy[BM_U];
  auto fetch = [&](int64_t r) {
#pragma unroll
    for (int u = 0; u < BM_U; ++u) {
      const int64_t ru = r + u * BM_ROWS;
      if (live && ru < r1) {
        const size_t i = (size_t)ru * cpr + chunk;
        qx[u] = x[i];
        qd[u] = dy[i];
        if (relu) qy[u] = y[i];
      }
    }
  };
  fetch(r0 + rsub);
  double sb, sg;
  bool has;
  if constexpr (WHOLE) has = bn_merged_totals_32<BN_THREADS>(part, slabs, C, first, sb, sg);
  else has = bn_merged_totals<BN_THREADS>(part, slabs, C, first, sb, sg);
  if (has) {
    const int c = first + threadIdx.x;
    const bool writer = blockIdx.y == 0;
    bn_bwd_coef(sb, sg, inv_rows, gamma[c], mean[c], invstd[c], writer ? dgamma16 + c : nullptr, writer ? dbeta16 + c : nullptr,
                &coef[0][threadIdx.x], BM_CH);
  }
  __syncthreads();
  float a[8], pc[8], qc[8];
  load8(&coef[0][(threadIdx.x & 7) * 8], a);
  load8(&coef[1][(threadIdx.x & 7) * 8], pc);
  load8(&coef[2][(threadIdx.x & 7) * 8], qc);
  for (int64_t r = r0 + rsub; r < r1; r += BM_U * BM_ROWS) {
    uint4 o[BM_U];
#pragma unroll
    for (int u = 0; u < BM_U; ++u) {
      float xv[8], gv[8], out[8];
      unpack8(qx[u], xv);
      unpack8(qd[u], gv);
      if (relu) {
        float yv[8];
        unpack8(qy[u], yv);
#pragma unroll
        for (int k = 0; k < 8; ++k) gv[k] = yv[k] > 0.f ? gv[k] : 0.f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) out[k] = bn_dx(a[k], gv[k], pc[k], xv[k], qc[k]);
      o[u] = pack8(out);
    }
    fetch(r + BM_U * BM_ROWS);
#pragma unroll
    for (int u = 0; u < BM_U; ++u) {
      const int64_t ru = r + u * BM_ROWS;
      if (live && ru < r1) dx[(size_t)ru * cpr + chunk] = o[u];
    }
  }
}

#include "jz_bn_whole.h"

// One launch for all (bn_whole): channel counts that are multiples of 64.  The plan is the statistics passes' with slabs for one workgroup
// per compute unit, so that the launches apart leave the same bits.
// Backward up to 128 passes of 64 rows a workgroup: beyond, most rows are read twice either way and the launches apart have more loads in
// flight (401408 x 256, 98 passes: 252 us apart, 217 in one; 200704 x 1024, 196 passes: 497 and 529).  Forward it is never slower (802816 x 256: 226
// and 218).
constexpr int64_t BW_MOST_PASSES_BWD = 128;
// Fewest rows of a workgroup.  A workgroup more is a slab more that all others read, and a flag more to wait for.  16384 x 64 forward / backward with
// ReLU, microseconds, with 64, 128 and 256 rows each: 9.8 / 10.7, 8.3 / 9.2, 7.8 / 8.6; 6272 x 64: 7.7 / 8.9, 7.1 / 8.0, 7.1 / 8.1; 392 x 2048: 6.7 / 7.9,
// 6.5 / 7.8, 6.7 / 8.2.  Up to 256 rows one workgroup has all and waits for nobody: 196 x 1024 5.6 / 6.5 instead of 6.4 / 7.4.
int64_t whole_min_rows(int64_t rows) { return rows <= 256 || rows >= 4096 ? 4 * BW_ROWS : 2 * BW_ROWS; }
// Launches apart on this plan, backward: whether the apply pass adds up the slabs itself.  Its slabs are few, so size decides: the pass over y that the
// mask's bits save is worth a finalize launch from some MB up (12544 x 1024, 16 slabs: 41.4 us merged, 38.5 with both; 1568 x 1024, 16 slabs: 11.7 and 12.1).
bool whole_merges_bwd(const BnPlan& p) { return p.slabs <= BN_MERGE_SLABS && p.rows * p.C * 2 <= BN_WIDE_BYTES; }
bool make_whole_plan(int64_t rows, int C, bool forward, BnPlan* p) {
  if (C % BW_CH != 0) return false;
  const int groups = C / BW_CH;
  int64_t per = (rows + BW_WGS / groups - 1) / (BW_WGS / groups);
  if (per < whole_min_rows(rows)) per = whole_min_rows(rows);
  p->rows = rows;
  p->C = C;
  p->cpr = C / 8;
  p->csplit = groups;
  p->threads = BW_THREADS;
  p->rpp = BW_ROWS;
  p->off_part = 0;
  p->slabs = (int)((rows + per - 1) / per);
  p->off_coef = up256((size_t)p->slabs * 2 * C * sizeof(BnSum<true>));
  const size_t coef = (size_t)4 * C * sizeof(float), flags = (size_t)p->slabs * groups * sizeof(unsigned long long);
  p->total = p->off_coef + up256(coef > flags ? coef : flags);
  p->rows_per_slab = per;
  p->mask_iters = (int)((per + BN_BWD_ROWS * BW_ROWS - 1) / (BN_BWD_ROWS * BW_ROWS));
  p->mask_bytes = whole_merges_bwd(*p) ? 0 : (size_t)p->slabs * groups * p->mask_iters * BW_THREADS * 4;
  return per * C * 2 < (int64_t(1) << 31) && (forward || per <= BW_MOST_PASSES_BWD * BW_ROWS);
}

// This plan may take more of the workspace than the other one, which is all that a call has to have.  A workspace of the reported size has room for
// either; with less, or with a tensor of the call where only this plan writes, the call has the other plan.
bool clear_of(const void* ws, size_t n, std::initializer_list<std::pair<const void*, size_t>> tensors) {
  for (const auto& t : tensors)
    if (jz::overlaps(ws, n, t.first, t.second)) return false;
  return true;
}

// Whether a result of the call lies where its parameters do, which the library accepts: in one launch the first workgroups write results while others have
// yet to read parameters; apart, a launch of its own reads them before the results are written.
bool over_parameters(std::initializer_list<std::pair<const void*, size_t>> results, std::initializer_list<const float*> parameters, size_t bytes) {
  for (const auto& r : results)
    for (const float* p : parameters)
      if (jz::overlaps(r.first, r.second, p, bytes)) return true;
  return false;
}

thread_local int t_bn_wait_us = 10;
// A counter that starts where the clock stood, of 62 bits, mixed by steps that keep different numbers different (odd factors, shifted xors): no launch of
// this process has had the result, and sums that an earlier call left in the workspace do not look like it.
unsigned long long bw_tag() {
  static std::atomic<unsigned long long> launches{(unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count()};
  constexpr unsigned long long BITS = (1ull << 62) - 1;
  unsigned long long z;
  do {
    z = 0x9e3779b97f4a7c15ull * launches.fetch_add(1, std::memory_order_relaxed) & BITS;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull & BITS;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull & BITS;
    z ^= z >> 31;
  } while (z == 0);  // what cleared memory holds
  return z << 2;
}

// Whether the stream's workgroups may run on all compute units.
bool bw_all_units(hipStream_t st) {
  uint32_t mask[BW_WGS / 32] = {};
  if (hipExtStreamGetCUMask(st, BW_WGS / 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  int n = 0;
  for (uint32_t m : mask) n += __builtin_popcount(m);
  return n >= BW_WGS;
}

// Whether a call on this stream may take bn_whole: it wants the chip to itself, and several of them from different streams would
// get in each other's way (four streams with 200704 x 64 each: 100 us a call instead of 21).  So one stream a device has it; another one
// gets it after 64 calls without one of the first, unless its workgroups are kept to a part of the chip.  Never while the stream is captured.  Those calls run the passes apart on the same plan, for the
// same bits.  Captured, microseconds, forward / backward with ReLU / block end, on the plan that other channel counts have and on this one:
//   196 x 1024   6.5 /  7.4 /  7.8    5.4 /  6.5 /  7.1      3136 x 2048   13.6 / 22.7 / 28.5    10.8 / 22.4 / 29.5
//   2048 x 128   6.4 /  7.6 /  7.8    6.9 /  7.7 /  8.6      12544 x 1024  17.2 / 39.2 / 46.8    14.3 / 38.5 / 48.5
//   3136 x 256   9.3 / 11.2 / 11.3    7.7 /  9.5 / 10.1      50176 x 512   29.4 / 65.7 / 88.7    28.2 / 67.1 / 92.2
//   3136 x 512  10.2 / 12.0 / 13.5    8.9 / 12.8 / 13.8      12544 x 256   11.0 / 15.5 / 18.4    10.6 / 14.2 / 16.9
//   6272 x 64    7.4 /  9.0 /  9.0    7.6 /  9.3 / 10.1      200704 x 256  54.6 / 120 / 163      54.2 / 121 / 164
//   25088 x 64  10.3 / 12.1 / 13.3   10.4 / 12.9 / 13.3      802816 x 64   54.1 / 120 / 162      53.5 / 118 / 165
// A block end loses up to 5 %, short ones a microsecond, where its rows are read in 128-byte pieces (an XCD for each range of whole rows: worse, 69.6 us backward at 50176 x 512).
// A call whose workgroups have all rows of their channels has nothing to wait for and always may.
bool bw_has_chip(const BnPlan& p, hipStream_t st) {
  if (p.slabs == 1) return true;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &capture) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  int dev = 0, cus = 0;
  if (capture != hipStreamCaptureStatusNone || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < BW_WGS) return false;
  struct Owner {
    std::atomic<uintptr_t> stream{~uintptr_t(0)};  // no stream's handle
    std::atomic<int> others{64};
  };
  static Owner owners[64];
  Owner& o = owners[dev];
  // each thread has its own stream of that name
  const uintptr_t me = st == hipStreamPerThread ? reinterpret_cast<uintptr_t>(&t_bn_wait_us) : reinterpret_cast<uintptr_t>(st);
  if (o.stream.load(std::memory_order_relaxed) != me) {
    if (o.others.fetch_add(1, std::memory_order_relaxed) < 64) return false;
    if (!bw_all_units(st)) {
      o.others.store(0, std::memory_order_relaxed);
      return false;
    }
    o.stream.store(me, std::memory_order_relaxed);
  }
  o.others.store(0, std::memory_order_relaxed);
  return true;
}

template <int MODE>
int launch_whole(const BnPlan& p, BnWholeArgs a, void* ws, hipStream_t st) {
  a.rows = p.rows;
  a.C = p.C;
  a.groups = p.csplit;
  a.wgs = p.slabs;
  a.rows_per_wg = (int)p.rows_per_slab;
  a.part = reinterpret_cast<double*>(static_cast<char*>(ws) + p.off_part);
  a.flags = reinterpret_cast<unsigned long long*>(static_cast<char*>(ws) + p.off_coef);
  a.tag = bw_tag();
  a.wait_ticks = (long long)t_bn_wait_us * 100;
  a.inv_rows = 1.0 / (double)p.rows;
  a.in_place = a.g_out != nullptr && (const void*)a.g_out == (const void*)a.dy;
  const int passes = (int)((p.rows_per_slab + BW_ROWS - 1) / BW_ROWS);
  auto go = [&](auto k_tag, auto l_tag, auto m_tag) {
    constexpr int K = decltype(k_tag)::value, KL = decltype(l_tag)::value, MASKS = decltype(m_tag)::value;
    constexpr size_t lds = ((size_t)KL * (MODE == BW_FWD ? 1 : 2) * 16 + MASKS) * BW_THREADS;
    static std::atomic<bool> lds_set{false};
    if (lds > 0 && !jz::allow_lds(reinterpret_cast<const void*>(bn_whole<MODE, K, KL, MASKS>), lds, lds_set)) return (int)JZ_ERR_LAUNCH;
    hipLaunchKernelGGL((bn_whole<MODE, K, KL, MASKS>), dim3((unsigned)(p.slabs * p.csplit)), dim3(BW_THREADS), lds, st, a);
    return jz::launch_status();
  };
  // the smallest kernel that keeps all passes, else the one that keeps the most: in registers as many as do not spill, then LDS (forward
  // LDS did not pay: 14 passes in LDS behind a full set of registers took 41.7 us at 200704 x 256, the registers alone 39.3)
#define JZ_BW(K, KL, MASKS) go(std::integral_constant<int, K>{}, std::integral_constant<int, KL>{}, std::integral_constant<int, MASKS>{})
  if (passes <= 4) return JZ_BW(4, 0, 0);
  if (passes <= 8) return JZ_BW(8, 0, 0);
  if constexpr (MODE == BW_FWD) return passes <= 16 ? JZ_BW(16, 0, 0) : passes <= 32 ? JZ_BW(32, 0, 0) : JZ_BW(43, 0, 0);
  else if constexpr (MODE == BW_RELU) return passes <= 14 ? JZ_BW(14, 0, 0) : passes <= 25 ? JZ_BW(18, 7, 0) : JZ_BW(18, 6, 56);
  else return passes <= 12 ? JZ_BW(8, 4, 0) : JZ_BW(10, 6, 0);
#undef JZ_BW
}

// grid of a merged apply pass: about `wgs` workgroups, at least one pass of `pass` rows each
dim3 merged_grid(int64_t rows, int C, int pass, int wgs, int* rows_per_wg) {
  const int64_t groups = (C + BM_CH - 1) / BM_CH;
  int64_t per = (rows * groups + wgs - 1) / wgs;
  per = (per + pass - 1) / pass * pass;
  *rows_per_wg = (int)per;
  return dim3((unsigned)groups, (unsigned)((rows + per - 1) / per));
}

unsigned apply_grid(int64_t n_chunks) {
  int64_t b = (n_chunks + BN_THREADS - 1) / BN_THREADS;
  const int64_t cap = 256 * 16;  // 16 workgroups per compute unit, grid-stride beyond that
  return (unsigned)(b < cap ? b : cap);
}

template <int MODE>
int launch_stats(const BnPlan& p, void* part, BnStatsArgs a, hipStream_t st) {
  a.part = part;
  a.rows = p.rows; a.rows_per_slab = p.rows_per_slab;
  a.C = p.C; a.cpr = p.cpr; a.rpp = p.rpp; a.csplit = p.csplit; a.mask_iters = p.mask_iters;
  const dim3 grid((unsigned)(p.slabs * p.csplit));
  if (p.threads == BN_THREADS) hipLaunchKernelGGL((bn_stats<MODE, BN_THREADS>), grid, dim3(BN_THREADS), 0, st, a);
  else hipLaunchKernelGGL((bn_stats<MODE, BW_THREADS>), grid, dim3(BW_THREADS), 0, st, a);
  return jz::launch_status();
}

// what follows the partial sums of the forward pass: totals, saved statistics, y = [relu](a x + b [+ res])
int launch_fwd_rest(const void* part, int slabs, float* coef, int64_t rows, int C, float eps, int relu, const float* gamma, const float* beta,
                    const uint4* x, const uint4* res, uint4* y, float* save_mean, float* save_invstd, hipStream_t st, bool whole = false) {
  const double inv_rows = 1.0 / (double)rows;
  const float* const part32 = static_cast<const float*>(part);
  const double* const part64 = static_cast<const double*>(part);
  auto merged = [&](auto kernel, auto* sums, int threads, int wgs) {
    int per;
    const dim3 grid = merged_grid(rows, C, threads / (BM_CH / 8), wgs, &per);
    hipLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), 0, st, x, res, y, rows, per, C, sums, slabs, inv_rows, eps, relu, gamma, beta, save_mean,
                       save_invstd);
    return jz::launch_status();
  };
  const int64_t nb = rows * C * 2;
  if (slabs <= (whole ? BN_MERGE_SLABS : BN_MERGE_SLABS_WIDE) && nb >= BN_WIDE_BYTES && nb <= BN_FEW_SLABS_BYTES)
    return whole ? merged(bn_apply_merged<0, 512, true>, part64, 512, 512)
           : res ? merged(bn_apply_merged<1, 512>, part32, 512, 512)
                 : merged(bn_apply_merged<0, 512>, part32, 512, 512);
  if (slabs <= BN_MERGE_SLABS && !(whole && nb > BN_FEW_SLABS_BYTES))
    return whole ? merged(bn_apply_merged<0, BN_THREADS, true>, part64, BN_THREADS, 2048)
           : res ? merged(bn_apply_merged<1, BN_THREADS>, part32, BN_THREADS, 2048)
                 : merged(bn_apply_merged<0, BN_THREADS>, part32, BN_THREADS, 2048);
  const dim3 fin((unsigned)((C + BN_FIN_C - 1) / BN_FIN_C));
  if (whole) hipLaunchKernelGGL(bn_fwd_final<double>, fin, dim3(BN_THREADS), 0, st, part64, slabs, C, inv_rows, eps, gamma, beta, save_mean, save_invstd, coef);
  else hipLaunchKernelGGL(bn_fwd_final<float>, fin, dim3(BN_THREADS), 0, st, part32, slabs, C, inv_rows, eps, gamma, beta, save_mean, save_invstd, coef);
  int rc = jz::launch_status();
  if (rc != JZ_OK) return rc;
  const int64_t n_chunks = rows * (C / 8);
  if (res)
    hipLaunchKernelGGL(bn_apply<1>, dim3(apply_grid(n_chunks)), dim3(BN_THREADS), 0, st, x, res, y, coef, n_chunks, C, C / 8, relu);
  else
    hipLaunchKernelGGL(bn_apply<0>, dim3(apply_grid(n_chunks)), dim3(BN_THREADS), 0, st, x, res, y, coef, n_chunks, C, C / 8, relu);
  return jz::launch_status();
}

// the same for the backward pass: parameter gradients, dx from g = dy (masked by y > 0 when relu)
int launch_bwd_rest(const void* part, int slabs, float* coef, int64_t rows, int C, int relu, const float* gamma, const float* mean,
                    const float* invstd, const uint4* x, const uint4* y, const uint4* dy, uint4* dx, void* dgamma16, void* dbeta16, hipStream_t st,
                    const unsigned* mask = nullptr, const BnPlan* p = nullptr) {
  const double inv_rows = 1.0 / (double)rows;
  unsigned short* dg = static_cast<unsigned short*>(dgamma16);
  unsigned short* db = static_cast<unsigned short*>(dbeta16);
  const bool whole = p && p->threads == BW_THREADS;
  const float* const part32 = static_cast<const float*>(part);
  const double* const part64 = static_cast<const double*>(part);
  if (whole ? whole_merges_bwd(*p) : slabs <= BN_MERGE_SLABS) {
    int per;
    const dim3 grid = merged_grid(rows, C, BM_ROWS, 2048, &per);
    if (whole)
      hipLaunchKernelGGL(bn_bwd_apply_merged<true>, grid, dim3(BN_THREADS), 0, st, x, y, dy, dx, rows, per, C, part64, slabs, inv_rows, relu, gamma, mean,
                         invstd, dg, db);
    else
      hipLaunchKernelGGL(bn_bwd_apply_merged<false>, grid, dim3(BN_THREADS), 0, st, x, y, dy, dx, rows, per, C, part32, slabs, inv_rows, relu, gamma, mean,
                         invstd, dg, db);
    return jz::launch_status();
  }
  const dim3 fin((unsigned)((C + BN_FIN_C - 1) / BN_FIN_C));
  if (whole) hipLaunchKernelGGL(bn_bwd_final<double>, fin, dim3(BN_THREADS), 0, st, part64, slabs, C, inv_rows, gamma, mean, invstd, dg, db, coef);
  else hipLaunchKernelGGL(bn_bwd_final<float>, fin, dim3(BN_THREADS), 0, st, part32, slabs, C, inv_rows, gamma, mean, invstd, dg, db, coef);
  int rc = jz::launch_status();
  if (rc != JZ_OK) return rc;
  const int64_t n_chunks = rows * (C / 8);
  const dim3 grid(mask ? (unsigned)(p->slabs * p->csplit) : apply_grid(n_chunks));
  if (mask && p->threads == BN_THREADS)
    hipLaunchKernelGGL(bn_bwd_apply_masked<BN_THREADS>, grid, dim3(BN_THREADS), 0, st, x, dy, dx, coef, mask, rows, C, p->cpr, p->rpp, p->rows_per_slab,
                       p->csplit);
  else if (mask)
    hipLaunchKernelGGL(bn_bwd_apply_masked<BW_THREADS>, grid, dim3(BW_THREADS), 0, st, x, dy, dx, coef, mask, rows, C, p->cpr, p->rpp, p->rows_per_slab,
                       p->csplit);
  else
    hipLaunchKernelGGL(bn_bwd_apply, grid, dim3(BN_THREADS), 0, st, x, y, dy, dx, coef, n_chunks, C, C / 8, relu);
  return jz::launch_status();
}

}  // namespace

extern "C" int jz_bn_tune_wait(int microseconds) {
  if (microseconds < 0 || microseconds > 1000000) return JZ_ERR_SHAPE;
  t_bn_wait_us = microseconds;
  return JZ_OK;
}

extern "C" int jz_bn_workspace_bytes(int64_t rows, int channels, size_t* bytes) {
  if (!bytes) return JZ_ERR_NULL;
  BnPlan p;
  int rc = make_bn_plan(rows, channels, false, &p);  // the forward plan fits where the backward one does
  if (rc != JZ_OK) return rc;
  // room for the plan that takes more, and behind it for the mask's bits (the whole plan's, where there is room for those)
  BnPlan w;
  *bytes = (make_whole_plan(rows, channels, true, &w) && w.total > p.total ? w.total : p.total) + p.mask_bytes;
  return JZ_OK;
}

extern "C" int jz_bn_relu_fwd(int64_t rows, int channels, const void* x16, const float* gamma, const float* beta, float eps,
                              int relu, void* y16, float* save_mean, float* save_invstd, void* ws, size_t ws_bytes,
                              void* hip_stream) {
  BnPlan p, b;
  int rc = make_bn_plan(rows, channels, true, &p);
  if (rc != JZ_OK) return rc;
  make_bn_plan(rows, channels, false, &b);  // one size for both directions
  if (p.total > b.total) p = b;             // it has no more slabs, for any size looked at
  if (!(eps >= 0.f)) return JZ_ERR_SHAPE;
  if (!x16 || !gamma || !beta || !y16 || !save_mean || !save_invstd) return JZ_ERR_NULL;
  if (!ws || ws_bytes < b.total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(x16) || !jz::aligned16(y16) || !jz::aligned16(ws) || !jz::aligned16(gamma) || !jz::aligned16(beta) ||
      !jz::aligned16(save_mean) || !jz::aligned16(save_invstd))
    return JZ_ERR_ALIGN;
  const size_t nb = (size_t)rows * channels * 2, nc = (size_t)channels * 4;
  if (jz::overlaps(y16, nb, x16, nb) || jz::overlaps(ws, p.total, x16, nb) || jz::overlaps(ws, p.total, y16, nb) ||
      jz::overlaps(save_mean, nc, x16, nb) || jz::overlaps(save_invstd, nc, x16, nb) || jz::overlaps(save_mean, nc, save_invstd, nc) ||
      jz::overlaps(save_mean, nc, y16, nb) || jz::overlaps(save_invstd, nc, y16, nb))
    return JZ_ERR_ALIAS;
  BnPlan wp;
  const bool whole = make_whole_plan(rows, channels, true, &wp) && ws_bytes >= wp.total &&
                     !over_parameters({{y16, nb}, {save_mean, nc}, {save_invstd, nc}}, {gamma, beta}, nc) &&
                     clear_of(ws, wp.total, {{x16, nb}, {y16, nb}, {gamma, nc}, {beta, nc}, {save_mean, nc}, {save_invstd, nc}});
  if (whole) p = wp;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_part);
  float* coef = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_coef);
  const uint4* x = static_cast<const uint4*>(x16);
  BnWholeArgs w;
  w.x = x; w.out = static_cast<uint4*>(y16);
  w.gamma = gamma; w.beta = beta; w.save_mean = save_mean; w.save_invstd = save_invstd;
  w.eps = eps; w.relu = relu ? 1 : 0;
  if (whole && bw_has_chip(p, st)) return launch_whole<BW_FWD>(p, w, ws, st);
  if ((rc = launch_stats<ST_SUM>(p, part, {.x = x}, st)) != JZ_OK) return rc;
  return launch_fwd_rest(part, p.slabs, coef, rows, channels, eps, relu ? 1 : 0, gamma, beta, x, nullptr, static_cast<uint4*>(y16), save_mean,
                         save_invstd, st, whole);
}

extern "C" int jz_bn_relu_bwd(int64_t rows, int channels, const void* x16, const void* y16, const void* dy16,
                              const float* gamma, const float* save_mean, const float* save_invstd, int relu, void* dx16,
                              void* dgamma16, void* dbeta16, void* ws, size_t ws_bytes, void* hip_stream) {
  BnPlan p;
  int rc = make_bn_plan(rows, channels, false, &p);
  if (rc != JZ_OK) return rc;
  if (!x16 || !dy16 || !gamma || !save_mean || !save_invstd || !dx16 || !dgamma16 || !dbeta16 || (relu && !y16)) return JZ_ERR_NULL;
  if (!ws || ws_bytes < p.total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(x16) || !jz::aligned16(dy16) || !jz::aligned16(dx16) || !jz::aligned16(ws) || (relu && !jz::aligned16(y16)) ||
      !jz::aligned16(gamma) || !jz::aligned16(save_mean) || !jz::aligned16(save_invstd))
    return JZ_ERR_ALIGN;
  const size_t nb = (size_t)rows * channels * 2, nh = (size_t)channels * 2, nf = (size_t)channels * 4;
  if (jz::overlaps(dx16, nb, x16, nb) || jz::overlaps(dx16, nb, dy16, nb) || (relu && jz::overlaps(dx16, nb, y16, nb)) ||
      jz::overlaps(ws, p.total, x16, nb) || jz::overlaps(ws, p.total, dy16, nb) || jz::overlaps(ws, p.total, dx16, nb) ||
      (relu && jz::overlaps(ws, p.total, y16, nb)) || jz::overlaps(dgamma16, nh, dbeta16, nh) || jz::overlaps(dgamma16, nh, dx16, nb) ||
      jz::overlaps(dbeta16, nh, dx16, nb) || jz::overlaps(dgamma16, nh, x16, nb) || jz::overlaps(dbeta16, nh, x16, nb) ||
      jz::overlaps(dgamma16, nh, dy16, nb) || jz::overlaps(dbeta16, nh, dy16, nb))
    return JZ_ERR_ALIAS;
  BnPlan wp;
  const bool whole = make_whole_plan(rows, channels, false, &wp) && ws_bytes >= wp.total &&
                     !over_parameters({{dx16, nb}, {dgamma16, nh}, {dbeta16, nh}}, {gamma, save_mean, save_invstd}, nf) &&
                     clear_of(ws, wp.total, {{x16, nb}, {relu ? y16 : nullptr, nb}, {dy16, nb}, {dx16, nb}, {gamma, nf}, {save_mean, nf}, {save_invstd, nf},
                                             {dgamma16, nh}, {dbeta16, nh}});
  if (whole) p = wp;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_part);
  float* coef = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_coef);
  // the mask's bits are optional: they go where the workspace has room behind what the call cannot do without, and none of its
  // tensors lies there (a workspace that is the head of a larger piece of memory)
  unsigned* mask = nullptr;
  if (relu && p.mask_bytes > 0 && ws_bytes >= p.total + p.mask_bytes) {
    char* const bits = static_cast<char*>(ws) + p.total;
    auto there = [&](const void* t, size_t n) { return jz::overlaps(bits, p.mask_bytes, t, n); };
    if (!there(x16, nb) && !there(y16, nb) && !there(dy16, nb) && !there(dx16, nb) && !there(gamma, nf) && !there(save_mean, nf) &&
        !there(save_invstd, nf) && !there(dgamma16, nh) && !there(dbeta16, nh))
      mask = reinterpret_cast<unsigned*>(bits);
  }
  const uint4* x = static_cast<const uint4*>(x16);
  const uint4* y = static_cast<const uint4*>(y16);
  const uint4* dy = static_cast<const uint4*>(dy16);
  BnWholeArgs w;
  w.x = x; w.y = y; w.dy = dy; w.out = static_cast<uint4*>(dx16);
  w.gamma = gamma; w.mean = save_mean; w.invstd = save_invstd;
  w.dgamma = static_cast<unsigned short*>(dgamma16); w.dbeta = static_cast<unsigned short*>(dbeta16);
  if (whole && bw_has_chip(p, st)) return relu ? launch_whole<BW_RELU>(p, w, ws, st) : launch_whole<BW_GRAD>(p, w, ws, st);
  const BnStatsArgs in{.x = x, .y = y, .dy = dy, .mask = mask, .mean = save_mean, .invstd = save_invstd};
  rc = !relu ? launch_stats<ST_GRAD>(p, part, in, st) : mask ? launch_stats<ST_MASK>(p, part, in, st) : launch_stats<ST_RELU>(p, part, in, st);
  if (rc != JZ_OK) return rc;
  return launch_bwd_rest(part, p.slabs, coef, rows, channels, relu ? 1 : 0, gamma, save_mean, save_invstd, x, y, dy, static_cast<uint4*>(dx16),
                         dgamma16, dbeta16, st, mask, &p);
}

extern "C" int jz_bn_bwd_block_end(int64_t rows, int channels, const void* x16, const void* y_out16, const void* dya16,
                                   const void* dyb16, const float* gamma, const float* save_mean, const float* save_invstd,
                                   void* g16, void* dx16, void* dgamma16, void* dbeta16, void* ws, size_t ws_bytes, void* hip_stream) {
  BnPlan p;
  int rc = make_bn_plan(rows, channels, false, &p);
  if (rc != JZ_OK) return rc;
  if (!x16 || !y_out16 || !dya16 || !gamma || !save_mean || !save_invstd || !g16 || !dx16 || !dgamma16 || !dbeta16) return JZ_ERR_NULL;
  if (!ws || ws_bytes < p.total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(x16) || !jz::aligned16(y_out16) || !jz::aligned16(dya16) || !jz::aligned16(dyb16) || !jz::aligned16(g16) ||
      !jz::aligned16(dx16) || !jz::aligned16(ws) || !jz::aligned16(gamma) || !jz::aligned16(save_mean) || !jz::aligned16(save_invstd))
    return JZ_ERR_ALIGN;
  const size_t nb = (size_t)rows * channels * 2, nh = (size_t)channels * 2;
  const void* ins[4] = {x16, y_out16, dya16, dyb16};
  void* outs[2] = {g16, dx16};
  for (void* o : outs) {
    for (const void* i : ins)
      if (jz::overlaps(o, nb, i, nb)) return JZ_ERR_ALIAS;
    if (jz::overlaps(o, nb, ws, p.total) || jz::overlaps(o, nb, dgamma16, nh) || jz::overlaps(o, nb, dbeta16, nh)) return JZ_ERR_ALIAS;
  }
  if (jz::overlaps(g16, nb, dx16, nb) || jz::overlaps(dgamma16, nh, dbeta16, nh)) return JZ_ERR_ALIAS;
  for (const void* i : ins)
    if (jz::overlaps(i, nb, ws, p.total) || jz::overlaps(i, nb, dgamma16, nh) || jz::overlaps(i, nb, dbeta16, nh)) return JZ_ERR_ALIAS;
  const size_t nf = (size_t)channels * 4;
  BnPlan wp;
  const bool whole = make_whole_plan(rows, channels, false, &wp) && ws_bytes >= wp.total &&
                     !over_parameters({{g16, nb}, {dx16, nb}, {dgamma16, nh}, {dbeta16, nh}}, {gamma, save_mean, save_invstd}, nf) &&
                     clear_of(ws, wp.total, {{x16, nb}, {y_out16, nb}, {dya16, nb}, {dyb16, nb}, {g16, nb}, {dx16, nb}, {gamma, nf}, {save_mean, nf},
                                             {save_invstd, nf}, {dgamma16, nh}, {dbeta16, nh}});
  if (whole) p = wp;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_part);
  float* coef = reinterpret_cast<float*>(static_cast<char*>(ws) + p.off_coef);
  const uint4* x = static_cast<const uint4*>(x16);
  BnWholeArgs w;
  w.x = x; w.y = static_cast<const uint4*>(y_out16); w.dy = static_cast<const uint4*>(dya16); w.dy2 = static_cast<const uint4*>(dyb16);
  w.g_out = static_cast<uint4*>(g16); w.out = static_cast<uint4*>(dx16);
  w.gamma = gamma; w.mean = save_mean; w.invstd = save_invstd;
  w.dgamma = static_cast<unsigned short*>(dgamma16); w.dbeta = static_cast<unsigned short*>(dbeta16);
  if (whole && bw_has_chip(p, st)) return launch_whole<BW_END>(p, w, ws, st);
  rc = launch_stats<ST_END>(p, part, {.x = x, .y = static_cast<const uint4*>(y_out16), .dy = static_cast<const uint4*>(dya16),
                                      .dy2 = static_cast<const uint4*>(dyb16), .g_out = static_cast<uint4*>(g16), .mean = save_mean,
                                      .invstd = save_invstd}, st);
  if (rc != JZ_OK) return rc;
  return launch_bwd_rest(part, p.slabs, coef, rows, channels, 0, gamma, save_mean, save_invstd, x, nullptr, static_cast<const uint4*>(g16),
                         static_cast<uint4*>(dx16), dgamma16, dbeta16, st, nullptr, &p);
}

// ---- convolution + batch normalization (+ ReLU), forward, with the statistics taken in the convolution's epilogue ----
namespace {

struct ConvBnPlan {
  BnPlan bn;
  size_t conv_ws = 0;   // the convolution's own workspace, at offset 0
  int tiles_m = 0;      // > 0: the convolution kernel leaves [tiles_m][2][C] column sums; 0: a statistics pass is needed
  size_t off_bn = 0, total = 0;
};

int make_conv_bn_plan(const jz_conv_desc* d, ConvBnPlan* p) {
  int rc = jz::conv_fwd_stats_plan(d, &p->conv_ws, &p->tiles_m);
  if (rc != JZ_OK) return rc;
  const int P = (d->H + 2 * d->pad_h - d->R) / d->stride_h + 1, Q = (d->W + 2 * d->pad_w - d->S) / d->stride_w + 1;
  rc = make_bn_plan((int64_t)d->N * P * Q, d->K, false, &p->bn);
  if (rc != JZ_OK) return rc;
  const int slabs = p->tiles_m > p->bn.slabs ? p->tiles_m : p->bn.slabs;
  p->off_bn = up256(p->conv_ws);
  // the batch-norm part of the workspace, laid out like BnPlan's but with room for either number of partial sums
  p->bn.off_part = 0;
  p->bn.off_coef = up256((size_t)slabs * 2 * d->K * sizeof(float));
  p->bn.total = p->bn.off_coef + up256((size_t)4 * d->K * sizeof(float));
  p->total = p->off_bn + p->bn.total;
  return JZ_OK;
}

}  // namespace

extern "C" int jz_conv2d_bn_relu_fwd_workspace_bytes(const jz_conv_desc* desc, size_t* bytes) {
  if (!bytes) return JZ_ERR_NULL;
  ConvBnPlan p;
  int rc = make_conv_bn_plan(desc, &p);
  if (rc != JZ_OK) return rc;
  *bytes = p.total;
  return JZ_OK;
}

extern "C" int jz_conv2d_bn_relu_fwd(const jz_conv_desc* desc, const void* x16, const void* w16, const float* gamma,
                                     const float* beta, float eps, const void* residual16, int relu, void* conv_out16, void* y16,
                                     float* save_mean, float* save_invstd, void* ws, size_t ws_bytes, void* hip_stream) {
  ConvBnPlan p;
  int rc = make_conv_bn_plan(desc, &p);
  if (rc != JZ_OK) return rc;
  if (!(eps >= 0.f)) return JZ_ERR_SHAPE;
  if (!x16 || !w16 || !gamma || !beta || !conv_out16 || !y16 || !save_mean || !save_invstd) return JZ_ERR_NULL;
  if (!ws || ws_bytes < p.total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(y16) || !jz::aligned16(ws) || !jz::aligned16(gamma) || !jz::aligned16(beta) || !jz::aligned16(save_mean) ||
      !jz::aligned16(save_invstd) || !jz::aligned16(residual16))
    return JZ_ERR_ALIGN;
  const int64_t rows = p.bn.rows;
  const int C = p.bn.C;
  const size_t nb = (size_t)rows * C * 2, nc = (size_t)C * 4;
  const size_t nx = (size_t)desc->N * desc->H * desc->W * desc->C * 2, nw = (size_t)desc->K * desc->R * desc->S * desc->C * 2;
  if (jz::overlaps(y16, nb, conv_out16, nb) || jz::overlaps(y16, nb, x16, nx) || jz::overlaps(y16, nb, w16, nw) ||
      jz::overlaps(ws, p.total, y16, nb) || jz::overlaps(save_mean, nc, save_invstd, nc) || jz::overlaps(y16, nb, residual16, nb) ||
      jz::overlaps(conv_out16, nb, residual16, nb) || jz::overlaps(ws, p.total, residual16, nb))
    return JZ_ERR_ALIAS;
  for (const float* sv : {save_mean, save_invstd})
    if (jz::overlaps(sv, nc, y16, nb) || jz::overlaps(sv, nc, conv_out16, nb) || jz::overlaps(sv, nc, x16, nx) ||
        jz::overlaps(sv, nc, w16, nw) || jz::overlaps(sv, nc, ws, p.total) || jz::overlaps(sv, nc, residual16, nb))
      return JZ_ERR_ALIAS;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char* bws = static_cast<char*>(ws) + p.off_bn;
  float* part = reinterpret_cast<float*>(bws + p.bn.off_part);
  float* coef = reinterpret_cast<float*>(bws + p.bn.off_coef);
  // the convolution (its own checks cover x, w, conv_out and its part of the workspace)
  jz::BnTail tail{.gamma = gamma, .beta = beta, .eps = eps, .relu = relu ? 1 : 0, .residual16 = residual16, .y16 = y16, .save_mean = save_mean,
                  .save_invstd = save_invstd};
  rc = jz::conv_fwd_run(desc, x16, w16, conv_out16, ws, p.conv_ws, p.tiles_m > 0 ? part : nullptr, p.tiles_m, &tail, hip_stream);
  if (rc != JZ_OK || tail.done) return rc;
  const uint4* c = static_cast<const uint4*>(conv_out16);
  int slabs = p.tiles_m;
  if (slabs == 0) {  // this convolution kernel cannot leave the sums: one more pass over its output
    slabs = p.bn.slabs;
    if ((rc = launch_stats<ST_SUM>(p.bn, part, {.x = c}, st)) != JZ_OK) return rc;
  }
  return launch_fwd_rest(part, slabs, coef, rows, C, eps, relu ? 1 : 0, gamma, beta, c, static_cast<const uint4*>(residual16),
                         static_cast<uint4*>(y16), save_mean, save_invstd, st);
}

// ---- backward-data of a convolution + the backward pass of the batch normalization + ReLU that produced its input ----
// The statistics pass of the normalization's backward (sum g, sum g x^ over g = dz where y > 0) reads dz, y and x; here
// the convolution's epilogue takes the sums while the dz tile is still on chip (it reads the matching y and x tiles), so
// that pass and its launch disappear.
namespace {

struct ConvBnBwdPlan {
  BnPlan bn;            // of the normalization: rows = N*H*W of the convolution's input, C = its channels
  size_t conv_ws = 0;
  int tiles_m = 0;      // > 0: the convolution kernel leaves [tiles_m][2][C] sums; 0: the statistics pass runs
  size_t off_bn = 0, total = 0;
  bool whole = false;   // bn_whole takes the normalization where there is room for `whole_bn`
  BnPlan whole_bn;
  size_t reported = 0;
};

int make_conv_bn_bwd_plan(const jz_conv_desc* d, ConvBnBwdPlan* p) {
  int rc = jz::conv_bwd_data_stats_plan(d, &p->conv_ws, &p->tiles_m);
  if (rc != JZ_OK) return rc;
  rc = make_bn_plan((int64_t)d->N * d->H * d->W, d->C, false, &p->bn);
  if (rc != JZ_OK) return rc;
  const int slabs = p->tiles_m > p->bn.slabs ? p->tiles_m : p->bn.slabs;
  p->off_bn = up256(p->conv_ws);
  p->bn.off_part = 0;
  p->bn.off_coef = up256((size_t)slabs * 2 * d->C * sizeof(float));
  p->bn.total = p->bn.off_coef + up256((size_t)4 * d->C * sizeof(float));
  p->total = p->reported = p->off_bn + p->bn.total;
  p->whole = p->tiles_m == 0 && make_whole_plan(p->bn.rows, d->C, false, &p->whole_bn);
  if (p->whole && p->whole_bn.total > p->bn.total) p->reported = p->off_bn + p->whole_bn.total;
  return JZ_OK;
}

}  // namespace

extern "C" int jz_conv2d_bwd_data_bn_relu_bwd_workspace_bytes(const jz_conv_desc* desc, size_t* bytes) {
  if (!bytes) return JZ_ERR_NULL;
  ConvBnBwdPlan p;
  int rc = make_conv_bn_bwd_plan(desc, &p);
  if (rc != JZ_OK) return rc;
  *bytes = p.reported;
  return JZ_OK;
}

// block_end false: dz = bwd_data, then the backward of y = relu(bn(x)) for dy = dz.
// block_end true:  y = relu(bn(x) + shortcut) is a residual block's output and bwd_data is one contribution to its gradient:
//                  g = RNE16(bwd_data [+ add]) where y > 0, else 0, goes to `out`, then the backward of bn(x) (no ReLU) for dy = g.
static int conv_bwd_data_bn_bwd(const jz_conv_desc* desc, const void* dy16, const void* w16, const void* bn_x16, const void* bn_y16,
                                const void* add16, bool block_end, const float* gamma, const float* save_mean, const float* save_invstd,
                                void* out16, void* bn_dx16, void* dgamma16, void* dbeta16, void* ws, size_t ws_bytes, void* hip_stream) {
  ConvBnBwdPlan p;
  int rc = make_conv_bn_bwd_plan(desc, &p);
  if (rc != JZ_OK) return rc;
  if (!dy16 || !w16 || !bn_x16 || !bn_y16 || !gamma || !save_mean || !save_invstd || !out16 || !bn_dx16 || !dgamma16 || !dbeta16)
    return JZ_ERR_NULL;
  if (!ws || ws_bytes < p.total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(bn_x16) || !jz::aligned16(bn_y16) || !jz::aligned16(add16) || !jz::aligned16(bn_dx16) || !jz::aligned16(ws) ||
      !jz::aligned16(gamma) || !jz::aligned16(save_mean) || !jz::aligned16(save_invstd))
    return JZ_ERR_ALIGN;
  const int64_t rows = p.bn.rows;
  const int C = p.bn.C;
  const size_t nb = (size_t)rows * C * 2, nh = (size_t)C * 2, nc = (size_t)C * 4;
  const int P = (desc->H + 2 * desc->pad_h - desc->R) / desc->stride_h + 1, Q = (desc->W + 2 * desc->pad_w - desc->S) / desc->stride_w + 1;
  const size_t ny = (size_t)desc->N * P * Q * desc->K * 2, nw = (size_t)desc->K * desc->R * desc->S * desc->C * 2;
  // outputs against everything else (the convolution's own checks cover dy, w, its output and its part of the workspace)
  const void* outs[4] = {out16, bn_dx16, dgamma16, dbeta16};
  const size_t outn[4] = {nb, nb, nh, nh};
  const void* ins[8] = {dy16, w16, bn_x16, bn_y16, gamma, save_mean, save_invstd, add16};
  const size_t inn[8] = {ny, nw, nb, nb, nc, nc, nc, add16 ? nb : 0};
  for (int i = 0; i < 4; ++i) {
    for (int j = 0; j < 8; ++j)
      if (inn[j] && jz::overlaps(outs[i], outn[i], ins[j], inn[j])) return JZ_ERR_ALIAS;
    for (int j = i + 1; j < 4; ++j)
      if (jz::overlaps(outs[i], outn[i], outs[j], outn[j])) return JZ_ERR_ALIAS;
    if (jz::overlaps(outs[i], outn[i], ws, p.total)) return JZ_ERR_ALIAS;
  }
  for (int j = 0; j < 8; ++j)
    if (inn[j] && jz::overlaps(ins[j], inn[j], ws, p.total)) return JZ_ERR_ALIAS;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char* bws = static_cast<char*>(ws) + p.off_bn;
  float* part = reinterpret_cast<float*>(bws + p.bn.off_part);
  float* coef = reinterpret_cast<float*>(bws + p.bn.off_coef);
  jz::BnBwdOperands bn{bn_x16, bn_y16, save_mean, save_invstd};
  bn.block_end = block_end;
  bn.add16 = add16;
  jz::BnTail tail{.gamma = gamma, .dx16 = bn_dx16, .dgamma16 = dgamma16, .dbeta16 = dbeta16};
  rc = jz::conv_bwd_data_run(desc, dy16, w16, out16, ws, p.conv_ws, p.tiles_m > 0 ? part : nullptr, p.tiles_m, &bn, &tail, hip_stream);
  if (rc != JZ_OK || tail.done) return rc;
  const uint4* x = static_cast<const uint4*>(bn_x16);
  const uint4* y = static_cast<const uint4*>(bn_y16);
  const uint4* dz = static_cast<const uint4*>(out16);
  if (p.tiles_m > 0)
    return launch_bwd_rest(part, p.tiles_m, coef, rows, C, block_end ? 0 : 1, gamma, save_mean, save_invstd, x, block_end ? nullptr : y, dz,
                           static_cast<uint4*>(bn_dx16), dgamma16, dbeta16, st);
  // This convolution kernel cannot leave the sums: the normalization as its own call takes it, a block end with g in place.  In one launch
  // 83 us at the block ends of ResNet-50's strided layers (batch 64, 200704 x 256 to 12544 x 1024, mean), as statistics and the rest 102.
  bool whole = p.whole && ws_bytes >= p.off_bn + p.whole_bn.total;
  for (int i = 0; i < 4; ++i) whole = whole && !jz::overlaps(bws, p.whole_bn.total, outs[i], outn[i]);
  for (int j = 0; j < 8; ++j) whole = whole && !jz::overlaps(bws, p.whole_bn.total, ins[j], inn[j]);
  if (whole) {
    p.bn = p.whole_bn;
    part = reinterpret_cast<float*>(bws + p.bn.off_part);
    coef = reinterpret_cast<float*>(bws + p.bn.off_coef);
  }
  uint4* const g = static_cast<uint4*>(out16);
  const uint4* const add = static_cast<const uint4*>(add16);
  if (whole && bw_has_chip(p.bn, st)) {
    BnWholeArgs w;
    w.x = x; w.y = y; w.dy = dz; w.dy2 = add;
    w.g_out = g; w.out = static_cast<uint4*>(bn_dx16);
    w.gamma = gamma; w.mean = save_mean; w.invstd = save_invstd;
    w.dgamma = static_cast<unsigned short*>(dgamma16); w.dbeta = static_cast<unsigned short*>(dbeta16);
    return block_end ? launch_whole<BW_END>(p.bn, w, bws, st) : launch_whole<BW_RELU>(p.bn, w, bws, st);
  }
  const BnStatsArgs in{.x = x, .y = y, .dy = dz, .dy2 = add, .g_out = g, .mean = save_mean, .invstd = save_invstd};
  rc = block_end ? launch_stats<ST_END>(p.bn, part, in, st) : launch_stats<ST_RELU>(p.bn, part, in, st);
  if (rc != JZ_OK) return rc;
  return launch_bwd_rest(part, p.bn.slabs, coef, rows, C, block_end ? 0 : 1, gamma, save_mean, save_invstd, x, block_end ? nullptr : y, dz,
                         static_cast<uint4*>(bn_dx16), dgamma16, dbeta16, st, nullptr, &p.bn);
}

extern "C" int jz_conv2d_bwd_data_bn_relu_bwd(const jz_conv_desc* desc, const void* dy16, const void* w16, const void* bn_x16,
                                              const void* bn_y16, const float* gamma, const float* save_mean,
                                              const float* save_invstd, void* dz16, void* bn_dx16, void* dgamma16, void* dbeta16,
                                              void* ws, size_t ws_bytes, void* hip_stream) {
  return conv_bwd_data_bn_bwd(desc, dy16, w16, bn_x16, bn_y16, nullptr, false, gamma, save_mean, save_invstd, dz16, bn_dx16, dgamma16,
                              dbeta16, ws, ws_bytes, hip_stream);
}

extern "C" int jz_conv2d_bwd_data_block_end_bwd(const jz_conv_desc* desc, const void* dy16, const void* w16, const void* dyb16,
                                                const void* bn_x16, const void* y_out16, const float* gamma, const float* save_mean,
                                                const float* save_invstd, void* g16, void* bn_dx16, void* dgamma16, void* dbeta16,
                                                void* ws, size_t ws_bytes, void* hip_stream) {
  return conv_bwd_data_bn_bwd(desc, dy16, w16, bn_x16, y_out16, dyb16, true, gamma, save_mean, save_invstd, g16, bn_dx16, dgamma16,
                              dbeta16, ws, ws_bytes, hip_stream);
}
