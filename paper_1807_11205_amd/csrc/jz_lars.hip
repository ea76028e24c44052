// Mixed-precision LARS update (Jia et al. 2018, Section 4.1, Eq. 1, Fig. 2) for gfx950.
//
// fp16 loss-scaled gradients and the fp32 master weights are widened, the layer-wise rate
// rho_t = eta*||w_t||/||g_t|| is formed, the momentum step is taken on the fp32 master copy and the
// result is narrowed to fp16 for the next forward pass.  The whole thing is HBM-bound (20 bytes per
// parameter must move), so it is organised as three stream-ordered launches over a fused flat buffer:
//
//   lars_reduce    per chunk (<= LARS_CH elements inside one tensor): the fp64 sum of g16^2 (and of w^2, unless the
//                  workspace still holds it from the previous update), not finite when a gradient is not, stored per
//                  chunk (no atomics => deterministic).  It runs at about 3 TB/s because the update in front of it left
//                  the last-level cache full of lines that have to be written out first (a persistent form that requests
//                  the next chunk ahead is no faster)
//   lars_finalize  one workgroup per tensor: adds that tensor's chunk sums in a fixed order, forms lr*rho_t.  A thread
//                  requests ten sums at once; 1024 threads when a tensor has more chunks than 256 threads take in one
//                  round (a 38 M-element tensor has 9216: 57 us with 256 threads and a sum per wavefront, 8 us now)
//   lars_update    one workgroup per chunk, walking the buffer in the opposite direction so that the
//                  tail the reduce pass touched last is still in the last-level cache; skips everything
//                  when any tensor raised the flag.  While writing w it accumulates the chunk's sum of w^2,
//                  which the next update's reduce pass then need not read w for.
//
// A set of at most LARS_SMALL_CHUNKS chunks is one launch of one workgroup (lars_small): three launches are 13 us of
// latency whatever they do.  Other small sets, and those with very large tensors, take two: a workgroup of the reduce pass takes
// a group of chunks of one tensor (lars_reduce_groups), so few that every workgroup of the update adds up its tensor's group sums
// itself while its chunk is on its way (lars_update<LARS_GROUPS>).
//
// When the kernels that produce the gradients also leave each tensor's sum of squares (jz_sumsq.h), the first two
// launches have nothing left to do at update time and the update is one launch ("presummed"):
//
//   lars_begin       at the start of a step, one workgroup per tensor: adds the partial sums of w^2 the last update left
//                    (or, for a fresh workspace, squares the tensor itself), clears the tensor's gradient sink
//   lars_grad_sumsq  the reduce pass for the tensors no other kernel covers (batch-norm scale / shift, bias), any time
//                    after their gradients exist
//   lars_update<LARS_PRE>  every wavefront forms lr*rho_t of its chunk's tensor itself from the sink and the sum lars_begin
//                    left; otherwise the same kernel
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "jz_internal.h"
#include "jz_sumsq.h"

namespace {

#ifndef JZ_LARS_CH
#define JZ_LARS_CH 4096
#endif
constexpr int LARS_CH = JZ_LARS_CH;  // elements per chunk; a multiple of 2048 (8 per thread and pass)
constexpr int LARS_THREADS = 256;
constexpr int LARS_WAVES = LARS_THREADS / 64;
constexpr int LARS_FIN_BATCH = 10;       // chunk sums a thread of the finalize kernel requests together
constexpr int LARS_SMALL_CHUNKS = 4;     // largest set lars_small takes: one chunk per group of threads (18 chunks: 37 us) ...
constexpr int LARS_SMALL_T = 64;         // ... and this many tensors
// Sets whose update works out its rates itself, which saves the finalize launch: at most LARS_MAX_GROUPS groups of chunks, two
// for every thread, and either few chunks in all or more in one tensor than the finalize kernel takes in one round of 256 threads.
// Updates in a row: 505 chunks 17.5 -> 15.3 us, 1075 chunks 25.3 -> 24.6, AlexNet's 15230 (9216 in one tensor, 11 us of the
// finalize launch) 259 -> 253; between those fewer, longer workgroups cost the reduce pass what the launch costs (1954 chunks 36.9
// and 37.4 us, ResNet-50's 6334 109.3 and 110.6).
constexpr int LARS_MAX_GROUPS = 2 * LARS_THREADS;
constexpr int64_t LARS_GROUPED_CHUNKS = 1536;
enum { LARS_PLAIN = 0, LARS_PRE = 1, LARS_GROUPS = 2 };  // where lars_update takes a tensor's rate from
constexpr uint64_t LARS_MAGIC = 0x4a5a4c4152533031ull;  // "JZLARS01"

// Everything a workgroup needs to know about its chunk in one 16-byte record: a kernel's first loads then depend on
// one table look-up, not on a chain of three (chunk -> tensor -> offsets), each a cold round trip to memory.
struct ChunkRec {
  int64_t start;  // first element
  int count;      // elements (<= LARS_CH)
  int tensor;
};

// Chunks chunk0, chunk0 + stride, ... of a tensor: the groups of a tensor interleave, so that workgroups side by side read side by side.
struct GroupRec {
  int chunk0, chunks, tensor, stride;
  int64_t start, end;  // of the first chunk, of the tensor
};

struct Layout {
  int64_t T = 0, P = 0, n_chunks = 0;
  int64_t group_chunks = 1, n_groups = 0;  // chunks of a group at most; 0 groups: the update takes the rates from lars_finalize
  int64_t most_chunks = 0;  // of one tensor
  size_t off_header = 0, off_offsets = 0, off_chunk_begin = 0, off_flags = 0, off_chunk_tensor = 0, off_chunk_rec = 0, off_group_rec = 0;
  size_t off_state = 0;
  size_t static_bytes = 0;  // everything up to here is written by prepare
  size_t off_psum_w = 0, off_psum_g = 0, off_coef = 0, off_tflag = 0;
  size_t off_gsum = 0, off_gflag = 0, off_wsum = 0, off_group_sum = 0, total = 0;  // presummed path: gradient sinks, their flags, sum of w^2
};

size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// The smallest of the group sizes 1, 2, 4, 8, 12, 16 ... that leaves at most LARS_MAX_GROUPS groups, for a set with no more tensors
// than that.  The layout is worked out by every call, so the sizes are not tried one after the other: size s leaves at least
// chunks / s groups and fewer than chunks / s + filled, and between those bounds the search halves (a set that takes groups costs one
// or two passes over its tensors, up to ten where nearly every tensor is a group of its own; the others none).
void choose_groups(const jz_param_set* ps, int64_t filled, Layout* L) {
  auto size = [](int64_t i) { return i < 2 ? i + 1 : 4 * (i - 1); };             // candidate i
  auto first_from = [](int64_t s) { return s <= 2 ? s - 1 : (s + 3) / 4 + 1; };  // the first candidate of at least s >= 1
  auto groups = [&](int64_t s) {
    int64_t n = 0;
    for (int64_t t = 0; t < L->T; ++t) {
      const unsigned nc = (unsigned)((ps->offsets[t + 1] - ps->offsets[t] + LARS_CH - 1) / LARS_CH);
      n += (nc + (unsigned)s - 1) / (unsigned)s;
    }
    return n;
  };
  const int64_t spare = LARS_MAX_GROUPS - filled, least = (L->n_chunks + LARS_MAX_GROUPS - 1) / LARS_MAX_GROUPS;
  int64_t enough = L->most_chunks;
  if (spare > 0 && (L->n_chunks + spare - 1) / spare < enough) enough = (L->n_chunks + spare - 1) / spare;
  int64_t lo = first_from(least < 1 ? 1 : least), hi = first_from(enough < 1 ? 1 : enough);
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (groups(size(mid)) <= LARS_MAX_GROUPS) hi = mid;
    else lo = mid + 1;
  }
  L->group_chunks = size(hi);
  L->n_groups = groups(L->group_chunks);
}

int make_layout(const jz_param_set* ps, Layout* L) {
  if (!ps) return JZ_ERR_NULL;
  if (ps->num_tensors < 0) return JZ_ERR_SHAPE;
  if (ps->num_tensors > 0 && (!ps->offsets || !ps->flags)) return JZ_ERR_NULL;
  L->T = ps->num_tensors;
  int64_t chunks = 0, filled = 0;  // tensors that have elements
  if (L->T > 0) {
    if (ps->offsets[0] != 0) return JZ_ERR_SHAPE;
    for (int64_t t = 0; t < L->T; ++t) {
      int64_t n = ps->offsets[t + 1] - ps->offsets[t];
      if (n < 0) return JZ_ERR_SHAPE;
      if (n >= (int64_t(1) << 31)) return JZ_ERR_UNSUPPORTED;
      const int64_t nc = (n + LARS_CH - 1) / LARS_CH;
      chunks += nc;
      filled += nc > 0 ? 1 : 0;
      if (nc > L->most_chunks) L->most_chunks = nc;
    }
    L->P = ps->offsets[L->T];
  }
  if (L->T >= (int64_t(1) << 24) || chunks >= (int64_t(1) << 30)) return JZ_ERR_UNSUPPORTED;
  L->n_chunks = chunks;
  if (filled <= LARS_MAX_GROUPS && (chunks <= LARS_GROUPED_CHUNKS || L->most_chunks > 256 * LARS_FIN_BATCH)) choose_groups(ps, filled, L);
  size_t o = 0;
  L->off_header = o;        o = up256(o + 64);
  L->off_offsets = o;       o = up256(o + sizeof(int64_t) * (L->T + 1));
  L->off_chunk_begin = o;   o = up256(o + sizeof(int) * (L->T + 1));
  L->off_flags = o;         o = up256(o + sizeof(int) * (L->T ? L->T : 1));
  L->off_chunk_tensor = o;  o = up256(o + sizeof(int) * (chunks ? chunks : 1));
  L->off_chunk_rec = o;     o = up256(o + sizeof(ChunkRec) * (chunks ? chunks : 1));
  L->off_group_rec = o;     o = up256(o + sizeof(GroupRec) * L->n_groups);
  L->off_state = o;         o = up256(o + 64);
  L->static_bytes = o;
  const size_t parts = (size_t)(chunks ? chunks : 1);
  L->off_psum_w = o;        o = up256(o + sizeof(double) * parts * LARS_WAVES);
  L->off_psum_g = o;        o = up256(o + sizeof(double) * parts);
  L->off_coef = o;          o = up256(o + sizeof(float) * (L->T ? L->T : 1));
  L->off_tflag = o;         o = up256(o + sizeof(int) * (L->T ? L->T : 1));
  L->off_gsum = o;          o = up256(o + jz::kSumsqSinkBytes * (L->T ? L->T : 1));
  L->off_gflag = o;         o = up256(o + sizeof(int) * (L->T ? L->T : 1));
  L->off_wsum = o;          o = up256(o + sizeof(double) * (L->T ? L->T : 1));
  L->off_group_sum = o;     o = up256(o + sizeof(double2) * L->n_groups);
  L->total = o;
  return JZ_OK;
}

uint64_t table_checksum(const jz_param_set* ps) {  // FNV-1a over T, offsets and flags
  uint64_t h = 1469598103934665603ull;
  auto mix = [&](const void* p, size_t n) {
    const unsigned char* b = static_cast<const unsigned char*>(p);
    for (size_t i = 0; i < n; ++i) { h ^= b[i]; h *= 1099511628211ull; }
  };
  int64_t T = ps->num_tensors;
  mix(&T, sizeof T);
  if (T > 0) { mix(ps->offsets, sizeof(int64_t) * (T + 1)); mix(ps->flags, T); }
  return h ? h : 1;
}

// host-side note of which workspace holds which table (the device header is checked as well)
// begun: jz_lars_begin_step has run since the last presummed update (and with which loss-scale state)
struct Prepared { void* ws; uint64_t sum; bool begun; const void* begun_state; };
std::mutex g_mu;
Prepared g_prepared[64];
int g_next = 0;

void remember(void* ws, uint64_t sum) {
  std::lock_guard<std::mutex> lk(g_mu);
  for (auto& e : g_prepared)
    if (e.ws == ws) { e = {ws, sum, false, nullptr}; return; }
  g_prepared[g_next] = {ws, sum, false, nullptr};
  g_next = (g_next + 1) % 64;
}
void set_begun(void* ws, bool begun, const void* state) {
  std::lock_guard<std::mutex> lk(g_mu);
  for (auto& e : g_prepared)
    if (e.ws == ws) { e.begun = begun; e.begun_state = state; }
}
bool has_begun(void* ws, const void* state) {
  std::lock_guard<std::mutex> lk(g_mu);
  for (auto& e : g_prepared)
    if (e.ws == ws) return e.begun && e.begun_state == state;
  return false;
}
bool is_prepared(void* ws, uint64_t sum) {
  std::lock_guard<std::mutex> lk(g_mu);
  for (auto& e : g_prepared)
    if (e.ws == ws) return e.sum == sum;
  return false;
}

// a chunk's sum of w^2 from its wavefronts' sums
__device__ __forceinline__ double chunk_sumsq_w(const double* __restrict__ psum_w, int c) {
  const double2 a = *reinterpret_cast<const double2*>(psum_w + (size_t)c * LARS_WAVES), b = *reinterpret_cast<const double2*>(psum_w + (size_t)c * LARS_WAVES + 2);
  return ((a.x + a.y) + b.x) + b.y;
}

struct Tables {
  const uint64_t* header;
  const int64_t* offsets;
  const int* chunk_begin;
  const int* flags;
  const int* chunk_tensor;
  const ChunkRec* chunk_rec;
  int* state;    // [0]: 1 when psum_w holds the sums of squares of the current master weights; [1], [2]: 1/S and S as
                 // float bits when the loss scale lives on the device (written by a launch before the update)
  double* psum_w;  // [n_chunks][LARS_WAVES] sums of w^2, one per wavefront: the update kernel then ends without a barrier
  double* psum_g;  // [n_chunks] sums of the squared (loss-scaled) gradients; Inf / NaN: a gradient of the chunk is not finite
  float* coef;  // lr * rho_t
  int* tflag;
  unsigned long long* gsum;  // [T][kSumsqSubs * kSumsqSubStride]: gradient sum-of-squares sinks
  int* gflag;                // [T]: non-finite gradient reported to the sink
  double* wsum;              // [T]: sum of squares of the master weights, written by lars_begin
  const GroupRec* group_rec;
  double2* group_sum;        // [n_groups] sums of w^2 and of g16^2
  int T, n_chunks, n_groups;
  uint64_t checksum;
};

__device__ __forceinline__ bool table_ok(const Tables& tb) { return tb.header[0] == LARS_MAGIC && tb.header[1] == tb.checksum; }

__device__ __forceinline__ bool half_nonfinite(unsigned short h) { return (h & 0x7c00u) == 0x7c00u; }
__device__ __forceinline__ float half_bits_to_float(unsigned short h) {
  _Float16 x;
  __builtin_memcpy(&x, &h, 2);
  return (float)x;
}
__device__ __forceinline__ unsigned short float_to_half_bits(float f) {
  _Float16 x = (_Float16)f;  // round to nearest even, overflow to Inf, subnormals kept
  unsigned short h;
  __builtin_memcpy(&h, &x, 2);
  return h;
}

// Sum over a workgroup of NW wavefronts in a fixed order: lanes by shuffle tree, then the wavefronts left to right.
template <int NW>
__device__ __forceinline__ double block_sum(double v, double* lds) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[wv] = v;
  __syncthreads();
  double t = lds[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) t += lds[i];
  return t;
}

// Workgroup barrier for data exchanged through LDS: unlike __syncthreads() it does not wait for the global stores in flight.
__device__ __forceinline__ void lds_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#endif
}

// Sum over the 64 lanes of a wavefront by a fixed shuffle tree; the total ends up in lane 0.
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

__device__ __forceinline__ void chunk_range(const ChunkRec& r, int* t_out, int64_t* start, int64_t* end) {
  *t_out = r.tensor;
  *start = r.start;
  *end = r.start + r.count;
}

constexpr int LARS_IT = LARS_CH / (LARS_THREADS * 8);     // 8-element groups per thread and chunk: gradients where nothing else is read
constexpr int LARS_QUADS = LARS_CH / (LARS_THREADS * 4);  // 4-element groups: weights, momentum and what goes with them

// 16-byte accesses of the update pass.  What it writes (w, v, the FP16 copy: 20 of 28 bytes an element) goes out with the
// non-temporal hint, or dirty lines of it are still being written back while the next pass reads: ResNet-50 113 -> 109 us,
// AlexNet 279 -> 260 us for updates one behind the other; an update of a state that was just written (133, 325 us) gains
// nothing.  The gradient, which the reduce pass has just read, is in the last-level cache: plain
// loads.  So is a part of the state when it fits there (204 MB for ResNet-50: 93 us for updates in a row, 108 with the hint);
// state that does not fit only displaces the gradient and is read with the hint (STREAM; AlexNet 261 -> 253 us).
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
constexpr int64_t LARS_STREAM_ELEMENTS = (256ll << 20) / 8;  // 8 bytes of state an element against 256 MiB of last-level cache
template <bool STREAM>
__device__ __forceinline__ float4 load_state_f4(const float* p) {
  if constexpr (!STREAM) return *reinterpret_cast<const float4*>(p);
  f32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(p));
  return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void store_stream_f4(float* p, float a, float b, float c, float d) {
  f32x4_t t = {a, b, c, d};
  __builtin_nontemporal_store(t, reinterpret_cast<f32x4_t*>(p));
}
__device__ __forceinline__ void store_stream_u2(unsigned short* p, unsigned a, unsigned b) {
  u32x2_t t = {a, b};
  __builtin_nontemporal_store(t, reinterpret_cast<u32x2_t*>(p));
}

// the 8-aligned body [b0,b1) of a chunk [s,e); the rest is at most 7 head and 7 tail elements
__device__ __forceinline__ void chunk_body(int64_t s, int64_t e, int64_t* b0, int64_t* b1) {
  int64_t a = (s + 7) & ~int64_t(7);
  if (a > e) a = e;
  *b0 = a;
  *b1 = a + ((e - a) & ~int64_t(7));
}

// A thread's weights of one chunk: its 4-element groups (zero where the chunk has none) and at most one head / tail element.  Whole
// chunks, nearly all, are loaded without conditions: behind a condition each, one group was waited for before the next was asked for.
struct ChunkWeights {
  float4 q[LARS_QUADS];
  float edge;
};
__device__ __forceinline__ ChunkWeights load_chunk_weights(const ChunkRec& rec, const float* __restrict__ w, int tid) {
  ChunkWeights r;
  if (rec.count == LARS_CH && (rec.start & 7) == 0) {
#pragma unroll
    for (int k = 0; k < LARS_QUADS; ++k) r.q[k] = *reinterpret_cast<const float4*>(w + rec.start + (k * LARS_THREADS + tid) * 4);
    r.edge = 0.f;
    return r;
  }
  int t;
  int64_t s, e, b0, b1;
  chunk_range(rec, &t, &s, &e);
  chunk_body(s, e, &b0, &b1);
#pragma unroll
  for (int k = 0; k < LARS_QUADS; ++k) {
    const int64_t i = b0 + (int64_t)(k * LARS_THREADS + tid) * 4;
    r.q[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < b1) r.q[k] = *reinterpret_cast<const float4*>(w + i);
  }
  const int64_t nh = b0 - s, nt = e - b1, k = tid;
  r.edge = k < nh + nt ? w[k < nh ? s + k : b1 + (k - nh)] : 0.f;
  return r;
}
// Its sum of squares, in the order lars_update adds it.
__device__ __forceinline__ double chunk_thread_sumsq_w(const ChunkWeights& r) {
  double sw = 0.0;
#pragma unroll
  for (int k = 0; k < LARS_QUADS; ++k) {
    const float wv[4] = {r.q[k].x, r.q[k].y, r.q[k].z, r.q[k].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) sw = fma((double)wv[j], (double)wv[j], sw);
  }
  return fma((double)r.edge, (double)r.edge, sw);
}

// A thread's gradients of one chunk: its 8-element groups (zero where the chunk has none) and at most one head / tail element.
struct ChunkGrads {
  uint4 q[LARS_IT];
  unsigned short edge;
};
__device__ __forceinline__ ChunkGrads load_chunk_grads(const ChunkRec& rec, const unsigned short* __restrict__ g16, int tid) {
  ChunkGrads r;
  int t;
  int64_t s, e, b0, b1;
  chunk_range(rec, &t, &s, &e);
  chunk_body(s, e, &b0, &b1);
#pragma unroll
  for (int k = 0; k < LARS_IT; ++k) {
    const int64_t i = b0 + (int64_t)(k * LARS_THREADS + tid) * 8;
    r.q[k] = make_uint4(0, 0, 0, 0);
    if (i < b1) r.q[k] = *reinterpret_cast<const uint4*>(g16 + i);
  }
  const int64_t nh = b0 - s, nt = e - b1, k = tid;
  r.edge = k < nh + nt ? g16[k < nh ? s + k : b1 + (k - nh)] : (unsigned short)0;
  return r;
}
// Its sum of squares; not finite when one of them is not (the sum of finite halves' squares cannot overflow in FP64), so
// nothing has to be tested per element: the pass is bound by vector arithmetic (13 instructions per element: 3.1 TB/s).
// The square of a half is exact in FP32 (22 bits), the sum is FP64.
__device__ __forceinline__ double chunk_thread_sumsq_g(const ChunkGrads& r) {
  double sg = 0.0;
#pragma unroll
  for (int k = 0; k < LARS_IT; ++k) {
    const unsigned gw[4] = {r.q[k].x, r.q[k].y, r.q[k].z, r.q[k].w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float g = half_bits_to_float((unsigned short)(gw[j >> 1] >> ((j & 1) * 16)));
      sg += (double)(g * g);
    }
  }
  const float g = half_bits_to_float(r.edge);
  return sg + (double)(g * g);
}
__device__ __forceinline__ bool sum_overflowed(double sg) { return !(sg <= 1.7e308); }  // Inf or NaN

__global__ __launch_bounds__(LARS_THREADS) void lars_reduce(Tables tb, const float* __restrict__ w, const unsigned short* __restrict__ g16) {
  __shared__ double red[LARS_WAVES];
  const int c = blockIdx.x;
  const ChunkRec rec = tb.chunk_rec[c];  // requested together with the header: garbage if the header is, but then unused
  const bool have_w = tb.state[0] != 0;  // written by the previous update, i.e. by an earlier launch
  if (!table_ok(tb)) return;
  const double sg = wave_sum(chunk_thread_sumsq_g(load_chunk_grads(rec, g16, threadIdx.x)));
  const double sw = have_w ? 0.0 : wave_sum(chunk_thread_sumsq_w(load_chunk_weights(rec, w, threadIdx.x)));
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = sg;
    if (!have_w) tb.psum_w[(size_t)c * LARS_WAVES + (threadIdx.x >> 6)] = sw;
  }
  lds_barrier();
  if (threadIdx.x == 0) tb.psum_g[c] = ((red[0] + red[1]) + red[2]) + red[3];
}

// The sums of a group of chunks for an update that works out the rates itself: it also finds the device-resident loss scale where
// it does not adjust it.
// 54 registers leave room for eight wavefronts a SIMD, two workgroups of 1024 threads a compute unit (with 71 and room for one AlexNet's update takes 224
// instead of 221 us): the first gradients are requested behind the sums of a fresh workspace; kept across them
// they spilled there (AlexNet's first call 74.9 us, 67.2 now).
template <int T>
__global__ __launch_bounds__(T) void lars_reduce_groups(Tables tb, const float* __restrict__ w, const unsigned short* __restrict__ g16,
                                                        const float* __restrict__ scale_dev) {
  __shared__ double red[2][T / 64];
  constexpr int U = 4, PIECES = LARS_CH / 8;     // 16-byte loads of a thread requested together; of a whole chunk
  const GroupRec gr = tb.group_rec[blockIdx.x];  // requested together with the header: garbage if the header is, but then unused
  const bool have_w = tb.state[0] != 0;          // written by the previous update, i.e. by an earlier launch
  if (!table_ok(tb)) return;
  const bool aligned = (gr.start & 7) == 0;
  double sw = 0.0, sg = 0.0;
  uint4 q[U];
  auto fetch = [&](int i) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = i + u * T;
      const int64_t at = gr.start + (int64_t)(p / PIECES * gr.stride) * LARS_CH + p % PIECES * 8;
      q[u] = make_uint4(0, 0, 0, 0);
      if (p < gr.chunks * PIECES && at + 8 <= gr.end) q[u] = *reinterpret_cast<const uint4*>(g16 + at);
    }
  };
  if (!have_w) {  // a fresh workspace: what the previous update would have left, chunk by chunk
    for (int j = (int)(threadIdx.x / LARS_THREADS); j < gr.chunks; j += T / LARS_THREADS) {
      const int c = gr.chunk0 + j * gr.stride;
      const double p = wave_sum(chunk_thread_sumsq_w(load_chunk_weights(tb.chunk_rec[c], w, threadIdx.x % LARS_THREADS)));
      if ((threadIdx.x & 63) == 0) tb.psum_w[(size_t)c * LARS_WAVES + (threadIdx.x % LARS_THREADS >> 6)] = p;
    }
    __threadfence_block();
    __syncthreads();
  }
  if (aligned) fetch(threadIdx.x);
  for (int i = threadIdx.x; i < gr.chunks * LARS_WAVES; i += T) {
    const double* const p = tb.psum_w + (size_t)(gr.chunk0 + i / LARS_WAVES * gr.stride) * LARS_WAVES + i % LARS_WAVES;
    // a fresh one's sums may share a line with a neighbour's that this compute unit has pulled in before they were written
    sw += have_w ? *p
                 : __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_AGENT));
  }
  if (aligned) {
    const int64_t end = gr.end & ~int64_t(7);  // the elements behind it belong to the tensor's last chunk
    if ((int)threadIdx.x < (int)(gr.end - end) && gr.end - gr.start <= ((int64_t)(gr.chunks - 1) * gr.stride + 1) * LARS_CH) {
      const float g = half_bits_to_float(g16[end + threadIdx.x]);
      sg = (double)(g * g);
    }
    for (int i = threadIdx.x; i < gr.chunks * PIECES; i += U * T) {
      uint4 now[U];
#pragma unroll
      for (int u = 0; u < U; ++u) now[u] = q[u];
      fetch(i + U * T);  // on its way while these squares are added
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const unsigned gw[4] = {now[u].x, now[u].y, now[u].z, now[u].w};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float g = half_bits_to_float((unsigned short)(gw[j >> 1] >> ((j & 1) * 16)));
          sg += (double)(g * g);
        }
      }
    }
  } else {
    for (int j = (int)(threadIdx.x / LARS_THREADS); j < gr.chunks; j += T / LARS_THREADS)
      sg += chunk_thread_sumsq_g(load_chunk_grads(tb.chunk_rec[gr.chunk0 + j * gr.stride], g16, threadIdx.x % LARS_THREADS));
  }
  sw = wave_sum(sw);
  sg = wave_sum(sg);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = sw;
    red[1][threadIdx.x >> 6] = sg;
  }
  if (scale_dev && blockIdx.x == 0 && threadIdx.x == 0) {
    const float scale = *scale_dev;
    tb.state[1] = __float_as_int(1.0f / scale);
    tb.state[2] = __float_as_int(scale);
  }
  lds_barrier();
  if (threadIdx.x == 0) {
    sw = red[0][0];
    sg = red[1][0];
#pragma unroll
    for (int i = 1; i < T / 64; ++i) {
      sw += red[0][i];
      sg += red[1][i];
    }
    tb.group_sum[blockIdx.x] = make_double2(sw, sg);
  }
}

// gamma rho_t of Eq. 1 on the un-scaled gradient
__device__ __forceinline__ float lars_rate(int flags, double sw, double sg, float lr, float eta, float loss_scale) {
  double rho = 1.0;
  if ((flags & JZ_PARAM_LARS) && sw > 0.0 && sg > 0.0) rho = (double)eta * sqrt(sw) / (sqrt(sg) / (double)loss_scale);
  return (float)((double)lr * rho);
}

// scale_dev != nullptr: the loss scale lives on the device (dynamic loss scaling) and replaces the argument
template <int THREADS>
__global__ __launch_bounds__(THREADS) void lars_finalize(Tables tb, float lr, float eta, float loss_scale,
                                                         const float* __restrict__ scale_dev) {
  __shared__ double red[THREADS / 64];
  if (scale_dev) loss_scale = *scale_dev;
  if (!table_ok(tb)) return;
  const int t = blockIdx.x;
  // the update kernel adjusts the device-resident scale itself, so its workgroups take 1/S from here instead
  if (scale_dev && t == 0 && threadIdx.x == 0) tb.state[1] = __float_as_int(1.0f / loss_scale);
  const int c0 = tb.chunk_begin[t], c1 = tb.chunk_begin[t + 1];
  double sw = 0.0, sg = 0.0;
  constexpr int U = LARS_FIN_BATCH;
  for (int c = c0 + (int)threadIdx.x; c < c1; c += U * THREADS) {
    double pw[U], pg[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int cj = c + j * THREADS;
      pw[j] = 0.0; pg[j] = 0.0;
      if (cj < c1) { pw[j] = chunk_sumsq_w(tb.psum_w, cj); pg[j] = tb.psum_g[cj]; }
    }
#pragma unroll
    for (int j = 0; j < U; ++j) { sw += pw[j]; sg += pg[j]; }
  }
  sw = block_sum<THREADS / 64>(sw, red);
  sg = block_sum<THREADS / 64>(sg, red);
  if (threadIdx.x == 0) {
    tb.coef[t] = lars_rate(tb.flags[t], sw, sg, lr, eta, loss_scale);
    tb.tflag[t] = sum_overflowed(sg) ? 1 : 0;
  }
}

// Start of a step on the presummed path, one workgroup per tensor (see the top of the file).
__global__ __launch_bounds__(LARS_THREADS) void lars_begin(Tables tb, const float* __restrict__ w,
                                                           const float* __restrict__ scale_dev) {
  __shared__ double red[LARS_WAVES];
  if (!table_ok(tb)) return;
  const int t = blockIdx.x;
  const bool have_w = tb.state[0] != 0;  // written by an earlier launch
  constexpr int SINK_WORDS = jz::kSumsqSubs * jz::kSumsqSubStride;
  for (int i = threadIdx.x; i < SINK_WORDS; i += LARS_THREADS) tb.gsum[(size_t)t * SINK_WORDS + i] = 0ull;
  if (threadIdx.x == 0) tb.gflag[t] = 0;
  if (scale_dev && t == 0 && threadIdx.x == 0) {  // the update adjusts the device-resident scale itself: it reads S from here
    const float S = *scale_dev;
    tb.state[1] = __float_as_int(1.0f / S);
    tb.state[2] = __float_as_int(S);
  }
  int c0 = tb.chunk_begin[t], c1 = tb.chunk_begin[t + 1];
  if (!have_w) {
    // Fresh workspace: leave in psum_w what lars_reduce would (same elements per thread, same order), chunk by chunk, so
    // that the sum below is the same bits whether the partial sums were carried or are recomputed here.  One workgroup
    // per tensor makes this slow for large tensors; it runs once per jz_lars_prepare.
    ChunkWeights next{};
    if (c0 < c1) next = load_chunk_weights(tb.chunk_rec[c0], w, threadIdx.x);
    for (int c = c0; c < c1; ++c) {
      const ChunkWeights now = next;
      if (c + 1 < c1) next = load_chunk_weights(tb.chunk_rec[c + 1], w, threadIdx.x);  // on its way while these are added
      const double p = wave_sum(chunk_thread_sumsq_w(now));
      if ((threadIdx.x & 63) == 0) tb.psum_w[(size_t)c * LARS_WAVES + (threadIdx.x >> 6)] = p;
    }
    __threadfence_block();
    __syncthreads();
  }
  c0 *= LARS_WAVES;
  c1 *= LARS_WAVES;
  // Loads that go past the compute unit's own cache: in the fresh case a partial sum written above may share a cache
  // line with a neighbouring tensor's, which another workgroup on this compute unit may have pulled in before the write.
  double sw = 0.0;
  if (have_w) {
    // carried sums, written by an earlier launch: plain loads, eight requested together, added in the same order as below
    for (int c = c0 + (int)threadIdx.x; c < c1; c += 8 * LARS_THREADS) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int cu = c + u * LARS_THREADS;
        v[u] = tb.psum_w[cu < c1 ? cu : c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c + u * LARS_THREADS < c1) sw += v[u];
    }
  } else {
    for (int c = c0 + (int)threadIdx.x; c < c1; c += LARS_THREADS)
      sw += __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(tb.psum_w + c),
                                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  }
  sw = block_sum<LARS_WAVES>(sw, red);
  if (threadIdx.x == 0) tb.wsum[t] = sw;
}

// The gradient reduce pass into the sinks, one workgroup per chunk, for chunks chunk0 .. chunk0 + gridDim.x - 1.
__global__ __launch_bounds__(LARS_THREADS) void lars_grad_sumsq(Tables tb, const unsigned short* __restrict__ g16, int chunk0) {
  __shared__ unsigned long long red[5];
  const int c = chunk0 + (int)blockIdx.x;
  const ChunkRec rec = tb.chunk_rec[c];
  if (!table_ok(tb)) return;
  if (threadIdx.x < 5) red[threadIdx.x] = 0ull;
  __syncthreads();
  int t;
  int64_t s, e, b0, b1;
  chunk_range(rec, &t, &s, &e);
  if (tb.flags[t] & JZ_PARAM_GRAD_PRESUMMED) return;  // its producer fills the sink
  chunk_body(s, e, &b0, &b1);
  jz::SumsqAcc sg;
  int bad = 0;
#pragma unroll
  for (int k = 0; k < LARS_IT; ++k) {
    int64_t i = b0 + (int64_t)(k * LARS_THREADS + threadIdx.x) * 8;
    if (i < b1) {
      const uint4 gq = *reinterpret_cast<const uint4*>(g16 + i);
      const unsigned gw[4] = {gq.x, gq.y, gq.z, gq.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) bad |= jz::sumsq_acc_add(sg, (unsigned short)(gw[j >> 1] >> ((j & 1) * 16)));
    }
  }
  {
    int64_t nh = b0 - s, nt = e - b1;
    int64_t k = threadIdx.x;
    if (k < nh + nt) bad |= jz::sumsq_acc_add(sg, g16[(k < nh) ? s + k : b1 + (k - nh)]);
  }
  jz::SumsqSink sink{tb.gsum + (size_t)t * (jz::kSumsqSubs * jz::kSumsqSubStride), tb.gflag + t};
  jz::sumsq_block_flush(sg, bad, sink, (unsigned)(c - tb.chunk_begin[t]), red);
}

// Dynamic loss scaling (Sections 4.1 and 5.3 name the loss scale; the policy is the usual skip / shrink / grow one).
struct DynScale {
  jz_loss_scale_state* st;  // nullptr: fixed loss scale
  float growth, backoff;
  int interval;
  float lo, hi;
};
__device__ __forceinline__ void loss_scale_step(const DynScale& d, int overflow) {
  float sc = d.st->scale;
  int good = d.st->good_steps;
  if (overflow) {
    sc = fmaxf(sc * d.backoff, d.lo);
    good = 0;
  } else if (++good >= d.interval) {
    sc = fminf(sc * d.growth, d.hi);
    good = 0;
  }
  d.st->scale = sc;
  d.st->good_steps = good;
}

__device__ __forceinline__ void lars_step(float& w, float& v, unsigned short gbits, float coef, float lam, float m,
                                          float inv_s, unsigned short& w16) {
  float g = half_bits_to_float(gbits) * inv_s;  // un-scale
  float u = fmaf(lam, w, g);                    // Eq. 2 differentiated: g + lambda*w
  float vn = fmaf(m, v, coef * u);              // momentum step with the local rate lr*rho
  float wn = w - vn;
  v = vn;
  w = wn;
  w16 = float_to_half_bits(wn);                 // cast back for the next forward pass
}

// One thread's share (tid of LARS_THREADS) of a chunk's state and gradients: every load is in flight before the first use.
// A lane takes four elements at a time, so that every access of a wavefront to weights or momentum is 1 KB without gaps.  With eight
// (two 16-byte accesses 32 bytes apart, each of which touches every line of 2 KB) the same stream, 20 bytes an element, ran at 5.35
// instead of 5.92 TB/s over 62 M elements.
struct ChunkState {
  float4 w[LARS_QUADS], v[LARS_QUADS];
  u32x2_t g[LARS_QUADS];
};
template <bool STREAM>
__device__ __forceinline__ ChunkState load_chunk_state(const ChunkRec& rec, int tid, const float* __restrict__ w, const float* __restrict__ v,
                                                       const unsigned short* __restrict__ g16) {
  ChunkState r;
  int t;
  int64_t s, e, b0, b1;
  chunk_range(rec, &t, &s, &e);
  chunk_body(s, e, &b0, &b1);
#pragma unroll
  for (int k = 0; k < LARS_QUADS; ++k) {
    int64_t i = b0 + (int64_t)(k * LARS_THREADS + tid) * 4;
    if (i < b1) {
      r.w[k] = load_state_f4<STREAM>(w + i);
      r.v[k] = load_state_f4<STREAM>(v + i);
      r.g[k] = *reinterpret_cast<const u32x2_t*>(g16 + i);
    }
  }
  return r;
}

// Its update; returns its share of the sum of squares of the new weights.
__device__ __forceinline__ double update_chunk(const ChunkState& q, const ChunkRec& rec, int tid, float* __restrict__ w, float* __restrict__ v,
                                               const unsigned short* __restrict__ g16, unsigned short* __restrict__ w16, float coef,
                                               float lam, float m, float inv_s) {
  int t;
  int64_t s, e, b0, b1;
  chunk_range(rec, &t, &s, &e);
  chunk_body(s, e, &b0, &b1);
  double sw = 0.0;  // sum of squares of the new weights, in the order lars_reduce would add them
#pragma unroll
  for (int k = 0; k < LARS_QUADS; ++k) {
    int64_t i = b0 + (int64_t)(k * LARS_THREADS + tid) * 4;
    if (i < b1) {
      float wv[4] = {q.w[k].x, q.w[k].y, q.w[k].z, q.w[k].w};
      float vv[4] = {q.v[k].x, q.v[k].y, q.v[k].z, q.v[k].w};
      unsigned ow[2];
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        const unsigned gw = q.g[k][j >> 1];
        unsigned short h0, h1;
        lars_step(wv[j], vv[j], (unsigned short)(gw & 0xffffu), coef, lam, m, inv_s, h0);
        lars_step(wv[j + 1], vv[j + 1], (unsigned short)(gw >> 16), coef, lam, m, inv_s, h1);
        ow[j >> 1] = (unsigned)h0 | ((unsigned)h1 << 16);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) sw = fma((double)wv[j], (double)wv[j], sw);
      store_stream_f4(w + i, wv[0], wv[1], wv[2], wv[3]);
      store_stream_f4(v + i, vv[0], vv[1], vv[2], vv[3]);
      store_stream_u2(w16 + i, ow[0], ow[1]);
    }
  }
  {
    int64_t nh = b0 - s, nt = e - b1;
    int64_t k = tid;
    if (k < nh + nt) {
      int64_t i = (k < nh) ? s + k : b1 + (k - nh);
      float wi = w[i], vi = v[i];
      unsigned short h;
      lars_step(wi, vi, g16[i], coef, lam, m, inv_s, h);
      w[i] = wi;
      v[i] = vi;
      w16[i] = h;
      sw = fma((double)wi, (double)wi, sw);
    }
  }
  return sw;
}

// PRE: the presummed path -- no lars_finalize ran; every wavefront forms its tensor's lr*rho_t itself (lr, eta and, for a
// fixed loss scale, S come as arguments) and the overflow flags are those of the sinks.
// 66 registers (78 where groups are summed here): seven wavefronts a SIMD (six).  Held to 64 for an eighth it spills eight of them, ResNet-50's update
// 107.6 -> 113.9 us, AlexNet's, which sums groups, the same.
template <int MODE, bool STREAM>
__global__ __launch_bounds__(LARS_THREADS) void lars_update(Tables tb, float* __restrict__ w, float* __restrict__ v,
                                                            const unsigned short* __restrict__ g16,
                                                            unsigned short* __restrict__ w16, float m, float wd,
                                                            float inv_s, int* __restrict__ found_inf, DynScale dyn,
                                                            float lr, float eta, float loss_scale) {
  constexpr bool PRE = MODE == LARS_PRE;
  if (dyn.st) {  // written by lars_finalize / lars_begin / lars_reduce_groups (not used when there is no tensor)
    inv_s = __int_as_float(tb.state[1]);
    if (MODE != LARS_PLAIN) loss_scale = __int_as_float(tb.state[2]);
  }
  // the header, this workgroup's chunk record and the tensor flags are requested together; nothing read through the
  // tables is used before the header has been checked
  const int cidx = (int)blockIdx.x < tb.n_chunks ? tb.n_chunks - 1 - (int)blockIdx.x : 0;
  const ChunkRec rec = tb.n_chunks > 0 ? tb.chunk_rec[cidx] : ChunkRec{0, 0, 0};
  int f = 0;  // every wavefront looks at all tensor flags (or group sums) itself
  double mw = 0.0, mg = 0.0;
  __shared__ double red[2][LARS_WAVES];
  __shared__ int red_f[LARS_WAVES];
  double2 gs[LARS_MAX_GROUPS / LARS_THREADS];
  int gt[LARS_MAX_GROUPS / LARS_THREADS];
  if constexpr (MODE == LARS_GROUPS) {  // is any gradient not finite, and what do this tensor's groups add up to
#pragma unroll
    for (int k = 0; k < LARS_MAX_GROUPS / LARS_THREADS; ++k) {
      const int i = k * LARS_THREADS + (int)threadIdx.x;
      gt[k] = -1;
      if (i < tb.n_groups) {
        gs[k] = tb.group_sum[i];
        gt[k] = tb.group_rec[i].tensor;
      }
    }
  } else {
    for (int t = threadIdx.x & 63; t < tb.T; t += 64) f |= PRE ? tb.gflag[t] : tb.tflag[t];
  }
  // PRE: this lane's share of the tensor's gradient sink (the tensor index is garbage if the header is: clamp it)
  // the first wavefront reads the sink (one quadruple per lane) and hands the total to the others through LDS
  __shared__ double sg_shared;
  unsigned long long d0 = 0, d1 = 0, d2 = 0, d3 = 0;
  double sw_t = 0.0;
  if (PRE && tb.n_chunks > 0) {
    const int ts = rec.tensor >= 0 && rec.tensor < tb.T ? rec.tensor : 0;
    static_assert(jz::kSumsqSubs == 64, "one counter quadruple per lane");
    if (threadIdx.x < 64) {
      const ulonglong2* a = reinterpret_cast<const ulonglong2*>(tb.gsum + ((size_t)ts * jz::kSumsqSubs + threadIdx.x) * jz::kSumsqSubStride);
      const ulonglong2 lo = a[0], hi = a[1];
      d0 = lo.x; d1 = lo.y; d2 = hi.x; d3 = hi.y;
    }
    sw_t = tb.wsum[ts];
  }
  if (!table_ok(tb)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *found_inf = -1;
    return;
  }
  ChunkState q;
  if constexpr (MODE == LARS_GROUPS) {
    q = load_chunk_state<STREAM>(rec, threadIdx.x, w, v, g16);  // on its way while the sums are added
#pragma unroll
    for (int k = 0; k < LARS_MAX_GROUPS / LARS_THREADS; ++k)
      if (gt[k] >= 0) {
        f |= sum_overflowed(gs[k].y) ? 1 : 0;
        if (gt[k] == rec.tensor) {
          mw += gs[k].x;
          mg += gs[k].y;
        }
      }
    mw = wave_sum(mw);
    mg = wave_sum(mg);
    f = __any(f);
    if ((threadIdx.x & 63) == 0) {
      red[0][threadIdx.x >> 6] = mw;
      red[1][threadIdx.x >> 6] = mg;
      red_f[threadIdx.x >> 6] = f;
    }
    lds_barrier();
    mw = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
    mg = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
    f = red_f[0] | red_f[1] | red_f[2] | red_f[3];
  } else {
    f = __any(f);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *found_inf = f ? 1 : 0;
    // skipped or not, psum_w describes the master weights as this launch leaves them: lars_reduce / lars_begin filled it in
    // for the weights as they were, and an update that goes through rewrites every chunk's sums
    tb.state[0] = 1;
    if (dyn.st) loss_scale_step(dyn, f);  // no workgroup of this launch reads dyn.st->scale
  }
  if (f) return;  // overflow under loss scaling: the step is skipped as a whole
  if ((int)blockIdx.x >= tb.n_chunks) return;
  const int c = cidx, t = rec.tensor;
  float coef;
  if (PRE) {
    if (threadIdx.x < 64) {  // integer sums: the order does not matter
      d0 = jz::wave_total_u64(d0);
      d1 = jz::wave_total_u64(d1);
      d2 = jz::wave_total_u64(d2);
      d3 = jz::wave_total_u64(d3);
      if (threadIdx.x == 63) sg_shared = jz::sumsq_value(d0, d1, d2, d3);
    }
    __syncthreads();  // every wavefront of the workgroup is here: the returns above depend on nothing wave-specific
    coef = lars_rate(tb.flags[t], sw_t, sg_shared, lr, eta, loss_scale);
  } else if (MODE == LARS_GROUPS) {
    coef = lars_rate(tb.flags[t], mw, mg, lr, eta, loss_scale);
  } else {
    coef = tb.coef[t];
  }
  const float lam = (tb.flags[t] & JZ_PARAM_WEIGHT_DECAY) ? wd : 0.0f;
  if constexpr (MODE != LARS_GROUPS) q = load_chunk_state<STREAM>(rec, threadIdx.x, w, v, g16);
  const double sw = wave_sum(update_chunk(q, rec, threadIdx.x, w, v, g16, w16, coef, lam, m, inv_s));
  if ((threadIdx.x & 63) == 0) tb.psum_w[(size_t)c * LARS_WAVES + (threadIdx.x >> 6)] = sw;
}

// The whole update of a small set in one launch of one workgroup: four groups of LARS_THREADS threads take the chunks in
// turn, the sums meet in LDS.  The same sums in the same order as the three launches.  What bounds it is three dependent
// round trips to memory (records, gradients, weights) and what one compute unit can move.
__global__ __launch_bounds__(1024) void lars_small(Tables tb, float* __restrict__ w, float* __restrict__ v,
                                                   const unsigned short* __restrict__ g16, unsigned short* __restrict__ w16, float m,
                                                   float wd, float inv_s, int* __restrict__ found_inf, DynScale dyn, float lr, float eta,
                                                   float loss_scale) {
  __shared__ double pg[LARS_SMALL_CHUNKS][LARS_WAVES], pw[LARS_SMALL_CHUNKS][LARS_WAVES];
  __shared__ float coef[LARS_SMALL_T];
  __shared__ int overflow;
  const int group = threadIdx.x / LARS_THREADS, tid = threadIdx.x % LARS_THREADS;
  const bool have_w = tb.state[0] != 0;
  if (dyn.st) {
    loss_scale = dyn.st->scale;
    inv_s = 1.0f / loss_scale;
  }
  if (!table_ok(tb)) {
    if (threadIdx.x == 0) *found_inf = -1;
    return;
  }
  if (threadIdx.x == 0) overflow = 0;
  for (int c = group; c < tb.n_chunks; c += 1024 / LARS_THREADS) {
    const ChunkRec rec = tb.chunk_rec[c];
    const double sg = wave_sum(chunk_thread_sumsq_g(load_chunk_grads(rec, g16, tid)));
    const double sw = have_w ? 0.0 : wave_sum(chunk_thread_sumsq_w(load_chunk_weights(rec, w, tid)));
    if ((tid & 63) == 0) {
      pg[c][tid >> 6] = sg;
      pw[c][tid >> 6] = sw;
      if (!have_w) tb.psum_w[(size_t)c * LARS_WAVES + (tid >> 6)] = sw;  // what a skipped update leaves
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < tb.T) {
    const int t = threadIdx.x;
    double sw = 0.0, sg = 0.0;
    for (int c = tb.chunk_begin[t]; c < tb.chunk_begin[t + 1]; ++c) {
      double cw;
      if (have_w) cw = chunk_sumsq_w(tb.psum_w, c);
      else cw = ((pw[c][0] + pw[c][1]) + pw[c][2]) + pw[c][3];
      sw += cw;
      sg += ((pg[c][0] + pg[c][1]) + pg[c][2]) + pg[c][3];
    }
    coef[t] = lars_rate(tb.flags[t], sw, sg, lr, eta, loss_scale);
    if (sum_overflowed(sg)) overflow = 1;
  }
  __syncthreads();
  const int f = overflow;
  if (threadIdx.x == 0) {
    *found_inf = f;
    tb.state[0] = 1;
    if (dyn.st) loss_scale_step(dyn, f);  // every thread has read the scale
  }
  if (f) return;
  for (int c = group; c < tb.n_chunks; c += 1024 / LARS_THREADS) {
    const ChunkRec rec = tb.chunk_rec[c];
    const float lam = (tb.flags[rec.tensor] & JZ_PARAM_WEIGHT_DECAY) ? wd : 0.0f;
    const double sw = wave_sum(update_chunk(load_chunk_state<false>(rec, tid, w, v, g16), rec, tid, w, v, g16, w16, coef[rec.tensor], lam, m, inv_s));
    if ((tid & 63) == 0) tb.psum_w[(size_t)c * LARS_WAVES + (tid >> 6)] = sw;
  }
}

__global__ void loss_scale_init(jz_loss_scale_state* __restrict__ st, float scale) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->scale = scale;
    st->good_steps = 0;
  }
}

Tables make_tables(const Layout& L, void* ws, uint64_t sum) {
  char* b = static_cast<char*>(ws);
  Tables tb;
  tb.header = reinterpret_cast<const uint64_t*>(b + L.off_header);
  tb.offsets = reinterpret_cast<const int64_t*>(b + L.off_offsets);
  tb.chunk_begin = reinterpret_cast<const int*>(b + L.off_chunk_begin);
  tb.flags = reinterpret_cast<const int*>(b + L.off_flags);
  tb.chunk_tensor = reinterpret_cast<const int*>(b + L.off_chunk_tensor);
  tb.chunk_rec = reinterpret_cast<const ChunkRec*>(b + L.off_chunk_rec);
  tb.state = reinterpret_cast<int*>(b + L.off_state);
  tb.psum_w = reinterpret_cast<double*>(b + L.off_psum_w);
  tb.psum_g = reinterpret_cast<double*>(b + L.off_psum_g);
  tb.coef = reinterpret_cast<float*>(b + L.off_coef);
  tb.tflag = reinterpret_cast<int*>(b + L.off_tflag);
  tb.gsum = reinterpret_cast<unsigned long long*>(b + L.off_gsum);
  tb.gflag = reinterpret_cast<int*>(b + L.off_gflag);
  tb.wsum = reinterpret_cast<double*>(b + L.off_wsum);
  tb.group_rec = reinterpret_cast<const GroupRec*>(b + L.off_group_rec);
  tb.group_sum = reinterpret_cast<double2*>(b + L.off_group_sum);
  tb.n_groups = (int)L.n_groups;
  tb.T = (int)L.T;
  tb.n_chunks = (int)L.n_chunks;
  tb.checksum = sum;
  return tb;
}

}  // namespace

extern "C" int jz_lars_workspace_bytes(const jz_param_set* ps, size_t* bytes) {
  if (!bytes) return JZ_ERR_NULL;
  Layout L;
  int rc = make_layout(ps, &L);
  if (rc != JZ_OK) return rc;
  *bytes = L.total;
  return JZ_OK;
}

extern "C" int jz_lars_prepare(const jz_param_set* ps, void* ws, size_t ws_bytes, void* hip_stream) {
  Layout L;
  int rc = make_layout(ps, &L);
  if (rc != JZ_OK) return rc;
  if (!ws || ws_bytes < L.total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(ws)) return JZ_ERR_ALIGN;
  std::vector<char> host(L.static_bytes, 0);
  uint64_t sum = table_checksum(ps);
  uint64_t* hdr = reinterpret_cast<uint64_t*>(host.data() + L.off_header);
  hdr[0] = LARS_MAGIC;
  hdr[1] = sum;
  hdr[2] = (uint64_t)L.T;
  hdr[3] = (uint64_t)L.n_chunks;
  hdr[4] = (uint64_t)L.P;
  int64_t* off = reinterpret_cast<int64_t*>(host.data() + L.off_offsets);
  int* cb = reinterpret_cast<int*>(host.data() + L.off_chunk_begin);
  int* fl = reinterpret_cast<int*>(host.data() + L.off_flags);
  int* ct = reinterpret_cast<int*>(host.data() + L.off_chunk_tensor);
  ChunkRec* cr = reinterpret_cast<ChunkRec*>(host.data() + L.off_chunk_rec);
  GroupRec* gr = reinterpret_cast<GroupRec*>(host.data() + L.off_group_rec);
  int c = 0;
  off[0] = 0;
  cb[0] = 0;
  for (int64_t t = 0; t < L.T; ++t) {
    off[t] = ps->offsets[t];
    off[t + 1] = ps->offsets[t + 1];
    fl[t] = ps->flags[t];
    int64_t n = ps->offsets[t + 1] - ps->offsets[t];
    int nc = (int)((n + LARS_CH - 1) / LARS_CH);
    for (int k = 0; k < nc; ++k) {
      ct[c + k] = (int)t;
      const int64_t st0 = ps->offsets[t] + (int64_t)k * LARS_CH;
      const int64_t en = st0 + LARS_CH < ps->offsets[t + 1] ? st0 + LARS_CH : ps->offsets[t + 1];
      cr[c + k] = ChunkRec{st0, (int)(en - st0), (int)t};
    }
    const int ng = (int)((nc + L.group_chunks - 1) / L.group_chunks);
    for (int k = 0; L.n_groups > 0 && k < ng; ++k) *gr++ = GroupRec{c + k, (nc - k + ng - 1) / ng, (int)t, ng, ps->offsets[t] + (int64_t)k * LARS_CH, ps->offsets[t + 1]};
    c += nc;
    cb[t + 1] = c;
  }
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (hipMemcpyAsync(ws, host.data(), L.static_bytes, hipMemcpyHostToDevice, st) != hipSuccess) return JZ_ERR_LAUNCH;
  if (hipStreamSynchronize(st) != hipSuccess) return JZ_ERR_LAUNCH;
  remember(ws, sum);
  return JZ_OK;
}

namespace {

// the update with a fixed loss scale (state == nullptr: hp->loss_scale) or with a device-resident one that the
// controller adjusts afterwards
int lars_run(const jz_param_set* ps, const jz_lars_hparams* hp, const jz_loss_scale_policy* pol, jz_loss_scale_state* state,
             int* found_inf_dev, void* ws, size_t ws_bytes, void* hip_stream, bool presummed = false) {
  if (!hp || !found_inf_dev) return JZ_ERR_NULL;
  Layout L;
  int rc = make_layout(ps, &L);
  if (rc != JZ_OK) return rc;
  if (!state && (!(hp->loss_scale > 0.0f) || !(hp->loss_scale < 3.0e38f))) return JZ_ERR_SHAPE;
  if (state) {
    if (!pol) return JZ_ERR_NULL;
    if (!(pol->growth_factor >= 1.0f) || !(pol->backoff_factor > 0.0f) || !(pol->backoff_factor <= 1.0f) ||
        pol->growth_interval < 1 || !(pol->min_scale > 0.0f) || !(pol->max_scale >= pol->min_scale) || !(pol->max_scale < 3.0e38f))
      return JZ_ERR_SHAPE;
    if (reinterpret_cast<uintptr_t>(state) & 7u) return JZ_ERR_ALIGN;
  }
  if (L.P > 0 && (!ps->master_w || !ps->momentum || !ps->grad16 || !ps->weight16)) return JZ_ERR_NULL;
  if (!ws || ws_bytes < L.total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(ws) || !jz::aligned16(ps->master_w) || !jz::aligned16(ps->momentum) ||
      !jz::aligned16(ps->grad16) || !jz::aligned16(ps->weight16) || (reinterpret_cast<uintptr_t>(found_inf_dev) & 3u))
    return JZ_ERR_ALIGN;
  const size_t P = (size_t)L.P;
  const void* bufs[4] = {ps->master_w, ps->momentum, ps->grad16, ps->weight16};
  const size_t lens[4] = {4 * P, 4 * P, 2 * P, 2 * P};
  for (int i = 0; i < 4; ++i) {
    if (jz::overlaps(bufs[i], lens[i], ws, L.total) || jz::overlaps(bufs[i], lens[i], found_inf_dev, sizeof(int)))
      return JZ_ERR_ALIAS;
    for (int j = i + 1; j < 4; ++j)
      if (jz::overlaps(bufs[i], lens[i], bufs[j], lens[j])) return JZ_ERR_ALIAS;
  }
  if (jz::overlaps(found_inf_dev, sizeof(int), ws, L.total)) return JZ_ERR_ALIAS;
  if (state) {
    if (jz::overlaps(state, sizeof(*state), ws, L.total) || jz::overlaps(state, sizeof(*state), found_inf_dev, sizeof(int)))
      return JZ_ERR_ALIAS;
    for (int i = 0; i < 4; ++i)
      if (jz::overlaps(bufs[i], lens[i], state, sizeof(*state))) return JZ_ERR_ALIAS;
  }
  uint64_t sum = table_checksum(ps);
  if (!is_prepared(ws, sum)) return JZ_ERR_NOT_PREPARED;
  // the presummed update consumes what jz_lars_begin_step set up (with the same loss-scale state) and the sinks filled since
  if (presummed && !has_begun(ws, state)) return JZ_ERR_NOT_PREPARED;

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  Tables tb = make_tables(L, ws, sum);
  const unsigned short* g16 = static_cast<const unsigned short*>(ps->grad16);
  const float* scale_dev = state ? &state->scale : nullptr;
  DynScale dyn{state, 1.0f, 1.0f, 1, 1.0f, 1.0f};
  if (state) dyn = DynScale{state, pol->growth_factor, pol->backoff_factor, pol->growth_interval, pol->min_scale, pol->max_scale};
  if (presummed) {
    set_begun(ws, false, nullptr);
    hipLaunchKernelGGL((L.P > LARS_STREAM_ELEMENTS ? lars_update<LARS_PRE, true> : lars_update<LARS_PRE, false>),
                       dim3((unsigned)(L.n_chunks > 0 ? L.n_chunks : 1)), dim3(LARS_THREADS), 0, st, tb, ps->master_w, ps->momentum, g16, static_cast<unsigned short*>(ps->weight16), hp->momentum,
                       hp->weight_decay, state ? 1.0f : 1.0f / hp->loss_scale, found_inf_dev, dyn, hp->lr, hp->trust_coef,
                       state ? 1.0f : hp->loss_scale);
    return jz::launch_status();
  }
  if (L.n_chunks <= LARS_SMALL_CHUNKS && L.T <= LARS_SMALL_T) {
    hipLaunchKernelGGL(lars_small, dim3(1), dim3(1024), 0, st, tb, ps->master_w, ps->momentum, g16,
                       static_cast<unsigned short*>(ps->weight16), hp->momentum, hp->weight_decay, state ? 1.0f : 1.0f / hp->loss_scale,
                       found_inf_dev, dyn, hp->lr, hp->trust_coef, state ? 1.0f : hp->loss_scale);
    return jz::launch_status();
  }
  if (L.n_groups > 0) {
    const dim3 groups((unsigned)L.n_groups);
    if (L.group_chunks == 1) hipLaunchKernelGGL(lars_reduce_groups<LARS_THREADS>, groups, dim3(LARS_THREADS), 0, st, tb, ps->master_w, g16, scale_dev);
    else hipLaunchKernelGGL(lars_reduce_groups<1024>, groups, dim3(1024), 0, st, tb, ps->master_w, g16, scale_dev);
    if ((rc = jz::launch_status()) != JZ_OK) return rc;
    hipLaunchKernelGGL((L.P > LARS_STREAM_ELEMENTS ? lars_update<LARS_GROUPS, true> : lars_update<LARS_GROUPS, false>), dim3((unsigned)L.n_chunks),
                       dim3(LARS_THREADS), 0, st, tb, ps->master_w, ps->momentum, g16, static_cast<unsigned short*>(ps->weight16), hp->momentum,
                       hp->weight_decay, state ? 1.0f : 1.0f / hp->loss_scale, found_inf_dev, dyn, hp->lr, hp->trust_coef,
                       state ? 1.0f : hp->loss_scale);
    return jz::launch_status();
  }
  if (L.n_chunks > 0) hipLaunchKernelGGL(lars_reduce, dim3((unsigned)L.n_chunks), dim3(LARS_THREADS), 0, st, tb, ps->master_w, g16);
  if (L.T > 0 && L.most_chunks <= 256 * LARS_FIN_BATCH)
    hipLaunchKernelGGL(lars_finalize<256>, dim3((unsigned)L.T), dim3(256), 0, st, tb, hp->lr, hp->trust_coef,
                       state ? 1.0f : hp->loss_scale, scale_dev);
  else if (L.T > 0)
    hipLaunchKernelGGL(lars_finalize<1024>, dim3((unsigned)L.T), dim3(1024), 0, st, tb, hp->lr, hp->trust_coef,
                       state ? 1.0f : hp->loss_scale, scale_dev);
  // at least one workgroup so that the flag is always written
  hipLaunchKernelGGL((L.P > LARS_STREAM_ELEMENTS ? lars_update<LARS_PLAIN, true> : lars_update<LARS_PLAIN, false>),
                     dim3((unsigned)(L.n_chunks > 0 ? L.n_chunks : 1)), dim3(LARS_THREADS), 0, st, tb, ps->master_w, ps->momentum, g16, static_cast<unsigned short*>(ps->weight16), hp->momentum,
                     hp->weight_decay, state ? 1.0f : 1.0f / hp->loss_scale, found_inf_dev, dyn, 0.0f, 0.0f, 1.0f);
  return jz::launch_status();
}

// what the entry points of the presummed path have in common: the table, the workspace and that it was prepared
int presummed_common(const jz_param_set* ps, void* ws, size_t ws_bytes, Layout* L, uint64_t* sum) {
  int rc = make_layout(ps, L);
  if (rc != JZ_OK) return rc;
  if (!ws || ws_bytes < L->total) return JZ_ERR_WORKSPACE;
  if (!jz::aligned16(ws)) return JZ_ERR_ALIGN;
  *sum = table_checksum(ps);
  if (!is_prepared(ws, *sum)) return JZ_ERR_NOT_PREPARED;
  return JZ_OK;
}

}  // namespace

extern "C" int jz_lars_mp_update(const jz_param_set* ps, const jz_lars_hparams* hp, int* found_inf_dev, void* ws,
                                 size_t ws_bytes, void* hip_stream) {
  return lars_run(ps, hp, nullptr, nullptr, found_inf_dev, ws, ws_bytes, hip_stream);
}

extern "C" int jz_lars_mp_update_dyn(const jz_param_set* ps, const jz_lars_hparams* hp, const jz_loss_scale_policy* policy,
                                     jz_loss_scale_state* state_dev, int* found_inf_dev, void* ws, size_t ws_bytes,
                                     void* hip_stream) {
  if (!state_dev) return JZ_ERR_NULL;
  return lars_run(ps, hp, policy, state_dev, found_inf_dev, ws, ws_bytes, hip_stream);
}

extern "C" int jz_lars_sumsq_sink(const jz_param_set* ps, void* ws, size_t ws_bytes, int64_t tensor, jz_sumsq_sink* sink) {
  if (!sink) return JZ_ERR_NULL;
  Layout L;
  uint64_t sum;
  int rc = presummed_common(ps, ws, ws_bytes, &L, &sum);
  if (rc != JZ_OK) return rc;
  if (tensor < 0 || tensor >= L.T) return JZ_ERR_SHAPE;
  static_assert(JZ_SUMSQ_SINK_BYTES == jz::kSumsqSinkBytes, "public and internal sink size");
  char* b = static_cast<char*>(ws);
  sink->sums = b + L.off_gsum + (size_t)tensor * jz::kSumsqSinkBytes;
  sink->nonfinite = reinterpret_cast<int*>(b + L.off_gflag) + tensor;
  return JZ_OK;
}

extern "C" int jz_lars_begin_step(const jz_param_set* ps, const jz_loss_scale_state* state_dev, void* ws, size_t ws_bytes,
                                  void* hip_stream) {
  Layout L;
  uint64_t sum;
  int rc = presummed_common(ps, ws, ws_bytes, &L, &sum);
  if (rc != JZ_OK) return rc;
  if (L.P > 0 && !ps->master_w) return JZ_ERR_NULL;
  if (!jz::aligned16(ps->master_w) || (reinterpret_cast<uintptr_t>(state_dev) & 7u)) return JZ_ERR_ALIGN;
  if (jz::overlaps(ps->master_w, 4 * (size_t)L.P, ws, L.total) || jz::overlaps(state_dev, sizeof(*state_dev), ws, L.total))
    return JZ_ERR_ALIAS;
  if (L.T > 0) {
    hipLaunchKernelGGL(lars_begin, dim3((unsigned)L.T), dim3(LARS_THREADS), 0, static_cast<hipStream_t>(hip_stream),
                       make_tables(L, ws, sum), ps->master_w, state_dev ? &state_dev->scale : nullptr);
    if ((rc = jz::launch_status()) != JZ_OK) return rc;
  }
  set_begun(ws, true, state_dev);
  return JZ_OK;
}

extern "C" int jz_lars_grad_sumsq(const jz_param_set* ps, int64_t first_tensor, int64_t num_tensors, void* ws, size_t ws_bytes,
                                  void* hip_stream) {
  Layout L;
  uint64_t sum;
  int rc = presummed_common(ps, ws, ws_bytes, &L, &sum);
  if (rc != JZ_OK) return rc;
  if (first_tensor < 0 || num_tensors < 0 || first_tensor + num_tensors > L.T) return JZ_ERR_SHAPE;
  if (L.P > 0 && !ps->grad16) return JZ_ERR_NULL;
  if (!jz::aligned16(ps->grad16)) return JZ_ERR_ALIGN;
  if (jz::overlaps(ps->grad16, 2 * (size_t)L.P, ws, L.total)) return JZ_ERR_ALIAS;
  int64_t c0 = 0, c1 = 0;  // chunks of tensors [first, first + num)
  for (int64_t t = 0; t < first_tensor + num_tensors; ++t) {
    const int64_t nc = (ps->offsets[t + 1] - ps->offsets[t] + LARS_CH - 1) / LARS_CH;
    if (t < first_tensor) c0 += nc;
    c1 += nc;
  }
  if (c1 > c0)
    hipLaunchKernelGGL(lars_grad_sumsq, dim3((unsigned)(c1 - c0)), dim3(LARS_THREADS), 0, static_cast<hipStream_t>(hip_stream),
                       make_tables(L, ws, sum), static_cast<const unsigned short*>(ps->grad16), (int)c0);
  return jz::launch_status();
}

extern "C" int jz_lars_mp_update_presummed(const jz_param_set* ps, const jz_lars_hparams* hp, int* found_inf_dev, void* ws,
                                           size_t ws_bytes, void* hip_stream) {
  return lars_run(ps, hp, nullptr, nullptr, found_inf_dev, ws, ws_bytes, hip_stream, true);
}

extern "C" int jz_lars_mp_update_presummed_dyn(const jz_param_set* ps, const jz_lars_hparams* hp,
                                               const jz_loss_scale_policy* policy, jz_loss_scale_state* state_dev,
                                               int* found_inf_dev, void* ws, size_t ws_bytes, void* hip_stream) {
  if (!state_dev) return JZ_ERR_NULL;
  return lars_run(ps, hp, policy, state_dev, found_inf_dev, ws, ws_bytes, hip_stream, true);
}

extern "C" int jz_loss_scale_init(jz_loss_scale_state* state_dev, float initial_scale, void* hip_stream) {
  if (!state_dev) return JZ_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(state_dev) & 7u) return JZ_ERR_ALIGN;
  if (!(initial_scale > 0.0f) || !(initial_scale < 3.0e38f)) return JZ_ERR_SHAPE;
  hipLaunchKernelGGL(loss_scale_init, dim3(1), dim3(64), 0, static_cast<hipStream_t>(hip_stream), state_dev, initial_scale);
  return jz::launch_status();
}
