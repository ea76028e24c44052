// Batch normalization of a whole tensor in one launch.  Included inside jz_bn.hip's anonymous namespace.
//
// The passes apart are bound by memory: forward they move 6 bytes an element, backward 12 (with the mask as bits), and the launch
// between them waits for the last workgroup and fills the chip anew.  Here one workgroup a compute unit keeps its rows in registers (FP16,
// 8 KB a pass) and LDS while the workgroups that share its 64 channels exchange their sums, so that a tensor of up to 43 passes = 90 MB
// forward, 25 = 52 MB backward with ReLU and 16 = 33 MB backward without or at a block's end is read once: 4 and 8 bytes an element.
// Rows beyond that are read again, with the mask's bits out of LDS.
// Measured, launches apart with their own plan (make_plan) and this, microseconds forward / backward with ReLU, in turn, different buffers:
//   3136 x 512    10.0 / 11.8    7.2 /  8.4        802816 x 64    53.0 / 119    43.8 / 93
//   12544 x 256   10.7 / 15.1    7.9 /  9.9        50176 x 512    29.0 / 65.0   23.8 / 44.0
//   12544 x 1024  16.9 / 38.6   13.4 / 24.8        200704 x 256   52.9 / 119    40.0 / 87.3
// ResNet-50's 53 layers at batch 64, both directions: 3.04 -> 2.22 ms.  What bounds it now: memory (5.1 TB/s read and written at
// 200704 x 256 forward, 4.7 backward with half of the rows kept) and, for short tensors, the launch and 3 us for the exchange.
// 64 channels are one 128-byte line of a row, the least that costs memory nothing; 512 threads are the fewest that can hold the register file.
#pragma once

constexpr int BW_WGS = 256;                      // workgroups at most: all of them run at the same time
constexpr int BW_U = 4;                          // passes beyond the kept ones whose loads are in flight together
constexpr int BW_UL = 2;                         // ... of the passes kept in LDS, and of rows taken over
constexpr int BW_Y = 2;                          // passes ahead of which y is requested: registers are what there is least of

typedef unsigned u32x4_bw __attribute__((ext_vector_type(4)));

struct BnWholeArgs {
  const uint4 *x = nullptr, *y = nullptr, *dy = nullptr, *dy2 = nullptr;  // y: the forward output (backward, ReLU mask)
  uint4 *out = nullptr, *g_out = nullptr;                                 // y forward, dx backward
  const float *gamma = nullptr, *beta = nullptr, *mean = nullptr, *invstd = nullptr;
  float *save_mean = nullptr, *save_invstd = nullptr;
  unsigned short *dgamma = nullptr, *dbeta = nullptr;
  double* part = nullptr;                // [slabs][2][C] sums
  unsigned long long* flags = nullptr;   // one a workgroup
  unsigned long long tag = 0;            // this launch's, two low bits clear
  long long wait_ticks = 0;              // of the 100 MHz clock: see look()
  int64_t rows = 0;
  int rows_per_wg = 0, C = 0, groups = 0, wgs = 0;  // groups of BW_CH channels, workgroups a group
  int relu = 0, in_place = 0;  // in_place: g_out is dy
  double inv_rows = 0;
  float eps = 0;
};

// what the flag of a workgroup's rows says in its two low bits, beside the launch's tag: someone has them in hand; their sums are there
enum { BW_CLAIMED = 1, BW_ARRIVED = 2 };
enum { BW_ALL_THERE = -1, BW_LOST = -2 };  // ends of the exchange, beside the rows to take over next
enum { BW_FWD, BW_GRAD, BW_RELU, BW_END };  // forward; backward of dy, of dy where y > 0, of RNE16(dy [+ dy2]) where y > 0

// Ties a value to its registers here.  The kept rows stay packed and their offsets are worked out again: left alone the compiler
// keeps the floats that the sums unpacked and an offset for every row, more registers than there are.
__device__ __forceinline__ void bw_pin(unsigned& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
}
__device__ __forceinline__ void bw_pin(uint4& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
#endif
}

__device__ __forceinline__ void bw_fence() {  // nothing is scheduled across
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// The wavefront's stores have been performed.  What workgroups tell each other goes through agent-scope atomics, which pass by
// the caches that are not shared; a store that has been performed is seen by every such load after it, so nothing has to be
// written back or thrown out: with release and acquire fences (which do that to a whole L2 each) the exchange took 20 us.
__device__ __forceinline__ void bw_performed() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}

__device__ __forceinline__ void bw_barrier() {  // orders accesses to LDS, waits for nothing else
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

// How the exchange ends.  A workgroup leaves its sums and its flag, then waits until all flags of its channels are there.  All
// workgroups fit the chip together, so on a chip of their own they do arrive.  Beside other streams some may not have started, and may not for
// as long as a kernel there holds a compute unit (a collective, another launch of this kernel).  So nobody waits for those: a workgroup whose time is
// up claims the rows of one that has not started, by one compare-and-swap on its flag, sums them out of memory in the order that their own
// workgroup would have, and looks again; when all sums are there it writes those rows' results too.  A workgroup that finds its flag claimed
// ends.  What is waited for is in the hands of a running workgroup, so every wait ends, and the bits do not depend on who did what.  Where
// the own workgroup is slow rather than absent both may sum the same rows, into the same bits, and the flag says who writes the results; only a block end
// in place, whose sums write g_out over dy, claims its rows before it starts (1 us more for short tensors).  So that slow ones are left alone the time to
// wait is what the own rows took, and 10 us.  Microseconds while another kernel holds one compute unit, forward / backward with ReLU: launches apart;
// waiting 100 us and leaving the rows of all to whoever comes last; this.
//   802816 x 64    55 / 103    3640 / 6770    84 / 164        50176 x 512    31 / 59    26 / 391    26 / 81
//   200704 x 256   55 / 103    1004 / 1210    78 / 150        12544 x 1024   19 / 38    13 / 199    14 / 56
// The flags need no clearing: they count only with the tag of this launch, 62 bits that no launch of the process had before.
// A captured graph would run the same tag again, so a capture takes the kernels in two launches.
template <int MODE, int K, int KL, int MASKS>
__global__ __launch_bounds__(BW_THREADS) void bn_whole(BnWholeArgs a) {
  constexpr bool GRAD = MODE != BW_FWD, NEEDS_Y = MODE == BW_RELU || MODE == BW_END;
  __shared__ __align__(16) float red[2][BW_THREADS][8];  // 32 KB: the lanes' sums, then the workgroups'
  __shared__ __align__(16) float coef[3][BW_CH];
  __shared__ unsigned short taken[BW_WGS];  // rows taken over
  __shared__ int next, owner;
  extern __shared__ __align__(16) uint4 kept[];  // [KL][x, and backward the gradient][lane]
  constexpr int TENSORS = GRAD ? 2 : 1;
  unsigned char* const mask = reinterpret_cast<unsigned char*>(kept + KL * TENSORS * BW_THREADS);  // [MASKS][lane]: y > 0 of a pass that is read again
  const int tid = threadIdx.x, chunk = tid & 7, rsub = tid >> 3;
  const int slab = blockIdx.x / a.groups, group = blockIdx.x % a.groups;
  const int c0 = group * BW_CH + chunk * 8;
  const unsigned pitch = (unsigned)a.C * 2u, step = pitch * BW_ROWS;

  struct Rows {  // the rows of one workgroup: descriptors that end with its last row, so that rows beyond it read as zeros and are not written
    __amdgpu_buffer_rsrc_t x, y, dy, dy2, out, g;
    int n;
  };
  auto rows_of = [&](int s) {
    const int64_t r0 = (int64_t)s * a.rows_per_wg;
    const int64_t left = a.rows - r0;
    Rows r;
    r.n = left < a.rows_per_wg ? (int)left : a.rows_per_wg;
    const int bytes = (int)((unsigned)r.n * pitch);
    const size_t off = (size_t)r0 * pitch;
    auto desc = [&](const void* p) { return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p + off), 0, p ? bytes : 0, 0x00020000); };
    r.x = desc(a.x);
    r.out = desc(a.out);
    if constexpr (GRAD) r.dy = desc(a.dy);
    if constexpr (NEEDS_Y) r.y = desc(a.y);
    if constexpr (MODE == BW_END) {
      r.dy2 = desc(a.dy2);
      r.g = desc(a.g_out);
    }
    return r;
  };
  auto get = [](__amdgpu_buffer_rsrc_t d, unsigned off) {
    const u32x4_bw v = __builtin_amdgcn_raw_buffer_load_b128(d, (int)off, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
  };
  auto put = [](__amdgpu_buffer_rsrc_t d, unsigned off, const uint4& v) {  // non-temporal, as store_streaming
    const u32x4_bw t = {v.x, v.y, v.z, v.w};
    __builtin_amdgcn_raw_buffer_store_b128(t, d, (int)off, 0, 2);
  };
  // the gradient behind the ReLU, FP16 (masking and the rounded sum are exact in it)
  auto masked = [&](const uint4& qd, const uint4& qy, const uint4& qe) {
    if constexpr (!NEEDS_Y) return qd;
    float gv[8], yv[8];
    unpack8(qd, gv);
    unpack8(qy, yv);
    if constexpr (MODE == BW_END)
      if (a.dy2) {
        float ev[8];
        unpack8(qe, ev);
#pragma unroll
        for (int e = 0; e < 8; ++e) gv[e] += ev[e];
      }
#pragma unroll
    for (int e = 0; e < 8; ++e) gv[e] = yv[e] > 0.f ? gv[e] : 0.f;
    return pack8(gv);
  };

  auto positive = [](const uint4& v) {  // bit e: element e > 0
    float f[8];
    unpack8(v, f);
    unsigned m = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) m |= f[e] > 0.f ? 1u << e : 0u;
    return (unsigned char)m;
  };
  auto masked_by = [](const uint4& v, unsigned m) {
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
    unsigned o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = w[i] & ((m >> (2 * i) & 1u ? 0xffffu : 0u) | (m >> (2 * i + 1) & 1u ? 0xffff0000u : 0u));
    return make_uint4(o[0], o[1], o[2], o[3]);
  };

  unsigned long long* const flags = a.flags + (size_t)group * a.wgs;
  const unsigned started = (unsigned)wall_clock64();
  unsigned long long stale = 0;  // what lies in the own flag: from before this launch, unless the rows have been claimed
  if (a.wgs > 1 && tid == 0) stale = __hip_atomic_load(flags + slab, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  auto claim = [&](int s, unsigned long long from, int as) {
    if ((from & ~3ull) == a.tag) return false;
    return __hip_atomic_compare_exchange_strong(flags + s, &from, a.tag | (unsigned long long)as, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };

  // ---- the workgroup's rows and their sums ---------------------------------------------------------------------------
  const Rows own = rows_of(slab);
  const unsigned voff = (unsigned)rsub * pitch + (unsigned)c0 * 2u;
  const int passes = (own.n + BW_ROWS - 1) / BW_ROWS;
  uint4 qx[K], qg[GRAD ? K : 1];
  float s0[8], s1[8], mu[8], is[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) s0[e] = s1[e] = mu[e] = is[e] = 0.f;
  auto add = [&](const uint4& x8, const uint4& g8) {
    float xv[8], gv[8];
    unpack8(x8, xv);
    if constexpr (GRAD) unpack8(g8, gv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (GRAD) {
        s0[e] += gv[e];
        s1[e] = fmaf(gv[e], (xv[e] - mu[e]) * is[e], s1[e]);
      } else {
        s0[e] += xv[e];
        s1[e] = fmaf(xv[e], xv[e], s1[e]);
      }
    }
  };
  if constexpr (GRAD) {
    load8(a.mean + c0, mu);
    load8(a.invstd + c0, is);
  }
  auto keep = [&](int k) {  // kept pass k has been added
    bw_pin(qx[k]);
    if constexpr (GRAD) bw_pin(qg[k]);
    bw_fence();
  };
  // everything that stays is requested at once; what only masks comes in behind it, BW_Y passes ahead of its use
  unsigned off = voff;
#pragma unroll
  for (int k = 0; k < K; ++k, off += step) {
    bw_pin(off);
    qx[k] = get(own.x, off);
    if constexpr (GRAD) qg[k] = get(own.dy, off);
  }
  if constexpr (NEEDS_Y) {
    uint4 y8[2][BW_Y], e8[2][BW_Y];
    unsigned off_g = voff;
    off = voff;
    auto request = [&](int b) {
#pragma unroll
      for (int u = 0; u < BW_Y; ++u, off += step) {
        bw_pin(off);
        y8[b][u] = get(own.y, off);
        if constexpr (MODE == BW_END) e8[b][u] = get(own.dy2, off);
      }
    };
    request(0);
    if constexpr (MODE == BW_END)
      if (a.in_place && a.wgs > 1) {
        if (tid == 0) owner = claim(slab, stale, BW_CLAIMED);
        bw_barrier();  // the loads stay in flight
        if (!owner) return;
      }
#pragma unroll
    for (int k = 0; k < K; k += BW_Y) {
      const int b = k / BW_Y % 2;
      if (k + BW_Y < K) request(b ^ 1);
#pragma unroll
      for (int u = 0; u < BW_Y; ++u) {
        qg[k + u] = masked(qg[k + u], y8[b][u], e8[b][u]);
        if constexpr (MODE == BW_END) {
          bw_pin(off_g);
          put(own.g, off_g, qg[k + u]);
          off_g += step;
        }
        add(qx[k + u], qg[k + u]);
        keep(k + u);
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      add(qx[k], qg[GRAD ? k : 0]);
      keep(k);
    }
  }
  enum { OWN, OWN_LDS, TAKEN };
  auto add_passes = [&](auto u_tag, auto whose_tag, const Rows& r, int p) {  // U passes from p on: the loads of all of them first
    constexpr int U = decltype(u_tag)::value, WHOSE = decltype(whose_tag)::value;
    uint4 x8[U], g8[U], y8[U], e8[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned o = voff + (unsigned)(p + u) * step;
      x8[u] = get(r.x, o);
      if constexpr (GRAD) g8[u] = get(r.dy, o);
      if constexpr (NEEDS_Y) y8[u] = get(r.y, o);
      if constexpr (MODE == BW_END) e8[u] = get(r.dy2, o);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      g8[u] = masked(g8[u], y8[u], e8[u]);
      if constexpr (MODE == BW_END) put(r.g, voff + (unsigned)(p + u) * step, g8[u]);
      if constexpr (WHOSE == OWN_LDS) {
        uint4* const slot = kept + (size_t)(p + u - K) * TENSORS * BW_THREADS + tid;
        slot[0] = x8[u];
        if constexpr (GRAD) slot[BW_THREADS] = g8[u];
      } else if constexpr (WHOSE == OWN && MASKS > 0) {
        if (p + u - K - KL < MASKS) mask[(p + u - K - KL) * BW_THREADS + tid] = positive(y8[u]);
      }
      add(x8[u], g8[u]);
    }
  };
  if constexpr (KL > 0) {
#pragma unroll 1
    for (int l = 0; l + BW_UL <= KL; l += BW_UL) add_passes(std::integral_constant<int, BW_UL>{}, std::integral_constant<int, OWN_LDS>{}, own, K + l);
    if constexpr (KL % BW_UL != 0) add_passes(std::integral_constant<int, 1>{}, std::integral_constant<int, OWN_LDS>{}, own, K + KL - 1);
  }
  for (int p = K + KL; p < passes; p += BW_U) add_passes(std::integral_constant<int, BW_U>{}, std::integral_constant<int, OWN>{}, own, p);
  // A lane's sums, of one in 64 of the workgroup's rows, are FP32; everything behind them is FP64, as in bn_stats for this plan's slabs.
  auto leave_sums = [&](int to) {
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      *reinterpret_cast<float4*>(&red[0][tid][e]) = make_float4(s0[e], s0[e + 1], s0[e + 2], s0[e + 3]);
      *reinterpret_cast<float4*>(&red[1][tid][e]) = make_float4(s1[e], s1[e + 1], s1[e + 2], s1[e + 3]);
    }
    __syncthreads();
    constexpr int SUMS = 2 * BW_CH, PARTS = BW_THREADS / SUMS;
    const int i = tid % SUMS, first = tid / SUMS;
    const float* p = &red[0][0][0] + (i < BW_CH ? i : BW_THREADS * 8 + i - BW_CH);  // [row of a pass][BW_CH]
    double t = 0;
    for (int j = first; j < BW_ROWS; j += PARTS) t += p[j * BW_CH];
    __syncthreads();
    double* const sums = reinterpret_cast<double*>(&red[0][0][0]);
    sums[first * SUMS + i] = t;
    __syncthreads();
    if (tid < SUMS) {
      t = 0;
#pragma unroll
      for (int k = 0; k < PARTS; ++k) t += sums[k * SUMS + tid];
      __hip_atomic_store(a.part + ((size_t)to * 2 + tid / BW_CH) * a.C + group * BW_CH + tid % BW_CH, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      bw_performed();
    }
    __syncthreads();  // also where no other workgroup has rows: two wavefronts have left the sums that any of them reads
  };
  leave_sums(slab);

  // ---- the exchange -----------------------------------------------------------------------------------------------------
  int n_taken = 0;
  bool first_rows = slab == 0;  // whoever has them writes what the call returns beside the tensor
  if (a.wgs > 1) {
    // the first wavefront looks, each lane at up to four flags: BW_ALL_THERE, or rows that it has claimed
    auto look = [&](unsigned since, unsigned patience) -> int {
      constexpr int F = BW_WGS / 64;
      for (;;) {
        unsigned long long v[F];
        bool all = true;
#pragma unroll
        for (int f = 0; f < F; ++f) {
          v[f] = a.tag | BW_ARRIVED;
          if (tid + 64 * f < a.wgs) v[f] = __hip_atomic_load(flags + tid + 64 * f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          all &= v[f] == (a.tag | BW_ARRIVED);
        }
        if (__all(all)) return BW_ALL_THERE;
        if ((unsigned)wall_clock64() - since >= patience) {
          unsigned long long absent[F];
          int n = 0;
#pragma unroll
          for (int f = 0; f < F; ++f) {
            absent[f] = __ballot((v[f] & ~3ull) != a.tag);
            n += __popcll(absent[f]);
          }
          if (n > 0) {  // one of them, another one for every workgroup that looks
            int rank = -(slab % n), won = 0;
#pragma unroll
            for (int f = 0; f < F; ++f) {
              const bool mine = rank + __popcll(absent[f] & ((1ull << tid) - 1ull)) == 0 && (absent[f] >> tid & 1ull) != 0;
              rank += __popcll(absent[f]);
              if (mine && claim(tid + 64 * f, v[f], BW_CLAIMED)) won = tid + 64 * f + 1;
            }
            const unsigned long long who = __ballot(won != 0);
            if (who != 0) return __shfl(won, __ffsll(who) - 1) - 1;
            continue;
          }
        }
        __builtin_amdgcn_s_sleep(1);
      }
    };
    unsigned since = 0, patience = 0;
    if (tid < 64) {
      int has = 1;
      if (tid == 0) {
        if (MODE == BW_END && a.in_place) __hip_atomic_store(flags + slab, a.tag | BW_ARRIVED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else has = claim(slab, stale, BW_ARRIVED);
      }
      has = __shfl(has, 0);
      since = (unsigned)wall_clock64();
      patience = a.wait_ticks > 0 ? (unsigned)a.wait_ticks + (since - started) : 0u;
      const int l = has ? look(since, patience) : (int)BW_LOST;
      if (tid == 0) next = l;
    }
    __syncthreads();
    int s;
    while ((s = next) >= 0) {
      if (tid == 0) taken[n_taken] = (unsigned short)s;
      ++n_taken;
      first_rows |= s == 0;
      const Rows r = rows_of(s);
#pragma unroll
      for (int e = 0; e < 8; ++e) s0[e] = s1[e] = 0.f;
      const int n = (r.n + BW_ROWS - 1) / BW_ROWS;
      for (int p = 0; p < n; p += BW_UL) add_passes(std::integral_constant<int, BW_UL>{}, std::integral_constant<int, TAKEN>{}, r, p);
      leave_sums(s);
      if (tid < 64) {
        if (tid == 0) __hip_atomic_store(flags + s, a.tag | BW_ARRIVED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int l = look(since, patience);
        if (tid == 0) next = l;
      }
      __syncthreads();
    }
    if (s == BW_LOST) return;
  }

  // ---- the channels' totals, FP64, in bn_slab_totals' order -----------------------------------------------------------
  double* const tot = reinterpret_cast<double*>(&red[0][0][0]);  // [lane][2 * BW_CH]
  {
    constexpr int Q = 2 * BW_CH / 2, OWN = BN_FIN_LANES / (BW_THREADS / Q), IN_FLIGHT = 2, LANES = BN_FIN_LANES / OWN;
    const int q = tid % Q, j = tid / Q;  // two channels' first or second sums, lanes j, j + 8, j + 16 and j + 24 of them
    // past the last workgroup's sums the loads return zeros; device scope, like the stores: they pass by the caches that are not shared
    constexpr int DEVICE_SCOPE = 16;
    const __amdgpu_buffer_rsrc_t sums = __builtin_amdgcn_make_buffer_rsrc((void*)a.part, 0, (int)((unsigned)a.wgs * (unsigned)a.C * 16u), 0x00020000);
    const unsigned slab_bytes = (unsigned)a.C * 16u, at = (unsigned)(q / (Q / 2)) * ((unsigned)a.C * 8u) + (unsigned)(group * BW_CH + q % (Q / 2) * 2) * 8u;
    double t[OWN][2];
#pragma unroll
    for (int o = 0; o < OWN; ++o) t[o][0] = t[o][1] = 0.0;
    for (int k = j; k < a.wgs; k += BN_FIN_LANES * IN_FLIGHT) {
      u32x4_bw v[IN_FLIGHT * OWN];
#pragma unroll
      for (int u = 0; u < IN_FLIGHT * OWN; ++u) v[u] = __builtin_amdgcn_raw_buffer_load_b128(sums, (int)(at + (unsigned)(k + u * LANES) * slab_bytes), 0, DEVICE_SCOPE);
#pragma unroll
      for (int u = 0; u < IN_FLIGHT * OWN; ++u) {
        t[u % OWN][0] += __hiloint2double((int)v[u].y, (int)v[u].x);
        t[u % OWN][1] += __hiloint2double((int)v[u].w, (int)v[u].z);
      }
    }
    __syncthreads();
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int e = 0; e < 2; ++e) tot[(j + o * LANES) * (2 * BW_CH) + q * 2 + e] = t[o][e];
    __syncthreads();
    if (tid < 2 * BW_CH) {
      double sum = 0.0;
      for (int l0 = 0; l0 < bn_lanes(a.wgs); l0 += 8) {  // eight read together; lanes beyond the workgroups hold zeros
        double v[8];
#pragma unroll
        for (int l = 0; l < 8; ++l) v[l] = tot[(l0 + l) * (2 * BW_CH) + tid];
#pragma unroll
        for (int l = 0; l < 8; ++l) sum += v[l];
      }
      tot[tid] = sum;
    }
    __syncthreads();
  }
  auto finish = [&](bool writer) {  // the coefficients; the workgroup of the first rows also writes what the call returns beside the tensor
    if (tid < BW_CH) {
      const int c = group * BW_CH + tid;
      if constexpr (GRAD)
        bn_bwd_coef(tot[tid], tot[BW_CH + tid], a.inv_rows, a.gamma[c], a.mean[c], a.invstd[c], writer ? a.dgamma + c : nullptr,
                    writer ? a.dbeta + c : nullptr, &coef[0][tid], BW_CH);
      else
        bn_fwd_coef(tot[tid], tot[BW_CH + tid], a.inv_rows, a.eps, a.gamma[c], a.beta[c], writer ? a.save_mean + c : nullptr,
                    writer ? a.save_invstd + c : nullptr, &coef[0][tid], BW_CH);
    }
    __syncthreads();
  };
  finish(first_rows);

  // ---- the results ------------------------------------------------------------------------------------------------------
  float ca[8], cb[8], cq[8];
  load8(&coef[0][chunk * 8], ca);
  load8(&coef[1][chunk * 8], cb);
  if constexpr (GRAD) load8(&coef[2][chunk * 8], cq);
  auto result = [&](const uint4& x8, const uint4& g8) {
    float xv[8], o[8];
    unpack8(x8, xv);
    if constexpr (GRAD) {
      float gv[8];
      unpack8(g8, gv);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = bn_dx(ca[e], gv[e], cb[e], xv[e], cq[e]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float z = fmaf(xv[e], ca[e], cb[e]);
        o[e] = (a.relu && !(z > 0.f)) ? 0.f : z;
      }
    }
    return pack8(o);
  };
  // passes from p on of a workgroup's rows out of memory.  Its own are masked already, by bits; a block end's are in g_out, also those taken
  // over (g_out may be dy, which is gone then)
  auto stream = [&](const Rows& r, int p, auto own_tag) {
    constexpr bool IS_OWN = decltype(own_tag)::value;
    const int n = (r.n + BW_ROWS - 1) / BW_ROWS;
    for (; p < n; p += BW_U) {
      uint4 x8[BW_U], g8[BW_U], y8[BW_U];
      const bool bits = IS_OWN && MASKS > 0 && p + BW_U - 1 - K - KL < MASKS;
#pragma unroll
      for (int u = 0; u < BW_U; ++u) {
        const unsigned o = voff + (unsigned)(p + u) * step;
        x8[u] = get(r.x, o);
        if constexpr (MODE == BW_END) {
          g8[u] = get(r.g, o);
        } else {
          if constexpr (GRAD) g8[u] = get(r.dy, o);
          if constexpr (NEEDS_Y)
            if (!bits) y8[u] = get(r.y, o);
        }
      }
#pragma unroll
      for (int u = 0; u < BW_U; ++u) {
        if constexpr (MODE != BW_END) {
          if (bits) g8[u] = masked_by(g8[u], mask[(p + u - K - KL) * BW_THREADS + tid]);
          else g8[u] = masked(g8[u], y8[u], g8[u]);
        }
        put(r.out, voff + (unsigned)(p + u) * step, result(x8[u], g8[u]));
      }
    }
  };
  stream(own, K + KL, std::true_type{});  // what was read last first: it is the likeliest to be in a cache
  if constexpr (KL > 0) {
#pragma unroll 1
    for (int l = 0; l < KL; ++l) {
      const uint4* const slot = kept + (size_t)l * TENSORS * BW_THREADS + tid;
      put(own.out, voff + (unsigned)(K + l) * step, result(slot[0], slot[GRAD ? BW_THREADS : 0]));
    }
  }
  off = voff;
#pragma unroll
  for (int k = 0; k < K; ++k, off += step) {
    bw_pin(off);
    put(own.out, off, result(qx[k], qg[GRAD ? k : 0]));
    bw_fence();
  }
  for (int i = 0; i < n_taken; ++i) stream(rows_of(taken[i]), 0, std::false_type{});
}
