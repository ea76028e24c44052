// Implicit GEMM of a convolution whose output grid is its input grid (unit stride, odd filter, "same" padding), forward and
// backward-data, with the input window of a tile kept in LDS.  Included by jz_conv_window_fwd.hip and jz_conv_window_bwd_data.hip behind jz_igemm_kernels.h.
//
// igemm_dma_kernel brings the gathered operand in once per filter tap: nine times for a 3x3 layer, and the path from L2 into LDS is what
// bounds those layers.  Here the BM pixels of a tile, which are consecutive in memory, and the pixels that their taps reach (a run of
// BM + (R-1) W + S-1 pixels, since every tap is a constant distance away) are brought in once per CK channels, and every tap
// reads its rows out of that run at its own distance.  Only the filter still goes through a ring, one (channels, tap) tile after another.
// Rows whose tap lies outside the image read a row of zeros instead: one bit per row and tap, as in the ring kernel.
//
//   LDS: NPB windows of PR rows | 1 KB of zeros | NST filter tiles.  A row is CK channels; chunk c of a row at LDS address x sits at
//   position c ^ ((x >> 8) & (CK / 8 - 1)), which sends any 16 consecutive rows' copies of a chunk to 16 different 16-byte bank groups.
//   While the taps of one block of channels are multiplied the window of the next comes in, PA loads a k tile; loads that are not needed
//   go to the zeros, out of range, so that every k tile requests the same number and the waits can count them.
//
// The reduction runs channel blocks outside, taps inside (the ring kernel: taps outside), in FP32 as there.
//
// Measured, ring kernel and this, microseconds forward / backward-data (different buffers in turn):
//   64 -> 64, 3x3, 64 x 56 x 56    31.4 / 31.0 23.3 / 25.1    128 -> 128, 3x3, 64 x 28 x 28     20.5 / 22.1   19.6 / 21.0
//   64 -> 64, 3x3, 32 x 56 x 56    19.5 / 18.2 13.0 / 13.9    384 -> 384, 3x3, 128 x 13 x 13    59.3 / 65.2   55.9 / 58.9
//   96 -> 256, 5x5, 128 x 27 x 27, backward-data   179 ... 184   167 ... 171 (256 channels read: the ring kernel's 128x128 tiles are 3 rounds)
// What bounds it now.  256x128 tiles: waits inside the loop, not the matrix pipes: over the 3x3 layers of 256 and 384 channels at 13 x 13 products
// are 57 % (forward) and 55 % (backward-data) of the compute units' busy cycles by counters, 54 % in the ring kernel.  256x64 tiles: two workgroups a
// compute unit, 3.06 rounds of work in four, and each waits for its window before its first product.
// Tried: wavefronts in two groups that share the reduction, with 128x64 of the tile each (a quarter fewer LDS reads, and one exchange of sums):
// 384 channels 51 -> 54 us, 128 channels 18.8 -> 22.5; 128x128 tiles (256 channels, 64 x 14 x 14: 20.1 us on eight wavefronts, 21.4 on four, the ring
// kernel 19.5); 64x128 and 128x64 tiles for small layers (9 ... 30 % slower than the ring kernel); blocks of 32 channels (0.93 ... 1.4).
#pragma once

namespace {

template <int OP_ARG, int BM, int BN, int CK, int NST, int PR, int NPB, int WGM, int WGN>
struct WindowShape {
  static constexpr int NT = 64 * WGM * WGN, RB = 2 * CK, CR = CK / 8;
  static constexpr int WIN = PR * RB, ZERO = NPB * WIN, RING = ZERO + 1024, STAGE = BN * RB;
  static constexpr int ring_bytes = RING + NST * STAGE;
  static constexpr int epi_bytes = BM / dma_epass(BM, BN) * (BN + 8) * 2;
  static constexpr int LDS = ring_bytes > epi_bytes ? ring_bytes : epi_bytes;
};

template <int OP_ARG, int BM, int BN, int CK, int NST, int PR, int NPB, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void conv_window(GemmArgs a) {
  constexpr int STATS = OP_ARG == OP_FWD_STATS ? 1 : (OP_ARG == OP_BWD_DATA_STATS ? 2 : (OP_ARG == OP_BWD_DATA_BLOCK_END ? 3 : 0));
  constexpr int OP = STATS == 1 ? OP_FWD : (STATS >= 2 ? OP_BWD_DATA : OP_ARG);
  using Shape = WindowShape<OP_ARG, BM, BN, CK, NST, PR, NPB, WGM, WGN>;
  constexpr bool B_KC = OP == OP_FWD;
  constexpr int NW = WGM * WGN, NT = 64 * NW;
  constexpr int WTM = BM / WGM, WTN = BN / WGN, TM = WTM / 32, TN = WTN / 32;
  constexpr int NKS = CK / 16, G = TM * TN, RB = Shape::RB, CR = Shape::CR;
  constexpr int RPI = 64 / CR;                    // rows of one load
  constexpr int LP = PR / (RPI * NW);             // loads per thread and window
  constexpr int PA = NPB == 1 ? 0 : (LP + 9 - NST + 1) / (9 - NST + 2);  // ... per k tile: in by the last but NST - 2 of nine taps
  constexpr int LB = BN * CR / NT, LPT = PA + LB;
  static_assert(LP * RPI * NW == PR && LB * NT == BN * CR && LB >= 1, "loads divide among the threads");
  static_assert(Shape::WIN % 2048 == 0, "the swizzle is the same in every window");
  static_assert(TM * 32 * WGM == BM && TN * 32 * WGN == BN && TM <= G && NST >= 3 && NKS >= 2, "tile");
  extern __shared__ __align__(16) unsigned short lds[];
  lds_byte* const ldsb = (lds_byte*)lds;
  const unsigned lds_base = (unsigned)(uintptr_t)JZ_LDS_PTR(lds);
  constexpr unsigned OOB = 0xffffffffu;

  const ConvGeom& g = a.g;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  unsigned L = xcd_remap(blockIdx.x, gridDim.x);
  const int tiles_mn = a.tiles_m * a.tiles_n;
  const int split = (int)fd_div(L, a.d_tiles_mn);
  L -= (unsigned)split * (unsigned)tiles_mn;
  const unsigned trow = fd_div(L, a.d_tiles_n);
  const int m0 = (int)trow * BM;
  const int n0 = (int)(L - trow * (unsigned)a.tiles_n) * BN;
  const int taps = g.R * g.S;
  const int kt_begin = split * a.kt_per_split;  // a multiple of the taps
  const int kt_end = kt_begin + a.kt_per_split < a.nkt ? kt_begin + a.kt_per_split : a.nkt;
  const int nk = kt_end - kt_begin;
  const int c_begin = kt_begin / taps * CK, c_end = kt_end / taps * CK;  // channels

  const __amdgpu_buffer_rsrc_t rsrcA = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, (int)a.bytesA, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB = __builtin_amdgcn_make_buffer_rsrc((void*)a.B, 0, (int)a.bytesB, 0x00020000);

  // ---- loads -----------------------------------------------------------------------------------
  // window row ii * NW * RPI + row0; rows that no tap reaches are not requested, pixels before and behind the tensor are out of range
  const int row0 = wave * RPI + lane / CR;
  const int chunk = (lane % CR) ^ (int)((unsigned)(row0 * RB) >> 8 & (CR - 1));
  const unsigned pitch = (unsigned)g.IC * 2u;
  const unsigned vP = (unsigned)row0 * pitch + (unsigned)chunk * 16u;
  const unsigned win_first = (unsigned)(m0 - g.ph * g.IW - g.pw) * pitch;
  const unsigned win_bytes = (unsigned)(BM + (g.R - 1) * g.IW + g.S - 1) * pitch;
  unsigned vB[LB];
  auto mc_k = [&](int ii) { constexpr int cpr = BN / 8; return (NW * ii + wave) * (64 / cpr) + lane / cpr; };
#pragma unroll
  for (int ii = 0; ii < LB; ++ii) {
    if (B_KC) {
      const int nn = n0 + NW * RPI * ii + row0;
      vB[ii] = nn < a.N ? (unsigned)(nn * a.Kred + chunk * 8) * 2u : OOB;
    } else {
      constexpr int cpr = BN / 8;
      const int k = mc_k(ii), nn = n0 + ((lane % cpr) ^ (cpr >= 16 ? 4 * (k & 3) : 2 * (k & 3))) * 8;
      vB[ii] = nn < a.N ? (unsigned)((k * taps) * a.N + nn) * 2u : OOB;
    }
  }
  auto load_window = [&](int buf, int c0, int ii, bool wanted) {
    const unsigned at = vP + (unsigned)(NW * RPI * ii) * pitch;
    const unsigned dst = wanted ? (unsigned)(buf * Shape::WIN + (NW * ii + wave) * 1024) : (unsigned)Shape::ZERO;
    jz_dma16s(rsrcA, ldsb + dst, at < (wanted ? win_bytes : 0u) ? at + win_first : OOB, (unsigned)c0 * 2u);
  };
  auto load_zeros = [&] { jz_dma16(rsrcA, ldsb + Shape::ZERO, OOB); };
  auto load_filter = [&](int st, int c0, int tap, auto ii_tag) {
    constexpr int ii = decltype(ii_tag)::value;
    const unsigned soff = B_KC ? (unsigned)(tap * g.IC + c0) * 2u : (unsigned)((c0 * taps + tap) * a.N) * 2u;
    jz_dma16s(rsrcB, ldsb + Shape::RING + st * Shape::STAGE + (NW * ii + wave) * 1024, vB[ii], soff);
  };

  load_zeros();
  static_for<0, LP>([&](auto ii) { load_window(0, c_begin, ii, true); });
#pragma unroll
  for (int s = 0; s < NST - 1; ++s) {  // at least nine k tiles
    static_for<0, PA>([&](auto) { load_zeros(); });
    static_for<0, LB>([&](auto ii) { load_filter(s, c_begin, s, ii); });
  }
  sched_fence();

  // ---- operand reads -----------------------------------------------------------------------------
  const int r31 = lane & 31, hi = lane >> 5;
  unsigned base[TM], inv[TM], adA[TM], adB[B_KC ? NKS : 2 * TN];
  const unsigned zero_at = lds_base + Shape::ZERO;
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int row = wm * WTM + 32 * t + r31, m = m0 + row;
    base[t] = lds_base + (unsigned)(row * RB);
    inv[t] = OOB;
    if (m < a.M) {
      const unsigned rem = (unsigned)m - fd_div((unsigned)m, g.d_ohow) * (unsigned)(g.OH * g.OW);
      const int oh = (int)fd_div(rem, g.d_ow), ow = (int)rem - oh * g.OW;
      // taps outside the image are a run at the start and one at the end along each axis, see igemm_dma_body
      constexpr int dir = OP == OP_FWD ? 1 : -1;
      const int ih0 = oh - dir * g.ph, iw0 = ow - dir * g.pw;
      const int lo_w = dir > 0 ? -iw0 : iw0 - g.IW + 1, hi_w = dir > 0 ? g.IW - iw0 : iw0 + 1;
      const int lo_h = dir > 0 ? -ih0 : ih0 - g.IH + 1, hi_h = dir > 0 ? g.IH - ih0 : ih0 + 1;
      const unsigned full = low_bits(g.S);
      const unsigned cm = low_bits(clamp_to(lo_w, g.S)) | (full & ~low_bits(clamp_to(hi_w, g.S)));
      inv[t] = cm * g.tap_rep | low_bits(clamp_to(lo_h, g.R) * g.S) | (low_bits(g.R * g.S) & ~low_bits(clamp_to(hi_h, g.R) * g.S));
    }
  }
  if (B_KC) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int row = wn * WTN + r31;
      adB[ks] = (unsigned)(row * RB + (((2 * ks + hi) ^ (int)((unsigned)(row * RB) >> 8 & (CR - 1))) * 16));
    }
  } else {
    constexpr int CPR = BN / 8;
    const int gi = lane >> 4, j = (lane >> 2) & 3, c4 = lane & 3;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const int k = 8 * (gi >> 1) + 4 * hf + j, c = (wn * WTN + 32 * t + 16 * (gi & 1) + 4 * c4) / 8;
        const int swz = CPR >= 16 ? 4 * (k & 3) : 2 * (k & 3);
        adB[t * 2 + hf] = (unsigned)(k * (BN * 2) + ((c ^ swz) * 16) + (c4 & 1) * 8);
      }
  }
  // where k step 0 of a tap is read; step ks flips bits 5 and 6.  dist: the tap's distance (and window) in bytes
  auto aim = [&](int t, unsigned dist, unsigned tap) {
    const unsigned row = base[t] + dist;
    const unsigned at = (row | (row >> 4 & (16u * (CR - 1)))) ^ (unsigned)(hi << 4);
    const unsigned bad = (unsigned)__builtin_amdgcn_sbfe(inv[t], tap, 1);
    adA[t] = (zero_at & bad) | (at & ~bad);
  };
  auto read_frags = [&](unsigned sb, auto ks_tag, half8 (&fa)[TM], half8 (&fb)[TN]) {
    constexpr int KS = decltype(ks_tag)::value;
#pragma unroll
    for (int t = 0; t < TM; ++t) fa[t] = lds_read_b128<0>(adA[t] ^ (unsigned)(KS << 5));
    if constexpr (B_KC) {
      fb[0] = lds_read_b128<0>(sb + adB[KS]);
      if constexpr (TN > 1) fb[1] = lds_read_b128<32 * RB>(sb + adB[KS]);
      if constexpr (TN > 2) fb[2] = lds_read_b128<64 * RB>(sb + adB[KS]);
      if constexpr (TN > 3) fb[3] = lds_read_b128<96 * RB>(sb + adB[KS]);
    } else {
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        half4v lo = lds_read_tr16_b64<KS * 16 * BN * 2>(sb + adB[t * 2]);
        half4v hv = lds_read_tr16_b64<KS * 16 * BN * 2>(sb + adB[t * 2 + 1]);
        fb[t] = __builtin_shufflevector(lo, hv, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    }
  };
  constexpr int READS = TM + (B_KC ? TN : 2 * TN);
  static_assert(READS <= 15, "lgkmcnt is a 4-bit counter");

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  auto wait_tiles = [&](int younger) {  // younger k tiles still in flight
    if (younger >= NST - 2) wait_vmcnt<(NST - 2) * LPT>();
    else if (NST - 2 > 1 && younger == 1) wait_vmcnt<LPT>();
    else wait_vmcnt<0>();
  };
  static_assert(NST <= 4, "wait_tiles");

  // ---- the loop: igemm_dma_body's, with the window's loads ahead of the filter's -----------------------------------
  constexpr int SPG = G > 1 ? G - 1 : 1, NSL = NKS * SPG;
  constexpr int LBAR = []() constexpr {
    int n = 0;
    for (int l = 0; l < LPT; ++l) n += ((l * NSL / LPT) / SPG <= NKS - 2) ? 1 : 0;
    return n;
  }();
  static_assert((NST - 3) * LPT + LBAR <= 63, "vmcnt range");
  // the k tile being multiplied, the one after it, and the one whose filter is requested
  struct At {
    int c0, tap, r, s, win;
  };
  auto advance = [&](At& p) {
    ++p.tap;
    if (++p.s == g.S) {
      p.s = 0;
      ++p.r;
    }
    if (p.tap == taps) {
      p.tap = p.r = 0;
      p.c0 += CK;
      p.win ^= NPB - 1;
    }
  };
  auto distance = [&](const At& p) {
    const int r = OP == OP_FWD ? p.r : g.R - 1 - p.r, s = OP == OP_FWD ? p.s : g.S - 1 - p.s;
    return (unsigned)(p.win * Shape::WIN + (r * g.IW + s) * RB);
  };
  At cur{c_begin, 0, 0, 0, 0}, next = cur, req{c_begin, NST - 1, 0, 0, 0};
  half8 fa0[TM], fb0[TN], fa1[TM], fb1[TN];
  auto iteration = [&](int st, auto steady_tag, int ist, bool has_next, int younger_after_next) {
    constexpr bool ISSUE = decltype(steady_tag)::value;
    const unsigned sb = lds_base + (unsigned)(Shape::RING + st * Shape::STAGE);
    const int st1 = st + 1 == NST ? 0 : st + 1;
    const unsigned sb_next = lds_base + (unsigned)(Shape::RING + st1 * Shape::STAGE);
    advance(next);
    const unsigned dist = distance(next);
    const bool more = cur.c0 + CK < c_end;
    static_for<0, NKS>([&](auto ks_tag) {
      constexpr int KS = decltype(ks_tag)::value;
      half8(&fa)[TM] = (KS % 2 == 0) ? fa0 : fa1;
      half8(&fb)[TN] = (KS % 2 == 0) ? fb0 : fb1;
      if constexpr (ISSUE) lds_wait<READS>();
      else lds_wait<0>();
#pragma unroll
      for (int t = 0; t < TM; ++t) lds_pin(fa[t]);
#pragma unroll
      for (int t = 0; t < TN; ++t) lds_pin(fb[t]);
      sched_fence();
      static_for<0, G>([&](auto q_tag) {
        constexpr int Q = decltype(q_tag)::value, I = Q / TN, J = Q % TN;
        acc[I][J] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[J], fa[I], acc[I][J], 0, 0, 0);
        sched_fence();
        if constexpr (KS == NKS - 2 && Q < TM) aim(Q, dist, (unsigned)next.tap);  // the reads of this k tile have all been requested
        if constexpr (ISSUE) {
          static_for<0, LPT>([&](auto l_tag) {
            constexpr int Lx = decltype(l_tag)::value, SLOT = Lx * NSL / LPT;
            if constexpr ((Q < G - 1 || G == 1) && SLOT / SPG == KS && SLOT % SPG == Q) {
              if constexpr (Lx < PA) {  // window load tap * PA + Lx of the next channels
                const int ii = cur.tap * PA + Lx;
                load_window(cur.win ^ 1, cur.c0 + CK, ii, more && ii < LP);
              } else {
                load_filter(ist, req.c0, req.tap, std::integral_constant<int, (Lx >= PA ? Lx - PA : 0)>{});
              }
            }
          });
        }
        sched_fence();
      });
      if constexpr (KS + 2 < NKS) {
        read_frags(sb, std::integral_constant<int, (KS + 2 < NKS ? KS + 2 : 0)>{}, fa, fb);
      } else {
        if (ISSUE || has_next) {
          if constexpr (KS == NKS - 2) {
            lds_wait<0>();
            if (ISSUE) wait_vmcnt<(NST - 3) * LPT + LBAR>();
            else wait_tiles(younger_after_next);
            __builtin_amdgcn_s_barrier();
          }
          read_frags(sb_next, std::integral_constant<int, (KS + 2 >= NKS ? KS + 2 - NKS : 0)>{}, fa, fb);
        }
      }
      sched_fence();
    });
    cur = next;
  };

  wait_vmcnt<(NST - 2) * LPT>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int t = 0; t < TM; ++t) aim(t, distance(cur), 0u);
  read_frags(lds_base + (unsigned)Shape::RING, std::integral_constant<int, 0>{}, fa0, fb0);
  read_frags(lds_base + (unsigned)Shape::RING, std::integral_constant<int, 1>{}, fa1, fb1);
  int i = 0, st = 0;
  for (; i + NST - 1 < nk; ++i) {
    iteration(st, std::true_type{}, st == 0 ? NST - 1 : st - 1, true, 0);
    advance(req);
    st = st + 1 == NST ? 0 : st + 1;
  }
  for (; i < nk; ++i) {
    iteration(st, std::false_type{}, 0, i + 1 < nk, nk - 2 - i);
    st = st + 1 == NST ? 0 : st + 1;
  }
  __syncthreads();
  igemm_epilogue_impl<BM, BN, TM, TN, NT, dma_epass(BM, BN), Shape::LDS, STATS>(a, acc, lds, m0, n0, split, tid, lane, wm * WTM, wn * WTN);
}

template <int OP, int BM, int BN, int CK, int NST, int PR, int NPB, int WGM, int WGN>
int launch_window_one(const GemmArgs& a, hipStream_t st) {
  using Shape = WindowShape<OP, BM, BN, CK, NST, PR, NPB, WGM, WGN>;
  static_assert(Shape::LDS <= 160 * 1024, "more LDS than a compute unit has");
  static std::atomic<bool> lds_set{false};
  if (!jz::allow_lds(reinterpret_cast<const void*>(&conv_window<OP, BM, BN, CK, NST, PR, NPB, WGM, WGN>), Shape::LDS, lds_set)) return JZ_ERR_LAUNCH;
  const unsigned grid = (unsigned)a.tiles_m * (unsigned)a.tiles_n * (unsigned)a.splits;
  hipLaunchKernelGGL((conv_window<OP, BM, BN, CK, NST, PR, NPB, WGM, WGN>), dim3(grid), dim3(Shape::NT), Shape::LDS, st, a);
  return jz::launch_status();
}

// one for every entry of kWindows; the window has to hold what the plan's geometry reaches
template <int OP>
int launch_window(const Plan& pl, hipStream_t st) {
  const GemmArgs& a = pl.args;
  const WindowVariant& v = kWindows[pl.window - 1];
  const int taps = a.g.R * a.g.S;
  if (v.BM + (a.g.R - 1) * a.g.IW + a.g.S - 1 > v.rows || a.g.IC % v.ck != 0 || (v.windows == 1 && a.g.IC != v.ck) || taps < 9 || taps > 32 ||
      a.g.ph * 2 + 1 != a.g.R || a.g.pw * 2 + 1 != a.g.S || a.g.IH != a.g.OH || a.g.IW != a.g.OW || a.kt_per_split % taps != 0 || a.sc_on)
    return JZ_ERR_UNSUPPORTED;
  switch (pl.window - 1) {
    case 0: return launch_window_one<OP, 256, 128, 64, 3, 384, 2, 4, 2>(a, st);
    case 1: return launch_window_one<OP, 256, 64, 64, 3, 384, 1, 4, 1>(a, st);
    default: return JZ_ERR_UNSUPPORTED;
  }
}

}  // namespace
