// FP32 implicit GEMM with LDS-direct loads for channel counts that are multiples of 4 (included by jz_f32_kernels.h inside its
// anonymous namespace; the table in jz_igemm.h says what A, B, m, n, k are in each operation): what a workgroup of either form loads
// and stores (F32Tile), and the form on the FP32 matrix instructions, which short launches take (choose_tiling_f32) and tiles with
// results that are not finite (jz_f32_split.h).
//
// What bounds that: the vector ALU.  The FP32 MFMAs run on it (their 157 TFLOP/s are the packed FP32 rate), so unlike beside FP16
// MFMAs every other vector instruction of the loop takes matrix time: a first version with plain per-load tap arithmetic,
// 60-80 vector instructions per k tile, stood at 115-126 TFLOP/s on a large GEMM.  Hence:
//   * operands go from memory to LDS directly, requested NST tiles ahead, one barrier per tile;
//   * a load's address is a per-lane offset that never changes plus a scalar offset (tap, channel block): one
//     v_bfe_i32 + one v_or per gathered load (bit mask of the row's invalid taps, an out-of-range offset delivers zeros),
//     none for the others (the last tile of a backward-weight reduction, whose rows can lie beyond the tensors, is the one
//     that compares: scalar offsets take no part in the descriptor's range check);
//   * the loop is unrolled over the ring's stages, so that LDS addresses are a register plus a constant.
// F32_TAPS keeps per-lane tap arithmetic, for channel counts that are not multiples of the k tile (the reduction then runs
// over the flattened (tap, channel) index) and more than 32 taps.  Backward-weight reads x as a plain matrix (1x1, unit stride,
// unpadded), at a constant distance per tap (F32_SAME: the output grid is the input grid) or by the input pixel's offset; as one
// kernel that looks at the launch's arguments a gathered load was 38 vector instructions, now 4, 17 and 20 (ResNet-50's weight
// gradients at N = 64, operands in parts: 3.63 -> 3.46 ms).
// The MFMA is the 16x16x4 form: in a loop of nothing else it reaches 152-154 TFLOP/s whatever the occupancy, the 32x32x2
// form 141 with one wavefront per SIMD, 151 with two and 124 with four.
//
// Reduction order inside a tile.  An MFMA multiplies four k, lanes 16 q .. 16 q + 15 hold the q-th.  Which four does not
// matter as long as both operands agree, so step j of a tile takes k = 4 q + j: a lane's four steps are then four
// consecutive k, one ds_read_b128 of a k-contiguous operand ("KC": rows of 16 floats in LDS, 16-byte chunk c of row r at
// position c ^ ((r >> 2) & 3), conflict-free for the writes and the reads).  An operand that is contiguous along its own
// m / n index ("MC") sits in LDS as [k][rows] and is read one float per lane and step; chunk c of k-row k is at position
// c ^ 4 ((k >> 2) & 3), so that the four 64-byte pieces a read takes from rows j, 4 + j, 8 + j, 12 + j lie in different banks.
#pragma once

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int OFF>
__device__ __forceinline__ f32x4 lds_read_f4(unsigned addr) {
  f32x4 v = {};
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
#endif
  return v;
}
template <int OFF>
__device__ __forceinline__ float lds_read_f1(unsigned addr) {
  float v = 0.f;
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
#endif
  return v;
}

// the k lowest bits, k in [0, 32]
__device__ __forceinline__ unsigned low_taps(int k) { return k >= 32 ? 0xffffffffu : (1u << k) - 1u; }
__device__ __forceinline__ int clamp_taps(int x, int hi) { return x < 0 ? 0 : (x > hi ? hi : x); }

// What the workgroup with number `block` of the `blocks` that the launch `a` consists of loads, and where its results go.
// SWZ: the places of the 16-byte chunks in LDS follow from the load (LDS-direct), so the lanes fetch them in swizzled order.
// TAPS_INSIDE: the k tiles go through the taps of 16 channels, then to the next channels (jz_f32_window.h: nine taps).
template <int OP, int BM, int BN, int FORM, bool SWZ, bool TAPS_INSIDE = false>
struct F32Tile {
  static constexpr bool GEN = OP != OP_BWD_WEIGHT && FORM == F32_TAPS;
  static constexpr bool MATRIX = OP == OP_BWD_WEIGHT && FORM == F32_MATRIX, SAME = OP == OP_BWD_WEIGHT && FORM == F32_SAME;
  static constexpr bool A_KC = OP != OP_BWD_WEIGHT, B_KC = OP == OP_FWD;
  static constexpr int A_BYTES = BM * FD_BK * 4, B_BYTES = BN * FD_BK * 4;
  static constexpr int LA = A_BYTES / 4096, LB = B_BYTES / 4096, LPT = LA + LB;  // 16-byte loads per thread and tile
  static_assert(LA >= 1 && LB >= 1, "tile too small for 256 loaders");
  static constexpr unsigned OOB = 0xffffffffu;

  const F32Args& a;
  const ConvGeom& g;
  int tid, lane, wave, wm, wn;   // 2 x 2 wavefronts
  bool whole;
  int split, m0, n0, kt_begin, nk;
  __amdgpu_buffer_rsrc_t rsrcA, rsrcB;
  // KC: 16 rows x 4 chunks a load of a wavefront; load ii of wavefront w covers rows (4 ii + w) 16 + lane / 4.  The swizzle is the
  // same for every ii.
  int kc_row, kc_chunk;
  // MC with ROWS mn: ROWS / 4 chunks per k-row
  __device__ __forceinline__ int mc_k(int rows, int ii) const { return ((4 * ii + wave) * 64 + lane) / (rows / 4); }
  __device__ __forceinline__ int mc_col(int rows, int ii) const {
    return ((lane % (rows / 4)) ^ (SWZ ? 4 * ((mc_k(rows, ii) >> 2) & 3) : 0)) * 4;
  }
  // vA / vB: the part of a load's byte offset that does not change over the k loop (OOB: the row or column does not exist);
  // invA: bit t set when filter tap t reads outside the image for this row (all bits for rows beyond M)
  unsigned vA[LA], invA[LA], vB[LB];
  int gh[LA], gw[LA];  // GEN: source coordinates of tap (0, 0)
  // backward-weight, gathered x: per load the row, the column and the byte offset of the input pixel at the lane's tap,
  // advanced by 16 output pixels per tile with one carry per digit.  The digits are kept as input coordinates (times the
  // stride, plus the tap): no multiplication in the loop, and exact for every size (a 24-bit product is not: grids and strides
  // reach beyond 2^23).  xp_end, xq_end: where they wrap.
  int xp[LB], xq[LB], xp_end[LB], xq_end[LB], bw_tp, bw_tp1, bw_tq, bw_rows, bw_cols;
  unsigned xoff[LB], bw_dv, bw_k1, bw_k2;

  __device__ __forceinline__ F32Tile(const F32Args& args, unsigned block, unsigned blocks) : a(args), g(args.g) {
    tid = threadIdx.x;
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    wm = wave >> 1;
    wn = wave & 1;
    // the first full_rows rows of tiles are computed whole, one workgroup each; the rest by `splits` workgroups a tile
    const unsigned full = (unsigned)(a.full_rows * a.tiles_n);
    whole = block < full;
    unsigned L = whole ? xcd_remap(block, full) : xcd_remap(block - full, blocks - full);
    split = whole ? 0 : (int)fd_div(L, a.d_tiles_mn);
    L -= (unsigned)split * (unsigned)((a.tiles_m - a.full_rows) * a.tiles_n);
    const unsigned trow = fd_div(L, a.d_tiles_n);
    m0 = ((int)trow + (whole ? 0 : a.full_rows)) * BM;
    n0 = (int)(L - trow * (unsigned)a.tiles_n) * BN;
    kt_begin = split * a.kt_per_split;
    const int kt_end = !whole && kt_begin + a.kt_per_split < a.nkt ? kt_begin + a.kt_per_split : a.nkt;
    nk = kt_end - kt_begin;

    // in-range taps of a gathered row can start before the tensor (padding): the descriptor's base is moved down by that much
    unsigned biasA = 0;
    if (!GEN && OP == OP_FWD) biasA = (unsigned)(g.ph * g.row_pitch + g.pw * g.IC) * 4u;
    if (!GEN && OP == OP_BWD_DATA) biasA = (unsigned)((g.R - 1) * g.row_pitch + (g.S - 1) * g.IC) * 4u;
    rsrcA = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)a.A - biasA), 0, (int)(a.bytesA + biasA), 0x00020000);
    // backward-weight of a layer whose output grid is its input grid (bw_same): pixel j at a tap is pixel j + constant of x, so the
    // offset is linear in j as for a plain matrix and only the image borders need the pixel's coordinates
    const unsigned biasB = SAME ? (unsigned)(g.ph * g.row_pitch + g.pw * g.IC) * 4u : 0u;
    rsrcB = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)a.B - biasB), 0, (int)(a.bytesB + biasB), 0x00020000);

    // ---- loader geometry: one load of a wavefront fills 1 KB ----------------------------------------
    kc_row = wave * 16 + lane / 4;
    kc_chunk = SWZ ? (lane & 3) ^ ((kc_row >> 2) & 3) : lane & 3;
    if constexpr (A_KC) {
#pragma unroll
      for (int ii = 0; ii < LA; ++ii) {
        const int m = m0 + 64 * ii + kc_row;
        gh[ii] = -(1 << 28); gw[ii] = 0; vA[ii] = 0; invA[ii] = OOB;
        if (m < a.M) {
          const unsigned n = fd_div((unsigned)m, g.d_ohow);
          const unsigned rem = (unsigned)m - n * (unsigned)(g.OH * g.OW);
          const int oh = (int)fd_div(rem, g.d_ow), ow = (int)rem - oh * g.OW;
          const int h0 = OP == OP_FWD ? oh * g.sh - g.ph : oh + g.ph, w0 = OP == OP_FWD ? ow * g.sw - g.pw : ow + g.pw;
          gh[ii] = h0; gw[ii] = w0;
          vA[ii] = (unsigned)(((int)n * g.IH + h0) * g.IW + w0) * (unsigned)g.IC;
          if constexpr (!GEN) {
            vA[ii] = (vA[ii] + (unsigned)kc_chunk * 4u) * 4u + (OP == OP_FWD ? biasA : 0u);
            invA[ii] = taps_outside(h0, w0);
          }
        }
      }
    } else {
#pragma unroll
      for (int ii = 0; ii < LA; ++ii) {
        const int mm = m0 + mc_col(BM, ii);
        vA[ii] = mm < a.M ? (unsigned)(mc_k(BM, ii) * a.M + mm) * 4u : OOB;
      }
    }
    if constexpr (OP == OP_FWD) {
#pragma unroll
      for (int ii = 0; ii < LB; ++ii) {
        const int nn = n0 + 64 * ii + kc_row;
        vB[ii] = nn < a.N ? (unsigned)(nn * a.Kred + kc_chunk * 4) * 4u : OOB;
      }
    } else if constexpr (OP == OP_BWD_DATA) {
#pragma unroll
      for (int ii = 0; ii < LB; ++ii) {
        const int nn = n0 + mc_col(BN, ii);
        vB[ii] = nn < a.N ? (unsigned)nn * 4u + (GEN ? 0u : (unsigned)(mc_k(BN, ii) * a.w_taps) * (unsigned)a.N * 4u) : OOB;
      }
    } else {
      bw_rows = g.OH * g.sh;
      bw_cols = g.OW * g.sw;
      const unsigned Pn = (unsigned)(g.IH * g.row_pitch) * 4u, Ph = (unsigned)(g.sh * g.row_pitch) * 4u, Pw = (unsigned)(g.sw * g.IC) * 4u;
      const unsigned ta = fd_div((unsigned)FD_BK, g.d_ohow), trem = (unsigned)FD_BK - ta * (unsigned)(g.OH * g.OW);
      const unsigned tp = fd_div(trem, g.d_ow), tq = trem - tp * (unsigned)g.OW;
      bw_tp = (int)tp * g.sh;
      bw_tp1 = bw_tp + g.sh;
      bw_tq = (int)tq * g.sw;
      bw_dv = ta * Pn + tp * Ph + tq * Pw;
      bw_k1 = Ph - (unsigned)g.OW * Pw;
      bw_k2 = Pn - (unsigned)g.OH * Ph;
#pragma unroll
      for (int ii = 0; ii < LB; ++ii) {
        const int nn = n0 + mc_col(BN, ii);
        int r0 = -(1 << 30), s0 = 0;  // a column that does not exist lies outside every image
        vB[ii] = nn < a.N ? (unsigned)(mc_k(BN, ii) * g.IC + nn) * 4u : OOB;  // 1x1, unit stride, unpadded: a plain matrix
        int ch = 0;
        if (nn < a.N) {
          const unsigned tap = fd_div((unsigned)nn, g.d_ic), r = fd_div(tap, g.d_s);
          ch = nn - (int)tap * g.IC;
          r0 = (int)r - g.ph;
          s0 = (int)(tap - r * (unsigned)g.S) - g.pw;
        }
        const unsigned j = (unsigned)(kt_begin * FD_BK + mc_k(BN, ii));
        const unsigned n = fd_div(j, g.d_ohow), rem = j - n * (unsigned)(g.OH * g.OW);
        const unsigned pp = fd_div(rem, g.d_ow);
        const unsigned qq = rem - pp * (unsigned)g.OW;
        xp[ii] = (int)pp * g.sh + r0;
        xq[ii] = (int)qq * g.sw + s0;
        xp_end[ii] = bw_rows + r0;
        xq_end[ii] = bw_cols + s0;
        if (SAME && nn < a.N) vB[ii] = (unsigned)((mc_k(BN, ii) + r0 * g.IW + s0) * g.IC + ch) * 4u + biasB;
        xoff[ii] = ((n * (unsigned)g.IH + (unsigned)xp[ii]) * (unsigned)g.row_pitch + (unsigned)xq[ii] * (unsigned)g.IC + (unsigned)ch) * 4u;
      }
    }
  }

  // The taps that read outside the image, for a row whose tap (0, 0) is at (h0, w0).  Along one axis they are a run at the start and a
  // run at the end of the filter (backward-data: the other way round); the column mask is copied into every filter row's slot by one
  // multiplication.
  __device__ __forceinline__ unsigned taps_outside(int h0, int w0) const {
    const int lo_w = OP == OP_FWD ? -w0 : w0 - g.IW + 1, hi_w = OP == OP_FWD ? g.IW - w0 : w0 + 1;
    const int lo_h = OP == OP_FWD ? -h0 : h0 - g.IH + 1, hi_h = OP == OP_FWD ? g.IH - h0 : h0 + 1;
    const unsigned cm = low_taps(clamp_taps(lo_w, g.S)) | (low_taps(g.S) & ~low_taps(clamp_taps(hi_w, g.S)));
    return cm * g.tap_rep | low_taps(clamp_taps(lo_h, g.R) * g.S) | (low_taps(g.R * g.S) & ~low_taps(clamp_taps(hi_h, g.R) * g.S));
  }
  __device__ __forceinline__ unsigned taps_outside(int m) const {
    if (m >= a.M) return OOB;
    const unsigned n = fd_div((unsigned)m, g.d_ohow), rem = (unsigned)m - n * (unsigned)(g.OH * g.OW);
    const int oh = (int)fd_div(rem, g.d_ow), ow = (int)rem - oh * g.OW;
    return OP == OP_FWD ? taps_outside(oh * g.sh - g.ph, ow * g.sw - g.pw) : taps_outside(oh + g.ph, ow + g.pw);
  }

  struct TileCtx {
    unsigned k0;
    unsigned tap, soffA, soffB;  // the same for the whole wavefront (the tile lies inside one tap)
    int r, s;                    // GEN, per lane: the tap of the lane's chunk (negated for backward-data) ...
    unsigned loff;               // ... the element offset it adds ...
    bool in;                     // ... and whether the chunk lies inside the reduction
    bool tail;                   // backward-weight, wave-uniform: some rows of the tile lie beyond the reduction
  };
  __device__ __forceinline__ TileCtx tile_ctx(int kt) const {
    TileCtx c{};
    c.k0 = (unsigned)(kt * FD_BK);
    if constexpr (TAPS_INSIDE) c.k0 = (unsigned)(kt % 9 * g.IC + kt / 9 * FD_BK);
    if constexpr (OP == OP_BWD_WEIGHT) {
      c.soffA = c.k0 * (unsigned)a.M * 4u;
      c.soffB = c.k0 * (unsigned)g.IC * 4u;
      c.tail = c.k0 + FD_BK > (unsigned)a.Kred;
    } else if constexpr (!GEN) {
      c.tap = fd_div(c.k0, g.d_ic);
      const unsigned ch = c.k0 - c.tap * (unsigned)g.IC;
      const unsigned r = fd_div(c.tap, g.d_s), s = c.tap - r * (unsigned)g.S;
      if constexpr (OP == OP_FWD) {
        c.soffA = (r * (unsigned)g.row_pitch + s * (unsigned)g.IC + ch) * 4u;
        c.soffB = c.k0 * 4u;
      } else {
        c.soffA = (((unsigned)g.R - 1u - r) * (unsigned)g.row_pitch + ((unsigned)g.S - 1u - s) * (unsigned)g.IC + ch) * 4u;
        c.soffB = (ch * (unsigned)a.w_taps + (unsigned)a.w_tap0 + r * (unsigned)a.w_tap_r + s * (unsigned)a.w_tap_s) * (unsigned)a.N * 4u;
      }
    } else {
      const unsigned kq = c.k0 + (unsigned)kc_chunk * 4u;
      const unsigned tap = fd_div(kq, g.d_ic), ch = kq - tap * (unsigned)g.IC;
      const int r = (int)fd_div(tap, g.d_s), s = (int)tap - r * g.S;
      c.r = OP == OP_FWD ? r : -r;
      c.s = OP == OP_FWD ? s : -s;
      c.loff = (unsigned)((c.r * g.IW + c.s) * g.IC) + ch;
      c.in = kq < (unsigned)a.Kred;
      c.soffB = c.k0 * 4u;
    }
    return c;
  }
  // the filter's part of it for 16 channels of one of nine taps (jz_f32_window.h)
  __device__ __forceinline__ TileCtx tile_at(int tap, int channel) const {
    TileCtx c{};
    c.soffB = OP == OP_FWD ? (unsigned)(tap * g.IC + channel) * 4u : (unsigned)(channel * 9 + tap) * (unsigned)a.N * 4u;
    return c;
  }
  // load Lx (A's, then B's) of the tile: f(descriptor, per-lane byte offset, scalar byte offset)
  template <int Lx, class F>
  __device__ __forceinline__ void load(const TileCtx& c, F&& f) {
    if constexpr (Lx < LA) {
      constexpr int ii = Lx;
      if constexpr (A_KC && GEN) {
        const bool ok = c.in && (unsigned)(gh[ii] + c.r) < (unsigned)g.IH && (unsigned)(gw[ii] + c.s) < (unsigned)g.IW;
        f(rsrcA, ok ? (vA[ii] + c.loff) * 4u : OOB, 0u);
      } else if constexpr (A_KC) {
        const unsigned bad = (unsigned)__builtin_amdgcn_sbfe(invA[ii], c.tap, 1);  // 0 / -1
        f(rsrcA, vA[ii] | bad, c.soffA);
      } else {
        f(rsrcA, c.tail && c.k0 + (unsigned)mc_k(BM, ii) >= (unsigned)a.Kred ? OOB : vA[ii], c.soffA);
      }
    } else {
      constexpr int ii = Lx - LA;
      if constexpr (OP == OP_FWD && GEN) {
        f(rsrcB, c.in ? vB[ii] : OOB, c.soffB);
      } else if constexpr (OP == OP_BWD_DATA && GEN) {
        // row k is filter w[ko][tap][.]; a strided layer's launch covers the taps of one residue of the stride
        const unsigned kk = c.k0 + (unsigned)mc_k(BN, ii);
        const unsigned tap = fd_div(kk, g.d_ic), ko = kk - tap * (unsigned)g.IC;
        const unsigned r = fd_div(tap, g.d_s), s = tap - r * (unsigned)g.S;
        const unsigned row = ko * (unsigned)a.w_taps + (unsigned)a.w_tap0 + r * (unsigned)a.w_tap_r + s * (unsigned)a.w_tap_s;
        f(rsrcB, kk < (unsigned)a.Kred && vB[ii] != OOB ? vB[ii] + row * (unsigned)a.N * 4u : OOB, 0u);
      } else if constexpr (OP != OP_BWD_WEIGHT) {
        f(rsrcB, vB[ii], c.soffB);
      } else {
        const bool beyond = c.tail && c.k0 + (unsigned)mc_k(BN, ii) >= (unsigned)a.Kred;
        if constexpr (MATRIX) {
          f(rsrcB, beyond ? OOB : vB[ii], c.soffB);
        } else {
          const bool ok = (unsigned)xp[ii] < (unsigned)g.IH && (unsigned)xq[ii] < (unsigned)g.IW && !beyond;
          f(rsrcB, ok ? (SAME ? vB[ii] : xoff[ii]) : OOB, SAME ? c.soffB : 0u);
          xq[ii] += bw_tq;
          const bool c1 = xq[ii] >= xq_end[ii];
          xq[ii] -= c1 ? bw_cols : 0;
          xp[ii] += c1 ? bw_tp1 : bw_tp;
          const bool c2 = xp[ii] >= xp_end[ii];
          xp[ii] -= c2 ? bw_rows : 0;
          if constexpr (!SAME) xoff[ii] += bw_dv + (c1 ? bw_k1 : 0u) + (c2 ? bw_k2 : 0u);
        }
      }
    }
  }

  // Results go through LDS, as many rows of wavefronts at a time as fit `lds_bytes`, so that a store instruction writes whole row
  // pieces.  put(floats): writes the wavefront's rows there, LDF floats apart.
  static constexpr int LDF = BN + 4;
  template <int LDS_BYTES, class F>
  __device__ __forceinline__ void store(float* lds_f, F&& put) {
    const int part_row = a.full_rows * BM;  // row 0 of the partial sums
    float* const out = whole ? a.D : a.Dpart + (size_t)split * (a.M - part_row) * a.N;
    constexpr int FCH = BN / 4, RPP = 256 / FCH;
    constexpr int PS = BM * LDF * 4 <= LDS_BYTES ? 1 : 2, RH = BM / PS;
    static_assert(RH * LDF * 4 <= LDS_BYTES, "the staged rows have to fit");
    const bool vec = (a.N & 3) == 0;
    const int fch = tid % FCH, frow = tid / FCH;
#pragma unroll
    for (int ps = 0; ps < PS; ++ps) {
      if (ps > 0) __syncthreads();
      if (PS == 1 || wm == ps) put(lds_f + (PS == 1 ? wm * (BM / 2) : 0) * LDF + wn * (BN / 2));
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RH / RPP; ++i) {
        const int row = frow + RPP * i, m = m0 + ps * RH + row, n = n0 + fch * 4;
        if (m >= a.M || n >= a.N) continue;
        size_t drow = (size_t)(whole ? m : m - part_row);
        if (a.sc_on) {  // row m = (n, p, q) of the strided grid goes to input pixel (n, p sh + oh, q sw + ow)
          const unsigned img = fd_div((unsigned)m, g.d_ohow);
          const unsigned rem = (unsigned)m - img * (unsigned)(g.OH * g.OW);
          const unsigned p = fd_div(rem, g.d_ow), q = rem - p * (unsigned)g.OW;
          drow = ((size_t)img * a.sc_H + p * a.sc_sh + a.sc_oh) * a.sc_W + q * a.sc_sw + a.sc_ow;
          // strided single tap: no output pixel reads the other pixels of this cell, their gradient is zero
          for (int i2 = 0; a.sc_fill && i2 < a.sc_sh; ++i2)
            for (int j2 = 0; j2 < a.sc_sw; ++j2) {
              if ((i2 | j2) == 0 || (int)(p * a.sc_sh) + i2 >= a.sc_H || (int)(q * a.sc_sw) + j2 >= a.sc_W) continue;
              *reinterpret_cast<float4*>(out + (drow + (size_t)i2 * a.sc_W + j2) * a.N + n) = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        const float4 v = *reinterpret_cast<const float4*>(lds_f + row * LDF + fch * 4);
        float* dst = out + drow * a.N + n;
        if (vec && whole) {  // non-temporal: written back at once, not while the next launch reads (partial sums are read at once)
          typedef float f32x4_t __attribute__((ext_vector_type(4)));
          const f32x4_t t = {v.x, v.y, v.z, v.w};
          __builtin_nontemporal_store(t, reinterpret_cast<f32x4_t*>(dst));
        } else if (vec) {
          *reinterpret_cast<float4*>(dst) = v;
        } else {
          const float e[4] = {v.x, v.y, v.z, v.w};
          for (int k = 0; k < 4 && n + k < a.N; ++k) dst[k] = e[k];
        }
      }
    }
  }
};

// the tile on the FP32 matrix instructions
template <int OP, int BM, int BN, int FORM, bool TAPS_INSIDE = false>
__device__ __forceinline__ void f32_dma_body(const F32Args& a, unsigned block, unsigned blocks) {
  using Tile = F32Tile<OP, BM, BN, FORM, true, TAPS_INSIDE>;
  constexpr bool A_KC = Tile::A_KC, B_KC = Tile::B_KC;
  constexpr int TM = BM / 32, TN = BN / 32;   // 16x16 MFMA tiles per wavefront
  constexpr int RB = FD_BK * 4;               // bytes per row of a KC tile
  constexpr int A_BYTES = Tile::A_BYTES, STAGE = A_BYTES + Tile::B_BYTES, LPT = Tile::LPT;
  extern __shared__ __align__(16) float lds_f[];
  lds_byte* const ldsb = (lds_byte*)lds_f;
  const unsigned lds_base = (unsigned)(uintptr_t)JZ_LDS_PTR(lds_f);
  Tile t(a, block, blocks);
  const int nk = t.nk, lane = t.lane, wm = t.wm, wn = t.wn;
  auto issue_load = [&](const typename Tile::TileCtx& c, int st, auto l_tag) {  // one load of a wavefront fills 1 KB
    constexpr int Lx = decltype(l_tag)::value;
    lds_byte* const dst = ldsb + st * STAGE + (Lx < Tile::LA ? 0 : A_BYTES) + (4 * (Lx < Tile::LA ? Lx : Lx - Tile::LA) + t.wave) * 1024;
    t.template load<Lx>(c, [&](__amdgpu_buffer_rsrc_t rsrc, unsigned voff, unsigned soff) { jz_dma16s(rsrc, dst, voff, soff); });
  };

#pragma unroll
  for (int s = 0; s < FD_NST; ++s)
    if (s < nk) {
      const typename Tile::TileCtx c = t.tile_ctx(t.kt_begin + s);
      static_for<0, LPT>([&](auto l) { issue_load(c, s, l); });
    }
  sched_fence();

  // ---- MFMA operand addresses -----------------------------------------------------------------------
  const int r15 = lane & 15, q4l = lane >> 4;
  // KC: row base + r15, chunk q at its swizzled place; 16-row sub-tiles are 16 RB bytes apart and share the swizzle.
  // MC: k-row 4 q + j, column base + r15: the swizzle moves whole groups of four chunks (16 columns), i.e. sub-tile t of a
  // wavefront sits where sub-tile t ^ q would: one address per sub-tile.
  unsigned adA[A_KC ? 1 : TM], adB[B_KC ? 1 : TN];
  if constexpr (A_KC) {
    adA[0] = lds_base + (unsigned)((wm * (BM / 2) + r15) * RB + ((q4l ^ ((r15 >> 2) & 3)) * 16));
  } else {
#pragma unroll
    for (int t = 0; t < TM; ++t) adA[t] = lds_base + (unsigned)((4 * q4l * BM + (((wm * (BM / 2)) / 16 + t) ^ q4l) * 16 + r15) * 4);
  }
  if constexpr (B_KC) {
    adB[0] = lds_base + (unsigned)(A_BYTES + (wn * (BN / 2) + r15) * RB + ((q4l ^ ((r15 >> 2) & 3)) * 16));
  } else {
#pragma unroll
    for (int t = 0; t < TN; ++t) adB[t] = lds_base + (unsigned)(A_BYTES + (4 * q4l * BN + (((wn * (BN / 2)) / 16 + t) ^ q4l) * 16 + r15) * 4);
  }

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

  f32x4 fa0[TM], fb0[TN], fa1[TM], fb1[TN];  // operands of one tile each
  auto read_tile = [&](auto st_tag, f32x4 (&va)[TM], f32x4 (&vb)[TN]) {
    constexpr int SO = decltype(st_tag)::value * STAGE;  // fits the instruction's 16-bit offset
    static_assert(FD_NST * STAGE <= 65536, "stage offsets are immediates");
    static_for<0, TM>([&](auto t_tag) {
      constexpr int T = decltype(t_tag)::value;
      if constexpr (A_KC) {
        va[T] = lds_read_f4<SO + 16 * T * RB>(adA[0]);
      } else {
        static_for<0, 4>([&](auto j_tag) {
          constexpr int J = decltype(j_tag)::value;
          va[T][J] = lds_read_f1<SO + J * BM * 4>(adA[A_KC ? 0 : T]);
        });
      }
    });
    static_for<0, TN>([&](auto t_tag) {
      constexpr int T = decltype(t_tag)::value;
      if constexpr (B_KC) {
        vb[T] = lds_read_f4<SO + 16 * T * RB>(adB[0]);
      } else {
        static_for<0, 4>([&](auto j_tag) {
          constexpr int J = decltype(j_tag)::value;
          vb[T][J] = lds_read_f1<SO + J * BN * 4>(adB[B_KC ? 0 : T]);
        });
      }
    });
  };
  auto wait_tiles = [&](int younger) {  // until at most `younger` later tiles are in flight
    if (younger >= 2) wait_vmcnt<2 * LPT>();
    else if (younger == 1) wait_vmcnt<LPT>();
    else wait_vmcnt<0>();
  };

  // One iteration multiplies tile i, whose operands were requested from LDS during tile i - 1.  Once they have arrived, tile
  // i + 1 has landed and every wavefront is at the barrier, stage i % NST is free: the next tile's operands are requested
  // from LDS and tile i + NST from memory between the MFMAs.
  static_assert(FD_NST == 4, "wait_tiles counts two younger tiles");
  auto iteration = [&](int i, auto st_tag, f32x4 (&va)[TM], f32x4 (&vb)[TN], f32x4 (&na)[TM], f32x4 (&nb)[TN]) {
    constexpr int ST = decltype(st_tag)::value;  // i % NST
    const bool more = i + FD_NST < nk;
    const typename Tile::TileCtx c = t.tile_ctx(t.kt_begin + i + FD_NST);  // unused when there is no such tile
    lds_wait<0>();
#pragma unroll
    for (int k = 0; k < TM; ++k) lds_pin(va[k]);
#pragma unroll
    for (int k = 0; k < TN; ++k) lds_pin(vb[k]);
    if (i + 1 < nk) {
      wait_tiles(nk - 2 - i);
      __builtin_amdgcn_s_barrier();
      read_tile(std::integral_constant<int, (ST + 1) % FD_NST>{}, na, nb);
    }
    sched_fence();
    static_for<0, 4>([&](auto j_tag) {
      constexpr int J = decltype(j_tag)::value;
#pragma unroll
      for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y)
          // n operand in the first slot: each lane then owns 4 consecutive n for one m (row = lane % 16)
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(vb[y][J], va[x][J], acc[x][y], 0, 0, 0);
      if (more)
        static_for<0, LPT>([&](auto l_tag) {
          if constexpr (decltype(l_tag)::value * 4 / LPT == J) issue_load(c, ST, l_tag);
        });
      sched_fence();
    });
  };
  if (nk > 0) {
    if (nk >= 4) wait_vmcnt<3 * LPT>();
    else wait_tiles(nk - 1);
    __builtin_amdgcn_s_barrier();
    read_tile(std::integral_constant<int, 0>{}, fa0, fb0);
  }
  for (int i = 0; i < nk; i += FD_NST) {
    iteration(i, std::integral_constant<int, 0>{}, fa0, fb0, fa1, fb1);
    if (i + 1 < nk) iteration(i + 1, std::integral_constant<int, 1>{}, fa1, fb1, fa0, fb0);
    if (i + 2 < nk) iteration(i + 2, std::integral_constant<int, 2>{}, fa0, fb0, fa1, fb1);
    if (i + 3 < nk) iteration(i + 3, std::integral_constant<int, 3>{}, fa1, fb1, fa0, fb0);
  }
  __syncthreads();  // the epilogue stages the tile in the ring

  // accumulator register r of tile (x,y): m = wrow + 16 x + lane % 16, n = wcol + 16 y + 4 (lane / 16) + r
  t.template store<FD_NST * STAGE>(lds_f, [&](float* rows) {
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
      for (int y = 0; y < TN; ++y)
        *reinterpret_cast<float4*>(rows + (16 * x + r15) * Tile::LDF + 16 * y + 4 * q4l) =
            make_float4(acc[x][y][0], acc[x][y][1], acc[x][y][2], acc[x][y][3]);
  });
}
