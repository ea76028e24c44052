// FP32 convolutions of 3x3 filters whose output grid is their input grid (unit stride, padding 1), forward and backward-data, on the
// bfloat16 matrix instructions, with the pixels under a tile taken apart once for all nine taps (included by jz_f32_kernels.h behind
// jz_f32_split.h, which says what the parts are).
//
// f32_split_body takes every value apart once per tap that reads it: 4.3 vector instructions per product for 128x128 tiles, 6.5 for
// 128x64, and energy, which is what bounds long reductions.  Here the 128 pixels of a tile, which are consecutive in memory, and what their
// taps reach (a run of 128 + 2 W + 2 pixels) are taken apart into LDS once per 16 channels, and each tap reads its rows out of that run at
// its own distance; rows whose tap lies outside the image read a row of zeros (one bit per row and tap).  Only the filter still is taken apart
// tile by tile.  That leaves about 3.2 vector instructions per product for 128x128 tiles: 2.2 for
// the filter, 0.4 for the pixels, 0.6 for the taps' addresses.
//
//   LDS: two windows, each three parts of PR rows of 16 bfloat16 and 16 rows of zeros | two stages of the filter's parts, as in
//   jz_f32_split.h.  Rows have the KC layout; its swizzle goes by the row's place in LDS, so any 16 consecutive rows read without conflicts.
//
// Measured (3x3, 64 images, us of a call, split reductions included, calls in a row on other buffers each, one box, forward / backward-data, every
// tap's values taken apart and this): 56x56, 64 channels 95 / 96 and 89 / 90; 28x28, 128 channels 92 / 93 and 79 / 79; 14x14, 256 channels
// 95 / 99 and 83 / 85; 28x28, 256 -> 512 570 / 587 and 557 / 561.  What bounds it: with the chip full, power (13x13, 384 channels, 128 images: pipes
// busy 82 % of the compute units' busy cycles at 1.7 GHz, where a loop of products alone has 1.74); with one or two workgroups a compute unit the
// waits of a tile (14x14: 61 % at 2.0 GHz; bank conflicts 3-8 % of the busy cycles).
//
// Relative errors against 64 bits, both directions of 21 layers, are 0.31 ... 1.00 of those of the form before.
//
// The reduction runs blocks of 16 channels outside, taps inside.  The loop is unrolled over two blocks, 18 k tiles, so that the tap, both LDS
// buffers and the register set of a load are constants: the window of the next block is requested behind the filter of one's second
// tap and taken apart during the last taps (loads return in order: with one window load a tap every filter tile waited for one).
#pragma once

template <int BN, int LP>
struct F32Window {
  static constexpr int BM = 128, PR = 64 * LP;                   // rows a window holds
  static constexpr int PART = (PR + 16) * 32, WIN = 3 * PART;    // a multiple of 512 bytes: the swizzle is the same in every part
  static constexpr int B0 = 2 * WIN, B_PART = BN * FD_BK * 2, STAGE = 3 * B_PART;
  static constexpr int OPERANDS = B0 + 2 * STAGE, RING = FD_NST * (BM + BN) * FD_BK * 4;
  static constexpr int LDS_BYTES = OPERANDS > RING ? OPERANDS : RING;
};

template <int OP, int BN, int LP>
__device__ __forceinline__ void f32_window_body(const F32Args& a, unsigned block, unsigned blocks) {
  using Lds = F32Window<BN, LP>;
  constexpr int BM = Lds::BM, PART = Lds::PART, WIN = Lds::WIN, B_PART = Lds::B_PART, STAGE = Lds::STAGE;
  using Tile = F32Tile<OP, BM, BN, F32_MASKS, false, true>;
  constexpr bool B_KC = Tile::B_KC;
  constexpr int TM = BM / 64, TN = BN / 64, TT = TM * TN, LA = Tile::LA, LB = Tile::LB, TAPS = 9;
  constexpr int SETS = BN == 64 ? 6 : LP == 3 ? 3 : 2;  // filter tiles on their way in registers: as many as there is room for
  extern __shared__ __align__(16) float lds_f[];
  lds_byte* const ldsb = (lds_byte*)lds_f;
  Tile t(a, block, blocks);
  const ConvGeom& g = a.g;
  const int nk = t.nk, lane = t.lane, wave = t.wave, wm = t.wm, wn = t.wn;  // nk, kt_begin: multiples of 18

  // ---- requests -----------------------------------------------------------------------------------------
  // Window row 64 l + kc_row; rows no tap reaches are not requested, pixels in front of the tensor wrap to offsets behind it.
  const unsigned pitch = (unsigned)g.IC * 4u;
  const unsigned vW = (unsigned)(t.m0 - g.IW - 1 + t.kc_row) * pitch + (unsigned)(lane & 3) * 16u, wrW = f32_kc_at(t.kc_row, lane & 3);
  const int chunk0 = t.kt_begin / TAPS, chunk_end = (t.kt_begin + nk) / TAPS;
  const auto rsrcW = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, (int)a.bytesA, 0x00020000);
  // A window comes in at once or, where its registers and those of 128-wide tiles are too many, in two halves.  At once, backward-data spilled 30
  // registers and waited for all its loads seven times in the loop: 24 images of 43x63, 128 -> 64, 50.0 -> 48.2 us, 41x41, 384 -> 128, 171 -> 167.
  constexpr int HALVES = BN == 128 && LP == 4 ? 2 : 1, LH = LP / HALVES;
  f32x4 rawW[LP], rawB[SETS][LB];  // in the loop the second half takes the places of the first
  auto request_window = [&](int chunk, auto l_tag, auto at_tag) {  // one that does not exist is requested out of range, as in jz_f32_split.h
    constexpr int Lx = decltype(l_tag)::value, AT = decltype(at_tag)::value;
    const int rows = chunk < chunk_end ? BM + 2 * g.IW + 2 - 64 * Lx : 0;
    const unsigned at = t.kc_row < rows ? vW + (unsigned)(64 * Lx) * pitch : Tile::OOB;
    rawW[AT] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rsrcW, (int)at, (int)((unsigned)chunk * FD_BK * 4u), 0));
  };
  auto request_filter = [&](int chunk, int tap, auto set_tag, auto l_tag) {
    constexpr int SET = decltype(set_tag)::value, Lx = decltype(l_tag)::value;
    const unsigned none = chunk < chunk_end ? 0u : Tile::OOB;
    t.template load<LA + Lx>(t.tile_at(tap, chunk * FD_BK), [&](__amdgpu_buffer_rsrc_t rsrc, unsigned voff, unsigned soff) {
      rawB[SET][Lx] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(voff | none), (int)soff, 0));
    });
  };
  static_for<0, LP>([&](auto l) { request_window(chunk0, l, l); });
  static_for<0, SETS>([&](auto s) { static_for<0, LB>([&](auto l) { request_filter(chunk0, decltype(s)::value, s, l); }); });
  sched_fence();
  // the zeros of both windows, 16 bytes a thread
  if (t.tid < 6 * 32) {
    const int p = t.tid / 32;
    *(__attribute__((address_space(3))) u32x4*)(ldsb + p * PART + Lds::PR * 32 + (t.tid % 32) * 16) = u32x4{0u, 0u, 0u, 0u};
  }

  // ---- where the parts go and are read ------------------------------------------------------------------
  unsigned wrB[LB], rdB[B_KC ? 1 : 2 * TN];
#pragma unroll
  for (int l = 0; l < LB; ++l)
    wrB[l] = Lds::B0 + (B_KC ? f32_kc_at(64 * l + t.kc_row, lane & 3) : f32_mc_at(BN, t.mc_k(BN, l), lane % (BN / 4)));
  f32_read_addr<B_KC, TN>(rdB, lane, wn * (BN / 2), BN, Lds::B0);
  unsigned rowA[TM], outside[TM], rdA[TM];
#pragma unroll
  for (int x = 0; x < TM; ++x) {
    const int row = wm * (BM / 2) + 32 * x + (lane & 31);
    rowA[x] = (unsigned)(row * 32);
    outside[x] = t.taps_outside(t.m0 + row);
  }
  const unsigned half = (unsigned)(lane >> 5) << 4;
  // tap `tap` out of the window at `win`.  Pinned: the addresses of all taps, which do not change from one pair of windows to the next,
  // would be kept across the loop, 36 registers that are not there (19 of them went to scratch memory, and each wait for one of those
  // is a wait for all loads in flight).
  auto aim = [&](int x, unsigned win, unsigned dist, int tap) {
    lds_pin(rowA[x]);
    const unsigned row = rowA[x] + dist + win;
    const unsigned at = (row | (row >> 4 & 16u)) ^ half;
    const unsigned bad = (unsigned)__builtin_amdgcn_sbfe(outside[x], (unsigned)tap, 1u);
    rdA[x] = (((unsigned)Lds::PR * 32u) & bad) | (at & ~bad);
  };
  unsigned dist[TAPS];  // bytes from a pixel's row to the row its tap reads
#pragma unroll
  for (int tap = 0; tap < TAPS; ++tap) {
    const int at = OP == OP_FWD ? tap : TAPS - 1 - tap;
    dist[tap] = (unsigned)(at / 3 * g.IW + at % 3) * 32u;
  }

  bf16x8 fa[3][TM], fb[3][TN];
  auto read_a = [&](int k) {
#pragma unroll
    for (int x = 0; x < TM; ++x) fa[k][x] = *(const __attribute__((address_space(3))) bf16x8*)(ldsb + rdA[x] + k * PART);
  };
  auto read_b = [&](int st, int k) {
#pragma unroll
    for (int y = 0; y < TN; ++y) fb[k][y] = f32_read_operand<B_KC>(ldsb, rdB, y, st * STAGE + k * B_PART);
  };
  u32x2 partW, partB[LB];
  auto split_filter = [&](auto set_tag, auto l_tag, auto step_tag, int st) {
    constexpr int SET = decltype(set_tag)::value, Lx = decltype(l_tag)::value;
    f32_split_step<decltype(step_tag)::value>(rawB[SET][Lx], partB[Lx], ldsb + wrB[Lx] + st * STAGE, B_PART);
  };
  auto split_window = [&](auto l_tag, auto at_tag, auto step_tag, int win) {
    constexpr int Lx = decltype(l_tag)::value;
    f32_split_step<decltype(step_tag)::value>(rawW[decltype(at_tag)::value], partW, ldsb + wrW + (win * WIN + Lx * 2048), PART);
  };

  // 64-wide tiles have registers left: the large sums of every nine or 18 k tiles are added up on their own (window_run_f32), so that they are
  // rounded no more often than those of a reduction split into many parts (roundings_f32 in jz_conv_f32.hip; the planner sees to it).  Behind
  // the products it costs at most 1 % over 35 layers (runs of 18 for every length: 28x28, 256 -> 512, backward-data 541 instead of 546 us).
  constexpr bool FOLD = BN == 64;
  f32x16 acc[TM][TN], low[TM][TN], sum[FOLD ? TM : 1][FOLD ? TN : 1];
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[x][y][r] = low[x][y][r] = 0.0f;
        if constexpr (FOLD) sum[x][y][r] = 0.0f;
      }
  const float end_run = window_run_f32(nk) == 9 ? 1.0f : 0.0f, keep_run = 1.0f - end_run;
  // The i-th of 16 TT sums, behind the second window (the products that follow start from the constant zero) or, where runs are nine k tiles,
  // behind the first.  Both products are exact.
  auto fold = [&](auto i_tag, auto window_tag) {
    constexpr int I = decltype(i_tag)::value, X = I / 16 / TN, Y = I / 16 % TN;
    f32x16& s = sum[FOLD ? X : 0][FOLD ? Y : 0];
    if constexpr (decltype(window_tag)::value == 0) {
      s[I % 16] = fmaf(acc[X][Y][I % 16], end_run, s[I % 16]);
      acc[X][Y][I % 16] *= keep_run;
    } else {
      s[I % 16] += acc[X][Y][I % 16];
      acc[X][Y][I % 16] = 0.0f;
    }
  };

  // The parts of the next tile are written behind the first kWritten products, the barrier that waits for them is kMeet products in, the operands
  // of the next tile's first groups are read behind it.  A window is taken apart during the last kWindowTiles taps.  Neither matters much: over 42
  // layers, both directions, 14 products of 24 before the barrier 0.6 % slower (4 % at most), 20 and the barrier 22 in 1.0 % (4 %), three taps 0.1 % (1 %).
  constexpr int kWritten = 18 * TT / 4, kMeet = 5 * TT;
  // Halves: the first during taps 3 and 4, then the other is requested, and taken apart during taps 7 and 8.
  constexpr int kWindowTiles = HALVES == 2 ? 2 : 5, kWindowSteps = LH * kSplitSteps;
  static_assert(kMeet >= 5 * TT && kWritten <= kMeet, "parts 0 and 1 of the pixels are multiplied for the last time by the fifth group of products");
  // the T-th of 18 k tiles: a tap of `chunk`
  auto tile = [&](int chunk, auto t_tag) {
    constexpr int T = decltype(t_tag)::value, TAP = T % TAPS, WINDOW = T / TAPS, PAR = T & 1, NEXT = 1 - PAR;
    constexpr int NEXT_TAP = (TAP + 1) % TAPS, NEXT_WINDOW = TAP + 1 == TAPS ? 1 - WINDOW : WINDOW;
    constexpr int kA[6] = {1, 0, 0, 1, 0, 2}, kB[6] = {1, 1, 0, 0, 2, 0};
    // the steps of taking the next window apart that fall to this tile
    constexpr int HALF = HALVES == 2 && TAP > 4 ? 1 : 0, SHARE = TAP - (HALVES == 2 && TAP <= 4 ? 3 : TAPS - kWindowTiles);
    constexpr int W0 = SHARE < 0 ? 0 : SHARE * kWindowSteps / kWindowTiles, W1 = SHARE < 0 ? 0 : (SHARE + 1) * kWindowSteps / kWindowTiles;
    constexpr int STEPS = kSplitSteps * LB + W1 - W0;
    read_b(PAR, 0);
    read_b(PAR, 2);
    read_a(2);
    sched_fence();
    static_for<0, 6 * TT>([&](auto s_tag) {
      constexpr int S = decltype(s_tag)::value, P = S / TT, X = S % TT / TN, Y = S % TN;
      if constexpr (S == kMeet) {
        f32_lds_meet();
        read_a(1);
        read_b(NEXT, 1);
        read_a(0);
        sched_fence();
      }
      f32x16& d = kA[P] + kB[P] == 0 ? acc[X][Y] : low[X][Y];
      // n operand in the first slot: each lane then owns 4 consecutive n for one m (row = lane % 32)
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kB[P]][Y], fa[kA[P]][X], d, 0, 0, 0);
      if constexpr (S < kWritten) {
        static_for<(S * STEPS + kWritten - 1) / kWritten, ((S + 1) * STEPS + kWritten - 1) / kWritten>([&](auto u_tag) {
          constexpr int U = decltype(u_tag)::value, W = W0 + U - kSplitSteps * LB;
          if constexpr (W < W0) {
            constexpr int Lx = U / kSplitSteps, K = U % kSplitSteps;
            constexpr std::integral_constant<int, (T + 1) % SETS> SET{};
            constexpr std::integral_constant<int, Lx> L{};
            split_filter(SET, L, std::integral_constant<int, K>{}, NEXT);
            if constexpr (K + 1 == kSplitSteps) request_filter(chunk + (TAP + 1 + SETS) / TAPS, (TAP + 1 + SETS) % TAPS, SET, L);
            if constexpr (U + 1 == kSplitSteps * LB && TAP == 0) static_for<0, LH>([&](auto w) { request_window(chunk + 1, w, w); });
          } else {
            constexpr int AT = W / kSplitSteps, K = W % kSplitSteps;
            constexpr std::integral_constant<int, AT> PLACE{};
            split_window(std::integral_constant<int, HALF * LH + AT>{}, PLACE, std::integral_constant<int, K>{}, 1 - WINDOW);
            if constexpr (HALVES == 2 && HALF == 0 && K + 1 == kSplitSteps) request_window(chunk + 1, std::integral_constant<int, LH + AT>{}, PLACE);
          }
        });
      }
      if constexpr (FOLD && TAP + 1 == TAPS && S > 3 * TT) {  // behind the products that follow the last large one (the third group)
        constexpr int FROM = S - 3 * TT - 1, OF = 3 * TT - 1;
        static_for<16 * TT * FROM / OF, 16 * TT * (FROM + 1) / OF>([&](auto i) { fold(i, std::integral_constant<int, WINDOW>{}); });
      }
      if constexpr (S >= 1 && S - 1 < TM) aim(S - 1, NEXT_WINDOW * WIN, dist[NEXT_TAP], NEXT_TAP);  // read_a(2) was the last of this tap
      sched_fence();
    });
  };
  if (nk > 0) {
    static_for<0, LP>([&](auto l) { static_for<0, kSplitSteps>([&](auto k) { split_window(l, l, k, 0); }); });
    constexpr std::integral_constant<int, 0> FIRST{};
    static_for<0, LB>([&](auto l) {
      static_for<0, kSplitSteps>([&](auto k) { split_filter(FIRST, l, k, 0); });
      request_filter(chunk0, SETS, FIRST, l);
    });
    f32_lds_meet();
#pragma unroll
    for (int x = 0; x < TM; ++x) aim(x, 0u, dist[0], 0);
    read_a(1);
    read_b(0, 1);
    read_a(0);
    sched_fence();
    for (int c = chunk0; c < chunk_end; c += 2) {
      static_for<0, 2 * TAPS>([&](auto k) { tile(c + decltype(k)::value / TAPS, k); });
    }
    if constexpr (FOLD) {
#pragma unroll
      for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y) acc[x][y] = sum[x][y];
    }
  }

  if (!f32_join_sums(acc, low, lane, wave)) {
    f32_dma_body<OP, BM, BN, F32_MASKS, true>(a, block, blocks);
    return;
  }
  t.template store<Lds::LDS_BYTES>(lds_f, [&](float* rows) { f32_put_rows<Tile::LDF>(rows, acc, lane); });
}

template <int OP, int BN, int LP>
__global__ __launch_bounds__(256, 2) void f32_window_kernel(F32Args a) {
  f32_window_body<OP, BN, LP>(a, blockIdx.x, gridDim.x);
}
