// FP32 implicit GEMM on the bfloat16 matrix instructions (included by jz_f32_kernels.h behind jz_f32_dma.h, whose F32Tile says what
// a workgroup loads and stores).
//
// An FP32 value is the sum of three bfloat16 values of eight significant bits each: p0 = a rounded to bfloat16, p1 = a - p0
// rounded, p2 = a - p0 - p1 (both differences and the last part are exact, the parts cover the 24 bits).  Of the nine products of
// two such sums the six of order 2^0 .. 2^-16 are added up, each exact in the FP32 accumulators; what is left out (two products of up
// to 2^-25 each, one of 2^-34) is at most 2^-24 of a product, what rounding the product to FP32 would lose, and of either sign.  The
// five smaller products have accumulators of their own: their sums are 2^-8 of the result, so their roundings do not count, and the
// large sums are rounded once in 16 k steps where the FP32 instructions round once in 4.  Errors measured against 64 bits are a third
// to two thirds of those of the FP32 instructions over the layers of ResNet-50 (one common set of accumulators would make them up to
// twice as large).
//
// Bfloat16 has FP32's exponents, so the last parts of a small value would fall below its normal range or out of it (unscaled, values
// below 2^-110 lost bits and subnormal ones all of them).  Every value is therefore multiplied by 2^24 on its way in and the sums by
// 2^-48: the last bit of the smallest FP32 value is then 2^-125, and no part of any value is subnormal.  It costs four vector
// instructions a load, 1.9 % of ResNet-50's operations at N = 64 (11.24 -> 11.45 ms).  Infinities, NaN, values of 2^104 and more (an
// infinite p0) and sums of 2^80 and more end in a result that is not finite: a workgroup that finds one in its tile computes the tile
// again with the FP32 instructions (f32_dma_body).
//
// Why: the FP32 matrix instructions reach 154 TFLOP/s and leave no issue slots beside them, the bfloat16 ones 1.9 PFLOP/s, 317 for
// six products.  Measured, FP32 instructions and parts: 3x3, 512 channels, 28x28, N = 64 1650 -> 1137 us (144 -> 208 TFLOP/s);
// 256 channels, 14x14 135 -> 96 us; 64 channels, 56x56 132 -> 94; 1x1 512 -> 128 on 28x28 68 -> 43; ResNet-50's operations at N = 64
// 13.94 -> 11.45 ms.
// What bounds it: issue slots, then, in long reductions, power.  A 32x32x16 product holds the matrix pipe for 32 cycles, eight issue slots of its SIMD;
// a loop of products with four vector instructions behind each runs at 95 % of the pipe, with four times as many behind every
// fourth at 68 %.  Taking the parts apart is 6.5 vector instructions a value.  A wavefront that did that for its own 64 + 64
// operand rows needed 7.3 of them per product (14x14 layer 129 us; v_dot2_f32_bf16 for the differences: 146).  So values are taken
// apart once per workgroup, on their way through registers into LDS, two instructions at a time between the products, and the
// operands are read from LDS as bfloat16: 4 to 5 instructions per product for 128x128 tiles.  On the 512-channel layer the pipes
// are then busy for 81 % of the compute units' busy cycles, without bank conflicts, at a clock that power holds at 1.4-1.5 GHz.  ResNet-50's
// own layers are not at that bound: 45-54 % in the main variants, 46 % over the stack, at 2.0-2.4 GHz under the profiler (short reductions:
// each workgroup's first tiles and its epilogue; the values of a 3x3 layer are taken apart once per tap, hence jz_f32_window.h).
//
// A tile's loads are requested two tiles ahead; the parts of tile i + 1 are made and written to the other of two stages between
// the products of tile i; one barrier a tile, in the last of the six groups of products.  LDS layouts of a part ("KC", "MC" as in jz_f32_dma.h): KC rows of 16 bfloat16, 16-byte half c of row r at place
// c ^ ((r >> 3) & 1); MC [16 k][rows], chunk c of eight at place c ^ 4 (k & 3) (64 rows: c ^ 2 (k & 3)), read with the transposing
// ds_read_b64_tr_b16.
#pragma once

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int BM, int BN>
struct F32Split {
  static constexpr int STAGE = 3 * (BM + BN) * FD_BK * 2;
  static constexpr int RING = FD_NST * (BM + BN) * FD_BK * 4;  // of f32_dma_body, in the same LDS
  static constexpr int LDS_BYTES = 2 * STAGE > RING ? 2 * STAGE : RING;
};

// Taking four values apart, in kSplitSteps steps of two vector instructions (the products hide four behind each of them): they are
// scaled, then the next eight bits of them go to LDS as part k at dst + k * part_bytes and, where another part follows, are taken
// off value by value (exact).
constexpr int kScaleSteps = 2, kSplitSteps = kScaleSteps + 11;
template <int STEP0>
__device__ __forceinline__ void f32_split_step(f32x4& v, u32x2& part, lds_byte* dst, int part_bytes) {
  constexpr int STEP = STEP0 - kScaleSteps, K = STEP / 5, E = STEP % 5 - 1;
  if constexpr (STEP < 0) {
    v[2 * STEP0] *= 0x1p24f;
    v[2 * STEP0 + 1] *= 0x1p24f;
  } else if constexpr (E < 0) {
    part = u32x2{__builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{v[0], v[1]}, bf16x2)),
                 __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{v[2], v[3]}, bf16x2))};
    *(__attribute__((address_space(3))) u32x2*)(dst + K * part_bytes) = part;
  } else {
    v[E] -= __builtin_bit_cast(float, E % 2 == 0 ? part[E / 2] << 16 : part[E / 2] & 0xffff0000u);
  }
}

// LDS offset of value (row, k 4 q .. 4 q + 3) of a KC part, and of (k, rows 4 q .. 4 q + 3) of an MC part of `rows` rows
__device__ __forceinline__ unsigned f32_kc_at(int row, int q) { return (unsigned)(row * 32 + (((q >> 1) ^ ((row >> 3) & 1)) * 16) + (q & 1) * 8); }
__device__ __forceinline__ unsigned f32_mc_at(int rows, int k, int q) {
  return (unsigned)(k * rows * 2 + (((q >> 1) ^ ((rows >= 128 ? 4 : 2) * (k & 3))) * 16) + (q & 1) * 8);
}
// Where a lane reads the operands of rows row0 .. of a part.  KC (one address): row r31, k 8 h .. 8 h + 7.  MC (two for each of the
// 32-row tiles): 16-lane group gi = lane / 16 reads half gi % 2 of the 32 rows and k block gi / 2; lane 4 j + c4 of the group addresses
// k-row j, the 8-byte piece c4 of those 16 rows.
template <bool KC, int TILES>
__device__ __forceinline__ void f32_read_addr(unsigned* rd, int lane, int row0, int rows, int base) {
  if constexpr (KC) {
    const int r31 = lane & 31, h = lane >> 5;
    rd[0] = (unsigned)(base + (row0 + r31) * 32 + ((h ^ ((r31 >> 3) & 1)) * 16));
  } else {
    const int gi = lane >> 4, j = (lane >> 2) & 3, c4 = lane & 3;
#pragma unroll
    for (int x = 0; x < TILES; ++x)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const int k = 8 * (gi >> 1) + 4 * hf + j, c = (row0 + 32 * x + 16 * (gi & 1) + 4 * c4) / 8;
        rd[2 * x + hf] = (unsigned)(base + k * rows * 2 + ((c ^ ((rows >= 128 ? 4 : 2) * (k & 3))) * 16) + (c4 & 1) * 8);
      }
  }
}
template <bool KC>
__device__ __forceinline__ bf16x8 f32_read_operand(lds_byte* ldsb, const unsigned* rd, int x, int off) {
  if constexpr (KC) return *(const __attribute__((address_space(3))) bf16x8*)(ldsb + rd[0] + (off + x * 1024));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  struct { s16x4 lo, hi; } v;
  v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(ldsb + rd[KC ? 0 : 2 * x] + off));
  v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(ldsb + rd[KC ? 0 : 2 * x + 1] + off));
  return __builtin_bit_cast(bf16x8, v);
}

// This wavefront's LDS writes have landed, and everyone else's; loads stay in flight.  Both sides of it are ordinary accesses,
// which the compiler may move across the barrier itself: the fences, of LDS alone, are what keeps them in place.
__device__ __forceinline__ void f32_lds_meet() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The two sums of every result added up and scaled back.  Whether all of the workgroup's are finite; every wavefront is past its
// last operand read then.
template <int TM, int TN>
__device__ __forceinline__ bool f32_join_sums(f32x16 (&acc)[TM][TN], f32x16 (&low)[TM][TN], int lane, int wave) {
  float odd = 0.f;  // 0 or, from a result that is not finite, NaN
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[x][y][r] = (acc[x][y][r] + low[x][y][r]) * 0x1p-48f;
        odd = fmaf(acc[x][y][r], 0.f, odd);
      }
  __shared__ int not_finite[4];
  const bool any = __ballot(odd != 0.f) != 0;
  if (lane == 0) not_finite[wave] = any;
  __syncthreads();  // and the tile is staged where the operands were
  return __builtin_amdgcn_readfirstlane(not_finite[0] | not_finite[1] | not_finite[2] | not_finite[3]) == 0;
}
// accumulator register r of tile (x,y): m = wrow + 32 x + lane % 32, n = wcol + 32 y + 8 (r / 4) + 4 (lane / 32) + r % 4
template <int LDF, int TM, int TN>
__device__ __forceinline__ void f32_put_rows(float* rows, const f32x16 (&acc)[TM][TN], int lane) {
  const int r31 = lane & 31, h = lane >> 5;
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(rows + (32 * x + r31) * LDF + 32 * y + 8 * q + 4 * h) =
            make_float4(acc[x][y][4 * q], acc[x][y][4 * q + 1], acc[x][y][4 * q + 2], acc[x][y][4 * q + 3]);
}

template <int OP, int BM, int BN, int FORM>
__device__ __forceinline__ void f32_split_body(const F32Args& a, unsigned block, unsigned blocks) {
  using Tile = F32Tile<OP, BM, BN, FORM, false>;
  using Lds = F32Split<BM, BN>;
  constexpr bool A_KC = Tile::A_KC, B_KC = Tile::B_KC;
  constexpr int TM = BM / 64, TN = BN / 64, TT = TM * TN;  // 32x32 MFMA tiles per wavefront
  constexpr int LA = Tile::LA, LPT = Tile::LPT;
  constexpr int A_PART = BM * FD_BK * 2, B_PART = BN * FD_BK * 2, B0 = 3 * A_PART, STAGE = Lds::STAGE;
  extern __shared__ __align__(16) float lds_f[];
  lds_byte* const ldsb = (lds_byte*)lds_f;
  Tile t(a, block, blocks);
  const int nk = t.nk, lane = t.lane, wave = t.wave, wm = t.wm, wn = t.wn;

  f32x4 raw[2][LPT];  // tiles on their way in
  // A tile that does not exist is requested too, out of range (zeros, nothing is fetched): a request under a condition would make
  // the compiler wait for all of them where one is used.
  struct Next {
    typename Tile::TileCtx c;
    unsigned none;
  };
  auto next = [&](int i) { return Next{t.tile_ctx(t.kt_begin + i), i < nk ? 0u : Tile::OOB}; };
  auto request = [&](const Next& n, auto set_tag, auto l_tag) {
    constexpr int SET = decltype(set_tag)::value, Lx = decltype(l_tag)::value;
    t.template load<Lx>(n.c, [&](__amdgpu_buffer_rsrc_t rsrc, unsigned voff, unsigned soff) {
      raw[SET][Lx] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(voff | n.none), (int)soff, 0));
    });
  };
  static_for<0, 2>([&](auto s_tag) {
    const Next n = next(decltype(s_tag)::value);
    static_for<0, LPT>([&](auto l_tag) { request(n, s_tag, l_tag); });
  });
  sched_fence();

  // ---- where a load's four values go in a part, where the operands are read ---------------------------
  unsigned wr[LPT];
#pragma unroll
  for (int l = 0; l < LPT; ++l) {
    const bool isA = l < LA;
    const int ii = isA ? l : l - LA, rows = isA ? BM : BN;
    if (isA ? A_KC : B_KC) wr[l] = f32_kc_at(64 * ii + t.kc_row, lane & 3);
    else wr[l] = f32_mc_at(rows, t.mc_k(rows, ii), lane % (rows / 4));
    if (!isA) wr[l] += (unsigned)B0;
  }
  unsigned rdA[A_KC ? 1 : 2 * TM], rdB[B_KC ? 1 : 2 * TN];
  f32_read_addr<A_KC, TM>(rdA, lane, wm * (BM / 2), BM, 0);
  f32_read_addr<B_KC, TN>(rdB, lane, wn * (BN / 2), BN, B0);

  bf16x8 fa[3][TM], fb[3][TN];
  auto read_a = [&](int st, int k) {
#pragma unroll
    for (int x = 0; x < TM; ++x) fa[k][x] = f32_read_operand<A_KC>(ldsb, rdA, x, st * STAGE + k * A_PART);
  };
  auto read_b = [&](int st, int k) {
#pragma unroll
    for (int y = 0; y < TN; ++y) fb[k][y] = f32_read_operand<B_KC>(ldsb, rdB, y, st * STAGE + k * B_PART);
  };
  // what the first two groups of products need, and what the last group leaves free
  auto read_first = [&](int st) {
    read_a(st, 1);
    read_b(st, 1);
    read_a(st, 0);
  };

  // step K of taking load l of register set SET apart
  constexpr int kSteps = kSplitSteps;
  u32x2 part[LPT];
  auto split_step = [&](auto set_tag, auto l_tag, auto step_tag, int st) {
    constexpr int Lx = decltype(l_tag)::value;
    f32_split_step<decltype(step_tag)::value>(raw[decltype(set_tag)::value][Lx], part[Lx], ldsb + wr[Lx] + st * STAGE, Lx < LA ? A_PART : B_PART);
  };

  f32x16 acc[TM][TN], low[TM][TN];
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = low[x][y][r] = 0.0f;

  // The parts of the next tile are written behind kWritten of the 6 TT products, the barrier that waits for them is kMeet products
  // in, with the reads of read_first behind it.  20 and 22 of 24; ResNet-50's operations at N = 64 with 18 and 22 11.50 ms, 20 and 22
  // 11.39, 21 and 22 11.43, 20 and 23 11.43.
  constexpr int kWritten = TT == 1 ? 5 : 5 * TT, kMeet = 11 * TT / 2;
  // Tile i out of stage PAR = i & 1.
  auto tile = [&](int i, auto par_tag) {
    constexpr int PAR = decltype(par_tag)::value, NEXT = 1 - PAR;
    constexpr int kA[6] = {1, 0, 0, 1, 0, 2}, kB[6] = {1, 1, 0, 0, 2, 0};
    const Next n = next(i + 3);
    read_b(PAR, 0);
    read_b(PAR, 2);
    read_a(PAR, 2);
    sched_fence();
    static_for<0, 6 * TT>([&](auto s_tag) {
      constexpr int S = decltype(s_tag)::value, P = S / TT, X = S % TT / TN, Y = S % TN;
      if constexpr (S == kMeet) {
        f32_lds_meet();
        read_first(NEXT);
        sched_fence();
      }
      f32x16& d = kA[P] + kB[P] == 0 ? acc[X][Y] : low[X][Y];
      // n operand in the first slot: each lane then owns 4 consecutive n for one m (row = lane % 32)
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kB[P]][Y], fa[kA[P]][X], d, 0, 0, 0);
      if constexpr (S < kWritten) {
        constexpr int STEPS = kSteps * LPT;
        static_for<(S * STEPS + kWritten - 1) / kWritten, ((S + 1) * STEPS + kWritten - 1) / kWritten>([&](auto u_tag) {
          constexpr int U = decltype(u_tag)::value, Lx = U / kSteps, K = U % kSteps;
          split_step(std::integral_constant<int, NEXT>{}, std::integral_constant<int, Lx>{}, std::integral_constant<int, K>{}, NEXT);
          if constexpr (K + 1 == kSteps) request(n, std::integral_constant<int, NEXT>{}, std::integral_constant<int, Lx>{});
        });
      }
      sched_fence();
    });
  };
  constexpr std::integral_constant<int, 0> EVEN{};
  constexpr std::integral_constant<int, 1> ODD{};
  if (nk > 0) {
    const Next n = next(2);
    static_for<0, LPT>([&](auto l_tag) {
      static_for<0, kSteps>([&](auto k_tag) { split_step(EVEN, l_tag, k_tag, 0); });
      request(n, EVEN, l_tag);
    });
    f32_lds_meet();
    read_first(0);
    sched_fence();
    // Behind an odd number of tiles there is one of zeros: with a condition around it the waits would count for a path without
    // it, an exit in front of it doubles the accumulators' registers.
    for (int i = 0; i < nk; i += 2) {
      tile(i, EVEN);
      tile(i + 1, ODD);
    }
  }

  if (!f32_join_sums(acc, low, lane, wave)) {
    f32_dma_body<OP, BM, BN, FORM>(a, block, blocks);
    return;
  }
  t.template store<Lds::LDS_BYTES>(lds_f, [&](float* rows) { f32_put_rows<Tile::LDF>(rows, acc, lane); });
}

template <int OP, int BM, int BN, int FORM, bool PARTS>
__device__ __forceinline__ void f32_body(const F32Args& a, unsigned block, unsigned blocks) {
  if constexpr (PARTS) f32_split_body<OP, BM, BN, FORM>(a, block, blocks);
  else f32_dma_body<OP, BM, BN, FORM>(a, block, blocks);
}
template <int OP, int BM, int BN, int FORM, bool PARTS>
__global__ __launch_bounds__(256, PARTS ? 2 : 1) void f32_kernel(F32Args a) {
  f32_body<OP, BM, BN, FORM, PARTS>(a, blockIdx.x, gridDim.x);
}

template <int BM, int BN, int FORM, bool PARTS>
__global__ __launch_bounds__(256, PARTS ? 2 : 1) void f32_set_kernel(F32Set s) {
  int k = 0;
  while (k + 1 < FD_MAX_SET && blockIdx.x >= s.first[k + 1]) ++k;
#if defined(__HIP_DEVICE_COMPILE__)
  // the member where it lies among the kernel's arguments: indexing the argument copies all of it to scratch memory first
  const F32Set& set = *(const F32Set*)(const __attribute__((address_space(4))) F32Set*)__builtin_amdgcn_kernarg_segment_ptr();
#else
  const F32Set& set = s;
#endif
  f32_body<OP_BWD_DATA, BM, BN, FORM, PARTS>(set.c[k], blockIdx.x - s.first[k], s.first[k + 1] - s.first[k]);
}
