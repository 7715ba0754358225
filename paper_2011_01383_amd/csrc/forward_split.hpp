// Forward kernels that contract on the bf16 matrix units with fp32 accuracy.
//
// Every fp32 operand x is split into three bf16 planes, x = p0 + p1 + p2 (each
// the round-to-nearest bf16 of what the planes before it leave: 3 x 8 significant
// bits, exact from |x| of about 2^-110; below, the third plane meets the end of
// bf16's range and up to 2^-134 is lost), and a product a*b is taken as the six
// plane products of order 2^-16 and above,
//   a0 b0  +  (a0 b1 + a1 b0 + a1 b1 + a0 b2 + a2 b0),
// the first in an accumulator of its own.  The dropped terms, a1 b2 + a2 b1 + a2 b2,
// reach 2^-24 of |a b| at worst (a = b = 1.0039: 2^-24.01) and pass 2^-26 for 3.6%
// of N(0,1) x U(-0.05, 0.05) products: about one fp32 rounding of the product, as
// every fp32 multiplication makes.  A 16x16x32 bf16 MFMA takes 16 cycles, so
// 32 k cost 96 cycles against 256 on the fp32 MFMA (8 x 32), and the sums are
// closer to the exact ones: against 64 bits, dot products of N(0,1) rows with
// U(-0.05, 0.05) weights are off by 0.47e-7 / 0.84e-7 / 1.75e-7 (2-norm,
// K = 64 / 256 / 1024) against 1.06e-7 / 2.04e-7 / 4.00e-7 for fp32 MFMA
// chains, since the large products are rounded K/32 times instead of K/4.
// (With all six products in one accumulator the unit's truncation of small
// addends shows: 0.91e-7 / 2.3e-7 / 4.9e-7.)
//
// Values that round to infinity in bf16 (infinities, |x| >= 3.396e38) cannot be
// split, and where products of finite values leave the fp32 range, plane products
// of both signs would (hi + lo is then infinity minus infinity).  Where a tile's
// operands or the weights allow either (split_limit), every wave forms its partial
// sums of the tile again on the fp32 matrix unit, operands and weights read from
// memory (one infinite weight, every tile of one slice: 64 grids 402 -> 1,757 us,
// 200 N-ary trees 188 -> 499, 200 child-sum trees 278 -> 576).  NaN needs no such
// path: it stays NaN in every plane.
#pragma once

namespace cortex {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

struct Split8 {
  bf16x8 p0, p1, p2;
};

// Two values rounded to bf16 (the first in the low half), and what that leaves of them.
__device__ __forceinline__ unsigned int bf16_pair(float a, float b) {
  const floatx2 v = {a, b};
  const bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(unsigned int, r);
}
__device__ __forceinline__ void bf16_rest(unsigned int pair, float &a, float &b) {
  a -= as_float(pair << 16);
  b -= as_float(pair & 0xFFFF0000u);
}

__device__ __forceinline__ Split8 split8(const float4 x, const float4 y) {
  float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
  u32x4 p[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    unsigned int q[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      q[k] = bf16_pair(v[2 * k], v[2 * k + 1]);
      if (i < 2) bf16_rest(q[k], v[2 * k], v[2 * k + 1]);
    }
    p[i] = u32x4{q[0], q[1], q[2], q[3]};
  }
  return Split8{__builtin_bit_cast(bf16x8, p[0]), __builtin_bit_cast(bf16x8, p[1]), __builtin_bit_cast(bf16x8, p[2])};
}

// f(integral_constant 0), ..., f(integral_constant N - 1): indices into register
// arrays stay compile-time constants through nested lambdas (a loop variable
// there would put the arrays in scratch memory).
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Largest magnitude (NaN ignored), and the magnitude from which it cannot be split.
constexpr float kSplitLimit = 3.3961775e38f;
__device__ __forceinline__ float max_abs(float m, const float4 v) {
  return fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
}
// The operand magnitude from which a wave whose weights reach wmax (this lane's
// share of them) must not use the planes: below it no sum of `terms` products can
// pass half of FLT_MAX, so no plane product or sum of them overflows.  Every
// magnitude, zero included, when a weight itself cannot be split.  Called by
// whole waves; the same value in every lane.
__device__ __forceinline__ float split_limit(float wmax, int terms) {
  // (rotations within 16 lanes, then one lane of each: no index registers, as
  // shuffles would take)
  static_for<4>([&](auto i) __attribute__((always_inline)) {
    const int x = (int)as_uint(wmax);
    wmax = fmaxf(wmax, as_float((unsigned int)__builtin_amdgcn_update_dpp(x, x, 0x120 + (8 >> i), 0xf, 0xf, false)));
  });
  const int x = (int)as_uint(wmax);
  wmax = fmaxf(fmaxf(as_float((unsigned int)__builtin_amdgcn_readlane(x, 0)), as_float((unsigned int)__builtin_amdgcn_readlane(x, 16))),
               fmaxf(as_float((unsigned int)__builtin_amdgcn_readlane(x, 32)), as_float((unsigned int)__builtin_amdgcn_readlane(x, 48))));
  const float limit = wmax >= kSplitLimit ? -1.f : fminf(kSplitLimit, 1.6e38f / ((float)terms * wmax));
  return as_float(__builtin_amdgcn_readfirstlane(as_uint(limit)));     // (a scalar register)
}

// The thread index, opaque to the compiler: what is derived from it is formed
// where it is used, not kept in registers through the loops around it.
__device__ __forceinline__ int fresh_tid() {
  int x = threadIdx.x;
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ floatx4 mfma_bf16(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 32 k of NT output tiles that share one A fragment: the six plane products,
// issued product-major so that consecutive MFMAs write different accumulators.
// between(i) runs after product i (0..5): loads placed there, one at a time, do
// not queue up ahead of the MFMAs in the address unit (64 bytes per clock).
template <int NT, typename Between>
__device__ __forceinline__ void mfma_split(const Split8 &a, const Split8 (&w)[NT], floatx4 (&hi)[NT], floatx4 (&lo)[NT],
                                           Between between) {
  static_for<6>([&](auto i) __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if constexpr (i == 0) lo[nt] = mfma_bf16(a.p2, w[nt].p0, lo[nt]);
      if constexpr (i == 1) lo[nt] = mfma_bf16(a.p1, w[nt].p1, lo[nt]);
      if constexpr (i == 2) lo[nt] = mfma_bf16(a.p0, w[nt].p2, lo[nt]);
      if constexpr (i == 3) lo[nt] = mfma_bf16(a.p1, w[nt].p0, lo[nt]);
      if constexpr (i == 4) lo[nt] = mfma_bf16(a.p0, w[nt].p1, lo[nt]);
      if constexpr (i == 5) hi[nt] = mfma_bf16(a.p0, w[nt].p0, hi[nt]);
    }
    between(i);
  });
}

// Exclusive prefix sum of one value per thread over the workgroup; wsum
// holds kFwdWaves + 1 ints of LDS.  Returns the exclusive sum, *total the sum.
__device__ __forceinline__ int block_excl_scan(int v, int *wsum, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int w = 0; w < kFwdWaves; ++w) {
      const int t = wsum[w];
      wsum[w] = run;
      run += t;
    }
    wsum[kFwdWaves] = run;
  }
  __syncthreads();
  const int ex = wsum[wave] + x - v;
  *total = wsum[kFwdWaves];
  __syncthreads();
  return ex;
}

// One block's four values: staged (two pairs of (value, tag) pairs) or plain.
// (By value: a choice between elements of the operand arrays would be made on
// their addresses and put the arrays in scratch memory.)
__device__ __forceinline__ float4 pick_block(bool staged, u32x4 lo, u32x4 hi, u32x4 plain) {
  const unsigned int a = staged ? lo.x : plain.x, b = staged ? lo.z : plain.y;
  const unsigned int c = staged ? hi.x : plain.z, d = staged ? hi.z : plain.w;
  return make_float4(as_float(a), as_float(b), as_float(c), as_float(d));
}

// ---------------------------------------------------------------------------
// The tiles of a node group, listed in LDS at entry with the operand sources of
// their rows, so that the level loop never reads the linearization and the next
// tile's operands can be requested across a level boundary.  A record is
//   row0, level end, level, level start (then -1 where a tile's operands cannot
//   be split), codes[16][CODES]
// (the codes of SrcCfg).  A group with more tiles than the list holds runs them
// a listed chunk at a time.
// ---------------------------------------------------------------------------
template <int CODES>
struct TileList {
  static constexpr int kHead = 4, kInts = kHead + kTileM * CODES;
};

// Records the tiles [first, first + cap) of this group over the levels
// [lo, hi) (row0 .. level; the codes are filled by the caller); returns the
// group's tile count.  One level per thread per round.  off(l) is the first row
// of level l; *bad is set when the offsets are not monotone from 0 to N.
template <int INTS, int ROWS = kTileM, typename Off>
__device__ __forceinline__ int list_tiles(const Off &off, int L, int N, int lo, int hi, int group, int Q, int first, int cap,
                                          int tid, int *list, int *wsum, int &bad) {
  int total = 0;
  for (int lb = 0; lb < L; lb += kFwdThreads) {
    const int l = lb + tid;
    int cnt = 0, r0 = 0, r1 = 0, uf = 0;
    if (l < L) {
      r0 = off(l);
      r1 = off(l + 1);
      const bool ok = r0 >= 0 && r1 >= r0 && r1 <= N && (l != 0 || r0 == 0) && (l != L - 1 || r1 == N);
      if (!ok) bad = 1;
      const int ntile = (ok && l >= lo && l < hi) ? (r1 - r0 + ROWS - 1) / ROWS : 0;
      uf = ((group - l) % Q + Q) % Q;
      cnt = uf < ntile ? (ntile - 1 - uf) / Q + 1 : 0;
    }
    int round_total;
    const int pos = total + block_excl_scan(cnt, wsum, &round_total) - first;
    for (int j = max(0, -pos); j < cnt && pos + j < cap; ++j) {
      int *t = &list[(pos + j) * INTS];
      t[0] = r0 + ROWS * (uf + j * Q);
      t[1] = r1;
      t[2] = l;
      t[3] = r0;
    }
    total += round_total;
  }
  return total;
}

// Deep, narrow batches.  A level that gives every group one tile at most costs
// the exchange and that tile, and the fp32 kernels' tile is the shorter one by 0.2
// to 0.7 us: its operands need no splitting, and the narrower slices have less
// epilogue.  The level count is known on the device only, so the split kernels
// hold the fp32 form as well and take it, every workgroup alike, where the levels
// above the leaves have fewer than `rows` rows on average, or fewer than `even` and
// the lowest of them less than twice the average (chains: in random trees it has
// four times the average or more, and that is where the split kernels gain).
//
// us per step, split / fp32 form, at rows per level:
//   N-ary TreeLSTM     16 918 / 824, 32 490 / 453, 41 (random) 105 / 115, 64 195 / 257
//   TreeRNN 256        J = 16: 32 202 / 191, 58 (random) 98 / 108, 64 142 / 137,
//                      96 91 / 96; J = 64: 64 239 / 203, 128 146 / 141, 130 (random)
//                      138 / 158, 192 125 / 135
//   TreeRNN 512        16 520 / 431, 58 (random) 163 / 174, 64 243 / 222, 96 256 / 256,
//                      128 136 / 150
//   child-sum          16 580 / 528, 32 378 / 366, 48 343 / 349, 64 345 / 433;
//                      linearization in LDS: 48 170 / 155, 60 (random) 111 / 121,
//                      64 147 / 141, 96 91 / 109
struct NarrowRule {
  int rows, even;
};
// off1, off2: first rows of levels 1 and 2.  (A scalar, and no branches: the rest
// of the kernel must stay in uniform control flow.)
__device__ __forceinline__ bool narrow_levels(int off1, int off2, int N, int L, NarrowRule r) {
  const int64_t above = L - 1, inner = N - off1, lowest = off2 - off1;
  const int narrow = (L > 1) & ((inner < r.rows * above) | ((inner < r.even * above) & (lowest * above < 2 * inner)));
  return __builtin_amdgcn_readfirstlane(narrow) != 0;
}

// ---------------------------------------------------------------------------
// TreeRNN, N-ary TreeLSTM and DAG-RNN at H = 256 and 512.
//
// Partition: workgroup b owns hidden slice b / Q (J units, all their gates) and
// node group b % Q, which takes the 16-row tiles u of level l with
// (u + l) % Q == group; a group's slices sit on one XCD when Q is a multiple
// of 8 (round-robin dispatch).  Wave w contracts H/4 columns of child slot w / 4
// (and H/8 columns of the node input, DAG-RNN); its weight fragments stay in
// registers, already split, for the whole launch.
//
// What bounds it: on narrow levels the chain of exchanges between workgroups
// (about 2 us each) and the one tile's contraction; on wide ones the number of
// tiles per group, and every slice loading the tile's operand rows again.  So
// wide batches take wide slices (J = 16 or 64: fewer, fuller tiles per group and
// fewer loads of each row), small ones narrow slices, whose tile costs less.
//
// Per tile: the input part, which waits for nothing; the wait for the children;
// per 32 columns, the split of the operands, the request of the next tile's and
// the MFMAs.  The eight partial sums meet in LDS, where four of the waves sum
// them and apply the gates (waves 0-3 for even tiles, 4-7 for odd ones) while
// the others go on to the next tile: one workgroup barrier per tile.
//
// A staged pair's first load, before any poll, carries no device-scope bit: the
// slices of a group then share their XCD's L2, and a stale line only shows an
// old tag, after which the polls are device-scope.
// ---------------------------------------------------------------------------
template <int CELL, int H, int J_, bool kHoisted = false>
struct SplitDims {
  static constexpr int J = J_, GATES = Cell<CELL, H>::GATES, GJ = GATES * J, NT = (GJ + 15) / 16;
  static constexpr bool kDag = CELL == CELL_DAG;
  static constexpr int CODES = SrcCfg<CELL>::SEGS;
  static constexpr int KX = kDag && !kHoisted ? H / 8 : 0, XS = KX / 32;          // input columns per wave, 32-column steps
  static constexpr int KR = 2 * H / 8, RS = KR / 32;                  // recurrent columns per wave
  // row stride of the partial sums: 4 rows apart is 16 banks apart, so neither
  // the MFMA-layout writes nor the unit-major reads conflict
  static constexpr int LDC = 16 * NT + 4;
  static constexpr int kPairs = kTileM * J;                           // (row, unit) pairs of a tile
  // DAG-RNN with 64 units: the input weights' planes sit in LDS (96 KB: in
  // registers they spill, 64 grids 570 against 385 us), so there is one buffer of
  // partial sums, and every thread takes part in the epilogue
  static constexpr bool kWxLds = XS > 0 && J == 64;
  static constexpr int ET = kDag && J == 64 ? 512 : 256;                       // epilogue threads
  static constexpr int PP = kPairs > ET ? kPairs / ET : 1;            // pairs per epilogue thread
  static constexpr int RSTEP = J == 64 ? ET / 64 : 4;                 // rows between a thread's pairs
  static constexpr int PARTS = kPairs < 256 ? 256 / kPairs : 1;       // threads per pair
  static constexpr NarrowRule kNarrowRule = CELL == CORTEX_NARY_TREELSTM ? NarrowRule{36, 36}
                                            : J == 64 ? NarrowRule{64, 150} : J == 32 ? NarrowRule{40, 100} : NarrowRule{40, 72};
  static_assert(KR % 32 == 0 && (!kDag || KX % 32 == 0) && 4 * KR == H, "whole 32-column steps, one child slot per wave");
  static_assert(PARTS <= 8 && H % J == 0 && J <= 64, "epilogue mapping");
};

// Bytes of dynamic LDS: the list; fused launches (DAG-RNN) add the linearizer's
// arrays.
template <int CODES>
constexpr size_t split_list_bytes(int cap) { return (size_t)cap * TileList<CODES>::kInts * sizeof(int); }
constexpr int kSplitCap = 128, kSplitFusedCap = 48;

// The kernel's arguments read again from the kernel argument segment, for a branch
// that shares nothing with the rest of the kernel: no argument register has to
// live across both (the LSTM cells; TreeRNN, with fewer, spills more scalars so).
__device__ __forceinline__ FwdArgs fresh_args() {
  typedef const __attribute__((address_space(4))) FwdArgs *Ptr;
  Ptr p = (Ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const FwdArgs *)p;
}

// kHoisted (ablation, DAG-RNN with 64 units): W x + b of every row is read from
// a.pre instead of being contracted here.  kNarrow: holds the form for deep, narrow
// batches, with the linearization in LDS (2) or not (1).
template <int CELL, int H, int J, bool kFused, bool kWeightsFromMemory = false, bool kHoisted = false, int kNarrow = 0>
__global__ void __launch_bounds__(kFwdThreads) slice_split_kernel(FwdArgs a) {
  using D = SplitDims<CELL, H, J, kHoisted>;
  using TL = TileList<D::CODES>;
  constexpr int NT = D::NT, XS = D::XS, RS = D::RS, GATES = D::GATES, LDC = D::LDC, PP = D::PP, PARTS = D::PARTS;
  constexpr int INTS = TL::kInts, HEAD = TL::kHead, CODES = D::CODES;
  constexpr bool kDag = D::kDag, kLstm = CELL == CORTEX_NARY_TREELSTM, kLeafInputs = !kDag;
  constexpr int kCap = kFused ? kSplitFusedCap : kSplitCap;
  constexpr int CBUF = kFwdWaves * kTileM * LDC;

  constexpr bool kWxLds = D::kWxLds, kOneBuffer = D::ET == 512;
  constexpr int WXP = XS * NT * kFwdThreads;    // one plane of the input weights, [step][tile][thread]
  constexpr int CS = (kOneBuffer ? 1 : 2) * CBUF;
  typedef SliceLds<CELL, H, Cell<CELL, H>::J> NarrowLds;
  constexpr int kPool = kNarrow && sizeof(NarrowLds) > CS * sizeof(float) ? (int)(sizeof(NarrowLds) + 3) / 4 : CS;
  __shared__ __attribute__((aligned(16))) float C_s[kPool];
  __shared__ u32x4 Wx_s[kWxLds ? 3 * WXP : 1];
  __shared__ int wsum[kFwdWaves + 1];
  __shared__ int stop_s[2];
  extern __shared__ int dyn[];
  int *list = dyn;                              // [kCap][INTS]

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g4 = lane >> 4;
  const int Q = a.Q, slice = blockIdx.x / Q, group = blockIdx.x % Q;
  const int hbase = slice * J, N = a.N, K = a.K;
  const uint32_t tag = launch_tag(a.sync);      // read with the status: one round trip
  const TagBuf hs(a.hs, (uint32_t)N * H * 8);
  const TagBuf cs(a.cs, kLstm ? (uint32_t)N * H * 8 : 0u);
  const InBuf xin(kDag ? (const void *)a.x : (const void *)a.x_table,
                  kDag ? (uint32_t)N * H * 4 : (a.x_table ? (uint32_t)a.x_rows * H * 4 : 0u));
  const InBuf pin(a.pre, kHoisted ? (uint32_t)N * H * 4 : 0u);
  const int rslot = wave >> 2, rcol = D::KR * (wave & 3) + 4 * g4;    // child slot; lane's first column in it
  const int xcol = D::KX * wave + 4 * g4;
  // epilogue: unit ej, part epart of the eight partial sums, rows erow + 4 p
  const int et = tid & (D::ET - 1), eside = kOneBuffer ? 0 : tid >> 8;
  const int ej = et % J, epart = J >= 16 ? 0 : (et & 15) / J;
  const int erow = J == 64 ? et >> 6 : (J == 32 ? 8 * ((et >> 5) & 1) + (et >> 6) : 4 * ((et >> 4) & 3) + (et >> 6));

  CORTEX_TRACE_KERNEL(0);
  const int status0 = load_status(a.status);
  // (before the weights: which form of the kernel runs is known when they are still on their way)
  int L = 0, off1 = 0, off2 = 0;
  if constexpr (!kFused) {
    L = *a.num_levels;
    off1 = a.level_offsets[1];
    if constexpr (kNarrow) off2 = a.level_offsets[N > 1 ? 2 : 1];
  }
  if (tid < 2) stop_s[tid] = 0;

  // ---- weights: fragment (step s, tile nt) = gate row 16 nt + i16, two
  // 16-column blocks of the step's 32 columns, four columns of each per lane
  auto wcol = [&](int s, int half) __attribute__((always_inline)) -> int {
    const int o = 32 * s + 16 * half;
    if (kDag) return s < XS ? xcol + o : H + rslot * H + rcol + o - 32 * XS;
    return rslot * H + rcol + o;
  };
  auto wfrag = [&](int s, int nt, int half, int row) __attribute__((always_inline)) -> float4 {
    return weight_slice_at<CELL, H, J>(a, hbase, 16 * nt + row, wcol(s, half));
  };
  constexpr int WS = kWeightsFromMemory ? 1 : XS + RS;
  constexpr int W0 = kWxLds ? XS : 0;           // steps whose weights are in LDS
  Split8 w[WS - W0][NT];
  float wmax = 0.f;
  float bias[GATES];
#pragma unroll
  for (int g = 0; g < GATES; ++g) bias[g] = a.b[g * H + hbase + ej];
  auto split_weights = [&](const float4 (&v)[WS][NT][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < WS; ++s)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        wmax = max_abs(max_abs(wmax, v[s][nt][0]), v[s][nt][1]);
        const Split8 p = split8(v[s][nt][0], v[s][nt][1]);
        if (s < W0) {
          // (each lane reads back only what it wrote: no barrier)
          u32x4 *o = &Wx_s[(s * NT + nt) * kFwdThreads + tid];
          o[0] = __builtin_bit_cast(u32x4, p.p0);
          o[WXP] = __builtin_bit_cast(u32x4, p.p1);
          o[2 * WXP] = __builtin_bit_cast(u32x4, p.p2);
        } else {
          w[s - W0 < 0 ? 0 : s - W0][nt] = p;
        }
      }
  };

  // ---- structure: the group's tiles and their operand sources ----
  int bad = 0, total = 0, listed = 0;
  SmallLin m;
  auto row_of_slot = [&](int idx) __attribute__((always_inline)) -> int {
    const int *t = &list[(idx / kTileM) * INTS];
    const int row = t[0] + idx % kTileM;
    return row < t[1] ? row : -1;
  };
  const int lvl_lo = kLeafInputs ? max(a.level_lo, 1) : a.level_lo;
  auto fill_fused = [&](int tid) __attribute__((always_inline)) {
    for (int idx = tid; idx < listed * kTileM; idx += kFwdThreads) {
      const int row = row_of_slot(idx);
      int *cd = &list[(idx / kTileM) * INTS + HEAD + (idx % kTileM) * CODES];
      const int v = row >= 0 ? m.order[row] : -1;
      cd[0] = v >= 0 ? -2 - v : -1;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int c = (v >= 0 && s < K) ? m.ch[v * K + s] : -1;
        cd[s + 1] = c >= 0 ? m.nrow[c] : -1;
      }
    }
  };
  // (three dependent loads per leaf child: child row, its node, its input row;
  // every slot of the chunk at once, so they cost one chain per chunk)
  auto fill_global = [&](int tid) __attribute__((always_inline)) {
    for (int idx = tid; idx < listed * kTileM; idx += kFwdThreads) {
      const int row = row_of_slot(idx);
      const int *t = &list[(idx / kTileM) * INTS];
      int *cd = const_cast<int *>(t) + HEAD + (idx % kTileM) * CODES;
      int c[2] = {-1, -1}, v = -1;
      if (row >= 0) {
#pragma unroll
        for (int s = 0; s < 2; ++s) c[s] = s < K ? a.child_rows[(size_t)row * K + s] : -1;
        if (kDag) {
          v = a.level_nodes[row];
          if (v < 0 || v >= N) {
            bad = 1;
            v = -1;
          }
        }
      }
      if (kDag) cd[0] = v >= 0 ? -2 - v : -1;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (c[s] < -1 || c[s] >= t[3]) {         // a child must sit in a lower level
          bad = 1;
          c[s] = -1;
        }
        if (kLeafInputs && !(a.ablate & 2) && c[s] >= 0 && c[s] < off1) {     // a leaf child: its input row
          const int lv = a.level_nodes[c[s]];
          int xi = -1;
          if (lv < 0 || lv >= N) bad = 1;
          else xi = a.x_index[lv];
          if (xi < -1 || xi >= a.x_rows) {
            raise_status(a.status, CORTEX_ST_INPUT_RANGE);
            xi = -1;
          }
          c[s] = xi >= 0 ? -2 - xi : -1;
        }
        cd[kDag ? s + 1 : s] = c[s];
      }
    }
  };
  auto list_chunk = [&](int first) __attribute__((always_inline)) {
    const int tid = fresh_tid();               // (nothing is kept through the tile loop for the next chunk)
    if constexpr (kFused) {
      total = list_tiles<INTS>([&](int l) { return l < L ? m.lcount[l] : N; }, L, N, lvl_lo, a.level_hi, group, Q, first,
                               kCap, tid, list, wsum, bad);
      listed = min(total - first, kCap);
      __syncthreads();
      fill_fused(tid);
    } else {
      total = list_tiles<INTS>([&](int l) { return a.level_offsets[l]; }, L, N, lvl_lo, a.level_hi, group, Q, first, kCap,
                               tid, list, wsum, bad);
      listed = min(total - first, kCap);
      if (__syncthreads_or(bad)) return;
      fill_global(tid);
    }
  };

  // (fused: the weight loads share the round trip of the linearizer's children)
  float4 wv[WS][NT][2];
  if constexpr (!kWeightsFromMemory) {
#pragma unroll
    for (int s = 0; s < WS; ++s)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) wv[s][nt][hf] = wfrag(s, nt, hf, i16);
  }
  if constexpr (kFused) {
    static_assert(kDag && !kWeightsFromMemory, "the DAG-RNN without ablations");
    L = small_linearize<kFwdThreads, kFusedPer>(a.children, N, K, a.status, dyn + kCap * INTS, m, fused_lin_stamps(a));
    if (L == 0) return;
    if (blockIdx.x == 0)
      small_lin_emit<kFwdThreads>(m, N, K, L, a.o_num_levels, a.o_height, a.o_level_offsets, a.o_level_nodes, a.o_node_row,
                                  a.o_child_rows);
    CORTEX_TRACE_KERNEL(9);
    CORTEX_TRACE_KERNEL(10);
    if (status0 != 0) return;
  } else {
    if (status0 != 0) return;
    if (L < 1 || L > N) {
      raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
      return;
    }
    if constexpr (kNarrow) {
      static_assert(kLeafInputs && !kWeightsFromMemory, "leaf-input cells");
      if (a.narrow_q > 0 && narrow_levels(off1, off2, N, L, D::kNarrowRule)) {
        NarrowLds &n = *(NarrowLds *)C_s;
        const FwdArgs b = kLstm ? fresh_args() : a;
        slice_forward<CELL, H, Cell<CELL, H>::J, kNarrow == 2>(b, b.narrow_q, n.W_s, n.C_s, n.Z_s, n.bias_s, n.chunk, dyn);
        return;
      }
    }
  }
  if constexpr (!kWeightsFromMemory) {
    split_weights(wv);
  } else {
#pragma unroll 1
    for (int k = 0; k < (XS + RS) * NT * 2; ++k) wmax = max_abs(wmax, wfrag(k / (2 * NT), k / 2 % NT, k & 1, i16));
  }
  const float limit = split_limit(wmax, D::KX + D::KR);
  constexpr float kLeast = kDag ? 1.f : 0.f;    // (DAG-RNN: every staged value is a tanh)

  int gave_up = 0, lvl = lvl_lo;
  u32x4 flo[2 * RS], fhi[2 * RS];     // staged child pairs: block b = columns rcol + 16 b .. +3
  u32x4 fp[kLeafInputs ? 2 * RS : 1]; // the same columns of a leaf child's input row
  u32x4 xv[XS > 0 ? 2 * XS : 1];      // DAG-RNN input: columns xcol + 16 b .. +3
  int cd = -1;                        // source code of this lane's row and child slot
  u32x2 cc[2];                        // N-ary: the children's memory cells of this thread's next epilogue
  int ce[2] = {-1, -1};

  auto code = [&](const int *t, int i, int seg) __attribute__((always_inline)) -> int {
    return t[0] + i < t[1] ? t[HEAD + i * CODES + seg] : -1;
  };
  // Requests of a tile's operands for source code c, one load each: every lane
  // issues both kinds (an offset beyond the buffer reads zeros without touching
  // memory), so nothing branches between the MFMAs they are placed among.
  constexpr int kLoads = kLeafInputs ? 6 * RS : 4 * RS;
  auto staged_off = [&](int c) __attribute__((always_inline)) -> uint32_t {
    return c >= 0 ? (uint32_t)(c * H + rcol) * 8u : kNoSource;
  };
  auto plain_off = [&](int c) __attribute__((always_inline)) -> uint32_t {
    return c <= -2 ? (uint32_t)((-2 - c) * H + rcol) * 4u : kNoSource;
  };
  auto issue_load = [&](uint32_t so, uint32_t po, auto k) __attribute__((always_inline)) {
    constexpr int PER = kLeafInputs ? 3 : 2, b = k / PER;
    if constexpr (k % PER == 0) flo[b] = hs.first2_at(so + 128u * b);
    if constexpr (k % PER == 1) fhi[b] = hs.first2_at(so + 128u * b + 16u);
    if constexpr (k % PER == 2) fp[b] = xin.load4(po + 64u * b);
  };
  auto block_ready = [&](int b) __attribute__((always_inline)) -> bool {
    return flo[b].y == tag && flo[b].w == tag && fhi[b].y == tag && fhi[b].w == tag;
  };
  auto block_value = [&](auto b) __attribute__((always_inline)) -> float4 {
    if constexpr (kLeafInputs) {
      return pick_block(cd >= 0, flo[b], fhi[b], fp[b]);
    } else {
      return make_float4(as_float(flo[b].x), as_float(flo[b].z), as_float(fhi[b].x), as_float(fhi[b].z));
    }
  };
  auto issue_x = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2 * XS; ++b)
      xv[b] = xin.load4(c <= -2 ? (uint32_t)(((-2 - c) * H + xcol + 16 * b) * 4) : kNoSource);
  };
  auto issue_cells = [&](const int *t, int e) __attribute__((always_inline)) {
    if (kLstm && eside == (e & 1)) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int c = code(t, erow, s);
        ce[s] = c >= 0 ? c * H + hbase + ej : -1;
        cc[s] = cs.load1_at(ce[s] >= 0 ? (uint32_t)ce[s] * 8u : kNoSource);
      }
    }
  };
  auto ready = [&](int e) __attribute__((always_inline)) -> bool {
    bool r = true;
#pragma unroll
    for (int b = 0; b < 2 * RS; ++b) r = r && block_ready(b);
    r = r || cd < 0;
    if (kLstm && eside == (e & 1)) {
#pragma unroll
      for (int s = 0; s < 2; ++s) r = r && (ce[s] < 0 || cc[s].y == tag);
    }
    return r;
  };

  // This wave's partial sums of tile t on the fp32 matrix unit: the same columns,
  // operands (all of them waited for) and weights from memory.
  auto fp32_tile = [&](const int *t, float *cb) __attribute__((always_inline)) {
    const int x0 = fresh_tid(), wave = x0 >> 6, i16 = x0 & 15, g4 = (x0 >> 4) & 3;
    const int rslot = wave >> 2, rcol = D::KR * (wave & 3) + 4 * g4, xcol = D::KX * wave + 4 * g4;
    const int xc = XS > 0 ? code(t, i16, 0) : -1, hc = code(t, i16, kDag ? 1 + rslot : rslot);
#pragma unroll 1
    for (int nt = 0; nt < NT; ++nt) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int b = 0; b < 2 * (XS + RS); ++b) {             // 16 columns at a time
        const bool in = b < 2 * XS;
        const int o = in ? xcol + 16 * b : rcol + 16 * (b - 2 * XS), c = in ? xc : hc;
        const uint32_t so = c >= 0 ? (uint32_t)(c * H + o) * 8u : kNoSource;
        const u32x4 plain = xin.load4(c <= -2 ? (uint32_t)((-2 - c) * H + o) * 4u : kNoSource);
        const float4 v = pick_block(c >= 0, hs.load2_at(so), hs.load2_at(so + 16u), plain);
        const int wc = kDag ? (in ? o : H + rslot * H + o) : rslot * H + o;
        acc = mfma_k16(v, weight_slice_at<CELL, H, J>(a, hbase, 16 * nt + i16, wc), acc);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) cb[(wave * kTileM + 4 * g4 + v) * LDC + 16 * nt + i16] = acc[v];
    }
  };

  for (int first = 0;; first += kCap) {
    if (first > 0) {
      if (first >= total) break;
      __syncthreads();                        // every wave is done with the last chunk's records
    }
    list_chunk(first);
    if (!kFused && first == 0) {
      if (kLstm && !bad && (size_t)(4 * N + 1) * sizeof(int) <= kStructCacheBudget) {
        // small batches: every row and input index is checked, also those that
        // no tile reads
#pragma unroll 1
        for (int r = blockIdx.x * kFwdThreads + tid; r < N; r += gridDim.x * kFwdThreads) {
          const int v = a.level_nodes[r], xi = a.x_index[r];
          bool ok = v >= 0 && v < N;
          for (int s = 0; s < K; ++s) {
            const int c = a.child_rows[(size_t)r * K + s];
            ok = ok && c >= -1 && (c < 0 || r >= off1);
          }
          if (!ok) raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
          if (xi < -1 || xi >= a.x_rows) raise_status(a.status, CORTEX_ST_INPUT_RANGE);
        }
      }
    }
    if (__syncthreads_or(bad)) {
      raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
      return;
    }
    if (first == 0) {
      CORTEX_TRACE_KERNEL(1);
      CORTEX_TRACE_KERNEL(2);
      if (!mark_entered(a.sync, tag, a.status)) return;
    }
    if (listed > 0) {
      cd = code(list, i16, kDag ? 1 + rslot : rslot);
      static_for<kLoads>([&](auto k) __attribute__((always_inline)) { issue_load(staged_off(cd), plain_off(cd), k); });
      if (XS > 0) issue_x(code(list, i16, 0));
      issue_cells(list, 0);
    }
    if constexpr (kLeafInputs) {
      // the leaf level: h = input row, c = 0 (its loads and stores overlap the
      // first tile's requests; no tile waits for these rows)
      if (first == 0 && a.level_lo == 0) write_leaf_outputs<H, kLstm>(a, nullptr, off1, hs, cs, tag);
    }
    // a tile's accumulators, and the largest operand met
    floatx4 hi[NT], lo[NT];
    float mx = kLeast;
    // 32 columns of step s: v0, v1 are this lane's four columns of its two blocks
    auto contract = [&](auto s, const float4 v0, const float4 v1, auto between) __attribute__((always_inline)) {
      if constexpr (kWeightsFromMemory) {
        Split8 wm[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const float4 w0 = wfrag(s, nt, 0, i16), w1 = wfrag(s, nt, 1, i16);
          wm[nt] = split8(w0, w1);
        }
        mfma_split<NT>(split8(v0, v1), wm, hi, lo, between);
      } else {
        if constexpr (s < W0) {
          Split8 wm[NT];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const u32x4 *o = &Wx_s[(s * NT + nt) * kFwdThreads + tid];
            wm[nt] = Split8{__builtin_bit_cast(bf16x8, o[0]), __builtin_bit_cast(bf16x8, o[WXP]),
                            __builtin_bit_cast(bf16x8, o[2 * WXP])};
          }
          mfma_split<NT>(split8(v0, v1), wm, hi, lo, between);
        } else {
          mfma_split<NT>(split8(v0, v1), w[s - W0], hi, lo, between);
        }
      }
    };
    for (int e = 0; e < listed; ++e) {
      const int *t = &list[e * INTS], *tn = &list[(e + 1 < listed ? e + 1 : e) * INTS];
      const bool more = e + 1 < listed;
      const int l = t[2];
      if (a.level_barrier) {
        for (; lvl < l; ++lvl)
          if (!grid_sync<false>(SyncWords{a.sync}, a.status, a.timeout)) return;
      }
      CORTEX_TRACE_POINT(l, 0);
      // the part that waits for nothing
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) hi[nt] = lo[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
      mx = kLeast;
      if constexpr (XS > 0) {
#pragma unroll
        for (int b = 0; b < 2 * XS; ++b) mx = max_abs(mx, as_float4(xv[b]));
        static_for<XS>([&](auto s) __attribute__((always_inline)) {
          contract(s, as_float4(xv[2 * s]), as_float4(xv[2 * s + 1]), [](auto) {});
        });
        issue_x(more ? code(tn, i16, 0) : -1);
      }
      float pv[PP];                            // hoisted: W x + b of this thread's outputs
      if constexpr (kHoisted) {
#pragma unroll
        for (int p = 0; p < PP; ++p) {
          const int row = t[0] + erow + D::RSTEP * p;
          pv[p] = as_float(pin.load1(row < t[1] ? (uint32_t)(row * H + hbase + ej) * 4u : kNoSource));
        }
      }
      CORTEX_TRACE_POINT(l, 1);
      if (!gave_up && !ready(e)) {
        const uint64_t t0 = wall_clock64();
        for (;;) {
          __builtin_amdgcn_s_sleep(1);
#pragma unroll
          for (int b = 0; b < 2 * RS; ++b)
            if (__any(cd >= 0 && !block_ready(b))) {       // (the whole wave: no masks to carry)
              flo[b] = hs.load2_at(staged_off(cd) + 128u * b);
              fhi[b] = hs.load2_at(staged_off(cd) + 128u * b + 16u);
            }
          if (kLstm && eside == (e & 1)) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
              if (ce[s] >= 0 && cc[s].y != tag) cc[s] = cs.load1_at((uint32_t)ce[s] * 8u);
          }
          const int stv = load_status(a.status);
          if (ready(e)) break;
          if (stv != 0) {
            gave_up = 1;
            break;
          }
          if (wall_clock64() - t0 > a.timeout) {
            raise_status(a.status, CORTEX_ST_BARRIER_TIMEOUT);
            gave_up = 1;
            break;
          }
        }
        if (gave_up) stop_s[e & 1] = 1;      // read by every wave after this tile's barrier
      }
      CORTEX_TRACE_POINT(l, 2);
      {
        const int ft = fresh_tid(), cdn = more ? code(tn, ft & 15, (kDag ? 1 : 0) + (ft >> 8)) : -1;     // (row i16, slot rslot)
        const uint32_t so = staged_off(cdn), po = plain_off(cdn);
        if (more) issue_cells(tn, e + 1);        // (for the other half's epilogue: not this tile's)
        // the next tile's operands are requested between a step's products, into the
        // registers whose values the step took
        static_for<RS>([&](auto s) __attribute__((always_inline)) {
          const float4 v0 = block_value(std::integral_constant<int, 2 * s>{}), v1 = block_value(std::integral_constant<int, 2 * s + 1>{});
          if constexpr (kLeafInputs) mx = max_abs(max_abs(mx, v0), v1);
          contract(std::integral_constant<int, XS + s>{}, v0, v1, [&](auto i) __attribute__((always_inline)) {
            // this step's loads, spread over its six products
            constexpr int PER = kLoads / RS, first = PER * s + PER * i / 6, last = PER * s + PER * (i + 1) / 6;
            static_for<last - first>([&](auto k) __attribute__((always_inline)) {
              issue_load(so, po, std::integral_constant<int, first + k>{});
            });
          });
        });
        cd = cdn;
        if (mx >= limit) list[e * INTS + 3] = -1;           // read after the tile's barrier
      }
      CORTEX_TRACE_WAVE(l);
      float *cb = &C_s[kOneBuffer ? 0 : (e & 1) * CBUF];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) cb[(wave * kTileM + 4 * g4 + v) * LDC + 16 * nt + i16] = hi[nt][v] + lo[nt][v];
      __syncthreads();
      CORTEX_TRACE_POINT(l, 3);
      const int stop = stop_s[e & 1], mark = t[3];
      if (stop) return;                      // a wave gave up its wait: every wave stops here
      if (__builtin_expect(mark < 0, 0)) {   // (the same for every wave)
        fp32_tile(t, cb);
        __syncthreads();
      }
      if (kOneBuffer || eside == (e & 1)) {
        // the eight partial sums in one order whatever J is, then the bias
        float z[PP][GATES];
#pragma unroll
        for (int p = 0; p < PP; ++p)
#pragma unroll
          for (int g = 0; g < GATES; ++g) {
            const float *c0 = &cb[(erow + D::RSTEP * p) * LDC + g * J + ej];
            float q[kFwdWaves];
#pragma unroll
            for (int k = 0; k < kFwdWaves / PARTS; ++k) q[k] = c0[(epart * (kFwdWaves / PARTS) + k) * kTileM * LDC];
#pragma unroll
            for (int n = kFwdWaves / PARTS; n > 1; n /= 2)
#pragma unroll
              for (int k = 0; k < n / 2; ++k) q[k] = q[2 * k] + q[2 * k + 1];
#pragma unroll
            for (int x = 1; x < PARTS; x *= 2) q[0] += __shfl_xor(q[0], J * x);
            z[p][g] = (kHoisted ? pv[p] : bias[g]) + q[0];
          }
        if constexpr (kOneBuffer) __syncthreads();     // the partial sums may be overwritten
        if constexpr (kLstm) {
          const int row = t[0] + erow;
          const float cn = sigmoidf(z[0][0]) * tanh_f(z[0][4]) + sigmoidf(z[0][1]) * as_float(cc[0].x) +
                           sigmoidf(z[0][2]) * as_float(cc[1].x);
          const float hv = sigmoidf(z[0][3]) * tanh_f(cn);
          if (epart == 0 && row < t[1]) {
            const uint32_t el = (uint32_t)(row * H + hbase + ej);
            cs.store1(el, cn, tag);
            hs.store1(el, hv, tag);
            a.c[el] = cn;
            a.h[el] = hv;
          }
        } else {
          float hv[PP];
#pragma unroll
          for (int p = 0; p < PP; ++p) hv[p] = tanh_f(z[p][0]);
          const int unit = hbase + (fresh_tid() & (J - 1));     // (hbase + ej: not an address kept, and spilled, through the loop)
          // the tagged pairs (what the next level waits for) first, then the outputs
#pragma unroll
          for (int p = 0; p < PP; ++p) {
            const int row = t[0] + erow + D::RSTEP * p;
            if (epart == 0 && row < t[1]) hs.store1((uint32_t)(row * H + unit), hv[p], tag);
          }
#pragma unroll
          for (int p = 0; p < PP; ++p) {
            const int row = t[0] + erow + D::RSTEP * p;
            if (epart == 0 && row < t[1]) *(float *)((char *)a.h + (uint32_t)(row * H + unit) * 4u) = hv[p];
          }
        }
      }
      CORTEX_TRACE_POINT(l, 4);
      CORTEX_TRACE_POINT(l, 5);
    }
  }
  if (a.level_barrier) {
    for (const int last = min(L, a.level_hi) - 1; lvl < last; ++lvl)
      if (!grid_sync<false>(SyncWords{a.sync}, a.status, a.timeout)) return;
  }
  CORTEX_TRACE_KERNEL(3);
  if (a.retire) retire_tag(a.sync, tag, a.status, a.timeout);
}

// ---------------------------------------------------------------------------
// Child-sum TreeLSTM at H = 256, batches beyond one launch (8 units per slice).
//
// Gate rows of a slice: (i, o | u, f) x 8, in two output tiles.  Wave w contracts
// 32 columns of the node input and of each of the four child slots, all slots of
// a row in one lane: the child sum h~ is then a sum of registers, and the first
// tile contracts h~ once instead of every child (seven products of 16 x 16 x 32
// per wave and tile; every slot with every gate would be ten).  The last tile
// contracts each slot: its f columns are U_f h_k, and its u columns sum over the
// slots to U_u h~.  An absent slot reads zeros.  The input weights' planes sit in
// LDS, the recurrent ones in registers beside the operands of two tiles.
//
// Leaves (more than half of the nodes) have no child: they run first, 64 rows
// per step, on their inputs alone.  The rest is as in slice_split_kernel.
//
// What bounds it: the operand loads, 16 per wave and tile through the address
// unit (0.85 us of a tile's 5), the two waves of a SIMD taking turns on the
// matrix unit and the vector ALU, and the epilogue of the waves on duty.  200
// trees (10,000 nodes) 496 -> 248 us per step against the fp32 kernel's 4-unit
// slices, which re-read every child row 64 times; 40 trees 132 -> 93.
// ---------------------------------------------------------------------------
struct ChildsumSplit {
  static constexpr int H = 256, J = 8, NT = J / 4, HT = NT - 1;               // gate tiles; those without f
  static constexpr int KW = H / 8, RS = KW / 32;                      // columns per wave of x and of each slot
  static constexpr int UB = 16 * HT, FB = UB + 16 - J;                // partial-sum columns: sums, then f_k
  static constexpr int COLS = FB + 4 * J, LDC = (COLS - 4 + 15) / 16 * 16 + 4;
  static constexpr int PARTS = 256 / (kTileM * J);
  static constexpr int CODES = 5, INTS = TileList<CODES>::kInts, HEAD = TileList<CODES>::kHead;
  static constexpr int LEAF = 64, LDL = 28;             // rows per leaf step, their partial-sum stride
  static constexpr int CBUF = kFwdWaves * kTileM * LDC;
  // the split input weights, in LDS: [step][tile][plane][wave][lane] x 16 bytes
  static constexpr int kWx = RS * NT * 3 * kFwdThreads;
  static constexpr int kCap = 64;
  static constexpr NarrowRule kNarrowRule = {40, 40}, kNarrowCachedRule = {40, 72};
  static_assert(J % 4 == 0 && J <= 8 && KW % 32 == 0 && kFwdWaves * LEAF * LDL <= 2 * CBUF, "tiling");
};

// kNarrowCached: the form for deep, narrow batches keeps the linearization in LDS.
template <bool kNarrowCached>
__global__ void __launch_bounds__(kFwdThreads) childsum_split_kernel(FwdArgs a) {
  using D = ChildsumSplit;
  constexpr int CELL = CORTEX_CHILDSUM_TREELSTM, H = D::H, J = D::J;
  constexpr int NT = D::NT, HT = D::HT, RS = D::RS, LDC = D::LDC, PARTS = D::PARTS, INTS = D::INTS, HEAD = D::HEAD;
  constexpr int CODES = D::CODES, CBUF = D::CBUF, LEAF = D::LEAF, LDL = D::LDL;
  constexpr int kCap = D::kCap;

  __shared__ __attribute__((aligned(16))) float C_s[2 * CBUF];
  __shared__ u32x4 Wx_s[D::kWx];
  __shared__ int wsum[kFwdWaves + 1];
  __shared__ int stop_s[2], big_s[2];
  __shared__ float bias_s[4 * J];
  extern __shared__ int dyn[];
  int *list = dyn;                              // [kCap][INTS]; the leaf rows' inputs before that

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g4 = lane >> 4;
  const int Q = a.Q, slice = blockIdx.x / Q, group = blockIdx.x % Q;
  const int hbase = slice * J, N = a.N, K = a.K;
  const uint32_t tag = launch_tag(a.sync);      // read with the status: one round trip
  const TagBuf hs(a.hs, (uint32_t)N * H * 8);
  const TagBuf cs(a.cs, (uint32_t)N * H * 8);
  const InBuf xin(a.x_table, a.x_table ? (uint32_t)a.x_rows * H * 4 : 0u);
  const int col = D::KW * wave + 4 * g4;        // this lane's first column of x and of every child
  const int et = tid & 255, eside = tid >> 8;
  const int ej = et % J, epart = (et & 15) / J, erow = 4 * ((et >> 4) & 3) + (et >> 6);

  CORTEX_TRACE_KERNEL(0);
  const int status0 = load_status(a.status);
  const int L = *a.num_levels, off1 = a.level_offsets[1], off2 = a.level_offsets[N > 1 ? 2 : 1];   // (before the weights, as in slice_split_kernel)
  if (tid < 2) stop_s[tid] = big_s[tid] = 0;

  auto wfrag = [&](int sg, int s, int nt, int half) __attribute__((always_inline)) -> float4 {
    return weight_slice_at<CELL, H, J>(a, hbase, 16 * nt + i16, sg * H + col + 32 * s + 16 * half);
  };
  float4 wv[2][RS][NT][2];
#pragma unroll
  for (int sg = 0; sg < 2; ++sg)
#pragma unroll
    for (int s = 0; s < RS; ++s)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) wv[sg][s][nt][hf] = wfrag(sg, s, nt, hf);
  if (tid < 4 * J) bias_s[tid] = a.b[childsum_gate(tid / J) * H + hbase + tid % J];     // i, o, u, f

  int bad = 0;
  if (status0 != 0) return;
  if (L < 1 || L > N || off1 < 1 || off1 > N) {
    raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
    return;
  }
  if (a.narrow_q > 0 && narrow_levels(off1, off2, N, L, kNarrowCached ? D::kNarrowCachedRule : D::kNarrowRule)) {
    ChildsumLds<H> &n = *(ChildsumLds<H> *)C_s;
    static_assert(sizeof(ChildsumLds<H>) <= sizeof(C_s), "the fp32 form's arrays take the place of the partial sums");
    const FwdArgs b = fresh_args();
    childsum_forward<H, kNarrowCached>(b, b.narrow_q, n.W_s, n.Cx, n.Ce, n.Z_s, n.bias_s, n.chunk, dyn);
    return;
  }
  Split8 wu[RS][NT];
  float wmax = 0.f;
#pragma unroll
  for (int s = 0; s < RS; ++s)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int sg = 0; sg < 2; ++sg) wmax = max_abs(max_abs(wmax, wv[sg][s][nt][0]), wv[sg][s][nt][1]);
      // (each lane reads back only what it wrote: no barrier)
      const Split8 x = split8(wv[0][s][nt][0], wv[0][s][nt][1]);
      u32x4 *o = &Wx_s[(s * NT + nt) * 3 * kFwdThreads + tid];
      o[0] = __builtin_bit_cast(u32x4, x.p0);
      o[kFwdThreads] = __builtin_bit_cast(u32x4, x.p1);
      o[2 * kFwdThreads] = __builtin_bit_cast(u32x4, x.p2);
      wu[s][nt] = split8(wv[1][s][nt][0], wv[1][s][nt][1]);
    }

  const float limit = split_limit(wmax, 5 * D::KW);     // (u: x and the four slots meet in one sum)

  auto wx = [&](int s, Split8 (&w)[NT]) __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const u32x4 *o = &Wx_s[(s * NT + nt) * 3 * kFwdThreads + tid];
      w[nt] = Split8{__builtin_bit_cast(bf16x8, o[0]), __builtin_bit_cast(bf16x8, o[kFwdThreads]),
                     __builtin_bit_cast(bf16x8, o[2 * kFwdThreads])};
    }
  };
  // The input row of row r, -1 = none (validated).
  auto input_row = [&](int r) __attribute__((always_inline)) -> int {
    const int v = a.level_nodes[r];
    if (v < 0 || v >= N) {
      bad = 1;
      return -1;
    }
    const int xi = a.x_index[v];
    if (xi < -1 || xi >= a.x_rows) {
      raise_status(a.status, CORTEX_ST_INPUT_RANGE);
      return -1;
    }
    return xi;
  };
  // 16 columns from column c (this lane's four of them) of gate tile nt on the
  // fp32 matrix unit: segment 0 is W, with input rows, 1 is U, with staged rows.
  auto fp32_block = [&](int sg, int c, int row, const float4 v, floatx4 acc) __attribute__((always_inline)) -> floatx4 {
    return mfma_k16(v, weight_slice_at<CELL, H, J>(a, hbase, row, sg * H + c), acc);
  };
  auto fp32_input = [&](int xr, int c) __attribute__((always_inline)) -> float4 {
    return as_float4(xin.load4(xr >= 0 ? (uint32_t)(xr * H + c) * 4u : kNoSource));
  };
  // Tree sum of this thread's part of the eight partial sums at c0 (stride:
  // floats between waves), then over the parts of the pair: one order whatever J.
  auto sum_parts = [&](const float *c0, int stride) __attribute__((always_inline)) -> float {
    float q[kFwdWaves];
#pragma unroll
    for (int k = 0; k < kFwdWaves / PARTS; ++k) q[k] = c0[(epart * (kFwdWaves / PARTS) + k) * stride];
#pragma unroll
    for (int n = kFwdWaves / PARTS; n > 1; n /= 2)
#pragma unroll
      for (int k = 0; k < n / 2; ++k) q[k] = q[2 * k] + q[2 * k + 1];
#pragma unroll
    for (int x = 1; x < PARTS; x *= 2) q[0] += __shfl_xor(q[0], J * x);
    return q[0];
  };

  if (!mark_entered(a.sync, tag, a.status)) return;
  CORTEX_TRACE_KERNEL(1);
  CORTEX_TRACE_KERNEL(2);

  // ---- level 0: c = i*u, h = o*tanh(c) on the inputs alone; step n of the
  // group takes the rows [64 (group + n Q), + 64)
  if (a.level_lo == 0) {
    constexpr int MT = LEAF / kTileM;
    const int nsteps = (off1 + LEAF - 1) / LEAF, mine = group < nsteps ? (nsteps - 1 - group) / Q + 1 : 0;
    constexpr int kChunk = kCap * INTS / LEAF;          // steps whose input rows the list holds
#pragma unroll 1
    for (int first = 0; first < mine; first += kChunk) {
      const int cnt = min(mine - first, kChunk);
      if (first > 0) __syncthreads();
#pragma unroll 1
      for (int idx = tid; idx < cnt * LEAF; idx += kFwdThreads) {
        const int row = LEAF * (group + (first + idx / LEAF) * Q) + idx % LEAF;
        list[idx] = row < off1 ? input_row(row) : -1;
      }
      if (__syncthreads_or(bad)) {
        raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
        return;
      }
      u32x4 xl[MT][2 * RS];
      auto issue_leaf = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          const int xr = n < cnt ? list[n * LEAF + t * kTileM + i16] : -1;
          const uint32_t o = xr >= 0 ? (uint32_t)(xr * H + col) * 4u : kNoSource;
#pragma unroll
          for (int b = 0; b < 2 * RS; ++b) xl[t][b] = xin.load4(o + 64u * b);
        }
      };
      // this wave's partial sums of leaf tile t
      auto leaf_sums = [&](int t, const floatx4 (&z)[NT]) __attribute__((always_inline)) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          if (16 * nt + i16 < 3 * J)
#pragma unroll
            for (int v = 0; v < 4; ++v) C_s[(wave * LEAF + t * kTileM + 4 * g4 + v) * LDL + 16 * nt + i16] = z[nt][v];
      };
      issue_leaf(0);
#pragma unroll 1
      for (int n = 0; n < cnt; ++n) {
        const int rowbase = LEAF * (group + (first + n) * Q);
        float mx = 0.f;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          floatx4 hi[NT], lo[NT];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) hi[nt] = lo[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
          static_for<RS>([&](auto s) __attribute__((always_inline)) {
            const float4 v0 = as_float4(xl[t][2 * s]), v1 = as_float4(xl[t][2 * s + 1]);
            mx = max_abs(max_abs(mx, v0), v1);
            Split8 w[NT];
            wx(s, w);
            mfma_split<NT>(split8(v0, v1), w, hi, lo, [](auto) {});
          });
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) hi[nt] += lo[nt];
          leaf_sums(t, hi);
        }
        issue_leaf(n + 1);
        if (mx >= limit) big_s[n & 1] = 1;
        __syncthreads();
        if (__builtin_expect(big_s[n & 1] != 0, 0)) {
          // (every wave) its partial sums again from the fp32 values
          const int x0 = fresh_tid(), r16 = x0 & 15, c0 = D::KW * (x0 >> 6) + 4 * ((x0 >> 4) & 3);
#pragma unroll 1
          for (int t = 0; t < MT; ++t) {
            const int xr = list[n * LEAF + t * kTileM + r16];
            floatx4 acc[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int b = 0; b < 2 * RS; ++b) {
              const float4 v = fp32_input(xr, c0 + 16 * b);
#pragma unroll
              for (int nt = 0; nt < NT; ++nt) acc[nt] = fp32_block(0, c0 + 16 * b, 16 * nt + r16, v, acc[nt]);
            }
            leaf_sums(t, acc);
          }
          __syncthreads();
        }
        if (tid < LEAF * J) {
          const int j = tid % J, i = tid / J, row = rowbase + i;
          float z[3];
#pragma unroll
          for (int g = 0; g < 3; ++g) {
            const float *c0 = &C_s[i * LDL + g * J + j];
            float q[kFwdWaves];
#pragma unroll
            for (int k = 0; k < kFwdWaves; ++k) q[k] = c0[k * LEAF * LDL];
#pragma unroll
            for (int w = kFwdWaves; w > 1; w /= 2)
#pragma unroll
              for (int k = 0; k < w / 2; ++k) q[k] = q[2 * k] + q[2 * k + 1];
            z[g] = bias_s[g * J + j] + q[0];
          }
          if (row < off1) {
            const float cn = sigmoidf(z[0]) * tanh_f(z[2]), hv = sigmoidf(z[1]) * tanh_f(cn);
            const uint32_t el = (uint32_t)(row * H + hbase + j);
            cs.store1(el, cn, tag);
            hs.store1(el, hv, tag);
            a.c[el] = cn;
            a.h[el] = hv;
          }
        }
        if (tid == 0) big_s[(n + 1) & 1] = 0;
        __syncthreads();                     // the partial sums may be overwritten
      }
    }
    if (L > 1 && a.level_hi > 1 && a.level_barrier && !grid_sync<false>(SyncWords{a.sync}, a.status, a.timeout)) return;
  }

  int gave_up = 0, lvl = max(a.level_lo, 1);
  u32x4 flo[4][2], fhi[4][2];         // child slot k, block b of a 32-column step
  u32x4 xv[2 * RS];
  int cd[4];                          // this lane's row: child rows, -1 = none
  u32x2 cc[4];                        // the children's memory cells of this thread's next epilogue
  unsigned int cmask = 0u;            // which of them exist

  auto code = [&](const int *t, int i, int k) __attribute__((always_inline)) -> int {
    return t[0] + i < t[1] ? t[HEAD + i * CODES + k] : -1;
  };
  auto child_off = [&](int c) __attribute__((always_inline)) -> uint32_t {
    return c >= 0 ? (uint32_t)(c * H + col) * 8u : kNoSource;
  };
  auto issue_slot = [&](uint32_t so, auto k, auto q) __attribute__((always_inline)) {     // load q (0..3) of slot k
    if constexpr (q % 2 == 0) flo[k][q / 2] = hs.first2_at(so + 128u * (q / 2));
    else fhi[k][q / 2] = hs.first2_at(so + 128u * (q / 2) + 16u);
  };
  auto issue_x = [&](int c) __attribute__((always_inline)) {
    const uint32_t o = c >= 0 ? (uint32_t)(c * H + col) * 4u : kNoSource;
#pragma unroll
    for (int b = 0; b < 2 * RS; ++b) xv[b] = xin.load4(o + 64u * b);
  };
  auto issue_cells = [&](const int *t, int e) __attribute__((always_inline)) {
    if (eside == (e & 1)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = code(t, erow, k);
        cmask = k == 0 ? (c >= 0) : cmask | (unsigned int)(c >= 0) << k;
        cc[k] = cs.load1_at(c >= 0 ? (uint32_t)(c * H + hbase + ej) * 8u : kNoSource);
      }
    }
  };

  // This wave's partial sums of a tile: z of x and h~ (the last gate tile of x
  // alone), f of each slot with the last gate tile.
  auto tile_sums = [&](float *cb, const floatx4 (&z)[NT], const floatx4 (&f)[4][1]) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float *c0 = &cb[(wave * kTileM + 4 * g4 + v) * LDC];
#pragma unroll
      for (int nt = 0; nt < HT; ++nt) c0[16 * nt + i16] = z[nt][v];
      const float x = z[NT - 1][v];
      if (i16 < 16 - J) {
        c0[D::UB + i16] = x + ((f[0][0][v] + f[1][0][v]) + (f[2][0][v] + f[3][0][v]));
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) c0[D::FB + k * J + i16 - (16 - J)] = x + f[k][0][v];
      }
    }
  };

  int total = 0, listed = 0;
#pragma unroll 1
  for (int first = 0;; first += kCap) {
    if (first > 0 && first >= total) break;
    __syncthreads();                          // every wave is done with the records (or the leaf inputs)
    {
      const int t0 = fresh_tid();
      total = list_tiles<INTS>([&](int l) { return a.level_offsets[l]; }, L, N, max(a.level_lo, 1), a.level_hi, group, Q, first,
                               kCap, t0, list, wsum, bad);
      listed = min(total - first, kCap);
      if (__syncthreads_or(bad)) {
        raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
        return;
      }
#pragma unroll 1
      for (int idx = t0; idx < listed * kTileM; idx += kFwdThreads) {
        int *t = &list[(idx / kTileM) * INTS], *o = t + HEAD + (idx % kTileM) * CODES;
        const int row = t[0] + idx % kTileM;
        const bool live = row < t[1];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          int c = -1;
          if (live && s < K) {
            c = a.child_rows[(size_t)row * K + s];
            if (c < -1 || c >= t[3]) {        // a child must sit in a lower level
              bad = 1;
              c = -1;
            }
          }
          o[s] = c;
        }
        o[4] = live ? input_row(row) : -1;
      }
      if (first == 0 && ((size_t)N * (K + 2) + 1) * sizeof(int) <= kStructCacheBudget) {
        // small batches: a leaf with children is refused
#pragma unroll 1
        for (int r = blockIdx.x * kFwdThreads + t0; r < off1; r += gridDim.x * kFwdThreads)
          for (int s = 0; s < K; ++s)
            if (a.child_rows[(size_t)r * K + s] != -1) raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
      }
    }
    if (__syncthreads_or(bad)) {
      raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
      return;
    }
    if (listed > 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) cd[k] = code(list, i16, k);
      static_for<4>([&](auto k) __attribute__((always_inline)) {
        static_for<4>([&](auto q) __attribute__((always_inline)) { issue_slot(child_off(cd[k]), k, q); });
      });
      issue_x(code(list, i16, 4));
      issue_cells(list, 0);
    }
#pragma unroll 1
    for (int e = 0; e < listed; ++e) {
      const int *t = &list[e * INTS], *tn = &list[(e + 1 < listed ? e + 1 : e) * INTS];
      const bool more = e + 1 < listed;
      const int l = t[2];
      if (a.level_barrier) {
        for (; lvl < l; ++lvl)
          if (!grid_sync<false>(SyncWords{a.sync}, a.status, a.timeout)) return;
      }
      CORTEX_TRACE_POINT(l, 0);
      float mx = 0.f;
      // the input part waits for nothing
      floatx4 hi[NT], lo[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) hi[nt] = lo[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
      static_for<RS>([&](auto s) __attribute__((always_inline)) {
        const float4 v0 = as_float4(xv[2 * s]), v1 = as_float4(xv[2 * s + 1]);
        mx = max_abs(max_abs(mx, v0), v1);
        Split8 w[NT];
        wx(s, w);
        mfma_split<NT>(split8(v0, v1), w, hi, lo, [](auto) {});
      });
      issue_x(more ? code(tn, i16, 4) : -1);
      CORTEX_TRACE_POINT(l, 1);
      floatx4 fh[4][1], fl[4][1];         // (the last step leaves the sum in fh)
#pragma unroll
      for (int k = 0; k < 4; ++k) fh[k][0] = fl[k][0] = floatx4{0.f, 0.f, 0.f, 0.f};
      int cdn[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) cdn[k] = more ? code(tn, i16, k) : -1;
      static_for<RS>([&](auto s) __attribute__((always_inline)) {
        // wait for step s of every child slot (and, before the first, the cells)
        auto slot_ready = [&](int k) __attribute__((always_inline)) -> bool {
          return cd[k] < 0 || (flo[k][0].y == tag && flo[k][0].w == tag && fhi[k][0].y == tag && fhi[k][0].w == tag &&
                               flo[k][1].y == tag && flo[k][1].w == tag && fhi[k][1].y == tag && fhi[k][1].w == tag);
        };
        auto ready = [&]() __attribute__((always_inline)) -> bool {
          bool r = true;
#pragma unroll
          for (int k = 0; k < 4; ++k) r = r && slot_ready(k);
          if (s == RS - 1 && eside == (e & 1)) {
#pragma unroll
            for (int k = 0; k < 4; ++k) r = r && (!((cmask >> k) & 1u) || cc[k].y == tag);
          }
          return r;
        };
        if (!gave_up && !ready()) {
          const uint64_t t0 = wall_clock64();
          for (;;) {
            __builtin_amdgcn_s_sleep(1);
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (__any(!slot_ready(k))) {       // (the whole wave: no masks to carry)
                const uint32_t so = child_off(cd[k]) + 256u * s;
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                  flo[k][b] = hs.load2_at(so + 128u * b);
                  fhi[k][b] = hs.load2_at(so + 128u * b + 16u);
                }
              }
            if (s == RS - 1 && eside == (e & 1)) {
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (((cmask >> k) & 1u) && cc[k].y != tag)
                  cc[k] = cs.load1_at((uint32_t)(code(t, erow, k) * H + hbase + ej) * 8u);
            }
            const int stv = load_status(a.status);
            if (ready()) break;
            if (stv != 0) {
              gave_up = 1;
              break;
            }
            if (wall_clock64() - t0 > a.timeout) {
              raise_status(a.status, CORTEX_ST_BARRIER_TIMEOUT);
              gave_up = 1;
              break;
            }
          }
          if (gave_up) stop_s[e & 1] = 1;    // read by every wave after this tile's barrier
        }
        CORTEX_TRACE_POINT(l, 2);
        float4 h0 = make_float4(0.f, 0.f, 0.f, 0.f), h1 = h0;     // h~ of this lane's columns
        static_for<4>([&](auto k) __attribute__((always_inline)) {
          const float4 v0 = make_float4(as_float(flo[k][0].x), as_float(flo[k][0].z), as_float(fhi[k][0].x), as_float(fhi[k][0].z));
          const float4 v1 = make_float4(as_float(flo[k][1].x), as_float(flo[k][1].z), as_float(fhi[k][1].x), as_float(fhi[k][1].z));
          // (an absent slot's loads read zeros)
          mx = max_abs(max_abs(mx, v0), v1);
          h0 = make_float4(h0.x + v0.x, h0.y + v0.y, h0.z + v0.z, h0.w + v0.w);
          h1 = make_float4(h1.x + v1.x, h1.y + v1.y, h1.z + v1.z, h1.w + v1.w);
          // the slot's next operands: the tile's next 32 columns, or the next tile's first
          const uint32_t so = s + 1 < RS ? child_off(cd[k]) + 256u * (s + 1) : child_off(cdn[k]);
          Split8 wl[1] = {wu[s][NT - 1]};
          mfma_split<1>(split8(v0, v1), wl, fh[k], fl[k], [&](auto i) __attribute__((always_inline)) {
            if constexpr (i < 4) issue_slot(so, k, i);
          });
          if constexpr (s == RS - 1) fh[k][0] += fl[k][0];
        });
        mx = max_abs(max_abs(mx, h0), h1);
        mfma_split<HT>(split8(h0, h1), reinterpret_cast<const Split8(&)[HT]>(wu[s]), reinterpret_cast<floatx4(&)[HT]>(hi),
                       reinterpret_cast<floatx4(&)[HT]>(lo), [](auto) {});
      });
      if (mx >= limit) list[e * INTS + 3] = -1;           // read after the tile's barrier
      CORTEX_TRACE_WAVE(l);
      float *cb = &C_s[(e & 1) * CBUF];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) hi[nt] += lo[nt];
      tile_sums(cb, hi, fh);
      // (the cells of the next tile go to the other half of the waves)
      if (more) issue_cells(tn, e + 1);
#pragma unroll
      for (int k = 0; k < 4; ++k) cd[k] = cdn[k];
      __syncthreads();
      CORTEX_TRACE_POINT(l, 3);
      const int stop = stop_s[e & 1], mark = t[3];
      if (stop) return;                      // a wave gave up its wait: every wave stops here
      if (__builtin_expect(mark < 0, 0)) {
        // (every wave) its partial sums again from the fp32 values, all waited for
        floatx4 z[NT], f[4][1];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) z[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k][0] = floatx4{0.f, 0.f, 0.f, 0.f};
        const int x0 = fresh_tid(), r16 = x0 & 15, c0 = D::KW * (x0 >> 6) + 4 * ((x0 >> 4) & 3);
#pragma unroll 1
        for (int c = c0; c < c0 + D::KW; c += 16) {
          const float4 x = fp32_input(code(t, r16, 4), c);
          float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) z[nt] = fp32_block(0, c, 16 * nt + r16, x, z[nt]);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int ch = code(t, r16, k);
            const uint32_t so = ch >= 0 ? (uint32_t)(ch * H + c) * 8u : kNoSource;
            const u32x4 lo = hs.load2_at(so), up = hs.load2_at(so + 16u);
            const float4 v = make_float4(as_float(lo.x), as_float(lo.z), as_float(up.x), as_float(up.z));
            h = make_float4(h.x + v.x, h.y + v.y, h.z + v.z, h.w + v.w);
            f[k][0] = fp32_block(1, c, 16 * (NT - 1) + r16, v, f[k][0]);
          }
#pragma unroll
          for (int nt = 0; nt < HT; ++nt) z[nt] = fp32_block(1, c, 16 * nt + r16, h, z[nt]);
        }
        tile_sums(cb, z, f);
        __syncthreads();
      }
      if (eside == (e & 1)) {
        const float *c0 = &cb[erow * LDC + ej];
        constexpr int WST = kTileM * LDC;
        float z[3], f[4];
#pragma unroll
        for (int g = 0; g < 3; ++g) z[g] = bias_s[g * J + ej] + sum_parts(c0 + g * J, WST);
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = bias_s[3 * J + ej] + sum_parts(c0 + D::FB + k * J, WST);
        float fc[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) fc[k] = (cmask >> k) & 1u ? sigmoidf(f[k]) * as_float(cc[k].x) : 0.f;
        const float cn = sigmoidf(z[0]) * tanh_f(z[2]) + ((fc[0] + fc[1]) + (fc[2] + fc[3]));
        const float hv = sigmoidf(z[1]) * tanh_f(cn);
        const int row = t[0] + erow;
        if (epart == 0 && row < t[1]) {
          const uint32_t el = (uint32_t)(row * H + hbase + ej);
          cs.store1(el, cn, tag);
          hs.store1(el, hv, tag);
          a.c[el] = cn;
          a.h[el] = hv;
        }
      }
      CORTEX_TRACE_POINT(l, 4);
      CORTEX_TRACE_POINT(l, 5);
    }
  }
  if (a.level_barrier) {
    for (const int last = min(L, a.level_hi) - 1; lvl < last; ++lvl)
      if (!grid_sync<false>(SyncWords{a.sync}, a.status, a.timeout)) return;
  }
  CORTEX_TRACE_KERNEL(3);
  if (a.retire) retire_tag(a.sync, tag, a.status, a.timeout);
}

// ---------------------------------------------------------------------------
// MV-RNN at d = 128: p = tanh(W [B a; A b]), P = W_M [A; B].
//
// Node-parallel by COLUMNS of P: workgroup (cb, group) computes the 16 columns
// [16 cb, + 16) of P for the nodes of its group (a level's nodes are dealt among
// the groups; a group's eight workgroups sit on one XCD), so it reads just
// those columns of A and B, an eighth of them, and every element of [A; B] is
// loaded once per node.  (By rows of P, each of the eight workgroups needs all of
// [A; B]: 256 KB of tagged pairs per node and workgroup, restaged through LDS.)
// Wave w holds W_M[:, 32 w .. 32 w + 31] in registers, split; it loads its 32
// rows x 16 columns of [A; B] straight into the MFMA operand layout, and the
// eight partial sums meet in LDS.
//
// B a and A b need whole rows of B and A: each workgroup forms the partial sums
// over its 16 columns from the operands it holds and publishes them (2 d values per
// node) in the workspace; once all eight are there, each workgroup adds them
// up and computes its 16 rows of p.  Within a level that second half runs one
// node late, so the exchange is not waited for.
//
// Leaf rows of the outputs are copied last, by workgroups with no node left to
// compute while the narrow top levels finish.
//
// kFused: every workgroup linearizes the batch in LDS itself (cortex_tree_infer
// up to kFusedRows nodes; one tree of two leaves 19.9 -> 16.8 us, ten 39.5 -> 36.0).
//
// 40 trees (1,960 nodes): 424 -> 260 us per step; ten trees 161 -> 104.
// ---------------------------------------------------------------------------
struct MvCols {
  static constexpr int D = 128, RB = D / 16, MT = D / 16;
  static constexpr int LDN = D + 4;                      // column stride of the partial sums
  static constexpr int INTS = 6;                         // node record: row, level end, level, level start / -1, two codes
  static constexpr int kCap = 512, kFusedCap = 32;       // records held at a time
  static constexpr int kFusedRows = 47;                  // one launch, and every node's input index checked, up to here
  static constexpr int kCheckRows = 640;                 // every entry of child_rows checked up to here
  static constexpr size_t kXchg = (size_t)RB * 2 * D;    // published partial sums per node
};

template <bool kFused>
__global__ void __launch_bounds__(kFwdThreads) mvrnn_cols_kernel(FwdArgs a) {
  using M = MvCols;
  constexpr int D = M::D, RB = M::RB, MT = M::MT, LDN = M::LDN, INTS = M::INTS, kCap = kFused ? M::kFusedCap : M::kCap;
  constexpr int CBUF = kFwdWaves * 16 * LDN;

  __shared__ __attribute__((aligned(16))) float C_s[2 * CBUF];
  __shared__ float bab_s[2][2][2 * D];          // [parity][half of the column blocks][B a; A b]
  __shared__ int list[kCap * INTS];
  __shared__ int wsum[kFwdWaves + 1];
  __shared__ int stop_s[2];
  __shared__ float limit_s[kFwdWaves];
  extern __shared__ int dyn[];                  // fused: the input row by node id, then the linearizer's arrays

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g4 = lane >> 4;
  const int ngroups = gridDim.x / RB, cb = blockIdx.x / ngroups, group = blockIdx.x % ngroups;
  const int N = a.N;
  const uint32_t tag = launch_tag(a.sync);      // read with the status: one round trip
  const TagBuf hs(a.hs, (uint32_t)N * D * 8);
  const TagBuf ps(a.cs, (uint32_t)N * D * D * 8);
  const TagBuf xs(a.keep, (uint32_t)N * (uint32_t)M::kXchg * 8u);
  const InBuf xv(a.x_table, a.x_table ? (uint32_t)a.x_rows * D * 4 : 0u);
  const InBuf xm(a.leaf_mat, a.leaf_mat ? (uint32_t)a.x_rows * D * D * 4 : 0u);
  const int side = wave >> 2, kk = 32 * (wave & 3) + 8 * g4;       // matrix (0: A, 1: B) and this lane's first row of it
  const int col = 16 * cb + i16;                                   // this lane's column of A, B and P
  const int status0 = load_status(a.status);
  int L = kFused ? 0 : *a.num_levels;
  SmallLin lin;
  if (tid < 2) stop_s[tid] = 0;
  Split8 wm[MT];
  float wmax = 0.f;
  {
    float4 v[MT][2];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        v[m][h] = *(const float4 *)&a.W_M[(size_t)(16 * m + i16) * 2 * D + 32 * wave + 8 * g4 + 4 * h];
    if constexpr (kFused) {
      // (the weight loads share the round trip of the linearizer's)
      static_assert(M::kFusedRows <= kFwdThreads, "a thread per node");
      int xi = tid < N ? a.x_index[tid] : -1;
      L = small_linearize<kFwdThreads, 1>(a.children, N, 2, a.status, dyn + N, lin, fused_lin_stamps(a));
      if (L == 0) return;
      if (blockIdx.x == 0)
        small_lin_emit<kFwdThreads>(lin, N, 2, L, a.o_num_levels, a.o_height, a.o_level_offsets, a.o_level_nodes, a.o_node_row,
                                    a.o_child_rows);
      if (xi < -1 || xi >= a.x_rows) {
        raise_status(a.status, CORTEX_ST_INPUT_RANGE);
        xi = -1;
      }
      if (tid < N) dyn[tid] = xi;
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      wmax = max_abs(max_abs(wmax, v[m][0]), v[m][1]);
      wm[m] = split8(v[m][0], v[m][1]);
    }
  }
  {
    const float limit = split_limit(wmax, 32);
    if (lane == 0) limit_s[wave] = limit;       // (in LDS: registers are short; a wave reads its own)
  }
  if (status0 != 0) return;
  if (L < 1 || L > N) {
    raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
    return;
  }
  if (!mark_entered(a.sync, tag, a.status)) return;

  int bad = 0, gave_up = 0;
  auto offset = [&](int l) __attribute__((always_inline)) -> int {
    if constexpr (kFused) return l < L ? lin.lcount[l] : N;
    else return a.level_offsets[l];
  };
  auto child_row = [&](int r, int s) __attribute__((always_inline)) -> int {
    if constexpr (kFused) {
      const int c = lin.ch[lin.order[r] * 2 + s];
      return c < 0 ? -1 : lin.nrow[c];
    } else {
      return a.child_rows[(size_t)r * 2 + s];
    }
  };
  // input row of leaf row r, -1 = none (validated)
  auto leaf_input = [&](int r) __attribute__((always_inline)) -> int {
    if constexpr (kFused) return dyn[lin.order[r]];
    const int v = a.level_nodes[r];
    if (v < 0 || v >= N) {
      raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
      return -1;
    }
    const int xi = a.x_index[v];
    if (xi < -1 || xi >= a.x_rows) {
      raise_status(a.status, CORTEX_ST_INPUT_RANGE);
      return -1;
    }
    return xi;
  };

  // a wave's operands: its 8 matrix elements per lane and one vector element
  // (a for the rows of B, b for the rows of A), staged (value, tag) or plain
  u32x2 f[8], fv;
  int cm = -1, cv = -1;                         // source codes of the matrix and of the vector (one per wave)
  auto issue = [&](const int *t) __attribute__((always_inline)) {
    cm = __builtin_amdgcn_readfirstlane(t[4 + side]);
    cv = __builtin_amdgcn_readfirstlane(t[4 + (side ^ 1)]);
    if (cm >= 0) {
#pragma unroll
      for (int j = 0; j < 8; ++j) f[j] = ps.first1_at((uint32_t)((cm * D + kk + j) * D + col) * 8u);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        f[j] = u32x2{xm.load1(cm <= -2 ? (uint32_t)(((-2 - cm) * D + kk + j) * D + col) * 4u : kNoSource), 0u};
    }
    if (cv >= 0) fv = hs.load1_at((uint32_t)(cv * D + col) * 8u);
    else fv = u32x2{xv.load1(cv <= -2 ? (uint32_t)((-2 - cv) * D + col) * 4u : kNoSource), 0u};
  };
  auto ready = [&]() __attribute__((always_inline)) -> bool {
    bool r = cv < 0 || fv.y == tag;
    if (cm >= 0) {
#pragma unroll
      for (int j = 0; j < 8; ++j) r = r && f[j].y == tag;
    }
    return r;
  };
  // bounded waits: poll() requests again what is missing
  auto wait_for = [&](auto is_ready, auto poll, int phase) __attribute__((always_inline)) {
    if (gave_up || is_ready()) return;
    const uint64_t t0 = wall_clock64();
    for (;;) {
      __builtin_amdgcn_s_sleep(1);
      poll();
      const int stv = load_status(a.status);
      if (is_ready()) break;
      if (stv != 0) {
        gave_up = 1;
        break;
      }
      if (wall_clock64() - t0 > a.timeout) {
        raise_status(a.status, CORTEX_ST_BARRIER_TIMEOUT);
        gave_up = 1;
        break;
      }
    }
    if (gave_up) stop_s[phase & 1] = 1;         // read by every wave after the barrier that closes the phase
  };
  // the published partial sums of a node: entry tid mod 2d of four column blocks
  u32x2 g[4];
  auto issue_gather = [&](int row) __attribute__((always_inline)) {
    const int x = fresh_tid();
    const uint32_t o = (uint32_t)((row * RB + 4 * (x >> 8)) * 2 * D + (x & (2 * D - 1))) * 8u;
#pragma unroll
    for (int c = 0; c < 4; ++c) g[c] = xs.load1_at(o + 16u * D * c);
  };
  int phase = 0;                                // barriers passed in the node loop
  // the second half of a node: its 16 rows of p; true when the kernel must stop
  auto vector_half = [&](int row) __attribute__((always_inline)) -> bool {
    // p: row 16 cb + po, columns [8 ppart, + 8) of W (from the caches: registers
    // are short)
    const int x0 = fresh_tid(), po = x0 >> 5, ppart = x0 & 31;
    const float4 w0 = *(const float4 *)&a.W[(size_t)(16 * cb + po) * 2 * D + 8 * ppart];
    const float4 w1 = *(const float4 *)&a.W[(size_t)(16 * cb + po) * 2 * D + 8 * ppart + 4];
    wait_for([&]() { return g[0].y == tag && g[1].y == tag && g[2].y == tag && g[3].y == tag; },
             [&]() { issue_gather(row); }, phase);
    (&bab_s[phase & 1][0][0])[x0] = (as_float(g[0].x) + as_float(g[1].x)) + (as_float(g[2].x) + as_float(g[3].x));
    __syncthreads();
    const bool stop = stop_s[phase & 1] != 0;
    const float *b0 = &bab_s[phase & 1][0][8 * ppart], *b1 = &bab_s[phase & 1][1][8 * ppart];
    const float wp[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) s = fmaf(wp[c], b0[c] + b1[c], s);
    ++phase;
    if (stop) return true;
#pragma unroll
    for (int x = 16; x > 0; x >>= 1) s += __shfl_xor(s, x, 32);
    if (ppart == 0) {
      const uint32_t el = (uint32_t)(row * D + 16 * cb + po);
      const float pv = tanh_f(s);
      hs.store1(el, pv, tag);
      a.h[el] = pv;
    }
    return false;
  };

  if (!kFused && N <= M::kCheckRows) {
    // small batches: every child row is in range, also those no node reads
#pragma unroll 1
    for (int i = blockIdx.x * kFwdThreads + fresh_tid(); i < 2 * N; i += gridDim.x * kFwdThreads) {
      const int c = a.child_rows[i];
      if (c < -1 || c >= N) raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
    }
  }
  int total = 0, listed = 0, off1 = 0;
#pragma unroll 1
  for (int first = 0;; first += kCap) {
    if (first > 0 && first >= total) break;
    __syncthreads();                            // every wave is done with the records
    {
      const int t0 = fresh_tid();
      total = list_tiles<INTS, 1>(offset, L, N, 1, L, group, ngroups, first, kCap, t0, list, wsum, bad);
      listed = min(total - first, kCap);
      if (__syncthreads_or(bad)) {
        raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
        return;
      }
      off1 = offset(1);
#pragma unroll 1
      for (int idx = t0; idx < 2 * listed; idx += kFwdThreads) {
        int *t = &list[(idx >> 1) * INTS];
        int c = child_row(t[0], idx & 1);
        if (c < -1 || c >= t[3]) {              // a child must sit in a lower level
          bad = 1;
          c = -1;
        }
        if (c >= 0 && c < off1) {
          const int xi = leaf_input(c);
          c = xi >= 0 ? -2 - xi : -1;
        }
        t[4 + (idx & 1)] = c;
      }
    }
    if (__syncthreads_or(bad)) {
      raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
      return;
    }
    if (listed > 0) issue(list);
    int pend = -1;                              // node whose second half is still to run
#pragma unroll 1
    for (int e = 0; e < listed; ++e) {
      int *t = &list[e * INTS];
      const bool more = e + 1 < listed;
      const int row = t[0];
      wait_for(ready, [&]() {
        if (cm >= 0) {
#pragma unroll
          for (int j = 0; j < 8; ++j) f[j] = ps.load1_at((uint32_t)((cm * D + kk + j) * D + col) * 8u);
        }
        if (cv >= 0) fv = hs.load1_at((uint32_t)(cv * D + col) * 8u);
      }, phase);
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = as_float(f[j].x);
      const float vec = as_float(fv.x);
      if (pend >= 0) issue_gather(pend);
      if (more) issue(t + INTS);
      // partial sums over this workgroup's columns: q[j] = M[kk + j][.] . vector,
      // folded so that lane i16 ends with row j = i16 / 2
      {
        float q[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) q[j] = v[j] * vec;
#pragma unroll
        for (int n = 4; n > 0; n >>= 1) {
          const bool up = (i16 & (2 * n)) != 0;
#pragma unroll
          for (int j = 0; j < n; ++j) {
            const float keep = up ? q[j + n] : q[j], give = up ? q[j] : q[j + n];
            q[j] = keep + __shfl_xor(give, 2 * n, 16);
          }
        }
        q[0] += __shfl_xor(q[0], 1, 16);
        // B a (rows of B) first, then A b
        if ((i16 & 1) == 0)
          xs.store1((uint32_t)((row * RB + cb) * 2 * D + (side ^ 1) * D + kk + (i16 >> 1)), q[0], tag);
      }
      const float4 v0 = make_float4(v[0], v[1], v[2], v[3]), v1 = make_float4(v[4], v[5], v[6], v[7]);
      // (also where a lane's elements are all below 2^-100: P is linear, and its
      // columns keep their own relative accuracy)
      const float top = max_abs(max_abs(0.f, v0), v1);
      if (top >= limit_s[wave] || as_uint(top) - 1u < as_uint(0x1p-100f) - 1u) t[3] = -1;     // read after the barrier
      const Split8 b = split8(v0, v1);
      // lane (column i16) receives rows 16 m + 4 g4 .. + 3; half of the row tiles
      // at a time, so the accumulators leave room for the next node's operands
      float *cbuf = &C_s[(e & 1) * CBUF];
      static_for<2>([&](auto half) __attribute__((always_inline)) {
        constexpr int HM = MT / 2, m0 = half * HM;
        floatx4 hi[HM], lo[HM];
#pragma unroll
        for (int m = 0; m < HM; ++m) lo[m] = mfma_bf16(wm[m0 + m].p2, b.p0, floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int m = 0; m < HM; ++m) lo[m] = mfma_bf16(wm[m0 + m].p1, b.p1, lo[m]);
#pragma unroll
        for (int m = 0; m < HM; ++m) lo[m] = mfma_bf16(wm[m0 + m].p0, b.p2, lo[m]);
#pragma unroll
        for (int m = 0; m < HM; ++m) lo[m] = mfma_bf16(wm[m0 + m].p1, b.p0, lo[m]);
#pragma unroll
        for (int m = 0; m < HM; ++m) lo[m] = mfma_bf16(wm[m0 + m].p0, b.p1, lo[m]);
#pragma unroll
        for (int m = 0; m < HM; ++m) hi[m] = mfma_bf16(wm[m0 + m].p0, b.p0, floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int m = 0; m < HM; ++m) *(floatx4 *)&cbuf[(wave * 16 + i16) * LDN + 16 * (m0 + m) + 4 * g4] = hi[m] + lo[m];
      });
      __syncthreads();
      const int stop = stop_s[phase & 1], mark = t[3];
      ++phase;
      if (stop) return;
      if (__builtin_expect(mark < 0, 0)) {
        // (every wave) its partial sums again on the fp32 matrix unit, operands
        // (all waited for) and weights from memory: step k takes the rows
        // 32 (wave & 3) + 8 g4 + k of this wave's matrix
        const int x0 = fresh_tid(), wave = x0 >> 6, i16 = x0 & 15, g4 = (x0 >> 4) & 3;
        const int c = t[4 + (wave >> 2)];
        const uint32_t at = (uint32_t)(((c >= 0 ? c : -2 - c) * D + 32 * (wave & 3) + 8 * g4) * D + 16 * cb + i16);
#pragma unroll 1
        for (int m = 0; m < MT; ++m) {
          floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int k = 0; k < 8; ++k) {
            float x = 0.f;
            if (c >= 0) x = as_float(ps.load1_at((at + k * D) * 8u).x);
            else if (c <= -2) x = as_float(xm.load1((at + k * D) * 4u));
            acc = mfma16x16x4(a.W_M[(size_t)(16 * m + i16) * 2 * D + 32 * wave + 8 * g4 + k], x, acc);
          }
          *(floatx4 *)&cbuf[(wave * 16 + i16) * LDN + 16 * m + 4 * g4] = acc;
        }
        __syncthreads();
      }
      {
        const int x0 = fresh_tid(), n = x0 & 15, r4 = 4 * (x0 >> 4);
        floatx4 s[kFwdWaves];
#pragma unroll
        for (int w = 0; w < kFwdWaves; ++w) s[w] = *(const floatx4 *)&cbuf[(w * 16 + n) * LDN + r4];
        const floatx4 sum = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
        const uint32_t el = (uint32_t)(row * D * D + r4 * D + 16 * cb + n);
#pragma unroll
        for (int i = 0; i < 4; ++i) ps.store1(el + i * D, sum[i], tag);
#pragma unroll
        for (int i = 0; i < 4; ++i) a.c[el + i * D] = sum[i];
      }
      // the previous node's second half, and this one's when it is the group's
      // last of its level: what follows may wait for its p
      const bool last = !more || t[INTS + 2] != t[2];
      int todo = pend;
      pend = row;
#pragma unroll 1
      for (;;) {
        if (todo >= 0 && vector_half(todo)) return;
        if (!last || pend < 0) break;
        issue_gather(pend);
        todo = pend;
        pend = -1;
      }
    }
  }
  // leaves: (p, P) = (x_table[x], leaf_mat[x]) or zeros, plain stores (no
  // workgroup reads them back)
  for (int r = blockIdx.x; r < off1; r += gridDim.x) {
    const int xi = leaf_input(r);
    if (tid < D / 4) {
      const float4 val = as_float4(xv.load4(xi >= 0 ? (uint32_t)((xi * D + tid * 4) * 4) : kNoSource));
      *(float4 *)&a.h[(size_t)r * D + tid * 4] = val;
    }
#pragma unroll
    for (int k = 0; k < D * D / 4 / kFwdThreads; ++k) {
      const int e = tid + k * kFwdThreads;
      const float4 val = as_float4(xm.load4(xi >= 0 ? (uint32_t)((xi * D * D + e * 4) * 4) : kNoSource));
      *(float4 *)&a.c[(size_t)r * D * D + e * 4] = val;
    }
  }
  if (a.retire) retire_tag(a.sync, tag, a.status, a.timeout);
}

}  // namespace cortex
