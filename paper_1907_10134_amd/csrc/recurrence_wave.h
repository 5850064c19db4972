// The walk of the tanh RNN with H <= 32 and at most four inputs by one wave per sample: what the launches of
// bppsa_forward and of a training iteration share.
#pragma once

#include "activations.h"
#include "barriers.h"
#include "bppsa_internal.h"
#include "train_parts.h"

namespace {

// Multiply-adds whose first factor is lane n of this lane's row of 16, several to a statement: between
// statements the compiler cannot see into it would put a wait state each.  A DPP operand may be read two
// wait states after a vector instruction wrote it, hence the s_nop in front.
#define BPPSA_FMAC_BARS(bar, acc, x, w, n) \
  "v_fmac_f32_dpp %" #acc ", " bar "%" #x bar ", " bar "%" #w bar " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
#define BPPSA_FMAC(acc, x, w, n) BPPSA_FMAC_BARS("", acc, x, w, n)

// orders the LDS accesses of the lanes of one wave
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Rows of 16 lanes (0 1 2 3): a and b exchange a's rows 1, 3 with b's rows 0, 2, giving
// a = (a0 b0 a2 b2), b = (a1 b1 a3 b3).
__device__ __forceinline__ void swap16(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// The same for halves of 32 lanes: a = (a0 a1 b0 b1), b = (a2 a3 b2 b3).
__device__ __forceinline__ void swap32(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}

// The largest magnitude in a wave whose rows 0 and 1, and 2 and 3, hold the same; a NaN if there is one (the bits of
// magnitudes are in the order of their values, with the NaNs last).  (The builtin of the swap, with one value as both
// operands, is compiled as if its two results were equal.)
__device__ __forceinline__ float max_of_rows(float x) {
  unsigned v = __builtin_bit_cast(unsigned, fabsf(x));
#define BPPSA_ROR(n) v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x120 + n, 0xf, 0xf, true))
  BPPSA_ROR(8);
  BPPSA_ROR(4);
  BPPSA_ROR(2);
  BPPSA_ROR(1);
#undef BPPSA_ROR
  float a = __builtin_bit_cast(float, v), b = a;
  swap32(a, b);
  return __builtin_bit_cast(float, max(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b)));
}

__device__ __forceinline__ void settle(float& x) { asm volatile("s_nop 1" : "+v"(x)); }

template <int Q>
struct Int {
  static constexpr int value = Q;
};

// ---- tanh RNN, H <= 32: one wave per sample ------------------------------------------------------
// Units and columns are cut in two halves A and B of C each (2 C >= H).  On even steps the rows of the wave hold
// (units, columns) = (A, A) (A, B) (B, A) (B, B), C of 16 lanes used: C multiply-adds, and one swap16 adds the two
// column halves.  That leaves the state as (A A B B), the order the columns of the transposed assignment
// (A, A) (B, A) (A, B) (B, B) need: odd steps use that one, and their swap32 gives back (A B A B).
constexpr int kWaveMaxI = 4;
constexpr int kWaveSteps = 16;       // steps per trip: their inputs are fetched one trip ahead

// a = sum of C columns + bias + lane Q of xs times wi, added up over the two rows that share the units (16 lanes
// apart on even steps, 32 on odd ones): both rows get the sum.  The first two instructions also are the wait states between the last write of s and its use.
// MAGNITUDES: the same of the absolute values.
template <int Q, int C, bool MAGNITUDES = false>
__device__ __forceinline__ float wave_product(const float (&w)[C], float s, float bias, float wi, float xs) {
  float a, p;
#define BPPSA_HEAD(bar)                                                                               \
  "v_mov_b32 %0, %4\n\t"                                                                              \
  "v_fmac_f32_dpp %0, " bar "%5" bar ", " bar "%3" bar " row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
#define BPPSA_TAIL(rows) "v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane" #rows "_swap_b32 %0, %1\n\tv_add_f32 %0, %0, %1"
#define BPPSA_ARGS "v"(s), "v"(wi), "v"(bias), "v"(xs), "n"(Q)
#define BPPSA_COL(bar, w, n) BPPSA_FMAC_BARS(bar, 0, 2, w, n)
#define BPPSA_COLS4(bar) BPPSA_COL(bar, 7, 0) BPPSA_COL(bar, 8, 1) BPPSA_COL(bar, 9, 2) BPPSA_COL(bar, 10, 3)
#define BPPSA_COLS10(bar)                                                                              \
  BPPSA_COLS4(bar) BPPSA_COL(bar, 11, 4) BPPSA_COL(bar, 12, 5) BPPSA_COL(bar, 13, 6) BPPSA_COL(bar, 14, 7) \
  BPPSA_COL(bar, 15, 8) BPPSA_COL(bar, 16, 9)
#define BPPSA_COLS16(bar)                                                                              \
  BPPSA_COLS10(bar) BPPSA_COL(bar, 17, 10) BPPSA_COL(bar, 18, 11) BPPSA_COL(bar, 19, 12) BPPSA_COL(bar, 20, 13) \
  BPPSA_COL(bar, 21, 14) BPPSA_COL(bar, 22, 15)
#define BPPSA_W4 "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3])
#define BPPSA_W10 BPPSA_W4, "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]), "v"(w[8]), "v"(w[9])
#define BPPSA_W16 BPPSA_W10, "v"(w[10]), "v"(w[11]), "v"(w[12]), "v"(w[13]), "v"(w[14]), "v"(w[15])
#define BPPSA_ROWS(n, bar, rows) \
  asm(BPPSA_HEAD(bar) BPPSA_COLS##n(bar) BPPSA_TAIL(rows) : "=&v"(a), "=&v"(p) : BPPSA_ARGS, BPPSA_W##n)
#define BPPSA_BOTH(n)                                                  \
  do {                                                                 \
    if constexpr (MAGNITUDES && Q % 2 == 0) BPPSA_ROWS(n, "|", 16);    \
    else if constexpr (MAGNITUDES) BPPSA_ROWS(n, "|", 32);             \
    else if constexpr (Q % 2 == 0) BPPSA_ROWS(n, "", 16);              \
    else BPPSA_ROWS(n, "", 32);                                        \
  } while (0)
  static_assert(C == 4 || C == 10 || C == 16, "no such form");
  if constexpr (C == 4) BPPSA_BOTH(4);
  else if constexpr (C == 10) BPPSA_BOTH(10);
  else BPPSA_BOTH(16);
#undef BPPSA_BOTH
#undef BPPSA_ROWS
#undef BPPSA_W16
#undef BPPSA_W10
#undef BPPSA_W4
#undef BPPSA_COLS16
#undef BPPSA_COLS10
#undef BPPSA_COLS4
#undef BPPSA_COL
#undef BPPSA_ARGS
#undef BPPSA_TAIL
#undef BPPSA_HEAD
  return a;
}

// N inputs per step, at most; the ones past the first come in through a scalar each.
// A second wave brings the inputs into LDS, a trip of kWaveSteps steps at a time: loads and stores share one counter
// and loads would wait for the stores before them, so the wave that stores the states loads nothing in its loop.
// (H = 20: 14 ns a step.)
template <int N>
using Ahead = float[2][N][kWaveSteps + 1];          // inputs of a trip, and a zero

// The second wave's part of a walk over the steps [t0, t1): barrier m says that the inputs of trip m are in LDS and
// those of trip m - 1 in registers.
template <int N>
__device__ __forceinline__ void feed_walk(Ahead<N>& ahead, int t0, int t1, int b, int B, int I, const float* __restrict__ x) {
  const int lane = threadIdx.x & 63;
  float even[N], odd[N];
  auto fetch = [&](float (&to)[N], int t) {
#pragma unroll
    for (int k = 0; k < N; ++k) to[k] = (k < I && t + lane < t1) ? x[((size_t)(t + lane) * B + b) * I + k] : 0.f;
  };
  if (lane < kWaveSteps) {
    fetch(even, t0);
    fetch(odd, t0 + kWaveSteps);
  }
  for (;; t0 += 2 * kWaveSteps) {
    auto pass = [&](float (&from)[N], int buf, int next) {
      if (lane < kWaveSteps) {
#pragma unroll
        for (int k = 0; k < N; ++k) ahead[buf][k][lane] = from[k];
        fetch(from, next);
      } else if (lane == kWaveSteps) {
#pragma unroll
        for (int k = 0; k < N; ++k) ahead[buf][k][lane] = 0.f;
      }
      lds_barrier();
    };
    pass(even, 0, t0 + 2 * kWaveSteps);            // the last one: a trip that does not exist
    if (t0 >= t1) return;
    pass(odd, 1, t0 + 3 * kWaveSteps);
    if (t0 + kWaveSteps >= t1) return;
  }
}

// The first wave's part, and single steps.
template <int C, int N, bool EXACT>                // EXACT: H = 2 C, every unit of the halves exists
struct WaveCell {
  // the unit whose rows a lane holds, on even and on odd steps
  int unit[2];
  float w[2][C], wi[2][N], bias[2];
  // the inputs and the bias enter through the rows of column half A, which also store the states
  bool first[2], exists[2];

  // (needed: whether this wave walks; the others should not queue for weights)
  __device__ __forceinline__ WaveCell(int H, int I, const float* __restrict__ w_ih, const float* __restrict__ w_hh,
                                      const float* __restrict__ b_ih, const float* __restrict__ b_hh, bool needed = true) {
    const int lane = threadIdx.x & 63, R = lane >> 4, i = lane & 15;
    unit[0] = C * (R >> 1) + i, unit[1] = C * (R & 1) + i;
    const int col0[2] = {C * (R & 1), C * (R >> 1)};
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const bool live = i < C && unit[f] < H;
      exists[f] = unit[f] < H;
      first[f] = live && col0[f] == 0;
      if (needed) {
#pragma unroll
        for (int n = 0; n < C; ++n) w[f][n] = (live && col0[f] + n < H) ? w_hh[(size_t)unit[f] * H + col0[f] + n] : 0.f;
#pragma unroll
        for (int k = 0; k < N; ++k) wi[f][k] = (first[f] && k < I) ? w_ih[(size_t)unit[f] * I + k] : 0.f;
        bias[f] = first[f] ? (b_ih ? b_ih[unit[f]] : 0.f) + (b_hh ? b_hh[unit[f]] : 0.f) : 0.f;
      } else {
#pragma unroll
        for (int n = 0; n < C; ++n) w[f][n] = 0.f;
#pragma unroll
        for (int k = 0; k < N; ++k) wi[f][k] = 0.f;
        bias[f] = 0.f;
      }
    }
  }

  // a state as even steps want it, (A B A B)
  __device__ __forceinline__ float load_state(const float* __restrict__ row, int H) const {
    return ((threadIdx.x & 15) < C && unit[1] < H) ? row[unit[1]] : 0.f;
  }

  template <int Q>
  __device__ __forceinline__ float step(float s, const float (&xs)[N]) const {
    constexpr int F = Q & 1;
    float in = bias[F];
#pragma unroll
    for (int k = 1; k < N; ++k)
      in = __builtin_fmaf(wi[F][k], __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, xs[k]),
                                                                                      0x150 + Q, 0xf, 0xf, true)), in);
    const float pre = wave_product<Q>(w[F], s, in, wi[F][0], xs[0]);
    s = EXACT && C == 10 ? bppsa_tanh_short(pre) : bppsa_tanh(pre);
    if (!EXACT) s = exists[F] ? s : 0.f;           // a column that does not exist must not carry a NaN
    return s;
  }

  // the magnitudes of what step<0> adds up
  __device__ __forceinline__ float terms(float s, const float (&xs)[N]) const {
    float in = fabsf(bias[0]);
#pragma unroll
    for (int k = 1; k < N; ++k)
      in = __builtin_fmaf(fabsf(wi[0][k]), __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(
                                               __builtin_bit_cast(int, fabsf(xs[k])), 0x150, 0xf, 0xf, true)), in);
    return wave_product<0, C, true>(w[0], s, in, wi[0][0], xs[0]);
  }

  // The states after the steps [t0, t1), t0 a multiple of kWaveSteps, from the state s before them; returns the last.
  // Rows up to `from` (a multiple of kWaveSteps) are not stored.
  __device__ __forceinline__ float walk(Ahead<N>& ahead, float s, int t0, int t1, int from, int b, int B, int H,
                                        float* __restrict__ h) const {
    const int lane = threadIdx.x & 63, R = lane >> 4, i = lane & 15;
    // Stores go through a buffer descriptor that ends with the trip's last row: lanes that own no unit
    // carry an offset past its end and store nothing, without a change of the lane mask.
    const unsigned row_bytes = (unsigned)B * (unsigned)H * 4u;
    unsigned voff[2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
      voff[f] = first[f] ? ((unsigned)b * (unsigned)H + (unsigned)unit[f]) * 4u : 0x80000000u;
    // lane i of a row holds the input of step t0 + i, in the rows of that step's column half A (elsewhere its
    // weight is zero, and the input must not be infinite)
    const int take = ((i & 1) ? R < 2 : (R & 1) == 0) ? i : kWaveSteps;
    auto fetch = [&](float (&xs)[N], int buf) {
      lds_barrier();
#pragma unroll
      for (int k = 0; k < N; ++k) xs[k] = ahead[buf][k][take];
    };
    float xs[N], xn[N];
    fetch(xs, 0);
    int buf = 1;
    for (; t0 + kWaveSteps <= t1; t0 += kWaveSteps) {
      fetch(xn, buf);
      buf ^= 1;
      const auto rows = __builtin_amdgcn_make_buffer_rsrc(h + (size_t)(t0 + 1) * B * H, 0,
                                                          t0 < from ? 0 : (int)(kWaveSteps * row_bytes), 0x00020000);
      settle(xs[0]);
      auto put = [&](auto q) {
        constexpr int Q = decltype(q)::value;
        s = step<Q>(s, xs);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, s), rows, (int)voff[Q & 1],
                                              (int)((unsigned)Q * row_bytes), 0);
      };
      put(Int<0>{}), put(Int<1>{}), put(Int<2>{}), put(Int<3>{}), put(Int<4>{}), put(Int<5>{}), put(Int<6>{}), put(Int<7>{});
      put(Int<8>{}), put(Int<9>{}), put(Int<10>{}), put(Int<11>{}), put(Int<12>{}), put(Int<13>{}), put(Int<14>{});
      put(Int<15>{});
#pragma unroll
      for (int k = 0; k < N; ++k) xs[k] = xn[k];
    }
    if (t0 < t1) lds_barrier();                    // the trip that does not exist
    // what is left of a trip: the inputs move down two lanes per pair of steps
    for (int t = t0; t < t1; t += 2) {
      settle(xs[0]);
      s = step<0>(s, xs);
      if (first[0]) h[((size_t)(t + 1) * B + b) * H + unit[0]] = s;
      if (t + 1 < t1) {
        s = step<1>(s, xs);
        if (first[1]) h[((size_t)(t + 2) * B + b) * H + unit[1]] = s;
      }
#pragma unroll
      for (int k = 0; k < N; ++k) xs[k] = __shfl_down(xs[k], 2, 16);
    }
    return s;
  }
};

// ---- the sequence in segments --------------------------------------------------------------------
// A walk is bound by the latency of its steps and leaves most of the chip idle, so a long sequence is cut into
// segments that are walked at the same time.  A segment does not know the state it starts from.  But a cell that
// forgets (with weights of the usual initialisation a state's influence halves with every step) reaches the states
// of the whole sequence from any other state after a number of steps, to the last bits, where rounding keeps two walks
// apart: a segment starts `warm` steps early, from zero, and stores nothing until its own first step.
// Nothing rests on that alone.  A second launch takes the step across every seam again, from the state stored before
// it, in the order of the walk, and compares with the state stored behind it, unit by unit.  A seam holds where no unit
// differs by more than the rounding of that step to it: 2^-22 of half its new state and of the magnitudes of its terms,
// as the derivatives of what follows the sums pass them on.  So a unit that is small or remembers is held to its own
// scale, whatever the others are.  Nor may it differ by more than kSeamMost of the largest state, which counts where terms
// cancel or overflow.  In 176000 seams of 8 to 30 sets of initial weights each (H = 9 to 128, bits and normal inputs) two
// walks that differ by rounding alone used up to 0.91 of the first bound, one seam in a thousand more than 0.68; of the
// second up to 0.91 (H = 20; one seam of H = 19 1.0).  Where a seam does not hold (long memories, a chaotic cell, NaN) the
// sequence is walked again from the state before it, up to the next seam that holds, by the wave form in rounds of
// four walks unless hardly a seam holds.
// Every step of the result is then a step of the cell to within the rounding of its own terms, for any weights and
// inputs.
// Errors against 64 bits, segments over one walk (2-norm, 8 sets of weights, T = 1000, B = 16): H = 20 1.000, with
// recurrent weights 1.5 times as large 1.003 and from 2 times on 1 (no seam holds: the same bits); H = 8 1.000 to
// 1.001, H = 32 1.000 to 1.006, H = 64 1.000 to 1.030, H = 128 0.999 to 1.019; GRU H = 20 0.999 to 1.003, H = 128 1.000 to
// 1.013.  Of a unit by itself, at worst: 1.04 with initial weights, 1.28 with larger ones.
constexpr float kSeam = 0x1p-22f, kSeamMost = 0x1p-21f;
constexpr float kSeamLeast = 0x1p-126f;            // below that numbers have no more digits to lose
// y: the step's result; own: half its magnitude and the terms'; most: the largest state.  A NaN does not hold.
__device__ __forceinline__ bool seam_holds(float y, float stored, float own, float limit) {
  const float off = fabsf(y - stored);
  return off <= __builtin_fmaf(kSeam, own, kSeamLeast) && off <= limit + kSeamLeast;
}

// Whether the step before step t from the state stored there leads to the state stored behind it; by a wave.
template <int C, int N, bool EXACT>
struct Seams {
  const WaveCell<C, N, EXACT>& cell;
  const float* x;
  float* hb;                                       // h of this sample
  int b, B, H, I;
  bool input, owns;
  __device__ __forceinline__ Seams(const WaveCell<C, N, EXACT>& cell, const float* x, float* h, int b, int B, int H, int I)
      : cell(cell), x(x), hb(h + (size_t)b * H), b(b), B(B), H(H), I(I), input((threadIdx.x >> 4 & 1) == 0),
        owns((threadIdx.x & 15) < C && cell.unit[0] < H) {}
  __device__ __forceinline__ size_t row() const { return (size_t)B * H; }
  __device__ __forceinline__ float state(int t) const { return cell.load_state(hb + (size_t)t * row(), H); }
  __device__ __forceinline__ float stored(int t) const { return owns ? hb[(size_t)(t + 1) * row() + cell.unit[0]] : 0.f; }
  __device__ __forceinline__ void inputs(float (&xs)[N], int t) const {
#pragma unroll
    for (int k = 0; k < N; ++k) xs[k] = (k < I && input) ? x[((size_t)t * B + b) * I + k] : 0.f;
  }
  // several at once, so that their exchanges between lanes overlap
  template <int K>
  __device__ __forceinline__ void hold(bool (&ok)[K], const float (&s)[K], float (&xs)[K][N], const float (&stored)[K]) const {
    float y[K], own[K], most[K];
#pragma unroll
    for (int u = 0; u < K; ++u) {
      settle(xs[u][0]);
      y[u] = cell.template step<0>(s[u], xs[u]);
      own[u] = __builtin_fmaf(__builtin_fmaf(-y[u], y[u], 1.f), cell.terms(s[u], xs[u]), 0.5f * fabsf(y[u]));
    }
#pragma unroll
    for (int u = 0; u < K; ++u) most[u] = max_of_rows(owns ? stored[u] : 0.f);
#pragma unroll
    for (int u = 0; u < K; ++u)
      ok[u] = __builtin_amdgcn_ballot_w64(owns && !seam_holds(y[u], stored[u], own[u], kSeamMost * most[u])) == 0;
  }
  __device__ __forceinline__ bool holds(int t) const {
    float s[1] = {state(t)}, xs[1][N];
    inputs(xs[0], t);
    const float y[1] = {stored(t)};
    bool ok[1];
    hold(ok, s, xs, y);
    return ok[0];
  }
};

// One sample by the 2 WALKS waves of a workgroup (the first half walk, the others feed them), in rounds: walk 0 goes on
// from the last true state and is as long as the others with their warm steps, the others start from that state too, a
// segment further on each, and the seams say how many of them count.  Where none does a round was no longer than the
// steps it took one walk, so a cell that does not forget costs little more than one walk, and one that holds on to
// something (training leads there) is soon in the right one of the states it was kept apart by.
template <int N, int WALKS>
struct RoundsLds {
  Ahead<N> ahead[WALKS];
  int joined[WALKS];
  float last[32];                                  // h_T, once a walk has got there
};
template <int WALKS, int C, int N, bool EXACT>
struct Rounds {
  RoundsLds<N, WALKS>& lds;
  const Seams<C, N, EXACT>& at;
  float* h;
  int T;

  // Walk 0 takes [base, base + lead) from the state stored there, walk p > 0 starts from it at base + p len and stores
  // [base + lead + (p - 1) len, ...), len steps.  Returns how far the states are true then.  base, len and, unless it
  // ends the sequence, lead are multiples of kWaveSteps.
  __device__ __forceinline__ int round(int base, int lead, int len, int walks) const {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), walk = wave & (WALKS - 1);
    const int from = walk ? base + lead + (walk - 1) * len : base, to = min(T, walk ? from + len : base + lead);
    const int t0 = base + walk * len, trips = (min(T, base + lead) - base + kWaveSteps - 1) / kWaveSteps;
    const bool has = walk == 0 || (walk < walks && from < T);
    if (has && wave < WALKS) {
      const float s = at.cell.walk(lds.ahead[walk], at.state(base), t0, to, from, at.b, at.B, at.H, h);
      const int u = to & 1 ? at.cell.unit[0] : at.cell.unit[1];
      if (to == T && (threadIdx.x & 15) < C && u < at.H) lds.last[u] = s;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // rows that other waves go on from
    } else if (has) {
      feed_walk<N>(lds.ahead[walk], t0, to, at.b, at.B, at.I, at.x);
    }
    // the barriers of the longest walk: one, and one a trip
    for (int k = has ? 1 + (to - t0 + kWaveSteps - 1) / kWaveSteps : 0; k < 1 + trips; ++k) lds_barrier();
    __syncthreads();
    if (walks == 1) return min(T, base + lead);
    if (wave < WALKS) {
      const bool ok = !has || walk == 0 || at.holds(from);
      if ((threadIdx.x & 63) == 0) lds.joined[walk] = ok;
    }
    __syncthreads();
    int past = 1;
    while (past < walks && lds.joined[past]) ++past;
    __syncthreads();
    return min(T, base + lead + (past - 1) * len);
  }

  // All of it from the state stored before step `base` on.  WALKS = 8: two walks on a SIMD take 1.4 times as long as one,
  // which pays for the first round only.
  __device__ __forceinline__ void run(int base) const {
    bool none = false;                             // no seam of the round before held
    for (int walks = WALKS; base < T; walks = WALKS < 4 ? WALKS : 4) {
      const int left = T - base, warm = left < 800 || base == 0 ? kRoundWarm : 160;
      int len = (left - warm) / walks / kWaveSteps * kWaveSteps + kWaveSteps;
      if (len < 2 * kWaveSteps) len = 2 * kWaveSteps;
      const int least = base == 0 ? rounds_from() : none ? 4 * warm : 2 * warm, lead = left <= least ? left : warm + len;
      const int next = round(base, lead, len, left <= least ? 1 : walks);
      none = next == base + lead;
      base = next;
    }
  }
  static constexpr int kRoundWarm = C < 8 ? 128 : 96;             // (segments: 128 below H = 16, see cut_of)
  // Longer sequences than this are begun in rounds.  H = 20, B = 200, one walk, rounds, and rounds of a cell that does
  // not forget: T = 250 23.7, 23.5, 33.2 us; T = 300 27.6, 24.0, 38.4; T = 500 42.5, 27.9, 53.8.
  static __device__ __forceinline__ int rounds_from() { return 3 * kRoundWarm; }
  // the waves that need the cell
  static __device__ __forceinline__ int walking(int T) { return T <= rounds_from() ? 1 : WALKS; }
};

// The classifier's seed dL/dh_T of one sample, by one wave: last = h_T, w_out and what else is read in LDS; dz is left
// there.  Returns entry `lane` of the seed.
__device__ __forceinline__ float head_of_sample(const bppsa_forward_tail& tail, int b, int B, int H, const float* w_out,
                                               float b_out, int label, const float* last, float* dz) {
  const int lane = threadIdx.x & 63, n = tail.C;
  float z = -INFINITY;
  if (lane < n) {
    z = b_out;
#pragma unroll 4
    for (int j = 0; j < H; ++j) z += w_out[lane * H + j] * last[j];
  }
  const float m = bppsa_wave_max(z);
  const float lse = m + logf(bppsa_wave_sum(lane < n ? expf(z - m) : 0.f));
  const float loss = lse - (label >= 0 && label < n ? __shfl(z, label, 64) : 0.f);
  if (lane < n) dz[lane] = (expf(z - lse) - (lane == label ? 1.f : 0.f)) * (1.0f / (float)B);
  wave_fence();
  float g = 0.f;
  if (lane < H) {
#pragma unroll 4
    for (int k = 0; k < n; ++k) g += dz[k] * w_out[k * H + lane];
    tail.seed[(size_t)b * H + lane] = g;
  }
  if (tail.share) {
    float* const share = tail.share + (size_t)b * tail.share_stride;
    for (int e = lane; e < n * (H + 1); e += 64) {
      const int c = e / (H + 1), j = e - c * (H + 1);
      share[e] = dz[c] * (j < H ? last[j] : 1.f);
    }
    if (lane == 0) share[n * (H + 1)] = loss * (1.0f / (float)B);
  }
  return g;
}
// What the launch does for the next one: thread `me` of `all`.
__device__ __forceinline__ void prepare_scan(const bppsa_forward_tail& tail, int H, const float* __restrict__ w_hh, int me, int all) {
  for (long long k = me; k < tail.words; k += all) tail.clear[k] = 0;
  if (tail.w_hh_t)
    for (int k = me; k < H * H; k += all) tail.w_hh_t[(k % H) * H + k / H] = w_hh[k];
}

}  // namespace
