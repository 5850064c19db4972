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
#define BPPSA_FMAC(acc, x, w, n) \
  "v_fmac_f32_dpp %" #acc ", %" #x ", %" #w " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"

// orders the LDS accesses of the lanes of one wave
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
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
template <int Q, int C>
__device__ __forceinline__ float wave_product(const float (&w)[C], float s, float bias, float wi, float xs) {
  float a, p;
#define BPPSA_HEAD                                                                                    \
  "v_mov_b32 %0, %4\n\t"                                                                              \
  "v_fmac_f32_dpp %0, %5, %3 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
#define BPPSA_TAIL(rows) "v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane" #rows "_swap_b32 %0, %1\n\tv_add_f32 %0, %0, %1"
#define BPPSA_ARGS "v"(s), "v"(wi), "v"(bias), "v"(xs), "n"(Q)
#define BPPSA_COL(w, n) BPPSA_FMAC(0, 2, w, n)
#define BPPSA_COLS4 BPPSA_COL(7, 0) BPPSA_COL(8, 1) BPPSA_COL(9, 2) BPPSA_COL(10, 3)
#define BPPSA_COLS10 \
  BPPSA_COLS4 BPPSA_COL(11, 4) BPPSA_COL(12, 5) BPPSA_COL(13, 6) BPPSA_COL(14, 7) BPPSA_COL(15, 8) BPPSA_COL(16, 9)
#define BPPSA_COLS16                                                                                       \
  BPPSA_COLS10 BPPSA_COL(17, 10) BPPSA_COL(18, 11) BPPSA_COL(19, 12) BPPSA_COL(20, 13) BPPSA_COL(21, 14) \
  BPPSA_COL(22, 15)
#define BPPSA_W4 "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3])
#define BPPSA_W10 BPPSA_W4, "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]), "v"(w[8]), "v"(w[9])
#define BPPSA_W16 BPPSA_W10, "v"(w[10]), "v"(w[11]), "v"(w[12]), "v"(w[13]), "v"(w[14]), "v"(w[15])
#define BPPSA_BOTH(n)                                                                                         \
  do {                                                                                                        \
    if constexpr (Q % 2 == 0)                                                                                 \
      asm(BPPSA_HEAD BPPSA_COLS##n BPPSA_TAIL(16) : "=&v"(a), "=&v"(p) : BPPSA_ARGS, BPPSA_W##n);             \
    else                                                                                                      \
      asm(BPPSA_HEAD BPPSA_COLS##n BPPSA_TAIL(32) : "=&v"(a), "=&v"(p) : BPPSA_ARGS, BPPSA_W##n);             \
  } while (0)
  static_assert(C == 4 || C == 10 || C == 16, "no such form");
  if constexpr (C == 4) BPPSA_BOTH(4);
  else if constexpr (C == 10) BPPSA_BOTH(10);
  else BPPSA_BOTH(16);
#undef BPPSA_BOTH
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

  __device__ __forceinline__ WaveCell(int H, int I, const float* __restrict__ w_ih, const float* __restrict__ w_hh,
                                      const float* __restrict__ b_ih, const float* __restrict__ b_hh) {
    const int lane = threadIdx.x & 63, R = lane >> 4, i = lane & 15;
    unit[0] = C * (R >> 1) + i, unit[1] = C * (R & 1) + i;
    const int col0[2] = {C * (R & 1), C * (R >> 1)};
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const bool live = i < C && unit[f] < H;
      exists[f] = unit[f] < H;
      first[f] = live && col0[f] == 0;
#pragma unroll
      for (int n = 0; n < C; ++n) w[f][n] = (live && col0[f] + n < H) ? w_hh[(size_t)unit[f] * H + col0[f] + n] : 0.f;
#pragma unroll
      for (int k = 0; k < N; ++k) wi[f][k] = (first[f] && k < I) ? w_ih[(size_t)unit[f] * I + k] : 0.f;
      bias[f] = first[f] ? (b_ih ? b_ih[unit[f]] : 0.f) + (b_hh ? b_hh[unit[f]] : 0.f) : 0.f;
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

// The classifier's seed dL/dh_T of one sample, by one wave: last = h_T, w_out and what else is read in LDS; dz is left
// there.  Returns the sample's loss and entry `lane` of the seed.
struct HeadOut {
  float loss, seed;
};
__device__ __forceinline__ HeadOut head_of_sample(const bppsa_forward_tail& tail, int b, int B, int H, const float* w_out,
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
  return {loss, g};
}
// What the launch does for the next one: thread `me` of `all`.
__device__ __forceinline__ void prepare_scan(const bppsa_forward_tail& tail, int H, const float* __restrict__ w_hh, int me, int all) {
  for (long long k = me; k < tail.words; k += all) tail.clear[k] = 0;
  if (tail.w_hh_t)
    for (int k = me; k < H * H; k += all) tail.w_hh_t[(k % H) * H + k / H] = w_hh[k];
}

}  // namespace
