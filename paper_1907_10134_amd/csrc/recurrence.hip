// bppsa_forward for hidden sizes up to 128: the walk over time, which no scan takes apart.
//
// A step is a matrix-vector product with weights that never change, a few transcendental functions and
// an exchange of H values, and the next step waits for all of it: T steps cost T times the latency of
// one, whatever the bandwidth.  So the weights stay in registers and the step is made of few
// instructions with short latencies (a wave issues one every four cycles; an LDS round trip is 60
// cycles, one with a workgroup barrier 125 to 170):
//   - the state is the DPP operand of the multiply-adds.  Lane i of a row of 16 lanes holds column i of
//     the state, and v_fmac_f32 with row_newbcast:n multiplies the weights of all 16 lanes by the value
//     of lane n: 16 columns from one register, and neither a broadcast read from LDS per column nor a
//     scalar register;
//   - the columns are dealt to the rows of a wave, and the partial sums of the rows meet in
//     v_permlane16_swap / v_permlane32_swap, which exchange rows between two registers in one
//     instruction (two values are reduced per exchange where there are several gates).
// Two forms:
//   rnn_forward_wave_kernel    tanh RNN, H <= 32, at most 4 inputs: one wave per sample walks, a second one
//                              fetches the inputs; no LDS and no barrier in a step.
//   forward_block_kernel       both cells, H <= 128, at most 40 inputs: a wave per 16 units, the state
//                              through LDS with one barrier per step, and two more waves that do the
//                              memory traffic (inputs fetched 16 steps ahead, states stored), so that no
//                              wave of the recurrence ever waits for memory.
// The inputs are further columns of the product: their weights sit in registers beside the others.
//
// Measured (bppsa_forward, before = one wave with the state in LDS for H = 20, one 1024-thread workgroup
// with two barriers per step for the GRU at H = 128, weights re-read from the cache every step elsewhere):
//   RNN H = 20, T = 1000, B = 16            219 -> 77 us     (0.074 us a step, about 0.015 of it the tanh)
//   RNN H = 64, T = 300, B = 7              344 -> 66 us
//   GRU H = 20, I = 24, T = 517, B = 32    1466 -> 162 us
//   GRU H = 128, I = 1, T = 4096, B = 16   4617 -> 2810 us   (0.69 us a step: 99 multiply-adds of each
//                                          of two waves per SIMD take two thirds of it)
//   GRU H = 128, I = 12, T = 1034, B = 5   6868 -> 750 us
// Past 40 inputs bppsa_forward falls back to a kernel that reads every weight from the cache in every step: 500 steps of
// 16 samples take 420 us at I = 40 and 6220 at I = 41 for the GRU of H = 128, 168 and 1836 for H = 20, 106 and 1577
// for the RNN of H = 20.  The RNN's step from the wave to the block form (I = 4 to 5) is 58 to 90 us.
#include "activations.h"
#include "bppsa_internal.h"
#include "train_parts.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// Multiply-adds whose first factor is lane n of this lane's row of 16, several to a statement: between
// statements the compiler cannot see into it would put a wait state each.  A DPP operand may be read two
// wait states after a vector instruction wrote it, hence the s_nop in front.
#define BPPSA_FMAC(acc, x, w, n) \
  "v_fmac_f32_dpp %" #acc ", %" #x ", %" #w " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
#define BPPSA_FMAC3(x, w0, w1, w2, n) BPPSA_FMAC(0, x, w0, n) BPPSA_FMAC(1, x, w1, n) BPPSA_FMAC(2, x, w2, n)
#define BPPSA_W3(w, c) "v"(w[0][c]), "v"(w[1][c]), "v"(w[2][c])

// acc[g] += sum of w[g][K + c] * (lane F + c of x), c < N: the blocks the forms below are made of
template <int N, int K, int F, int C>
__device__ __forceinline__ void fmac_block(float (&a)[3], const float (&w)[3][C], float x) {
  if constexpr (N == 1 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC3(3, 4, 5, 6, 0) : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]) : "v"(x), BPPSA_W3(w, K));
  else if constexpr (N == 3 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC3(3, 4, 5, 6, 0) BPPSA_FMAC3(3, 7, 8, 9, 1) BPPSA_FMAC3(3, 10, 11, 12, 2)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]) : "v"(x), BPPSA_W3(w, K), BPPSA_W3(w, K + 1), BPPSA_W3(w, K + 2));
  else if constexpr (N == 5 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC3(3, 4, 5, 6, 0) BPPSA_FMAC3(3, 7, 8, 9, 1) BPPSA_FMAC3(3, 10, 11, 12, 2)
        BPPSA_FMAC3(3, 13, 14, 15, 3) BPPSA_FMAC3(3, 16, 17, 18, 4)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2])
        : "v"(x), BPPSA_W3(w, K), BPPSA_W3(w, K + 1), BPPSA_W3(w, K + 2), BPPSA_W3(w, K + 3), BPPSA_W3(w, K + 4));
  else if constexpr (N == 5 && F == 5)
    asm("s_nop 1\n\t" BPPSA_FMAC3(3, 4, 5, 6, 5) BPPSA_FMAC3(3, 7, 8, 9, 6) BPPSA_FMAC3(3, 10, 11, 12, 7)
        BPPSA_FMAC3(3, 13, 14, 15, 8) BPPSA_FMAC3(3, 16, 17, 18, 9)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2])
        : "v"(x), BPPSA_W3(w, K), BPPSA_W3(w, K + 1), BPPSA_W3(w, K + 2), BPPSA_W3(w, K + 3), BPPSA_W3(w, K + 4));
  else if constexpr (N == 8 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC3(3, 4, 5, 6, 0) BPPSA_FMAC3(3, 7, 8, 9, 1) BPPSA_FMAC3(3, 10, 11, 12, 2)
        BPPSA_FMAC3(3, 13, 14, 15, 3) BPPSA_FMAC3(3, 16, 17, 18, 4) BPPSA_FMAC3(3, 19, 20, 21, 5)
        BPPSA_FMAC3(3, 22, 23, 24, 6) BPPSA_FMAC3(3, 25, 26, 27, 7)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2])
        : "v"(x), BPPSA_W3(w, K), BPPSA_W3(w, K + 1), BPPSA_W3(w, K + 2), BPPSA_W3(w, K + 3), BPPSA_W3(w, K + 4),
          BPPSA_W3(w, K + 5), BPPSA_W3(w, K + 6), BPPSA_W3(w, K + 7));
  else {
    static_assert(N == 8 && F == 8, "no such block");
    asm("s_nop 1\n\t" BPPSA_FMAC3(3, 4, 5, 6, 8) BPPSA_FMAC3(3, 7, 8, 9, 9) BPPSA_FMAC3(3, 10, 11, 12, 10)
        BPPSA_FMAC3(3, 13, 14, 15, 11) BPPSA_FMAC3(3, 16, 17, 18, 12) BPPSA_FMAC3(3, 19, 20, 21, 13)
        BPPSA_FMAC3(3, 22, 23, 24, 14) BPPSA_FMAC3(3, 25, 26, 27, 15)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2])
        : "v"(x), BPPSA_W3(w, K), BPPSA_W3(w, K + 1), BPPSA_W3(w, K + 2), BPPSA_W3(w, K + 3), BPPSA_W3(w, K + 4),
          BPPSA_W3(w, K + 5), BPPSA_W3(w, K + 6), BPPSA_W3(w, K + 7));
  }
}
template <int N, int K, int F, int C>
__device__ __forceinline__ void fmac_block(float (&a)[1], const float (&w)[1][C], float x) {
#define BPPSA_W1(c) "v"(w[0][c])
  if constexpr (N == 1 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC(0, 1, 2, 0) : "+v"(a[0]) : "v"(x), BPPSA_W1(K));
  else if constexpr (N == 3 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC(0, 1, 2, 0) BPPSA_FMAC(0, 1, 3, 1) BPPSA_FMAC(0, 1, 4, 2)
        : "+v"(a[0]) : "v"(x), BPPSA_W1(K), BPPSA_W1(K + 1), BPPSA_W1(K + 2));
  else if constexpr (N == 5 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC(0, 1, 2, 0) BPPSA_FMAC(0, 1, 3, 1) BPPSA_FMAC(0, 1, 4, 2) BPPSA_FMAC(0, 1, 5, 3)
        BPPSA_FMAC(0, 1, 6, 4)
        : "+v"(a[0]) : "v"(x), BPPSA_W1(K), BPPSA_W1(K + 1), BPPSA_W1(K + 2), BPPSA_W1(K + 3), BPPSA_W1(K + 4));
  else if constexpr (N == 5 && F == 5)
    asm("s_nop 1\n\t" BPPSA_FMAC(0, 1, 2, 5) BPPSA_FMAC(0, 1, 3, 6) BPPSA_FMAC(0, 1, 4, 7) BPPSA_FMAC(0, 1, 5, 8)
        BPPSA_FMAC(0, 1, 6, 9)
        : "+v"(a[0]) : "v"(x), BPPSA_W1(K), BPPSA_W1(K + 1), BPPSA_W1(K + 2), BPPSA_W1(K + 3), BPPSA_W1(K + 4));
  else if constexpr (N == 8 && F == 0)
    asm("s_nop 1\n\t" BPPSA_FMAC(0, 1, 2, 0) BPPSA_FMAC(0, 1, 3, 1) BPPSA_FMAC(0, 1, 4, 2) BPPSA_FMAC(0, 1, 5, 3)
        BPPSA_FMAC(0, 1, 6, 4) BPPSA_FMAC(0, 1, 7, 5) BPPSA_FMAC(0, 1, 8, 6) BPPSA_FMAC(0, 1, 9, 7)
        : "+v"(a[0])
        : "v"(x), BPPSA_W1(K), BPPSA_W1(K + 1), BPPSA_W1(K + 2), BPPSA_W1(K + 3), BPPSA_W1(K + 4), BPPSA_W1(K + 5),
          BPPSA_W1(K + 6), BPPSA_W1(K + 7));
  else {
    static_assert(N == 8 && F == 8, "no such block");
    asm("s_nop 1\n\t" BPPSA_FMAC(0, 1, 2, 8) BPPSA_FMAC(0, 1, 3, 9) BPPSA_FMAC(0, 1, 4, 10) BPPSA_FMAC(0, 1, 5, 11)
        BPPSA_FMAC(0, 1, 6, 12) BPPSA_FMAC(0, 1, 7, 13) BPPSA_FMAC(0, 1, 8, 14) BPPSA_FMAC(0, 1, 9, 15)
        : "+v"(a[0])
        : "v"(x), BPPSA_W1(K), BPPSA_W1(K + 1), BPPSA_W1(K + 2), BPPSA_W1(K + 3), BPPSA_W1(K + 4), BPPSA_W1(K + 5),
          BPPSA_W1(K + 6), BPPSA_W1(K + 7));
  }
#undef BPPSA_W1
}

// acc[g] += sum over C columns of w[g][c] * x[column c]; x0 holds columns 0..15, x1 columns 16..31.
template <int G, int C>
__device__ __forceinline__ void add_columns(float (&acc)[G], const float (&w)[G][C], float x0, float x1) {
  if constexpr (C < 8) {
    fmac_block<C, 0, 0>(acc, w, x0);
  } else if constexpr (C == 10) {
    fmac_block<5, 0, 0>(acc, w, x0);
    fmac_block<5, 5, 5>(acc, w, x0);
  } else {
    static_assert(C % 8 == 0 && C <= 32, "no such block");
    fmac_block<8, 0, 0>(acc, w, x0);
    if constexpr (C >= 16) fmac_block<8, 8, 8>(acc, w, x0);
    if constexpr (C >= 24) fmac_block<8, 16, 0>(acc, w, x1);
    if constexpr (C >= 32) fmac_block<8, 24, 8>(acc, w, x1);
  }
}

// barriers that leave loads and stores outstanding
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
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

// Rows of 16 lanes (0 1 2 3): a and b exchange a's rows 1, 3 with b's rows 0, 2, giving
// a = (a0 b0 a2 b2), b = (a1 b1 a3 b3).
__device__ __forceinline__ void swap16(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// The same for halves of 32 lanes: a = (a0 a1 b0 b1), b = (a2 a3 b2 b3).
__device__ __forceinline__ void swap32(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}

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
// HEAD: the classifier's seed dL/dh_T follows in the same launch (a training iteration): each sample's last state is
// still in its wave's registers, and a launch of its own takes 6 us.  The workgroups also zero the words the next
// launch wants zeroed.
template <int C, int N, bool EXACT, bool HEAD>      // EXACT: H = 2 C, every unit of the halves exists
__global__ void __launch_bounds__(128)
rnn_forward_wave_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                        const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                        const float* __restrict__ b_hh, float* __restrict__ h, const bppsa_forward_tail tail) {
  __shared__ float w_out[HEAD ? 64 * 2 * C : 1], last[HEAD ? 2 * C : 1], dz[HEAD ? 64 : 1];
  __shared__ int label;
  __shared__ float ahead[2][N][kWaveSteps + 1];    // inputs of a trip, and a zero
  const int b = blockIdx.x, lane = threadIdx.x & 63, R = lane >> 4, i = lane & 15;
  if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 1) {
    // barrier m: the inputs of trip m are in LDS, those of trip m - 1 are in registers
    float even[N], odd[N];
    auto fetch = [&](float (&to)[N], int t0) {
#pragma unroll
      for (int k = 0; k < N; ++k) to[k] = (k < I && t0 + lane < T) ? x[((size_t)(t0 + lane) * B + b) * I + k] : 0.f;
    };
    if (lane < kWaveSteps) {
      fetch(even, 0);
      fetch(odd, kWaveSteps);
    }
    for (int t0 = 0;; t0 += 2 * kWaveSteps) {
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
      pass(even, 0, t0 + 2 * kWaveSteps);          // the last one: a trip that does not exist
      if (t0 >= T) return;
      pass(odd, 1, t0 + 3 * kWaveSteps);
      if (t0 + kWaveSteps >= T) return;
    }
  }
  float b_out = 0.f;
  if constexpr (HEAD) {
    for (long long k = (long long)b * 64 + lane; k < tail.words; k += (long long)B * 64) tail.clear[k] = 0;
    if (tail.w_hh_t)
      for (int k = b * 64 + lane; k < H * H; k += B * 64) tail.w_hh_t[(k % H) * H + k / H] = w_hh[k];
    const int n = tail.C * H;
    for (int k0 = lane; k0 < n; k0 += 4 * 64) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = tail.w_out[k0 + 64 * u < n ? k0 + 64 * u : n - 1];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k0 + 64 * u < n) w_out[k0 + 64 * u] = v[u];
    }
    if (lane < tail.C) b_out = tail.b_out[lane];
    if (lane == 0) label = tail.labels[b];
  }
  // the unit whose rows a lane holds and the first of its columns, on even and on odd steps
  const int unit[2] = {C * (R >> 1) + i, C * (R & 1) + i}, col0[2] = {C * (R & 1), C * (R >> 1)};
  float w[2][C], wi[2][N], bias[2];
  // the inputs and the bias enter through the rows of column half A, which also store the states
  bool first[2], exists[2];
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
  float s = (i < C && unit[1] < H) ? h[(size_t)b * H + unit[1]] : 0.f;         // (A B A B)
  // Stores go through a buffer descriptor that ends with the trip's last row: lanes that own no unit
  // carry an offset past its end and store nothing, without a change of the lane mask.
  const unsigned row_bytes = (unsigned)B * (unsigned)H * 4u;
  unsigned voff[2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
    voff[f] = first[f] ? ((unsigned)b * (unsigned)H + (unsigned)unit[f]) * 4u : 0x80000000u;

  // lane i of a row holds the input of step t0 + i, in the rows of that step's column half A (elsewhere its
  // weight is zero, and the input must not be infinite)
  const int from = ((i & 1) ? R < 2 : (R & 1) == 0) ? i : kWaveSteps;
  auto fetch = [&](float (&xs)[N], int buf) {
    lds_barrier();
#pragma unroll
    for (int k = 0; k < N; ++k) xs[k] = ahead[buf][k][from];
  };
  auto step = [&](auto q, const float (&xs)[N]) {
    constexpr int Q = decltype(q)::value, F = Q & 1;
    float in = bias[F];
#pragma unroll
    for (int k = 1; k < N; ++k)
      in = __builtin_fmaf(wi[F][k], __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, xs[k]),
                                                                                      0x150 + Q, 0xf, 0xf, true)), in);
    const float pre = wave_product<Q>(w[F], s, in, wi[F][0], xs[0]);
    s = EXACT && C == 10 ? bppsa_tanh_short(pre) : bppsa_tanh(pre);
    if (!EXACT) s = exists[F] ? s : 0.f;       // a column that does not exist must not carry a NaN
  };

  float xs[N], xn[N];
  fetch(xs, 0);
  int t0 = 0, buf = 1;
  for (; t0 + kWaveSteps <= T; t0 += kWaveSteps) {
    fetch(xn, buf);
    buf ^= 1;
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(h + (size_t)(t0 + 1) * B * H, 0, (int)(kWaveSteps * row_bytes),
                                                        0x00020000);
    settle(xs[0]);
    auto put = [&](auto q) {
      step(q, xs);
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, s), rows, (int)voff[decltype(q)::value & 1],
                                            (int)((unsigned)decltype(q)::value * row_bytes), 0);
    };
    put(Int<0>{}), put(Int<1>{}), put(Int<2>{}), put(Int<3>{}), put(Int<4>{}), put(Int<5>{}), put(Int<6>{}), put(Int<7>{});
    put(Int<8>{}), put(Int<9>{}), put(Int<10>{}), put(Int<11>{}), put(Int<12>{}), put(Int<13>{}), put(Int<14>{});
    put(Int<15>{});
#pragma unroll
    for (int k = 0; k < N; ++k) xs[k] = xn[k];
  }
  if (t0 < T) lds_barrier();                       // the trip that does not exist
  // what is left of a trip: the inputs move down two lanes per pair of steps
  for (int t = t0; t < T; t += 2) {
    settle(xs[0]);
    step(Int<0>{}, xs);
    if (first[0]) h[((size_t)(t + 1) * B + b) * H + unit[0]] = s;
    if (t + 1 < T) {
      step(Int<1>{}, xs);
      if (first[1]) h[((size_t)(t + 2) * B + b) * H + unit[1]] = s;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) xs[k] = __shfl_down(xs[k], 2, 16);
  }
  if constexpr (HEAD) {
    const int n = tail.C, u = unit[T & 1 ? 0 : 1];
    if (i < C && u < H) last[u] = s;
    wave_fence();
    float z = -INFINITY;
    if (lane < n) {
      z = b_out;
#pragma unroll 4
      for (int j = 0; j < H; ++j) z += w_out[lane * H + j] * last[j];
    }
    const float m = bppsa_wave_max(z);
    const float lse = m + logf(bppsa_wave_sum(lane < n ? expf(z - m) : 0.f));
    if (lane < n) dz[lane] = (expf(z - lse) - (lane == label ? 1.f : 0.f)) * (1.0f / (float)B);
    wave_fence();
    if (lane < H) {
      float g = 0.f;
#pragma unroll 4
      for (int k = 0; k < n; ++k) g += dz[k] * w_out[k * H + lane];
      tail.seed[(size_t)b * H + lane] = g;
    }
  }
}

// ---- both cells, H <= 128: a wave per 16 units ---------------------------------------------------
// Row R of a wave holds the columns C R .. C R + C - 1 of the state (C = ceil(H / 4) rounded up to a
// built size) and IX R .. IX R + IX - 1 of the input.  The four rows' sums of the GRU's four values
// (r, z, hidden part of n, input part of n) are reduced together: two swap16 and one swap32 leave
// row 0 with r, row 1 with z, row 2 with the hidden and row 3 with the input part.
constexpr int kBlockSteps = 16;      // steps per trip
constexpr int kBlockMaxI = 40;
constexpr int kBlockMaxWaves = 8 + 2;

template <bool GRU, int C, int IX>
__global__ void __launch_bounds__(64 * kBlockMaxWaves)
forward_block_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                     const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                     const float* __restrict__ b_hh, float* __restrict__ h) {
  constexpr int G = GRU ? 3 : 1;
  constexpr int kState = 128 + 32;                 // rows read up to 16 (32) columns from C R on
  constexpr int kXRow = 4 * IX;
  __shared__ float hs[2][kState];
  __shared__ float xs[2][kBlockSteps * kXRow + 64];
  __shared__ float dump[64];                       // where lanes that own no unit write
  const int b = blockIdx.x, lane = threadIdx.x & 63, R = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nrec = (H + 15) >> 4;                  // waves of the recurrence; then the storer, the loader
  for (int e = threadIdx.x; e < 2 * kState; e += blockDim.x) hs[0][e] = 0.f;
  for (int e = threadIdx.x; e < 2 * (kBlockSteps * kXRow + 64); e += blockDim.x) xs[0][e] = 0.f;
  __syncthreads();
  for (int e = threadIdx.x; e < H; e += blockDim.x) hs[0][e] = h[(size_t)b * H + e];

  if (wave > nrec) {
    // ---- loader: x of 16 steps at a time, element e = step * I + column -----------------------------
    constexpr int kLoads = (kBlockSteps * kXRow + 63) / 64;
    float v[kLoads];
    int dst[kLoads], off[kLoads];
    const int count = kBlockSteps * I;
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int e = lane + 64 * k, q = e / I, c = e - q * I;
      dst[k] = e < count ? q * kXRow + c : kBlockSteps * kXRow + (lane & 15);
      off[k] = e < count ? q : 0x3fffffff;         // step within the trip
    }
    auto fetch = [&](int t0) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k) {
        const int e = lane + 64 * k, q = off[k], c = e - q * I;
        v[k] = (e < count && q < T - t0) ? x[((size_t)(t0 + q) * B + b) * I + c] : 0.f;
      }
    };
    auto put = [&](int buf) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k) xs[buf][dst[k]] = v[k];
    };
    fetch(0);
    put(0);
    __syncthreads();
    int buf = 0;
    for (int t0 = 0; t0 < T; t0 += kBlockSteps) {
      fetch(t0 + kBlockSteps);
      const int n = T - t0 < kBlockSteps ? T - t0 : kBlockSteps;
      for (int q = 0; q < n; ++q) {
        if (q == kBlockSteps - 2) put(buf ^ 1);    // in LDS one barrier before the trip that reads it
        lds_barrier();
      }
      buf ^= 1;
    }
    return;
  }
  if (wave == nrec) {
    // ---- storer: the state of step t, while the recurrence forms step t + 1 -------------------------
    __syncthreads();
    const int j1 = lane + 64;
    float* dst = h + ((size_t)B + b) * H;
    const size_t stride = (size_t)B * H;
    for (int t = 1; t <= T; ++t, dst += stride) {
      lds_barrier();
      if (lane < H) dst[lane] = hs[t & 1][lane];
      if (j1 < H) dst[j1] = hs[t & 1][j1];
    }
    return;
  }

  // ---- recurrence ------------------------------------------------------------------------------
  const int unit = 16 * wave + i;
  const bool live = unit < H;
  float w[G][C], wx[G][IX];
#pragma unroll
  for (int g = 0; g < G; ++g) {
#pragma unroll
    for (int c = 0; c < C; ++c)
      w[g][c] = (live && C * R + c < H) ? w_hh[(size_t)(g * H + unit) * H + C * R + c] : 0.f;
#pragma unroll
    for (int c = 0; c < IX; ++c)
      wx[g][c] = (live && IX * R + c < I) ? w_ih[(size_t)(g * H + unit) * I + IX * R + c] : 0.f;
  }
  // biases enter the sums through row 0
  const bool own = live && R == 0;
  float bi[G], bh[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    bi[g] = (own && b_ih) ? b_ih[g * H + unit] : 0.f;
    bh[g] = (own && b_hh) ? b_hh[g * H + unit] : 0.f;
  }
  __syncthreads();
  float hold = hs[0][unit];
  float* const out0 = own ? &hs[1][unit] : &dump[lane];
  float* const out1 = own ? &hs[0][unit] : &dump[lane];

  // xv holds the input columns of this step; those of the next one (row `xnext`) are requested together
  // with the state, and this step's are multiplied while the state is on its way
  float xv = xs[0][IX * R + i];
  auto step = [&](int from, const float* xnext, float* out) {
    const float s0 = hs[from][C * R + i], s1 = C > 16 ? hs[from][C * R + 16 + i] : 0.f;
    const float xn = xnext[IX * R + i];
    __builtin_amdgcn_sched_barrier(0);
    float y;
    if constexpr (GRU) {
      float acc[3] = {bi[0] + bh[0], bi[1] + bh[1], bh[2]};
      float xa[3] = {acc[0], acc[1], bi[2]};
      add_columns(xa, wx, xv, xv);                 // r and z take the input into the same sum
      acc[0] = xa[0];
      acc[1] = xa[1];
      add_columns(acc, w, s0, s1);
      float r = acc[0], z = acc[1], nh = acc[2], nx = xa[2];
      swap16(r, z);
      swap16(nh, nx);
      float u = r + z, v = nh + nx;                // rows (r z r z) and (nh nx nh nx), two partial sums each
      swap32(u, v);
      const float sum = u + v;                     // rows (r z nh nx)
      const float sg = bppsa_sigmoid(sum);
      float hi = sum, lo = sum;
      swap32(lo, hi);                              // hi: rows (nh nx nh nx)
      float nxa = hi;
      swap16(hi, nxa);                             // hi = nh, nxa = nx in every row
      float rg = sg, zg = sg;
      swap16(rg, zg);                              // rows 0, 1: r and z
      const float n = bppsa_tanh(__builtin_fmaf(rg, hi, nxa));
      y = __builtin_fmaf(zg, hold - n, n);         // (1 - z) n + z h
      hold = y;
    } else {
      float acc[1] = {bi[0] + bh[0]};
      add_columns(acc, wx, xv, xv);
      add_columns(acc, w, s0, s1);
      float p = acc[0];
      swap16(acc[0], p);
      float a = acc[0] + p, a2 = a;
      swap32(a, a2);
      y = bppsa_tanh(a + a2);
    }
    *out = y;
    xv = xn;
    lds_barrier();
  };
  int buf = 0;
  for (int t0 = 0; t0 < T; t0 += kBlockSteps) {
    const int n = T - t0 < kBlockSteps ? T - t0 : kBlockSteps;
    const float* xrow = xs[buf];
    int q = 0;
    for (; q + 2 <= n; q += 2, xrow += 2 * kXRow) {
      step(0, xrow + kXRow, out0);
      step(1, q + 2 < kBlockSteps ? xrow + 2 * kXRow : xs[buf ^ 1], out1);
    }
    if (q < n) step(0, xrow, out0);                // only in the last trip: 16 is even
    buf ^= 1;
  }
}

}  // namespace

// RNN with H <= 32 and I <= 4: wave form; else H <= 128 and I <= 40: block form; BPPSA_EUNSUPPORTED
// beyond (the caller has a kernel for any size).  A tail is taken by the wave form only.  The column counts are rounded up to the next built
// size; columns past H have zero weights.
bppsa_status bppsa_recurrence(int cell, int T, int B, int H, int I, const float* x, const float* w_ih,
                              const float* w_hh, const float* b_ih, const float* b_hh, float* h, hipStream_t s,
                              const bppsa_forward_tail* tail) {
  // the trip's rows must lie within a buffer descriptor's 2 GB
  if (cell == BPPSA_RNN_TANH && H <= 32 && I <= kWaveMaxI && (size_t)B * H * 4 * kWaveSteps < ((size_t)1 << 31)) {
#define BPPSA_WAVE_LAUNCH(C, N, E)                                                                                \
  do {                                                                                                            \
    if (tail) rnn_forward_wave_kernel<C, N, E, true><<<B, 128, 0, s>>>(T, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h, *tail); \
    else rnn_forward_wave_kernel<C, N, E, false><<<B, 128, 0, s>>>(T, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h, {});    \
  } while (0)
#define BPPSA_WAVE_FORM(C)                                                                               \
  do {                                                                                                   \
    if (I == 1 && H == 2 * C) BPPSA_WAVE_LAUNCH(C, 1, true);                                              \
    else if (I == 1) BPPSA_WAVE_LAUNCH(C, 1, false);                                                      \
    else BPPSA_WAVE_LAUNCH(C, kWaveMaxI, false);                                                          \
  } while (0)
    if (H <= 8) BPPSA_WAVE_FORM(4);
    else if (H <= 20) BPPSA_WAVE_FORM(10);
    else BPPSA_WAVE_FORM(16);
#undef BPPSA_WAVE_FORM
#undef BPPSA_WAVE_LAUNCH
    BPPSA_CHECK_LAUNCH();
    return BPPSA_OK;
  }
  if (tail || H > 128 || I > kBlockMaxI) return BPPSA_EUNSUPPORTED;
  const int threads = 64 * (bppsa_ceil_div(H, 16) + 2);
#define BPPSA_BLOCK_FORM(GR, C, X) \
  forward_block_kernel<GR, C, X><<<B, threads, 0, s>>>(T, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h)
#define BPPSA_BLOCK_COLUMNS(GR, C)              \
  do {                                          \
    if (I <= 4) BPPSA_BLOCK_FORM(GR, C, 1);     \
    else if (I <= 12) BPPSA_BLOCK_FORM(GR, C, 3); \
    else if (I <= 20) BPPSA_BLOCK_FORM(GR, C, 5); \
    else if (I <= 32) BPPSA_BLOCK_FORM(GR, C, 8); \
    else BPPSA_BLOCK_FORM(GR, C, 10);           \
  } while (0)
#define BPPSA_BLOCK_SIZES(GR)                   \
  do {                                          \
    if (H <= 20) BPPSA_BLOCK_COLUMNS(GR, 5);    \
    else if (H <= 32) BPPSA_BLOCK_COLUMNS(GR, 8); \
    else if (H <= 64) BPPSA_BLOCK_COLUMNS(GR, 16); \
    else if (H <= 96) BPPSA_BLOCK_COLUMNS(GR, 24); \
    else BPPSA_BLOCK_COLUMNS(GR, 32);           \
  } while (0)
  if (cell == BPPSA_GRU) BPPSA_BLOCK_SIZES(true);
  else BPPSA_BLOCK_SIZES(false);
#undef BPPSA_BLOCK_SIZES
#undef BPPSA_BLOCK_COLUMNS
#undef BPPSA_BLOCK_FORM
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
