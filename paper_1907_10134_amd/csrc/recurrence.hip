// bppsa_forward for hidden sizes up to 128: the walk over time, of a short sequence in one go and of a long one as
// segments that are walked at the same time and then joined (see Cut).
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
// Two forms, each of one walk, of segments with a launch that joins them, and the first also of rounds (Rounds: fewer
// walks than segments, in one workgroup, for batches that leave a sample no more than its compute unit):
//   rnn_forward_wave_kernel    tanh RNN, H <= 32, at most 4 inputs: one wave per walk, a second one
//                              fetches the inputs; no LDS and no barrier in a step.
//   forward_block_kernel       both cells, H <= 128, at most 40 inputs: a wave per 16 units, the state
//                              through LDS with one barrier per step, and two more waves that do the
//                              memory traffic (inputs fetched 16 steps ahead, states stored), so that no
//                              wave of the recurrence ever waits for memory.
// The inputs are further columns of the product: their weights sit in registers beside the others.
//
// A step takes 0.074 us for the RNN of H = 20 (about 0.015 of it the tanh), 0.22 for H = 64, 0.31 for the GRU of H = 20
// and 0.69 for that of H = 128 (99 multiply-adds of each of two waves per SIMD take two thirds of it).
// Measured (bppsa_forward, one call between two events): the whole sequence in one walk, as it is walked now with
// weights of the usual initialisation, and with weights that do not forget (recurrent weights six times as large: all of
// it is walked again):
//   RNN H = 20, T = 1000, B = 16              80      22      87 us
//   RNN H = 20, T = 1000, B = 256             83      40     105   (rounds)
//   RNN H = 20, T = 30000, B = 16           2228      63    2195
//   RNN H = 64, T = 300, B = 7                69      38      76
//   GRU H = 20, I = 24, T = 517, B = 32      165      55     187
//   GRU H = 128, I = 1, T = 4096, B = 16    2823     259    2887
//   GRU H = 128, I = 12, T = 1034, B = 5     754     106     783
// The launch that joins, with each unit held to its own rounding rather than to 2^-21 of the largest state (2^-20 in the
// block form, its sums there in an order of their own), which let wrong states through: T = 1034 above 99 -> 106,
// the others as before.
// Past 40 inputs bppsa_forward falls back to a kernel that reads every weight from the cache in every step: 500 steps of
// 16 samples take 420 us at I = 40 and 6220 at I = 41 for the GRU of H = 128, 168 and 1836 for H = 20, 106 and 1577
// for the RNN of H = 20.  The RNN's step from the wave to the block form (I = 4 to 5) is 58 to 90 us.
#include "recurrence_wave.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8h __attribute__((ext_vector_type(8)));

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

// ---- tanh RNN, H <= 32: one wave per sample (recurrence_wave.h) ----------------------------------
// HEAD: the classifier's seed dL/dh_T follows in the same launch (a training iteration; on segments, in the second):
// each sample's last state is still in its wave's registers, and a launch of its own takes 6 us.  The workgroups also
// zero the words the next launch wants zeroed.
template <int C, int N, bool EXACT, bool HEAD>
__global__ void __launch_bounds__(128)
rnn_forward_wave_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                        const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                        const float* __restrict__ b_hh, float* __restrict__ h, const bppsa_forward_tail tail) {
  __shared__ float w_out[HEAD ? 64 * 2 * C : 1], last[HEAD ? 2 * C : 1], dz[HEAD ? 64 : 1];
  __shared__ int label;
  __shared__ Ahead<N> ahead;
  const int b = blockIdx.x, lane = threadIdx.x & 63;
  if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 1) return feed_walk<N>(ahead, 0, T, b, B, I, x);
  float b_out = 0.f;
  if constexpr (HEAD) {
    prepare_scan(tail, H, w_hh, b * 64 + lane, B * 64);
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
  const WaveCell<C, N, EXACT> cell(H, I, w_ih, w_hh, b_ih, b_hh);
  const float s = cell.walk(ahead, cell.load_state(h + (size_t)b * H, H), 0, T, 0, b, B, H, h);
  if constexpr (HEAD) {
    const int u = T & 1 ? cell.unit[0] : cell.unit[1];
    if ((lane & 15) < C && u < H) last[u] = s;
    wave_fence();
    head_of_sample(tail, b, B, H, w_out, b_out, label, last, dz);
  }
}

// The first segment takes the steps that the others spend warming up as well: [0, warm + len), then len each.
struct Cut {
  int segs, len, warm;                             // len and warm are multiples of kWaveSteps
  __device__ __forceinline__ int seam(int g) const { return g ? warm + g * len : 0; }       // first step of segment g
  __device__ __forceinline__ int end(int g, int T) const { return min(T, warm + (g + 1) * len); }
  __device__ __forceinline__ int start(int g) const { return g * len; }
};
constexpr int kWaveChains = 4;                     // chains of a workgroup: a walking wave for each SIMD
constexpr int kMaxSegs = 256;
constexpr int kSettleThreads = 1024;
constexpr int kRoundWalks = 4, kFirstWalks = 8;

template <int C, int N, bool EXACT>
__global__ void __launch_bounds__(128 * kWaveChains)
rnn_forward_segments_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                            const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                            const float* __restrict__ b_hh, float* __restrict__ h, const Cut cut) {
  __shared__ Ahead<N> ahead[kWaveChains];
  // waves 0..3 walk, waves 4..7 feed them; barriers wait for the waves that are left
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pair = wave & (kWaveChains - 1);
  const int chain = blockIdx.x * kWaveChains + pair, b = chain % B, seg = chain / B;
  if (seg >= cut.segs) return;
  const int t0 = cut.start(seg), to = cut.end(seg, T);
  if (wave >= kWaveChains) return feed_walk<N>(ahead[pair], t0, to, b, B, I, x);
  const WaveCell<C, N, EXACT> cell(H, I, w_ih, w_hh, b_ih, b_hh);
  const float s0 = seg == 0 ? cell.load_state(h + (size_t)b * H, H) : 0.f;
  cell.walk(ahead[pair], s0, t0, to, cut.seam(seg), b, B, H, h);
}

// A workgroup per sample: the seams are dealt to its waves.  A seam that is broken by itself has the segment behind it
// walked again, otherwise the rest of the sequence is walked in rounds.
template <int C, int N, bool EXACT, bool HEAD>
__global__ void __launch_bounds__(kSettleThreads)
rnn_forward_settle_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                          const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                          const float* __restrict__ b_hh, float* __restrict__ h, const bppsa_forward_tail tail,
                          const Cut cut) {
  constexpr int kAtOnce = 4;
  __shared__ float w_out[HEAD ? 64 * 2 * C : 1], last[HEAD ? 2 * C : 1], dz[HEAD ? 64 : 1];
  __shared__ RoundsLds<N, kRoundWalks> lds;
  __shared__ int broken[kMaxSegs];
  const int b = blockIdx.x, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // all that is read is requested before any of it is waited for
  const WaveCell<C, N, EXACT> cell(H, I, w_ih, w_hh, b_ih, b_hh);
  const Seams<C, N, EXACT> at(cell, x, h, b, B, H, I);
  const float* const h_last = at.hb + (size_t)T * at.row();
  float s[kAtOnce], y[kAtOnce], xs[kAtOnce][N];
  auto load_seams = [&](int g0) {
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int g = g0 + u * waves < cut.segs ? g0 + u * waves : cut.segs - 1, t = cut.seam(g);
      s[u] = at.state(t);
      y[u] = at.stored(t);
      at.inputs(xs[u], t);
    }
  };
  load_seams(1 + wave);
  float b_out = 0.f, end = 0.f, wv = 0.f;
  int label = 0;
  const bool head_wave = HEAD && wave == 0;
  if constexpr (HEAD) {
    if ((int)threadIdx.x < tail.C * H) wv = tail.w_out[threadIdx.x];
    if (head_wave) {
      if (lane < tail.C) b_out = tail.b_out[lane];
      if (lane < H) end = h_last[lane];
      label = tail.labels[b];
    }
    prepare_scan(tail, H, w_hh, b * blockDim.x + threadIdx.x, B * blockDim.x);
  }
  bool bad = false;
  for (int g0 = 1 + wave; g0 < cut.segs; g0 += kAtOnce * waves) {
    if (g0 != 1 + wave) load_seams(g0);
    bool ok[kAtOnce];
    at.hold(ok, s, xs, y);
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int g = g0 + u * waves;
      if (g < cut.segs) {
        bad |= !ok[u];
        if (lane == 0) broken[g] = !ok[u];
      }
    }
  }
  if constexpr (HEAD) {
    if ((int)threadIdx.x < tail.C * H) w_out[threadIdx.x] = wv;
    for (int k = threadIdx.x + blockDim.x; k < tail.C * H; k += blockDim.x) w_out[k] = tail.w_out[k];
    if (head_wave && lane < H) last[lane] = end;
  }
  const bool any = __syncthreads_or(bad);
  if (any) {
    if (wave >= 2 * kRoundWalks) return;
    const Rounds<kRoundWalks, C, N, EXACT> rounds{lds, at, h, T};
    int base = T;                                  // where the rounds begin
    for (int g = 1; g < cut.segs; ++g) {
      if (!broken[g]) continue;
      if (g + 1 < cut.segs && broken[g + 1]) {
        base = cut.seam(g);
        break;
      }
      const int to = rounds.round(cut.seam(g), cut.end(g, T) - cut.seam(g), 0, 1);
      if (to >= T) break;
      if (wave == 0) {                             // whether the next seam holds from the new end
        const bool ok = at.holds(to);
        if (lane == 0) lds.joined[0] = ok;
      }
      __syncthreads();
      const bool ok = lds.joined[0] != 0;
      __syncthreads();
      if (!ok) {
        base = to;
        break;
      }
    }
    // Where hardly a seam holds rounds are longer than one walk: T = 30000, B = 16, a cell that does not forget 2383 us
    // in rounds, 2195 here; from half the seams on, samples that rounds bring back would lose more (an iteration of
    // T = 5000, B = 13 between 357 and 525 us in rounds, 474 in one walk; of T = 2000, B = 30 150 to 258 and 238).
    int count = 0;
    for (int g = 1; g < cut.segs; g += 64)
      count += __popcll(__ballot(g + lane < cut.segs && broken[min(g + lane, cut.segs - 1)] != 0));
    if (base < T && 8 * count >= 7 * (cut.segs - 1)) rounds.round(base, T - base, 0, 1);
    else rounds.run(base);
    if constexpr (HEAD) {
      // (a seam in the middle put right by itself leaves h_T as it was)
      if (head_wave && lane < H) last[lane] = h_last[lane];
    }
  }
  if constexpr (HEAD) {
    if (!head_wave) return;
    wave_fence();
    head_of_sample(tail, b, B, H, w_out, b_out, label, last, dz);
  }
}

// A sequence that eight walks of one workgroup are enough for: one launch, and little lost where the cell does not
// forget.
template <int C, int N, bool EXACT, bool HEAD>
__global__ void __launch_bounds__(128 * kFirstWalks)
rnn_forward_rounds_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                          const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                          const float* __restrict__ b_hh, float* __restrict__ h, const bppsa_forward_tail tail) {
  __shared__ float w_out[HEAD ? 64 * 2 * C : 1], dz[HEAD ? 64 : 1];
  __shared__ RoundsLds<N, kFirstWalks> lds;
  const int b = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const WaveCell<C, N, EXACT> cell(H, I, w_ih, w_hh, b_ih, b_hh, wave < kFirstWalks);
  const Seams<C, N, EXACT> at(cell, x, h, b, B, H, I);
  float b_out = 0.f;
  int label = 0;
  if constexpr (HEAD) {
    for (int k = threadIdx.x; k < tail.C * H; k += 128 * kFirstWalks) w_out[k] = tail.w_out[k];
    if (wave == 0 && lane < tail.C) b_out = tail.b_out[lane];
    if (wave == 0) label = tail.labels[b];
    // by waves that walk no further than the others
    prepare_scan(tail, H, w_hh, b * 128 * kFirstWalks + threadIdx.x, B * 128 * kFirstWalks);
  }
  Rounds<kFirstWalks, C, N, EXACT>{lds, at, h, T}.run(0);
  if constexpr (HEAD) {
    if (wave != 0) return;
    head_of_sample(tail, b, B, H, w_out, b_out, label, lds.last, dz);
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

template <int IX>
struct BlockLds {
  float hs[2][128 + 32];                           // rows of lanes read up to 16 (32) columns from C R on
  float xs[2][kBlockSteps * 4 * IX + 64];
  float dump[64];                                  // where lanes that own no unit write
};

// Columns from .. from + N - 1 of a row of n weights, those that exist.  Every lane reads a row of its own, so what a
// load costs is the 64 lines it touches: in pieces of four where rows start on 16 bytes (GRU, H = 128: the weights
// of a workgroup are there after 6 us, after 22 one by one).
template <int N>
__device__ __forceinline__ void load_columns(float (&w)[N], const float* __restrict__ row, int from, int n, bool live,
                                             const float* base) {
  if (N % 4 == 0 && (n & 3) == 0 && ((uintptr_t)base & 15) == 0) {
#pragma unroll
    for (int c = 0; c + 3 < N; c += 4) {
      v4f v = {0.f, 0.f, 0.f, 0.f};
      if (live && from + c < n) v = *reinterpret_cast<const v4f*>(row + from + c);
      w[c] = v[0], w[c + 1] = v[1], w[c + 2] = v[2], w[c + 3] = v[3];
    }
  } else {
#pragma unroll
    for (int c = 0; c < N; ++c) w[c] = (live && from + c < n) ? row[from + c] : 0.f;
  }
}

// The states after the steps [t0, t1) of sample b, from the stored state before them or from zero, by a whole
// workgroup; rows past `from` and up to `to` are stored.  The last one is left in hs[(t1 - t0) & 1].
template <bool GRU, int C, int IX>
__device__ __forceinline__ void block_walk(BlockLds<IX>& lds, int t0, int t1, bool stored, int from, int to, int b, int B,
                                           int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                                           const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                                           const float* __restrict__ b_hh, float* h) {
  constexpr int G = GRU ? 3 : 1;
  constexpr int kXRow = 4 * IX;
  auto& hs = lds.hs;
  auto& xs = lds.xs;
  auto& dump = lds.dump;
  const int lane = threadIdx.x & 63, R = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nrec = (H + 15) >> 4;                  // waves of the recurrence; then the storer, the loader
  for (int e = threadIdx.x; e < (int)(sizeof(hs) / sizeof(float)); e += blockDim.x) hs[0][e] = 0.f;
  for (int e = threadIdx.x; e < (int)(sizeof(xs) / sizeof(float)); e += blockDim.x) xs[0][e] = 0.f;
  __syncthreads();
  if (stored)
    for (int e = threadIdx.x; e < H; e += blockDim.x) hs[0][e] = h[((size_t)t0 * B + b) * H + e];

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
    auto fetch = [&](int t) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k) {
        const int e = lane + 64 * k, q = off[k], c = e - q * I;
        v[k] = (e < count && q < t1 - t) ? x[((size_t)(t + q) * B + b) * I + c] : 0.f;
      }
    };
    auto put = [&](int buf) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k) xs[buf][dst[k]] = v[k];
    };
    fetch(t0);
    put(0);
    __syncthreads();
    int buf = 0;
    for (int t = t0; t < t1; t += kBlockSteps) {
      fetch(t + kBlockSteps);
      const int n = t1 - t < kBlockSteps ? t1 - t : kBlockSteps;
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
    const size_t stride = (size_t)B * H;
    float* dst = h + (size_t)(t0 + 1) * stride + (size_t)b * H;
    for (int n = 1; n <= t1 - t0; ++n, dst += stride) {
      lds_barrier();
      if (t0 + n <= from || t0 + n > to) continue;
      if (lane < H) dst[lane] = hs[n & 1][lane];
      if (j1 < H) dst[j1] = hs[n & 1][j1];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // whoever goes on from here may read the last row
    return;
  }

  // ---- recurrence ------------------------------------------------------------------------------
  const int unit = 16 * wave + i;
  const bool live = unit < H;
  float w[G][C], wx[G][IX];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    load_columns<C>(w[g], w_hh + (size_t)(g * H + unit) * H, C * R, H, live, w_hh);
    load_columns<IX>(wx[g], w_ih + (size_t)(g * H + unit) * I, IX * R, I, live, w_ih);
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
  for (int t = t0; t < t1; t += kBlockSteps) {
    const int n = t1 - t < kBlockSteps ? t1 - t : kBlockSteps;
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

// (a segment of a longer sequence, or all of it: see Cut)
template <bool GRU, int C, int IX>
__global__ void __launch_bounds__(64 * kBlockMaxWaves)
forward_block_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                     const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                     const float* __restrict__ b_hh, float* __restrict__ h, const Cut cut) {
  __shared__ BlockLds<IX> lds;
  const int b = blockIdx.x % B, seg = blockIdx.x / B, to = cut.end(seg, T);
  block_walk<GRU, C, IX>(lds, cut.start(seg), to, seg == 0, cut.seam(seg), to, b, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h);
}

// ---- the steps across seams, block form ------------------------------------------------------------
// 16 or 32 of them at a time on the matrix cores, since a walking step each would take as long as a segment.  The bits are
// those of the walk: a wave forms 16 units of 16 steps at once with v_mfma_f32_16x16x1_4b_f32, whose four blocks are the four
// rows of the walking wave, one column of each per instruction in the walk's order; a lane supplies the weight that it
// holds in the walk, and gets the four partial sums of four steps of one unit.  (Sums in another order differ from the
// walk's by as much again as two walks do.)
// Two tiles of 16 for each time the weights are loaded, where these take longer than a tile's products (GRU H = 128,
// I = 12, T = 1034, B = 5: forward 107 -> 104 us; H = 20, I = 24, T = 517, B = 32 52.0 -> 54.2, RNN H = 64 36.2 -> 37.4).
template <int C>
constexpr int kSeamTiles = C > 16 ? 2 : 1;
constexpr float kSeamMostBlock = 0x1p-20f;         // for sums of up to 168 terms

// rows of [state | x] in LDS, as the walk pads them; odd, so that 16 rows lie in 16 banks
template <int C, int IX>
constexpr int kSeamStride = 4 * (C + IX) + 1;

// sums of products, and of their magnitudes, for four steps of this lane's unit
struct SeamSums {
  float sum[4], terms[4];
};

// columns [at + N R, at + N R + N) of the staged rows times the weights of a lane (R, unit); of the magnitudes eight
// columns of all four rows at a time, in bf16: a bound need not be exact to more than 2^-8
template <int N>
__device__ __forceinline__ void add_seam_columns(v16f& acc, v4f& mag, const float* row, const float (&w)[N]) {
#pragma unroll
  for (int c0 = 0; c0 < N; c0 += 8) {
    v8h a8, w8;
#pragma unroll
    for (int c = c0; c < c0 + 8; ++c) {
      const float a = c < N ? row[c] : 0.f, b = c < N ? w[c < N ? c : 0] : 0.f;
      if (c < N) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, acc, 0, 0, 0);
      a8[c - c0] = (__bf16)fabsf(a), w8[c - c0] = (__bf16)fabsf(b);
    }
    mag = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8, w8, mag, 0, 0, 0);
  }
}
__device__ __forceinline__ v16f seam_bias(float bias) {        // enters through the walk's row 0
  v16f acc;
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = k < 4 ? bias : 0.f;
  return acc;
}
__device__ __forceinline__ v4f seam_terms(float bias) { return v4f{fabsf(bias), fabsf(bias), fabsf(bias), fabsf(bias)}; }
__device__ __forceinline__ SeamSums seam_sums(const v16f& acc, const v4f& mag) {
  SeamSums s;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    s.sum[v] = (acc[v] + acc[4 + v]) + (acc[8 + v] + acc[12 + v]);
    s.terms[v] = mag[v];
    asm volatile("" : "+v"(s.sum[v]));             // added here, not where they are used: 4 registers for 16
  }
  return s;
}

// The steps from the first `count` staged rows for the 16 units of this wave: emit(row, unit, new state, what its rounding
// may be, in units of kSeam) by every lane whose unit exists.
template <bool GRU, int C, int IX, class F>
__device__ __forceinline__ void seam_steps(int count, int H, int I, const float* __restrict__ w_ih,
                                           const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                                           const float* __restrict__ b_hh, const float* rows, F&& emit) {
  constexpr int kStride = kSeamStride<C, IX>, kTiles = kSeamTiles<C>;
  const int lane = threadIdx.x & 63, R = lane >> 4, i = lane & 15;
  const int unit = 16 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + i;
  const bool live = unit < H;
  const float* const state = rows + i * kStride + C * R;
  const float* const input = rows + i * kStride + 4 * C + IX * R;
  float w[C], wx[IX];
  auto load = [&](int g) {                         // one gate at a time: the registers hold no more
    const float *hh = w_hh, *ih = w_ih;
    asm volatile("" : "+s"(hh), "+s"(ih));         // nor ahead of a loop around
    __builtin_amdgcn_sched_barrier(0);
    load_columns<C>(w, hh + (size_t)(g * H + unit) * H, C * R, H, live, w_hh);
    load_columns<IX>(wx, ih + (size_t)(g * H + unit) * I, IX * R, I, live, w_ih);
  };
  auto bias_ih = [&](int g) { return live && b_ih ? b_ih[g * H + unit] : 0.f; };
  auto bias_hh = [&](int g) { return live && b_hh ? b_hh[g * H + unit] : 0.f; };
  auto sums = [&](SeamSums (&to)[kTiles], float bias, bool of_input, bool of_state) {
#pragma unroll
    for (int k = 0; k < kTiles; ++k) {
      if (16 * k >= count) break;
      v16f acc = seam_bias(bias);
      v4f mag = seam_terms(bias);
      if (of_input) add_seam_columns(acc, mag, input + 16 * k * kStride, wx);
      if (of_state) add_seam_columns(acc, mag, state + 16 * k * kStride, w);
      to[k] = seam_sums(acc, mag);
    }
  };
  load(0);
  if constexpr (GRU) {
    SeamSums r_in[kTiles] = {}, z_in[kTiles] = {}, nx[kTiles] = {}, nh[kTiles] = {};
    sums(r_in, bias_ih(0) + bias_hh(0), true, true);
    load(1);
    sums(z_in, bias_ih(1) + bias_hh(1), true, true);
    load(2);
    sums(nx, bias_ih(2), true, false);
    sums(nh, bias_hh(2), false, true);
    if (!live) return;
#pragma unroll
    for (int k = 0; k < kTiles; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * k + 4 * R + v;
        if (row >= count) break;
        const float r = bppsa_sigmoid(r_in[k].sum[v]), z = bppsa_sigmoid(z_in[k].sum[v]);
        const float n = bppsa_tanh(__builtin_fmaf(r, nh[k].sum[v], nx[k].sum[v]));
        const float off = rows[row * kStride + unit] - n, y = __builtin_fmaf(z, off, n);
        const float of_n = 0.5f * fabsf(n) + (1.f - n * n) * (nx[k].terms[v] + r * nh[k].terms[v] +
                                                              fabsf(nh[k].sum[v]) * r * (1.f - r) * r_in[k].terms[v]);
        const float of_z = z * (0.5f + (1.f - z) * z_in[k].terms[v]);
        emit(row, unit, y, 0.5f * fabsf(y) + (1.f - z) * of_n + fabsf(off) * of_z);
      }
  } else {
    SeamSums in[kTiles] = {};
    sums(in, bias_ih(0) + bias_hh(0), true, true);
    if (!live) return;
#pragma unroll
    for (int k = 0; k < kTiles; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * k + 4 * R + v;
        if (row >= count) break;
        const float y = bppsa_tanh(in[k].sum[v]);
        emit(row, unit, y, 0.5f * fabsf(y) + __builtin_fmaf(-y, y, 1.f) * in[k].terms[v]);
      }
  }
}

// A workgroup per sample, the waves of a walk: the seams, then the segments behind those that do not hold.
template <bool GRU, int C, int IX>
__global__ void __launch_bounds__(64 * kBlockMaxWaves)
forward_block_settle_kernel(int T, int B, int H, int I, const float* __restrict__ x, const float* __restrict__ w_ih,
                            const float* __restrict__ w_hh, const float* __restrict__ b_ih,
                            const float* __restrict__ b_hh, float* __restrict__ h, const Cut cut) {
  constexpr int kAtOnce = 4, kStride = kSeamStride<C, IX>, kSeamRows = 16 * kSeamTiles<C>;
  __shared__ BlockLds<IX> lds;
  __shared__ float rows[kSeamRows * kStride];
  __shared__ float most[kSeamRows];
  __shared__ int broken[kMaxSegs];
  const int b = blockIdx.x, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const size_t row = (size_t)B * H;
  float* const hb = h + (size_t)b * H;
  for (int g = threadIdx.x; g < cut.segs; g += blockDim.x) broken[g] = 0;
  // marks those of `count` seams from g0 on that do not hold; returns whether this thread found one
  auto check = [&](int g0, int count) {
    bool bad = false;
    __syncthreads();
    for (int r0 = wave; r0 < kSeamRows; r0 += kAtOnce * waves) {
      float now[kAtOnce][2], next[kAtOnce][2], in[kAtOnce];
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        const int r = r0 + u * waves, t = cut.seam(g0 + (r < count ? r : 0));
        const float* at = hb + (size_t)t * row;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const bool has = r < count && lane + 64 * k < H;
          now[u][k] = has ? at[lane + 64 * k] : 0.f;
          next[u][k] = has ? at[row + lane + 64 * k] : 0.f;
        }
        in[u] = (r < count && lane < I) ? x[((size_t)t * B + b) * I + lane] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        const int r = r0 + u * waves;
        if (r >= kSeamRows) break;
        float* to = rows + r * kStride;
#pragma unroll
        for (int k = 0; k < 2; ++k)
          if (lane + 64 * k < 4 * C) to[lane + 64 * k] = now[u][k];
        if (lane < 4 * IX) to[4 * C + lane] = in[u];
        const float m = bppsa_wave_max(fmaxf(fabsf(next[u][0]), fabsf(next[u][1])));
        if (lane == 0) most[r] = m;
      }
    }
    __syncthreads();
    if (wave * 16 < H)
      seam_steps<GRU, C, IX>(count, H, I, w_ih, w_hh, b_ih, b_hh, rows, [&](int r, int unit, float y, float own) {
        const float stored = hb[(size_t)(cut.seam(g0 + r) + 1) * row + unit];
        if (!seam_holds(y, stored, own, kSeamMostBlock * most[r])) {
          broken[g0 + r] = 1;
          bad = true;
        }
      });
    return bad;
  };
  bool bad = false, all = true;                    // all: on the way through the seams for the first time
  for (int g0 = 1, g = 1;;) {
    if (g0 < cut.segs) bad |= check(g0, all ? min(kSeamRows, cut.segs - g0) : 1);
    if (all) {
      g0 += kSeamRows;
      if (g0 < cut.segs) continue;
      all = false;
      if (!__syncthreads_or(bad)) return;
    }
    __syncthreads();
    while (g < cut.segs && !broken[g]) ++g;
    if (g >= cut.segs) return;
    int past = g;
    while (past < cut.segs && broken[past]) ++past;
    const int from = cut.seam(g), to = cut.end(past - 1, T);
    block_walk<GRU, C, IX>(lds, from, to, true, from, to, b, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h);
    g = g0 = past;                                 // does the next seam hold from its true state?
  }
}

}  // namespace

// How a sequence is cut for `chains` walks of one sample at a time; one segment: not at all.  Segments are as short as
// fills the chip, but not below 32 steps, where the warm steps are most of the walk.  settle_steps: what the second
// launch costs, in steps; share: the price where a cell does not forget (that launch and the walks for nothing) may be
// this much of one walk.
// warm: steps until a walk from zero was within 2^-21 of the true one, at most over seams of 2000 sets of initial
// weights: H = 20 112 (99.8 % of the sets within 64), H = 32 64, H = 8 a set in a thousand beyond 192; GRU 64.  Segments
// take 96, 128 below H = 16, and 64 for the GRU; rounds 96, and 128 up to H = 8 (kRoundWarm), since a seam that does
// not hold costs them less.
// Training makes a tanh RNN remember: after 4000 to 8000 iterations on one batch of 16 samples (T = 1000, rate 1e-5) 64
// steps leave a sample with a broken seam in most sets of weights, 96 in one of five, and the iteration takes 72 us
// with 64 and 52 with 96.  A large batch always has such a sample, so it is walked in one go.
static Cut cut_of(int T, int chains, int warm, int settle_steps, double share) {
  const Cut whole = {1, T, 0};
  if (chains < 2) return whole;
  if (chains > kMaxSegs) chains = kMaxSegs;
  const int each = bppsa_ceil_div(T, chains), quarter = each / 4 / kWaveSteps * kWaveSteps;
  if (warm < quarter) warm = quarter < 128 ? quarter : 128;          // costs little
  int len = (bppsa_ceil_div(T > warm ? T - warm : 1, chains) + kWaveSteps - 1) / kWaveSteps * kWaveSteps;
  if (len < 2 * kWaveSteps) len = 2 * kWaveSteps;
  if (warm + len + settle_steps > share * T) return whole;
  return Cut{bppsa_ceil_div(T - warm, len), len, warm};
}
// workgroups of a compute unit: as many as there are SIMDs for two walking waves each (H = 128: one)
static Cut block_cut(int cell, int T, int B, int H) {
  const int walking = bppsa_ceil_div(H, 16), at_once = walking >= 8 ? 1 : 8 / walking;
  return cut_of(T, at_once * bppsa_compute_units() / B, cell == BPPSA_GRU ? 64 : H < 16 ? 128 : 96, 24, 0.6);
}
// two walking waves per SIMD (T = 30000, B = 16 takes 46 us with two and 55 with one)
static Cut wave_cut(int T, int B, int H) {
  const int chains = 2 * kWaveChains * bppsa_compute_units() / B;
  return cut_of(T, chains < 32 ? 1 : chains, H < 16 ? 128 : 96, 64, 0.5);
}
// a compute unit for each sample; sequences that rounds shorten (Rounds::rounds_from)
static bool wave_rounds(int T, int B, int H) {
  return T > 3 * (H <= 8 ? 128 : 96) && B <= bppsa_compute_units() && wave_cut(T, B, H).segs == 1;
}

// the trip's rows must lie within a buffer descriptor's 2 GB
static bool wave_form(int B, int H, int I) {
  return H <= 32 && I <= kWaveMaxI && (size_t)B * H * 4 * kWaveSteps < ((size_t)1 << 31);
}
bool bppsa_wave_walks_whole(int T, int B, int H, int I) { return wave_form(B, H, I) && wave_cut(T, B, H).segs == 1; }

// RNN with H <= 32 and I <= 4: wave form; else H <= 128 and I <= 40: block form; BPPSA_EUNSUPPORTED
// beyond (the caller has a kernel for any size).  A tail is taken by the wave form only.  The column counts are rounded up to the next built
// size; columns past H have zero weights.
bppsa_status bppsa_recurrence(int cell, int T, int B, int H, int I, const float* x, const float* w_ih,
                              const float* w_hh, const float* b_ih, const float* b_hh, float* h, hipStream_t s,
                              const bppsa_forward_tail* tail) {
  if (cell == BPPSA_RNN_TANH && wave_form(B, H, I)) {
    const Cut cut = wave_cut(T, B, H);
    const bool rounds = wave_rounds(T, B, H);
#define BPPSA_WAVE_ARGS T, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h
#define BPPSA_WAVE_LAUNCH(C, N, E)                                                                           \
  do {                                                                                                       \
    if (rounds) {                                                                                            \
      if (tail) rnn_forward_rounds_kernel<C, N, E, true><<<B, 128 * kFirstWalks, 0, s>>>(BPPSA_WAVE_ARGS, *tail); \
      else rnn_forward_rounds_kernel<C, N, E, false><<<B, 128 * kFirstWalks, 0, s>>>(BPPSA_WAVE_ARGS, {});   \
    } else if (cut.segs > 1) {                                                                               \
      const int groups = bppsa_ceil_div(B * cut.segs, kWaveChains);                                          \
      rnn_forward_segments_kernel<C, N, E><<<groups, 128 * kWaveChains, 0, s>>>(BPPSA_WAVE_ARGS, cut);       \
      BPPSA_CHECK_LAUNCH();                                                                                  \
      const int threads = cut.segs > 64 ? kSettleThreads : 128 * kRoundWalks;                                \
      if (tail) rnn_forward_settle_kernel<C, N, E, true><<<B, threads, 0, s>>>(BPPSA_WAVE_ARGS, *tail, cut); \
      else rnn_forward_settle_kernel<C, N, E, false><<<B, threads, 0, s>>>(BPPSA_WAVE_ARGS, {}, cut);        \
    } else if (tail) {                                                                                       \
      rnn_forward_wave_kernel<C, N, E, true><<<B, 128, 0, s>>>(BPPSA_WAVE_ARGS, *tail);                      \
    } else {                                                                                                 \
      rnn_forward_wave_kernel<C, N, E, false><<<B, 128, 0, s>>>(BPPSA_WAVE_ARGS, {});                        \
    }                                                                                                        \
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
#undef BPPSA_WAVE_ARGS
    BPPSA_CHECK_LAUNCH();
    return BPPSA_OK;
  }
  if (tail || H > 128 || I > kBlockMaxI) return BPPSA_EUNSUPPORTED;
  const int threads = 64 * (bppsa_ceil_div(H, 16) + 2);
  const Cut cut = block_cut(cell, T, B, H);
#define BPPSA_BLOCK_FORM(GR, C, X)                                                                                 \
  do {                                                                                                             \
    forward_block_kernel<GR, C, X><<<B * cut.segs, threads, 0, s>>>(T, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h, cut); \
    if (cut.segs > 1) {                                                                                            \
      BPPSA_CHECK_LAUNCH();                                                                                        \
      forward_block_settle_kernel<GR, C, X><<<B, threads, 0, s>>>(T, B, H, I, x, w_ih, w_hh, b_ih, b_hh, h, cut); \
    }                                                                                                              \
  } while (0)
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
