// What the parts of a training iteration hand to one another.
#pragma once

#include "bppsa_internal.h"

// What the forward launch of a training iteration does besides the states (see rnn_forward_wave_kernel).
struct bppsa_forward_tail {
  const float* w_out;          // [C][H], C <= 64
  const float* b_out;
  const int32_t* labels;
  float* seed;                 // [B][H], dL/dh_T
  int C;
  int* clear;                  // words to zero for the scan
  long long words;
  float* w_hh_t;               // W_hh transposed for the scan, or null
  float* share;                // each sample's share of the head's gradients, [C][H + 1] (dW_out | db_out), and of the loss,
  int share_stride;            // sample b's at share + b share_stride; or null
};

// bppsa_forward for the sizes the kernels of recurrence.hip take; BPPSA_EUNSUPPORTED for the others.
bppsa_status bppsa_recurrence(int cell, int T, int B, int H, int I, const float* x, const float* w_ih,
                              const float* w_hh, const float* b_ih, const float* b_hh, float* h, hipStream_t s,
                              const bppsa_forward_tail* tail = nullptr);

// Whether bppsa_recurrence walks such a sequence of the tanh RNN in one go, by a wave per sample.
bool bppsa_wave_walks_whole(int T, int B, int H, int I);

// H = 20, sequences that are walked in one go: states, seed and head (tail), gradients G and each sample's share of the
// cell's parameter gradients in one launch: [20][20 + I + 1] (dW_hh | dW_ih | db) at part + b stride.
// T >= 2, I <= 4; `error` receives 0.
inline int bppsa_head_entries(int H, int C) { return C * (H + 1) + 1; }
inline int bppsa_walk_entries(int I, int C) { return 20 * (21 + I) + bppsa_head_entries(20, C); }
bppsa_status bppsa_train_walk_h20(int T, int B, int I, const float* x, const float* w_ih, const float* w_hh,
                                  const float* b_ih, const float* b_hh, float* h, const bppsa_forward_tail& tail, float* G,
                                  int* error, float* part, int stride, hipStream_t s);

// The first half of bppsa_param_grads for the tanh RNN: *nparts partial sums [H][H + I + 1], columns [dW_hh | dW_ih | db].
bppsa_status bppsa_rnn_param_partials(int T, int B, int H, int I, const float* h, const float* x, const float* G,
                                      void* workspace, size_t workspace_bytes, int* nparts, hipStream_t s);

__device__ __forceinline__ float bppsa_wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ float bppsa_wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Adds nparts partials of E elements, `stride` apart, in a fixed order: a workgroup of sixteen waves owns 64 consecutive elements, each
// wave adds every sixteenth partial (consecutive lanes read consecutive addresses, sixteen independent loads in
// flight per thread), and the sixteen sums are added in wave order.  The sum of element first + lane, in wave 0.
constexpr int kFinishWaves = 16;
__device__ __forceinline__ float bppsa_add_partials(int nparts, int E, int stride, int first, const float* __restrict__ part,
                                                    float (&red)[kFinishWaves][64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = first + lane;
  float s = 0.f;
  if (e < E) {
    for (int k0 = wave; k0 < nparts; k0 += 16 * kFinishWaves) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int k = k0 + u * kFinishWaves;
        v[u] = k < nparts ? part[(size_t)k * stride + e] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) s += v[u];
    }
  }
  red[wave][lane] = s;
  __syncthreads();
  float t = 0.f;
  if (wave == 0) {
    t = red[0][lane];
#pragma unroll
    for (int w = 1; w < kFinishWaves; ++w) t += red[w][lane];
  }
  return t;
}
