// The walks of a training iteration at H = 20 in one launch, for sequences short enough to be walked in one go both
// ways: a workgroup per sample goes through the states, the classifier's seed, the gradients and the sample's share of
// all parameter gradients.  Short iterations are made of launches (about 2 us before the first load comes back and as
// much between one and the next), and what one phase leaves for the next lies in this compute unit's own caches.
// T = 10, B = 16: 15.6 us in the forward, scan and gradient launches and as long as two launches between them, 13.1
// here (the iteration 21.0 -> 15.1); T = 1000, B = 256: 158 and 103.
#include "chain_h20.h"
#include "recurrence_wave.h"
#include "scan_plan.h"

namespace {

constexpr int H = 20;
constexpr int kWalks = chain_h20::kParamThreads / 128;

template <int N, bool EXACT>
__global__ void __launch_bounds__(chain_h20::kParamThreads)
train_walk_h20_kernel(int T, int B, const float* __restrict__ w_ih, const float* __restrict__ w_hh,
                      const float* __restrict__ b_ih, const float* __restrict__ b_hh, float* h,
                      const bppsa_forward_tail tail, float* __restrict__ G, float* __restrict__ g0,
                      int* __restrict__ error, const chain_h20::ParamSums params) {
  __shared__ chain_h20::Lds lds;
  __shared__ RoundsLds<N, kWalks> rounds;
  __shared__ float w_out[64 * H], dz[64], seed[H];
  const int b = blockIdx.x, lane = threadIdx.x & 63, I = params.I;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  chain_h20::Weights weights;
  weights.load(w_hh);
  for (int k = threadIdx.x; k < tail.C * H; k += chain_h20::kParamThreads) w_out[k] = tail.w_out[k];
  {
    const WaveCell<10, N, EXACT> cell(H, I, w_ih, w_hh, b_ih, b_hh, wave < Rounds<kWalks, 10, N, EXACT>::walking(T));
    const Seams<10, N, EXACT> at(cell, params.x, h, b, B, H, I);
    const float b_out = wave == 0 && lane < tail.C ? tail.b_out[lane] : 0.f;
    const int label = wave == 0 ? tail.labels[b] : 0;
    Rounds<kWalks, 10, N, EXACT>{rounds, at, h, T}.run(0);
    if (wave == 0) {
      const float g = head_of_sample(tail, b, B, H, w_out, b_out, label, rounds.last, dz);
      if (lane < H) seed[lane] = g;
    }
  }
  __syncthreads();
  chain_h20::walk<true, true>(lds, weights, T, B, T - 1, b, nullptr, h, seed, G, g0, error, params);   // no g0: T - 1 elements
}

}  // namespace

bppsa_status bppsa_train_walk_h20(int T, int B, int I, const float* x, const float* w_ih, const float* w_hh,
                                  const float* b_ih, const float* b_hh, float* h, const bppsa_forward_tail& tail, float* G,
                                  int* error, float* part, int stride, hipStream_t s) {
  if (T < 2 || I < 1 || I > kWaveMaxI || I > chain_h20::kMaxI) return BPPSA_EUNSUPPORTED;
  const chain_h20::ParamSums params = {x, I, part, stride};
  // (the cell as bppsa_forward instantiates it: the same bits where a sequence is walked in one go.  From
  // Rounds::rounds_from on it is cut for four walks here, for eight there, and differs by rounding behind the seams.)
  if (I == 1)
    train_walk_h20_kernel<1, true><<<B, chain_h20::kParamThreads, 0, s>>>(T, B, w_ih, w_hh, b_ih, b_hh, h, tail, G, nullptr, error, params);
  else
    train_walk_h20_kernel<kWaveMaxI, false><<<B, chain_h20::kParamThreads, 0, s>>>(T, B, w_ih, w_hh, b_ih, b_hh, h, tail, G, nullptr, error, params);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
