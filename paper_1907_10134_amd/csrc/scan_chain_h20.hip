// The launches of the serial chain at H = 20, and when it is the cheaper form.
#include "chain_h20.h"
#include "scan_plan.h"

namespace {

template <bool GEN, bool STREAM>
__global__ void __launch_bounds__(chain_h20::kThreads)
chain_h20_kernel(int T, int B, int n, const float* __restrict__ Jt, const float* __restrict__ h,
                 const float* __restrict__ w_hh, const float* __restrict__ seed, float* __restrict__ G,
                 float* __restrict__ g0, int* __restrict__ error) {
  __shared__ chain_h20::Lds lds;
  chain_h20::Weights weights;
  if (GEN) weights.load(w_hh);
  const int b = blockIdx.x;
  chain_h20::walk<GEN, false, STREAM>(lds, weights, T, B, n, b, Jt, h, seed + (size_t)b * chain_h20::H, G, g0, error, {});
}

}  // namespace

bppsa_status bppsa_chain_h20(int T, int B, const float* Jt, const float* seed, float* G, float* g0, int* error,
                             hipStream_t stream, const float* h, const float* w_hh) {
  const int n = g0 ? T : T - 1;
  if (n < 1) return BPPSA_EINVAL;
  using namespace chain_h20;
  if (Jt && bppsa_stream_jacobians(T, B, H))
    chain_h20_kernel<false, true><<<B, kThreads, 0, stream>>>(T, B, n, Jt, nullptr, nullptr, seed, G, g0, error);
  else if (Jt)
    chain_h20_kernel<false, false><<<B, kThreads, 0, stream>>>(T, B, n, Jt, nullptr, nullptr, seed, G, g0, error);
  else chain_h20_kernel<true, false><<<B, kThreads, 0, stream>>>(T, B, n, nullptr, h, w_hh, seed, G, g0, error);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

// What the two forms take, in us, fitted to both sources over T = 10 .. 3000, B = 1 .. 256: the chain 0.055 a step
// (one compute unit per sample, so batches beyond the device's units take turns) and 4 for the launch; the tree 12.5
// for its two launches and one unit, then 0.5 per thousand tiles, with the device filled.
//   T = 100,  B = 16:  9.1 against 14.6         T = 1000, B = 16:   58 against 21 (so the tree)
//   T = 1000, B = 256: 63 generated, 84 stored (tiles at 4.9 TB/s), against 124 and 139
bool bppsa_prefer_chain_h20(int n, int B) {
  const double turns = bppsa_ceil_div(B, bppsa_compute_units());
  return 4.0 + 0.055 * n * turns < 12.5 + 0.0005 * n * B;
}
