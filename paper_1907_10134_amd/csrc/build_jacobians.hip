// bppsa_build_jacobians: materialise Jt[t][b] = (d h[t+1] / d h[t])^T, the
// matrix entries of the scan's input array (Section 3.1, Eq. 5).
//
// RNN (Section 4.1): d h[t+1][j] / d h[t][i] = (1 - h[t+1][j]^2) W_hh[j][i], so
// the transposed Jacobian is W_hh^T with column j scaled by 1 - h[t+1][j]^2.
// The kernels are a pure streaming write (4 H^2 bytes out per 4 H bytes in): a thread owns one piece
// position of the tile, with its weights in registers, and walks over tiles; consecutive lanes write
// consecutive addresses.
#include "bppsa_internal.h"

namespace {

// Any H: pieces of V floats (16 bytes where H is a multiple of four), blockIdx.y tells stretches of 256 pieces apart,
// and where a tile has fewer, a workgroup takes several tiles at once.  Eight tiles per trip: their reads of h
// are issued before the first result is formed.
// 2100 tiles of H = 64 (34 MB): 22 -> 11 us, against weights in LDS and one read of h in front of every store; 16000 of
// H = 100 (640 MB): 245 -> 126 (5.1 TB/s); of H = 33: 36 -> 19; of H = 5: 4.6 -> 4.0.
constexpr int kThreads = 256, kTrip = 8;
template <int V, bool STREAM>
__global__ void __launch_bounds__(kThreads)
rnn_jacobians_kernel(long long tiles, int B, int H, const float* __restrict__ h, const float* __restrict__ w_hh,
                     float* __restrict__ Jt) {
  typedef float piece __attribute__((ext_vector_type(V)));
  typedef float piece_of_h __attribute__((ext_vector_type(V), aligned(4)));      // h may lie at any float
  const int hv = H / V;                            // pieces per row
  const long long pieces = (long long)hv * H;
  const int at_once = pieces < kThreads ? kThreads / (int)pieces : 1;
  const int slot = pieces < kThreads ? (int)threadIdx.x / (int)pieces : 0;
  if (slot >= at_once) return;
  const long long step = (long long)gridDim.x * at_once;
  for (long long p = (long long)blockIdx.y * kThreads + (int)threadIdx.x - slot * pieces; p < pieces;
       p += (long long)gridDim.y * kThreads) {
    const int i = (int)(p / hv), j = (int)(p - (long long)i * hv) * V;
    piece w;
#pragma unroll
    for (int u = 0; u < V; ++u) w[u] = w_hh[(size_t)(j + u) * H + i];
    for (long long m0 = (long long)blockIdx.x * at_once + slot; m0 < tiles; m0 += kTrip * step) {
      piece hv8[kTrip];
#pragma unroll
      for (int u = 0; u < kTrip; ++u) {
        const long long m = m0 + u * step < tiles ? m0 + u * step : m0;
        hv8[u] = *reinterpret_cast<const piece_of_h*>(h + (size_t)(m + B) * H + j);       // h[t+1][b][j..]
      }
#pragma unroll
      for (int u = 0; u < kTrip; ++u) {
        const long long m = m0 + u * step;
        if (m < tiles) {
          piece o;
#pragma unroll
          for (int c = 0; c < V; ++c) o[c] = w[c] * __builtin_fmaf(-hv8[u][c], hv8[u][c], 1.0f);
          piece* dst = reinterpret_cast<piece*>(Jt + (size_t)m * H * H + (size_t)p * V);
          if (STREAM) __builtin_nontemporal_store(o, dst);   // far larger than the caches: do not allocate
          else *dst = o;                                     // small enough to be read back from cache
        }
      }
    }
  }
}

// H = 20 (the paper's RNN size): a tile is 100 pieces of 16 bytes.  A thread keeps one fixed
// piece position (row i, columns j4..j4+3), so its four weights live in registers, and walks
// over tiles: per tile it reads 16 bytes of h, multiplies and issues one 16-byte store.
// 500 of the 512 threads of a workgroup cover five tiles per pass.
constexpr int kH20Threads = 512;
constexpr int kH20TilesPerPass = 5;

typedef float bj_v4f __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(kH20Threads)
rnn_jacobians_h20_kernel(int tiles, int B, const float* __restrict__ h, const float* __restrict__ w_hh,
                         float* __restrict__ Jt) {
  constexpr int H = 20;
  const int tid = threadIdx.x;
  const int slot = tid / 100, p = tid - slot * 100;
  if (slot >= kH20TilesPerPass) return;
  const int i = p / 5, j4 = (p - i * 5) * 4;
  bj_v4f w;
#pragma unroll
  for (int u = 0; u < 4; ++u) w[u] = w_hh[(j4 + u) * H + i];
  const int step = gridDim.x * kH20TilesPerPass;
  // Eight tiles per trip: the eight 16-byte reads of h are issued before the first result is
  // formed, so a thread waits for memory once per eight stores instead of once per store.
  constexpr int kTrip = 8;
  for (int m0 = blockIdx.x * kH20TilesPerPass + slot; m0 < tiles; m0 += kTrip * step) {
    bj_v4f hv[kTrip];
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {
      const int m = m0 + u * step;
      hv[u] = bj_v4f{0.f, 0.f, 0.f, 0.f};
      if (m < tiles) hv[u] = *reinterpret_cast<const bj_v4f*>(h + (size_t)(m + B) * H + j4);   // h[t+1][b][j4..]
    }
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {
      const int m = m0 + u * step;
      if (m < tiles) {
        // 1 - h^2 as one fused multiply-add, spelled out: the fused scan forms the same tile and
        // must get the same bits whatever the compiler would contract
        bj_v4f o;
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = w[c] * __builtin_fmaf(-hv[u][c], hv[u][c], 1.0f);
        *reinterpret_cast<bj_v4f*>(Jt + (size_t)m * H * H + p * 4) = o;
      }
    }
  }
}

// The same for outputs far larger than the caches.  What bounds it is how the memory takes the stores: fastest when
// everything in flight lies close together, so workgroups write whole lines side by side (256 pieces; the stride over
// pieces, 256 x 500, is a multiple of the 100 of a tile, so a thread keeps its position) and 500 workgroups with four
// stores to a wave are in flight at a time.  T = 30000, B = 16 (768 MB): 150 us with the workgroups of five tiles above
// (8000 bytes each, 512 of them, eight stores), 129 like this; 250 to 4000 workgroups with eight stores 130 to 147,
// with one store 171 and more (the reads of h are then waited for), ordinary stores 172 and more.
constexpr int kH20StreamThreads = 256, kH20StreamGroups = 500;

__global__ void __launch_bounds__(kH20StreamThreads)
rnn_jacobians_h20_stream_kernel(unsigned tiles, int B, const float* __restrict__ h, const float* __restrict__ w_hh,
                                float* __restrict__ Jt) {
  constexpr int H = 20, kTrip = 4;
  constexpr unsigned kStep = kH20StreamThreads * kH20StreamGroups / 100;         // tiles
  static_assert(kH20StreamThreads * kH20StreamGroups % 100 == 0, "a thread keeps its place in the tile");
  const unsigned first = blockIdx.x * kH20StreamThreads + threadIdx.x, p = first % 100;
  const int i = (int)p / 5, j4 = ((int)p - i * 5) * 4;
  bj_v4f w;
#pragma unroll
  for (int u = 0; u < 4; ++u) w[u] = w_hh[(j4 + u) * H + i];
  for (unsigned m0 = first / 100; m0 < tiles; m0 += kTrip * kStep) {
    bj_v4f hv[kTrip];
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {
      const unsigned m = m0 + u * kStep < tiles ? m0 + u * kStep : m0;
      hv[u] = *reinterpret_cast<const bj_v4f*>(h + (size_t)(m + B) * H + j4);   // h[t+1][b][j4..]
    }
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {
      const unsigned m = m0 + u * kStep;
      if (m < tiles) {
        bj_v4f o;                                  // the same arithmetic as above
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = w[c] * __builtin_fmaf(-hv[u][c], hv[u][c], 1.0f);
        __builtin_nontemporal_store(o, reinterpret_cast<bj_v4f*>(Jt + (size_t)m * H * H + p * 4));
      }
    }
  }
}

}  // namespace

bppsa_status bppsa_build_jacobians_gru(int T, int B, int H, int I,
                                       const float* h, const float* x,
                                       const float* w_ih, const float* w_hh,
                                       const float* b_ih, const float* b_hh,
                                       float* Jt, hipStream_t stream);

extern "C" bppsa_status bppsa_build_jacobians(int cell, int T, int B, int H, int I,
                                              const float* h, const float* x,
                                              const float* w_ih, const float* w_hh,
                                              const float* b_ih, const float* b_hh,
                                              float* Jt, void* stream) {
  if (!h || !w_hh || !Jt) return BPPSA_EINVAL;
  if (T < 1 || B < 1 || H < 1) return BPPSA_EINVAL;
  if (bppsa_mul_overflows(T, B, H, H)) return BPPSA_EOVERFLOW;
  hipStream_t s = (hipStream_t)stream;
  if (cell == BPPSA_GRU) {
    if (!x || !w_ih || I < 1) return BPPSA_EINVAL;
    return bppsa_build_jacobians_gru(T, B, H, I, h, x, w_ih, w_hh, b_ih, b_hh, Jt, s);
  }
  if (cell != BPPSA_RNN_TANH) return BPPSA_EUNSUPPORTED;

  if (H == 20 && (long long)T * B < 0x7fffffffLL - 65536) {
    const int tiles = T * B;
    int grid = bppsa_ceil_div(tiles, kH20TilesPerPass);
    if (grid > 512) grid = 512;
    if (bppsa_stream_jacobians(T, B, H))
      rnn_jacobians_h20_stream_kernel<<<kH20StreamGroups, kH20StreamThreads, 0, s>>>((unsigned)tiles, B, h, w_hh, Jt);
    else
      rnn_jacobians_h20_kernel<<<grid, kH20Threads, 0, s>>>(tiles, B, h, w_hh, Jt);
    BPPSA_CHECK_LAUNCH();
    return BPPSA_OK;
  }
  const int vec = (H % 4 == 0) ? 4 : 1;
  const long long tiles = (long long)T * B, pieces = (long long)H * H / vec;
  const int at_once = pieces < kThreads ? kThreads / (int)pieces : 1;
  const long long stretches = (pieces + kThreads - 1) / kThreads;
  const int gy = (int)(stretches < 65535 ? stretches : 65535);
  // Up to eight workgroups to a compute unit, with a trip of eight tiles to a thread before there are more than two:
  // a workgroup's weights are gathered across their rows, so fewer of them cost less than the second trip that four
  // tiles to a thread avoid.  2100 tiles of H = 64 12.3 -> 10.5 us, 1000 of H = 80 10.3 -> 8.3, of H = 96 12.8 -> 10.7.
  const long long passes = (tiles + at_once - 1) / at_once;
  const auto share = [&](long long groups) { return groups > gy ? groups / gy : 1; };
  long long gx = passes / 8 > share(512) ? passes / 8 : share(512);
  if (gx > share(2048)) gx = share(2048);
  if (gx > passes) gx = passes;
  const dim3 grid((unsigned)gx, (unsigned)gy);
  const bool stream_out = bppsa_stream_jacobians(T, B, H);
#define BPPSA_JACOBIANS(V, S) rnn_jacobians_kernel<V, S><<<grid, kThreads, 0, s>>>(tiles, B, H, h, w_hh, Jt)
  if (vec == 4 && stream_out) BPPSA_JACOBIANS(4, true);
  else if (vec == 4) BPPSA_JACOBIANS(4, false);
  else if (stream_out) BPPSA_JACOBIANS(1, true);
  else BPPSA_JACOBIANS(1, false);
#undef BPPSA_JACOBIANS
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
