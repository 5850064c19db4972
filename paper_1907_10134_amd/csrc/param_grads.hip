// bppsa_param_grads: Eq. 2 of Section 2.1 summed over the time steps that share
// the parameters.  Once dL/dh[t] is known for every t the terms are independent,
// so the sum is one tall-skinny contraction over the T*B (step, sample) rows:
//     [dW_hh | dW_ih | db] = sum_rows  delta_row (x) [h_prev_row | x_row | 1],
// with delta[t] = (1 - h[t]^2) o dL/dh[t] for the tanh RNN (Section 4.1).
// It reads each of G, h and x once (HBM bound).  Blocks reduce disjoint row
// ranges into fp32 partials; a second kernel adds the partials in a fixed order.
#include "train_parts.h"

namespace {

typedef float pg_v4f __attribute__((ext_vector_type(4)));

constexpr int kTileRows = 32;
constexpr int kMaxBlocks = 1024;

// Any size: the H x W output, W = H + I + 1, is cut into tiles of 16 x 16 dealt to eight waves, K of them to each,
// and v_mfma_f32_16x16x4 contracts four of the 32 staged rows at a time.  The rows lie in LDS as in memory, strides
// ld and lu an odd multiple of 16 so that the four rows of an operand fall on different banks.  A thread holds up to
// kLoads elements of the next 32 rows of h_t, h_{t-1} and G while the current ones are multiplied.
// 2100 rows of H = 64: 36 -> 8 us, against one thread per output entry and scalar reads of LDS; 16000 of
// H = 100: 113 -> 14; of H = 33: 19 -> 6; of H = 8: 5.2, as before.
constexpr int kWaves = 8, kThreads = 64 * kWaves, kMaxTiles = 12;
constexpr int kMaxE = 16384;                       // entries of the output, which also keeps H below 128
constexpr int kLoads = kTileRows * 127 / kThreads + 1;

template <int K>
__global__ void __launch_bounds__(kThreads)
rnn_param_partials_kernel(long long rows, int B, int H, int I, int rows_per_block, int ld, int lu,
                          const float* __restrict__ h, const float* __restrict__ x,
                          const float* __restrict__ G, float* __restrict__ part) {
  extern __shared__ float smem[];
  const int W = H + I + 1;             // columns of the right-hand rows [h_prev | x | 1]
  float* D = smem;                     // [kTileRows][ld]   delta
  float* U = smem + kTileRows * ld;    // [kTileRows][lu]
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nu = (H + 15) >> 4, tiles = nu * ((W + 15) >> 4);
  const long long r_begin = (long long)blockIdx.x * rows_per_block;
  long long r_end = r_begin + rows_per_block;
  if (r_end > rows) r_end = rows;
  const float* hcur = h + (size_t)B * H;   // row r of hcur is h[t][b], r = (t-1)*B + b
  pg_v4f acc[K];
  int aoff[K], boff[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int t = wave + kWaves * k < tiles ? wave + kWaves * k : 0;
    acc[k] = pg_v4f{0.f, 0.f, 0.f, 0.f};
    aoff[k] = q * ld + 16 * (t % nu) + l16;
    boff[k] = q * lu + 16 * (t / nu) + l16;
  }
  // element tid + k kThreads of 32 rows, and where it goes; what lies behind H and W in the rows feeds entries
  // that are not stored
  const int loads = (kTileRows * H + kThreads - 1) / kThreads;
  int dto[kLoads], uto[kLoads];
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    const int e = tid + k * kThreads, rr = e / H, c = e - rr * H;
    dto[k] = rr * ld + c;
    uto[k] = rr * lu + c;
  }
  const int xr = tid / I, xto = xr * lu + H + tid - xr * I;
  for (int rr = tid; rr < kTileRows; rr += kThreads) U[rr * lu + H + I] = 1.f;
  float hc[kLoads], hp[kLoads], gv[kLoads], xv = 0.f;
  auto fetch = [&](long long r0) {                 // elements past the end repeat the last one and are not used
    const long long left = r_end - r0;
    const int live = (int)(left < kTileRows ? left : kTileRows);
    const size_t base = (size_t)r0 * H;
#pragma unroll
    for (int k = 0; k < kLoads; ++k)
      if (k < loads) {
        const int e = tid + k * kThreads < live * H ? tid + k * kThreads : live * H - 1;
        hc[k] = hcur[base + e];
        gv[k] = G[base + e];
        hp[k] = h[base + e];
      }
    xv = x[(size_t)r0 * I + (tid < live * I ? tid : live * I - 1)];
  };
  if (r_begin < r_end) fetch(r_begin);
  for (long long r0 = r_begin; r0 < r_end; r0 += kTileRows) {
    const int nr = (int)((r_end - r0 < kTileRows) ? (r_end - r0) : kTileRows);
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int e = tid + k * kThreads;
      if (e < kTileRows * H) {
        D[dto[k]] = e < nr * H ? (1.0f - hc[k] * hc[k]) * gv[k] : 0.f;
        U[uto[k]] = e < nr * H ? hp[k] : 0.f;
      }
    }
    if (tid < kTileRows * I) U[xto] = tid < nr * I ? xv : 0.f;
    for (int e = tid + kThreads; e < kTileRows * I; e += kThreads) {     // more than 16 inputs
      const int rr = e / I, c = e - rr * I;
      U[rr * lu + H + c] = rr < nr ? x[(size_t)(r0 + rr) * I + c] : 0.f;
    }
    __syncthreads();
    if (r0 + kTileRows < r_end) fetch(r0 + kTileRows);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (wave + kWaves * k < tiles) {             // uniform
#pragma unroll
        for (int s = 0; s < kTileRows / 4; ++s)
          acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(D[aoff[k] + 4 * s * ld], U[boff[k] + 4 * s * lu], acc[k], 0, 0, 0);
      }
    __syncthreads();
  }
  float* dst = part + (size_t)blockIdx.x * H * W;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int t = wave + kWaves * k;
    if (t >= tiles) continue;
    const int c = 16 * (t / nu) + l16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * (t % nu) + 4 * q + v;
      if (i < H && c < W) dst[(size_t)i * W + c] = acc[k][v];
    }
  }
}

// H = 20 (the paper's RNN size), up to 3 inputs: the same contraction on the matrix cores.
// The 20 x W output (W = 20 + I + 1 <= 24) is 5 x 6 blocks of 4 x 4; v_mfma_f32_4x4x1 handles 16
// blocks per issue, so two issues per (step, sample) row accumulate all of it:
// D_blk[i][j] += delta[row][4 I + i] * u[row][4 J + j], lane (blk, idx) supplying both operands
// from a tile staged in LDS.  Each wave takes every fifth row of a tile and keeps its own
// accumulators; the five waves' sums are added in a fixed order at the end.
// A tile is one 16-byte piece of h_t, h_{t-1} and G for each of 320 threads.  The pieces of the next tile are
// requested before the current one is multiplied and there are two tiles in LDS, so a tile costs one barrier and
// its memory latency is hidden.  480000 rows: 33.8 -> 23.9 us (79 MB, 3.3 TB/s), 256000: 18.1 -> 13.6 us, against
// four waves, one tile and the loads in front of every tile.
constexpr int kMfmaRows = 64;     // rows per staged tile
constexpr int kUW = 24;           // padded width of [h_prev | x | 1 | 0]
constexpr int kMfmaWaves = 5, kMfmaThreads = 64 * kMfmaWaves;
static_assert(kMfmaThreads == kMfmaRows * 5, "one piece per thread");

__global__ void __launch_bounds__(kMfmaThreads)
rnn_param_partials_h20_kernel(long long rows, int B, int I, int rows_per_block,
                              const float* __restrict__ h, const float* __restrict__ x,
                              const float* __restrict__ G, float* __restrict__ part) {
  constexpr int H = 20;
  __shared__ __attribute__((aligned(16))) float D[2][kMfmaRows * H];
  __shared__ __attribute__((aligned(16))) float U[2][kMfmaRows * kUW];
  __shared__ float red[kMfmaWaves][H * kUW];
  const int W = H + I + 1;
  const int tid = threadIdx.x, lane = tid & 63, blk = lane >> 2, idx = lane & 3;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long r_begin = (long long)blockIdx.x * rows_per_block;
  long long r_end = r_begin + rows_per_block;
  if (r_end > rows) r_end = rows;
  const float* hcur = h + (size_t)B * H;          // row r of hcur is h[t][b], r = (t-1)*B + b
  // operand offsets of this lane for the two issues (block ids blk and 16 + blk; ids 30, 31 idle)
  int aoff[2], boff[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    int id = 16 * n + blk;
    id = id < 30 ? id : 29;
    aoff[n] = 4 * (id / 6) + idx;
    boff[n] = 4 * (id % 6) + idx;
  }
  // this thread's piece of a tile, and its element of [x | 1 | 0]
  const int pr = tid / 5, pc = (tid - 5 * pr) * 4, xr = tid >> 2, xc = tid & 3;
  pg_v4f hc, hp, gv;
  float xv = 0.f;
  auto fetch = [&](long long r0) {                // rows past the end repeat the last one and are not used
    const long long rp = r0 + pr < r_end ? r0 + pr : r_end - 1;
    const size_t g = (size_t)rp * H + pc;
    hc = *reinterpret_cast<const pg_v4f*>(hcur + g);
    gv = *reinterpret_cast<const pg_v4f*>(G + g);
    hp = *reinterpret_cast<const pg_v4f*>(h + g);
    const long long rx = r0 + xr < r_end ? r0 + xr : r_end - 1;
    if (tid < 4 * kMfmaRows) xv = xc < I ? x[(size_t)rx * I + xc] : xc == I ? 1.f : 0.f;
  };
  auto put = [&](long long r0, float* d, float* u) {
    const bool live = r0 + pr < r_end;
    const pg_v4f zero = {0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<pg_v4f*>(d + pr * H + pc) = live ? (1.0f - hc * hc) * gv : zero;
    *reinterpret_cast<pg_v4f*>(u + pr * kUW + pc) = live ? hp : zero;
    if (tid < 4 * kMfmaRows) u[xr * kUW + H + xc] = r0 + xr < r_end ? xv : 0.f;
  };
  pg_v4f acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  if (r_begin < r_end) fetch(r_begin);
  int buf = 0;
  for (long long r0 = r_begin; r0 < r_end; r0 += kMfmaRows, buf ^= 1) {
    put(r0, D[buf], U[buf]);
    __syncthreads();
    if (r0 + kMfmaRows < r_end) fetch(r0 + kMfmaRows);
    const float *d = D[buf], *u = U[buf];
#pragma unroll
    for (int k = 0; k < (kMfmaRows + kMfmaWaves - 1) / kMfmaWaves; ++k) {
      const int rr = wave + k * kMfmaWaves;
      if (rr < kMfmaRows) {                       // uniform; false in the last trip of the last wave only
        const float a0 = d[rr * H + aoff[0]], b0 = u[rr * kUW + boff[0]];
        const float a1 = d[rr * H + aoff[1]], b1 = u[rr * kUW + boff[1]];
        acc[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a0, b0, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a1, b1, acc[1], 0, 0, 0);
      }
    }
  }
  // accumulator register v of lane (blk, idx) is element (4 I + v, 4 J + idx) of its block
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int id = 16 * n + blk;
    if (id < 30) {
      const int bi = id / 6, bj = id % 6;
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][(4 * bi + v) * kUW + 4 * bj + idx] = acc[n][v];
    }
  }
  __syncthreads();
  float* dst = part + (size_t)blockIdx.x * H * W;
  for (int e = tid; e < H * W; e += kMfmaThreads) {
    const int i = e / W, c = e - i * W;
    const int o = i * kUW + c;
    dst[e] = ((red[0][o] + red[1][o]) + (red[2][o] + red[3][o])) + red[4][o];
  }
}

// Adds the per-block partials in a fixed order (deterministic).
__global__ void __launch_bounds__(64 * kFinishWaves)
rnn_param_finish_kernel(int nblocks, int H, int I, const float* __restrict__ part,
                        float* __restrict__ dW_ih, float* __restrict__ dW_hh,
                        float* __restrict__ db_ih, float* __restrict__ db_hh) {
  __shared__ float red[kFinishWaves][64];
  const int W = H + I + 1;
  const int E = H * W, e = blockIdx.x * 64 + (int)(threadIdx.x & 63);
  const float t = bppsa_add_partials(nblocks, E, E, blockIdx.x * 64, part, red);
  if (threadIdx.x >= 64 || e >= E) return;
  const int i = e / W, c = e - i * W;
  if (c < H) dW_hh[(size_t)i * H + c] = t;
  else if (c < H + I) dW_ih[(size_t)i * I + (c - H)] = t;
  else {
    db_ih[i] = t;
    if (db_hh) db_hh[i] = t;
  }
}

int rnn_blocks(long long rows) {
  long long nb = (rows + 2 * kTileRows - 1) / (2 * kTileRows);
  if (nb > kMaxBlocks) nb = kMaxBlocks;
  return (int)nb;
}

}  // namespace

bppsa_status bppsa_rnn_param_partials(int T, int B, int H, int I, const float* h, const float* x, const float* G,
                                      void* workspace, size_t workspace_bytes, int* nparts, hipStream_t s) {
  const int W = H + I + 1;
  const int E = H * W;
  if (E > kMaxE) return BPPSA_EUNSUPPORTED;
  if ((size_t)kTileRows * (H + W) * sizeof(float) > 64 * 1024) return BPPSA_EUNSUPPORTED;
  const long long rows = (long long)T * B;
  const int nb = rnn_blocks(rows);
  const size_t need = bppsa_align_up((size_t)nb * E * sizeof(float), 256);
  if (!workspace || workspace_bytes < need) return BPPSA_EWORKSPACE;
  float* part = static_cast<float*>(workspace);
  long long rpb = (rows + nb - 1) / nb;
  if (H == 20 && I <= 3) {
    rpb = (rpb + kMfmaRows - 1) / kMfmaRows * kMfmaRows;
    rnn_param_partials_h20_kernel<<<nb, kMfmaThreads, 0, s>>>(rows, B, I, (int)rpb, h, x, G, part);
  } else {
    rpb = (rpb + kTileRows - 1) / kTileRows * kTileRows;
    auto stride = [](int n) { return (bppsa_ceil_div(n, 16) | 1) * 16; };
    const int ld = stride(H), lu = stride(W), tiles = bppsa_ceil_div(H, 16) * bppsa_ceil_div(W, 16);
    const size_t lds = (size_t)kTileRows * (ld + lu) * sizeof(float);
    // H + W <= 512 and H W <= 16384 leave at most 90 tiles (H = 33, W = 479)
    if (tiles > kWaves * kMaxTiles) return BPPSA_EUNSUPPORTED;
#define BPPSA_LAUNCH_PARTIALS(K)                                                                                   \
  do {                                                                                                             \
    if (lds > 48 * 1024)                                                                                           \
      BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)rnn_param_partials_kernel<K>,                                 \
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));                   \
    rnn_param_partials_kernel<K><<<nb, kThreads, lds, s>>>(rows, B, H, I, (int)rpb, ld, lu, h, x, G, part);        \
  } while (0)
    if (tiles <= kWaves) BPPSA_LAUNCH_PARTIALS(1);
    else if (tiles <= 3 * kWaves) BPPSA_LAUNCH_PARTIALS(3);
    else if (tiles <= 6 * kWaves) BPPSA_LAUNCH_PARTIALS(6);
    else BPPSA_LAUNCH_PARTIALS(kMaxTiles);
#undef BPPSA_LAUNCH_PARTIALS
  }
  BPPSA_CHECK_LAUNCH();
  *nparts = nb;
  return BPPSA_OK;
}

size_t bppsa_param_grads_gru_ws(int T, int B, int H, int I);
bppsa_status bppsa_param_grads_gru(int T, int B, int H, int I,
                                   const float* h, const float* x, const float* G,
                                   const float* w_ih, const float* w_hh,
                                   const float* b_ih, const float* b_hh,
                                   float* dW_ih, float* dW_hh, float* db_ih, float* db_hh,
                                   void* workspace, size_t workspace_bytes, hipStream_t stream);

extern "C" size_t bppsa_param_grads_workspace_bytes(int cell, int T, int B, int H, int I) {
  if (T < 1 || B < 1 || H < 1 || I < 1) return 0;
  if (cell == BPPSA_GRU) return bppsa_param_grads_gru_ws(T, B, H, I);
  if (cell != BPPSA_RNN_TANH) return 0;
  const long long rows = (long long)T * B;
  return bppsa_align_up((size_t)rnn_blocks(rows) * H * (H + I + 1) * sizeof(float), 256);
}

extern "C" bppsa_status bppsa_param_grads(int cell, int T, int B, int H, int I,
                                          const float* h, const float* x, const float* G,
                                          const float* w_ih, const float* w_hh,
                                          const float* b_ih, const float* b_hh,
                                          float* dW_ih, float* dW_hh,
                                          float* db_ih, float* db_hh,
                                          void* workspace, size_t workspace_bytes,
                                          void* stream) {
  if (T < 1 || B < 1 || H < 1 || I < 1) return BPPSA_EINVAL;
  if (!h || !x || !G || !dW_ih || !dW_hh || !db_ih) return BPPSA_EINVAL;
  if (bppsa_mul_overflows((int64_t)T + 1, B, H, 1) || bppsa_mul_overflows(T, B, I, 1))
    return BPPSA_EOVERFLOW;
  hipStream_t s = (hipStream_t)stream;
  if (cell == BPPSA_GRU) {
    if (!w_ih || !w_hh || !db_hh) return BPPSA_EINVAL;
    return bppsa_param_grads_gru(T, B, H, I, h, x, G, w_ih, w_hh, b_ih, b_hh,
                                 dW_ih, dW_hh, db_ih, db_hh, workspace, workspace_bytes, s);
  }
  if (cell != BPPSA_RNN_TANH) return BPPSA_EUNSUPPORTED;
  int nb = 0;
  BPPSA_TRY(bppsa_rnn_param_partials(T, B, H, I, h, x, G, workspace, workspace_bytes, &nb, s));
  // blocks past the last row range wrote zeros, so summing all nb partials is exact
  rnn_param_finish_kernel<<<bppsa_ceil_div(H * (H + I + 1), 64), 64 * kFinishWaves, 0, s>>>(
      nb, H, I, static_cast<const float*>(workspace), dW_ih, dW_hh, db_ih, db_hh);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
