// The GRU Jacobian stream at H = 128: the gates of 32 rows at a time on the matrix cores (gru_gates.h), then the
// tiles (Appendix E) streamed out with the three recurrent weight matrices held in registers.
#include "gru_gates.h"

namespace {

constexpr int H = 128;

// Jt[i][j] = W_hr[j][i] a_j + W_hn[j][i] c_j + W_hz[j][i] e_j + [i == j] z_j   (Appendix E)
// Persistent workgroups of 512 threads.  Thread (i0 = tid / 32, j4 = 4 (tid % 32)) owns the
// elements (i0 + 16 q, j4 .. j4 + 3), q < 8, of every tile and keeps the matching 3 x 32 weights
// in registers, so a tile costs 16 coefficient reads from LDS, 96 multiply-adds and eight
// 16-byte streaming stores per thread.
__global__ void __launch_bounds__(kGruThreads, 2)
gru_jacobians_h128_kernel(const GruShape s, long long rows, long long tiles, const float* __restrict__ h,
                          const float* __restrict__ x, const GruWeights32 wt, float* __restrict__ Jt) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* As = smem;                        // [32][LA]
  float* coef = smem + kGruRows * s.LA;    // [32][4][H]: a, c, e, z
  const int tid = threadIdx.x;
  const int j4 = (tid & 31) * 4, i0 = tid >> 5;
  v4f wr[8], wn[8], wz[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int i = i0 + 16 * q;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      wr[q][u] = wt.w_hh[(size_t)(j4 + u) * H + i];
      wz[q][u] = wt.w_hh[(size_t)(H + j4 + u) * H + i];
      wn[q][u] = wt.w_hh[(size_t)(2 * H + j4 + u) * H + i];
    }
  }
  GruBias bias = {};
  gru_share<2>(s, [&](int ub, int) { bias = gru_bias(s, wt, 16 * ub + (tid & 15)); });
  for (long long tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const long long row0 = tile * kGruRows;
    const int nrows = (int)((rows - row0 < kGruRows) ? (rows - row0) : kGruRows);
    gru_stage_rows(s, row0, rows, h, x, As);
    __syncthreads();
    gru_share<2>(s, [&](int ub, int sub0) {
      gru_gates<2>(s, wt, bias, ub, sub0, As, x + (size_t)row0 * s.I, nrows, [&](int, int row, int j, float r, float z, float n, float M) {
        const GruCoefs f = gru_coefs_of(r, z, n, M, As[row * s.LA + j]);
        float* c = coef + row * 4 * H + j;
        c[0] = f.a, c[H] = f.c, c[2 * H] = f.e, c[3 * H] = z;
      });
    });
    __syncthreads();
    for (int r = 0; r < nrows; ++r) {
      const float* c = coef + r * 4 * H + j4;
      const v4f ca = *reinterpret_cast<const v4f*>(c);
      const v4f cc = *reinterpret_cast<const v4f*>(c + H);
      const v4f ce = *reinterpret_cast<const v4f*>(c + 2 * H);
      const v4f cz = *reinterpret_cast<const v4f*>(c + 3 * H);
      float* dst = Jt + (size_t)(row0 + r) * H * H + j4;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int i = i0 + 16 * q;
        v4f o = wr[q] * ca + wn[q] * cc + wz[q] * ce;
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] += (i == j4 + u) ? cz[u] : 0.f;
        __builtin_nontemporal_store(o, reinterpret_cast<v4f*>(dst + (size_t)i * H));
      }
    }
    __syncthreads();                   // As and coef are rewritten by the next tile
  }
}

}  // namespace

bppsa_status bppsa_build_jacobians_gru_h128(int T, int B, int I, const float* h, const float* x,
                                            const float* w_ih, const float* w_hh, const float* b_ih,
                                            const float* b_hh, float* Jt, hipStream_t stream) {
  const GruShape s = gru_shape(H, I);
  const long long rows = (long long)T * B;
  const long long tiles = (rows + kGruRows - 1) / kGruRows;
  const int cus = bppsa_compute_units();
  const long long grid = tiles < cus ? tiles : cus;       // one workgroup of 80 KB per compute unit
  const size_t lds = gru_rows_lds(s) + (size_t)kGruRows * 4 * H * sizeof(float);
  if (lds > 160 * 1024) return BPPSA_EUNSUPPORTED;
  BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)gru_jacobians_h128_kernel,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  gru_jacobians_h128_kernel<<<(int)grid, kGruThreads, lds, stream>>>(s, rows, tiles, h, x,
                                                                     GruWeights32{w_ih, w_hh, b_ih, b_hh}, Jt);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
