// The GRU Jacobian stream at H = 128: the gates of 32 rows at a time on the matrix cores (gru_gates.h), then the
// tiles (Appendix E) streamed out with the three recurrent weight matrices held in registers.
#include "gru_gates.h"

namespace {

constexpr int H = 128;

// Jt[i][j] = W_hr[j][i] a_j + W_hn[j][i] c_j + W_hz[j][i] e_j + [i == j] z_j   (Appendix E)
// Persistent workgroups of 512 threads.  Thread (i0 = tid / 32, j4 = 4 (tid % 32)) owns the
// elements (i0 + 16 q, j4 .. j4 + 3), q < 8, of every tile and keeps the matching 3 x 32 weights
// in registers, so a tile costs 16 coefficient reads from LDS, 96 multiply-adds and eight
// 16-byte stores per thread.
// Bound by the stores.  The 32 rows that a workgroup takes at a time lie gridDim.x apart, so that all workgroups write
// near one another, and the stores are ordinary ones: 4.3 GB written in 777 us as streaming stores with a stretch of
// 32 rows to each workgroup, in 740 like this, without the arithmetic.  With TWICE the coefficients have two buffers,
// and the rows of one set are stored between the products that give the gates of the next, 8 us a set; without (inputs
// too wide for the second buffer) after them, all at once, and then with streaming stores where there is much to write
// (I = 250, 1034 x 5 rows 339 MB 95.5 -> 94 us, 8000 rows 524 MB 135 -> 130, 16000 253 -> 236, 32000 489 -> 424).
// T = 4096, B = 16: 843 -> 772 us; T = 1034, B = 5 (339 MB): 97 -> 80; 60 rows, which two workgroups had before: 51 -> 21.5.
template <bool TWICE, bool STREAM>
__global__ void __launch_bounds__(kGruThreads, 2)
gru_jacobians_h128_kernel(const GruShape s, long long rows, const float* __restrict__ h,
                          const float* __restrict__ x, const GruWeights32 wt, float* __restrict__ Jt) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* As = smem;                        // [32][LA]
  float* coef = smem + kGruRows * s.LA;    // [32][4][H]: a, c, e, z; one buffer, or two
  const int tid = threadIdx.x, apart = gridDim.x;
  const int j4 = (tid & 31) * 4, i0 = tid >> 5;
  // The weights come through LDS: gathered across their rows, 32 lines to a request, they take 15 us
  // longer.
  v4f wr[8], wn[8], wz[8];
  auto weights = [&](v4f (&w)[8], int gate) {
    constexpr int kRow = H + 1;
#pragma unroll
    for (int k = 0; k < H * H / kGruThreads; ++k) {
      const int e = tid + kGruThreads * k;
      smem[(e / H) * kRow + e % H] = wt.w_hh[(size_t)gate * H * H + e];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int u = 0; u < 4; ++u) w[q][u] = smem[(j4 + u) * kRow + i0 + 16 * q];
    __syncthreads();
  };
  weights(wr, 0);
  weights(wz, 1);
  weights(wn, 2);
  GruBias bias = {};
  gru_share<2>(s, [&](int ub, int) { bias = gru_bias(s, wt, 16 * ub + (tid & 15)); });
  // rows first, first + apart, ... below `rows`, 32 at most
  auto rows_of = [&](long long first) {
    const long long left = first < rows ? (rows - first + apart - 1) / apart : 0;
    return (int)(left < kGruRows ? left : kGruRows);
  };
  auto store_row = [&](const float* buf, long long first, int r) {
    const float* c = buf + r * 4 * H + j4;
    const v4f ca = *reinterpret_cast<const v4f*>(c);
    const v4f cc = *reinterpret_cast<const v4f*>(c + H);
    const v4f ce = *reinterpret_cast<const v4f*>(c + 2 * H);
    const v4f cz = *reinterpret_cast<const v4f*>(c + 3 * H);
    float* dst = Jt + (size_t)(first + (long long)r * apart) * H * H + j4;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int i = i0 + 16 * q;
      v4f o = wr[q] * ca + wn[q] * cc + wz[q] * ce;
#pragma unroll
      for (int u = 0; u < 4; ++u) o[u] += (i == j4 + u) ? cz[u] : 0.f;
      if (STREAM) __builtin_nontemporal_store(o, reinterpret_cast<v4f*>(dst + (size_t)i * H));
      else *reinterpret_cast<v4f*>(dst + (size_t)i * H) = o;
    }
  };
  constexpr int kBlocks = H / 16, kEach = kGruRows / kBlocks;      // rows stored behind each block of hidden units
  int buf = 0, have = 0;                                           // the set of rows whose coefficients are there
  long long had = 0;
  for (long long first = blockIdx.x; first < rows; first += (long long)kGruRows * apart) {
    const int nrows = rows_of(first);
    float* next = coef + (TWICE ? (buf ^ 1) * kGruRows * 4 * H : 0);
    const float* last = coef + buf * kGruRows * 4 * H;
    gru_stage_rows(s, first, rows, h, x, As, apart);
    __syncthreads();
    gru_share<2>(s, [&](int ub, int sub0) {
      gru_gates<2>(s, wt, bias, ub, sub0, As, x + (size_t)first * s.I, nrows,
                   [&](int, int row, int j, float r, float z, float n, float M) {
                     const GruCoefs f = gru_coefs_of(r, z, n, M, As[row * s.LA + j]);
                     float* c = next + row * 4 * H + j;
                     c[0] = f.a, c[H] = f.c, c[2 * H] = f.e, c[3 * H] = z;
                   },
                   apart,
                   [&](int kb) {
                     if (!TWICE) return;
#pragma unroll 1
                     for (int r = kEach * kb; r < min(kEach * kb + kEach, have); ++r) store_row(last, had, r);
                   });
    });
    __syncthreads();                       // As is rewritten by the next set, and the coefficients are complete
    if (TWICE) {
      buf ^= 1, have = nrows, had = first;
    } else {
      for (int r = 0; r < nrows; ++r) store_row(coef, first, r);
      __syncthreads();
    }
  }
  if (TWICE)
    for (int r = 0; r < have; ++r) store_row(coef + buf * kGruRows * 4 * H, had, r);
}

}  // namespace

bppsa_status bppsa_build_jacobians_gru_h128(int T, int B, int I, const float* h, const float* x,
                                            const float* w_ih, const float* w_hh, const float* b_ih,
                                            const float* b_hh, float* Jt, hipStream_t stream) {
  const GruShape s = gru_shape(H, I);
  const long long rows = (long long)T * B;
  // one workgroup of 83 or, with the second buffer, 147 KB (up to 16 inputs) per compute unit; short inputs are dealt out
  // evenly
  const int cus = bppsa_compute_units();
  const int grid = (int)(rows < cus ? rows : cus);
  const size_t one = (size_t)kGruRows * 4 * H * sizeof(float), lds = gru_rows_lds(s) + one;
  if (lds > 160 * 1024) return BPPSA_EUNSUPPORTED;
  const bool twice = lds + one <= 160 * 1024;
  const auto kernel = twice                                ? gru_jacobians_h128_kernel<true, false>
                      : rows * (64 << 10) > (384LL << 20) ? gru_jacobians_h128_kernel<false, true>      // bytes written
                                                            : gru_jacobians_h128_kernel<false, false>;
  BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)(twice ? lds + one : lds)));
  kernel<<<grid, kGruThreads, twice ? lds + one : lds, stream>>>(s, rows, h, x, GruWeights32{w_ih, w_hh, b_ih, b_hh}, Jt);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
