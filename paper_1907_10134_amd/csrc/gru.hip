// GRU variants of the Jacobian builder (H < 128) and, for every H <= 128, of the coefficient vectors the fused
// scan reads and of the parameter-gradient reduction.
//
// Cell (Section 4.2; Appendix E's rewrite with pre-activations R, Z, M, N):
//   r = sigmoid(R), z = sigmoid(Z), n = tanh(N), N = W_in x + b_in + r o M,
//   M = W_hn h' + b_hn, h = (1 - z) o n + z o h'.
// The gates are not inputs: they are recomputed from (h', x, weights) for all steps in parallel, as the paper
// does (Appendix E, last paragraph), on the matrix cores (gru_gates.h).
#include "gru_gates.h"
#include "train_parts.h"

namespace {

// Jacobians of 32 rows at a time: coefficients into LDS, then the tiles are streamed out.  A piece is W floats
// of a tile row (16 bytes where H is a multiple of four); a thread owns the same P pieces of every tile, with
// their 3 W P recurrent weights in registers, or, where a tile has fewer pieces than the workgroup threads,
// one piece of every (512 / pieces)-th tile.  More than P 512 pieces: blockIdx.y tells the ranges apart.  Bound by
// the stores.
// (H = 20, I = 24, T = 517, B = 32: 26 MB in 19.6 us, with three workgroups to a compute unit where a tile is one piece
// a thread, 80 registers, 21.6 with two; 512 tiles, which two rounds of 256 hold, 15.5 and 16.4.)
template <int W, int P, int NSUB, bool STREAM>
__global__ void __launch_bounds__(kGruThreads, P == 1 ? 6 : 1)
gru_jacobians_kernel(const GruShape s, long long rows, long long tiles, const float* __restrict__ h,
                     const float* __restrict__ x, const GruWeights32 wt, float* __restrict__ Jt) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int H = s.H, tid = threadIdx.x;
  const int HC = (H + 3) & ~3;
  float* As = smem;                                // [32][LA]
  float* coef = smem + kGruRows * s.LA;            // [32][4][HC]: a, c, e, z
  const int per_row = H / W, pieces = H * per_row;
  const int side = P == 1 ? kGruThreads / pieces : 1;                 // tiles side by side
  const int slot = side > 1 ? tid / pieces : 0;
  const int p0 = tid - slot * pieces + blockIdx.y * P * kGruThreads;
  const bool owner = slot < side;
  float wr[P][W], wn[P][W], wz[P][W];
  int pi[P], pj[P];
#pragma unroll
  for (int k = 0; k < P; ++k) {
    const int p = p0 + kGruThreads * k;
    pi[k] = p < pieces ? p / per_row : 0;
    pj[k] = p < pieces ? (p - pi[k] * per_row) * W : 0;
#pragma unroll
    for (int u = 0; u < W; ++u) {
      wr[k][u] = wt.w_hh[(size_t)(pj[k] + u) * H + pi[k]];
      wz[k][u] = wt.w_hh[(size_t)(H + pj[k] + u) * H + pi[k]];
      wn[k][u] = wt.w_hh[(size_t)(2 * H + pj[k] + u) * H + pi[k]];
    }
  }
  GruBias bias = {};
  gru_share<NSUB>(s, [&](int ub, int) { bias = gru_bias(s, wt, 16 * ub + (tid & 15)); });
  for (long long tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const long long row0 = tile * kGruRows;
    const int nrows = (int)((rows - row0 < kGruRows) ? (rows - row0) : kGruRows);
    gru_stage_rows(s, row0, rows, h, x, As);
    __syncthreads();
    gru_share<NSUB>(s, [&](int ub, int sub0) {
      gru_gates<NSUB>(s, wt, bias, ub, sub0, As, x + (size_t)row0 * s.I, nrows, [&](int, int row, int j, float r, float z, float n, float M) {
        const GruCoefs f = gru_coefs_of(r, z, n, M, As[row * s.LA + j]);
        float* c = coef + row * 4 * HC + j;
        c[0] = f.a, c[HC] = f.c, c[2 * HC] = f.e, c[3 * HC] = z;
      });
    });
    __syncthreads();
    if (owner) {
      for (int r = slot; r < nrows; r += side) {
        const float* c = coef + r * 4 * HC;
        float* dst = Jt + (size_t)(row0 + r) * H * H;
#pragma unroll
        for (int k = 0; k < P; ++k) {
          if (P > 1 && p0 + kGruThreads * k >= pieces) continue;
          float o[W];
#pragma unroll
          for (int u = 0; u < W; ++u) {
            const int j = pj[k] + u;
            o[u] = wr[k][u] * c[j] + wn[k][u] * c[HC + j] + wz[k][u] * c[2 * HC + j] + (pi[k] == j ? c[3 * HC + j] : 0.f);
          }
          if constexpr (W == 4) {
            v4f* to = reinterpret_cast<v4f*>(dst + pi[k] * H + pj[k]);
            const v4f val = {o[0], o[1], o[2], o[3]};
            if (STREAM) __builtin_nontemporal_store(val, to);
            else *to = val;
          } else {
            if (STREAM) __builtin_nontemporal_store(o[0], dst + pi[k] * H + pj[k]);
            else dst[pi[k] * H + pj[k]] = o[0];
          }
        }
      }
    }
    __syncthreads();                               // As and coef are rewritten by the next tile
  }
}

// coef[row][4][H] = (a, c, e, z), for a scan that generates the Jacobians itself instead of reading them
// (H = 128, 5170 rows: 17.5 us, 52 us with the products in scalar loops), and, by the workgroups past those of the
// rows, wT[g][i][j] = W_hg[j][i] for g = r, n, z (the order of the coefficients a, c, e; by itself 5 us in front).
template <int NSUB>
__global__ void __launch_bounds__(kGruThreads)
gru_coefs_kernel(const GruShape s, long long rows, int tiles, const float* __restrict__ h, const float* __restrict__ x,
                 const GruWeights32 wt, float* __restrict__ coef, float* __restrict__ wT) {
  extern __shared__ __attribute__((aligned(16))) float As[];
  if ((int)blockIdx.x >= tiles) {                // uniform over the workgroup
    const int H = s.H, e = ((int)blockIdx.x - tiles) * kGruThreads + (int)threadIdx.x;      // over 3 * H * H
    if (e >= 3 * H * H) return;
    const int g = e / (H * H), rem = e - g * H * H, i = rem / H, j = rem - i * H;
    const int src_gate = g == 0 ? 0 : (g == 1 ? 2 : 1);     // w_hh rows are ordered r, z, n
    wT[e] = wt.w_hh[((size_t)src_gate * H + j) * H + i];
    return;
  }
  const long long row0 = (long long)blockIdx.x * kGruRows;
  const int nrows = (int)((rows - row0 < kGruRows) ? (rows - row0) : kGruRows);
  gru_stage_rows(s, row0, rows, h, x, As);
  __syncthreads();
  gru_share<NSUB>(s, [&](int ub, int sub0) {
    const GruBias bias = gru_bias(s, wt, 16 * ub + (threadIdx.x & 15));
    gru_gates<NSUB>(s, wt, bias, ub, sub0, As, x + (size_t)row0 * s.I, nrows, [&](int, int row, int j, float r, float z, float n, float M) {
      if (row >= nrows) return;
      const GruCoefs f = gru_coefs_of(r, z, n, M, As[row * s.LA + j]);
      float* c = coef + (size_t)(row0 + row) * 4 * s.H + j;
      c[0] = f.a, c[s.H] = f.c, c[2 * s.H] = f.e, c[3 * s.H] = z;
    });
  });
}

// Parameter gradients (Eq. 2, summed over steps and samples) in one pass over the rows:
//   dW_hh = sum Dh^T h', db_hh = sum Dh, dW_ih = sum Di^T x, db_ih = sum Di,
// with Dh = (dR, dZ, dM), Di = (dR, dZ, dN) from the recomputed gates and g = dL/dh[t+1].  A persistent
// workgroup takes 32 rows at a time.  A wave forms the gates of a block of 16 units, leaves the four deltas in LDS with
// the rows innermost, and contracts them over the rows with all columns of [h' | 1] and [x | 1], read out of the staged
// rows, as 16x16x4 fp32 MFMA: nobody else reads its deltas and there are two buffers of rows, so that one barrier to a
// set is enough, and 3 CT tiles of sums stay in registers for the workgroup's whole life.  Each workgroup leaves one
// partial, [3H][H + 1 + I + 1].  More column tiles than CT: another launch, from ct0 on.
//   HALVES: two waves to a block of units, 16 rows each, whose sums are added at the end (cells of up to 64 units);
//   otherwise a wave to a block, and blockIdx.y tells the blocks apart that do not fit the workgroup's waves.
//   GROUPS: this many times the waves, each with its share of the column tiles; the gates are formed by each.
// Two or more workgroups of four waves fit on a compute unit, with a wave of each on every SIMD, so that one's products
// run beside the other's gates and staging; where inputs are wide, one of eight waves.  Bound by the products and by the
// latencies of a set.
// Before, one set of 32 rows and all units went to a workgroup of eight waves, with the products behind two more barriers
// and the columns copied to where four rows of one lie together.  With the sum of the partials 4096 x 16 rows
// of H = 128, I = 1 take 176 us (245 then), 1034 x 5 of I = 12 42 (75), 1034 x 64 of H = 64, I = 38 95 (133), of H = 20,
// I = 38 51 (67), 517 x 32 of H = 20, I = 24 19 (23); 60 rows of H = 128 34 (66); the smallest the same.  For inputs of 64
// columns and more see the rule at the launch; five blocks of units with 11 or 12 column tiles, which leave three of eight
// waves idle, are the one form that was faster then, by 3 to 7 % (H = 72, I = 110 117 us, 125 now).
template <int CT, int WAVES, bool HALVES, int GROUPS = 1>
__global__ void __launch_bounds__(64 * WAVES, HALVES ? (CT <= 4 ? 3 : CT <= 8 ? 2 : 1) : (CT <= 10 ? 2 : 1))
gru_param_kernel(const GruShape s, int ct0, int ct_count, long long rows, long long tiles, const float* __restrict__ h,
                 const float* __restrict__ x, const float* __restrict__ G, const GruWeights32 wt,
                 float* __restrict__ part) {
  constexpr int kRows = HALVES ? 16 : kGruRows, kSubs = kRows / 16, LR = kRows + 4, kKind = 16 * LR;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int H = s.H, I = s.I, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cth = (H + 16) / 16;                   // column tiles of [h' | 1]
  constexpr int kGroup = WAVES / GROUPS;           // waves that share the column tiles of a group
  if (GROUPS > 1) {
    const int each = (ct_count + GROUPS - 1) / GROUPS, before = wave / kGroup * each;
    ct0 += before;
    ct_count = min(each, ct_count - before);
  }
  const int block = (HALVES ? wave % kGroup >> 1 : wave % kGroup), sub = HALVES ? wave & 1 : 0;
  const int ub = (int)blockIdx.y * kGroup + block, unit = 16 * ub + l16;
  const bool busy = ub < s.NB;                     // uniform over the wave
  float* const delta = smem + 2 * kGruRows * s.LA + wave * 4 * kKind + l16 * LR;           // [4][16][LR]: dR, dZ, dN, dM
  v4f acc[3][CT];
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[g][c] = v4f{0.f, 0.f, 0.f, 0.f};
  GruBias bias = {};
  if (busy) bias = gru_bias(s, wt, unit);
  if (unit >= H)                                   // units past H stay zero
    for (int k = 0; k < 4; ++k)
      for (int r = q; r < kRows; r += 4) delta[k * kKind + r] = 0.f;
  GruRowRequests<WAVES, HALVES ? 1 : 2> next;
  next.fetch(s, (long long)blockIdx.x * kGruRows, rows, h, x);
  int buf = 0;
  for (long long tile = blockIdx.x; tile < tiles; tile += gridDim.x, buf ^= 1) {
    const long long row0 = tile * kGruRows;
    const int nrows = (int)((rows - row0 < kGruRows) ? (rows - row0) : kGruRows);
    float* As = smem + buf * kGruRows * s.LA;      // last read two sets ago, in front of a barrier
    next.put(s, row0, rows, x, As);
    __syncthreads();
    const long long row_next = (tile + gridDim.x) * kGruRows;         // past the end: reads nothing
    if (!busy) {
      next.fetch(s, row_next, rows, h, x);
      continue;
    }
    float g[4 * kSubs];                            // dL/dh of this lane's rows, requested ahead of the gates
#pragma unroll
    for (int v = 0; v < 4 * kSubs; ++v) {
      const int row = 16 * (sub + (v >> 2)) + 4 * q + (v & 3);
      g[v] = (row < nrows && unit < H) ? G[(size_t)(row0 + row) * H + unit] : 0.f;
    }
    gru_gates<kSubs>(s, wt, bias, ub, sub, As, x + (size_t)row0 * I, nrows,
                     [&](int v, int row, int j, float r, float z, float n, float M) {
      const float dN = g[v] * (1.f - z) * (1.f - n * n);
      const bool in = row < nrows;                 // past the end the gates of an infinite weight are NaN
      float* d = delta + row - 16 * sub;
      d[0] = in ? dN * M * r * (1.f - r) : 0.f;
      d[kKind] = in ? g[v] * (As[row * s.LA + j] - n) * z * (1.f - z) : 0.f;
      d[2 * kKind] = in ? dN : 0.f;
      d[3 * kKind] = in ? dN * r : 0.f;
    });
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    __builtin_amdgcn_sched_barrier(0);
    next.fetch(s, row_next, rows, h, x);           // (not under the gates: registers)
#pragma unroll 1
    for (int kc = 0; kc < kSubs; ++kc) {
      v4f d[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) d[k] = *reinterpret_cast<const v4f*>(delta + k * kKind + 16 * kc + 4 * q);
      const float* const rowq = As + (16 * (sub + kc) + 4 * q) * s.LA + l16;
      int tile0 = ct0;
      asm volatile("" : "+s"(tile0));              // what follows from it is not kept for every c
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        if (c < ct_count) {                        // uniform, like everything that follows from it
          const bool of_h = tile0 + c < cth;
          const int first = 16 * (of_h ? tile0 + c : tile0 + c - cth), have = (of_h ? H : I) - first;
          const float* from = rowq + first + (of_h ? 0 : 16 * s.NB);
          float b[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) b[v] = from[v * s.LA];
          if (have < 16) {                         // the tile with the ones
#pragma unroll
            for (int v = 0; v < 4; ++v) b[v] = l16 < have ? b[v] : l16 == have ? 1.f : 0.f;
          }
          const v4f dn = of_h ? d[3] : d[2];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            acc[0][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[0][v], b[v], acc[0][c], 0, 0, 0);
            acc[1][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[1][v], b[v], acc[1][c], 0, 0, 0);
            acc[2][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(dn[v], b[v], acc[2][c], 0, 0, 0);
          }
        }
      }
    }
  }
  if (HALVES) {                                    // the second half's sums join the first's
    v4f* const red = reinterpret_cast<v4f*>(smem) + (wave >> 1) * 3 * CT * 64 + lane;
    __syncthreads();
    if (busy && sub == 1) {
#pragma unroll
      for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int c = 0; c < CT; ++c) red[(g * CT + c) * 64] = acc[g][c];
    }
    __syncthreads();
    if (sub == 1) return;
    if (busy) {
#pragma unroll
      for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[g][c] += red[(g * CT + c) * 64];
    }
  }
  if (!busy) return;
  const int W = H + 1 + I + 1;
  float* out = part + (size_t)blockIdx.x * 3 * H * W;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int col = 16 * (ct0 + c) + l16, cx = col - 16 * cth;
    const int at = c >= ct_count ? -1 : cx < 0 ? (col <= H ? col : -1) : (cx <= I ? H + 1 + cx : -1);
#pragma unroll
    for (int g = 0; g < 3; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int to = 16 * ub + 4 * q + v;
        if (to < H && at >= 0) out[(size_t)(g * H + to) * W + at] = acc[g][c][v];
      }
  }
}

// Adds the partials in a fixed order (256 partials of H = 128: 11 us; one thread per element took 34).
__global__ void __launch_bounds__(64 * kFinishWaves)
gru_param_finish_kernel(int nsplit, int H, int I, const float* __restrict__ part, float* __restrict__ dW_ih,
                        float* __restrict__ dW_hh, float* __restrict__ db_ih, float* __restrict__ db_hh) {
  __shared__ float red[kFinishWaves][64];
  const int W = H + 1 + I + 1, E = 3 * H * W, e = blockIdx.x * 64 + (int)(threadIdx.x & 63);
  const float t = bppsa_add_partials(nsplit, E, E, blockIdx.x * 64, part, red);
  if (threadIdx.x >= 64 || e >= E) return;
  const int g = e / W, c = e - g * W;
  if (c < H) dW_hh[(size_t)g * H + c] = t;
  else if (c == H) db_hh[g] = t;
  else if (c < H + 1 + I) dW_ih[(size_t)g * I + (c - H - 1)] = t;
  else db_ih[g] = t;
}

// partials of the reduction: a workgroup per unit, at least two tiles each, at most kMaxSplits
constexpr int kMaxSplits = 256;
int gru_splits(long long rows) {
  long long ns = (rows + 2 * kGruRows - 1) / (2 * kGruRows);
  if (ns > kMaxSplits) ns = kMaxSplits;
  if (ns < 1) ns = 1;
  return (int)ns;
}

constexpr size_t kMaxLds = 160 * 1024;

template <class K>
bppsa_status allow_lds(K kernel, size_t lds) {
  if (lds > kMaxLds) return BPPSA_EUNSUPPORTED;
  if (lds > 48 * 1024)
    BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  return BPPSA_OK;
}

}  // namespace

// the 4 GB streams of H = 128
bppsa_status bppsa_build_jacobians_gru_h128(int T, int B, int I, const float* h, const float* x,
                                            const float* w_ih, const float* w_hh, const float* b_ih,
                                            const float* b_hh, float* Jt, hipStream_t stream);

bppsa_status bppsa_build_jacobians_gru(int T, int B, int H, int I,
                                       const float* h, const float* x,
                                       const float* w_ih, const float* w_hh,
                                       const float* b_ih, const float* b_hh,
                                       float* Jt, hipStream_t stream) {
  if (H > 128) return BPPSA_EUNSUPPORTED;
  if (H == 128) return bppsa_build_jacobians_gru_h128(T, B, I, h, x, w_ih, w_hh, b_ih, b_hh, Jt, stream);
  const GruShape s = gru_shape(H, I);
  const GruWeights32 wt = {w_ih, w_hh, b_ih, b_hh};
  const long long rows = (long long)T * B, tiles = (rows + kGruRows - 1) / kGruRows;
  const size_t lds = gru_rows_lds(s) + (size_t)kGruRows * 4 * ((H + 3) & ~3) * sizeof(float);
  const bool vec = H % 4 == 0 && ((uintptr_t)Jt & 15) == 0;
  const int pieces = H * H / (vec ? 4 : 1), P = (pieces + kGruThreads - 1) / kGruThreads;
  const bool stream_out = bppsa_stream_jacobians(T, B, H);
  const long long most = (P == 1 ? 3LL : 2LL) * bppsa_compute_units();
#define BPPSA_JAC_RUN(...)                                                                             \
  do {                                                                                                 \
    BPPSA_TRY(allow_lds(__VA_ARGS__, lds));                                                            \
    __VA_ARGS__<<<grid, kGruThreads, lds, stream>>>(s, rows, tiles, h, x, wt, Jt);                     \
  } while (0)
#define BPPSA_JAC(W, PP, N)                                                                            \
  do {                                                                                                 \
    const dim3 grid((int)(tiles < most ? tiles : most), bppsa_ceil_div(P, PP));                        \
    if (stream_out) BPPSA_JAC_RUN(gru_jacobians_kernel<W, PP, N, true>);                               \
    else BPPSA_JAC_RUN(gru_jacobians_kernel<W, PP, N, false>);                                         \
  } while (0)
  if (vec) {                                       // H <= 44 one piece, <= 64 two, <= 124 ranges of four
    if (P == 1) BPPSA_JAC(4, 1, 1);
    else if (P == 2) BPPSA_JAC(4, 2, 1);
    else BPPSA_JAC(4, 4, 2);
  } else {                                         // H <= 22 one, <= 63 eight, <= 127 two ranges of sixteen
    if (P == 1) BPPSA_JAC(1, 1, 1);
    else if (P <= 8) BPPSA_JAC(1, 8, 1);
    else BPPSA_JAC(1, 16, 2);
  }
#undef BPPSA_JAC
#undef BPPSA_JAC_RUN
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_gru_coefs_h128(long long rows, int I, const float* h, const float* x, const float* w_ih,
                                  const float* w_hh, const float* b_ih, const float* b_hh, float* coef,
                                  float* wT, hipStream_t stream) {
  const int H = 128;
  const GruShape s = gru_shape(H, I);
  const long long tiles = (rows + kGruRows - 1) / kGruRows;
  const int transposing = (3 * H * H + kGruThreads - 1) / kGruThreads;
  if (tiles > 0x7fffffffLL - transposing) return BPPSA_EOVERFLOW;
  BPPSA_TRY(allow_lds(gru_coefs_kernel<2>, gru_rows_lds(s)));
  gru_coefs_kernel<2><<<(int)tiles + transposing, kGruThreads, gru_rows_lds(s), stream>>>(
      s, rows, (int)tiles, h, x, GruWeights32{w_ih, w_hh, b_ih, b_hh}, coef, wT);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

// The kernels use room for the partials (gru_splits); what is asked for, and refused below, is never less than the
// four deltas per row and 128 partials of earlier versions, on which callers may count (134 MB at T = 4096, B = 16,
// H = 128, of which 52 are used).
size_t bppsa_param_grads_gru_ws(int T, int B, int H, int I) {
  const long long rows = (long long)T * B;
  const size_t W = (size_t)H + 1 + I + 1, one = 3 * (size_t)H * W * sizeof(float);
  long long splits = (rows + 127) / 128;
  if (splits > 128) splits = 128;
  const size_t floor = bppsa_align_up((size_t)rows * 4 * H * sizeof(float), 256) + bppsa_align_up((size_t)splits * one, 256);
  const size_t need = bppsa_align_up((size_t)gru_splits(rows) * one, 256);
  return need > floor ? need : floor;
}

bppsa_status bppsa_param_grads_gru(int T, int B, int H, int I,
                                   const float* h, const float* x, const float* G,
                                   const float* w_ih, const float* w_hh,
                                   const float* b_ih, const float* b_hh,
                                   float* dW_ih, float* dW_hh, float* db_ih, float* db_hh,
                                   void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (H > 128) return BPPSA_EUNSUPPORTED;
  const long long rows = (long long)T * B, tiles = (rows + kGruRows - 1) / kGruRows;
  const int W = H + 1 + I + 1;
  if (W > 256) return BPPSA_EUNSUPPORTED;
  if (!workspace || workspace_bytes < bppsa_param_grads_gru_ws(T, B, H, I)) return BPPSA_EWORKSPACE;
  const GruShape s = gru_shape(H, I);
  const GruWeights32 wt = {w_ih, w_hh, b_ih, b_hh};
  float* part = static_cast<float*>(workspace);
  const int cth = (H + 16) / 16, ctx = (I + 16) / 16, all = cth + ctx;
  // Which form (4096 x 8 rows, us, and with workgroups of four waves and no groups):
  //   one block of units: both pairs of waves would hold the same units, so they split the columns
  //     (H = 8, I = 100 29.5, 40.6; I = 200, then in two launches, 62, 120; H = 16, I = 1 16.6, 18.1);
  //   two: the same with twice the waves, if two workgroups of four do not have the registers for the columns
  //     (H = 20, I = 126 50.8, 54.2; I = 200 71, 129; I = 64, for which they have them, 43, 32.5);
  //   more: workgroups of four waves in pairs on a compute unit; where registers or LDS have room for one only, of eight
  //     waves (H = 33, I = 200 147, 184; H = 64, I = 126 128, 142; H = 80, I = 126 189, 276; H = 128, I = 126 236, 321),
  //     unless there are so few rows that not all units have work, or of four blocks two sets (1034 x 5 rows: H = 128,
  //     I = 126 124, 97; H = 64, I = 88 44.9, 42.7).
  const bool two_groups = s.NB == 1 || (s.NB == 2 && all > 8);
  const int launches = bppsa_ceil_div(all, two_groups ? 20 : 12), each_launch = bppsa_ceil_div(all, launches);
  const int ct = two_groups ? (each_launch + 1) / 2 : each_launch;                      // 10 and 12 at most
  const int sums_for = s.NB == 1 ? (ct + 1) / 2 * 2 : s.NB == 2 ? (two_groups ? (ct <= 6 ? 6 : 10) : ct <= 4 ? 4 : 8)
                                                                : (ct <= 8 ? 8 : ct <= 10 ? 10 : 12);      // CT
  bool halves = s.NB <= 2;
  int waves = s.NB == 2 && two_groups ? 8 : 4;
  auto lds_of = [&]() {
    const size_t deltas = (size_t)waves * 4 * 16 * ((halves ? 16 : kGruRows) + 4) * sizeof(float);
    const size_t sums = halves ? (size_t)(waves / 2) * 3 * sums_for * 64 * sizeof(v4f) : 0;
    const size_t need = 2 * gru_rows_lds(s) + deltas;
    return need > sums ? need : sums;
  };
  const int cus = bppsa_compute_units();
  int ns = gru_splits(rows);
  if (s.NB > 2 && (ct > 10 || 2 * lds_of() > kMaxLds) &&
      (s.NB == 3 || (s.NB == 4 ? tiles > 2 * cus : 2 * ns > cus))) {
    waves = 8;
    halves = s.NB <= 4;
  }
  const size_t lds = lds_of();
  if (s.NB <= 4 || waves == 8) {
    // All workgroups take the same number of sets, with as many partials as the least workspace holds.  Of one, two and three
    // workgroups to a unit, what the fullest unit does counts, 0.7 of it where they overlap.
    long long fit = waves == 8 ? 1 : halves ? (ct <= 4 ? 3 : ct <= 8 ? 2 : 1) : ct <= 10 ? 2 : 1;
    while (fit > 1 && fit * lds > kMaxLds) --fit;
    const long long room = (long long)(bppsa_param_grads_gru_ws(T, B, H, I) / (3 * (size_t)H * W * sizeof(float)));
    double least = 1e300;
    for (const long long last = all <= 4 ? fit : 1; fit >= last; --fit) {
      const long long most = fit * cus < room ? fit * cus : room, each = (tiles + most - 1) / most;
      const long long groups = (tiles + each - 1) / each, fullest = (groups + cus - 1) / cus * each;
      const double cost = (double)fullest * (groups > cus ? 0.7 : 1.0);
      if (cost < least) least = cost, ns = (int)groups;
    }
  }
  for (int ct0 = 0; ct0 < all; ct0 += each_launch) {
    const int left = all - ct0, n = left < each_launch ? left : each_launch;
#define BPPSA_PART(...)                                                                                           \
  do {                                                                                                            \
    const dim3 grid(ns, halves ? 1 : bppsa_ceil_div(s.NB, waves));                                                \
    BPPSA_TRY(allow_lds(gru_param_kernel<__VA_ARGS__>, lds));                                                     \
    gru_param_kernel<__VA_ARGS__><<<grid, 64 * waves, lds, stream>>>(s, ct0, n, rows, tiles, h, x, G, wt, part);  \
  } while (0)
#define BPPSA_PART_WIDE(WAVES, HALVES)                         \
  do {                                                         \
    if (sums_for == 8) BPPSA_PART(8, WAVES, HALVES, 1);        \
    else if (sums_for == 10) BPPSA_PART(10, WAVES, HALVES, 1); \
    else BPPSA_PART(12, WAVES, HALVES, 1);                     \
  } while (0)
    if (s.NB == 1) {
      if (sums_for == 2) BPPSA_PART(2, 4, true, 2);
      else if (sums_for == 4) BPPSA_PART(4, 4, true, 2);
      else if (sums_for == 6) BPPSA_PART(6, 4, true, 2);
      else if (sums_for == 8) BPPSA_PART(8, 4, true, 2);
      else BPPSA_PART(10, 4, true, 2);
    } else if (two_groups) {
      if (sums_for == 6) BPPSA_PART(6, 8, true, 2);
      else BPPSA_PART(10, 8, true, 2);
    } else if (s.NB == 2) {
      if (sums_for == 4) BPPSA_PART(4, 4, true, 1);
      else BPPSA_PART(8, 4, true, 1);
    } else if (waves == 8 && halves) {
      BPPSA_PART_WIDE(8, true);
    } else if (waves == 8) {
      BPPSA_PART_WIDE(8, false);
    } else {
      BPPSA_PART_WIDE(4, false);
    }
#undef BPPSA_PART_WIDE
#undef BPPSA_PART
    BPPSA_CHECK_LAUNCH();
  }
  gru_param_finish_kernel<<<bppsa_ceil_div(3 * H * W, 64), 64 * kFinishWaves, 0, stream>>>(ns, H, I, part, dW_ih, dW_hh,
                                                                                          db_ih, db_hh);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
