// The gates of a GRU (Section 4.2) recomputed for many (step, sample) rows at once, for every H <= 128:
//   R = W_ir x + b_ir + W_hr h' + b_hr,  Z likewise,  M = W_hn h' + b_hn,  N = W_in x + b_in + r M,
//   r = sigmoid(R), z = sigmoid(Z), n = tanh(N).
// A workgroup stages 32 rows of [h' | x] in LDS, and a wave forms the four values of 16 units for 16 or 32 of
// those rows as v_mfma_f32_16x16x4_f32 products over k = columns of h' and x: lane l supplies
// A[row l % 16][k] from LDS and B[k][unit l % 16] from the weights (read through buffer descriptors: zero past
// the end of a matrix; padding columns are zero on both sides), with k = 16 kb + 4 (l / 16) + s in issue s of
// block kb, so one 16-byte read of either serves four issues.  The four results land in the same
// lane and register, so everything that follows per (row, unit) happens in registers.
#pragma once

#include "activations.h"
#include "bppsa_internal.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kGruRows = 32;
constexpr int kGruThreads = 512;                   // eight waves

struct GruShape {
  int H, I;
  int NB;                                          // blocks of 16 units
  int KX;                                          // blocks of 16 inputs
  int LA;                                          // floats per staged row
};
// (inputs past kGruMaxStaged do not fit beside the rest: they are added one by one in the epilogue)
constexpr int kGruMaxStaged = 256;
static inline GruShape gru_shape(int H, int I) {
  const int nb = (H + 15) / 16, kx = I <= kGruMaxStaged ? (I + 15) / 16 : 0;
  return GruShape{H, I, nb, kx, 16 * (nb + kx) + 4};
}
static inline size_t gru_rows_lds(const GruShape& s) { return (size_t)kGruRows * s.LA * sizeof(float); }

struct GruWeights32 {
  const float* w_ih;
  const float* w_hh;
  const float* b_ih;
  const float* b_hh;
};

// rows row0, row0 + apart, ... (32 of them) of [h' | 0 | x | 0] into As; rows past the end read as zero
__device__ __forceinline__ void gru_stage_rows(const GruShape& s, long long row0, long long rows,
                                               const float* __restrict__ h, const float* __restrict__ x, float* As,
                                               int apart = 1) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int xcol = 16 * s.NB, cols = xcol + 16 * s.KX;
  for (int r = wave; r < kGruRows; r += nw) {
    const long long row = row0 + (long long)r * apart;
    const bool in = row < rows;
    const float* hr = h + (size_t)row * s.H;
    const float* xr = x + (size_t)row * s.I;
    for (int c = lane; c < cols; c += 64) {
      float v = 0.f;
      if (in && c < s.H) v = hr[c];
      if (in && c >= xcol && c - xcol < s.I) v = xr[c - xcol];
      As[r * s.LA + c] = v;
    }
  }
}

// The same through registers, so that the next rows are on their way while these are worked on, by WAVES waves: columns
// of h' below 64 HS and of x below 64 are fetched ahead, any others of x when the rows are put down.  Requests through
// buffer descriptors read zero past the end; branches around them cost more registers than the rows.
template <int WAVES, int HS>
struct GruRowRequests {
  static constexpr int kEach = kGruRows / WAVES;
  float u[kEach][HS], v[kEach];
  __device__ __forceinline__ void fetch(const GruShape& s, long long row0, long long rows, const float* __restrict__ h,
                                        const float* __restrict__ x) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int left = row0 < rows ? (int)(rows - row0 < kGruRows ? rows - row0 : kGruRows) : 0;
    const size_t at = left > 0 ? (size_t)row0 : 0;
    const auto rh = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(h + at * s.H), 0, left * s.H * 4, 0x00020000);
    const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x + at * s.I), 0, left * s.I * 4, 0x00020000);
    constexpr unsigned kPast = 0x80000000u;        // no 32 rows reach it: zero
    const unsigned cx = lane < s.I ? 4 * lane : kPast;
    unsigned ch[HS];
#pragma unroll
    for (int j = 0; j < HS; ++j) ch[j] = lane + 64 * j < s.H ? 4 * (lane + 64 * j) : kPast;
#pragma unroll
    for (int r = 0; r < kEach; ++r) {
      const int row = wave + WAVES * r;
#pragma unroll
      for (int j = 0; j < HS; ++j)
        u[r][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rh, ch[j] + row * s.H * 4, 0, 0));
      v[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, cx + row * s.I * 4, 0, 0));
    }
  }
  __device__ __forceinline__ void put(const GruShape& s, long long row0, long long rows, const float* __restrict__ x,
                                      float* As) const {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), xcol = 16 * s.NB;
#pragma unroll
    for (int r = 0; r < kEach; ++r) {
      float* to = As + (wave + WAVES * r) * s.LA;
#pragma unroll
      for (int j = 0; j < HS; ++j)
        if (lane + 64 * j < xcol) to[lane + 64 * j] = u[r][j];
      if (lane < 16 * s.KX) to[xcol + lane] = v[r];
    }
    if (s.KX > 4)                                  // uniform
      for (int r = wave; r < kGruRows; r += WAVES)
        for (int c = 64 + lane; c < 16 * s.KX; c += 64)
          As[r * s.LA + xcol + c] = (row0 + r < rows && c < s.I) ? x[(size_t)(row0 + r) * s.I + c] : 0.f;
  }
};

// what a lane adds to its unit's values
struct GruBias {
  float r, z, m, n;
};
__device__ __forceinline__ GruBias gru_bias(const GruShape& s, const GruWeights32& w, int unit) {
  GruBias b = {0.f, 0.f, 0.f, 0.f};
  if (unit < s.H) {
    if (w.b_ih) b.r = w.b_ih[unit], b.z = w.b_ih[s.H + unit], b.n = w.b_ih[2 * s.H + unit];
    if (w.b_hh) b.r += w.b_hh[unit], b.z += w.b_hh[s.H + unit], b.m = w.b_hh[2 * s.H + unit];
  }
  return b;
}

// Columns from n on become zero: a piece read past the end of its row holds the next unit's weights, and where one
// of those is infinite the zeros of the padded rows do not keep it out.
__device__ __forceinline__ void gru_cut(v4f& r, v4f& z, v4f& n_, int col, int n) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const bool in = col + v < n;
    r[v] = in ? r[v] : 0.f, z[v] = in ? z[v] : 0.f, n_[v] = in ? n_[v] : 0.f;
  }
}

// Units 16 ub .. + 15 for the rows 16 (sub0 + s) .. + 15, s < NSUB, of the staged tile, by one wave.
// emit(4 s + register, row in tile, unit, r, z, n, M) for every unit < H (also for rows past the end: gates of zeros).
// xrows: x of the tile's first row, `nrows` of which exist, rows `apart` apart; read only where the inputs are not
// staged.  between(kb) is called behind the products of every block of hidden units.
struct GruNothingBetween {
  __device__ __forceinline__ void operator()(int) const {}
};
template <int NSUB, class F, class Between = GruNothingBetween>
__device__ __forceinline__ void gru_gates(const GruShape& s, const GruWeights32& w, const GruBias& bias, int ub, int sub0,
                                          const float* As, const float* __restrict__ xrows, int nrows, F&& emit,
                                          int apart = 1, Between&& between = Between()) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
  const int unit = 16 * ub + l16;
  const auto rh = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w.w_hh), 0, 3 * s.H * s.H * 4, 0x00020000);
  const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w.w_ih), 0, s.KX ? 3 * s.H * s.I * 4 : 0, 0x00020000);
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f R[NSUB], Z[NSUB], M[NSUB], N[NSUB];
#pragma unroll
  for (int k = 0; k < NSUB; ++k) R[k] = zero, Z[k] = zero, M[k] = zero, N[k] = zero;
  const float* arow = As + (16 * sub0 + l16) * s.LA + 4 * q;
#define BPPSA_LOAD4(rsrc, off) __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off), 0, 0))
#define BPPSA_MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0)
  // the weights of the next block are on their way while this one's are multiplied
  v4f br, bz, bn;
  {
    const unsigned step = (unsigned)s.H * (unsigned)s.H * 4u;
    unsigned off = ((unsigned)unit * (unsigned)s.H + 4u * q) * 4u;
    br = BPPSA_LOAD4(rh, off), bz = BPPSA_LOAD4(rh, off + step), bn = BPPSA_LOAD4(rh, off + 2u * step);
    for (int kb = 0; kb < s.NB; ++kb) {
      off += 64u;
      const v4f nr = BPPSA_LOAD4(rh, off), nz = BPPSA_LOAD4(rh, off + step), nn = BPPSA_LOAD4(rh, off + 2u * step);
      __builtin_amdgcn_sched_barrier(0);
      if (16 * kb + 16 > s.H) gru_cut(br, bz, bn, 16 * kb + 4 * q, s.H);
#pragma unroll
      for (int k = 0; k < NSUB; ++k) {
        const v4f a = *reinterpret_cast<const v4f*>(arow + 16 * k * s.LA + 16 * kb);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          R[k] = BPPSA_MFMA(a[v], br[v], R[k]);
          Z[k] = BPPSA_MFMA(a[v], bz[v], Z[k]);
          M[k] = BPPSA_MFMA(a[v], bn[v], M[k]);
        }
      }
      br = nr, bz = nz, bn = nn;
      between(kb);
    }
  }
  {
    const unsigned step = (unsigned)s.H * (unsigned)s.I * 4u;
    unsigned off = ((unsigned)unit * (unsigned)s.I + 4u * q) * 4u;
    for (int kb = 0; kb < s.KX; ++kb, off += 64u) {
      br = BPPSA_LOAD4(rx, off), bz = BPPSA_LOAD4(rx, off + step), bn = BPPSA_LOAD4(rx, off + 2u * step);
      if (16 * kb + 16 > s.I) gru_cut(br, bz, bn, 16 * kb + 4 * q, s.I);
#pragma unroll
      for (int k = 0; k < NSUB; ++k) {
        const v4f a = *reinterpret_cast<const v4f*>(arow + 16 * k * s.LA + 16 * (s.NB + kb));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          R[k] = BPPSA_MFMA(a[v], br[v], R[k]);
          Z[k] = BPPSA_MFMA(a[v], bz[v], Z[k]);
          N[k] = BPPSA_MFMA(a[v], bn[v], N[k]);
        }
      }
    }
  }
#undef BPPSA_MFMA
#undef BPPSA_LOAD4
  if (unit >= s.H) return;
#pragma unroll
  for (int k = 0; k < NSUB; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 * (sub0 + k) + 4 * q + v;
      float ir = R[k][v] + bias.r, iz = Z[k][v] + bias.z, in = N[k][v] + bias.n;
      const float m = M[k][v] + bias.m;
      if (s.KX == 0 && row < nrows) {
        const float* xr = xrows + (size_t)row * apart * s.I;
        const float* wi = w.w_ih + (size_t)unit * s.I;
        const size_t gate = (size_t)s.H * s.I;
        for (int i = 0; i < s.I; ++i) ir += wi[i] * xr[i], iz += wi[gate + i] * xr[i], in += wi[2 * gate + i] * xr[i];
      }
      const float r = bppsa_sigmoid(ir), z = bppsa_sigmoid(iz);
      emit(4 * k + v, row, unit, r, z, bppsa_tanh(in + r * m), m);
    }
}

// How the eight waves share a tile's units: up to four blocks of units, a wave per (block, half of the rows);
// beyond, a wave per block for all rows.  body(ub, sub0) is called with what this wave does, if anything.
template <int NSUB, class F>
__device__ __forceinline__ void gru_share(const GruShape& s, F&& body) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ub = NSUB == 1 ? wave >> 1 : wave, sub0 = NSUB == 1 ? wave & 1 : 0;
  if (ub < s.NB) body(ub, sub0);
}

// The coefficients of Appendix E's closed form of the transposed Jacobian,
//   Jt[i][j] = W_hr[j][i] a_j + W_hn[j][i] c_j + W_hz[j][i] e_j + [i == j] z_j.
struct GruCoefs {
  float a, c, e;
};
__device__ __forceinline__ GruCoefs gru_coefs_of(float r, float z, float n, float M, float hprev) {
  const float dn = (1.f - z) * (1.f - n * n);
  return GruCoefs{dn * M * r * (1.f - r), dn * r, (hprev - n) * z * (1.f - z)};
}

}  // namespace
