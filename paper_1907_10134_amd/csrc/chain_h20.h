// Scan for H = 20 as what it is a bracketing of: one matrix-vector product after the other, a workgroup per
// sample.  It does a twentieth of the arithmetic of the tree of products and reads every tile once, but its T
// steps wait for one another, so it is the form for chains that are short or for batches that fill the chip by
// themselves; bppsa_chain_h20_us says what it costs.
//
// Seven waves (eight) share the work so that the one that walks the chain never waits for memory:
//   wave 0       the chain.  Rows and columns of a tile are cut in halves A and B of ten.  On even steps the four
//                rows of 16 lanes hold (rows, columns) = (A, A) (A, B) (B, A) (B, B): ten multiply-adds with the
//                vector as DPP operand, and one v_permlane16_swap adds the two column halves.  That leaves the
//                vector as (A A B B), which is what the transposed assignment (A, A) (B, A) (A, B) (B, B) of the
//                odd steps needs; its v_permlane32_swap gives back (A B A B).  Tile rows come from LDS, three
//                steps ahead;
//   waves 1..5   bring tiles into LDS in chunks of 16: read from memory two chunks ahead, or formed from the
//                hidden states and W_hh (tanh RNN) by the arithmetic of the builder, so that both sources give
//                the same bits;
//   wave 6       stores the gradients, so that no load ever waits behind a store;
//   wave 7       in a training iteration: the sums of the parameter gradients, on the matrix cores, which saves the
//                launch that would read states and gradients again.
// One barrier per chunk.
#pragma once

#include "barriers.h"
#include "bppsa_internal.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));

namespace chain_h20 {

constexpr int H = 20;
constexpr int HH = H * H;
constexpr int kC = H / 2;
constexpr int kChunk = 16;
constexpr int kBring = 320;                       // threads that bring tiles: five pieces of 16 bytes per chunk each
constexpr int kPieces = kChunk * HH / 4 / kBring;
constexpr int kStorer = 1 + kBring / 64;             // its wave; behind it the wave of the parameter sums
constexpr int kThreads = 64 * (kStorer + 1), kParamThreads = kThreads + 64;
constexpr int kOutRow = 24;                       // columns 20..23 take what the idle lanes write
constexpr int kOutChunk = kChunk * kOutRow;

// Member i of half A or B: {0..7, 16, 17} and {8..15, 18, 19}, so that a half row is two aligned pieces of 16 bytes
// and one of 8.
__device__ __forceinline__ int unit_of(int half, int i) { return i < 8 ? 8 * half + i : 8 + 2 * half + i; }

// a = product of the ten columns with lanes 0..9 of this lane's row of s, summed with the row 16 (FORM 0) or 32
// (FORM 1) lanes away.  A DPP operand may be read two wait states after it was written.
template <int FORM>
__device__ __forceinline__ float chain_product(const float (&w)[kC], float s) {
  float a, p;
#define BPPSA_STEP(op, w, n) #op "_f32_dpp %0, %2, %" #w " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
#define BPPSA_TEN                                                                                                   \
  "s_nop 1\n\t" BPPSA_STEP(v_mul, 3, 0) BPPSA_STEP(v_fmac, 4, 1) BPPSA_STEP(v_fmac, 5, 2) BPPSA_STEP(v_fmac, 6, 3)   \
  BPPSA_STEP(v_fmac, 7, 4) BPPSA_STEP(v_fmac, 8, 5) BPPSA_STEP(v_fmac, 9, 6) BPPSA_STEP(v_fmac, 10, 7)              \
  BPPSA_STEP(v_fmac, 11, 8) BPPSA_STEP(v_fmac, 12, 9) "v_mov_b32 %1, %0\n\ts_nop 1\n\t"
#define BPPSA_ARGS                                                                                                  \
  "=&v"(a), "=&v"(p)                                                                                                \
      : "v"(s), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]), "v"(w[8]), "v"(w[9])
  if constexpr (FORM == 0) asm(BPPSA_TEN "v_permlane16_swap_b32 %0, %1\n\tv_add_f32 %0, %0, %1" : BPPSA_ARGS);
  else asm(BPPSA_TEN "v_permlane32_swap_b32 %0, %1\n\tv_add_f32 %0, %0, %1" : BPPSA_ARGS);
#undef BPPSA_ARGS
#undef BPPSA_TEN
#undef BPPSA_STEP
  return a;
}

struct Lds {
  __attribute__((aligned(16))) float tiles[3 * kChunk * HH];
  __attribute__((aligned(16))) float outs[4 * kOutChunk];
};

// The pieces of W_hh that a thread of the bringing waves scales (generated tiles).
struct Weights {
  v4f v[kPieces];
  __device__ __forceinline__ void load(const float* __restrict__ w_hh) {
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      // (the piece of thread 64 + e is e modulo 100; other waves load some piece and do not use it)
      const int pc = ((int)threadIdx.x + 36 + kBring * k) % (HH / 4), row = pc / 5, j4 = (pc - row * 5) * 4;
#pragma unroll
      for (int u = 0; u < 4; ++u) v[k][u] = w_hh[(j4 + u) * H + row];
    }
  }
};

// One sample's share of the cell's parameter gradients (Eq. 2), [H][W], W = H + I + 1: columns [dW_hh | dW_ih | db].
struct ParamSums {
  const float* x;              // [T][B][I]
  int I;                       // at most kMaxI
  float* part;                 // sample b's at part + b stride
  int stride;
};
constexpr int kMaxI = 4;

// Chain element c is tile T - 1 - c; its product is the gradient of row T - 2 - c (c = T - 1: of the initial state).
// n >= 1 elements.  Barrier m (0 .. M + 1, M chunks): from it on chunk m may be read, buffer m - 2 be written again,
// and the results of chunk m - 2 be stored.
template <bool GEN, bool PARAMS, bool STREAM = false>
__device__ __forceinline__ void walk(Lds& lds, const Weights& weights, int T, int B, int n, int b, const float* Jt, const float* h,
                                     const float* seed, float* G, float* g0, int* error, const ParamSums params) {
  float* const tiles = lds.tiles;
  float* const outs = lds.outs;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int M = (n + kChunk - 1) / kChunk;
  if (wave == 0) {
    const int R = lane >> 4, i = lane & 15, ic = i < kC ? i : 0;
    const int unit[2] = {unit_of(R >> 1, ic), unit_of(R & 1, ic)};
    int src[2], dst[2];
    src[0] = unit[0] * H, src[1] = unit[1] * H;
    const int last[2] = {src[0] + 16 + 2 * (R & 1), src[1] + 16 + 2 * (R >> 1)};
    src[0] += 8 * (R & 1), src[1] += 8 * (R >> 1);
#pragma unroll
    for (int f = 0; f < 2; ++f) dst[f] = i < kC ? unit[f] : H + (i & 3);
    float s = seed[unit[1]];                       // (A B A B)
    __builtin_amdgcn_s_setprio(3);
    float w[4][kC];
    auto fetch = [&](float (&to)[kC], const float* tile, int form) {
      const v4f x = *reinterpret_cast<const v4f*>(tile + src[form]), y = *reinterpret_cast<const v4f*>(tile + src[form] + 4);
      const v2f z = *reinterpret_cast<const v2f*>(tile + last[form]);
#pragma unroll
      for (int k = 0; k < 4; ++k) to[k] = x[k], to[4 + k] = y[k];
      to[8] = z[0], to[9] = z[1];
    };
    bare_barrier();
#pragma unroll
    for (int q = 0; q < 3; ++q) fetch(w[q], tiles + q * HH, q & 1);
    int at = 0;
    for (int m = 0; m < M; ++m) {
      const float* now = tiles + at * kChunk * HH;
      at = at == 2 ? 0 : at + 1;
      const float* then = tiles + at * kChunk * HH;
      float* out = outs + (m & 3) * kOutChunk;
#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        if (q == kChunk - 3) bare_barrier();       // chunk m + 1 is there
        fetch(w[(q + 3) & 3], q + 3 < kChunk ? now + (q + 3) * HH : then + (q + 3 - kChunk) * HH, (q + 3) & 1);
        __builtin_amdgcn_sched_barrier(0);         // not all of the chunk's reads at once
        s = q & 1 ? chain_product<1>(w[q & 3], s) : chain_product<0>(w[q & 3], s);
        out[q * kOutRow + dst[q & 1]] = s;
      }
    }
    lds_barrier();                                 // barrier M + 1
  } else if (wave <= kBring / 64) {
    const int p = tid - 64;
    size_t off[kPieces];                           // of the piece within its chunk's first tile's row, going down in time
    int el[kPieces];
    const size_t step = (size_t)B * (GEN ? H : HH);
    const float* arr = GEN ? h + (size_t)B * H : Jt;                     // h[t + 1] stands for tile t
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      const int e = p + kBring * k, pc = e % (HH / 4), j4 = pc % 5 * 4;
      el[k] = e / (HH / 4);
      off[k] = (size_t)b * (GEN ? H : HH) + (GEN ? j4 : 4 * pc);
    }
    auto load = [&](v4f (&to)[kPieces], int m) {
#pragma unroll
      for (int k = 0; k < kPieces; ++k) {
        int c = m * kChunk + el[k];
        c = c < n ? c : n - 1;                     // past the end: any tile
        const v4f* from = reinterpret_cast<const v4f*>(arr + (size_t)(T - 1 - c) * step + off[k]);
        to[k] = STREAM ? __builtin_nontemporal_load(from) : *from;
      }
    };
    auto put = [&](const v4f (&from)[kPieces], int buf) {
      v4f* to = reinterpret_cast<v4f*>(tiles + buf * kChunk * HH) + p;
#pragma unroll
      for (int k = 0; k < kPieces; ++k) {
        v4f v = from[k];
        if (GEN) {
          // Jt[i][j] = W_hh[j][i] (1 - h[t+1][j]^2), the arithmetic of the builder
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = weights.v[k][u] * __builtin_fmaf(-v[u], v[u], 1.0f);
        }
        to[kBring * k] = v;
      }
    };
    v4f even[kPieces], odd[kPieces];
    load(even, 0);
    load(odd, 1);
    put(even, 0);
    load(even, 2);
    lds_barrier();                                 // barrier 0
    int buf = 1;
    for (int m = 1; m <= M; m += 2) {
      put(odd, buf);                               // chunk m (past the end: never read)
      buf = buf == 2 ? 0 : buf + 1;
      load(odd, m + 2);
      lds_barrier();
      if (m + 1 > M) break;
      put(even, buf);
      buf = buf == 2 ? 0 : buf + 1;
      load(even, m + 3);
      lds_barrier();
    }
    bare_barrier();                                // barrier M + 1
  } else if (!PARAMS || wave == kStorer) {
    if (lane < H) G[((size_t)(T - 1) * B + b) * H + lane] = seed[lane];
    if (b == 0 && lane == 0 && error) *error = 0;
    bare_barrier();
    bare_barrier();
    for (int m = 0; m < M; ++m) {
      bare_barrier();                              // barrier m + 2
      const float* out = outs + (m & 3) * kOutChunk;
#pragma unroll
      for (int k = 0; k < kChunk * H / 64; ++k) {
        const int e = lane + 64 * k, q = e / H, j = e - q * H, c = m * kChunk + q;
        const float v = out[q * kOutRow + j];
        float* to = c == T - 1 ? g0 + (size_t)b * H : G + ((size_t)(T - 2 - c) * B + b) * H;
        if (c < n) to[j] = v;
      }
    }
  } else {
    // The sums of 32 x 32, of which 20 x W are used, two steps to an issue of v_mfma_f32_32x32x2_f32: half the lanes
    // supply delta = (1 - h[t+1]^2) dL/dh[t+1] and [h[t] | x[t] | 1] of one step.  Chunk m stands for the steps of its
    // gradients, t = T - 2 - 16 m and below; the last step, whose gradient is the seed, comes first by itself.
    const int l32 = lane & 31, half = lane >> 5, I = params.I, W = H + I + 1, k = l32 - H;
    const float* const hb = h + (size_t)b * H + (l32 < H ? l32 : 0);
    const float* const xb = params.x + (size_t)b * I + (k >= 0 && k < I ? k : 0);
    const size_t hs = (size_t)B * H, xs = (size_t)B * I;
    const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    v16f acc = zero, sum = zero;
    struct Steps {
      float next[kChunk / 2], now[kChunk / 2], in[kChunk / 2];
    };
    // rows of a chunk from its last element up, as 32-bit offsets; the chunk that ends the sequence clamps them
    unsigned hoff[kChunk / 2], xoff[kChunk / 2];
#pragma unroll
    for (int q = 0; q < kChunk / 2; ++q) {
      hoff[q] = (unsigned)(kChunk - 1 - 2 * q - half) * (unsigned)hs;
      xoff[q] = (unsigned)(kChunk - 1 - 2 * q - half) * (unsigned)xs;
    }
    auto load = [&](Steps& to, int m) {
      const int t0 = T - 1 - kChunk - m * kChunk;
      if (t0 >= 0) {
        const float* const h0 = hb + (size_t)t0 * hs;
        const float* const x0 = xb + (size_t)t0 * xs;
#pragma unroll
        for (int q = 0; q < kChunk / 2; ++q) {
          to.now[q] = h0[hoff[q]];
          to.next[q] = h0[hoff[q] + (unsigned)hs];
          to.in[q] = x0[xoff[q]];
        }
      } else {
#pragma unroll
        for (int q = 0; q < kChunk / 2; ++q) {
          const int r = t0 + kChunk - 1 - 2 * q - half, t = r > 0 ? r : 0;
          to.now[q] = hb[(size_t)t * hs];
          to.next[q] = hb[(size_t)(t + 1) * hs];
          to.in[q] = xb[(size_t)t * xs];
        }
      }
    };
    auto column = [&](float now, float in) { return l32 < H ? now : k < I ? in : k == I ? 1.f : 0.f; };
    auto delta = [&](float g, float next) { return l32 < H ? (1.0f - next * next) * g : 0.f; };
    Steps steps[3];                                // requested two chunks (1.8 us) ahead
    load(steps[0], 0);
    load(steps[1], 1);
    {
      const float g = l32 < H ? seed[l32] : 0.f, next = hb[(size_t)T * hs], now = hb[(size_t)(T - 1) * hs];
      const float a = half == 0 ? delta(g, next) : 0.f, u = half == 0 ? column(now, xb[(size_t)(T - 1) * xs]) : 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, u, acc, 0, 0, 0);
    }
    bare_barrier();
    bare_barrier();
    auto chunk = [&](const Steps& cur, int m) {
      bare_barrier();                              // barrier m + 2
      const float* out = outs + (m & 3) * kOutChunk + half * kOutRow + (l32 < H ? l32 : 0);
#pragma unroll
      for (int q = 0; q < kChunk / 2; ++q) {
        const bool in = m * kChunk + 2 * q + half < T - 1;          // chain element T - 1 is the initial state's
        const float g = out[2 * q * kOutRow];
        const float a = in ? delta(g, cur.next[q]) : 0.f, u = in ? column(cur.now[q], cur.in[q]) : 0.f;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, u, acc, 0, 0, 0);
      }
    };
    for (int m = 0; m < M; m += 3) {
      if (m % 24 == 21) {                          // not too many terms in a row
        sum += acc;
        acc = zero;
      }
      load(steps[2], m + 2);
      chunk(steps[0], m);
      if (m + 1 >= M) break;
      load(steps[0], m + 3);
      chunk(steps[1], m + 1);
      if (m + 2 >= M) break;
      load(steps[1], m + 4);
      chunk(steps[2], m + 2);
    }
    sum += acc;
    float* to = params.part + (size_t)b * params.stride;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = 8 * (v >> 2) + 4 * half + (v & 3);
      if (i < H && l32 < W) to[i * W + l32] = sum[v];
    }
  }
}

}  // namespace chain_h20
}  // namespace
