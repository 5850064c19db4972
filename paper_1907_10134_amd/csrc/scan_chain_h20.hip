// Scan for H = 20 as what it is a bracketing of: one matrix-vector product after the other, a workgroup per
// sample.  It does a twentieth of the arithmetic of the tree of products and reads every tile once, but its T
// steps wait for one another, so it is the form for chains that are short or for batches that fill the chip by
// themselves; bppsa_chain_h20_us says what it costs.
//
// Seven waves share the work so that the one that walks the chain never waits for memory:
//   wave 0       the chain.  Rows and columns of a tile are cut in halves A and B of ten.  On even steps the four
//                rows of 16 lanes hold (rows, columns) = (A, A) (A, B) (B, A) (B, B): ten multiply-adds with the
//                vector as DPP operand, and one v_permlane16_swap adds the two column halves.  That leaves the
//                vector as (A A B B), which is what the transposed assignment (A, A) (B, A) (A, B) (B, B) of the
//                odd steps needs; its v_permlane32_swap gives back (A B A B).  Tile rows come from LDS, three
//                steps ahead;
//   waves 1..5   bring tiles into LDS in chunks of 16: read from memory two chunks ahead, or formed from the
//                hidden states and W_hh (tanh RNN) by the arithmetic of the builder, so that both sources give
//                the same bits;
//   wave 6       stores the gradients, so that no load ever waits behind a store.
// One barrier per chunk.
#include "bppsa_internal.h"
#include "scan_plan.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int H = 20;
constexpr int HH = H * H;
constexpr int kC = H / 2;
constexpr int kChunk = 16;
constexpr int kBring = 320;                       // threads that bring tiles: five pieces of 16 bytes per chunk each
constexpr int kPieces = kChunk * HH / 4 / kBring;
constexpr int kThreads = 64 + kBring + 64;
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

// a barrier that waits for nothing but what the caller says
__device__ __forceinline__ void bare_barrier() { asm volatile("s_barrier" ::: "memory"); }
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Chain element c is tile T - 1 - c; its product is the gradient of row T - 2 - c (c = T - 1: of the initial state).
// n >= 1 elements.  Barrier m (0 .. M + 1, M chunks): from it on chunk m may be read, buffer m - 2 be written again,
// and the results of chunk m - 2 be stored.
template <bool GEN>
__global__ void __launch_bounds__(kThreads)
chain_h20_kernel(int T, int B, int n, const float* __restrict__ Jt, const float* __restrict__ h,
                 const float* __restrict__ w_hh, const float* __restrict__ seed, float* __restrict__ G,
                 float* __restrict__ g0, int* __restrict__ error) {
  __shared__ __attribute__((aligned(16))) float tiles[3 * kChunk * HH];
  __shared__ __attribute__((aligned(16))) float outs[4 * kOutChunk];
  const int b = blockIdx.x, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
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
    float s = seed[(size_t)b * H + unit[1]];       // (A B A B)
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
    v4f wv[kPieces];
    size_t off[kPieces];                           // of the piece within its chunk's first tile's row, going down in time
    int el[kPieces];
    const size_t step = (size_t)B * (GEN ? H : HH);
    const float* arr = GEN ? h + (size_t)B * H : Jt;                     // h[t + 1] stands for tile t
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      const int e = p + kBring * k, pc = e % (HH / 4), row = pc / 5, j4 = (pc - row * 5) * 4;
      el[k] = e / (HH / 4);
      off[k] = (size_t)b * (GEN ? H : HH) + (GEN ? j4 : 4 * pc);
      if (GEN) {
#pragma unroll
        for (int u = 0; u < 4; ++u) wv[k][u] = w_hh[(j4 + u) * H + row];
      }
    }
    auto load = [&](v4f (&to)[kPieces], int m) {
#pragma unroll
      for (int k = 0; k < kPieces; ++k) {
        int c = m * kChunk + el[k];
        c = c < n ? c : n - 1;                     // past the end: any tile
        to[k] = *reinterpret_cast<const v4f*>(arr + (size_t)(T - 1 - c) * step + off[k]);
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
          for (int u = 0; u < 4; ++u) v[u] = wv[k][u] * __builtin_fmaf(-v[u], v[u], 1.0f);
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
  } else {
    if (lane < H) G[((size_t)(T - 1) * B + b) * H + lane] = seed[(size_t)b * H + lane];
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
  }
}

}  // namespace

bppsa_status bppsa_chain_h20(int T, int B, const float* Jt, const float* seed, float* G, float* g0, int* error,
                             hipStream_t stream, const float* h, const float* w_hh) {
  const int n = g0 ? T : T - 1;
  if (n < 1) return BPPSA_EINVAL;
  if (Jt) chain_h20_kernel<false><<<B, kThreads, 0, stream>>>(T, B, n, Jt, nullptr, nullptr, seed, G, g0, error);
  else chain_h20_kernel<true><<<B, kThreads, 0, stream>>>(T, B, n, nullptr, h, w_hh, seed, G, g0, error);
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
