// One training iteration of the tanh RNN of Section 4.1 on a mini-batch, as one call: forward
// recurrence, softmax cross-entropy head, the backward pass as a scan (Section 3.1) with its
// parameter gradients (Eq. 2), and an Adam update of every parameter (learning rate 1e-5 in the
// paper's runs).  The call chains the parts of the library's own entry points on the caller's stream.  A launch costs
// about 4.5 us on its own, so what is small rides along: the head's seed and each sample's share of the head's
// parameter gradients with the forward launch (H <= 32), the optimiser step with the last sum of the gradients; and at
// H = 20 sequences that are walked in one go both ways take one launch for everything before that sum
// (train_walk_h20.hip).
#include <cmath>

#include "scan_plan.h"
#include "train_parts.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// Softmax cross-entropy head with all its gradients, by one workgroup of sixteen waves.  Everything is a small product
// on the matrix cores (v_mfma_f32_16x16x4_f32) with operands in LDS, where [h_T | 1] and [W_out | b_out] are copied
// first (rows of odd length: consecutive rows in different banks):
//   logits   a wave per 16 samples; the log-sum-exp is an exchange between the 16 lanes that hold a sample's classes;
//   seed     dL/dh_T = dz W_out, a wave per tile of 16 x 16;
//   dW_out, db_out = dz^T [h_T | 1], the samples dealt to several waves per tile where tiles are few, whose sums are
//            added in a fixed order: the same bits on every run.
// What is left is latency.  (B = 256, H = 20, C = 10: 75 us with a wave per sample and one thread per entry of dW_out;
// 14 us with all threads on scalar products out of LDS, which one compute unit cannot issue faster.)
constexpr int kHeadThreads = 1024;
constexpr int kHeadWaves = kHeadThreads / 64;

struct HeadShape {
  int B, H, C;
  int ct;                      // tiles of 16 classes
  int pitch, dpitch;           // floats per row of [h_T | 1 | 0] and [W_out | b_out | 0], of dz
  int parts;                   // waves per tile of dW_out
  bool staged;                 // whether it all fits into LDS; otherwise head_plain
};
size_t head_lds(const HeadShape& s) {
  const size_t bp = bppsa_align_up((size_t)s.B, 16);
  if (!s.staged) return ((size_t)s.B * (s.C + 1) + kHeadThreads) * sizeof(float);
  return ((bp + 16 * s.ct) * s.pitch + bp * (s.dpitch + 1) + s.B + 16 + (s.parts > 1 ? kHeadWaves * 256 : 0)) * sizeof(float);
}
HeadShape head_shape(int B, int H, int C) {
  HeadShape s = {B, H, C, (C + 15) / 16, (H + 4) / 4 * 4 + 1, 0, 1, true};
  s.dpitch = 16 * s.ct + 1;
  const int tiles = s.ct * ((H + 16) / 16), most = (B + 15) / 16;
  s.parts = tiles < kHeadWaves ? kHeadWaves / tiles : 1;
  if (s.parts > most) s.parts = most;
  s.staged = (size_t)B * (H + 4) <= 32768 && (size_t)H * C <= 16384 && head_lds(s) <= 150 * 1024;
  return s;
}

// rows x 16-column product tile: a(row, k), b(k, column), k < 4 steps
template <class FA, class FB>
__device__ __forceinline__ v4f head_tile(int steps, FA&& a, FB&& b) {
  const int l16 = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
  v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int k = 0; k < steps; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a(l16, 4 * k + q), b(4 * k + q, l16), acc, 0, 0, 0);
  return acc;
}

// emit(c, j, v): v = dW_out[c][j], j < H; emit(c, H, v): v = db_out[c].  seed, loss may be null.
template <class F>
__device__ __forceinline__ void head_staged(const HeadShape s, float* lds, const float* __restrict__ h_last,
                                            const float* __restrict__ w_out, const float* __restrict__ b_out,
                                            const int32_t* __restrict__ labels, float* __restrict__ seed,
                                            float* __restrict__ loss, F&& emit) {
  const int B = s.B, H = s.H, C = s.C, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), bt = (B + 15) / 16, jt = (H + 16) / 16;
  float* w = lds;                                  // [16 ct][pitch]
  float* h = w + 16 * s.ct * s.pitch;              // [16 bt][pitch]
  float* dz = h + 16 * bt * s.pitch;               // [16 bt][dpitch]
  int* ys = reinterpret_cast<int*>(dz + 16 * bt * s.dpitch);                      // [16 bt] labels
  float* lb = dz + 16 * bt * (s.dpitch + 1);       // [B] per-sample loss, then what a tile reads past the end
  float* red = lb + B + 16;                        // [16 waves][256]
  const int nw = 16 * s.ct * s.pitch, nh = 16 * bt * s.pitch, most = nw > nh ? nw : nh;
  // the copies in trips of nine loads per thread, all in flight at once
  for (int e0 = tid; e0 < most; e0 += 4 * kHeadThreads) {
    float wv[4], hv[4];
    const int y = labels[e0 < B ? e0 : B - 1];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * kHeadThreads, r = e / s.pitch, j = e - r * s.pitch;
      const bool in_w = r < C && j <= H, in_h = r < B && j < H;
      wv[u] = *(in_w && j < H ? w_out + (size_t)r * H + j : b_out + (in_w ? r : 0));
      hv[u] = h_last[in_h ? (size_t)r * H + j : 0];
      wv[u] = in_w ? wv[u] : 0.f;
      hv[u] = in_h ? hv[u] : (r < B && j == H ? 1.f : 0.f);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * kHeadThreads;
      if (e < nw) w[e] = wv[u];
      if (e < nh) h[e] = hv[u];
    }
    if (e0 < 16 * bt) ys[e0] = y;
  }
  for (int b = tid + kHeadThreads; b < 16 * bt; b += kHeadThreads) ys[b] = labels[b < B ? b : B - 1];
  __syncthreads();
  const float invB = 1.0f / (float)B;
  for (int t = wave; t < bt; t += kHeadWaves) {
    v4f z[4];
    float m[4], lse[4];
    int y[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int b = 16 * t + 4 * q + v;
      y[v] = ys[b];
      m[v] = -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u < s.ct) {
        z[u] = head_tile((H + 4) / 4, [&](int r, int k) { return h[(16 * t + r) * s.pitch + k]; },
                         [&](int k, int c) { return w[(16 * u + c) * s.pitch + k]; });
#pragma unroll
        for (int v = 0; v < 4; ++v) m[v] = 16 * u + l16 < C ? fmaxf(m[v], z[u][v]) : m[v];
      }
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
      for (int v = 0; v < 4; ++v) m[v] = fmaxf(m[v], __shfl_xor(m[v], off, 64));
#pragma unroll
    for (int v = 0; v < 4; ++v) lse[v] = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < s.ct && 16 * u + l16 < C) {
#pragma unroll
        for (int v = 0; v < 4; ++v) lse[v] += expf(z[u][v] - m[v]);
      }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
      for (int v = 0; v < 4; ++v) lse[v] += __shfl_xor(lse[v], off, 64);
#pragma unroll
    for (int v = 0; v < 4; ++v) lse[v] = m[v] + logf(lse[v]);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < s.ct) {
        const int c = 16 * u + l16;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int b = 16 * t + 4 * q + v;
          const bool in = b < B && c < C;
          dz[b * s.dpitch + c] = in ? (expf(z[u][v] - lse[v]) - (c == y[v] ? 1.f : 0.f)) * invB : 0.f;
          if (in && c == y[v]) lb[b] = lse[v] - z[u][v];
        }
      }
  }
  __syncthreads();
  if (seed) {
    const int ht = (H + 15) / 16;
    for (int t = wave; t < bt * ht; t += kHeadWaves) {
      const int tb = t / ht, j = 16 * (t - tb * ht);
      const v4f g = head_tile((C + 3) / 4, [&](int r, int k) { return dz[(16 * tb + r) * s.dpitch + k]; },
                              [&](int k, int c) { return w[k * s.pitch + j + c]; });
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int b = 16 * tb + 4 * q + v;
        if (b < B && j + l16 < H) seed[(size_t)b * H + j + l16] = g[v];
      }
    }
  }
  // tile t of dW_out is classes 16 (t / jt) .., columns 16 (t % jt) ..; part p of it takes its share of the samples
  const int tiles = s.ct * jt, share = 4 * ((4 * bt + s.parts - 1) / s.parts);
  for (int t = wave; t < tiles * s.parts; t += kHeadWaves) {
    const int tile = t / s.parts, p = t - tile * s.parts, u = tile / jt, j = 16 * (tile - u * jt), b0 = p * share;
    const int left = 16 * bt - b0, take = left < share ? left : share;
    const v4f g = head_tile(take > 0 ? take / 4 : 0, [&](int r, int k) { return dz[(b0 + k) * s.dpitch + 16 * u + r]; },
                            [&](int k, int c) { return h[(b0 + k) * s.pitch + j + c]; });
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 * u + 4 * q + v;
      if (s.parts > 1) red[t * 256 + 16 * (4 * q + v) + l16] = g[v];
      else if (c < C && j + l16 <= H) emit(c, j + l16, g[v]);
    }
  }
  if (s.parts > 1) {
    __syncthreads();
    for (int e = tid; e < tiles * 256; e += kHeadThreads) {
      const int tile = e >> 8, u = tile / jt, c = 16 * u + ((e >> 4) & 15), j = 16 * (tile - u * jt) + (e & 15);
      const float* r = red + tile * s.parts * 256 + (e & 255);
      float g = r[0];
      for (int p = 1; p < s.parts; ++p) g += r[p * 256];
      if (c < C && j <= H) emit(c, j, g);
    }
  }
  if (loss && wave == 0) {
    float acc = 0.f;
    for (int b = lane; b < B; b += 64) acc += lb[b];
    acc = bppsa_wave_sum(acc);
    if (lane == 0) *loss = acc * invB;
  }
}

// The same for heads too large for LDS, a thread per logit, per entry of the seed and per entry of dW_out.
template <class F>
__device__ __forceinline__ void head_plain(const HeadShape s, float* lds, const float* __restrict__ h,
                                           const float* __restrict__ w, const float* __restrict__ b_out,
                                           const int32_t* __restrict__ labels, float* __restrict__ seed,
                                           float* __restrict__ loss, F&& emit) {
  const int B = s.B, H = s.H, C = s.C, tid = threadIdx.x;
  float* dz = lds;                  // [B][C] logits, then dL/dz
  float* lb = dz + B * C;           // [B] per-sample loss
  const float invB = 1.0f / (float)B;
  for (int e = tid; e < B * C; e += kHeadThreads) {
    const int b = e / C, c = e - b * C;
    float acc = b_out[c];
    for (int j = 0; j < H; ++j) acc += w[(size_t)c * H + j] * h[(size_t)b * H + j];
    dz[e] = acc;
  }
  __syncthreads();
  for (int b = tid; b < B; b += kHeadThreads) {
    float* z = dz + b * C;
    const int y = labels[b];
    float m = z[0], sum = 0.f;
    for (int k = 1; k < C; ++k) m = fmaxf(m, z[k]);
    for (int k = 0; k < C; ++k) sum += expf(z[k] - m);
    const float lse = m + logf(sum);
    lb[b] = lse - (y >= 0 && y < C ? z[y] : 0.f);
    for (int k = 0; k < C; ++k) z[k] = (expf(z[k] - lse) - (k == y ? 1.f : 0.f)) * invB;
  }
  __syncthreads();
  if (seed) {
    for (size_t e = tid; e < (size_t)B * H; e += kHeadThreads) {
      const int b = (int)(e / H), j = (int)(e - (size_t)b * H);
      float acc = 0.f;
      for (int k = 0; k < C; ++k) acc += dz[b * C + k] * w[(size_t)k * H + j];
      seed[e] = acc;
    }
  }
  for (int e = tid; e < C * (H + 1); e += kHeadThreads) {
    const int c = e / (H + 1), j = e - c * (H + 1);
    float acc = 0.f;
    for (int b = 0; b < B; ++b) acc += dz[b * C + c] * (j < H ? h[(size_t)b * H + j] : 1.f);
    emit(c, j, acc);
  }
  if (loss && tid < 64) {
    float acc = 0.f;
    for (int b = tid; b < B; b += 64) acc += lb[b];
    acc = bppsa_wave_sum(acc);
    if (tid == 0) *loss = acc * invB;
  }
}

template <class F>
__device__ __forceinline__ void head_all(const HeadShape s, float* lds, const float* __restrict__ h_last,
                                         const float* __restrict__ w_out, const float* __restrict__ b_out,
                                         const int32_t* __restrict__ labels, float* __restrict__ seed,
                                         float* __restrict__ loss, F&& emit) {
  if (s.staged) head_staged(s, lds, h_last, w_out, b_out, labels, seed, loss, emit);
  else head_plain(s, lds, h_last, w_out, b_out, labels, seed, loss, emit);
}

__global__ void __launch_bounds__(kHeadThreads)
head_backward_kernel(const HeadShape s, const float* __restrict__ h_last, const float* __restrict__ w_out,
                     const float* __restrict__ b_out, const int32_t* __restrict__ labels,
                     float* __restrict__ seed, float* __restrict__ loss, float* __restrict__ dW_out,
                     float* __restrict__ db_out) {
  extern __shared__ float lds[];
  head_all(s, lds, h_last, w_out, b_out, labels, seed, loss, [&](int c, int j, float v) {
    if (j < s.H) {
      if (dW_out) dW_out[(size_t)c * s.H + j] = v;
    } else if (db_out) {
      db_out[c] = v;
    }
  });
}

// Adam (Kingma & Ba, Algorithm 1).  1 - beta and the bias corrections c1 = 1 / (1 - beta1^t),
// c2 = 1 / (1 - beta2^t) are formed on the host in double precision and rounded once.
struct Adam {
  float* theta;
  float* m;
  float* v;
  float lr, beta1, one_minus_beta1, beta2, one_minus_beta2, eps, c1, c2;
  struct Entry {
    float theta, m, v;
  };
  // an entry can be fetched while its gradient is still on its way
  __device__ __forceinline__ Entry fetch(size_t i) const { return {theta[i], m[i], v[i]}; }
  __device__ __forceinline__ void update(size_t i, float gi, const Entry& was) const {
    const float mi = beta1 * was.m + one_minus_beta1 * gi;
    const float vi = beta2 * was.v + one_minus_beta2 * gi * gi;
    m[i] = mi;
    v[i] = vi;
    theta[i] = was.theta - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
  }
  __device__ __forceinline__ void update(size_t i, float gi) const { update(i, gi, fetch(i)); }
};

Adam make_adam(float* theta, float* m, float* v, int step, double lr, double beta1, double beta2, double eps) {
  const float c1 = (float)(1.0 / (1.0 - std::pow(beta1, (double)step)));
  const float c2 = (float)(1.0 / (1.0 - std::pow(beta2, (double)step)));
  return Adam{theta, m, v, (float)lr, (float)beta1, (float)(1.0 - beta1), (float)beta2, (float)(1.0 - beta2), (float)eps, c1, c2};
}

__global__ void __launch_bounds__(256)
adam_kernel(int n, const float* __restrict__ g, const Adam adam) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) adam.update(i, g[i]);
}

// Where the parameters lie in the flat layout: W_ih | W_hh | b_ih | b_hh | W_out | b_out.
struct Offsets {
  size_t whh, bih, bhh, wout, bout, all;
};
Offsets offsets_of(int H, int I, int C) {
  Offsets o;
  o.whh = (size_t)H * I, o.bih = o.whh + (size_t)H * H, o.bhh = o.bih + H, o.wout = o.bhh + H;
  o.bout = o.wout + (size_t)C * H, o.all = o.bout + C;
  return o;
}

// The end of an iteration: the last sum of the cell's parameter gradients, 64 entries to a workgroup, and one more
// workgroup for the head's parameters - their gradients too unless they are there already (with_head = false) - each
// entry updated by the thread that has its gradient.
__global__ void __launch_bounds__(kHeadThreads)
train_finish_kernel(const HeadShape s, const Offsets o, int I, int nparts, const float* __restrict__ part, bool with_head,
                    const float* __restrict__ h_last, const int32_t* __restrict__ labels, float* __restrict__ grads,
                    float* __restrict__ loss, const Adam adam) {
  static_assert(kHeadThreads == 64 * kFinishWaves, "one launch for both");
  extern __shared__ float lds[];
  __shared__ float red[kFinishWaves][64];
  const int H = s.H, W = H + I + 1, E = H * W;
  auto give = [&](size_t i, float g) {
    grads[i] = g;
    adam.update(i, g);
  };
  if (blockIdx.x == 0) {
    if (with_head) {
      // W_out and b_out change only after every thread has read them: no gradient is given before the barrier behind
      // the logits
      head_all(s, lds, h_last, adam.theta + o.wout, adam.theta + o.bout, labels, nullptr, loss,
               [&](int c, int j, float v) { give(j < H ? o.wout + (size_t)c * H + j : o.bout + c, v); });
    } else {
      for (size_t i = o.wout + threadIdx.x; i < o.all; i += kHeadThreads) adam.update(i, grads[i]);
    }
    return;
  }
  const int first = (blockIdx.x - 1) * 64, e = first + (int)(threadIdx.x & 63), r = e < E ? e / W : 0, c = e - r * W;
  const size_t i = e >= E ? 0 : c < H ? o.whh + (size_t)r * H + c : c < H + I ? (size_t)r * I + (c - H) : o.bih + r;
  const size_t i2 = e < E && c == H + I ? o.bhh + r : i;      // both bias vectors have this gradient
  Adam::Entry was = {}, was2 = {};
  if (threadIdx.x < 64) was = adam.fetch(i), was2 = adam.fetch(i2);
  const float t = bppsa_add_partials(nparts, E, E, first, part, red);
  if (threadIdx.x >= 64 || e >= E) return;
  grads[i] = t;
  adam.update(i, t, was);
  if (i2 != i) {
    grads[i2] = t;
    adam.update(i2, t, was2);
  }
}

// The same where the samples' shares of the head's gradients are there too: sums only.  4 us against 6.4 with the head
// in a workgroup of this launch (B = 16), 5 against 11 (B = 256).
struct Shares {
  const float* part;
  int count, stride;
};
__global__ void __launch_bounds__(kHeadThreads)
train_sum_kernel(const Offsets o, int H, int I, int C, const Shares cell, const Shares head, float* __restrict__ grads,
                 float* __restrict__ loss, const Adam adam) {
  __shared__ float red[kFinishWaves][64];
  const int W = H + I + 1, E = H * W, cell_groups = (E + 63) / 64, entries = C * (H + 1) + 1;
  const bool of_cell = (int)blockIdx.x < cell_groups;
  const int first = 64 * (of_cell ? blockIdx.x : blockIdx.x - cell_groups), e = first + (int)(threadIdx.x & 63);
  const bool is_loss = !of_cell && e == entries - 1, live = of_cell ? e < E : e < entries - 1;
  size_t i = 0, i2 = 0;                            // both bias vectors of the cell have one gradient
  if (live && of_cell) {
    const int r = e / W, c = e - r * W;
    i2 = i = c < H ? o.whh + (size_t)r * H + c : c < H + I ? (size_t)r * I + (c - H) : o.bih + r;
    if (c == H + I) i2 = o.bhh + r;
  } else if (live) {
    const int r = e / (H + 1), c = e - r * (H + 1);
    i2 = i = c < H ? o.wout + (size_t)r * H + c : o.bout + r;
  }
  Adam::Entry was = {}, was2 = {};
  if (threadIdx.x < 64) was = adam.fetch(i), was2 = adam.fetch(i2);
  const Shares& s = of_cell ? cell : head;
  const float t = bppsa_add_partials(s.count, of_cell ? E : entries, s.stride, first, s.part, red);
  if (threadIdx.x >= 64) return;
  if (live) {
    grads[i] = t;
    adam.update(i, t, was);
    if (i2 != i) {
      grads[i2] = t;
      adam.update(i2, t, was2);
    }
  } else if (is_loss && loss) {
    *loss = t;
  }
}

bppsa_status allow_head_lds(const void* kernel, size_t lds) {
  if (lds > 48 * 1024) BPPSA_HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  return BPPSA_OK;
}
bool head_fits(int B, int C) { return C <= 64 && ((size_t)B * C + (size_t)B) * sizeof(float) <= 48 * 1024; }

}  // namespace

extern "C" bppsa_status bppsa_head_backward(int B, int H, int C, const float* h_last, const float* w_out,
                                            const float* b_out, const int32_t* labels, float* seed, float* loss,
                                            float* dW_out, float* db_out, void* stream) {
  if (!h_last || !w_out || !b_out || !labels || !seed) return BPPSA_EINVAL;
  if (B < 1 || H < 1 || C < 1) return BPPSA_EINVAL;
  if (!head_fits(B, C)) return BPPSA_ESHAPE;
  const HeadShape s = head_shape(B, H, C);
  const size_t lds = head_lds(s);
  BPPSA_TRY(allow_head_lds((const void*)head_backward_kernel, lds));
  head_backward_kernel<<<1, kHeadThreads, lds, (hipStream_t)stream>>>(s, h_last, w_out, b_out, labels, seed, loss,
                                                                      dW_out, db_out);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

extern "C" bppsa_status bppsa_adam_step(int64_t n, float* theta, const float* grad, float* m, float* v, int step,
                                        double lr, double beta1, double beta2, double eps, void* stream) {
  if (!theta || !grad || !m || !v) return BPPSA_EINVAL;
  if (n < 1 || step < 1 || n > INT32_MAX - 256) return BPPSA_EINVAL;
  if (!(beta1 >= 0. && beta1 < 1.) || !(beta2 >= 0. && beta2 < 1.)) return BPPSA_EINVAL;
  adam_kernel<<<bppsa_ceil_div((int)n, 256), 256, 0, (hipStream_t)stream>>>(
      (int)n, grad, make_adam(theta, m, v, step, lr, beta1, beta2, eps));
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

extern "C" size_t bppsa_rnn_param_count(int H, int I, int C) {
  if (H < 1 || I < 1 || C < 1) return 0;
  return (size_t)H * I + (size_t)H * H + 2 * (size_t)H + (size_t)C * H + (size_t)C;
}

// The scan's part comes first and stays untouched by the later calls, so its error word (the
// first four bytes, H = 20) can still be read after the iteration.
static size_t train_scan_ws_bytes(int T, int B, int H) { return bppsa_align_up(bppsa_scan_workspace_bytes(T, B, H), 256); }

// What a call needs, and what the query asks for: room for the samples' shares of the gradients as well, behind the rest
// (those of the head, for up to 16 classes) or over it where one launch walks both ways.
static size_t train_ws_least(int T, int B, int H, int I) {
  return train_scan_ws_bytes(T, B, H) + bppsa_param_grads_workspace_bytes(BPPSA_RNN_TANH, T, B, H, I);
}
static size_t head_shares_bytes(int B, int H, int C) { return (size_t)B * bppsa_head_entries(H, C) * sizeof(float); }
static size_t walk_shares_bytes(int B, int I, int C) {
  return 256 + (size_t)B * bppsa_walk_entries(I, C) * sizeof(float);
}
extern "C" size_t bppsa_rnn_train_workspace_bytes(int T, int B, int H, int I) {
  const size_t least = train_ws_least(T, B, H, I);
  if (least == 0 || H > 32 || I > 4) return least;
  const size_t more = least + head_shares_bytes(B, H, 16), walk = H == 20 ? walk_shares_bytes(B, I, 16) : 0;
  return walk > more ? walk : more;
}

extern "C" bppsa_status bppsa_rnn_train_step(int T, int B, int H, int I, int C, const float* x,
                                             const int32_t* labels, const bppsa_rnn_train_state* st, int step,
                                             double lr, double beta1, double beta2, double eps, void* stream) {
  if (!x || !labels || !st) return BPPSA_EINVAL;
  if (!st->params || !st->grads || !st->adam_m || !st->adam_v || !st->h || !st->G || !st->seed || !st->workspace)
    return BPPSA_EINVAL;
  if (T < 1 || B < 1 || H < 1 || I < 1 || C < 1 || step < 1) return BPPSA_EINVAL;
  if (st->workspace_bytes < train_ws_least(T, B, H, I)) return BPPSA_EWORKSPACE;
  if (!(beta1 >= 0. && beta1 < 1.) || !(beta2 >= 0. && beta2 < 1.)) return BPPSA_EINVAL;
  if (bppsa_mul_overflows((int64_t)T + 1, B, H, H) || bppsa_mul_overflows(T, B, I, 1)) return BPPSA_EOVERFLOW;
  if (!head_fits(B, C)) return BPPSA_ESHAPE;
  const Offsets o = offsets_of(H, I, C);
  const float* p = st->params;
  float* g = st->grads;
  const float* h_last = st->h + (size_t)T * B * H;
  hipStream_t s = (hipStream_t)stream;
  const size_t scan_bytes = train_scan_ws_bytes(T, B, H);
  void* pg_ws = static_cast<char*>(st->workspace) + scan_bytes;
  const size_t pg_bytes = st->workspace_bytes - scan_bytes;
  // H = 20: the scan's own entry, whose zeroed words are left to the forward launch
  const bool h20 = H == 20 && B <= 65535 && ((uintptr_t)st->workspace & 255) == 0;
  bppsa_forward_tail tail = {p + o.wout, p + o.bout, labels, st->seed, C, static_cast<int*>(st->workspace), 0, nullptr, nullptr, 0};
  const Adam adam = make_adam(st->params, st->adam_m, st->adam_v, step, lr, beta1, beta2, eps);
  auto sum_up = [&](const Shares& cell, const Shares& head) -> bppsa_status {
    const int groups = bppsa_ceil_div(H * (H + I + 1), 64) + bppsa_ceil_div(bppsa_head_entries(H, C), 64);
    train_sum_kernel<<<groups, kHeadThreads, 0, s>>>(o, H, I, C, cell, head, g, st->loss, adam);
    BPPSA_CHECK_LAUNCH();
    return BPPSA_OK;
  };
  // H = 20, walked in one go both ways: two launches.  The samples' shares lie behind the scan's error word, over
  // what the other forms use.
  if (h20 && T > 1 && I <= 4 && !st->Jt && st->workspace_bytes >= walk_shares_bytes(B, I, C) &&
      bppsa_prefer_chain_h20(T - 1, B) && bppsa_wave_walks_whole(T, B, H, I)) {
    const int stride = bppsa_walk_entries(I, C), cell = H * (H + I + 1);
    float* part = reinterpret_cast<float*>(static_cast<char*>(st->workspace) + 256);
    tail.share = part + cell, tail.share_stride = stride;
    BPPSA_TRY(bppsa_train_walk_h20(T, B, I, x, p, p + o.whh, p + o.bih, p + o.bhh, st->h, tail, st->G,
                                   static_cast<int*>(st->workspace), part, stride, s));
    return sum_up({part, B, stride}, {part + cell, B, stride});
  }
  if (st->workspace_bytes >= train_ws_least(T, B, H, I) + head_shares_bytes(B, H, C)) {
    tail.share = reinterpret_cast<float*>(static_cast<char*>(st->workspace) + train_ws_least(T, B, H, I));
    tail.share_stride = bppsa_head_entries(H, C);
  }
  if (h20) bppsa_h20_clears(T, B, false, st->workspace, &tail.words, &tail.w_hh_t);
  if (st->Jt) tail.w_hh_t = nullptr;
  const bppsa_status walked = bppsa_recurrence(BPPSA_RNN_TANH, T, B, H, I, x, p, p + o.whh, p + o.bih, p + o.bhh, st->h, s, &tail);
  const bool seeded = walked == BPPSA_OK;
  if (!seeded) {
    if (walked != BPPSA_EUNSUPPORTED) return walked;
    BPPSA_TRY(bppsa_forward(BPPSA_RNN_TANH, T, B, H, I, x, p, p + o.whh, p + o.bih, p + o.bhh, st->h, stream));
    BPPSA_TRY(bppsa_head_backward(B, H, C, h_last, p + o.wout, p + o.bout, labels, st->seed, st->loss, g + o.wout,
                                  g + o.bout, stream));
  }
  // the backward pass over the T steps as a scan; the seed is dL/dh_T (Eq. 5)
  if (st->Jt)
    BPPSA_TRY(bppsa_build_jacobians(BPPSA_RNN_TANH, T, B, H, I, st->h, nullptr, nullptr, p + o.whh, nullptr, nullptr,
                                    st->Jt, stream));
  if (h20)
    BPPSA_TRY(bppsa_any_scan_h20(T, B, st->Jt, st->seed, st->G, nullptr, st->workspace, s, st->h, p + o.whh, seeded));
  else if (st->Jt)
    BPPSA_TRY(bppsa_scan(T, B, H, st->Jt, st->seed, st->G, nullptr, st->workspace, scan_bytes, stream));
  else
    BPPSA_TRY(bppsa_rnn_scan_fused(T, B, H, st->h, p + o.whh, st->seed, st->G, nullptr, st->workspace, scan_bytes,
                                   stream));
  int nparts = 0;
  BPPSA_TRY(bppsa_rnn_param_partials(T, B, H, I, st->h, x, st->G, pg_ws, pg_bytes, &nparts, s));
  if (seeded && tail.share)
    return sum_up({static_cast<const float*>(pg_ws), nparts, H * (H + I + 1)}, {tail.share, B, tail.share_stride});
  const HeadShape hs = head_shape(B, H, C);
  const size_t lds = seeded ? head_lds(hs) : 0;
  BPPSA_TRY(allow_head_lds((const void*)train_finish_kernel, lds));
  train_finish_kernel<<<1 + bppsa_ceil_div(H * (H + I + 1), 64), kHeadThreads, lds, s>>>(
      hs, o, I, nparts, static_cast<const float*>(pg_ws), seeded, h_last, labels, g, st->loss,
      adam);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
