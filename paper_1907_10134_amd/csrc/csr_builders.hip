// Analytic generation of transposed Jacobians directly in CSR (Appendix D):
// 3x3 convolution (and the convolution of any kernel size, stride, padding and dilation), ReLU,
// 2x2 max-pooling and the fully connected layer.
// What a row pointer adds up is known in closed form where the layer allows it (3x3 convolution: nine
// counts per input channel; pooling: one entry per window); elsewhere it comes from a count pass and an
// exclusive prefix sum.  Column indices within a row ascend because candidates are enumerated in column
// order and compacted with wave-level prefix counts.
#include "bppsa_internal.h"
#include "sparse_common.h"

namespace {

// A mask that may be absent (everything kept), read without a branch: a load inside one is waited for on the
// spot, so a loop of them pays a memory latency each.  Without a mask the bytes read are the weights', which
// are at least as many, and do not count.
struct KeptBytes {
  const uint8_t* bytes;
  bool all;
  __device__ __forceinline__ KeptBytes(const uint8_t* mask, const float* weight)
      : bytes(mask ? mask : reinterpret_cast<const uint8_t*>(weight)), all(mask == nullptr) {}
};

// Candidate q of row (c, y, x) of a convolution Jacobian: q = co * 9 + tap, tap = (dy+1)*3 + (dx+1).
struct ConvCand {
  bool valid;
  int col;
  int widx;
};

__device__ __forceinline__ ConvCand conv_candidate(int q, int c, int y, int x, int ci, int h, int w,
                                                   const uint8_t* __restrict__ mask) {
  ConvCand r;
  const int co = q / 9, tap = q - co * 9;
  const int dy = tap / 3 - 1, dx = tap - (tap / 3) * 3 - 1;
  const int yy = y + dy, xx = x + dx;
  r.widx = ((co * ci + c) * 3 + (1 - dy)) * 3 + (1 - dx);
  r.col = co * h * w + yy * w + xx;
  r.valid = (yy >= 0) && (yy < h) && (xx >= 0) && (xx < w) && (mask == nullptr || mask[r.widx] != 0);
  return r;
}

// Indices and values of the 3x3 convolution, one wave per row, candidates tested one by one.
// For weights whose list (conv_fill_kernel) does not fit LDS.
__global__ void __launch_bounds__(256)
conv_rows_kernel(int ci, int co, int h, int w, const float* __restrict__ weight,
                 const uint8_t* __restrict__ mask, const int32_t* __restrict__ indptr,
                 int32_t* __restrict__ indices, float* __restrict__ data) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int rows = ci * h * w;
  if (row >= rows) return;
  const int c = row / (h * w);
  const int rem = row - c * h * w;
  const int y = rem / w, x = rem - y * w;
  const int ncand = co * 9;
  int count = indptr[row];
  for (int q0 = 0; q0 < ncand; q0 += 64) {
    const int q = q0 + lane;
    ConvCand cd;
    cd.valid = false;
    if (q < ncand) cd = conv_candidate(q, c, y, x, ci, h, w, mask);
    const unsigned long long bal = __ballot(cd.valid);
    if (cd.valid) {
      const int to = count + __popcll(bal & ((1ull << lane) - 1ull));
      indices[to] = cd.col;
      data[to] = weight[cd.widx];
    }
    count += __popcll(bal);
  }
}

// Row pointers of the 3x3 convolution.  With A[dy][dx] the number of kept weights of channel c that read
// neighbour (dy, dx), row (y, x) holds the sum of A over the neighbours inside the image, so every row
// pointer is a few multiplications away from the nine counts and the entries of the channels before.
// Up to kDirectRows rows: the row lengths, and their prefix sum.  Beyond: counts and total per channel, kept
// in the channel's own stretch of indptr (place 0: the total, 1 + tap: the counts; such an image has more
// than ten pixels); prefix sum of the totals; pointers.
// (Counting every row's candidates one by one took 30 us a layer of VGG-11, these take about 6.)
constexpr int kCountChannels = 16, kCountThreads = 1024, kDirectRows = 16384;
template <bool DIRECT>
__global__ void __launch_bounds__(kCountThreads)
conv_channel_counts_kernel(int ci, int co, int h, int w, const uint8_t* __restrict__ mask, int32_t* __restrict__ indptr) {
  // 144 (channel, tap) pairs: four to a thread where the mask's rows are whole words, 28 ways over co (18 loads
  // a thread for 512 output channels), else one to a thread, 7 ways
  constexpr int E = 9 * kCountChannels, SPLIT = 28;
  __shared__ int part[SPLIT][E];
  const int c0 = blockIdx.x * kCountChannels;
  const int here = (ci - c0 < kCountChannels ? ci - c0 : kCountChannels) * 9;       // pairs of this workgroup
  const size_t stride = (size_t)ci * 9;
  const bool words = (stride & 3) == 0 && ((uintptr_t)mask & 3) == 0;               // uniform
  const int ways = !mask ? 1 : words ? SPLIT : kCountThreads / E;
  if (!mask) {
    if (threadIdx.x < E) part[0][threadIdx.x] = (int)threadIdx.x < here ? co : 0;
  } else if (words) {
    const int e = (threadIdx.x % (E / 4)) * 4, s = threadIdx.x / (E / 4);
    if (s < SPLIT) {
      int n[4] = {0, 0, 0, 0};
      if (e < here) {                              // here is a multiple of 4 as well: ci is
        const uint8_t* m = mask + (size_t)c0 * 9 + e;
        for (int o0 = s; o0 < co; o0 += 10 * SPLIT) {      // ten loads at a time, past the end repeated and not counted
          uint32_t v[10];
#pragma unroll
          for (int k = 0; k < 10; ++k) {
            const int o = o0 + k * SPLIT;
            v[k] = *reinterpret_cast<const uint32_t*>(m + (size_t)(o < co ? o : o0) * stride);
          }
#pragma unroll
          for (int k = 0; k < 10; ++k)
#pragma unroll
            for (int u = 0; u < 4; ++u) n[u] += o0 + k * SPLIT < co && ((v[k] >> (8 * u)) & 0xffu) != 0;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) part[s][e + u] = n[u];
    }
  } else {
    const int e = threadIdx.x % E, s = threadIdx.x / E;
    if (s < kCountThreads / E) {
      int n = 0;
      if (e < here) {
        const uint8_t* m = mask + (size_t)c0 * 9 + e;
        for (int o0 = s; o0 < co; o0 += 10 * (kCountThreads / E)) {
          uint8_t v[10];
#pragma unroll
          for (int k = 0; k < 10; ++k) {
            const int o = o0 + k * (kCountThreads / E);
            v[k] = m[(size_t)(o < co ? o : o0) * stride];
          }
#pragma unroll
          for (int k = 0; k < 10; ++k) n += o0 + k * (kCountThreads / E) < co && v[k] != 0;
        }
      }
      part[s][e] = n;
    }
  }
  __syncthreads();
  if (threadIdx.x < E) {
    const int e = threadIdx.x;
    int n = 0;
    for (int k = 0; k < ways; ++k) n += part[k][e];
    part[0][e] = n;
    if (!DIRECT && e < here) indptr[(size_t)(c0 + e / 9) * h * w + 1 + e % 9] = n;
  }
  __syncthreads();
  if (DIRECT) {
    const int hw = h * w, rows = (ci - c0 < kCountChannels ? ci - c0 : kCountChannels) * hw;
    for (int r = threadIdx.x; r < rows; r += blockDim.x) {
      const int c = r / hw, i = r - c * hw, y = i / w, x = i - y * w;
      const int* A = part[0] + 9 * c;              // weight tap k reads neighbour (1 - k / 3, 1 - k % 3)
      int n = 0;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int yy = y + 1 - k / 3, xx = x + 1 - k % 3;
        n += (yy >= 0 && yy < h && xx >= 0 && xx < w) ? A[k] : 0;
      }
      indptr[(size_t)c0 * hw + r] = n;
    }
    return;
  }
  if (threadIdx.x < kCountChannels && c0 + (int)threadIdx.x < ci) {
    int total = 0;
    for (int tap = 0; tap < 9; ++tap) {
      const int dy = tap / 3 - 1, dx = tap % 3 - 1;
      total += part[0][threadIdx.x * 9 + tap] * (h - (dy != 0)) * (w - (dx != 0));
    }
    indptr[(size_t)(c0 + threadIdx.x) * h * w] = total;
  }
}

__global__ void __launch_bounds__(256)
conv_pointers_kernel(int h, int w, int32_t* __restrict__ indptr) {
  const int hw = h * w;
  int32_t* p = indptr + (size_t)blockIdx.x * hw;
  const int base = p[0];
  int A[3][3];                                     // [dy + 1][dx + 1]; weight tap (1 - dy, 1 - dx)
#pragma unroll
  for (int k = 0; k < 9; ++k) A[2 - k / 3][2 - k % 3] = p[1 + k];
  __syncthreads();                                 // everyone has read the counts: they may be overwritten
  int whole[3];                                    // entries of a whole image row through neighbours of row dy
#pragma unroll
  for (int d = 0; d < 3; ++d) whole[d] = w * A[d][1] + (w - 1) * (A[d][0] + A[d][2]);
  for (int i = threadIdx.x; i < hw; i += blockDim.x) {
    const int y = i / w, x = i - y * w;
    const int up = y > 0 ? 1 : 0, down = y + 1 < h ? 1 : 0;
    int n = base + y * whole[1] + (y > 0 ? y - 1 : 0) * whole[0] + (y < h - 1 ? y : h - 1) * whole[2];
    n += (x > 0 ? x - 1 : 0) * (up * A[0][0] + A[1][0] + down * A[2][0]) + x * (up * A[0][1] + A[1][1] + down * A[2][1]) +
         (x < w - 1 ? x : w - 1) * (up * A[0][2] + A[1][2] + down * A[2][2]);
    p[i] = n;
  }
}

// Indices and values of the 3x3 convolution.  The kept weights of an input channel are the same list for
// every pixel: a workgroup compacts it once into LDS (column offset, value, tap, in column order) and then
// writes the rows of its stretch of pixels, a wave per row: inside the image plain copies of the list with
// the pixel's position added, at the border the entries whose neighbour exists.  (Testing all 9 co
// candidates for every row took 50 us a layer of VGG-11 at 90 % pruned, this takes a tenth.)
constexpr size_t kConvListBytes = 64 * 1024;
constexpr int kFillWaves = 8, kMaxBatches = 16;
static_assert(kConvListBytes / 9 / kFillWaves + 9 <= 64 * kMaxBatches, "a wave's share of the longest list");
__global__ void __launch_bounds__(64 * kFillWaves)
conv_fill_kernel(int ci, int co, int h, int w, int pixels_per_group, const float* __restrict__ weight,
                 const uint8_t* __restrict__ mask, const int32_t* __restrict__ indptr, int32_t* __restrict__ indices,
                 float* __restrict__ data) {
  extern __shared__ __attribute__((aligned(8))) unsigned char conv_lds[];
  __shared__ int share[kFillWaves];
  const int cand = co * 9;
  int2* list = reinterpret_cast<int2*>(conv_lds);                     // (column offset, bits of the value)
  uint8_t* taps = conv_lds + (size_t)cand * sizeof(int2);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hw = h * w;
  // The weights of neighbouring channels share cache lines: workgroups that the dispatcher puts on one
  // compute die (ids equal modulo 8) take a contiguous eighth of the channels, so that a die's L2 fetches
  // an eighth of the weights instead of all of them.
  const int groups = (hw + pixels_per_group - 1) / pixels_per_group;
  const int share_of_die = (ci + 7) / 8, turn = blockIdx.x >> 3;
  const int c = (blockIdx.x & 7) * share_of_die + turn / groups;
  if (turn / groups >= share_of_die || c >= ci) return;               // uniform over the workgroup
  const int first = (turn % groups) * pixels_per_group;
  int next_start = indptr[(size_t)c * hw + (first + wave < hw ? first + wave : 0)];     // of this wave's first row
  const size_t wbase = (size_t)c * 9, wstride = (size_t)ci * 9;
  // Each wave compacts an eighth of the output channels, 64 candidates at a time: the masks and weights of
  // all of them first, all in flight together, then, once every wave's count is known, the kept ones.
  const int o0 = co * wave / kFillWaves, q0 = o0 * 9, q_end = (co * (wave + 1) / kFillWaves) * 9;
  const int batches = (q_end - q0 + 63) >> 6;      // at most kMaxBatches for a list of kConvListBytes
  const KeptBytes kb(mask, weight);
  float v[kMaxBatches];
  unsigned keeps = 0;                              // bit s: this lane's candidate of batch s
  int count = 0;
#pragma unroll
  for (int s0 = 0; s0 < kMaxBatches; s0 += 8)
    if (s0 < batches) {
      uint8_t m[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = q0 + 64 * (s0 + u) + lane, qc = q < q_end ? q : q_end - 1;
        const int o = qc / 9;
        const size_t at = wbase + o * wstride + (8 - (qc - 9 * o));
        m[u] = kb.bytes[at];
        v[s0 + u] = weight[at];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool keep = (kb.all || m[u] != 0) && q0 + 64 * (s0 + u) + lane < q_end;
        keeps |= (unsigned)keep << (s0 + u);
        count += keep;
      }
    }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) count += __shfl_xor(count, off);
  if (lane == 0) share[wave] = count;
  __syncthreads();
  int pos = 0, n = 0;
  for (int k = 0; k < kFillWaves; ++k) {
    if (k < wave) pos += share[k];
    n += share[k];
  }
#pragma unroll
  for (int s = 0; s < kMaxBatches; ++s) {
    if (s >= batches) break;
    const int q = q0 + 64 * s + lane;
    const bool keep = ((keeps >> s) & 1u) != 0;
    const unsigned long long bal = __ballot(keep);
    if (keep) {
      const int o = q / 9, tap = q - 9 * o, to = pos + __popcll(bal & ((1ull << lane) - 1ull));
      list[to] = make_int2(o * hw + (tap / 3 - 1) * w + tap % 3 - 1, __float_as_int(v[s]));
      taps[to] = (uint8_t)tap;
    }
    pos += __popcll(bal);
  }
  __syncthreads();
  const int end = first + pixels_per_group < hw ? first + pixels_per_group : hw;
  for (int i = first + wave; i < end; i += kFillWaves) {
    const int y = i / w, x = i - y * w;
    const int s = next_start;
    next_start = indptr[(size_t)c * hw + (i + kFillWaves < end ? i + kFillWaves : i)];
    int32_t* idx = indices + s;
    float* val = data + s;
    if (y > 0 && y + 1 < h && x > 0 && x + 1 < w) {
      for (int k = lane; k < n; k += 64) {
        const int2 e = list[k];
        idx[k] = e.x + i;
        val[k] = __int_as_float(e.y);
      }
    } else {
      // bit `tap` set: the neighbour of that tap lies in the image
      unsigned ok = 0x1ffu;
      if (y == 0) ok &= ~0x007u;
      if (y == h - 1) ok &= ~0x1c0u;
      if (x == 0) ok &= ~0x049u;
      if (x == w - 1) ok &= ~0x124u;
      int done = 0;
      for (int k0 = 0; k0 < n; k0 += 64) {
        const int k = k0 + lane;
        const bool in = k < n && ((ok >> taps[k < n ? k : 0]) & 1u) != 0;
        const unsigned long long bal = __ballot(in);
        if (in) {
          const int2 e = list[k];
          const int to = done + __popcll(bal & ((1ull << lane) - 1ull));
          idx[to] = e.x + i;
          val[to] = __int_as_float(e.y);
        }
        done += __popcll(bal);
      }
    }
  }
}

// Any kernel size, stride, zero padding and dilation (the generic routine the footnote of Appendix
// D.1 leaves open).  Input (c, y, x) feeds output (o, oy, ox) through tap (ky, kx) when
// y = oy sh - ph + ky dh and x = ox sw - pw + kx dw; for a given output the tap is unique, so
// no entry is a sum.  Candidate q = o * kh * kw + tap with the taps taken from the last to the
// first, which makes (oy, ox) and with it the column ascend along a row.
struct ConvGeom {
  int kh, kw, sh, sw, ph, pw, dh, dw, oh, ow;
};

__device__ __forceinline__ ConvCand conv2d_candidate(int q, int c, int y, int x, int ci, const ConvGeom& g,
                                                     const uint8_t* __restrict__ mask) {
  ConvCand r;
  const int taps = g.kh * g.kw;
  const int o = q / taps, tap = q - o * taps;
  const int ky = g.kh - 1 - tap / g.kw, kx = g.kw - 1 - (tap - (tap / g.kw) * g.kw);
  const int ny = y + g.ph - ky * g.dh, nx = x + g.pw - kx * g.dw;      // oy sh and ox sw
  const int oy = ny / g.sh, ox = nx / g.sw;
  r.widx = ((o * ci + c) * g.kh + ky) * g.kw + kx;
  r.col = (o * g.oh + oy) * g.ow + ox;
  r.valid = ny >= 0 && nx >= 0 && oy * g.sh == ny && ox * g.sw == nx && oy < g.oh && ox < g.ow &&
            (mask == nullptr || mask[r.widx] != 0);
  return r;
}

template <int FILL>
__global__ void __launch_bounds__(256)
conv2d_rows_kernel(int ci, int co, int h, int w, ConvGeom g, const float* __restrict__ weight,
                   const uint8_t* __restrict__ mask, int32_t* __restrict__ indptr,
                   int32_t* __restrict__ indices, float* __restrict__ data) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int rows = ci * h * w;
  if (row >= rows) return;
  const int c = row / (h * w);
  const int rem = row - c * h * w;
  const int y = rem / w, x = rem - y * w;
  const int ncand = co * g.kh * g.kw;
  int count = 0;
  const int base = FILL ? indptr[row] : 0;
  for (int q0 = 0; q0 < ncand; q0 += 64) {
    const int q = q0 + lane;
    ConvCand cd;
    cd.valid = false;
    if (q < ncand) cd = conv2d_candidate(q, c, y, x, ci, g, mask);
    const unsigned long long bal = __ballot(cd.valid);
    if (FILL && cd.valid) {
      const int off = count + __popcll(bal & ((1ull << lane) - 1ull));
      indices[base + off] = cd.col;
      data[base + off] = weight[cd.widx];
    }
    count += __popcll(bal);
  }
  if (!FILL && lane == 0) indptr[row] = count;
}

// host: checks the geometry, fills in the output size; false if a size does not fit 32 bits
bppsa_status conv2d_geometry(int ci, int co, int h, int w, const bppsa_conv2d_geometry* in, ConvGeom* g) {
  if (!in || ci < 1 || co < 1 || h < 1 || w < 1) return BPPSA_EINVAL;
  if (in->kh < 1 || in->kw < 1 || in->stride_h < 1 || in->stride_w < 1 || in->pad_h < 0 || in->pad_w < 0 ||
      in->dil_h < 1 || in->dil_w < 1)
    return BPPSA_EINVAL;
  const int64_t span_h = (int64_t)h + 2LL * in->pad_h - (int64_t)in->dil_h * (in->kh - 1) - 1;
  const int64_t span_w = (int64_t)w + 2LL * in->pad_w - (int64_t)in->dil_w * (in->kw - 1) - 1;
  if (span_h < 0 || span_w < 0) return BPPSA_ESHAPE;               // the kernel does not fit: no output
  const int64_t oh = span_h / in->stride_h + 1, ow = span_w / in->stride_w + 1;
  const int64_t rows = (int64_t)ci * h * w, cols = (int64_t)co * oh * ow;
  const int64_t taps = (int64_t)in->kh * in->kw;
  if (rows >= INT32_MAX || cols >= INT32_MAX || taps >= INT32_MAX || (int64_t)co * taps >= INT32_MAX ||
      (int64_t)co * ci * taps >= INT32_MAX)
    return BPPSA_EOVERFLOW;
  // every stored entry is one (output element, input channel, tap) triple
  if ((double)cols * (double)ci * (double)taps >= (double)INT32_MAX) return BPPSA_EOVERFLOW;
  // intermediate coordinates: y + pad and ky * dil
  if ((int64_t)h + in->pad_h >= INT32_MAX || (int64_t)w + in->pad_w >= INT32_MAX ||
      (int64_t)in->dil_h * in->kh >= INT32_MAX || (int64_t)in->dil_w * in->kw >= INT32_MAX)
    return BPPSA_EOVERFLOW;
  *g = ConvGeom{in->kh, in->kw, in->stride_h, in->stride_w, in->pad_h, in->pad_w, in->dil_h, in->dil_w, (int)oh, (int)ow};
  return BPPSA_OK;
}

// A workgroup owns 64 input features (a lane each, so mask and weight rows are read along the lanes) and
// its sixteen waves share the outputs out in order; each lane counts, and then appends, its own entries.
constexpr int kLinearWaves = 16;
template <int FILL>
__global__ void __launch_bounds__(64 * kLinearWaves)
linear_rows_kernel(int out, int in, const float* __restrict__ weight, const uint8_t* __restrict__ mask,
                   int32_t* __restrict__ indptr, int32_t* __restrict__ indices, float* __restrict__ data) {
  __shared__ int counts[kLinearWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x * 64 + lane;                             // input feature
  const int j0 = (int)((long long)out * wave / kLinearWaves), j1 = (int)((long long)out * (wave + 1) / kLinearWaves);
  int count = 0;
  if (row < in) {
    if (mask) {
      for (int jb = j0; jb < j1; jb += 16) {                         // sixteen loads at a time
        uint8_t m[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) m[u] = mask[(size_t)(jb + u < j1 ? jb + u : jb) * in + row];
#pragma unroll
        for (int u = 0; u < 16; ++u) count += jb + u < j1 && m[u] != 0;
      }
    } else {
      count = j1 - j0;
    }
  }
  counts[wave][lane] = count;
  __syncthreads();
  if (!FILL) {
    if (wave == 0 && row < in) {
      int n = 0;
      for (int k = 0; k < kLinearWaves; ++k) n += counts[k][lane];
      indptr[row] = n;
    }
    return;
  }
  if (row >= in) return;
  int pos = indptr[row];
  for (int k = 0; k < wave; ++k) pos += counts[k][lane];
  const KeptBytes kb(mask, weight);
  constexpr int kBatch = 32;                                          // loads in flight ahead of the stores
  for (int jb = j0; jb < j1; jb += kBatch) {
    uint8_t m[kBatch];
    float v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const size_t at = (size_t)(jb + u < j1 ? jb + u : j1 - 1) * in + row;
      m[u] = kb.bytes[at];
      v[u] = weight[at];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if ((kb.all || m[u] != 0) && jb + u < j1) {
        indices[pos] = jb + u;
        data[pos] = v[u];
        ++pos;
      }
  }
}

__global__ void relu_kernel(int d, const float* __restrict__ x, int32_t* __restrict__ indptr,
                            int32_t* __restrict__ indices, float* __restrict__ data) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < d) {
    indptr[i] = i;
    indices[i] = i;
    data[i] = x[i] > 0.f ? 1.f : 0.f;
  }
  if (i == d) indptr[d] = d;
}

// Every window has exactly one entry, so the rows of a pair of image rows hold w / 2 entries together and
// start at (pair of rows) * w / 2: a wave takes a pair, a lane a window, and what is left to count is how many
// windows before this one had their maximum in the upper image row.  First maximum in row-major window order.
__global__ void __launch_bounds__(256)
pool_kernel(int pairs, int h, int w, const float* __restrict__ x, int32_t* __restrict__ indptr,
            int32_t* __restrict__ indices, float* __restrict__ data) {
  const int lane = threadIdx.x & 63;
  const int pair = blockIdx.x * 4 + (threadIdx.x >> 6);               // = channel * (h / 2) + window row
  if (pair >= pairs) return;
  const int nw = w / 2;
  const float* top = x + (size_t)pair * 2 * w;
  const size_t row0 = (size_t)pair * 2 * w, row1 = row0 + w;
  const int base = pair * nw;
  // which of the four is the window's first maximum; 4 for lanes without a window
  auto winner = [&](int k) {
    if (k >= nw) return 4;
    const float a = top[2 * k], b = top[2 * k + 1], c = top[w + 2 * k], d = top[w + 2 * k + 1];
    float best = a;
    int at = 0;
    if (b > best) { best = b; at = 1; }
    if (c > best) { best = c; at = 2; }
    if (d > best) { best = d; at = 3; }
    return at;
  };
  int upper = 0;                                                      // windows with their maximum in the upper row
  for (int k0 = 0; k0 < nw; k0 += 64) upper += __popcll(__ballot(winner(k0 + lane) < 2));
  int seen0 = base, seen1 = base + upper;
  for (int k0 = 0; k0 < nw; k0 += 64) {
    const int k = k0 + lane, at = winner(k);
    const unsigned long long before = (1ull << lane) - 1ull;
    const unsigned long long up = __ballot(at < 2), low = __ballot(at == 2 || at == 3);
    const int p0 = seen0 + __popcll(up & before), p1 = seen1 + __popcll(low & before);
    if (k < nw) {
      indptr[row0 + 2 * k] = p0;
      indptr[row0 + 2 * k + 1] = p0 + (at == 0);
      indptr[row1 + 2 * k] = p1;
      indptr[row1 + 2 * k + 1] = p1 + (at == 2);
      const int p = at < 2 ? p0 : p1;
      indices[p] = base + k;
      data[p] = 1.f;
    }
    seen0 += __popcll(up);
    seen1 += __popcll(low);
  }
  if (pair == pairs - 1 && lane == 0) indptr[(size_t)pairs * 2 * w] = pairs * nw;
}

}  // namespace

static bppsa_status conv3x3_indptr(int ci, int co, int h, int w, const uint8_t* mask, int32_t* indptr,
                                   int32_t* report, hipStream_t s) {
  if (ci < 1 || co < 1 || h < 1 || w < 1 || !indptr) return BPPSA_EINVAL;
  const int64_t rows = (int64_t)ci * h * w, cols = (int64_t)co * h * w;
  const int64_t nnz_max = (int64_t)ci * co * (3LL * h - 2) * (3LL * w - 2);
  if (rows >= INT32_MAX || cols >= INT32_MAX || nnz_max >= INT32_MAX || (int64_t)co * ci * 9 >= INT32_MAX)
    return BPPSA_EOVERFLOW;
  const int groups = bppsa_ceil_div(ci, kCountChannels);
  if (rows <= kDirectRows || h * w < 10) {
    conv_channel_counts_kernel<true><<<groups, kCountThreads, 0, s>>>(ci, co, h, w, mask, indptr);
    BPPSA_CHECK_LAUNCH();
    return bppsa_lengths_to_indptr(indptr, (int)rows, s, 1, report);
  }
  conv_channel_counts_kernel<false><<<groups, kCountThreads, 0, s>>>(ci, co, h, w, mask, indptr);
  BPPSA_CHECK_LAUNCH();
  BPPSA_TRY(bppsa_lengths_to_indptr(indptr, ci, s, h * w, report));
  conv_pointers_kernel<<<ci, 256, 0, s>>>(h, w, indptr);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

extern "C" bppsa_status bppsa_csr_conv3x3_indptr(int ci, int co, int h, int w, const uint8_t* mask,
                                                 int32_t* indptr, void* stream) {
  return conv3x3_indptr(ci, co, h, w, mask, indptr, nullptr, (hipStream_t)stream);
}

// ---- the two-call pattern's first half with the total handed to the host ------------------------------------
// The prefix sum's kernel stores the total in the caller's pinned memory the moment it has it, and the host
// watches that word: a few microseconds instead of a copy and a stream synchronisation (about 25 us, during
// which the device is idle).  After kSpins looks the host blocks on the stream instead.
static bppsa_status prepare_report(volatile int32_t* report, int64_t* nnz, hipStream_t s) {
  if (!report || !nnz) return BPPSA_EINVAL;
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &capturing) != hipSuccess || capturing != hipStreamCaptureStatusNone) return BPPSA_EHIP;
  *report = -1;
  __atomic_thread_fence(__ATOMIC_SEQ_CST);
  return BPPSA_OK;
}
static bppsa_status await_report(volatile int32_t* report, int64_t* nnz, hipStream_t s) {
  constexpr int kSpins = 20000;
  int32_t v = *report;
  for (int k = 0; v == -1 && k < kSpins; ++k) {
    __builtin_ia32_pause();
    v = *report;
  }
  if (v == -1) {
    BPPSA_HIP_TRY(hipStreamSynchronize(s));
    __atomic_thread_fence(__ATOMIC_SEQ_CST);
    v = *report;
  }
  if (v < 0) return v == -1 ? BPPSA_EHIP : BPPSA_EOVERFLOW;
  *nnz = v;
  return BPPSA_OK;
}

extern "C" bppsa_status bppsa_csr_conv3x3_indptr_nnz(int ci, int co, int h, int w, const uint8_t* mask, int32_t* indptr,
                                                     int32_t* report, int64_t* nnz, void* stream) {
  BPPSA_TRY(prepare_report(report, nnz, (hipStream_t)stream));
  BPPSA_TRY(conv3x3_indptr(ci, co, h, w, mask, indptr, report, (hipStream_t)stream));
  return await_report(report, nnz, (hipStream_t)stream);
}

extern "C" bppsa_status bppsa_csr_conv3x3_fill(int ci, int co, int h, int w, const float* weight,
                                               const uint8_t* mask, const int32_t* indptr,
                                               int32_t* indices, float* data, void* stream) {
  if (ci < 1 || co < 1 || h < 1 || w < 1 || !weight || !indptr || !indices || !data) return BPPSA_EINVAL;
  const int64_t rows = (int64_t)ci * h * w;
  const int64_t nnz_max = (int64_t)ci * co * (3LL * h - 2) * (3LL * w - 2);
  if (rows >= INT32_MAX || (int64_t)co * h * w >= INT32_MAX || nnz_max >= INT32_MAX) return BPPSA_EOVERFLOW;
  const size_t list = (size_t)co * 9 * (sizeof(int2) + 1);
  if (list <= kConvListBytes) {
    // a stretch of pixels per workgroup: enough workgroups to fill the device twice over, and at least eight
    // rows to each list
    const int hw = h * w;
    int groups = bppsa_ceil_div(512, ci);
    if (groups > bppsa_ceil_div(hw, 8)) groups = bppsa_ceil_div(hw, 8);
    const int pixels = bppsa_ceil_div(hw, groups);
    if (list > 48 * 1024)
      BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)conv_fill_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)kConvListBytes));
    conv_fill_kernel<<<8 * bppsa_ceil_div(ci, 8) * bppsa_ceil_div(hw, pixels), 64 * kFillWaves, list, (hipStream_t)stream>>>(
        ci, co, h, w, pixels, weight, mask, indptr, indices, data);
    BPPSA_CHECK_LAUNCH();
    return BPPSA_OK;
  }
  conv_rows_kernel<<<bppsa_ceil_div((int)rows, 4), 256, 0, (hipStream_t)stream>>>(
      ci, co, h, w, weight, mask, indptr, indices, data);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

static bppsa_status conv2d_indptr(int ci, int co, int h, int w, const bppsa_conv2d_geometry* geometry,
                                  const uint8_t* mask, int32_t* indptr, int32_t* report, hipStream_t s) {
  if (!indptr) return BPPSA_EINVAL;
  ConvGeom g;
  BPPSA_TRY(conv2d_geometry(ci, co, h, w, geometry, &g));
  const int rows = ci * h * w;
  conv2d_rows_kernel<0><<<bppsa_ceil_div(rows, 4), 256, 0, s>>>(ci, co, h, w, g, nullptr, mask, indptr, nullptr, nullptr);
  BPPSA_CHECK_LAUNCH();
  return bppsa_lengths_to_indptr(indptr, rows, s, 1, report);
}

extern "C" bppsa_status bppsa_csr_conv2d_indptr(int ci, int co, int h, int w, const bppsa_conv2d_geometry* geometry,
                                                const uint8_t* mask, int32_t* indptr, void* stream) {
  return conv2d_indptr(ci, co, h, w, geometry, mask, indptr, nullptr, (hipStream_t)stream);
}

extern "C" bppsa_status bppsa_csr_conv2d_indptr_nnz(int ci, int co, int h, int w, const bppsa_conv2d_geometry* geometry,
                                                    const uint8_t* mask, int32_t* indptr, int32_t* report, int64_t* nnz,
                                                    void* stream) {
  BPPSA_TRY(prepare_report(report, nnz, (hipStream_t)stream));
  BPPSA_TRY(conv2d_indptr(ci, co, h, w, geometry, mask, indptr, report, (hipStream_t)stream));
  return await_report(report, nnz, (hipStream_t)stream);
}

extern "C" bppsa_status bppsa_csr_conv2d_fill(int ci, int co, int h, int w, const bppsa_conv2d_geometry* geometry,
                                              const float* weight, const uint8_t* mask, const int32_t* indptr,
                                              int32_t* indices, float* data, void* stream) {
  if (!weight || !indptr || !indices || !data) return BPPSA_EINVAL;
  ConvGeom g;
  BPPSA_TRY(conv2d_geometry(ci, co, h, w, geometry, &g));
  conv2d_rows_kernel<1><<<bppsa_ceil_div(ci * h * w, 4), 256, 0, (hipStream_t)stream>>>(
      ci, co, h, w, g, weight, mask, const_cast<int32_t*>(indptr), indices, data);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

extern "C" bppsa_status bppsa_csr_relu(int d, const float* x, int32_t* indptr, int32_t* indices,
                                       float* data, void* stream) {
  if (d < 1 || !x || !indptr || !indices || !data) return BPPSA_EINVAL;
  if (d == INT32_MAX) return BPPSA_EOVERFLOW;
  relu_kernel<<<bppsa_ceil_div(d + 1, 256), 256, 0, (hipStream_t)stream>>>(d, x, indptr, indices, data);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

extern "C" bppsa_status bppsa_csr_maxpool2x2(int c, int h, int w, const float* x, int32_t* indptr,
                                             int32_t* indices, float* data, void* stream) {
  if (c < 1 || h < 2 || w < 2 || !x || !indptr || !indices || !data) return BPPSA_EINVAL;
  if ((h & 1) || (w & 1)) return BPPSA_ESHAPE;
  const int64_t rows = (int64_t)c * h * w;
  if (rows >= INT32_MAX) return BPPSA_EOVERFLOW;
  hipStream_t s = (hipStream_t)stream;
  const int pairs = c * (h / 2);
  pool_kernel<<<bppsa_ceil_div(pairs, 4), 256, 0, s>>>(pairs, h, w, x, indptr, indices, data);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

static bppsa_status linear_indptr(int out, int in, const uint8_t* mask, int32_t* indptr, int32_t* report, hipStream_t s) {
  if (out < 1 || in < 1 || !indptr) return BPPSA_EINVAL;
  if ((int64_t)out * in >= INT32_MAX) return BPPSA_EOVERFLOW;
  linear_rows_kernel<0><<<bppsa_ceil_div(in, 64), 64 * kLinearWaves, 0, s>>>(out, in, nullptr, mask, indptr, nullptr, nullptr);
  BPPSA_CHECK_LAUNCH();
  return bppsa_lengths_to_indptr(indptr, in, s, 1, report);
}

extern "C" bppsa_status bppsa_csr_linear_indptr(int out, int in, const uint8_t* mask, int32_t* indptr,
                                                void* stream) {
  return linear_indptr(out, in, mask, indptr, nullptr, (hipStream_t)stream);
}

extern "C" bppsa_status bppsa_csr_linear_indptr_nnz(int out, int in, const uint8_t* mask, int32_t* indptr,
                                                    int32_t* report, int64_t* nnz, void* stream) {
  BPPSA_TRY(prepare_report(report, nnz, (hipStream_t)stream));
  BPPSA_TRY(linear_indptr(out, in, mask, indptr, report, (hipStream_t)stream));
  return await_report(report, nnz, (hipStream_t)stream);
}

extern "C" bppsa_status bppsa_csr_linear_fill(int out, int in, const float* weight, const uint8_t* mask,
                                              const int32_t* indptr, int32_t* indices, float* data,
                                              void* stream) {
  if (out < 1 || in < 1 || !weight || !indptr || !indices || !data) return BPPSA_EINVAL;
  if ((int64_t)out * in >= INT32_MAX) return BPPSA_EOVERFLOW;
  linear_rows_kernel<1><<<bppsa_ceil_div(in, 64), 64 * kLinearWaves, 0, (hipStream_t)stream>>>(
      out, in, weight, mask, const_cast<int32_t*>(indptr), indices, data);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
