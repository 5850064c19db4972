// bppsa_scan for every H <= 128 that has no kernel of its own (H = 20 and 128 do).
//
// The chain of n elements, element c = Jt[T-1-c] counted from the seed, is cut as
//     [ top | segment 0 | segment 1 | ... | segment s-1 ]      (Section 5.3's hybrid)
// and walked in three launches:
//   1. one workgroup per sample walks the top with matrix-vector products from the seed while the others
//      form the total of every segment but the last with matrix-matrix products on the matrix cores;
//   2. one workgroup per sample walks the totals, which gives every segment its incoming vector;
//   3. one workgroup per (segment, sample) walks the segment with matrix-vector products.
// Short chains, and batches that fill the device by themselves, are all top: one launch, no product.
// Where the cuts lie is a cost model's choice (plan_tiles), within the workspace the caller gave.
//
// Sizes are rounded up to NT = ceil(H / 16) blocks of 16 and a workgroup has NT waves (one more stores
// gradients); rows and columns past H read as zero through the bounds of a buffer descriptor.
//
// This file is compiled with MFMA results in ordinary vector registers (see the build script): the running
// product's results are the next step's B operands.
#include "bppsa_internal.h"
#include "scan_plan.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kMaxNT = 8;
constexpr unsigned kOut = 0x80000000u;             // a byte offset no tile reaches: reads zero

// Orders LDS accesses of the workgroup; outstanding global loads and stores stay outstanding.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// How the threads of a workgroup share a tile.  LPR lanes own a row, so 64 NT / LPR rows are held by a pass
// and a thread has RP rows g + PASS r (g = tid / LPR) of NC pieces at columns W l + W LPR c (l = tid % LPR).
// VEC: pieces of 16 bytes, for H a multiple of four: a unit keeps about 64 KB of requests in flight, and only
// requests of whole lines make that 64 KB of data (with 4-byte pieces the walk at H = 64 drew 45 GB/s).
template <int NT_, bool VEC_>
struct Share {
  static constexpr int NT = NT_;
  static constexpr bool VEC = VEC_;
  static constexpr int W = VEC ? 4 : 1;
  static constexpr int LPR = VEC ? (NT == 1 ? 4 : NT == 2 ? 8 : 16) : 16;
  static constexpr int PASS = 64 * NT / LPR;
  static constexpr int RP = LPR / 4;
  static constexpr int NC = VEC ? (NT > 4 ? 2 : 1) : NT;
  static constexpr int HP = 16 * NT;               // rows of a padded tile; columns reach W LPR NC >= HP
  // tiles in flight per walk, up to about 128 registers of them: a step takes 0.13 to 0.35 us, a fetch 1 to 2 us
  static constexpr int REGS = RP * NC * W;
  static constexpr int D = REGS <= 4 ? 16 : REGS <= 8 ? 12 : REGS <= 16 ? 7 : REGS <= 20 ? 5 : 4;
  float m[RP][NC][W];
};

// Byte offsets of a thread's pieces in a tile: first column block of its rows, and the last one (which may
// end early).
template <class S>
struct Places {
  unsigned row[S::RP], last[S::RP];
  __device__ __forceinline__ Places(int tid, int H) {
    const int g = tid / S::LPR, l = tid % S::LPR;
    constexpr int kLast = S::W * S::LPR * (S::NC - 1);
#pragma unroll
    for (int r = 0; r < S::RP; ++r) {
      const int i = g + S::PASS * r;
      row[r] = (i < H && S::W * l < H) ? (unsigned)(i * H + S::W * l) * 4u : kOut;
      last[r] = (i < H && S::W * l + kLast < H) ? (unsigned)(i * H + S::W * l + kLast) * 4u : kOut;
    }
  }
};
template <class S>
__device__ __forceinline__ void load_tile(S& t, const float* tile, int H, const Places<S>& p) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(tile), 0, H * H * 4, 0x00020000);
#pragma unroll
  for (int r = 0; r < S::RP; ++r)
#pragma unroll
    for (int c = 0; c < S::NC; ++c) {
      const int off = (int)(c == S::NC - 1 ? p.last[r] : p.row[r] + 4u * S::W * S::LPR * c);
      if constexpr (S::VEC) {
        const v4f x = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
#pragma unroll
        for (int u = 0; u < 4; ++u) t.m[r][c][u] = x[u];
      } else {
        t.m[r][c][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0));
      }
    }
}

// sum over the N lanes of a group (4, 8 or 16), in every lane
template <int CTRL>
__device__ __forceinline__ float dpp_from(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ float group_sum(float x) {
  x += dpp_from<0xB1>(x);                          // quad_perm [1,0,3,2]
  x += dpp_from<0x4E>(x);                          // quad_perm [2,3,0,1]
  if (N >= 8) x += dpp_from<0x141>(x);             // row_half_mirror
  if (N >= 16) x += dpp_from<0x140>(x);            // row_mirror
  return x;
}

// v <- tile_s v for s = 0 .. steps-1, tile_s at src + s * stride (floats); vector s goes to dst + s * dstride,
// the last one to `last` instead where that is not null.  The entering vector is in vs[0..H) and both
// buffers of vs (of kVec floats) are zero past H.  Called by all NT + 1 waves; wave NT only stores, so that
// the others have nothing but loads outstanding and can wait for the oldest tile alone (a wait behind a
// pending store waits for everything).  One barrier per step.
constexpr int kVec = 128;
template <class S>
__device__ __forceinline__ void walk(const float* src, long long stride, int steps, int H, float* vs, float* dst,
                                     long long dstride, float* last) {
  const int tid = threadIdx.x;
  if (tid >= 64 * S::NT) {
    const int lane = tid - 64 * S::NT;
    for (int s = 0; s < steps; ++s) {
      lds_barrier();
      const float* v = vs + ((s + 1) & 1) * kVec;
      float* out = (last && s == steps - 1) ? last : dst + s * dstride;
      if (lane < H) out[lane] = v[lane];
      if (S::NT > 4 && lane + 64 < H) out[lane + 64] = v[lane + 64];
    }
    return;
  }
  const Places<S> p(tid, H);
  const int g = tid / S::LPR, l = tid % S::LPR;
  const int myrow = g + S::PASS * l;               // the row this lane hands on, if it is one of l < RP
  const bool writer = l < S::RP && myrow < H;
  S t[S::D];
#pragma unroll
  for (int k = 0; k < S::D; ++k) load_tile(t[k], src + (long long)min(k, steps - 1) * stride, H, p);
  for (int s0 = 0; s0 < steps; s0 += S::D) {
#pragma unroll
    for (int k = 0; k < S::D; ++k) {
      const int s = s0 + k;
      if (s >= steps) break;                       // uniform
      const float* v = vs + (s & 1) * kVec;
      float x[S::NC][S::W], sum[S::RP];
#pragma unroll
      for (int c = 0; c < S::NC; ++c) {
        if constexpr (S::VEC) {
          const v4f xv = *reinterpret_cast<const v4f*>(v + 4 * (l + S::LPR * c));
#pragma unroll
          for (int u = 0; u < 4; ++u) x[c][u] = xv[u];
        } else {
          x[c][0] = v[l + S::LPR * c];
        }
      }
#pragma unroll
      for (int r = 0; r < S::RP; ++r) {
        float a = t[k].m[r][0][0] * x[0][0];
#pragma unroll
        for (int e = 1; e < S::NC * S::W; ++e) a = __builtin_fmaf(t[k].m[r][e / S::W][e % S::W], x[e / S::W][e % S::W], a);
        sum[r] = a;
      }
      load_tile(t[k], src + (long long)min(s + S::D, steps - 1) * stride, H, p);
#pragma unroll
      for (int r = 0; r < S::RP; ++r) sum[r] = group_sum<S::LPR>(sum[r]);
      float y = sum[0];
      if (S::RP >= 2) y = (l & 1) ? sum[S::RP >= 2 ? 1 : 0] : y;
      if (S::RP == 4) y = (l & 2) ? ((l & 1) ? sum[S::RP - 1] : sum[S::RP / 2]) : y;
      if (writer) vs[((s + 1) & 1) * kVec + myrow] = y;
      lds_barrier();
    }
  }
}

// P <- J P for J = tile_1, ..., tile_{steps-1} from P = tile_0 (tile_s at src + s * stride); tot = P.
//
// v_mfma_f32_16x16x4_f32: lane l supplies A[l % 16][k] and B[k][l % 16] of one k per quarter wave l / 16 and
// holds D[4 (l / 16) + v][l % 16] in register v.  Any assignment of k values to (issue, quarter) will do
// as long as A and B agree: issue (kb, v) takes k = 16 kb + 4 (l / 16) + v, the row register v of
// row-block kb holds, so the results of one product are the B operands of the next and P never leaves
// the registers.  Wave w owns columns 16 w .. 16 w + 15.  The Jacobians go through LDS, one buffer read
// while the next tile is written to the other; one barrier per product.
template <class S>
__device__ __forceinline__ void reduce(const float* src, long long stride, int steps, int H, float* lds, float* tot) {
  constexpr int NT = S::NT, LS = 16 * NT + 4, TILE = 16 * NT * LS;
  const int tid = threadIdx.x;
  if (tid >= 64 * NT) return;                      // the storing wave has nothing to do here
  const int wave = tid >> 6, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const Places<S> p(tid, H);
  const int g = tid / S::LPR, l = tid % S::LPR;
  S t;
  auto stage = [&](float* buf) {
#pragma unroll
    for (int r = 0; r < S::RP; ++r)
#pragma unroll
      for (int c = 0; c < S::NC; ++c) {
        const int col = S::W * (l + S::LPR * c);
        float* to = buf + (g + S::PASS * r) * LS + col;
        if constexpr (S::VEC) {
          if (S::W * S::LPR * S::NC == S::HP || col < S::HP)
            *reinterpret_cast<v4f*>(to) = v4f{t.m[r][c][0], t.m[r][c][1], t.m[r][c][2], t.m[r][c][3]};
        } else {
          *to = t.m[r][c][0];
        }
      }
  };
  load_tile(t, src, H, p);
  stage(lds);
  load_tile(t, src + (long long)min(1, steps - 1) * stride, H, p);
  lds_barrier();
  v4f P[NT];
#pragma unroll
  for (int kb = 0; kb < NT; ++kb)
#pragma unroll
    for (int v = 0; v < 4; ++v) P[kb][v] = lds[(16 * kb + 4 * q + v) * LS + 16 * wave + l16];
  stage(lds + TILE);
  load_tile(t, src + (long long)min(2, steps - 1) * stride, H, p);
  lds_barrier();
  const int pad = 16 * (NT - 1) + 4 * q;           // the last row block's rows of this lane
  for (int s = 1; s < steps; ++s) {
    const float* A = lds + (s & 1) * TILE + l16 * LS + 4 * q;
    v4f Q[NT];
#pragma unroll
    for (int bi = 0; bi < NT; ++bi) Q[bi] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < NT; ++kb) {
      v4f a[NT];
#pragma unroll
      for (int bi = 0; bi < NT; ++bi) a[bi] = *reinterpret_cast<const v4f*>(A + 16 * bi * LS + 16 * kb);
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int bi = 0; bi < NT; ++bi) Q[bi] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[bi][v], P[kb][v], Q[bi], 0, 0, 0);
      // the tile of step s + 1 goes to the other buffer, which every wave left at the last barrier
      if (kb == 0) {
        stage(lds + ((s + 1) & 1) * TILE);
        load_tile(t, src + (long long)min(s + 2, steps - 1) * stride, H, p);
      }
    }
    // the padding rows, zeros times P, are put back to zero: an Inf of P left NaN there, which the next
    // tile's padding columns, zeros too, would bring into every row
#pragma unroll
    for (int v = 0; v < 4; ++v) Q[NT - 1][v] = pad + v < H ? Q[NT - 1][v] : 0.f;
#pragma unroll
    for (int bi = 0; bi < NT; ++bi) P[bi] = Q[bi];
    lds_barrier();
  }
  const int col = 16 * wave + l16;
#pragma unroll
  for (int bi = 0; bi < NT; ++bi)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 * bi + 4 * q + v;
      if (row < H && col < H) tot[row * H + col] = P[bi][v];
    }
}

// How a call is cut: `top` elements, then nseg segments of `len` (the last one may be shorter).
struct Cut {
  int top, len, nseg;
};

struct Chain {
  int T, B, H, n;
  const float* __restrict__ Jt;
  const float* __restrict__ seed;
  float* __restrict__ G;
  float* __restrict__ g0;
  float* __restrict__ tot;           // [nseg - 1][B][H][H]
  float* __restrict__ vin;           // [nseg][B][H]
  Cut cut;
};

__device__ __forceinline__ const float* tile_of(const Chain& ch, int c, int b) {
  return ch.Jt + ((size_t)(ch.T - 1 - c) * ch.B + b) * ch.H * ch.H;
}
// walks elements [c0, c0 + count) of sample b: vector c goes to G[T-2-c], the one of c = T-1 to g0
template <class S>
__device__ __forceinline__ void walk_elements(const Chain& ch, int c0, int count, int b, float* vs) {
  const long long row = (long long)ch.B * ch.H;
  const bool tail = c0 + count == ch.T;             // only with g0
  walk<S>(tile_of(ch, c0, b), -row * ch.H, count, ch.H, vs, ch.G + (long long)(ch.T - 2 - c0) * row + (long long)b * ch.H,
           -row, tail ? ch.g0 + (size_t)b * ch.H : nullptr);
}
__device__ __forceinline__ void enter(float* vs, const float* v, int H) {
  for (int e = threadIdx.x; e < 2 * kVec; e += blockDim.x) vs[e] = e < H ? v[e] : 0.f;
  lds_barrier();
}

template <class S>
__global__ void __launch_bounds__(64 * (S::NT + 1))
tiles_top_kernel(const Chain ch) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int H = ch.H, B = ch.B;
  if ((int)blockIdx.x >= B) {
    const int id = blockIdx.x - B, seg = id / B, b = id - seg * B;
    const int c0 = ch.cut.top + seg * ch.cut.len;
    reduce<S>(tile_of(ch, c0, b), -(long long)B * H * H, ch.cut.len, H, lds, ch.tot + ((size_t)seg * B + b) * H * H);
    return;
  }
  const int b = blockIdx.x;
  const float* seed = ch.seed + (size_t)b * H;
  float* first = ch.G + ((size_t)(ch.T - 1) * B + b) * H;
  if (first != seed)
    for (int e = threadIdx.x; e < H; e += blockDim.x) first[e] = seed[e];
  enter(lds, seed, H);
  if (ch.cut.top < 1) return;
  walk_elements<S>(ch, 0, ch.cut.top, b, lds);
  if (ch.cut.nseg > 0) {
    lds_barrier();
    float* out = ch.vin + (size_t)b * H;
    for (int e = threadIdx.x; e < H; e += blockDim.x) out[e] = lds[(ch.cut.top & 1) * kVec + e];
  }
}

// vin[k + 1] = tot[k] vin[k]
template <class S>
__global__ void __launch_bounds__(64 * (S::NT + 1))
tiles_chain_kernel(const Chain ch) {
  __shared__ __attribute__((aligned(16))) float vs[2 * kVec];
  const int b = blockIdx.x, H = ch.H;
  const long long row = (long long)ch.B * H;
  enter(vs, ch.vin + (size_t)b * H, H);
  walk<S>(ch.tot + (size_t)b * H * H, row * H, ch.cut.nseg - 1, H, vs, ch.vin + row + (size_t)b * H, row, nullptr);
}

template <class S>
__global__ void __launch_bounds__(64 * (S::NT + 1))
tiles_apply_kernel(const Chain ch) {
  __shared__ __attribute__((aligned(16))) float vs[2 * kVec];
  const int seg = blockIdx.x / ch.B, b = blockIdx.x - seg * ch.B;
  const int c0 = ch.cut.top + seg * ch.cut.len;
  enter(vs, ch.vin + ((size_t)seg * ch.B + b) * ch.H, ch.H);
  walk_elements<S>(ch, c0, min(ch.cut.len, ch.n - c0), b, vs);
}

size_t tot_bytes(int nseg, int B, int H) { return nseg > 1 ? bppsa_align_up((size_t)(nseg - 1) * B * H * H * sizeof(float), 256) : 0; }
size_t vin_bytes(int nseg, int B, int H) { return bppsa_align_up((size_t)nseg * B * H * sizeof(float), 256); }

// The cut with the least estimated time that needs at most `room` bytes.  Times in microseconds, measured on
// MI355X: a matrix-vector step costs the latency of its exchange, or what one unit draws from memory (62 KB
// per us), or, with many workgroups, its share of the device's memory rate; a product costs the latency of
// its 4 NT^2 issues per wave, or the matrix-core time (32 NT^3 cycles) of all the products its unit holds.
// Measured beside the best of fifty cuts (us; all top in brackets): T=300 B=7 H=64 32.5, best 32.5 [81];
// T=1000 B=16 H=32 36.7, 35.2 [136]; T=1000 B=16 H=8 18.7, 18.3 [98]; T=200 B=3 H=33 23.3, 22.3 [52].
Cut plan_tiles(int n, int B, int H, int cus, size_t room) {
  const int nt = (H + 15) / 16;
  const double mhz = 2300.0, tile = 4.0 * H * H, device_rate = 4.0e6, unit_rate = 62.0e3, launch = 4.0;
  const double mv = H % 4 == 0 ? 0.08 + 0.028 * nt : 0.10 + 0.05 * nt, draw = tile / unit_rate;
  const double mm = 0.25 + nt * nt * 4.0 * 32.0 / mhz * (nt > 4 ? nt / 4.0 : 1.0);
  const double mm_full = 32.0 * nt * nt * nt / mhz;
  const auto larger = [](double a, double b) { return a > b ? a : b; };
  const auto held = [&](double groups) { return (double)(((long long)groups + cus - 1) / cus); };
  const auto mv_step = [&](double groups) {        // a step of `groups` workgroups side by side
    return larger(larger(mv, draw), groups * tile / device_rate);
  };
  Cut best = {n, 0, 0};
  double best_us = launch + n * mv_step(B);
  for (int len = 2; len <= 256 && len < n; len += len < 16 ? 1 : len / 8)
    for (int half = 1; half <= 12; half += half < 4 ? 1 : 2) {             // the top: half to six segments
      const int top = len * half / 2;
      if (top > n - 2) break;
      const int nseg = (n - top + len - 1) / len;
      if (nseg < 2 || tot_bytes(nseg, B, H) + vin_bytes(nseg, B, H) > room) continue;
      // a unit works through the tops and totals it holds; the matrix cores are theirs to share
      const double reduce_us = (len - 1) * larger(mm, held((double)nseg * B) * mm_full);
      const double us = 3 * launch + larger(top * mv_step(B), reduce_us) + (nseg - 1) * mv_step(B) +
                        len * mv_step((double)nseg * B);
      if (us < best_us) {
        best_us = us;
        best = Cut{top, len, nseg};
      }
    }
  return best;
}

// The search takes a few microseconds, and a training loop asks for the same sizes every iteration: each
// host thread remembers its last answer.
Cut planned(int n, int B, int H, int cus, size_t room) {
  struct Memo {
    int n, B, H, cus;
    size_t room;
    Cut cut;
  };
  static thread_local Memo memo = {-1, 0, 0, 0, 0, {0, 0, 0}};
  if (memo.n != n || memo.B != B || memo.H != H || memo.cus != cus || memo.room != room)
    memo = Memo{n, B, H, cus, room, plan_tiles(n, B, H, cus, room)};
  return memo.cut;
}

template <class S>
bppsa_status launch(const Chain& ch, hipStream_t s) {
  const Cut& cut = ch.cut;
  constexpr int NT = S::NT;
  const size_t vec = 2 * kVec * sizeof(float), tiles = (size_t)2 * 16 * NT * (16 * NT + 4) * sizeof(float);
  const size_t lds = cut.nseg > 1 && tiles > vec ? tiles : vec;
  if (lds > 48 * 1024)
    BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)tiles_top_kernel<S>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds));
  const int extra = cut.nseg > 1 ? (cut.nseg - 1) * ch.B : 0;
  tiles_top_kernel<S><<<ch.B + extra, 64 * (NT + 1), lds, s>>>(ch);
  BPPSA_CHECK_LAUNCH();
  if (cut.nseg < 1) return BPPSA_OK;
  if (cut.nseg > 1) {
    tiles_chain_kernel<S><<<ch.B, 64 * (NT + 1), 0, s>>>(ch);
    BPPSA_CHECK_LAUNCH();
  }
  tiles_apply_kernel<S><<<cut.nseg * ch.B, 64 * (NT + 1), 0, s>>>(ch);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

}  // namespace

// Workspace the preferred cut needs on a device of 256 compute units (with less, a coarser one is taken).
size_t bppsa_tiles_scan_ws(int T, int B, int H) {
  size_t most = 0;
  for (int t_min = 0; t_min <= 1; ++t_min) {
    if (T - t_min < 1) continue;
    const Cut cut = plan_tiles(T - t_min, B, H, 256, (size_t)1 << 40);
    const size_t need = cut.nseg > 0 ? tot_bytes(cut.nseg, B, H) + vin_bytes(cut.nseg, B, H) : 0;
    if (need > most) most = need;
  }
  return most;
}

bppsa_status bppsa_scan_tiles(int T, int B, int H, const float* Jt, const float* seed, float* G, float* g0,
                              void* workspace, size_t workspace_bytes, hipStream_t s) {
  Chain ch;
  ch.T = T; ch.B = B; ch.H = H; ch.n = g0 ? T : T - 1;
  ch.Jt = Jt; ch.seed = seed; ch.G = G; ch.g0 = g0;
  ch.cut = ch.n > 0 ? planned(ch.n, B, H, bppsa_compute_units(), workspace ? workspace_bytes : 0) : Cut{0, 0, 0};
  if ((long long)(ch.cut.nseg + 1) * B > 0x7fffffffLL) return BPPSA_EOVERFLOW;
  ch.tot = static_cast<float*>(workspace);
  ch.vin = reinterpret_cast<float*>(static_cast<char*>(workspace) + tot_bytes(ch.cut.nseg, B, H));
  // 16-byte pieces need rows, and with them tiles, of a multiple of 16 bytes
  const bool vec = H % 4 == 0 && ((uintptr_t)Jt & 15) == 0;
#define BPPSA_TILES(NT) return vec ? launch<Share<NT, true>>(ch, s) : launch<Share<NT, false>>(ch, s)
  switch ((H + 15) / 16) {
    case 1: BPPSA_TILES(1);
    case 2: BPPSA_TILES(2);
    case 3: BPPSA_TILES(3);
    case 4: BPPSA_TILES(4);
    case 5: BPPSA_TILES(5);
    case 6: BPPSA_TILES(6);
    case 7: BPPSA_TILES(7);
    case 8: BPPSA_TILES(8);
    default: return BPPSA_EUNSUPPORTED;
  }
#undef BPPSA_TILES
}
