// Sparse kernels behind the CSR form of A <> B = B A (Section 3.3): a
// row-parallel CSR x dense-vector product for everything that touches the
// gradient vector, and a row-parallel CSR x CSR product for interior up-sweep
// nodes, split into a symbolic phase (row lengths, then ascending column
// indices, both from a per-row bitmap of B's columns held in LDS) and a numeric
// phase, so that the symbolic work can be done once ahead of the training loop
// (Section 4.3).  The numeric phase adds the terms of every value in a fixed order.
#include "bppsa_internal.h"
#include "sparse_common.h"

namespace {

// Positions in a matrix are unsigned: it may have up to 2^31 - 2 entries, and lanes that look up to some 1000 entries past
// the end of a row must not wrap round to the front.

// One workgroup; a thread takes eight consecutive lengths per trip, in two 16-byte pieces where they are
// consecutive in memory, so 8192 of them cost one memory latency and two barriers.
template <bool VEC>
__global__ void __launch_bounds__(1024)
lengths_to_indptr_kernel(int32_t* __restrict__ a, int n, int stride, int32_t* report) {
  constexpr int kPer = 8;
  __shared__ int wave_sum[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int carry = 0;
  for (int base = 0; base < n; base += 1024 * kPer) {
    const int i0 = base + (int)threadIdx.x * kPer;
    int v[kPer], own = 0;
    const bool whole = VEC && i0 + kPer <= n;
    if (whole) {
      const int4 lo = *reinterpret_cast<const int4*>(a + i0), hi = *reinterpret_cast<const int4*>(a + i0 + 4);
      v[0] = lo.x, v[1] = lo.y, v[2] = lo.z, v[3] = lo.w;
      v[4] = hi.x, v[5] = hi.y, v[6] = hi.z, v[7] = hi.w;
    } else {
#pragma unroll
      for (int u = 0; u < kPer; ++u) v[u] = i0 + u < n ? a[(size_t)(i0 + u) * stride] : 0;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) own += v[u];
    int incl = own;
    for (int off = 1; off < 64; off <<= 1) {
      const int t = __shfl_up(incl, off);
      if (lane >= off) incl += t;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = carry, all = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int s = wave_sum[k];
      before += k < wave ? s : 0;
      all += s;
    }
    before += incl - own;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int mine = v[u];
      v[u] = before;
      before += mine;
    }
    if (whole) {
      *reinterpret_cast<int4*>(a + i0) = make_int4(v[0], v[1], v[2], v[3]);
      *reinterpret_cast<int4*>(a + i0 + 4) = make_int4(v[4], v[5], v[6], v[7]);
    } else {
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if (i0 + u < n) a[(size_t)(i0 + u) * stride] = v[u];
    }
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a[(size_t)n * stride] = carry;
    if (report) __hip_atomic_store(report, carry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// LPR lanes per row, FLIGHT entries per lane in flight.  A row is a chain of three memory latencies (bounds,
// entries, gathered values), about 4 us, however long it is up to LPR * FLIGHT entries; the number of rows a
// wave holds side by side (64 / LPR) then decides how many such chains follow one another.
template <int LPR, int FLIGHT>
__global__ void __launch_bounds__(256)
spmv_rows_kernel(int rows, const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                 const float* __restrict__ data, const float* __restrict__ x, float* __restrict__ y,
                 const float* __restrict__ d, float* __restrict__ y2) {
  const int lane = threadIdx.x % LPR;
  const unsigned row = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
  if (row >= (unsigned)rows) return;
  const unsigned s = indptr[row], e = indptr[row + 1];
  const float dv = y2 ? d[row] : 0.f;
  float acc = 0.f;
  for (unsigned p0 = s + lane; p0 < e; p0 += FLIGHT * LPR) {
    int col[FLIGHT];
    float v[FLIGHT], g[FLIGHT];
#pragma unroll
    for (int u = 0; u < FLIGHT; ++u) {
      const unsigned p = p0 + u * LPR;
      col[u] = 0;
      v[u] = 0.f;
      if (p < e) {
        col[u] = indices[p];
        v[u] = data[p];
      }
    }
#pragma unroll
    for (int u = 0; u < FLIGHT; ++u) g[u] = x[col[u]];
#pragma unroll
    for (int u = 0; u < FLIGHT; ++u) acc += p0 + u * LPR < e ? v[u] * g[u] : 0.f;
  }
#pragma unroll
  for (int m = LPR / 2; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
  if (lane == 0) {
    y[row] = acc;
    if (y2) y2[row] = dv * acc;
  }
}

// A wave per row and the vector in LDS: gathered from memory, a vector that does not fit the 32 KB of a compute
// unit's cache costs the lines of every gather again.  The next kTrip entries of a lane are on their way while the
// current ones are added.  Bound by the matrix' bytes: 16384 rows of 2330 (305 MB) by 16384 columns 88 -> 62 us,
// 40000 rows of 1200 (384 MB) by 40960 columns 205 -> 71.
constexpr int kTrip = 4;
constexpr int kSpmvLdsCols = 40960;                // 160 KB, one workgroup of 16 waves to a compute unit
__global__ void __launch_bounds__(1024)
spmv_lds_kernel(int rows, int cols, const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                const float* __restrict__ data, const float* __restrict__ x, float* __restrict__ y,
                const float* __restrict__ d, float* __restrict__ y2) {
  extern __shared__ float xs[];
  const int lane = threadIdx.x & 63, first = blockIdx.x * 16 + (threadIdx.x >> 6), stride = gridDim.x * 16;
  unsigned s = 0, e = 0;
  if (first < rows) {
    s = indptr[first];
    e = indptr[first + 1];
  }
  for (int c0 = threadIdx.x; c0 < cols; c0 += 4 * 1024) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = x[c0 + 1024 * u < cols ? c0 + 1024 * u : cols - 1];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (c0 + 1024 * u < cols) xs[c0 + 1024 * u] = v[u];
  }
  __syncthreads();
  struct Trip {
    int col[kTrip];
    float v[kTrip];
  };
  auto fetch = [&](Trip& t, unsigned p0) {         // past the end of the row: its last entry, not added
#pragma unroll
    for (int u = 0; u < kTrip; ++u) {
      const unsigned p = min(p0 + u * 64, e - 1);
      t.col[u] = indices[p];
      t.v[u] = data[p];
    }
  };
  for (int row = first; row < rows; row += stride) {
    const float dv = y2 ? d[row] : 0.f;
    float acc = 0.f;
    auto add = [&](const Trip& t, unsigned p0) {
#pragma unroll
      for (int u = 0; u < kTrip; ++u) acc += p0 + u * 64 < e ? t.v[u] * xs[t.col[u]] : 0.f;
    };
    if (e > s) {                                   // uniform over the wave
      Trip even, odd;
      unsigned p0 = s + lane;                      // trips start at the same place for all lanes of the wave
      fetch(even, p0);
      for (unsigned base = s;; base += 2 * kTrip * 64, p0 += 2 * kTrip * 64) {
        fetch(odd, p0 + kTrip * 64);
        add(even, p0);
        if (base + kTrip * 64 >= e) break;
        fetch(even, p0 + 2 * kTrip * 64);
        add(odd, p0 + kTrip * 64);
        if (base + 2 * kTrip * 64 >= e) break;
      }
    }
    if (row + stride < rows) {
      s = indptr[row + stride];
      e = indptr[row + stride + 1];
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
    if (lane == 0) {
      y[row] = acc;
      if (y2) y2[row] = dv * acc;
    }
  }
}

// One lane per row: for matrices with about one entry per row (ReLU, max-pooling).
__global__ void __launch_bounds__(256)
spmv_lane_kernel(int rows, const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                 const float* __restrict__ data, const float* __restrict__ x, float* __restrict__ y,
                 const float* __restrict__ d, float* __restrict__ y2) {
  const unsigned row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= (unsigned)rows) return;
  const int s = indptr[row], e = indptr[row + 1];
  float acc = 0.f;
  for (int p = s; p < e; ++p) acc += data[p] * x[indices[p]];
  y[row] = acc;
  if (y2) y2[row] = d[row] * acc;
}

__global__ void __launch_bounds__(256)
check_diagonals_kernel(bppsa_diagonal_batch batch, int* __restrict__ bad) {
  const int k = blockIdx.y, rows = batch.rows[k];
  const int32_t* __restrict__ indptr = batch.indptr[k];
  const int32_t* __restrict__ indices = batch.indices[k];
  bool ok = true;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i <= rows; i += gridDim.x * blockDim.x) {
    ok = ok && indptr[i] == i;
    if (i < rows) ok = ok && indices[i] == i;
  }
  if (!ok) bad[k] = 1;
}

// *bad is set if the arrays differ.
__global__ void __launch_bounds__(256)
check_same_kernel(long long n, const int32_t* __restrict__ a, const int32_t* __restrict__ b, int* __restrict__ bad) {
  bool ok = true;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    ok = ok && a[i] == b[i];
  if (!ok) *bad = 1;
}

// Mark, in an LDS bitmap, every column of B reachable from row `row` of A.  Waves take
// entries of A's row, lanes take entries of the matching row of B.  Returns (to every
// thread of wave 0, lane 0 only is used) nothing; the caller syncs.
__device__ __forceinline__ unsigned long long
mark_row(int row, const int32_t* __restrict__ a_indptr, const int32_t* __restrict__ a_indices,
         const int32_t* __restrict__ b_indptr, const int32_t* __restrict__ b_indices,
         unsigned int* bitmap) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
  const unsigned as = a_indptr[row], ae = a_indptr[row + 1];
  unsigned long long work = 0;
  for (unsigned p = as + wave; p < ae; p += nwave) {
    const int k = a_indices[p];
    const unsigned bs = b_indptr[k], be = b_indptr[k + 1];
    for (unsigned q = bs + lane; q < be; q += 64) {
      const int col = b_indices[q];
      atomicOr(&bitmap[col >> 5], 1u << (col & 31));
    }
    if (lane == 0) work += (unsigned long long)(be - bs);
  }
  return work;
}

// MODE 0: row length -> c_indptr[row], multiply-add count -> *madds.
// MODE 1: ascending column indices -> c_indices[c_indptr[row] ...].
template <int MODE>
__global__ void __launch_bounds__(256)
spgemm_symbolic_kernel(int words, const int32_t* __restrict__ a_indptr,
                       const int32_t* __restrict__ a_indices, const int32_t* __restrict__ b_indptr,
                       const int32_t* __restrict__ b_indices, int32_t* __restrict__ c_indptr,
                       int32_t* __restrict__ c_indices, unsigned long long* __restrict__ madds) {
  extern __shared__ unsigned int bitmap[];
  __shared__ int wave_sum[4];
  __shared__ int carry_s;
  const int row = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int wd = threadIdx.x; wd < words; wd += blockDim.x) bitmap[wd] = 0u;
  __syncthreads();
  const unsigned long long work = mark_row(row, a_indptr, a_indices, b_indptr, b_indices, bitmap);
  __syncthreads();
  if (MODE == 0) {
    int cnt = 0;
    for (int wd = threadIdx.x; wd < words; wd += blockDim.x) cnt += __popc(bitmap[wd]);
    for (int m = 32; m >= 1; m >>= 1) cnt += __shfl_xor(cnt, m);
    if (lane == 0) wave_sum[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) c_indptr[row] = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    if (lane == 0 && work) atomicAdd(madds, work);
  } else {
    int carry = c_indptr[row];
    for (int base = 0; base < words; base += 256) {
      const int wd = base + threadIdx.x;
      unsigned int bits = (wd < words) ? bitmap[wd] : 0u;
      const int v = __popc(bits);
      int incl = v;
      for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(incl, off);
        if (lane >= off) incl += t;
      }
      if (lane == 63) wave_sum[wave] = incl;
      __syncthreads();
      int woff = 0;
      for (int k = 0; k < wave; ++k) woff += wave_sum[k];
      int pos = carry + woff + incl - v;
      while (bits) {
        const int b = __ffs(bits) - 1;
        c_indices[pos++] = wd * 32 + b;
        bits &= bits - 1u;
      }
      if (threadIdx.x == 255) carry_s = carry + woff + incl;
      __syncthreads();
      carry = carry_s;
      __syncthreads();
    }
  }
}

// ---- fingerprint of an index array ----------------------------------------------------------------
// Each element contributes two 64-bit words, bit-mixed from (position, value, salt) with the
// multiply-xorshift finaliser of the SplitMix64 generator; the words of all elements are summed
// modulo 2^64, so the result is independent of the order in which waves arrive.
__device__ __forceinline__ unsigned long long mix64(unsigned long long x) {
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  x ^= x >> 31;
  return x;
}

__global__ void __launch_bounds__(256)
pattern_hash_kernel(bppsa_hash_batch batch, unsigned long long* __restrict__ out) {
  const int32_t* __restrict__ a = batch.array[blockIdx.y];
  const long long count = batch.count[blockIdx.y];
  const unsigned long long salt = batch.salt[blockIdx.y];
  unsigned long long h0 = 0, h1 = 0;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
    const unsigned long long x = ((unsigned long long)i << 32) | (unsigned int)a[i];
    h0 += mix64(x ^ (salt * 0x9e3779b97f4a7c15ull));
    h1 += mix64((x + salt) * 0xd1342543de82ef95ull + 1);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    h0 += __shfl_down(h0, off, 64);
    h1 += __shfl_down(h1, off, 64);
  }
  if ((threadIdx.x & 63) == 0 && (h0 | h1) != 0) {
    atomicAdd(out, h0);
    atomicAdd(out + 1, h1);
  }
}

// ---- numeric phase of C = A B for a known structure ---------------------------------------------
// Every value of C is formed by ONE wave, which adds the terms of an entry in an order fixed by
// the structure of A and B alone, so the values are the same bits on every run; no two waves ever
// add to the same accumulator.  Three kernels, chosen once per product when the plan is built:
//
//   single : every entry of C is exactly one product a * b (the number of multiply-adds equals
//            nnz(C): a diagonal or selection matrix on either side, i.e. every product with a ReLU
//            or pooling Jacobian).  Nothing is summed; one wave per row writes the products to
//            their places.
//   scale  : one side is an input with the pattern of the identity and C has the other side's indices
//            entry for entry: its values times the row's or the column's factor.
//   wave   : rows of C of up to kWaveRowCap entries: one wave per row stages the row's column
//            indices in LDS, walks A's row and adds each term at the slot found by binary search.
//   block  : longer rows: one workgroup of 4, 8 or 16 waves per row (bppsa_spgemm_ways).  The columns are
//            cut into as many equal ranges, one per wave, and a table built with the plan says where
//            each row of B crosses those boundaries, so a wave reads exactly its share of every row
//            of B and owns its share of the accumulators: one per column of B, or one per entry of
//            the longest row of C plus a rank table (whichever takes less LDS), or, when neither
//            fits kBlockLdsBytes, the row itself in global memory.
constexpr int kWaveRowCap = 1024;
// Most LDS one workgroup of the BLOCK kinds takes: all that a compute unit has.  A row that does not fit is
// added up in global memory at a tenth of the speed: 4096 rows, 24000 columns, 2048 rows of 512 in B, 9912 us
// with 64 KB as the most, 766 with one workgroup of 16 waves to a compute unit.
constexpr size_t kBlockLdsBytes = 160 * 1024;

// first position in sorted idx[0..n) whose value is >= col
__device__ __forceinline__ int lower_bound_i32(const int32_t* idx, int n, int col) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (idx[mid] < col) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// split[(ways - 1) k + j] = first entry of row k of B whose column is >= (j + 1) * ceil(cols / ways)
__global__ void __launch_bounds__(256)
row_splits_kernel(int rows, int cols, int ways, const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                  int32_t* __restrict__ split) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (ways - 1) * rows) return;
  const int k = t / (ways - 1), j = t - (ways - 1) * k;
  const int range = (cols + ways - 1) / ways;
  const int s = indptr[k], e = indptr[k + 1];
  split[t] = s + lower_bound_i32(indices + s, e - s, (j + 1) * range);
}

__global__ void __launch_bounds__(256)
spgemm_numeric_single_kernel(int rows, const int32_t* __restrict__ a_indptr, const int32_t* __restrict__ a_indices,
                             const float* __restrict__ a_data, const int32_t* __restrict__ b_indptr,
                             const int32_t* __restrict__ b_indices, const float* __restrict__ b_data,
                             const int32_t* __restrict__ c_indptr, const int32_t* __restrict__ c_indices,
                             float* __restrict__ c_data) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int cs = c_indptr[row], n = c_indptr[row + 1] - cs;
  if (n == 0) return;
  const unsigned as = a_indptr[row], ae = a_indptr[row + 1];
  if (ae - as == 1) {                            // the row of C is a scaled copy of one row of B
    const int k = a_indices[as];
    const float av = a_data[as];
    const int bs = b_indptr[k];
    for (int j = lane; j < n; j += 64) c_data[cs + j] = av * b_data[bs + j];
    return;
  }
  // One lane per entry of A's row, with its (short) row of B.  Where B keeps the order of the columns (a
  // diagonal, and a selection inside one row of the image) an entry's place is the number of entries before
  // it: one coalesced read of C's indices confirms that, and only the lanes it does not fit search.  The
  // search is eight to thirteen dependent loads and was most of the kernel's time: 8192 rows of a product with a
// diagonal, 47 -> 27 us.
  int before = 0;
  for (unsigned p0 = as; p0 < ae; p0 += 64) {
    const unsigned p = p0 + lane;
    int bs = 0, be = 0;
    float av = 0.f;
    if (p < ae) {
      const int k = a_indices[p];
      av = a_data[p];
      bs = b_indptr[k];
      be = b_indptr[k + 1];
    }
    const unsigned long long with = __ballot(be > bs);
    int guess = before + __builtin_amdgcn_mbcnt_hi((unsigned)(with >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)with, 0u));
    before += __builtin_popcountll(with);
    for (int q = bs; q < be; ++q, ++guess) {
      const int col = b_indices[q];
      int slot = guess;
      if (slot >= n || c_indices[cs + slot] != col) slot = lower_bound_i32(c_indices + cs, n, col);
      c_data[cs + slot] = av * b_data[q];
    }
  }
}

// C = D B and C = A D for a diagonal D, where C has the other factor's pattern.  The kernel above finds a
// diagonal's entry through its row pointers and indices, four gathers of 64 lines each per 64 entries (the bound:
// four stretches in flight instead of one changed nothing), and reads C's indices as well; here one gather is
// left, or none.  8192 rows of 320 by a diagonal: 27.5 -> 12.5 us; a diagonal by 16384 rows of 194: 28 -> 8.
__global__ void __launch_bounds__(256)
scale_rows_kernel(int rows, const int32_t* __restrict__ indptr, const float* __restrict__ d,
                  const float* __restrict__ b_data, float* __restrict__ c_data) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const unsigned s = indptr[row], e = indptr[row + 1];
  const float dv = d[row];
  for (unsigned p0 = s + lane; p0 < e; p0 += 256) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = b_data[min(p0 + 64 * u, e - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (p0 + 64 * u < e) c_data[p0 + 64 * u] = dv * v[u];
  }
}

__global__ void __launch_bounds__(256)
scale_columns_kernel(int64_t nnz, const int32_t* __restrict__ indices, const float* __restrict__ a_data,
                     const float* __restrict__ d, float* __restrict__ c_data) {
  const int64_t p0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  int col[4];
  float v[4], f[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t p = p0 + 256 * u < nnz ? p0 + 256 * u : nnz - 1;
    col[u] = indices[p];
    v[u] = a_data[p];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) f[u] = d[col[u]];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (p0 + 256 * u < nnz) c_data[p0 + 256 * u] = v[u] * f[u];
}

__global__ void __launch_bounds__(256)
spgemm_numeric_wave_kernel(int rows, const int32_t* __restrict__ a_indptr, const int32_t* __restrict__ a_indices,
                           const float* __restrict__ a_data, const int32_t* __restrict__ b_indptr,
                           const int32_t* __restrict__ b_indices, const float* __restrict__ b_data,
                           const int32_t* __restrict__ c_indptr, const int32_t* __restrict__ c_indices,
                           float* __restrict__ c_data) {
  __shared__ int32_t cidx_s[4][kWaveRowCap];
  __shared__ float acc_s[4][kWaveRowCap];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x * 4 + wave;
  if (row >= rows) return;                       // no workgroup barrier below: waves are independent
  int32_t* cidx = cidx_s[wave];
  float* acc = acc_s[wave];
  const int cs = c_indptr[row], n = c_indptr[row + 1] - cs;
  if (n == 0) return;
  const unsigned as = a_indptr[row], ae = a_indptr[row + 1];
  for (int j = lane; j < n; j += 64) {
    cidx[j] = c_indices[cs + j];
    acc[j] = 0.f;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  // Entries of A's row in storage order; the entries of one row of B have distinct columns, so
  // the lanes of one step never meet at a slot, and LDS operations of a wave complete in order.
  // Each lane first fetches one entry of A's row and the bounds of its row of B; the wave then
  // takes them four at a time so that the loads of four rows of B are in flight together.
  for (unsigned p0 = as; p0 < ae; p0 += 64) {
    const unsigned mine = p0 + lane;
    int bs_l = 0, be_l = 0;
    float av_l = 0.f;
    if (mine < ae) {
      const int k = a_indices[mine];
      av_l = a_data[mine];
      bs_l = b_indptr[k];
      be_l = b_indptr[k + 1];
    }
    const int cnt = (ae - p0 < 64) ? (int)(ae - p0) : 64;
    for (int e = 0; e < cnt; e += 4) {
      unsigned bs[4], be[4];
      int col[4];
      float av[4], bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int src = (e + u < cnt) ? e + u : e;
        bs[u] = __builtin_amdgcn_readlane(bs_l, src);
        be[u] = (e + u < cnt) ? __builtin_amdgcn_readlane(be_l, src) : bs[u];
        av[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, av_l), src));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned q = bs[u] + lane;
        col[u] = (q < be[u]) ? b_indices[q] : -1;
        bv[u] = (q < be[u]) ? b_data[q] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (col[u] >= 0) acc[lower_bound_i32(cidx, n, col[u])] += av[u] * bv[u];
        for (unsigned q0 = bs[u] + 64 + lane; q0 < be[u]; q0 += 64)      // a row of B longer than one wave
          acc[lower_bound_i32(cidx, n, b_indices[q0])] += av[u] * b_data[q0];
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  for (int j = lane; j < n; j += 64) c_data[cs + j] = acc[j];
}

// Where an accumulator lies: its column with the six bits that say the LDS bank turned by a hash of the others.  The
// columns of a convolution's row are a few positions of many channels, which fall into few banks (conflicts 118 -> 73 M
// cycles, 1 % of the time).
__device__ __forceinline__ int turned(int c) { return c ^ (int)((((unsigned)c >> 6) * 0x9E3779B1u) >> 26); }

__global__ void __launch_bounds__(256)
cols16_kernel(long long nnz, const int32_t* __restrict__ indices, uint16_t* __restrict__ cols) {
  for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < nnz; p += (long long)gridDim.x * 256)
    cols[p] = (uint16_t)turned(indices[p]);
}

// One workgroup of WAYS waves per row of C; wave w owns the columns [w q, (w + 1) q), q = ceil(cols / WAYS),
// and with them every value of the row that falls there, so each value is summed by one wave in
// one order.
//   MODE 0: one LDS accumulator per column of B.
//   MODE 1: one LDS accumulator per entry of the row; the place of a column is its rank among the
//           row's columns, read from a table of (bits, entries before) per 32 columns.
//   MODE 2: the row stays in global memory, places by binary search; the additions are memory-side
//           add operations, all additions to one entry issued by one wave in program order.
// The wave walks A's row 64 entries at a time (one per lane: value and the bounds of its share of
// the row of B), and takes their shares in pieces of 64 entries: first pieces of all entries, then
// second pieces, and so on.  Pieces are fetched kDepth at a time and the fetch of the next kDepth
// is issued before the current ones are added, so the additions run under the memory latency.  For
// that the loads stand outside every branch (a lane past the end of its share repeats the last
// entry) and the two sets take turns without a copy: behind a branch, or for a copy, the compiler waits
// for everything in flight.  Three at a time, with stretches of 128 rows: two are better where B comes from
// the die's L2 (544 us for the first product below) and worse where it does not (4096 rows of 100 random columns by
// 16384 columns, 320 a row: 407, against 392 with three and 391 with four); six 585.
// What bounds it is the path that returns loads (busy all the time in the counters), with the dies' L2 behind it: half of
// the requests miss it and take 6 TB/s.  So the columns are read as 16 bits from a copy that the plan keeps, six bytes an
// entry instead of eight, and a batch of 64 entries that all have a piece is walked four pieces at a time without looking
// for the next entry (14 scalar instructions a piece before, 7 now).  4096 x 8192 by 8192 x 8192,
// 320 entries a row in both, 454 M multiply-adds: 876 us at first, 675 with the order of the rows (85) and 32-bit
// offsets (25), 580 with eight waves, 571 with longer stretches, 514 with 16-bit columns, 462 now; 8192 rows of a
// smaller product 126, 92, 91, 81; MODE 1, 16384 rows 222, 199 with batches fetched ahead, 189 now.  Not kept, for their
// instructions: two neighbouring entries a lane
// (1040 us), a scalar base per piece (754); LDS add operations
// in place of read, add and write (2880); 3, 5 and 6 waves, which fill their pieces better (754, 660 and 650
// against 682 with 4 and 587 with 8) but leave the four SIMDs unequal shares.  Columns cut among the dies, so that each
// reads a range of B that its L2 holds, with a wave to a row and range: a third of the misses and no less time (455), with
// any number of ranges; column and value packed into one record of eight bytes there: 523, more accesses for the bytes.
constexpr int kDepth = 3;

typedef float v4f __attribute__((ext_vector_type(4)));

struct Pieces {
  int col[kDepth];
  float bv[kDepth];
  float av[kDepth];
  bool on[kDepth];
};

// How a kernel reads B's columns: its own indices with a 32-bit offset, with a 64-bit one (B has 2^30 entries or more),
// or the plan's copy in 16 bits, turned (MODE 0).
enum { kCols32, kCols64, kCols16 };

// takes up to kDepth entries out of `todo` (one bit per lane whose share has a piece number `round`);
// `src` is a lane with such a piece, and the last one taken afterwards
template <int COLS>
__device__ __forceinline__ void fetch_pieces(Pieces& pc, unsigned long long& todo, int& src, int round, int lane,
                                             int bs_l, int be_l, float av_l, const void* __restrict__ b_cols,
                                             const float* __restrict__ b_data) {
#pragma unroll
  for (int u = 0; u < kDepth; ++u) {
    const bool more = todo != 0;                         // uniform over the wave
    src = more ? __builtin_ctzll(todo) : src;
    todo &= todo - 1;
    const unsigned e = __builtin_amdgcn_readlane(be_l, src);
    unsigned q = __builtin_amdgcn_readlane(bs_l, src) + 64u * round + lane;
    pc.av[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, av_l), src));
    pc.on[u] = more && q < e;
    q = min(q, e - 1);                                   // (a lane that is taken has entries)
    if (COLS == kCols64) {
      pc.col[u] = static_cast<const int32_t*>(b_cols)[q];
      pc.bv[u] = b_data[q];
    } else {                                             // the arrays' own bases and a 32-bit offset per lane
      const unsigned off = 4u * q;
      if (COLS == kCols16) pc.col[u] = *reinterpret_cast<const uint16_t*>(static_cast<const char*>(b_cols) + 2u * q);
      else pc.col[u] = *reinterpret_cast<const int32_t*>(static_cast<const char*>(b_cols) + off);
      pc.bv[u] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(b_data) + off);
    }
  }
}

// The same for lanes src .. src + kRun - 1, all of which have a first piece.
constexpr int kRun = 4;

struct Run {
  int col[kRun];
  float bv[kRun];
  float av[kRun];
  bool on[kRun];
};

template <int COLS>
__device__ __forceinline__ void fetch_run(Run& pc, int src, int lane, int bs_l, int be_l, float av_l,
                                          const void* __restrict__ b_cols, const float* __restrict__ b_data) {
#pragma unroll
  for (int u = 0; u < kRun; ++u) {
    const unsigned e = __builtin_amdgcn_readlane(be_l, src + u);
    unsigned q = __builtin_amdgcn_readlane(bs_l, src + u) + (unsigned)lane;
    pc.av[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, av_l), src + u));
    pc.on[u] = q < e;
    q = min(q, e - 1);
    if (COLS == kCols64) {
      pc.col[u] = static_cast<const int32_t*>(b_cols)[q];
      pc.bv[u] = b_data[q];
    } else {
      const unsigned off = 4u * q;
      if (COLS == kCols16) pc.col[u] = *reinterpret_cast<const uint16_t*>(static_cast<const char*>(b_cols) + 2u * q);
      else pc.col[u] = *reinterpret_cast<const int32_t*>(static_cast<const char*>(b_cols) + off);
      pc.bv[u] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(b_data) + off);
    }
  }
}

// Neighbouring rows of a convolution's Jacobian (the positions of one channel) meet the same rows of B, so
// stretches of rows go to one die, whose L2 then serves them: workgroup b runs on die b % 8.  `stretch` is
// short enough that every die gets four (128 against 64: 4096 rows of 320 by rows of 320 580 -> 570 us, 16384 rows of
// 106 by rows of 194 199 -> 193).
__host__ __device__ __forceinline__ int block_stretch(int rows) { return rows >= 4096 ? 128 : rows / 32 + 1; }
__host__ __device__ __forceinline__ int block_grid(int rows) {
  const int s = 8 * block_stretch(rows);
  return (rows + s - 1) / s * s;
}

template <int MODE, int COLS, int WAYS>
__global__ void __launch_bounds__(64 * WAYS)
spgemm_numeric_block_kernel(int rows, int b_cols, const int32_t* __restrict__ a_indptr,
                            const int32_t* __restrict__ a_indices, const float* __restrict__ a_data,
                            const int32_t* __restrict__ b_indptr, const void* __restrict__ b_indices,
                            const float* __restrict__ b_data, const int32_t* __restrict__ b_split,
                            const int32_t* __restrict__ c_indptr, const int32_t* __restrict__ c_indices,
                            float* __restrict__ c_data) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int stretch = block_stretch(rows);
  const int turn = blockIdx.x >> 3;
  const int row = (turn / stretch * 8 + (int)(blockIdx.x & 7)) * stretch + turn % stretch;
  if (row >= rows) return;                       // uniform over the workgroup
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cs = c_indptr[row], n = c_indptr[row + 1] - cs;
  const unsigned as = a_indptr[row], ae = a_indptr[row + 1];
  if (n == 0) return;                            // uniform over the workgroup
  // This lane's entry of A's row: value and bounds of its share of the row of B.  Fetched one batch ahead, the
  // first one before the accumulators are cleared: three loads that wait for one another.
  int bs_l, be_l;
  float av_l;
  auto fetch_batch = [&](unsigned p0) {
    const unsigned mine = p0 + lane, at = mine < ae ? mine : ae - 1;         // n > 0: A's row has entries
    const int k = a_indices[at];
    av_l = a_data[at];
    bs_l = wave == 0 ? b_indptr[k] : b_split[(WAYS - 1) * k + wave - 1];
    be_l = wave == WAYS - 1 ? b_indptr[k + 1] : b_split[(WAYS - 1) * k + wave];
    be_l = mine < ae ? be_l : bs_l;
  };
  fetch_batch(as);
  // the row's columns, four loads of a thread in flight at a time
  constexpr int kThreads = 64 * WAYS;
  auto each_column = [&](auto&& use) {
    for (int p0 = threadIdx.x; p0 < n; p0 += 4 * kThreads) {
      int c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) c[u] = c_indices[cs + (p0 + u * kThreads < n ? p0 + u * kThreads : n - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (p0 + u * kThreads < n) use(p0 + u * kThreads, c[u]);
    }
  };
  // MODE 1: rank table first (8 bytes per 32 columns), then the accumulators
  const int words = (b_cols + 31) >> 5;
  uint2* rk = reinterpret_cast<uint2*>(lds);
  float* cacc = lds + 2 * words;
  if (MODE == 0 && b_cols <= 8 * n) {            // (uniform; all of it: four at a time, and no index is read)
    const int all = COLS == kCols16 ? (b_cols + 63) & ~63 : b_cols;
    for (int p = 4 * threadIdx.x; p < all; p += 4 * kThreads) *reinterpret_cast<v4f*>(lds + p) = v4f{0.f, 0.f, 0.f, 0.f};
  } else if (MODE == 0) {
    each_column([&](int, int c) { lds[COLS == kCols16 ? turned(c) : c] = 0.f; });
  } else if (MODE == 1) {
    for (int w = threadIdx.x; w < words; w += blockDim.x) rk[w] = make_uint2(0u, 0u);
    __syncthreads();
    each_column([&](int p, int c) {
      atomicOr(&rk[c >> 5].x, 1u << (c & 31));   // integer: the result does not depend on the order
      int before = __shfl_up(c, 1);
      if (lane == 0) before = p > 0 ? c_indices[cs + p - 1] : -1;
      if ((before >> 5) != (c >> 5)) rk[c >> 5].y = (unsigned)p;
      cacc[p] = 0.f;
    });
  } else {
    for (int p = threadIdx.x; p < n; p += blockDim.x) c_data[cs + p] = 0.f;
  }
  __syncthreads();
  const int range = (b_cols + WAYS - 1) / WAYS;
  int slot_lo = 0, slot_n = n;                   // MODE 2: the places of this wave's columns
  if (MODE == 2) {
    slot_lo = lower_bound_i32(c_indices + cs, n, wave * range);
    slot_n = lower_bound_i32(c_indices + cs, n, (wave + 1) * range) - slot_lo;
  }
  auto add = [&](const auto& pc) {
#pragma unroll
    for (int u = 0; u < (int)(sizeof(pc.col) / sizeof(pc.col[0])); ++u) {
      const int c = pc.col[u];
      if (pc.on[u]) {                            // the lanes of one piece hold distinct columns
        const float t = pc.av[u] * pc.bv[u];
        if (MODE == 0) {
          lds[c] += t;
        } else if (MODE == 1) {
          const uint2 r = rk[c >> 5];
          cacc[r.y + __builtin_popcount(r.x & ((1u << (c & 31)) - 1u))] += t;
        } else {
          atomicAdd(&c_data[cs + slot_lo + lower_bound_i32(c_indices + cs + slot_lo, slot_n, c)], t);
        }
      }
    }
  };
  for (unsigned p0 = as; p0 < ae; p0 += 64) {
    const int bs = bs_l, be = be_l;
    const float av = av_l;
    if (p0 + 64 < ae) fetch_batch(p0 + 64);
    for (int round = 0;; ++round) {
      unsigned long long todo = __ballot(be - bs > 64 * round);
      if (todo == 0) break;
      if (round == 0 && todo == ~0ull) {           // a full batch: no entry is looked for
        Run even, odd;
        fetch_run<COLS>(even, 0, lane, bs, be, av, b_indices, b_data);
#pragma unroll 1
        for (int src = 0;; src += 2 * kRun) {
          fetch_run<COLS>(odd, src + kRun, lane, bs, be, av, b_indices, b_data);
          add(even);
          if (src + 2 * kRun >= 64) break;
          fetch_run<COLS>(even, src + 2 * kRun, lane, bs, be, av, b_indices, b_data);
          add(odd);
        }
        add(odd);
        continue;
      }
      int src = __builtin_ctzll(todo);
      Pieces even, odd;
      fetch_pieces<COLS>(even, todo, src, round, lane, bs, be, av, b_indices, b_data);
      while (true) {
        const bool then = todo != 0;
        fetch_pieces<COLS>(odd, todo, src, round, lane, bs, be, av, b_indices, b_data);
        add(even);
        if (!then) break;
        const bool again = todo != 0;
        fetch_pieces<COLS>(even, todo, src, round, lane, bs, be, av, b_indices, b_data);
        add(odd);
        if (!again) break;
      }
    }
  }
  if (MODE == 2) return;
  __syncthreads();
  if (MODE == 0) {
    each_column([&](int p, int c) { c_data[cs + p] = lds[COLS == kCols16 ? turned(c) : c]; });
  } else {
    for (int p = threadIdx.x; p < n; p += blockDim.x) c_data[cs + p] = cacc[p];
  }
}

}  // namespace

bppsa_status bppsa_lengths_to_indptr(int32_t* a, int n, hipStream_t stream, int stride, int32_t* report) {
  if (stride == 1 && ((uintptr_t)a & 15) == 0)
    lengths_to_indptr_kernel<true><<<1, 1024, 0, stream>>>(a, n, stride, report);
  else
    lengths_to_indptr_kernel<false><<<1, 1024, 0, stream>>>(a, n, stride, report);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_launch_spmv(const bppsa_csr& A, const float* x, float* y, hipStream_t stream,
                               const float* d, float* y2) {
  if (A.rows < 1) return BPPSA_OK;
#define BPPSA_SPMV(LPR, FLIGHT)                                                                          \
  spmv_rows_kernel<LPR, FLIGHT><<<bppsa_ceil_div(A.rows, 256 / LPR), 256, 0, stream>>>(                  \
      A.rows, A.indptr, A.indices, A.data, x, y, d, y2)
  // Measured over means of 10 to 6300 entries a row, thirteen forms: the fewest lanes with which a row takes
  // one or two trips.  16384 rows of 160: 9.1 us (64 lanes, four in flight: 9.9); 65536 of 100: 16.9 (20.8);
  // 4096 of 6300: 67.7 (72.6); 512 of 51: 6.4 (7.0).
  const int64_t mean = A.nnz / A.rows;
  // The vector in LDS, where there are entries enough to make up for staging it, rows enough for the waves and
  // trips enough for a wave; up to 8192 columns the cache holds it, and fewer waves to a compute unit than the
  // kernels below put there cost more.  us, those against this one, 16384 columns: 4096 rows of 450 6.3 / 7.6, of
  // 600 9.8 / 6.3; 16384 rows of 106 7.1 / 8.4, of 194 11.1 / 9.5, of 600 34.7 / 16.6; 2048 rows of 2400 9.5 / 11.1;
  // 4096 columns, 16384 rows of 600 15.8 / 14.3; 2048 columns, of 320 9.0 / 9.7.
  if (mean >= 192 && A.nnz >= 2400000 && A.rows >= (A.cols > 8192 ? 4096 : 8192) && A.cols >= 4096 &&
      A.cols <= kSpmvLdsCols) {
    const size_t lds = (size_t)A.cols * sizeof(float);
    if (lds > 48 * 1024)
      BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)spmv_lds_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        kSpmvLdsCols * (int)sizeof(float)));
    const int most = A.cols > kSpmvLdsCols / 2 ? 256 : 512, groups = bppsa_ceil_div(A.rows, 16);
    spmv_lds_kernel<<<groups < most ? groups : most, 1024, lds, stream>>>(A.rows, A.cols, A.indptr, A.indices, A.data, x,
                                                                          y, d, y2);
  } else if (mean >= 512) BPPSA_SPMV(64, 8);
  else if (mean >= 64) BPPSA_SPMV(32, 4);
  else if (mean >= 16) BPPSA_SPMV(16, 4);
  else if (mean >= 4) BPPSA_SPMV(8, 4);
  else
    spmv_lane_kernel<<<bppsa_ceil_div(A.rows, 256), 256, 0, stream>>>(A.rows, A.indptr, A.indices, A.data, x, y,
                                                                      d, y2);
#undef BPPSA_SPMV
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_launch_check_diagonals(const bppsa_diagonal_batch& batch, int n, int* bad, hipStream_t stream) {
  if (n < 1) return BPPSA_OK;
  if (n > BPPSA_DIAGONAL_BATCH) return BPPSA_EINVAL;
  int most = 0;
  for (int k = 0; k < n; ++k) most = batch.rows[k] > most ? batch.rows[k] : most;
  int groups = most / (256 * 4) + 1;
  if (groups > 64) groups = 64;
  check_diagonals_kernel<<<dim3(groups, n), 256, 0, stream>>>(batch, bad);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_launch_check_same(int64_t n, const int32_t* a, const int32_t* b, int* bad, hipStream_t stream) {
  if (n < 1) return BPPSA_OK;
  const int64_t groups = (n + 1023) / 1024;
  check_same_kernel<<<groups < 1024 ? (int)groups : 1024, 256, 0, stream>>>(n, a, b, bad);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

static int bitmap_words(const bppsa_csr& B) { return (B.cols + 31) / 32; }

bppsa_status bppsa_launch_spgemm_count(const bppsa_csr& A, const bppsa_csr& B, int32_t* c_indptr,
                                       unsigned long long* madds, hipStream_t stream) {
  if (B.cols > kBppsaMaxSpgemmCols) return BPPSA_ESHAPE;
  const int words = bitmap_words(B);
  const size_t lds = (size_t)words * sizeof(unsigned int);
  if (lds > 48 * 1024)
    BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)spgemm_symbolic_kernel<0>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  spgemm_symbolic_kernel<0><<<A.rows, 256, lds, stream>>>(words, A.indptr, A.indices, B.indptr, B.indices,
                                                          c_indptr, nullptr, madds);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_launch_spgemm_indices(const bppsa_csr& A, const bppsa_csr& B, const int32_t* c_indptr,
                                         int32_t* c_indices, hipStream_t stream) {
  if (B.cols > kBppsaMaxSpgemmCols) return BPPSA_ESHAPE;
  const int words = bitmap_words(B);
  const size_t lds = (size_t)words * sizeof(unsigned int);
  if (lds > 48 * 1024)
    BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)spgemm_symbolic_kernel<1>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  spgemm_symbolic_kernel<1><<<A.rows, 256, lds, stream>>>(words, A.indptr, A.indices, B.indptr, B.indices,
                                                          const_cast<int32_t*>(c_indptr), c_indices, nullptr);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_launch_pattern_hash(const bppsa_hash_batch& batch, int n, unsigned long long* out,
                                       hipStream_t stream) {
  if (n < 1) return BPPSA_OK;
  if (n > BPPSA_HASH_BATCH) return BPPSA_EINVAL;
  pattern_hash_kernel<<<dim3(64, n), 256, 0, stream>>>(batch, out);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_launch_row_splits(const bppsa_csr& B, int ways, int32_t* split, hipStream_t stream) {
  if (B.rows < 1) return BPPSA_OK;
  row_splits_kernel<<<bppsa_ceil_div((ways - 1) * B.rows, 256), 256, 0, stream>>>(B.rows, B.cols, ways, B.indptr,
                                                                                  B.indices, split);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

bppsa_status bppsa_launch_cols16(const bppsa_csr& B, uint16_t* cols, hipStream_t stream) {
  if (B.nnz < 1) return BPPSA_OK;
  const int64_t groups = (B.nnz + 1023) / 1024;
  cols16_kernel<<<(int)(groups < 2048 ? groups : 2048), 256, 0, stream>>>(B.nnz, B.indices, cols);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

static size_t dense_lds_bytes(int b_cols) { return (size_t)b_cols * sizeof(float); }
static size_t ranked_lds_bytes(int c_max_row, int b_cols) {
  return (size_t)c_max_row * sizeof(float) + (size_t)((b_cols + 31) / 32) * 8;
}

int bppsa_spgemm_numeric_kind(int64_t madds, int64_t c_nnz, int c_max_row, int b_cols) {
  if (madds == c_nnz) return BPPSA_SPGEMM_SINGLE;
  if (c_max_row <= kWaveRowCap) return BPPSA_SPGEMM_WAVE;
  const size_t dense = dense_lds_bytes(b_cols), ranked = ranked_lds_bytes(c_max_row, b_cols);
  // one accumulator per column costs one LDS access less per term: it wins unless the rank table
  // and the row's accumulators are clearly smaller (more workgroups per compute unit)
  if (dense <= kBlockLdsBytes && (dense <= 16 * 1024 || 4 * dense <= 5 * ranked)) return BPPSA_SPGEMM_BLOCK_DENSE;
  if (ranked <= kBlockLdsBytes) return BPPSA_SPGEMM_BLOCK_STAGED;
  return BPPSA_SPGEMM_BLOCK_GLOBAL;
}

// Waves of a workgroup of the BLOCK kinds.  The accumulators' LDS says how many workgroups a compute unit
// holds: eight of four waves up to 20 KB, then four of eight, then two or one of sixteen, as long as a wave's
// share of a row of B stays worth a piece.  Rows of 640 entries and more take sixteen waves in any case: four
// would walk them in three and more rounds.  4096 rows of 100 entries by 2048 rows, us with 4 / 8 / 16 waves:
//   columns of B   96 a row          160               320               512               800
//    4096          113 / 155 / 259   117 / 159 / 263   167 / 161 / 269   235 / 231 / 272   397 / 424 / 328
//    8192          184 / 173 / 276   205 / 189 / 288   284 / 207 / 306   331 / 283 / 316   458 / 481 / 376
//   16384          223 / 231 / 362   390 / 348 / 441   686 / 457 / 412   788 / 546 / 438   942 / 656 / 500
int bppsa_spgemm_ways(int kind, int c_max_row, const bppsa_csr& B) {
  const size_t lds = kind == BPPSA_SPGEMM_BLOCK_DENSE    ? dense_lds_bytes(B.cols)
                     : kind == BPPSA_SPGEMM_BLOCK_STAGED ? ranked_lds_bytes(c_max_row, B.cols)
                                                         : kBlockLdsBytes;
  const int64_t mean = B.rows > 0 ? B.nnz / B.rows : 0;
  if (mean >= 640 || (mean >= 200 && lds > 40 * 1024)) return 16;
  return mean >= 96 && lds > 20 * 1024 ? 8 : 4;
}

template <int MODE, int WAYS>
static bppsa_status launch_block(size_t lds, const bppsa_csr& A, const bppsa_csr& B, const int32_t* b_split,
                                 const uint16_t* b_cols16,
                                 const int32_t* c_indptr, const int32_t* c_indices, float* c_data,
                                 hipStream_t stream) {
  const bool narrow = MODE == 0 && b_cols16;
  const auto kernel = narrow                        ? spgemm_numeric_block_kernel<MODE, MODE == 0 ? kCols16 : kCols32, WAYS>
                      : B.nnz >= (int64_t)1 << 30 ? spgemm_numeric_block_kernel<MODE, kCols64, WAYS>
                                                    : spgemm_numeric_block_kernel<MODE, kCols32, WAYS>;
  const void* cols = narrow ? static_cast<const void*>(b_cols16) : B.indices;
  if (lds > 48 * 1024)
    BPPSA_HIP_TRY(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)kBlockLdsBytes));
  kernel<<<block_grid(A.rows), 64 * WAYS, lds, stream>>>(A.rows, B.cols, A.indptr, A.indices, A.data, B.indptr,
                                                         cols, B.data, b_split, c_indptr, c_indices, c_data);
  return BPPSA_OK;
}

bppsa_status bppsa_launch_spgemm_numeric(int kind, int ways, const bppsa_csr& A, const bppsa_csr& B,
                                         const int32_t* b_split, const uint16_t* b_cols16, const int32_t* c_indptr,
                                         const int32_t* c_indices, float* c_data, int c_max_row, hipStream_t stream) {
  if (A.rows < 1) return BPPSA_OK;
#define BPPSA_NUMERIC_ARGS A.indptr, A.indices, A.data, B.indptr, B.indices, B.data
#define BPPSA_BLOCK_WAYS(MODE, WAYS, LDS) launch_block<MODE, WAYS>(LDS, A, B, b_split, b_cols16, c_indptr, c_indices, c_data, stream)
#define BPPSA_BLOCK(MODE, LDS)                                                                                   \
  (ways == 16 ? BPPSA_BLOCK_WAYS(MODE, 16, LDS) : ways == 8 ? BPPSA_BLOCK_WAYS(MODE, 8, LDS) : BPPSA_BLOCK_WAYS(MODE, 4, LDS))
  switch (kind) {
    case BPPSA_SPGEMM_SINGLE:
      spgemm_numeric_single_kernel<<<bppsa_ceil_div(A.rows, 4), 256, 0, stream>>>(A.rows, BPPSA_NUMERIC_ARGS, c_indptr,
                                                                                  c_indices, c_data);
      break;
    case BPPSA_SPGEMM_SCALE_ROWS:
      scale_rows_kernel<<<bppsa_ceil_div(A.rows, 4), 256, 0, stream>>>(A.rows, c_indptr, A.data, B.data, c_data);
      break;
    case BPPSA_SPGEMM_SCALE_COLUMNS:
      if (A.nnz < 1) return BPPSA_OK;
      scale_columns_kernel<<<(int)((A.nnz + 1023) / 1024), 256, 0, stream>>>(A.nnz, A.indices, A.data, B.data, c_data);
      break;
    case BPPSA_SPGEMM_WAVE:
      spgemm_numeric_wave_kernel<<<bppsa_ceil_div(A.rows, 4), 256, 0, stream>>>(A.rows, BPPSA_NUMERIC_ARGS, c_indptr,
                                                                                c_indices, c_data);
      break;
    case BPPSA_SPGEMM_BLOCK_DENSE:
      if (!b_split) return BPPSA_EINVAL;
      if (dense_lds_bytes(B.cols) > kBlockLdsBytes) return BPPSA_EINVAL;
      BPPSA_TRY(BPPSA_BLOCK(0, dense_lds_bytes((B.cols + 63) & ~63)));
      break;
    case BPPSA_SPGEMM_BLOCK_STAGED:
      if (!b_split) return BPPSA_EINVAL;
      if (ranked_lds_bytes(c_max_row, B.cols) > kBlockLdsBytes) return BPPSA_EINVAL;
      BPPSA_TRY(BPPSA_BLOCK(1, ranked_lds_bytes(c_max_row, B.cols)));
      break;
    case BPPSA_SPGEMM_BLOCK_GLOBAL:
      if (!b_split) return BPPSA_EINVAL;
      BPPSA_TRY(BPPSA_BLOCK(2, 0));
      break;
    default:
      return BPPSA_EINVAL;
  }
#undef BPPSA_BLOCK
#undef BPPSA_BLOCK_WAYS
#undef BPPSA_NUMERIC_ARGS
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}

extern "C" bppsa_status bppsa_spmv(const bppsa_csr* A, const float* x, float* y, void* stream) {
  if (!A || !x || !y || !A->indptr || (A->nnz > 0 && (!A->indices || !A->data))) return BPPSA_EINVAL;
  if (A->rows < 1 || A->cols < 1 || A->nnz < 0) return BPPSA_EINVAL;
  if (A->nnz >= INT32_MAX) return BPPSA_EOVERFLOW;
  return bppsa_launch_spmv(*A, x, y, (hipStream_t)stream);
}
