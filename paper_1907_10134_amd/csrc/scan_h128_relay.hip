// The seed-side stretch of an H = 128 chain, walked by several compute units a sample.
//
// A step of the walk is 0.25 us of arithmetic, but one compute unit draws 55 to 65 GB/s from memory, a tile in 1.0 us
// (1.17 beside the matrix-core kernel), however many requests it has outstanding; and on Jacobians that are generated it
// has three times the arithmetic (0.70 us).  So the units of a sample take blocks of kBlock steps in turn: a unit gets the
// tiles of its next block into registers while the others walk theirs, and when the vector entering that block arrives it
// goes through the block with nothing else to do (requests spread over the steps would hold a wave at every one of them
// until earlier tiles have come).  The vector is handed on in 64-bit pieces of (value, tag), stored and polled with agent
// scope, so that value and arrival are one access; 0.9 us from unit to unit.  us a step, T = 1025, B = 16, stored, by
// units a sample: 1 1.0, 2 0.70, 3 0.48, 4 0.40, 5 0.43 (then the hand-over is what is left); beside the totals 0.45, as
// on generated Jacobians.  gru_step, T = 4096, B = 16: the scan 2.00 -> 1.35 ms stored, 1.61 -> 1.35 generated.
//
// No unit depends on another one being resident: a unit that waits for longer than `patience` goes on alone from the last
// vector it had, block after block to the end.  All units compute a block with the same instructions, so what two of
// them write is the same to the bit.  (Two and three scans on streams of their own share the device at 1.1 to 3.9 times
// the speed of one unit a sample.  Blocks claimed by running units in place of fixed turns, so that nobody waits for one
// without a place: the claim takes longer than a block and costs 0.08 us a step, T = 300, B = 8 130 -> 160 us, and beside
// large matrix products or copies, where a scan waits for whole free units, nothing is gained.)
#include "barriers.h"
#include "scan_h128_common.h"

namespace {

typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int kRelayThreads = 1024;
constexpr int kRelayPieces = HH / 4 / kRelayThreads;   // 4
constexpr int kBlock = BPPSA_H128_RELAY_BLOCK;         // even: a block's last vector lies where its first one did
constexpr int kStreaming = 2;                          // the nt bit of a buffer request
static_assert(kBlock % 2 == 0, "the vector of a whole block returns to buffer 0");

template <bool GEN>
__global__ void __launch_bounds__(kRelayThreads)
relay_h128_kernel(int B, int workers, int lo, int hi, const float* __restrict__ Jt, const float* __restrict__ seed,
                  float* __restrict__ G, float* __restrict__ g0, float* __restrict__ v_out,
                  unsigned long long* __restrict__ mail, unsigned base, long long patience,
                  const float* __restrict__ coef, const float* __restrict__ wT) {
  __shared__ __attribute__((aligned(16))) float vs[2][H];
  __shared__ float kept[H];                        // the vector entering block `have`
  __shared__ int seen[2];
  // (workgroups are dealt to the dies in turn, so this leaves every die as many free units, which the totals beside the
  // chain need; all units of a sample on one die: the same time a step)
  const int turn = blockIdx.x / B, b = blockIdx.x % B;
  const int tid = threadIdx.x;
  const int c = tid & 15, r = tid >> 4;            // columns 4c.., 64 + 4c.. of rows r and r + 64
  const int n = hi - lo + 1, blocks = (n + kBlock - 1) / kBlock;
  const bool upper = (c & 8) != 0;                 // the half of a row group that ends up with row r + 64
  const int row = r + (upper ? 64 : 0);
  const bool writer = (c & 7) == 0;
  const bool storer = __builtin_amdgcn_readfirstlane(tid) < H;      // the first two waves
  unsigned long long* box = mail + (size_t)b * H;

  v4f pre[kBlock][kRelayPieces];
  const int at_row = 4 * (H * r + 4 * c);
  const uint64_t stride = (uint64_t)B * HH * 4;
  // The tiles of block j formed in place of being fetched: Jt = W_hr^T diag(a) + W_hn^T diag(c) + W_hz^T diag(e) + diag(z),
  // the coefficients of the block staged in LDS, a piece of the weights (from the cache) for all its tiles.  The diagonal,
  // far larger than the rest, is left to the step: rounded into the tile it would cost half of the accuracy.
  __shared__ __attribute__((aligned(16))) float cfs[GEN ? kBlock : 1][4 * H];
  auto generate = [&](int j) __attribute__((always_inline)) {
    if (tid < kBlock * H) {
      const int k = tid >> 7;                      // one wave, one step
      const size_t at = (size_t)max(hi - j * kBlock - k, lo) * B + b;
      reinterpret_cast<v4f*>(&cfs[k][0])[tid & 127] = reinterpret_cast<const v4f*>(coef + at * 4 * H)[tid & 127];
    }
    lds_barrier();
    // Two columns at a time (pieces of four would not fit the registers beside the tiles), the weights anew for every block
    // (the offset is opaque, or they would be kept in registers that are not there); the tiles are opaque too, or their
    // products would wait for the steps that use them.
    int none = 0;
    asm volatile("" : "+s"(none));
    const float* w = wT + none;
#pragma unroll
    for (int p = 0; p < kRelayPieces; ++p) {       // columns 64 half + 4 c + u and the next, of both rows
      const int half = p >> 1, u = 2 * (p & 1), col = 64 * half + 4 * c + u;
      v2f wr[2], wn[2], wz[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float* at = w + H * (r + 64 * i) + col;
        wr[i] = *reinterpret_cast<const v2f*>(at);
        wn[i] = *reinterpret_cast<const v2f*>(at + HH);
        wz[i] = *reinterpret_cast<const v2f*>(at + 2 * HH);
      }
#pragma unroll
      for (int k = 0; k < kBlock; ++k) {
        const float* f = &cfs[k][col];
        const v2f a = *reinterpret_cast<const v2f*>(f), n = *reinterpret_cast<const v2f*>(f + H),
                  e = *reinterpret_cast<const v2f*>(f + 2 * H);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            float o = wr[i][d] * a[d];
            o += wn[i][d] * n[d];
            o += wz[i][d] * e[d];
            asm volatile("" : "+v"(o));
            pre[k][2 * i + half][u + d] = o;
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto request = [&](int j) __attribute__((always_inline)) {                      // the tiles of block j; below lo: tile lo, which nobody uses
    if (GEN) return generate(j);
    const uint64_t top = (uint64_t)(Jt + ((size_t)max(hi - j * kBlock, lo) * B + b) * HH);
    uint64_t next = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(top >> 32)) << 32 |
                    (uint32_t)__builtin_amdgcn_readfirstlane((int)top);
    int left = n - 1 - j * kBlock;                 // tiles below `next`
#pragma unroll
    for (int k = 0; k < kBlock; ++k) {
      const auto tile = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float*>(next), 0, HH * 4, 0x00020000);
#pragma unroll
      for (int q = 0; q < kRelayPieces; ++q)       // row r + 64 (q / 2), columns 64 (q % 2) + 4 c ..
        pre[k][q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                        tile, at_row, 4 * (64 * H * (q >> 1) + 64 * (q & 1)), kStreaming));
      next -= left > 0 ? stride : 0;
      --left;
    }
  };

  int j = turn, ahead = workers, have = 0;
  if (tid < H) {
    const float first = seed[(size_t)b * H + tid];
    vs[0][tid] = kept[tid] = first;
    if (turn == 0) G[((size_t)hi * B + b) * H + tid] = first;          // to its own row
  }
  if (j >= blocks) return;
  request(j);
  __syncthreads();
  for (;;) {
    bool walk = true;
    if (have < j) {
      // the two waves hold a vector when all 64 pieces of each carry one and the same tag, of block j or a later one
      if (storer) {
        const long long since = wall_clock64();
        bool whole;
        uint32_t block;
        unsigned long long piece;
        do {
          piece = __hip_atomic_load(box + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const uint32_t tag = (uint32_t)(piece >> 32);
          block = (uint32_t)__builtin_amdgcn_readfirstlane((int)tag) - base;     // stale tags: below base, or of another launch
          whole = __builtin_amdgcn_ballot_w64(tag - base == block) == ~0ull && block >= (uint32_t)j && block <= (uint32_t)blocks;
        } while (!whole && wall_clock64() - since < patience);
        vs[0][tid] = __uint_as_float((uint32_t)piece);
        if ((tid & 63) == 0) seen[tid >> 6] = whole ? (int)block : -1;
      }
      lds_barrier();
      const int first = seen[0], second = seen[1];
      if (first < 0 || first != second) {          // go on alone
        lds_barrier();
        if (tid < H) vs[0][tid] = kept[tid];
        j = have;
        ahead = 1;
        walk = false;
      } else if (first > j) {                      // somebody else went on alone and has passed block j
        have = first;
        if (tid < H) kept[tid] = vs[0][tid];
        j += (have - j + ahead - 1) / ahead * ahead;
        walk = false;
      }
    }
    if (walk) {
      const int n0 = j * kBlock, steps = min(kBlock, n - n0);
      float* out = G + ((size_t)(hi - n0) * B + b) * H;      // the row of the vector a step starts from
      float own = GEN ? vs[0][row] : 0.f;          // the vector's value in this thread's row
#pragma unroll
      for (int k = 0; k < kBlock; ++k) {
        if (k < steps) {                             // uniform
          const v4f x0 = *reinterpret_cast<const v4f*>(&vs[k & 1][4 * c]);
          const v4f x1 = *reinterpret_cast<const v4f*>(&vs[k & 1][64 + 4 * c]);
          const float z = GEN ? cfs[GEN ? k : 0][3 * H + row] : 0.f;
          float part[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {              // row r + 64 i
            const v4f p = pre[k][2 * i], q = pre[k][2 * i + 1];
            float acc0 = p[0] * x0[0], acc1 = q[0] * x1[0];      // (two sums: no less exact than pairs)
#pragma unroll
            for (int u = 1; u < 4; ++u) acc0 += p[u] * x0[u], acc1 += q[u] * x1[u];
            part[i] = acc0 + acc1;
          }
          if (k > 0 && storer) out[tid] = vs[k & 1][tid];
          out -= (size_t)B * H;
          float sum = (upper ? part[1] : part[0]) + dpp_from<kDppMirror>(upper ? part[0] : part[1]);
          sum += dpp_from<kDppXor1>(sum);
          sum += dpp_from<kDppXor2>(sum);
          sum += dpp_from<kDppHalfMirror>(sum);
          if (GEN) own = sum += z * own;
          if (writer) {
            vs[(k & 1) ^ 1][row] = sum;
            if (k == steps - 1)
              __hip_atomic_store(box + row, (unsigned long long)(base + (uint32_t)j + 1) << 32 | __float_as_uint(sum),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          lds_barrier();
        }
      }
      have = j + 1;
      j += ahead;
      if (storer) {
        const int below = hi - n0 - steps;           // the row of the block's last vector
        const float last = vs[steps & 1][tid];
        kept[tid] = last;
        (below >= 0 ? G + ((size_t)below * B + b) * H : g0 + (size_t)b * H)[tid] = last;
        if (v_out && have == blocks) v_out[(size_t)b * H + tid] = last;
      }
    }
    if (j >= blocks) break;
    request(j);                                    // (ahead of the barrier: 10 % of a step)
    __syncthreads();
  }
}

}  // namespace

bppsa_status bppsa_relay_h128(int B, int lo, int hi, const float* Jt, const float* seed, float* G, float* g0, float* v_out,
                              const bppsa_h128_relay& relay, hipStream_t s, const bppsa_gru_tiles* gen) {
  // tags of one launch: 1 + launch * 2^24 and the blocks of the stretch behind it
  if (relay.launch < 0 || relay.launch > 127 || (hi - lo) / kBlock >= (1 << 24) - 2) return BPPSA_EINVAL;
  const unsigned base = 1u + ((unsigned)relay.launch << 24);
  unsigned long long* mail = static_cast<unsigned long long*>(relay.mail);
  if (gen)
    relay_h128_kernel<true><<<relay.workers * B, kRelayThreads, 0, s>>>(B, relay.workers, lo, hi, nullptr, seed, G, g0, v_out,
                                                                        mail, base, relay.patience, gen->coef, gen->wT);
  else
    relay_h128_kernel<false><<<relay.workers * B, kRelayThreads, 0, s>>>(B, relay.workers, lo, hi, Jt, seed, G, g0, v_out,
                                                                         mail, base, relay.patience, nullptr, nullptr);
  BPPSA_CHECK_LAUNCH();
  return BPPSA_OK;
}
