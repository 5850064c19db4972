// bppsa_scan and bppsa_gru_scan_fused at H = 128: the host side (kernels in scan_h128.hip).
//
// The time axis is cut into segments of S steps.  This is the hybrid schedule
// the paper itself uses when n is much larger than the number of workers
// (Section 5.3: a truncated up-sweep, a scan of the partial results, then the
// down-sweep; Section 3.6: step complexity n/p + log p):
//   reduce : every interior segment multiplies its S transposed Jacobians into
//            one H x H total (the matrix-matrix side of the up-sweep);
//   top    : the segment that touches the seed only ever needs matrix-vector
//            products (Section 3.1: A may be a vector), so it is applied
//            directly and hands its last vector on as the next level's seed;
//   recurse: the totals form a shorter chain of the same kind - scan it;
//   apply  : every other segment walks its steps with matrix-vector products
//            from its incoming vector (the down-sweep side).
// Any bracketing gives the same gradients up to rounding (Section 3.5).
#include <mutex>

#include "bppsa_internal.h"
#include "scan_plan.h"

namespace {

constexpr int H = 128;

__global__ void copy_rows_kernel(long long n, const float* __restrict__ src, float* __restrict__ dst) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}
// the same, and the mail of the relays (a 64-bit piece to every value of a vector) is zeroed
__global__ void copy_rows_clear_kernel(long long n, const float* __restrict__ src, float* __restrict__ dst,
                                       unsigned long long* __restrict__ mail) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (src != dst) dst[i] = src[i];
  mail[i] = 0;
}

// A second stream and the events that order it against the caller's stream; one set per
// device, created on first use and kept until the process ends.  `lock` is held while a call
// enqueues work that uses them, so that the records and waits of two host threads do not
// interleave.
constexpr int kMaxSlabs = BPPSA_H128_MAX_SLABS;
struct SideStream {
  hipStream_t stream;
  hipEvent_t fork, join, slab[kMaxSlabs];
  std::mutex lock;
};
SideStream* side_stream() {
  constexpr int kMaxDevices = 64;
  static SideStream table[kMaxDevices];
  static bool made[kMaxDevices];
  static std::mutex table_lock;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> hold(table_lock);
  if (!made[dev]) {
    SideStream& st = table[dev];
    if (hipStreamCreateWithFlags(&st.stream, hipStreamNonBlocking) != hipSuccess) return nullptr;
    if (hipEventCreateWithFlags(&st.fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&st.join, hipEventDisableTiming) != hipSuccess)
      return nullptr;
    for (int i = 0; i < kMaxSlabs; ++i)
      if (hipEventCreateWithFlags(&st.slab[i], hipEventDisableTiming) != hipSuccess) return nullptr;
    made[dev] = true;
  }
  return &table[dev];
}

// H = 128, long chains: the schedule of bppsa_h128_plan.  The caller's stream walks the serial chain of
// the segments nearest the seed (up to four 1024-thread workgroups per sample, which have their compute units
// to themselves) while a second stream forms the totals of the segments below it on the matrix
// cores, slab by slab, nearest the seed first, a slab filling the other units once.  Behind the
// chain and behind each slab's totals the caller's stream runs the chain over the slab's totals,
// entered by the vector handed on from above, and then the slab's own matrix-vector pass (bound
// by HBM, or by the vector ALUs on generated Jacobians), which shares the units with the totals
// of the next slab: 242 + 148 registers per lane, 135 KB + 1 KB of LDS.
// (The chain is the one that does not wait for an event: totals of more than one round, started first, would hold all
// units until their first round is over.  T = 1034, B = 16, generated: 523 -> 389 us.)
bppsa_status scan_h128_pipelined(int T, int B, int t_min, int S, int nseg, const float* Jt, const float* seed,
                                 float* G, float* g0, float* tot, float* vin, float* fine_tot, float* fine_vin,
                                 hipStream_t s, SideStream* side, const bppsa_h128_plan& plan, int fine_segments,
                                 const bppsa_gru_tiles* gen, bppsa_h128_relay relay) {
  const size_t row = (size_t)B * H;
  const int R = nseg - plan.chain_segments;       // segments R-1 .. 0 lie below the serial chain
  std::lock_guard<std::mutex> hold(side->lock);
  hipStream_t s2 = side->stream;
  BPPSA_HIP_TRY(hipEventRecord(side->fork, s));
  BPPSA_HIP_TRY(hipStreamWaitEvent(s2, side->fork, 0));
  // From here on the second stream carries work of this call, so every way out - an error
  // included - goes through the join below: the caller's stream waits for whatever was enqueued
  // on the second stream (and a capturing stream gets its fork joined) before the status returns.
  bppsa_status st = [&]() -> bppsa_status {
    // the serial chain; its last vector enters segment R-1
    relay.workers = plan.workers;
    bppsa_status e = bppsa_chain_h128(B, t_min + R * S, T - 1, Jt, seed, G, g0, vin + (size_t)(R - 1) * row, s, gen, &relay);
    if (e != BPPSA_OK) return e;
    int j = 0;
    for (int hi = R - 1; hi >= 0; ++j) {
      if (j >= kMaxSlabs) return BPPSA_EINVAL;
      const bppsa_h128_slab sl = bppsa_h128_next_slab(hi, plan.slab);
      // this slab's own view of its stretch of the chain: segments [lo, top] of `steps` steps counted
      // from t_min, totals and incoming vectors in `stot` and `svin` (indexed by segment), the
      // vector entering segment `top` in vin[sl.hi]
      int steps = S, lo = sl.lo, rlo = sl.rlo, top = sl.hi;
      float *stot = tot, *svin = vin;
      if (sl.lo == 0 && plan.last_steps < S) {
        // the slab farthest from the seed, cut into shorter segments with room of their own
        const int f = S / plan.last_steps;
        steps = plan.last_steps;
        top = (sl.hi + 1) * f - 1;
        rlo = 1;
        stot = fine_tot;
        svin = fine_vin;
        if (top + 1 > fine_segments) return BPPSA_EINVAL;
      }
      const bool stream = bppsa_stream_h128((int64_t)(top - lo + 1) * steps, B, true);
      if (top >= rlo) {
        e = bppsa_reduce_h128(t_min + (top + 1) * steps, B, t_min, steps, rlo, top - rlo + 1, Jt, stream, stot, s2, gen);
        if (e != BPPSA_OK) return e;
      }
      BPPSA_HIP_TRY(hipEventRecord(side->slab[j], s2));
      BPPSA_HIP_TRY(hipStreamWaitEvent(s, side->slab[j], 0));
      if (top >= rlo) {
        // svin[seg-1] = stot[seg] svin[seg] for seg = top .. rlo: the totals as a chain of
        // top-rlo+1 steps, entered by svin[top]; also gives the next slab its entering vector
        // (on the compute units the serial chain has left: beside the matrix-core kernel a
        // 256-thread workgroup would take 6 to 10 us per step)
        // (the slab farthest from the seed has no totals beside it, and the whole device for its chain)
        ++relay.launch;
        relay.workers = bppsa_h128_totals_workers(top - rlo + 1, sl.lo == 0 ? bppsa_compute_units() / B : plan.workers);
        // It writes the vector it starts from to svin[top], where the pass looks for it (a copy in front cost 5 us and a launch).
        e = bppsa_chain_h128(B, rlo, top, stot, vin + (size_t)sl.hi * row, svin, nullptr, nullptr, s, nullptr, &relay);
        if (e != BPPSA_OK) return e;
      }
      e = bppsa_apply_h128(svin == vin ? T : t_min + (top + 1) * steps, B, t_min, steps, lo, top - lo + 1, Jt, stream, svin, 0, G, g0,
                           nullptr, s, gen);
      if (e != BPPSA_OK) return e;
      hi = sl.lo - 1;
    }
    return BPPSA_OK;
  }();
  const bool joined = hipEventRecord(side->join, s2) == hipSuccess &&
                      hipStreamWaitEvent(s, side->join, 0) == hipSuccess;
  if (st != BPPSA_OK) return st;
  return joined ? BPPSA_OK : BPPSA_EHIP;
}

// One level of the recursion; `ws` is the unused tail of the workspace.
bppsa_status scan_level(int T, int B, const float* Jt, const float* seed,
                        float* G, float* g0, char* ws, int fine_segments, hipStream_t s,
                        const bppsa_gru_tiles* gen = nullptr,
                        const bppsa_h128_plan* forced = nullptr, long long patience = BPPSA_H128_PATIENCE) {
  const size_t row = (size_t)B * H;
  const int t_min = g0 ? 0 : 1;
  const int n = T - t_min;
  const int S = BPPSA_H128_SEGMENT;
  bppsa_h128_plan plan = {0, 0, 0, S, 0.0, 1};
  if (n > S) plan = forced ? *forced : bppsa_plan_h128(n, B, bppsa_compute_units(), gen != nullptr, fine_segments);
  const int copy_blocks = (int)(((long long)row + 255) / 256);
  float* const last = G + (size_t)(T - 1) * row;
  if (plan.chain_segments >= 1) {
    // the mail of the relays lies where segment 0's total would: no form of the scan makes that one
    copy_rows_clear_kernel<<<copy_blocks, 256, 0, s>>>((long long)row, seed, last, reinterpret_cast<unsigned long long*>(ws));
    BPPSA_CHECK_LAUNCH();
  } else if (seed != last) {
    copy_rows_kernel<<<copy_blocks, 256, 0, s>>>((long long)row, seed, last);
    BPPSA_CHECK_LAUNCH();
  }
  if (n <= 0) return BPPSA_OK;
  const bool stream = bppsa_stream_h128(n, B, n > S);
  if (n <= S) return bppsa_apply_h128(T, B, t_min, n, 0, 1, Jt, stream, seed, 1, G, g0, nullptr, s, gen);

  const int nseg = bppsa_ceil_div(n, S);
  const int T2 = nseg - 1;                               // length of the chain of totals
  float* tot = reinterpret_cast<float*>(ws);
  ws += bppsa_align_up((size_t)T2 * row * H * sizeof(float), 256);
  float* vin = reinterpret_cast<float*>(ws);
  ws += bppsa_align_up((size_t)T2 * row * sizeof(float), 256);

  bppsa_status st;
  const bppsa_h128_relay relay = {plan.workers, tot, 0, patience};
  if (plan.chain_segments >= nseg) return bppsa_chain_h128(B, t_min, T - 1, Jt, seed, G, g0, nullptr, s, gen, &relay);
  if (plan.chain_segments >= 1) {
    SideStream* side = side_stream();
    if (side) {
      float* fine_tot = reinterpret_cast<float*>(ws);
      float* fine_vin = reinterpret_cast<float*>(
          ws + bppsa_align_up((size_t)fine_segments * row * H * sizeof(float), 256));
      return scan_h128_pipelined(T, B, t_min, S, nseg, Jt, seed, G, g0, tot, vin, fine_tot, fine_vin, s, side, plan,
                                 fine_segments, gen, relay);
    }
  }
  // interior segments 1..nseg-2: matrix-matrix totals (segment 0's total reaches no output)
  st = bppsa_reduce_h128(T, B, t_min, S, 1, nseg - 2, Jt, stream, tot, s, gen);
  if (st != BPPSA_OK) return st;
  // seed-side segment: matrix-vector only; its last vector seeds the chain of totals
  st = bppsa_apply_h128(T, B, t_min, S, nseg - 1, 1, Jt, stream, seed, 1, G, g0, vin + (size_t)(T2 - 1) * row, s, gen);
  if (st != BPPSA_OK) return st;
  // incoming vectors of segments 0..nseg-2 = scan over the totals
  st = scan_level(T2, B, tot, vin + (size_t)(T2 - 1) * row, vin, nullptr, ws, fine_segments, s);
  if (st != BPPSA_OK) return st;
  return bppsa_apply_h128(T, B, t_min, S, 0, nseg - 1, Jt, stream, vin, 0, G, g0, nullptr, s, gen);
}

}  // namespace

bppsa_status bppsa_scan_h128(int T, int B, const float* Jt, const float* seed, float* G, float* g0, void* workspace,
                             int fine_segments, hipStream_t stream, const bppsa_gru_tiles* gen,
                             const bppsa_h128_plan* plan, long long patience) {
  return scan_level(T, B, Jt, seed, G, g0, static_cast<char*>(workspace), fine_segments, stream, gen, plan, patience);
}
