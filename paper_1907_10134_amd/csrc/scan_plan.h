// Host-side planning shared by the workspace query and the scan launcher.
#pragma once

#include "bppsa_internal.h"

// Segment length of the H = 128 scan (and of the schedule that sets the least workspace at any other size).
#define BPPSA_H128_SEGMENT 64

// Workspace of the H = 128 scan: per recursion level, the chain of segment
// totals [nseg-1, B, H, H] and their incoming vectors [nseg-1, B, H].  Also the least workspace
// bppsa_scan accepts at any other size.
static inline size_t bppsa_generic_scan_ws(int T, int B, int H, int want_g0) {
  size_t total = 0;
  int t_min = want_g0 ? 0 : 1;
  for (;;) {
    const int n = T - t_min;
    const int S = BPPSA_H128_SEGMENT;
    if (n <= S) break;
    const int T2 = bppsa_ceil_div(n, S) - 1;
    total += bppsa_align_up((size_t)T2 * B * H * H * sizeof(float), 256);
    total += bppsa_align_up((size_t)T2 * B * H * sizeof(float), 256);
    T = T2;
    t_min = 1;
  }
  return total;
}

// H = 128: the slab of segments farthest from the seed may be cut into shorter segments (see
// bppsa_h128_plan); their totals and incoming vectors have room of their own: for 32 of them in the least
// workspace a call accepts, and in the one the query asks for as many as the compute units take at once, where
// that is more.  A segment's product is serial, so a small batch on 32 long segments leaves most of the device
// idle.  Room for 32, and for 256 / B up to 128 (8 MB a sample, 16 MB for any batch), us per scan:
//   generated  T = 1034, B = 1  294, 218;  B = 5  324, 235;  T = 2000, B = 2  520, 265;  T = 4096, B = 1  670, 403
//   stored     T = 700, B = 2   189, 192;  T = 1034, B = 1  314, 194;  T = 2000, B = 2  461, 257
#define BPPSA_H128_FINE_SEGMENTS 32
static inline int bppsa_h128_fine_preferred(int T, int B) {
  const int S = BPPSA_H128_SEGMENT, all = (bppsa_ceil_div(T, S) - 1) * 4;   // S / 4 steps each, below the chain
  int most = 256 / B < 128 ? 256 / B : 128;
  if (most > all) most = all;
  return most > BPPSA_H128_FINE_SEGMENTS ? most : BPPSA_H128_FINE_SEGMENTS;
}
static inline size_t bppsa_h128_fine_ws(int T, int B, int want_g0, int segments) {
  if (T - (want_g0 ? 0 : 1) <= BPPSA_H128_SEGMENT) return 0;
  return bppsa_align_up((size_t)segments * B * 128 * 128 * sizeof(float), 256) +
         bppsa_align_up((size_t)segments * B * 128 * sizeof(float), 256);
}

// ---- single-pass path for H = 20 --------------------------------------------------------
#define BPPSA_H20_SEGMENT 32
#define BPPSA_H20_AGG_STRIDE 416   /* floats: a 20x20 total padded to 13 cache lines */
#define BPPSA_H20_INC_STRIDE 32    /* floats: a 20-vector padded to one cache line */
#define BPPSA_H20_HEADER_BYTES 4096

// Workspace of the single-pass scan: header, one status word and one hop count per (unit,
// sample), one published total and one published inclusive vector per (unit, sample), and the
// transposed weights of the fused form.  Sized for units of one half (the larger case).
static inline size_t bppsa_h20_scan_ws(int T, int B) {
  const size_t nblk = (size_t)bppsa_ceil_div(T, BPPSA_H20_SEGMENT) * B;
  return BPPSA_H20_HEADER_BYTES + 2 * bppsa_align_up(nblk * sizeof(int), 256) +
         nblk * (BPPSA_H20_AGG_STRIDE + BPPSA_H20_INC_STRIDE) * sizeof(float) + 20 * 20 * sizeof(float);
}

// skip_dies (bit mask of compute dies whose workgroups stand aside) and unit_halves (0 = chosen
// from the sizes, 1 or 2 = forced) are 0 except in the diagnostic call.
bppsa_status bppsa_scan_h20(int T, int B, const float* Jt, const float* seed, float* G, float* g0,
                            void* workspace, hipStream_t stream, const float* h = nullptr,
                            const float* w_hh = nullptr, int skip_dies = 0, int unit_halves = 0, bool cleared = false);
// What that call zeroes first, from the start of the workspace, and where the fused form puts W_hh transposed (null:
// nowhere); a caller that has done both passes cleared = true.
void bppsa_scan_h20_clears(int T, int B, bool want_g0, void* workspace, long long* words, float** wt);

// The same scan as one serial chain per sample; `error` (may be null) receives 0.  At least one Jacobian.
bppsa_status bppsa_chain_h20(int T, int B, const float* Jt, const float* seed, float* G, float* g0, int* error,
                             hipStream_t stream, const float* h = nullptr, const float* w_hh = nullptr);
bool bppsa_prefer_chain_h20(int n, int B);

// Either of them, whichever costs less.  bppsa_h20_clears says what a caller that passes cleared = true must have
// done: zeroed `words` words at the start of the workspace and, for the fused form, transposed W_hh into wt unless null.
bppsa_status bppsa_any_scan_h20(int T, int B, const float* Jt, const float* seed, float* G, float* g0, void* workspace,
                                hipStream_t stream, const float* h = nullptr, const float* w_hh = nullptr,
                                bool cleared = false);
void bppsa_h20_clears(int T, int B, bool want_g0, void* workspace, long long* words, float** wt);

bppsa_status bppsa_scan_h20_hops(int T, int B, int want_g0, int unit_halves, const void* workspace,
                                 long long* out, hipStream_t stream);

// GRU transposed Jacobians (H = 128) given by what generates them instead of as tiles: coef
// [T*B][4][H] = the per-step vectors (a, c, e, z) of Appendix E's closed form, wT [3][H][H] =
// W_hr^T, W_hn^T, W_hz^T.  With such a source the top level of the scan reads no Jt.
struct bppsa_gru_tiles {
  const float* coef;
  const float* wT;
};

// ---- schedule of a long H = 128 chain ---------------------------------------------------
// The chain is cut into segments of BPPSA_H128_SEGMENT steps, counted from the far end (the
// last one, nearest the seed, may be shorter).  At this size a step of the matrix-matrix side
// costs 128 times the arithmetic of a matrix-vector step, so the hybrid schedule of Section 5.3
// is taken one step further: the `chain_segments` segments nearest the seed are walked by one
// serial matrix-vector chain per sample, on one to four compute units of its own, while the totals of the
// other segments are formed on the matrix cores in slabs of `slab` segments; behind the chain and
// each slab's totals come the slab's matrix-vector passes.  chain_segments = 0: the two-level
// form without the serial chain (used when the batch alone fills the device); chain_segments =
// all segments: no matrix-matrix product at all.
#define BPPSA_H128_MAX_SLABS 32
// Up to this many compute units take turns on a sample's serial chain, this many steps at a time
// (see relay_h128_kernel).  More units than four give no more: what is left is handing the vector on.
#define BPPSA_H128_WORKERS 4
#define BPPSA_H128_RELAY_BLOCK 6
struct bppsa_h128_plan {
  int chain_segments;
  int slab;
  int slabs;
  int last_steps;       // segment length inside the slab farthest from the seed (S, S/2 or S/4): a
                        // slab that would fill less than half of the device is cut finer, which
                        // shortens its products in proportion
  double model_us;      // the estimate the choice was made on
  int workers;          // compute units a sample that walk the serial chain in turn
};

// What the units of a relay share: one vector a sample in 64-bit pieces (zeroed before the call's first launch), the
// launch's number within the call, and how long (ticks of 10 ns) a unit waits for the one before it until it goes on
// alone.  A hand-over takes 1 us and a turn 10; 200 us pass only if the unit before has found no place on the device.
#define BPPSA_H128_PATIENCE 20000
struct bppsa_h128_relay {
  int workers;
  void* mail;
  int launch;
  long long patience;
};

// Units for the chain over `totals` totals, of which `room` a sample are free: one for every block.
static inline int bppsa_h128_totals_workers(int totals, int room) {
  const int blocks = bppsa_ceil_div(totals, BPPSA_H128_RELAY_BLOCK);
  return blocks < room ? blocks : room < 1 ? 1 : room;
}
static inline double bppsa_h128_totals_us(int totals, int workers) {
  return workers > 1 ? 9.0 + 0.4 * totals : 1.2 * totals;
}

// One slab of the walk below the serial chain, shared by the cost model and the launcher:
// segments [lo, hi] of S steps, totals for [rlo, hi].
struct bppsa_h128_slab {
  int lo, hi, rlo;
};
static inline bppsa_h128_slab bppsa_h128_next_slab(int hi, int slab) {
  int lo = hi - slab + 1;
  if (lo <= 1) lo = 0;                        // segment 0 has no total: it rides with the last slab
  return bppsa_h128_slab{lo, hi, lo < 1 ? 1 : lo};
}

// The schedule of the cost model below, or the one the caller forces (force_chain >= 0; force_slab
// and force_last 0 = not forced).  Times in microseconds, measured on MI355X: a step of the serial
// chain (1024 threads on one to four compute units a sample; bound by what one unit draws from memory, or
// by its vector ALUs when the Jacobians are generated), a step of a segment's running product on
// the matrix cores with the other units full, a step of the chain over a slab's totals, and the
// matrix-vector pass of a slab (HBM-bound on stored Jacobians, ALU-bound on generated ones).
static inline bppsa_h128_plan bppsa_plan_h128(int n, int B, int cus, bool generated, int fine_segments,
                                              int force_chain = -1, int force_slab = 0, int force_last = 0) {
  const int S = BPPSA_H128_SEGMENT;
  const int nseg = bppsa_ceil_div(n, S);
  bppsa_h128_plan best = {0, 0, 0, S, 0.0, 1};
  if (cus < 2 * B || nseg < 2) return best;
  // The search below takes 2 to 190 us (T = 705, B = 2 and T = 30000, B = 16; without its bounds 4 and 1200): a training
  // loop asks for the same sizes every iteration, for a few lengths in turn, or with and without g0, so each host
  // thread remembers its last answers.
  struct Memo {
    int key[8];
    bppsa_h128_plan plan;
  };
  constexpr int kMemos = 16;
  static thread_local Memo memo[kMemos] = {};      // (n is never 0)
  static thread_local unsigned next_memo = 0;
  const int key[8] = {n, B, cus, (int)generated, fine_segments, force_chain, force_slab, force_last};
  for (const Memo& m : memo) {
    bool same = true;
    for (int k = 0; k < 8; ++k) same &= m.key[k] == key[k];
    if (same) return m.plan;
  }
  const double stored_step[BPPSA_H128_WORKERS] = {1.17, 0.72, 0.52, 0.46};
  const double generated_step[BPPSA_H128_WORKERS] = {0.70, 0.70, 0.52, 0.42};
  const int top_steps = n - (nseg - 1) * S;
  double best_us = 1e300;
  const int k_lo = force_chain >= 0 ? (force_chain < 1 ? 1 : force_chain > nseg ? nseg : force_chain) : 1;
  const int k_hi = force_chain >= 0 ? k_lo : nseg;
  for (int workers = 1; workers <= BPPSA_H128_WORKERS && (workers == 1 || cus >= 2 * workers * B); ++workers) {
    // the serial chains keep their units to themselves, and workgroups go to the eight dies in turn, so what
    // counts is the die with the most of them: a workgroup more than it holds is a second round
    const int left_units = cus - 8 * bppsa_ceil_div(workers * B, 8), free_units = left_units > 1 ? left_units : 1;
    // a slab's times: its totals on the matrix cores, the chain over them, its pass, and that pass beside other totals
    struct Slab {
      double reduce_us, chain_us, apply_us, beside_us, after_us;
    };
    auto slab_times = [&](int totals, int segs, int steps, bool farthest) {
      // (the clock falls with the number of units whose matrix cores are busy: 7.2 us with less than half of them)
      const double product_step = generated ? 8.5 : 2 * totals * B > cus ? 8.1 : 7.2;
      Slab t;
      t.reduce_us = totals > 0 ? (generated ? 20.0 : 8.0) + (steps - 1) * product_step * bppsa_ceil_div(totals * B, free_units) : 0.0;
      t.chain_us = bppsa_h128_totals_us(totals, bppsa_h128_totals_workers(totals, farthest ? cus / B : workers));
      // Beside the matrix-core kernel the matrix-vector pass on stored Jacobians gets a
      // fraction of its speed; the pass on generated ones (242 registers) does not fit on a
      // compute unit beside the totals kernel of that form (313) and waits for it.
      const double apply_us = generated ? steps * 1.1 * bppsa_ceil_div(segs * B, cus)
                                        : (double)segs * B * steps * (128.0 * 128.0 * 4.0) / 5.3e6;
      const double alone = 15.0 + 0.8 * steps;                       // a workgroup by itself
      const double beside = generated ? apply_us : apply_us * 2.8;
      t.apply_us = apply_us < alone ? alone : apply_us;
      t.beside_us = beside < alone ? alone : beside;
      // (waiting for the totals and starting the next launches; with 20 for shorter segments, chains of 363 to 636 steps at
      // B = 1 to 24 are cut, at 1.05 to 1.2 times what they take in one)
      t.after_us = steps < S ? 25.0 : 10.0;
      return t;
    };
    for (int K = k_lo; K <= k_hi; ++K) {
      const double chain_us = (generated && workers == 1 ? 0.0 : 9.0) +
                              (double)(top_steps + (K - 1) * S) * (generated ? generated_step : stored_step)[workers - 1];
      // (nothing below is without cost: no plan with this chain or a longer one takes less)
      if (chain_us >= best_us) break;
      const int R = nseg - K;                         // segments R-1 .. 0 lie below the chain
      int slab = 0, full = 0;                         // all slabs but the farthest are full
      Slab each{};
      if (R > 0) {
        slab = force_slab > 0 ? force_slab : free_units / B;
        if (slab < 1) slab = 1;
        if (bppsa_ceil_div(R, slab) > BPPSA_H128_MAX_SLABS) slab = bppsa_ceil_div(R, BPPSA_H128_MAX_SLABS);
        full = R >= 2 ? (R - 2) / slab : 0;           // (bppsa_h128_next_slab: segment 0 rides with the farthest)
        if (full > 0) each = slab_times(slab, slab, S, false);
      }
      for (int last = S; last >= S / 4; last /= 2) {
        if (R > 0 ? (force_last > 0 && last != force_last) : last != S) continue;   // no slab: nothing to cut
        double cur = chain_us;
        if (R > 0) {
          const int top = R - 1 - full * slab, segs = (top + 1) * (S / last);       // the slab farthest from the seed
          if (last < S && segs > fine_segments) continue;
          const Slab far = slab_times(segs - 1, segs, last, true);
          double reduce_all = 0.0, reduce_end = 0.0;      // when the totals of all slabs, and of those so far, are done
          for (int j = 0; j < full; ++j) reduce_all += each.reduce_us;
          reduce_all += far.reduce_us;
          if (reduce_all >= best_us) continue;
          for (int j = 0; j <= full; ++j) {
            const Slab& t = j < full ? each : far;
            reduce_end += t.reduce_us;
            double start = (cur > reduce_end ? cur : reduce_end) + t.chain_us;
            const bool beside = start < reduce_all;
            if (generated && beside) start = reduce_all;
            cur = start + (beside ? t.beside_us : t.apply_us) + t.after_us;
          }
        }
        // Plans that near are not told apart by these figures.  Stored Jacobians: a longer chain for more than 2 % only, as what
        // it draws from memory is taken from the passes beside it.  Generated ones: more units to a chain for more than 1 %
        // only, as four take 0.42 us a step by themselves and 0.45 and more beside the totals (T = 2751, B = 8 721 us with four
        // units, 686 with one; T = 2490, B = 7 697, 679; T = 1034, B = 5 237, 224 with fewer; T = 4096, B = 2 402, 404 with one).
        const bool doubtful = generated ? workers > best.workers : K > best.chain_segments;
        if (cur < best_us * (!doubtful ? 1.0 : generated ? 0.99 : 0.98)) {
          best_us = cur;
          best = {K, slab, R > 0 ? full + 1 : 0, last, cur, workers};
        }
      }
    }
  }
  Memo& m = memo[next_memo++ % kMemos];
  for (int k = 0; k < 8; ++k) m.key[k] = key[k];
  m.plan = best;
  return best;
}

// fine_segments: how many of the last slab's shorter segments the workspace has room for (at least
// BPPSA_H128_FINE_SEGMENTS); plan: null = chosen by bppsa_plan_h128, otherwise the schedule to use
bppsa_status bppsa_scan_h128(int T, int B, const float* Jt, const float* seed, float* G, float* g0, void* workspace,
                             int fine_segments, hipStream_t stream, const bppsa_gru_tiles* gen = nullptr,
                             const bppsa_h128_plan* plan = nullptr, long long patience = BPPSA_H128_PATIENCE);

// ---- every H <= 128 without kernels of its own: cut by a cost model within the workspace given (also
// none), preferred size from the query ----
size_t bppsa_tiles_scan_ws(int T, int B, int H);
bppsa_status bppsa_scan_tiles(int T, int B, int H, const float* Jt, const float* seed, float* G, float* g0,
                              void* workspace, size_t workspace_bytes, hipStream_t s);

// ---- matrix-core kernels for H = 128; stream: Jt is read past the caches (bppsa_stream_h128) ----
bppsa_status bppsa_reduce_h128(int T, int B, int t_min, int S, int seg_begin, int seg_count,
                               const float* Jt, bool stream, float* tot, hipStream_t s, const bppsa_gru_tiles* gen = nullptr);
// The same totals with the tiles generated (gen is not null); called by bppsa_reduce_h128.
bppsa_status bppsa_reduce_h128_gen(int T, int B, int t_min, int S, int seg_begin, int seg_count, float* tot,
                                   hipStream_t s, const bppsa_gru_tiles* gen);
bppsa_status bppsa_apply_h128(int T, int B, int t_min, int S, int seg_begin, int seg_count,
                              const float* Jt, bool stream, const float* vin, int vin_is_seed, float* G, float* g0,
                              float* v_out, hipStream_t s, const bppsa_gru_tiles* gen = nullptr);

// One serial chain per sample over steps hi..lo (seeded by seed [B, H]); g[t] goes to G[t-1] (g0 for
// t = 0, which must not be null if lo = 0), the last vector to v_out [B, H] if not null, and, but for generated Jacobians
// and one unit, the seed to G[hi].
bppsa_status bppsa_chain_h128(int B, int lo, int hi, const float* Jt, const float* seed, float* G, float* g0,
                              float* v_out, hipStream_t s, const bppsa_gru_tiles* gen = nullptr,
                              const bppsa_h128_relay* relay = nullptr);
// The same by several compute units a sample; relay.mail: 8 H bytes a sample.
bppsa_status bppsa_relay_h128(int B, int lo, int hi, const float* Jt, const float* seed, float* G, float* g0, float* v_out,
                              const bppsa_h128_relay& relay, hipStream_t s, const bppsa_gru_tiles* gen = nullptr);

// coef and wT of bppsa_gru_tiles from the hidden states, inputs and weights (gates recomputed).
bppsa_status bppsa_gru_coefs_h128(long long rows, int I, const float* h, const float* x, const float* w_ih,
                                  const float* w_hh, const float* b_ih, const float* b_hh, float* coef,
                                  float* wT, hipStream_t stream);
