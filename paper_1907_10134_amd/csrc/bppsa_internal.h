// Internal helpers shared by the HIP translation units of libbppsa (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "bppsa.h"

#define BPPSA_WAVE 64

// Returns BPPSA_EHIP from the enclosing function if the last launch failed.
#define BPPSA_CHECK_LAUNCH()                                  \
  do {                                                        \
    if (hipGetLastError() != hipSuccess) return BPPSA_EHIP;   \
  } while (0)

#define BPPSA_TRY(expr)                                       \
  do {                                                        \
    const bppsa_status st__ = (expr);                         \
    if (st__ != BPPSA_OK) return st__;                        \
  } while (0)

#define BPPSA_HIP_TRY(expr)                                   \
  do {                                                        \
    if ((expr) != hipSuccess) return BPPSA_EHIP;              \
  } while (0)

static inline size_t bppsa_align_up(size_t n, size_t a) { return (n + a - 1) / a * a; }

static inline int bppsa_ceil_div(int a, int b) { return a / b + (a % b > 0); }

// A product of sizes that must fit a signed 64-bit element count and whose
// per-array element count must stay below 2^40 (far above 288 GB of fp32).
static inline bool bppsa_mul_overflows(int64_t a, int64_t b, int64_t c, int64_t d) {
  const int64_t lim = (int64_t)1 << 40;
  if (a <= 0 || b <= 0 || c <= 0 || d <= 0) return true;
  if (a > lim / b) return true;
  int64_t ab = a * b;
  if (ab > lim / c) return true;
  int64_t abc = ab * c;
  if (abc > lim / d) return true;
  return false;
}

// Stored Jacobians that the caches do not hold from one call to the next are written and read with streaming accesses
// (plain loads leave the caches full of lines that the next writer has to displace: the builder's 768 MB at T = 30000,
// B = 16, H = 20 take 204 us behind a scan with plain loads, 129 behind one with streaming loads; at 77 MB, where the
// builder's lines are still there, streaming loads cost 2 us of 62).  For the builders, and the readers of H = 20.
__host__ __device__ static inline bool bppsa_stream_jacobians(int64_t T, int64_t B, int64_t H) {
  return T * B * H * H * (int64_t)sizeof(float) > (int64_t)128 << 20;
}
// The same for totals and passes of H = 128, whose builder writes with ordinary stores at every size.  us with ordinary and
// with streaming loads, of the scan and of builder and scan.  One matrix-vector pass over `steps` steps is read again in
// the next call: past the caches where it is more than they hold (256 MB and eight times 4):
//   T = 20, B = 3 20, 27 and 45, 44;  T = 65, B = 3 63, 86 and 92, 89;  T = 65, B = 16 66, 95 and 97, 104;
//   T = 20, B = 127 (159 MB) 26, 37 and 76, 74;  T = 60, B = 64 (240 MB) 63, 99 and 121, 123;
//   T = 60, B = 150 (562 MB) 123, 113 and 268, 249
// A slab is read twice, for the totals and for its pass, beside a chain that reads too:
//   T = 500, B = 5 (120 MB) 177, 189 and 221, 235;  T = 1034, B = 5 (240 MB) 216, 222 and 313, 286;
//   T = 1034, B = 8 (256 MB) 319, 331 and 436, 439;  T = 2000, B = 5 (480 MB) 385, 372 and 514, 494
static inline bool bppsa_stream_h128(int64_t steps, int64_t B, bool slab) {
  return steps * B * 128 * 128 * (int64_t)sizeof(float) > (int64_t)(slab ? 224 : 288) << 20;
}

// Compute units of the current device (256 on an MI355X); queried from the runtime on every
// call, so nothing is remembered across devices.  Falls back to 256 if the query fails.
static inline int bppsa_compute_units() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  return cus;
}
