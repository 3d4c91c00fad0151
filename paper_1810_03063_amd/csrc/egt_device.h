// Device helpers of the single-launch passes (smoothed best response, regrets).
#pragma once

#include <hip/hip_runtime.h>

namespace egt {

// Bijection of [0, total): workgroup L (on XCD L % 8) -> position, with each
// XCD's workgroups on consecutive positions.
__device__ inline int xcd_spread(int L, int total) {
  const int q = total / 8, r = total % 8;
  const int x = L % 8, j = L / 8;
  return x * q + min(x, r) + j;
}

constexpr int kFusedPad = 16;  // entries past the end of an LDS array that a run may read

// x + p[0] + p[HB] + ... (cnt > 0 entries, added in order).  The last run reads
// up to three entries past the end; the arrays leave room for that.
template <int HB>
__device__ __forceinline__ double add_run(double x, const double* p, int cnt) {
  for (int c = 0; c < cnt; c += 4, p += 4 * HB) {
    const double v0 = p[0], v1 = p[HB], v2 = p[2 * HB], v3 = p[3 * HB];
    x += v0;
    if (c + 1 < cnt) x += v1;
    if (c + 2 < cnt) x += v2;
    if (c + 3 < cnt) x += v3;
  }
  return x;
}

}  // namespace egt
