// Launch places of work units that are dealt to the XCDs in order. No HIP, so
// that it can be checked on the host.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define SELL_HOST_DEVICE __host__ __device__
#else
#define SELL_HOST_DEVICE
#endif

namespace sell {

// Place of the k-th of n units, W to a workgroup, where workgroup b runs on XCD
// b mod X: eighth q (X = 8) of the units goes to workgroups q, q + X, q + 2X, ..., in
// whole workgroups; the last n mod (W * X) units follow.
SELL_HOST_DEVICE inline int64_t xcd_place(int64_t k, int64_t n, int W, int X) {
  const int64_t per = n / ((int64_t)W * X) * W;  // units of an XCD
  if (k >= per * X) return k;
  const int64_t q = k / per, t = k - q * per;
  return (t / W * X + q) * W + t % W;
}

}  // namespace sell
