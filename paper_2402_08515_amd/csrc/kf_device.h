// Device helpers shared by the time-stepping kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace kf {

inline int ceil_div64(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Consecutive workgroup ids are dealt round-robin to the 8 XCDs; renumber
// them so that each XCD receives one contiguous range of row slices and its
// L2 keeps the neighbouring rows it gathers.
__device__ __forceinline__ int xcd_map(int i, int nblk) {
  const int q = nblk >> 3, r = nblk & 7;
  const int x = i & 7, t = i >> 3;
  return (x < r) ? x * (q + 1) + t : r * (q + 1) + (x - r) * q + t;
}

// B consecutive columns of a block's row, loaded and stored at once
template <typename T, int B>
struct alignas((B * sizeof(T)) >= 16 ? 16 : (B * sizeof(T))) Row {
  T v[B];
};

}  // namespace kf
