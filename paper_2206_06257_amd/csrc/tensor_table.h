// Walking the tensor table on the device: shared by the quantizer, the aggregation and the optimizer kernels.
#pragma once
#include "common.h"

namespace dat {

// Largest t with off[t] <= i (off[0] = 0, off[T] = d > i); empty tensors are skipped.
__device__ __forceinline__ int find_tensor(const int64_t* off, int T, int64_t i) {
  int lo = 0, hi = T;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// The offset table in LDS (T <= kTabMax): the binary search and every tensor boundary a thread crosses then
// cost LDS reads instead of dependent global loads.  Returns the table to use (generic pointer).
constexpr int kTabMax = 1024;
__device__ __forceinline__ const int64_t* stage_offsets(const int64_t* __restrict__ off, int T, int64_t* s_off) {
  if (T > kTabMax) return off;
  for (int i = threadIdx.x; i <= T; i += blockDim.x) s_off[i] = off[i];
  __syncthreads();
  return s_off;
}

}  // namespace dat
