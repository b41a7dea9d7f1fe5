// Device-side pieces of the dispatch shared by the kernels that place (token, rank) pairs.
#pragma once

#include "internal.h"

namespace mm {
namespace {

__device__ __forceinline__ unsigned long long lanemask_lt(int lane) {
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// expert of rank j of token t, at idx[at]; -1 if that is no pair
__device__ __forceinline__ int pair_expert(const int32_t* __restrict__ idx, const int32_t* __restrict__ k_t,
                                           int j_lo, int t, int j, size_t at, int E, int K) {
  int kt = k_t[t];
  kt = kt < 0 ? 0 : (kt > K ? K : kt);
  const int e = idx[at];
  return j >= j_lo && j < kt && (unsigned)e < (unsigned)E ? e : -1;
}

}  // namespace
}  // namespace mm
