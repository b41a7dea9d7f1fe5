// Device-side pieces of the dispatch shared by the kernels that place (token, rank) pairs.
#pragma once

#include "internal.h"

namespace mm {
namespace {

__device__ __forceinline__ unsigned long long lanemask_lt(int lane) {
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Inclusive sum over the lanes of a wave, without LDS: within the rows of 16, then lane 15 of a row into the next one and lane 31 into
// the upper half.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);     // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);     // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);     // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);     // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // row_bcast:31 into rows 2, 3
  return v;
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
