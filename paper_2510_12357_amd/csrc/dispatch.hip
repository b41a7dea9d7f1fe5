// Token-to-expert dispatch with a variable expert count per token (k_t = k_big for important
// tokens, k_little otherwise; Sec. III-A).  The execution stage (Sec. II-A) wants the
// (token, rank) pairs grouped per expert; the order is fixed to (expert asc, token asc), i.e. a
// stable counting sort of the pair list by expert id.
//
// The order is produced without order-dependent operations: every pair sets its token's bit in its
// expert's token mask in LDS (atomic OR, which does not depend on the order), and a pair's position is its
// expert's offset plus the number of bits below its token's, so the result is unique and reproducible,
// and all pairs are placed at once (the masks took the place of a loop over the experts that scanned
// the tokens for each: 200 tokens 12.4 -> 4.8 us, 64 tokens 5.5 -> 4.6; the scatter kernel at 2048 tokens, 8 of 64
// experts, 11.3 -> 7.2).  The experts of one token must be distinct,
// as the selection stage produces them.  Two shapes:
//   * T <= kSmallDispatchT: one workgroup, one launch.
//   * larger T: one workgroup per chunk of 128 tokens; a count kernel, then a scatter kernel
//     that rebuilds the prefixes of the counts itself.  In a step of one call the selection kernel may have counted
//     already, per 16 tokens, and the count kernel is not launched (selection_counts has the rule).
#include "internal.h"
#include "dispatch_device.h"

namespace mm {
namespace {

constexpr int kSmallThreads = 1024;
constexpr int kBigThreads = 256;

__global__ __launch_bounds__(kSmallThreads) void dispatch_small_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ k_t, int j_lo, int T, int E, int K,
    int32_t* __restrict__ offsets, int32_t* __restrict__ sorted_token,
    int32_t* __restrict__ sorted_rank, int32_t* __restrict__ inv_pos) {
  constexpr int kWords = kSmallDispatchT / 64, kPerThread = kSmallDispatchT * MOE_MAX_TOPK / kSmallThreads;
  __shared__ unsigned long long s_mask[MOE_MAX_EXPERTS][kWords];
  __shared__ int s_off[MOE_MAX_EXPERTS + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = T * K;
  int pe[kPerThread];                                  // this thread's pairs tid, tid + kSmallThreads, ..
#pragma unroll
  for (int c = 0; c < kPerThread; ++c) {
    const int i = tid + c * kSmallThreads, t = i / K;
    pe[c] = i < n ? pair_expert(idx, k_t, j_lo, t, i - t * K, i, E, K) : -1;
  }
  for (int i = tid; i < E * kWords; i += kSmallThreads) (&s_mask[0][0])[i] = 0;
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kPerThread; ++c) {
    const int t = (tid + c * kSmallThreads) / K;
    if (pe[c] >= 0) atomicOr(&s_mask[pe[c]][t >> 6], 1ull << (t & 63));
  }
  __syncthreads();
  if (wave == 0) {                                     // exclusive prefix over <= 256 experts
    constexpr int C = MOE_MAX_EXPERTS / 64;
    int loc[C], sum = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int e = lane * C + c;
      loc[c] = 0;
      if (e < E)
#pragma unroll
        for (int w = 0; w < kWords; ++w) loc[c] += __popcll(s_mask[e][w]);
      sum += loc[c];
    }
    const int incl = wave_scan(sum);
    int run = incl - sum;
#pragma unroll
    for (int c = 0; c < C; ++c) { const int e = lane * C + c; if (e < E) s_off[e] = run; run += loc[c]; }
    if (lane == 63) s_off[E] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kPerThread; ++c) {
    const int i = tid + c * kSmallThreads;
    if (i >= n) break;
    int p = -1;
    if (pe[c] >= 0) {
      const int t = i / K;
      p = s_off[pe[c]] + __popcll(s_mask[pe[c]][t >> 6] & lanemask_lt(t & 63));
#pragma unroll
      for (int w = 0; w < kWords - 1; ++w) if (w < t >> 6) p += __popcll(s_mask[pe[c]][w]);
      sorted_token[p] = t;
      sorted_rank[p] = i - t * K;
    }
    inv_pos[i] = p;
  }
  for (int e = tid; e <= E; e += kSmallThreads) offsets[e] = s_off[e];
  for (int i = s_off[E] + tid; i < n; i += kSmallThreads) { sorted_token[i] = -1; sorted_rank[i] = -1; }
}

// ---- large T: one workgroup per chunk of kChunk tokens ------------------------------------------
// Pass 1 counts, per chunk, the pairs of every expert (LDS integer atomics: a sum, so the result
// does not depend on their order).  Pass 2 turns the counts into each chunk's first position
// inside every expert segment, then places the chunk's pairs by their bits in the experts' token masks,
// which keeps tokens ascending inside a segment.
constexpr int kChunk = 128;
static_assert(kChunk == 128, "two mask words per chunk");
static_assert(MOE_MAX_EXPERTS <= kBigThreads, "one thread per expert");

__global__ __launch_bounds__(kBigThreads) void dispatch_count_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ k_t, int j_lo, int T, int E, int K,
    int32_t* __restrict__ counts /* [chunks][E] */) {
  __shared__ int s_hist[MOE_MAX_EXPERTS];
  const int t0 = blockIdx.x * kChunk, n = min(kChunk, T - t0) * K;
  for (int e = threadIdx.x; e < E; e += kBigThreads) s_hist[e] = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += kBigThreads) {
    const int tl = i / K, e = pair_expert(idx, k_t, j_lo, t0 + tl, i - tl * K, (size_t)t0 * K + i, E, K);
    if (e >= 0) atomicAdd(&s_hist[e], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += kBigThreads) counts[(size_t)blockIdx.x * E + e] = s_hist[e];
}

__global__ __launch_bounds__(kBigThreads) void dispatch_scatter_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ k_t, int j_lo, int T, int E, int K,
    const int32_t* __restrict__ counts, int n_chunks, int per_chunk, int32_t* __restrict__ offsets,
    int32_t* __restrict__ sorted_token, int32_t* __restrict__ sorted_rank,
    int32_t* __restrict__ inv_pos) {
  constexpr int kWords = kChunk / 64, kPerThread = kChunk * MOE_MAX_TOPK / kBigThreads;
  __shared__ unsigned long long s_mask[MOE_MAX_EXPERTS][kWords];
  __shared__ int s_base[MOE_MAX_EXPERTS];       // first position of this chunk inside expert e's segment
  __shared__ int s_before[MOE_MAX_EXPERTS], s_tot[MOE_MAX_EXPERTS];
  __shared__ int s_wsum[kBigThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int chunk = blockIdx.x, t0 = chunk * kChunk, np = min(kChunk, T - t0) * K;
  int pe[kPerThread];                                  // this thread's pairs of the chunk
#pragma unroll
  for (int c = 0; c < kPerThread; ++c) {
    const int i = tid + c * kBigThreads, tl = i / K;
    pe[c] = i < np ? pair_expert(idx, k_t, j_lo, t0 + tl, i - tl * K, (size_t)t0 * K + i, E, K) : -1;
  }
  for (int i = tid; i < E * kWords; i += kBigThreads) (&s_mask[0][0])[i] = 0;
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kPerThread; ++c) {
    const int tl = (tid + c * kBigThreads) / K;
    if (pe[c] >= 0) atomicOr(&s_mask[pe[c]][tl >> 6], 1ull << (tl & 63));
  }
  // per expert (one thread each, E <= 256 = kBigThreads): pairs in earlier chunks, pairs in all
  // chunks.  The count table (per_chunk rows for a chunk) is read with coalesced loads by all threads, each of which adds up
  // every 256/E-th row of an expert; the parts meet in LDS (a per-thread loop over global memory would pay one
  // memory latency per row).
  const int first_row = chunk * per_chunk, n_rows = n_chunks * per_chunk, parts = kBigThreads / E;
  if (tid < E) s_before[tid] = s_tot[tid] = 0;
  __syncthreads();
  if (tid < parts * E) {
    const int e = tid % E;
    int bf = 0, all = 0;
    for (int r0 = tid / E; r0 < n_rows; r0 += 8 * parts) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { const int r = r0 + u * parts; v[u] = r < n_rows ? counts[(size_t)r * E + e] : 0; }
#pragma unroll
      for (int u = 0; u < 8; ++u) { all += v[u]; if (r0 + u * parts < first_row) bf += v[u]; }
    }
    atomicAdd(&s_before[e], bf);
    atomicAdd(&s_tot[e], all);
  }
  __syncthreads();
  const int before = tid < E ? s_before[tid] : 0, tot = tid < E ? s_tot[tid] : 0;
  // exclusive prefix of tot over the experts -> expert_offsets
  const int incl = wave_scan(tot);
  if (lane == 63) s_wsum[wave] = incl;
  __syncthreads();
  int wbase = 0, P = 0;
#pragma unroll
  for (int w = 0; w < kBigThreads / 64; ++w) { if (w < wave) wbase += s_wsum[w]; P += s_wsum[w]; }
  const int off_e = wbase + incl - tot;
  if (tid < E) {
    s_base[tid] = off_e + before;
    if (chunk == 0) offsets[tid] = off_e;
  }
  if (chunk == 0 && tid == 0) offsets[E] = P;
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kPerThread; ++c) {
    const int i = tid + c * kBigThreads;
    if (i >= np) break;
    int p = -1;
    if (pe[c] >= 0) {
      const int tl = i / K;
      p = s_base[pe[c]] + __popcll(s_mask[pe[c]][tl >> 6] & lanemask_lt(tl & 63));
      if (tl >= 64) p += __popcll(s_mask[pe[c]][0]);
      sorted_token[p] = t0 + tl;
      sorted_rank[p] = i - tl * K;
    }
    inv_pos[(size_t)t0 * K + i] = p;
  }
  // positions beyond P are not pairs
  const int n = T * K;
  for (int i = P + chunk * kBigThreads + tid; i < n; i += n_chunks * kBigThreads) { sorted_token[i] = -1; sorted_rank[i] = -1; }
}

// T == 0: only the offsets exist
__global__ void dispatch_empty_kernel(int E, int32_t* offsets) {
  for (int e = threadIdx.x; e <= E; e += blockDim.x) offsets[e] = 0;
}

}  // namespace

int dispatch_chunks(int T) { return (T + kChunk - 1) / kChunk; }
int route_count_rows(int T) { return dispatch_chunks(T) * (kChunk / kRouteTokens); }

int launch_dispatch(const moe_config& c, const int32_t* idx, const int32_t* k_t, int j_lo, int32_t* offsets,
                    int32_t* sorted_token, int32_t* sorted_rank, int32_t* inv_pos, int32_t* counts,
                    bool counted, hipStream_t s) {
  if (c.T == 0) {
    hipLaunchKernelGGL(dispatch_empty_kernel, dim3(1), dim3(256), 0, s, c.E, offsets);
  } else if (c.T <= kSmallDispatchT) {
    hipLaunchKernelGGL(dispatch_small_kernel, dim3(1), dim3(kSmallThreads), 0, s, idx, k_t, j_lo, c.T, c.E,
                       c.k_big, offsets, sorted_token, sorted_rank, inv_pos);
  } else {
    const int n_chunks = dispatch_chunks(c.T);
    if (!counted)
      hipLaunchKernelGGL(dispatch_count_kernel, dim3((unsigned)n_chunks), dim3(kBigThreads), 0, s, idx, k_t,
                         j_lo, c.T, c.E, c.k_big, counts);
    // rows behind the last 16 tokens do not exist: the selection kernel writes zeros there
    hipLaunchKernelGGL(dispatch_scatter_kernel, dim3((unsigned)n_chunks), dim3(kBigThreads), 0, s, idx, k_t,
                       j_lo, c.T, c.E, c.k_big, counts, n_chunks, counted ? kChunk / kRouteTokens : 1, offsets,
                       sorted_token, sorted_rank, inv_pos);
  }
  return hip_fail(hipGetLastError(), "dispatch launch");
}

}  // namespace mm
