// Selection stage (Sec. II-A) with the big-little rule (Sec. III-A, Alg. 1): softmax over all
// experts, importance flag from the token's confidence, and the k_t best experts in the order
// (logit descending, expert id ascending).
//
// Selection runs in one wavefront per token; an expert row of up to 256 logits lives in
// registers (4 per lane) and every reduction is a butterfly of cross-lane shuffles.  All
// selection decisions are comparisons on the fp32 logits, so they are exact and reproducible.
//
// Kernels:
//   gate_route_kernel router logits and selection of one token per workgroup (small steps)
//   gate_gemv_kernel  router logits alone (65 to 256 tokens that the former is not for): plain fp32
//                     FMAs, one wave per block of 2 experts x 4 tokens
//   gate_mfma_kernel  router logits alone (more than 256 tokens): MFMA
//   route_kernel      softmax / importance / top-k on given logits, and the number of pairs of each expert for the dispatch
#include "internal.h"
#include "groups.h"
#include "route_device.h"

namespace mm {
namespace {

// COUNT: kRouteTokens tokens per workgroup, and a row of `counts` with the pairs of each expert among them.  Rows
// behind the last token are zeros.
template <int WAVES, bool COUNT>
__global__ __launch_bounds__(WAVES * 64) void route_kernel(const float* __restrict__ logits, int32_t* __restrict__ counts,
                                                            const RouteParams P) {
  __shared__ int s_hist[COUNT ? MOE_MAX_EXPERTS : 1];
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * WAVES + (threadIdx.x >> 6);
  if (COUNT) {
    for (int e = threadIdx.x; e < P.E; e += WAVES * 64) s_hist[e] = 0;
    __syncthreads();
  }
  if (t < P.T) {
    float raw[kPerLane];
#pragma unroll
    for (int c = 0; c < kPerLane; ++c) {
      const int e = lane + 64 * c;
      raw[c] = (e < P.E) ? logits[(size_t)t * P.E + e] : 0.f;
    }
    const Selection sel = select_token(P, t, lane, raw);
    if (COUNT && lane < sel.k) atomicAdd(&s_hist[sel.expert], 1);
  }
  if (!COUNT) return;
  __syncthreads();
  for (int e = threadIdx.x; e < P.E; e += WAVES * 64) counts[(size_t)blockIdx.x * P.E + e] = s_hist[e];
}

// One wave per block of TE experts x TT tokens: the lanes split the hidden dimension, every
// operand chunk is a 16/32-byte load, and the block's sums are reduced with shuffles.
constexpr int kGemvWaves = 4;

template <typename S, int TE, int TT>
__global__ __launch_bounds__(kGemvWaves * 64) void gate_gemv_kernel(const S* __restrict__ x,
                                                                     const S* __restrict__ Wg,
                                                                     const float* __restrict__ bias, int T,
                                                                     int H, int E,
                                                                     float* __restrict__ logits) {
  const int lane = threadIdx.x & 63;
  const int wid = blockIdx.x * kGemvWaves + (threadIdx.x >> 6);
  const int n_eb = (E + TE - 1) / TE, n_tb = (T + TT - 1) / TT;
  if (wid >= n_eb * n_tb) return;                      // whole wave leaves together
  const int e0 = (wid % n_eb) * TE, t0 = (wid / n_eb) * TT;
  float acc[TE][TT];
#pragma unroll
  for (int a = 0; a < TE; ++a)
#pragma unroll
    for (int b = 0; b < TT; ++b) acc[a][b] = 0.f;
  const int nchunk = H >> 3;                           // 8 elements per chunk
  // U chunks per trip with all loads issued before the first FMA: a lane has only H/512 chunks,
  // so with one chunk per trip the kernel would be a chain of exposed load latencies.  The FMA
  // order per accumulator (chunks ascending) is the same for every U.
  constexpr int U = sizeof(S) == 2 ? 4 : 2;
  for (int c0 = lane; c0 < nchunk; c0 += 64 * U) {
    Raw8<S> xr[U][TT], wr[U][TE];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = min(c0 + 64 * u, nchunk - 1);      // a chunk past the end is loaded again and skipped
#pragma unroll
      for (int b = 0; b < TT; ++b) xr[u][b].load(x + (size_t)min(t0 + b, T - 1) * H + c * 8);
#pragma unroll
      for (int a = 0; a < TE; ++a) wr[u][a].load(Wg + (size_t)min(e0 + a, E - 1) * H + c * 8);   // clamped rows are discarded below
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c0 + 64 * u < nchunk) {
        float xv[TT][8];
#pragma unroll
        for (int b = 0; b < TT; ++b) xr[u][b].get(xv[b]);
#pragma unroll
        for (int a = 0; a < TE; ++a) {
          float wv[8];
          wr[u][a].get(wv);
#pragma unroll
          for (int b = 0; b < TT; ++b)
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[a][b] = fmaf(xv[b][i], wv[i], acc[a][b]);
        }
      }
    }
  }
#pragma unroll
  for (int a = 0; a < TE; ++a)
#pragma unroll
    for (int b = 0; b < TT; ++b) {
      const float sum = wave_sum(acc[a][b]);
      const int e = e0 + a, t = t0 + b;
      if (lane == 0 && e < E && t < T) logits[(size_t)t * E + e] = sum + (bias ? bias[e] : 0.f);
    }
}

template <typename S, int TE, int TT>
void launch_gemv(const moe_config& c, const void* x, const void* Wg, const float* bias, float* logits,
                 hipStream_t s) {
  const int waves = ((c.E + TE - 1) / TE) * ((c.T + TT - 1) / TT);
  hipLaunchKernelGGL((gate_gemv_kernel<S, TE, TT>), dim3((unsigned)((waves + kGemvWaves - 1) / kGemvWaves)),
                     dim3(kGemvWaves * 64), 0, s, static_cast<const S*>(x), static_cast<const S*>(Wg), bias,
                     c.T, c.H, c.E, logits);
}

// Router logits and selection of one token in one workgroup (small steps): the waves split the
// experts, every wave sums its experts' dot products exactly as gate_gemv_kernel does (per lane
// the 8-element chunks lane, lane + 64, ... in ascending order, then the same shuffle reduction),
// so the logits are bit-identical to that kernel's; they go to global memory and to LDS, and wave
// 0 selects from LDS.  One launch instead of two dependent ones.
constexpr int kFusedWaves = 16;

template <typename S>
__global__ __launch_bounds__(kFusedWaves * 64) void gate_route_kernel(const S* __restrict__ x,
                                                                       const S* __restrict__ Wg,
                                                                       const float* __restrict__ bias, int H,
                                                                       float* __restrict__ logits,
                                                                       const RouteParams P) {
  __shared__ float s_logit[MOE_MAX_EXPERTS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.x, E = P.E;
  float* const logits_row = logits + (size_t)t * E;
  gate_logits_token<S, kFusedWaves>(x + (size_t)t * H, Wg, bias, H, E, 0, E, wave, lane,
                                    [&](int e, float z) { logits_row[e] = z; s_logit[e] = z; });
  __syncthreads();
  if (wave != 0) return;
  float raw[kPerLane];
#pragma unroll
  for (int c = 0; c < kPerLane; ++c) {
    const int e = lane + 64 * c;
    raw[c] = (e < E) ? s_logit[e] : 0.f;
  }
  select_token(P, t, lane, raw);
}

// Router logits of more than 256 tokens: MT x 16 tokens and NT x 16 experts per workgroup of 16 waves, which split the
// contraction.  What bounds it is what one CU fetches of rows that the weight stream has pushed out of the caches: about 50
// bytes per ns, whatever is in flight.  So the tile is the smallest whose workgroups still fit the CUs at once (128 KB for one
// tile of either at a hidden size of 2048), a wave issues the loads of whole cache lines of all its rows before the
// first product, and the partial sums meet in LDS.  us, a register-ring GEMM with items of 16 tokens x 32 experts on four waves /
// here: 64 experts of 2048, 300 tokens 10.7 / 6.0, 700 tokens 10.6 / 6.1, 2000 tokens 11.2 / 8.1, 4000 tokens 18.0 / 11.0; 8 experts of
// 4096, 300 tokens 11.3 / 8.0, 4000 tokens 15.1 / 13.4.  Steps that do not fit take 32 tokens x 32 experts, with up to 16 experts x 16: half of the
// larger tile would not exist (in a graph, 32 x 32 / 32 x 16: 8 of 4096, 4500 tokens 16.1 / 15.0, 32768 tokens 58.9 / 55.3; 16 of 2048, 16384 tokens
// 21.5 / 20.2; rows from memory the same; 16 x 16, two workgroups per CU 31.1 / 28.0 from memory there but 37 / 30 at 16 of 7168, 4112 tokens).  Measured and not kept: all experts and the selection in the same workgroup (300 tokens, 64
// experts of 2048: 14.2, against 6.8 and a selection of 4.6: 320 KB through one CU).
constexpr int kMfmaWaves = 16;

typedef __attribute__((ext_vector_type(4))) float f32x4;

// 8 consecutive k of one row: the operand of one 16x16x32 product, or of eight 16x16x4 ones, whose i-th takes
// the i-th element of every lane's eight
template <typename S> struct Frag8;
template <> struct Frag8<uint16_t> {
  bf16x8 v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned off, int soff) {
    v = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, soff, 0));
  }
  static __device__ __forceinline__ f32x4 mma(const Frag8& a, const Frag8& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
  }
};
template <> struct Frag8<float> {
  f32x4 lo, hi;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, unsigned off, int soff) {
    lo = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, soff, 0));
    hi = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off + 16u), soff, 0));   // kOob + 16 is out of range too
  }
  static __device__ __forceinline__ f32x4 mma(const Frag8& a, const Frag8& b, f32x4 c) {
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.lo[i], b.lo[i], c, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.hi[i], b.hi[i], c, 0, 0, 0);
    return c;
  }
};

template <typename S, int MT, int NT>
__global__ __launch_bounds__(kMfmaWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void gate_mfma_kernel(
    const S* __restrict__ x, const S* __restrict__ Wg, const float* __restrict__ bias, int T, int H, int E, float* __restrict__ logits) {
  constexpr int U = sizeof(S) == 2 ? 4 : 2;              // k-steps of 32 per trip: 256 bytes of a row
  constexpr int kRow = 20;                               // floats of a tile's row: the lanes of a store meet a bank twice at most
  constexpr unsigned esz = sizeof(S);
  __shared__ float s_part[kMfmaWaves][MT * NT][16][kRow];
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int q = lane >> 4, c16 = lane & 15;
  const int t0 = blockIdx.x * MT * 16, e0 = blockIdx.y * NT * 16;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(x, (unsigned)T * (unsigned)H * esz), rw = make_rsrc(Wg, (unsigned)E * (unsigned)H * esz);
  const unsigned row = (unsigned)H * esz;
  unsigned xo[MT], wo[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) xo[i] = t0 + 16 * i + c16 < T ? (unsigned)(t0 + 16 * i + c16) * row + (unsigned)q * 8u * esz : kOob;
#pragma unroll
  for (int j = 0; j < NT; ++j) wo[j] = e0 + 16 * j + c16 < E ? (unsigned)(e0 + 16 * j + c16) * row + (unsigned)q * 8u * esz : kOob;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // groups of U k-steps, dealt to the waves; then the k-steps left over, one by one
  const int groups = H / (32 * U), steps = (H + 31) >> 5;
  for (int g = wave; g < groups; g += kMfmaWaves) {
    const int k = uniform(g * U * 32);
    Frag8<S> fx[U][MT], fw[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < MT; ++i) fx[u][i].load(rx, xo[i], (k + 32 * u) * (int)esz);
#pragma unroll
      for (int j = 0; j < NT; ++j) fw[u][j].load(rw, wo[j], (k + 32 * u) * (int)esz);
    }
    __builtin_amdgcn_sched_barrier(0);                   // all loads before the first product
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = Frag8<S>::mma(fx[u][i], fw[u][j], acc[i][j]);
  }
  for (int st = groups * U + wave; st < steps; st += kMfmaWaves) {
    const unsigned none = st * 32 + q * 8 < H ? 0u : kOob;   // beyond the row: zeros
    Frag8<S> fx[MT], fw[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) fx[i].load(rx, (xo[i] + (unsigned)(st * 32) * esz) | none, 0);
#pragma unroll
    for (int j = 0; j < NT; ++j) fw[j].load(rw, (wo[j] + (unsigned)(st * 32) * esz) | none, 0);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = Frag8<S>::mma(fx[i], fw[j], acc[i][j]);
  }
  // accumulator v of a lane: token 4 q + v, expert c16 of the tile
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) s_part[wave][i * NT + j][4 * q + v][c16] = acc[i][j][v];
  __syncthreads();
  if (tid < MT * NT * 256) {
    const int r = tid / (16 * NT), c = tid % (16 * NT), t = t0 + r, e = e0 + c;
    float z = 0.f;
#pragma unroll
    for (int w = 0; w < kMfmaWaves; ++w) z += s_part[w][(r >> 4) * NT + (c >> 4)][r & 15][c & 15];
    if (t < T && e < E) logits[(size_t)t * E + e] = z + (bias ? bias[e] : 0.f);
  }
}

template <typename S, int MT, int NT>
void launch_gate_mfma_tile(const moe_config& c, const void* x, const void* Wg, const float* bias, float* logits, hipStream_t s) {
  const dim3 grid((unsigned)((c.T + 16 * MT - 1) / (16 * MT)), (unsigned)((c.E + 16 * NT - 1) / (16 * NT)));
  hipLaunchKernelGGL((gate_mfma_kernel<S, MT, NT>), grid, dim3(kMfmaWaves * 64), 0, s, static_cast<const S*>(x),
                     static_cast<const S*>(Wg), bias, c.T, c.H, c.E, logits);
}
template <typename S>
void launch_gate_mfma_typed(const moe_config& c, const void* x, const void* Wg, const float* bias, float* logits, hipStream_t s) {
  const int tt = (c.T + 15) / 16, et = (c.E + 15) / 16, cus = device_cu_count();
  if (tt * et <= cus) launch_gate_mfma_tile<S, 1, 1>(c, x, Wg, bias, logits, s);
  else if (tt * ((et + 1) / 2) <= cus) launch_gate_mfma_tile<S, 1, 2>(c, x, Wg, bias, logits, s);
  else if (et == 1) launch_gate_mfma_tile<S, 2, 1>(c, x, Wg, bias, logits, s);
  else launch_gate_mfma_tile<S, 2, 2>(c, x, Wg, bias, logits, s);
}

// conf[t] = 1 / sum_v exp(z_tv - max_v z_tv): one workgroup per token, one sweep over the row.
// Bound: a single CU's share of the work, since a row stays in one workgroup (the call has no
// workspace through which several could meet): one v_exp_f32 and a few more vector instructions per
// logit, under 16-byte loads, kConfUnroll of them in flight per thread.  Every thread keeps a running
// maximum m and s = sum exp(z - m) over the values seen, rescaled when a batch of loads raises m, so the row is
// read once.  T = 64, V = 131072: 206 us with one 4-byte load in flight per thread and two sweeps, 10.4 us so.
constexpr int kConfUnroll = 8;

struct ExpSum { float m, s; };                          // s = sum exp(z - m)

// exp(d), d <= 0, is e = exp2(p) with p = d log2 e rounded: off by about |d| 2^-24 of it, on top of the
// hardware's own error.  EXACT adds up e times the low half of d log2 e in `low`: e + ln 2 low has expf's error.
constexpr float kLog2eHi = 1.44269504088896341f, kLog2eLo = 1.92596299e-8f;
template <bool EXACT>
__device__ __forceinline__ float conf_exp(float d) { return EXACT ? expf(d) : __builtin_amdgcn_exp2f(d * kLog2eHi); }
template <bool EXACT>
__device__ __forceinline__ void conf_add(float d, float& sum, float& low) {
  const float p = d * kLog2eHi, e = __builtin_amdgcn_exp2f(p);
  sum += e;
  // -inf: e is 0 and the low half NaN, which the median turns into a number
  if (EXACT) low = fmaf(e, __builtin_amdgcn_fmed3f(fmaf(d, kLog2eLo, fmaf(d, kLog2eHi, -p)), -1.f, 1.f), low);
}
// nothing but -inf seen yet: every term is exp(-inf) = 0
__device__ __forceinline__ float conf_base(float m) { return m == -INFINITY ? 0.f : m; }
template <bool EXACT>
__device__ __forceinline__ float conf_rescale(ExpSum a, float m) { return a.m == m ? a.s : a.s * conf_exp<EXACT>(a.m - m); }

template <int THREADS, bool EXACT>
__global__ __launch_bounds__(THREADS) void confidence_kernel(const float* __restrict__ z, int V,
                                                              float* __restrict__ conf) {
  constexpr int kWaves = THREADS / 64;
  __shared__ float s_m[kWaves], s_s[kWaves];
  const float* row = z + (size_t)blockIdx.x * V;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  ExpSum a = {-INFINITY, 0.f};
  // rows of an odd V start anywhere: single values up to the first 16-byte boundary, and behind the last
  const int head = min(V, (int)((16u - ((unsigned)(uintptr_t)row & 15u)) & 15u) >> 2);
  const int n4 = (V - head) >> 2, tail = head + 4 * n4;
  const float4* body = reinterpret_cast<const float4*>(row + head);
  for (int i0 = tid; i0 < n4; i0 += THREADS * kConfUnroll) {
    float4 v[kConfUnroll];
#pragma unroll
    for (int u = 0; u < kConfUnroll; ++u) {
      const int i = i0 + u * THREADS;
      v[u] = i < n4 ? body[i] : float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
    float m = a.m;
#pragma unroll
    for (int u = 0; u < kConfUnroll; ++u) m = fmaxf(fmaxf(fmaxf(m, v[u].x), fmaxf(v[u].y, v[u].z)), v[u].w);
    a.s = conf_rescale<EXACT>(a, m);
    a.m = m;
    const float mb = conf_base(m);
    float part[4] = {0.f, 0.f, 0.f, 0.f}, low[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < kConfUnroll; ++u) {
      conf_add<EXACT>(v[u].x - mb, part[0], low[0]); conf_add<EXACT>(v[u].y - mb, part[1], low[1]);
      conf_add<EXACT>(v[u].z - mb, part[2], low[2]); conf_add<EXACT>(v[u].w - mb, part[3], low[3]);
    }
    a.s += fmaf((low[0] + low[1]) + (low[2] + low[3]), 0.693147180559945309f, (part[0] + part[1]) + (part[2] + part[3]));
  }
  const int extra = tid < head ? tid : tail + tid - head;   // at most 3 + 3 single values
  if (extra < V && tid < head + (V - tail)) {
    const float x = row[extra], m = fmaxf(a.m, x);
    a.s = conf_rescale<EXACT>(a, m);
    a.m = m;
    a.s += conf_exp<EXACT>(x - conf_base(m));
  }
  // the workgroup's maximum, then every thread's sum brought to it (EXACT: in one step, with one rounding less)
  const float wm = wave_max(a.m);
  float m, tot;
  if constexpr (EXACT) {
    if (lane == 0) s_m[wave] = wm;
    __syncthreads();
    m = wave_max(lane < kWaves ? s_m[lane] : -INFINITY);
    const float ws = wave_sum(conf_rescale<EXACT>(a, m));
    if (lane == 0) s_s[wave] = ws;
    __syncthreads();
    if (wave != 0) return;
    tot = wave_sum(lane < kWaves ? s_s[lane] : 0.f);
  } else {
    const float ws = wave_sum(conf_rescale<EXACT>(a, wm));
    if (lane == 0) { s_m[wave] = wm; s_s[wave] = ws; }
    __syncthreads();
    if (wave != 0) return;
    const ExpSum w = {lane < kWaves ? s_m[lane] : -INFINITY, lane < kWaves ? s_s[lane] : 0.f};
    m = wave_max(w.m);
    tot = wave_sum(conf_rescale<EXACT>(w, m));
  }
  if (lane != 0) return;
  conf[blockIdx.x] = m == -INFINITY ? NAN : 1.f / tot;   // a row of -inf has no distribution
}

RouteParams make_params(const moe_config& c, const float* conf, int32_t* idx, float* w, uint8_t* important,
                        int32_t* k_t) {
  RouteParams P;
  P.conf = conf; P.gamma = c.gamma; P.T = c.T; P.E = c.E; P.k_big = c.k_big; P.k_little = c.k_little;
  P.renorm = c.renorm; P.idx = idx; P.w = w; P.important = important; P.k_t = k_t;
  return P;
}

}  // namespace

int launch_route(const moe_config& c, const float* conf, const float* logits, int32_t* idx, float* w,
                 uint8_t* important, int32_t* k_t, int32_t* counts, hipStream_t s) {
  if (c.T == 0) return MOE_OK;
  const RouteParams P = make_params(c, conf, idx, w, important, k_t);
  if (counts)
    hipLaunchKernelGGL((route_kernel<kRouteTokens, true>), dim3((unsigned)route_count_rows(c.T)), dim3(kRouteTokens * 64), 0, s, logits, counts, P);
  else
    hipLaunchKernelGGL((route_kernel<kWavesPerBlock, false>), dim3((unsigned)((c.T + kWavesPerBlock - 1) / kWavesPerBlock)),
                       dim3(kWavesPerBlock * 64), 0, s, logits, counts, P);
  return hip_fail(hipGetLastError(), "route_kernel launch");
}

// Router logits + selection in one launch; for small steps (rule in moe_route).
int launch_gate_route(const moe_config& c, const void* x, const void* Wg, const float* bias, const float* conf,
                      float* logits, int32_t* idx, float* w, uint8_t* important, int32_t* k_t, hipStream_t s) {
  if (c.T == 0) return MOE_OK;
  const RouteParams P = make_params(c, conf, idx, w, important, k_t);
  if (c.dtype != MOE_FP32)
    hipLaunchKernelGGL(gate_route_kernel<uint16_t>, dim3((unsigned)c.T), dim3(kFusedWaves * 64), 0, s,
                       static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(Wg), bias, c.H, logits, P);
  else
    hipLaunchKernelGGL(gate_route_kernel<float>, dim3((unsigned)c.T), dim3(kFusedWaves * 64), 0, s,
                       static_cast<const float*>(x), static_cast<const float*>(Wg), bias, c.H, logits, P);
  return hip_fail(hipGetLastError(), "gate_route_kernel launch");
}

int launch_gate_mfma(const moe_config& c, const void* x, const void* Wg, const float* bias, float* logits, hipStream_t s) {
  if (c.T == 0) return MOE_OK;
  if (c.dtype != MOE_FP32) launch_gate_mfma_typed<uint16_t>(c, x, Wg, bias, logits, s);
  else launch_gate_mfma_typed<float>(c, x, Wg, bias, logits, s);
  return hip_fail(hipGetLastError(), "gate_mfma_kernel launch");
}

int launch_gate_gemv(const moe_config& c, const void* x, const void* Wg, const float* bias, float* logits,
                     hipStream_t s) {
  if (c.T == 0) return MOE_OK;
  const bool bf = c.dtype != MOE_FP32;
  if (bf) launch_gemv<uint16_t, 2, 4>(c, x, Wg, bias, logits, s); else launch_gemv<float, 2, 4>(c, x, Wg, bias, logits, s);
  return hip_fail(hipGetLastError(), "gate_gemv_kernel launch");
}

// Long rows do without the low halves: error against 64 bits there is below that of the two sweeps with expf that
// this kernel replaced, whose chains of additions grew with the row, while the low halves cost four more
// vector instructions per logit (64 rows of 131072 9.4 -> 13.3 us).  RMS of the relative error, 1e-8, two sweeps /
// without / with: random rows of 1000 6.0 / 6.4 / 5.8, 8193 6.0 / 6.5 / 5.3, 32768 7.7 / 6.8 / 5.2, 50257 7.8 / 6.9,
// 131072 15 / 7.5; rows of one value beside a larger one, 1000 8.6 / 9.9 / 5.3, 8192 28 / 16 / 6, 65536 175 / 21.
// Up to 36864 values with them take the time without: 64 rows of 32001 6.8 us (two sweeps 35.3).
constexpr int kConfExactMaxV = 36864;

int launch_confidence(const float* z, int T, int V, float* conf, hipStream_t s) {
  if (T == 0) return MOE_OK;
  // a row of at most 8192 values is one batch of loads of 256 threads; a larger workgroup would only add waves
  // without a load to the reduction (T = 64, both about 7.4 us, the rate of launches)
  if (V <= 8192) hipLaunchKernelGGL((confidence_kernel<256, true>), dim3((unsigned)T), dim3(256), 0, s, z, V, conf);
  else if (V <= kConfExactMaxV) hipLaunchKernelGGL((confidence_kernel<1024, true>), dim3((unsigned)T), dim3(1024), 0, s, z, V, conf);
  else hipLaunchKernelGGL((confidence_kernel<1024, false>), dim3((unsigned)T), dim3(1024), 0, s, z, V, conf);
  return hip_fail(hipGetLastError(), "confidence_kernel launch");
}

}  // namespace mm
