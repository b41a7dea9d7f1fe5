// Device-side pieces of the selection stage (Sec. II-A with the big-little rule of Sec. III-A,
// Alg. 1) shared by the kernels that route tokens: wave-wide reductions, the selection of one token
// by one wavefront, and the router dot products of one token.
#pragma once

#include <math.h>

#include <type_traits>

#include "internal.h"

namespace mm {
namespace {

constexpr int kPerLane = MOE_MAX_EXPERTS / 64;   // 4
constexpr int kWavesPerBlock = 4;

// Wave-wide reductions on the data-parallel-primitive path (no LDS round trips): quads, half
// rows and rows with quad_perm / row_half_mirror / row_mirror, then lane 15 of a row into the
// next row and lane 31 into rows 2 and 3, so that lane 63 holds the result, which is read back
// as a scalar.  `ident` is what a lane outside the row mask contributes.
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, T ident, Op op) {
  const auto dpp = [](T old, T x, auto ctrl, auto rows) {
    const int r = __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, x),
                                              decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    return __builtin_bit_cast(T, r);
  };
  using std::integral_constant;
  v = op(v, dpp(v, v, integral_constant<int, 0xB1>{}, integral_constant<int, 0xf>{}));    // quad_perm [1,0,3,2]
  v = op(v, dpp(v, v, integral_constant<int, 0x4E>{}, integral_constant<int, 0xf>{}));    // quad_perm [2,3,0,1]
  v = op(v, dpp(v, v, integral_constant<int, 0x141>{}, integral_constant<int, 0xf>{}));   // row_half_mirror
  v = op(v, dpp(v, v, integral_constant<int, 0x140>{}, integral_constant<int, 0xf>{}));   // row_mirror
  v = op(v, dpp(ident, v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{}));   // row_bcast:15 into rows 1, 3
  v = op(v, dpp(ident, v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{}));   // row_bcast:31 into rows 2, 3
  return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_reduce(v, 0.f, [](float a, float b) { return a + b; });
}

struct RouteParams {
  const float* conf;
  float gamma;
  int T, E, k_big, k_little, renorm;
  int32_t* idx;
  float* w;
  uint8_t* important;
  int32_t* k_t;
};

// What one wave decides for a token: lane j < k_big holds the j-th selected expert and its routing
// weight (-1 / 0 from rank k on); k and imp are the same in all lanes.
struct Selection {
  int expert;
  float weight;
  int k;
  bool imp;
};

// One wave selects for token t.  raw[c] = logit of expert lane + 64*c (anything for e >= E); E <= 64 PL.
// A round costs one reduction: the best value's expert is the first bit of a ballot and its probability one lane's.  With
// a second reduction for the lowest id and a third for the probability, and four experts per lane whatever E, route_kernel took, us, now /
// then: 8 / 4 of 64 experts, 300 tokens 4.8 / 5.5, 2000 tokens 4.9 / 6.3, 4000 tokens 5.2 / 8.3 (4.6 is what any launch takes there).
// Lanes of several experts keep their best one beside them, so that a ballot for each set of 64 is only taken where lanes tie.  us in a
// graph, moe_route on given logits, three reductions / a ballot per set in every round / so: 16 of 65 experts, 64 tokens 7.3 / 8.4 / 6.7, 8 of 128, 64
// tokens 4.8 / 5.3 / 4.5, 2048 tokens 6.0 / 6.1 / 5.1.
template <int PL>
__device__ __forceinline__ Selection select_values(const RouteParams& P, int t, int lane, const float* raw) {
  const float NINF = -INFINITY;
  const int E = P.E;
  float v[PL];
  unsigned open = 0;                                   // bit c: this lane's c-th expert exists and is not taken
#pragma unroll
  for (int c = 0; c < PL; ++c) {
    const bool ok = lane + 64 * c < E;
    const float x = ok ? raw[c] : NINF;
    v[c] = (x != x) ? NINF : x;                        // NaN counts as -inf
    open |= ok ? 1u << c : 0u;
  }
  // softmax statistics over all E
  float m = v[0];
#pragma unroll
  for (int c = 1; c < PL; ++c) m = fmaxf(m, v[c]);
  m = wave_max(m);
  float p[PL];
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < PL; ++c) {
    p[c] = (lane + 64 * c < E && m != NINF) ? expf(v[c] - m) : 0.f;
    s += p[c];
  }
  s = wave_sum(s);
  const float inv_s = s > 0.f ? 1.f / s : 0.f;

  // Alg. 1: the little result is kept only if the confidence is strictly above gamma
  const bool imp = P.conf ? !(P.conf[t] > P.gamma) : true;
  const int k = __builtin_amdgcn_readfirstlane(imp ? P.k_big : P.k_little);   // one token: the same in all lanes

  // k rounds of "best expert not taken yet"
  float my_w = 0.f;                                    // lane j keeps the j-th weight
  int my_e = -1;
  float wsum = 0.f;
  float best = m;                                      // of the experts not taken
  // PL > 1: this lane's best expert not taken, the lowest of equal ones: value, probability, set (PL: none left)
  float mine = NINF, p_mine = p[0];
  int c_mine = 0;
  auto best_of_lane = [&] {
    mine = NINF; c_mine = PL;
#pragma unroll
    for (int c = PL - 1; c >= 0; --c)
      if (((open >> c) & 1u) && v[c] >= mine) { mine = v[c]; p_mine = p[c]; c_mine = c; }
  };
  if (PL > 1) best_of_lane();
  for (int j = 0; j < k; ++j) {
    const unsigned long long at = __ballot(PL > 1 ? c_mine < PL && mine == best : (open & 1u) && v[0] == best);   // some lane holds it
    int l = (int)__builtin_ctzll(at), set = 0;
    if (PL > 1) {
      if (at & (at - 1)) {                             // several: the lowest set goes first
#pragma unroll
        for (int c = PL - 1; c >= 0; --c) {
          const unsigned long long in_set = __ballot(c_mine == c && mine == best);
          if (in_set) l = (int)__builtin_ctzll(in_set);
        }
      }
      set = __builtin_amdgcn_readlane(c_mine, l);
    }
    const int sel = 64 * set + l;
    const float psel = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, p_mine), l)) * inv_s;
    if (lane == l) open &= ~(1u << set);
    wsum += psel;
    if (lane == j) { my_w = psel; my_e = sel; }
    if (j + 1 < k) {
      if (PL > 1) best_of_lane();
      else mine = open & 1u ? v[0] : NINF;
      best = wave_max(mine);
    }
  }
  if (P.renorm) my_w = wsum > 0.f ? my_w / wsum : 0.f;
  Selection sel;
  sel.expert = lane < k ? my_e : -1;
  sel.weight = lane < k ? my_w : 0.f;
  sel.k = k;
  sel.imp = imp;
  return sel;
}
__device__ __forceinline__ Selection select_token_values(const RouteParams& P, int t, int lane,
                                                         const float (&raw)[kPerLane]) {
  return P.E <= 64 ? select_values<1>(P, t, lane, raw) : select_values<kPerLane>(P, t, lane, raw);
}

// ... and writes the token's rows of the four output arrays.
__device__ __forceinline__ Selection select_token(const RouteParams& P, int t, int lane, const float (&raw)[kPerLane]) {
  const Selection sel = select_token_values(P, t, lane, raw);
  if (lane < P.k_big) {
    P.idx[(size_t)t * P.k_big + lane] = sel.expert;
    P.w[(size_t)t * P.k_big + lane] = sel.weight;
  }
  if (lane == 0) {
    P.important[t] = sel.imp ? 1 : 0;
    P.k_t[t] = sel.k;
  }
  return sel;
}

// Eight consecutive elements as loaded (16 or 32 bytes), converted to fp32 on demand.
template <typename S> struct Raw8;
template <> struct Raw8<uint16_t> {
  uint4 u;
  __device__ __forceinline__ void load(const uint16_t* p) { u = *reinterpret_cast<const uint4*>(p); }
  __device__ __forceinline__ void get(float (&f)[8]) const {
    const unsigned w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);            // bf16 -> fp32 is a 16-bit shift
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};
template <> struct Raw8<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const float4*>(p); b = *reinterpret_cast<const float4*>(p + 4);
  }
  __device__ __forceinline__ void get(float (&f)[8]) const {
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
};

// Router logits of one token for the experts [e_begin, e_end), computed by the NWAVES waves of a
// workgroup: the waves split the experts, every wave sums its experts' dot products with the lanes
// striding the 8-element chunks of the hidden dimension (chunks lane, lane + 64, ... in ascending
// order, U chunks per trip with all loads issued before the first FMA) and reduces with the same
// shuffles everywhere, so a logit has the same bits whichever kernel calls this and however the
// experts are split.  Lane 0 of the wave that owns expert e calls store(e, logit).
template <typename S, int NWAVES, typename Store>
__device__ __forceinline__ void gate_logits_token(const S* __restrict__ xr, const S* __restrict__ Wg,
                                                  const float* __restrict__ bias, int H, int E, int e_begin,
                                                  int e_end, int wave, int lane, Store store) {
  const int nchunk = H >> 3;
  constexpr int U = sizeof(S) == 2 ? 4 : 2;
  constexpr int TE = 4;                                // experts per pass of a wave
  for (int e0 = e_begin + wave * TE; e0 < e_end; e0 += NWAVES * TE) {
    float acc[TE];
#pragma unroll
    for (int a = 0; a < TE; ++a) acc[a] = 0.f;
    for (int c0 = lane; c0 < nchunk; c0 += 64 * U) {
      Raw8<S> xv[U], wv[U][TE];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = min(c0 + 64 * u, nchunk - 1);    // a chunk past the end is loaded again and skipped
        xv[u].load(xr + c * 8);
#pragma unroll
        for (int a = 0; a < TE; ++a) wv[u][a].load(Wg + (size_t)min(e0 + a, E - 1) * H + c * 8);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (c0 + 64 * u < nchunk) {
          float xf[8];
          xv[u].get(xf);
#pragma unroll
          for (int a = 0; a < TE; ++a) {
            float wf[8];
            wv[u][a].get(wf);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[a] = fmaf(xf[i], wf[i], acc[a]);
          }
        }
      }
    }
#pragma unroll
    for (int a = 0; a < TE; ++a) {
      const float sum = wave_sum(acc[a]);
      const int e = e0 + a;
      if (lane == 0 && e < e_end) store(e, sum + (bias ? bias[e] : 0.f));
    }
  }
}

}  // namespace
}  // namespace mm
