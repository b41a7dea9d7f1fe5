// Skinny grouped GEMM for the decode regime of large layers and for prefill of few rows per expert (bf16 activations; bf16,
// 8-bit or MXFP4 weights): the operation and, per element, the order of additions of the kernel that it stands in for, so that
// either gives the same bits, and a step has the same ones whether it is issued whole or in parts: fewer than 256 tokens
// those of stream_lds.hip, from there on (MANY) those of ffn_tiled.hip and ffn_wide.hip.
//
//   kGateUp  h = silu(W_gate x) * (W_up x)     (execution stage of Sec. II-A, SwiGLU)
//   kDown    y = W_down h
//
// What bounds it: the weight stream from HBM.  In stream_lds.hip the waves that compute load the token rows from L2 one
// chunk ahead, in a queue behind the loaders' stream, with two barriers of the workgroup per 16 KB of weights; the
// narrower the weights, the shorter 16 KB last.  Here every wave streams its own rows through a ring of its own in LDS
// and nothing in the loop over k waits for another wave:
//   * One workgroup of eight waves per CU.  A wave loads units of 16 weight rows x 256 bytes (four loads into LDS of four rows
//     each; MXFP4: a fifth for the scales), waits by count for its oldest unit, reads it as MFMA fragments and at once
//     loads the next one into its place.  Three units in flight for bf16, two for the narrow formats, whose computing
//     takes longer than the latency and whose token rows need the room.
//   * The token rows of a panel come through LDS as well, in slices of as many units of k as half of the token
//     buffer holds, one slice ahead, shared by the eight waves: one barrier per slice.  Loads complete in order, so
//     a wave's count of units behind a slice tells when its part has landed.
//   * A quad is four weight rows: gate/up: two gate rows and the same two up rows, so that one lane holds both; down: four
//     rows.  A panel is up to 32 quads of one group for up to 64 token rows, a tile of up to four quads per wave.
//     All groups' panels form one list, dealt to the workgroups in rounds.  The panel's size is the smallest that needs no more
//     rounds than the largest, so that every workgroup ends at the same time: 1342 panels of 32 quads on 256 CUs
//     are 5.2 rounds, 1525 of 28.2 fill six (60 experts, 64 tokens, gate/up: the last workgroup ended 27 us behind the
//     median, now 7).
//   * With many token rows it is the reads from LDS that bound the narrow formats: 16 KB of a panel's token rows for every 4 KB of
//     weights.  RT = 2 makes a wave's share two tiles of up to four quads, whose products share the fragments of the token rows:
//     8 experts of 14336, MXFP4, 256 tokens, gate/up + down 327 / 306, 8-bit 370 tokens 450 / 400, 64 of 1408 + 2 shared, MXFP4 420 tokens
//     142 / 132, 60 of 1408 + 5632, 8-bit 420 tokens 185 / 171.  The 16 quads' accumulators still fit 256 registers at 64 rows.
//   * Steps of 256 tokens and more (MANY) have token numbers of two bytes, too many for LDS at once: the workgroup
//     looks them up for 32 of its panels at a time.  Their weights pass the caches as well: loaded through them the steps
//     were slower.
//   * In a step of one call below 256 tokens the gate/up launch builds the dispatch for itself: 0.8 us more, where a launch of
//     its own takes 3.5 to 4.8 (60 experts, 8 tokens bf16, whole step 78.7 -> 75.2, 64 tokens MXFP4 93.0 -> 88.8).  Measured and not kept: the
//     shared experts' gate/up as a launch of its own in which other workgroups select (1 token 5.7 + 20.8 -> 15.6 + 16.1: the
//     selection's loads wait behind the weight stream, and two launches fill the pipeline twice).
//   * What stands in front of the first load counts twice in a step.  From a workgroup's first instruction to its first loads of weights,
//     us: gate/up 4.7 -> 4.1 (1.9 of them for the dispatch), down 3.8 -> 3.3; the first data come 2 us later.  Measured and not kept:
//     the first loads before the table of panels, and token rows before weights (first product as late as before).
//   * Groups of more token rows are several blocks of even length, whose panels over the same weights are eight places
//     apart, i.e. on one XCD at one time.
//   * The two sums per output (even and odd groups of four 16-byte columns) are those of the two k parts in stream_lds.hip.
//     The one sum of MANY is that of the tiled kernels: a product of 32 k adds up as two of theirs of 16 k do, and tile_order()
//     gives it the k of those two.
//
// us, gate/up + down, stream_lds / here.  60 experts of 1408 + 5632: bf16, 1 token 25 + 15 / 20 + 15, 64 tokens 124 + 67 / 120 + 63,
// 255 tokens 171 + 98 / 153 + 83; 8-bit, 16 tokens 40 + 25 / 36 + 24, 64 tokens 71 + 44 / 69 + 42, 255 tokens 107 + 67 / 94 + 55;
// MXFP4, 16 tokens 31 + 22 / 26 + 19, 64 tokens 56 + 35 / 47 + 32, 255 tokens 88 + 54 / 75 + 47.  8 experts of 14336, 255 tokens:
// bf16 431 + 227 / 320 + 168, 8-bit 334 + 187 / 199 + 109, MXFP4 294 + 177 / 187 + 151.  MXFP4 at 64 tokens: 187 MB in 42 us behind the
// first load; without the products 36, without the token rows too 33.
// Measured and not kept: contiguous ranges of quads per workgroup (pieces of groups that a wave has little of last as
// long as whole ones); slices of half a unit; two tiles per wave and panel for bf16 weights (as fast, the rounds balance worse); three or four
// token buffers with a mark per load (1 - 2 % slower: the counts are no constants any more); weights and token rows
// read in one go (MXFP4 5 % slower: the next load waits for the token rows); units of 1 or 2 quads and 4 or 2 times the k for
// panels of few quads (8 experts, 1 token, down 51 -> 42, everything else 1 % slower).
#include <type_traits>

#include "internal.h"
#include "groups.h"
#include "dispatch_device.h"

namespace mm {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kWaves = 8;
constexpr int kThreadsP = kWaves * 64;
constexpr int kPanelsMany = 32;                           // panels that a workgroup of a step of 256 tokens and more looks up at a time
constexpr int kIndexMax = (kTiledMinT - 1) * MOE_MAX_TOPK;
static_assert(kTiledMinT <= 256, "the token numbers of such a step fit a byte");

// WB as in groups.h: 2 = bf16, 1 = 8-bit codes with row scales, 0 = MXFP4
template <int WB> struct Unit {
  static constexpr int kPerColumn = WB ? 16 / WB : 32;  // k per 16-byte column
  static constexpr int kK = 16 * kPerColumn;            // k per unit
  static constexpr int kParts = kK / 128;               // 128 k each: 256 bytes of a token row
  static constexpr int kRowShift = WB == 2 ? 8 : (WB == 1 ? 9 : 10);   // bytes of a token row per unit
  static constexpr int kRowsPerLoad = 4 / kParts;       // token rows of a load
  static constexpr int kBytes = 4096 + (WB == 0 ? 256 : 0);            // MXFP4: 16 scale bytes per row
  static constexpr int kLoads = 4 + (WB == 0 ? 1 : 0);
  static constexpr int kStages = WB == 2 ? 3 : 2;                      // units of a wave in flight
  static constexpr int kBuffer = (155 * 1024 - kWaves * kStages * kBytes) / 2048 * 1024;   // bytes of a slice of token rows
  static constexpr int kBlock = (kBuffer >> kRowShift) < 64 ? kBuffer >> kRowShift : 64;   // token rows of a block
  static constexpr int kTiles = (kBlock + 15) / 16;
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
#define MM_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0f70 | ((n) & 15) | (((n) >> 4) << 14))
// waits until at most BASE + extra loads of this wave are outstanding (more than 4 count as 4: a longer wait)
template <int BASE>
__device__ __forceinline__ void wait_vm(int extra) {
  switch (extra) {
    case 0: MM_WAIT_VM(BASE); break;
    case 1: MM_WAIT_VM(BASE + 1); break;
    case 2: MM_WAIT_VM(BASE + 2); break;
    case 3: MM_WAIT_VM(BASE + 3); break;
    default: MM_WAIT_VM(BASE + 4); break;
  }
  asm volatile("" ::: "memory");
}
// waits until at most n units of PER loads are
template <int PER>
__device__ __forceinline__ void wait_units(int n) {
  switch (n) {
    case 0: MM_WAIT_VM(0); break;
    case 1: MM_WAIT_VM(PER); break;
    case 2: MM_WAIT_VM(2 * PER); break;
    default: MM_WAIT_VM(3 * PER); break;
  }
  asm volatile("" ::: "memory");
}
// LDS reads of the main loop, each with its wait: what the compiler issues itself would also wait for the loads into LDS
__device__ __forceinline__ unsigned lds_read_u8(unsigned addr) {
  unsigned v;
  asm volatile("ds_read_u8 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
  return v;
}
__device__ __forceinline__ unsigned lds_read_u16(unsigned addr) {
  unsigned v;
  asm volatile("ds_read_u16 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
  return v;
}
#define MM_RD(D, A, O) "ds_read_b128 %" #D ", %" #A " offset:" #O "\n\t"
#define MM_RD4(D0, D1, D2, D3, A0, A1, A2, A3, O) MM_RD(D0, A0, O) MM_RD(D1, A1, O) MM_RD(D2, A2, O) MM_RD(D3, A3, O)
#define MM_OUT4(V) "=&v"((V)[0]), "=&v"((V)[1]), "=&v"((V)[2]), "=&v"((V)[3])
#define MM_IN4(A) "v"((A)[0]), "v"((A)[1]), "v"((A)[2]), "v"((A)[3])
// the weights of a unit; MXFP4: and the scales of this lane's row
__device__ __forceinline__ void read_weights(i32x4 (&w)[4], const unsigned (&aw)[4]) {
  asm volatile(MM_RD4(0, 1, 2, 3, 4, 5, 6, 7, 0) "s_waitcnt lgkmcnt(0)" : MM_OUT4(w) : MM_IN4(aw) : "memory");
}
__device__ __forceinline__ void read_weights(i32x4 (&w)[4], i32x4& sc, const unsigned (&aw)[4], unsigned as) {
  asm volatile(MM_RD(4, 9, 0) MM_RD4(0, 1, 2, 3, 5, 6, 7, 8, 0) "s_waitcnt lgkmcnt(0)" : MM_OUT4(w), "=&v"(sc) : MM_IN4(aw), "v"(as) : "memory");
}
// a tile of token rows
__device__ __forceinline__ void read_tokens(i32x4 (&b)[1][4], const unsigned (&ab)[4]) {
  asm volatile(MM_RD4(0, 1, 2, 3, 4, 5, 6, 7, 0) "s_waitcnt lgkmcnt(0)" : MM_OUT4(b[0]) : MM_IN4(ab) : "memory");
}
__device__ __forceinline__ void read_tokens(i32x4 (&b)[2][4], const unsigned (&ab)[4]) {
  asm volatile(MM_RD4(0, 1, 2, 3, 8, 9, 10, 11, 0) MM_RD4(4, 5, 6, 7, 8, 9, 10, 11, 256) "s_waitcnt lgkmcnt(0)"
               : MM_OUT4(b[0]), MM_OUT4(b[1]) : MM_IN4(ab) : "memory");
}
__device__ __forceinline__ void read_tokens(i32x4 (&b)[4][4], const unsigned (&ab)[4]) {
  asm volatile(MM_RD4(0, 1, 2, 3, 16, 17, 18, 19, 0) MM_RD4(4, 5, 6, 7, 16, 17, 18, 19, 256) MM_RD4(8, 9, 10, 11, 16, 17, 18, 19, 512)
               MM_RD4(12, 13, 14, 15, 16, 17, 18, 19, 768) "s_waitcnt lgkmcnt(0)"
               : MM_OUT4(b[0]), MM_OUT4(b[1]), MM_OUT4(b[2]), MM_OUT4(b[3]) : MM_IN4(ab) : "memory");
}

// Brings the codes of four 16-byte columns of a weight row, one in the lanes of each q, into the order in which the tiled
// kernel takes their k: q and q + 2 exchange halves of their columns.
//   8-bit (64 k = 8 groups of 8): products of the groups 0, 2, 1, 3 and 4, 6, 5, 7 (from the lanes of q = 0, 1, 2, 3)
//   MXFP4 (128 k = 16 groups):    of 0, 4, 1, 5, of 2, 6, 3, 7, of 8, 12, 9, 13 and of 10, 14, 11, 15
template <int WB>
__device__ __forceinline__ void tile_order(i32x4& w) {
  constexpr int far = WB == 1 ? 2 : 1;
  const auto a = __builtin_amdgcn_permlane32_swap((unsigned)w[0], (unsigned)w[far], false, false);
  const auto b = __builtin_amdgcn_permlane32_swap((unsigned)w[3 - far], (unsigned)w[3], false, false);
  w = i32x4{(int)a[0], (int)b[0], (int)a[1], (int)b[1]};
}

// Column c of a token row sits at c ^ token_key(row & 15).  A read is free of bank conflicts while the lanes of neighbouring q
// take columns whose numbers differ in a bit that the keys of rows 0 .. 3, 12 .. 15 and of rows 4 .. 11 do not differ in alone: 4 columns
// apart (MXFP4 in the tiles' order) want the bits 1 and 2 of the row exchanged.
template <int WB, bool MANY>
__device__ __forceinline__ int token_key(int row) {
  return WB == 0 && MANY ? (row & 9) | (row & 2) << 1 | (row & 4) >> 1 : row;
}

template <int WB> __device__ __forceinline__ int token_blocks(int m) { return (m + Unit<WB>::kBlock - 1) / Unit<WB>::kBlock; }

template <int WB>
struct __attribute__((aligned(1024))) SmemP {
  char tok[2][Unit<WB>::kBuffer];     // in front of the ring: reads for tokens that do not exist run into it
  char ring[kWaves][Unit<WB>::kStages * Unit<WB>::kBytes];
  union {
    unsigned char index[kIndexMax];   // fewer than 256 tokens: token of each dispatch position (gate/up)
    unsigned short rows[kPanelsMany][64];   // more: token of each row of the workgroup's panels
  };
};

// The dispatch of a step of fewer than 256 tokens, built by a whole workgroup for itself: as dispatch.hip has it (token masks by
// LDS atomic OR, positions by bit counts), with the token of each position in sm.index and the experts' rows in the lanes of every wave.
// `scratch` holds the masks and the offsets until the token rows come.  `write`: this workgroup fills the arrays of the C ABI.
struct DispatchScratch {
  unsigned long long mask[MOE_MAX_EXPERTS][kTiledMinT / 64];
  int off[MOE_MAX_EXPERTS + 1];
};
// PER: pairs of a thread
template <int NE, int PER>
__device__ __forceinline__ void build_dispatch(const StreamArgs& a, const StepDispatch& d, DispatchScratch& sc, unsigned char* index, int tid,
                                               bool write, int (&v_m)[NE], int (&v_row0)[NE]) {
  constexpr int kWords = kTiledMinT / 64;
  const int lane = tid & 63, wave = tid >> 6, E = a.E, K = d.k_big, n = a.T * K;
  const float inv_k = 1.f / (float)K;
  int pe[PER], pt[PER];                                  // this thread's pairs tid, tid + kThreadsP, ..: expert (-1: none) and token
  {
    int kt[PER];
#pragma unroll
    for (int c = 0; c < PER; ++c) {                      // all loads before the first use
      const int i = min(tid + c * kThreadsP, n - 1);
      pt[c] = (int)(((float)i + 0.5f) * inv_k);          // i / K: i < 2^12, K <= 16
      pe[c] = d.topk_idx[i];
      kt[c] = d.k_t[pt[c]];
    }
    for (int i = tid; i < E * kWords; i += kThreadsP) (&sc.mask[0][0])[i] = 0;
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const int i = tid + c * kThreadsP, j = i - pt[c] * K;
      if (!(i < n && j >= d.j_lo && j < min(kt[c], K) && (unsigned)pe[c] < (unsigned)E)) pe[c] = -1;
    }
  }
  lds_barrier();
#pragma unroll
  for (int c = 0; c < PER; ++c)
    if (pe[c] >= 0) atomicOr(&sc.mask[pe[c]][pt[c] >> 6], 1ull << (pt[c] & 63));
  lds_barrier();
  int base = 0;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    v_m[j] = v_row0[j] = 0;
    if (64 * j < E) {
      const int e = 64 * j + lane;
      int m = 0;
      if (e < E)
#pragma unroll
        for (int w = 0; w < kWords; ++w) m += __popcll(sc.mask[e][w]);
      const int incl = wave_scan(m);
      v_m[j] = m; v_row0[j] = base + incl - m;
      if (wave == 0 && e < E) { sc.off[e] = base + incl - m; if (e == E - 1) sc.off[E] = base + incl; }
      base += __builtin_amdgcn_readlane(incl, 63);
    }
  }
  lds_barrier();
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    const int i = tid + c * kThreadsP, t = pt[c];
    int p = -1;
    if (pe[c] >= 0) {
      p = sc.off[pe[c]] + __popcll(sc.mask[pe[c]][t >> 6] & lanemask_lt(t & 63));
#pragma unroll
      for (int w = 0; w < kWords - 1; ++w) if (w < t >> 6) p += __popcll(sc.mask[pe[c]][w]);
      index[p] = (unsigned char)t;
      if (write) { d.sorted_token[p] = t; d.sorted_rank[p] = i - t * K; }
    }
    if (write && i < n) d.inv_pos[i] = p;
  }
  if (write) {
    for (int e = tid; e <= E; e += kThreadsP) d.offsets[e] = sc.off[e];
    for (int i = base + tid; i < n; i += kThreadsP) { d.sorted_token[i] = -1; d.sorted_rank[i] = -1; }
  }
}

// MANY: 256 tokens and more; RT: tiles of four quads of a wave in a panel, at most
template <int MODE, int WB, bool MANY, int RT>
__global__ __launch_bounds__(kThreadsP) __attribute__((amdgpu_waves_per_eu(2, 2))) void stream_panel_kernel(const StreamArgs a, const StepDispatch d) {
  constexpr bool DISPATCH = MODE == kGateUp && !MANY;
  typedef Unit<WB> U;
  constexpr int OQ = MODE == kGateUp ? 2 : 4;            // output columns per quad
  constexpr int kPanelQuads = 4 * RT * kWaves;           // quads of a panel, at most
  __shared__ SmemP<WB> sm;
  fetch_arguments<sizeof(StreamArgs) + (DISPATCH ? sizeof(StepDispatch) : 0)>();
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int q = lane >> 4, c16 = lane & 15;
  const int n_sh = MODE == kDown ? a.n_slabs : a.n_shared;
  const unsigned ring = (unsigned)(size_t)sm.ring[wave], tok = (unsigned)(size_t)sm.tok[0], s_index = (unsigned)(size_t)sm.index;

  // ---- routed experts: expert 64 j + lane in this lane ----
  constexpr int NE = MOE_MAX_EXPERTS / 64;
  int v_end[NE], v_m[NE], v_row0[NE], v_lo[NE], v_hi[NE];   // token blocks up to and with the expert; rows, first dispatch position; weights
  int routed_blocks = 0;
  const bool dispatch = DISPATCH && d.on != 0;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    v_end[j] = v_m[j] = v_row0[j] = v_lo[j] = v_hi[j] = 0;
    if (64 * j + lane < a.n_routed) {
      GroupSrc src = {};
      if (dispatch) src.blob = a.expert_w[64 * j + lane];
      else src = load_group_src<MODE>(a, n_sh + 64 * j + lane);
      v_m[j] = src.m; v_row0[j] = src.row0;
      v_lo[j] = (int)(uint64_t)src.blob; v_hi[j] = (int)((uint64_t)src.blob >> 32);
    }
  }
  if constexpr (DISPATCH) {
    static_assert(sizeof(DispatchScratch) <= sizeof(sm.tok), "the token rows' place");
    if (dispatch) {
      DispatchScratch& sc = *reinterpret_cast<DispatchScratch*>(sm.tok[0]);
      const bool write = blockIdx.x == gridDim.x - 1;
      if (a.max_pairs <= kThreadsP) build_dispatch<NE, 1>(a, d, sc, sm.index, tid, write, v_m, v_row0);
      else if (a.max_pairs <= 2 * kThreadsP) build_dispatch<NE, 2>(a, d, sc, sm.index, tid, write, v_m, v_row0);
      else build_dispatch<NE, (kIndexMax + kThreadsP - 1) / kThreadsP>(a, d, sc, sm.index, tid, write, v_m, v_row0);
#pragma unroll
      for (int j = 0; j < NE; ++j)
        if ((v_lo[j] | v_hi[j]) == 0) v_m[j] = 0;              // an expert without weights
    }
  }
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    if (64 * j < a.n_routed) {
      int nb = token_blocks<WB>(v_m[j]);
      nb = wave_scan(nb);
      v_end[j] = routed_blocks + nb;
      routed_blocks = __builtin_amdgcn_readlane(v_end[j], 63);
    }
  }
  if (DISPATCH && a.n_routed && !dispatch)
    for (int i = tid; i < a.max_pairs; i += kThreadsP) sm.index[i] = (unsigned char)clampi(a.sorted_token[i], 0, a.T - 1);

  // ---- panels: every group's quads in panels of at most `per`, the smallest size that needs no more rounds of workgroups ----
  const int sh_blocks = n_sh ? token_blocks<WB>(a.T) : 0, grid = (int)gridDim.x;
  const int Qr = (MODE == kGateUp ? a.I : a.H) / OQ;
  auto shared_quads = [&](int g) -> int { return (MODE == kGateUp ? a.shared_I[g] : a.H) / OQ; };
  auto panels_with = [&](int per) -> int {
    int n = routed_blocks * quotient(Qr + per - 1, per);
    for (int g = 0; g < n_sh; ++g) n += sh_blocks * quotient(shared_quads(g) + per - 1, per);
    return n;
  };
  int per;
  {
    const int rounds = quotient(panels_with(kPanelQuads) + grid - 1, grid);
    const uint64_t fits = __ballot(panels_with(min(lane + 1, kPanelQuads)) <= rounds * grid);
    per = uniform((int)__builtin_ctzll(fits | 1ull << (kPanelQuads - 1)) + 1);
  }
  const int npr = quotient(Qr + per - 1, per);
  const int total = panels_with(per), total_sh = total - routed_blocks * npr;

  // this lane's 16 bytes of the four column groups of a unit of weights, and of four k-steps of a token row; column c of row r
  // sits at c ^ (r & 15), which keeps the reads free of bank conflicts
  unsigned a_rd[4], b_rd[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    a_rd[j] = ring + (unsigned)(c16 * 256 + (((4 * j + q) ^ c16) << 4));
    int low = WB == 2 ? 4 * j + q : (WB == 1 ? 8 * (j >> 1) + 2 * q + (j & 1) : 4 * q + j);
    if (MANY && WB != 2) low = 8 * (j >> 1) + (WB == 1 ? 4 : 2) * (j & 1) + (WB == 1 ? 2 : 4) * (q & 1) + (q >> 1);   // tile_order()
    b_rd[j] = tok + (unsigned)((c16 << U::kRowShift) + ((low ^ token_key<WB, MANY>(c16)) << 4));
  }

  constexpr int kLook = MANY ? kPanelsMany : 64;
#pragma unroll 1
  for (int first = blockIdx.x; first < total; first += kLook * grid) {
    // ---- panels first, first + grid, ..: one per lane ----
    const int np = min(kLook, quotient(total - first + grid - 1, grid));
    int p_g = 0, p_qa = 0, p_n = 0, p_r0 = 0, p_rows = 0, p_m = a.T, p_row0 = 0, p_lo = 0, p_hi = 0;
    {
      int item = first + min(lane, np - 1) * grid, nb = sh_blocks, panels = npr, Q = Qr;
      const bool sh = item < total_sh;
      int rest = sh ? item : 0x7fffffff;                 // counts down to this lane's group: an index of its own would be a load from memory per lane
      for (int g = 0; g < n_sh; ++g) {
        const int Qg = shared_quads(g), pg = quotient(Qg + per - 1, per), n = sh_blocks * pg;
        const uint64_t blob = (uint64_t)a.shared_w[MODE == kDown ? a.slab_shared[g] : g];
        const bool here = rest >= 0 && rest < n;
        p_g = here ? g : p_g; Q = here ? Qg : Q; panels = here ? pg : panels; item = here ? rest : item;
        p_lo = here ? (int)blob : p_lo; p_hi = here ? (int)(blob >> 32) : p_hi;
        rest -= n;
      }
      if (!sh) item -= total_sh;
      const int blk = sh ? 0 : quotient(item, npr);               // the expert that holds this block: the first whose blocks end behind it
      int e = 0, m = a.T, row0 = 0, lo = 0, hi = 0, end = 0;
#pragma unroll
      for (int j = 0; j < NE; ++j) {
        if (64 * j < a.n_routed) {
          int at = 0;
#pragma unroll
          for (int d = 32; d > 0; d >>= 1)
            if (__shfl(v_end[j], at + d - 1) <= blk) at += d;
          const bool here = j == 0 || e == 64 * j;       // every expert of the sets before ends in front of the block
          const int l = min(at, 63);
          const int nm = __shfl(v_m[j], l), nrow0 = __shfl(v_row0[j], l), nlo = __shfl(v_lo[j], l), nhi = __shfl(v_hi[j], l), nend = __shfl(v_end[j], l);
          if (here) { e = 64 * j + (__shfl(v_end[j], 63) <= blk ? 64 : at); m = nm; row0 = nrow0; lo = nlo; hi = nhi; end = nend; }
        }
      }
      if (!sh) {
        p_g = n_sh + min(e, a.n_routed - 1); p_m = m; p_row0 = row0; p_lo = lo; p_hi = hi;
        nb = token_blocks<WB>(m);
        item -= (end - nb) * npr;
      }
      // all token blocks of panel 8 b + i are 8 panels apart: at the same time on one XCD
      m = p_m;
      int tb = 0, panel = item;
      if (nb > 1) {
        const int b8 = quotient(item, 8 * nb), rem = item - b8 * 8 * nb, w8 = min(8, panels - 8 * b8);
        tb = quotient(rem, w8); panel = 8 * b8 + (rem - tb * w8);
      }
      const int block = nb > 1 ? quotient(m + nb - 1, nb) : m, base = quotient(Q, panels), more = Q - base * panels;
      p_qa = panel * base + min(panel, more);
      p_n = base + (panel < more ? 1 : 0);
      p_r0 = tb * block; p_rows = min(block, m - p_r0);
    }
    struct Panel { int qa, n, r0, rows; };
    auto get_panel = [&](int i, Group& G) -> Panel {
      Panel p;
      const int g = __builtin_amdgcn_readlane(p_g, i);
      p.qa = __builtin_amdgcn_readlane(p_qa, i); p.n = __builtin_amdgcn_readlane(p_n, i);
      p.r0 = __builtin_amdgcn_readlane(p_r0, i); p.rows = __builtin_amdgcn_readlane(p_rows, i);
      GroupSrc src;
      src.m = __builtin_amdgcn_readlane(p_m, i); src.row0 = __builtin_amdgcn_readlane(p_row0, i);
      src.blob = (const void*)(((uint64_t)(unsigned)__builtin_amdgcn_readlane(p_hi, i) << 32) | (unsigned)__builtin_amdgcn_readlane(p_lo, i));
      G = make_group<uint16_t, MODE, WB>(a, g, src);
      return p;
    };
    if (MANY && MODE == kGateUp) {
      for (int i = wave; i < np; i += kWaves) {
        const int r0 = __builtin_amdgcn_readlane(p_r0, i), rows = __builtin_amdgcn_readlane(p_rows, i);
        if (__builtin_amdgcn_readlane(p_g, i) >= n_sh && lane < rows)
          sm.rows[i][lane] = (unsigned short)clampi(a.sorted_token[__builtin_amdgcn_readlane(p_row0, i) + r0 + lane], 0, a.T - 1);
      }
    }
    // a panel's quads are dealt to the waves in contiguous parts that differ by one at most
    auto wave_part = [&](const Panel& p, int i, int& wa, int& wn) {
      const int w = (wave + 3 * i) & (kWaves - 1), more = p.n & (kWaves - 1);
      wn = p.n / kWaves + (w < more ? 1 : 0);
      wa = p.qa + (p.n / kWaves) * w + min(w, more);
    };
    // a wave's quads as one tile of up to four, or two even ones
    auto tiles_of = [](int wn) -> int { return RT > 1 && wn > 4 ? 2 : 1; };
    auto tile_start = [](int wn, int r) -> int { return r == 0 ? 0 : (RT > 1 && wn > 4 && r == 1 ? (wn + 1) / 2 : wn); };
    auto slice_rows = [](const Panel& p) -> int { return (p.rows + U::kRowsPerLoad - 1) & ~(U::kRowsPerLoad - 1); };
    // units per slice of token rows
    auto slice_units = [&](const Panel& p, int nu) -> int { return min(nu, quotient(U::kBuffer >> U::kRowShift, slice_rows(p))); };

    // ---- weight cursor ----
    int w_p = -1, w_u = 0, w_nu = 0, w_left = 0, w_n = 0, w_tile = 0, w_tiles = 1, slot = 0;
    unsigned addr[RT][4], s_addr[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      s_addr[r] = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) addr[r][i] = 0;
    }
    __amdgpu_buffer_rsrc_t rw = make_rsrc(a.x, 0), rsc = rw;
    auto next_weights = [&]() {
      w_u = 0; w_n = 0; w_nu = 1 << 30;                  // nothing is left: loads that only fill LDS with zeros
      int wa = 0;
      Group G;
      while (w_n == 0 && ++w_p < np) {
        const Panel p = get_panel(w_p, G);
        wave_part(p, w_p, wa, w_n);
      }
      if (w_n > 0) {
        const unsigned ld = WB ? (unsigned)G.ldw * WB : (unsigned)G.ldw / 2u;
        rw = make_rsrc(G.w0, G.wbytes);
        w_left = G.K; w_nu = (G.K + U::kK - 1) / U::kK;
        w_tiles = tiles_of(w_n);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const int n0 = (wa + tile_start(w_n, r)) * OQ, tn = tile_start(w_n, r + 1) - tile_start(w_n, r);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // quad i of the tile: gate/up: rows n, n + 1 of W_gate and the same of W_up behind it
            const int n = MODE == kGateUp ? n0 + 2 * i + (q & 1) + ((q & 2) ? G.N : 0) : n0 + 4 * i + q;
            addr[r][i] = ((unsigned)n * ld + (unsigned)((c16 ^ (4 * i + q)) << 4)) | (i < tn ? 0u : kOob);
          }
          if (WB == 0) {
            const unsigned lds = (unsigned)G.ldw >> 5;
            rsc = make_rsrc(G.scale, (unsigned)((MODE == kGateUp ? 2 : 1) * G.N - 1) * lds + ((unsigned)G.K >> 5));
            const int row = lane >> 2;                   // one dword = four blocks of one row
            const int n = MODE == kGateUp ? n0 + 2 * (row >> 2) + (row & 1) + ((row & 2) ? G.N : 0) : n0 + row;
            s_addr[r] = ((unsigned)n * lds + 4u * (lane & 3)) | ((row >> 2) < tn ? 0u : kOob);
          }
        }
      } else {
        w_tiles = 1;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          s_addr[r] = kOob;
#pragma unroll
          for (int i = 0; i < 4; ++i) addr[r][i] = kOob;
        }
      }
      w_tile = 0;
    };
    auto issue = [&]() {
      char* const st = sm.ring[wave] + slot * U::kBytes;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ok = (c16 ^ (4 * i + q)) * U::kPerColumn < w_left;            // k behind the row's end: out of range
        const unsigned at = RT > 1 && w_tile ? addr[RT - 1][i] : addr[0][i];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)(st + i * 1024), 16, (int)(at | (ok ? 0u : kOob)), 0, 0, kStreamOnce);
      }
      if (WB == 0) {
        const unsigned at = RT > 1 && w_tile ? s_addr[RT - 1] : s_addr[0];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsc, (lds_void*)(st + 4096), 4, (int)(at | ((lane & 3) * 128 < w_left ? 0u : kOob)), 0, 0, 0);
      }
      slot = slot + 1 == U::kStages ? 0 : slot + 1;
      if (RT > 1 && w_tile + 1 < w_tiles) w_tile = 1;
      else {
        w_tile = 0;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
          for (int i = 0; i < 4; ++i) addr[r][i] += 256u;              // kOob + a row stays out of range
          s_addr[r] += 16u;
        }
        w_left -= U::kK;
        if (++w_u == w_nu) next_weights();
      }
    };

    // ---- token cursor ----
    int t_p = -1, t_u = 0, t_nu = 0, t_us = 1, t_rows = 0, t_loads = 0, t_r0 = 0, t_K = 0, t_gather = 0, t_row0 = 0;
    unsigned t_ld = 0, t_bytes = 0;
    const void* t_base = a.x;
    auto next_tokens = [&]() {
      if (++t_p < np) {
        Group G;
        const Panel p = get_panel(t_p, G);
        t_base = G.b; t_bytes = G.bbytes;
        t_rows = p.rows; t_r0 = p.r0; t_K = G.K; t_ld = (unsigned)G.ldw * 2u; t_gather = G.gather; t_row0 = G.row0;
        t_nu = (G.K + U::kK - 1) / U::kK; t_us = slice_units(p, t_nu); t_loads = slice_rows(p) / U::kRowsPerLoad; t_u = 0;
      }
    };
    // the token rows of the next slice into buffer `buf`; returns the loads this wave issued
    auto issue_tokens = [&](int buf) -> int {
      int issued = 0;
      if (t_p < np) {
        const int n = min(t_us, t_nu - t_u) * t_loads;
        char* const dst = sm.tok[buf];
        const __amdgpu_buffer_rsrc_t rt = make_rsrc(t_base, t_bytes);
        int u = t_u, r = wave;
        for (int i = wave; i < n; i += kWaves, r += kWaves) {
          while (r >= t_loads) { r -= t_loads; ++u; }
          constexpr int cols = 16 * U::kParts;
          const int row = U::kRowsPerLoad * r + lane / cols, kk = u * U::kK + (((lane % cols) ^ token_key<WB, MANY>(row & 15)) << 3);
          int src = t_r0 + min(row, t_rows - 1);
          if (t_gather) src = MANY ? (int)lds_read_u16(s_index + (unsigned)(t_p * 64 + min(row, t_rows - 1)) * 2u) : (int)lds_read_u8(s_index + (unsigned)(t_row0 + src));
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rt, (lds_void*)(dst + i * 1024), 16,
              (int)(((unsigned)src * t_ld + (unsigned)kk * 2u) | (row < t_rows && kk < t_K ? 0u : kOob)), 0, 0, 0);
          ++issued;
        }
        t_u += t_us;
        if (t_u >= t_nu) next_tokens();
      }
      return issued;
    };

    next_weights();
#pragma unroll 1
    for (int i = 0; i < U::kStages; ++i) issue();
    slot = 0;
    lds_barrier();                             // the index table is complete
    next_tokens();
    issue_tokens(0);

    int buf = 1, since = 0;                    // units issued behind the latest token rows
#pragma unroll 1
    for (int ip = 0; ip < np; ++ip) {
      Group G;
      const Panel p = get_panel(ip, G);
      int wa, wn;
      wave_part(p, ip, wa, wn);
      const int nt = (p.rows + 15) >> 4, nu = (G.K + U::kK - 1) / U::kK, us = slice_units(p, nu);
      const unsigned unit_bytes = (unsigned)slice_rows(p) << U::kRowShift;
      constexpr int kSums = MANY ? 1 : 2;      // per token tile; two: even and odd groups of four columns
      f32x4 acc[RT][U::kTiles][kSums];
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < U::kTiles; ++t) acc[r][t][0] = acc[r][t][kSums - 1] = f32x4{0, 0, 0, 0};
      const bool both = RT > 1 && wn > 4;
#pragma unroll 1
      for (int u0 = 0; u0 < nu; u0 += us) {
        if (since <= U::kStages) wait_units<U::kLoads>(since);          // this wave's part of the slice has landed
        lds_barrier();                                                  // ... and every other wave's; the other buffer is free
        const int extra = issue_tokens(buf);
        since = 0;
        buf ^= 1;
        const int u1 = wn > 0 ? min(nu, u0 + us) : 0;
        unsigned ab[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) ab[j] = b_rd[j] + (unsigned)(buf * U::kBuffer);
#pragma unroll 1
        for (int u = u0; u < u1; ++u) {
          i32x4 w[RT][4], sc4[RT];
          auto take_unit = [&](int r) {
            // the units issued in front of the slice's token rows may have those behind them as well
            if (since < U::kStages) wait_vm<(U::kStages - 1) * U::kLoads>(extra); else MM_WAIT_VM((U::kStages - 1) * U::kLoads);
            const unsigned so = (unsigned)(slot * U::kBytes);
            const unsigned aw[4] = {a_rd[0] + so, a_rd[1] + so, a_rd[2] + so, a_rd[3] + so};
            if constexpr (WB == 0) read_weights(w[r], sc4[r], aw, ring + so + 4096u + (unsigned)c16 * 16u);
            else read_weights(w[r], aw);
            if constexpr (MANY && WB != 2) {
#pragma unroll
              for (int j = 0; j < 4; ++j) tile_order<WB>(w[r][j]);
            }
            issue();
            ++since;
          };
          take_unit(0);
          if constexpr (RT > 1) if (both) take_unit(1);
          // weights of the k-steps of a part of unit r
          auto widen = [&](int r, int part, bf16x8 (&f)[4]) {
            float s0 = WB == 0 ? e8m0_to_f32(((unsigned)sc4[r][part] >> (8 * q)) & 0xffu) : 0.f, s1 = s0;
            if (WB == 0 && MANY) {                       // behind tile_order(): of the blocks q & 1 and 2 + (q & 1)
              const auto both_halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(s0), __float_as_uint(s0), false, false);
              s0 = __uint_as_float(both_halves[0]); s1 = __uint_as_float(both_halves[1]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if constexpr (WB == 2) f[j] = __builtin_bit_cast(bf16x8, w[r][j]);
              else if constexpr (WB == 1) f[j] = widen_e4m3(w[r][2 * part + (j >> 1)][2 * (j & 1)], w[r][2 * part + (j >> 1)][2 * (j & 1) + 1]);
              else f[j] = widen_mx4(w[r][part][j], j < 2 ? s0 : s1);
            }
          };
          auto multiply = [&](int r, int t, int part, const bf16x8 (&f)[4], const i32x4 (&b)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int odd = MANY ? 0 : (WB == 2 ? j & 1 : (WB == 1 ? j >> 1 : part & 1));
              acc[r][t][odd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[j], __builtin_bit_cast(bf16x8, b[j]), acc[r][t][odd], 0, 0, 0);
            }
          };
          if constexpr (RT == 1 || WB != 0) {
            bf16x8 f[RT][U::kParts][4];
#pragma unroll
            for (int part = 0; part < U::kParts; ++part) widen(0, part, f[0][part]);
            if constexpr (RT > 1) {
              if (both) {
#pragma unroll
                for (int part = 0; part < U::kParts; ++part) widen(1, part, f[1][part]);
              }
            }
            auto token_tile = [&](auto tc) {
              constexpr int t = decltype(tc)::value;
              if constexpr (t < U::kTiles) {
                if (t < nt) {
                  constexpr unsigned far = (unsigned)t << (U::kRowShift + 4);
                  const unsigned at[4] = {ab[0] + far, ab[1] + far, ab[2] + far, ab[3] + far};
                  i32x4 b[U::kParts][4];
                  read_tokens(b, at);
#pragma unroll
                  for (int part = 0; part < U::kParts; ++part) multiply(0, t, part, f[0][part], b[part]);
                  if constexpr (RT > 1) {
                    if (both) {
#pragma unroll
                      for (int part = 0; part < U::kParts; ++part) multiply(1, t, part, f[1][part], b[part]);
                    }
                  }
                }
              }
            };
            token_tile(std::integral_constant<int, 0>{});
            token_tile(std::integral_constant<int, 1>{});
            token_tile(std::integral_constant<int, 2>{});
            token_tile(std::integral_constant<int, 3>{});
          } else {
#pragma unroll
            for (int part = 0; part < U::kParts; ++part) {
              bf16x8 f[RT][4];
              widen(0, part, f[0]);
              if (both) widen(1, part, f[RT - 1]);
#pragma unroll
              for (int t = 0; t < U::kTiles; ++t) {
                if (t < nt) {
                  const unsigned far = ((unsigned)t << (U::kRowShift + 4)) + 256u * part;
                  const unsigned at[4] = {ab[0] + far, ab[1] + far, ab[2] + far, ab[3] + far};
                  i32x4 b[1][4];
                  read_tokens(b, at);
                  multiply(0, t, part, f[0], b[0]);
                  if (both) multiply(1, t, part, f[RT - 1], b[0]);
                }
              }
            }
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) ab[j] += unit_bytes;
        }
      }
      // ---- epilogue ----
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int tn = tile_start(wn, r + 1) - tile_start(wn, r), n0 = (wa + tile_start(wn, r)) * OQ;
        if (tn <= 0) continue;
        float sc[4] = {1.f, 1.f, 1.f, 1.f};
        if (WB == 1) {
          typedef const __attribute__((address_space(4))) float* cfloat;
          cfloat s0 = (cfloat)(uintptr_t)G.scale;
          auto pick = [&](int from, int step, int limit) -> float {     // scale from + q * step
            const float v0 = s0[min(from, limit)], v1 = s0[min(from + step, limit)], v2 = s0[min(from + 2 * step, limit)], v3 = s0[min(from + 3 * step, limit)];
            return q == 0 ? v0 : (q == 1 ? v1 : (q == 2 ? v2 : v3));
          };
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (MODE == kGateUp) sc[v] = pick((v >= 2 ? G.N : 0) + n0 + (v & 1), 2, 2 * G.N - 1);
            else sc[v] = pick(n0 + v, 4, G.N - 1);
          }
        }
#pragma unroll
        for (int t = 0; t < U::kTiles; ++t) {
          const int row = 16 * t + c16;
          if (row < p.rows && q < tn) {
            float val[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              val[v] = MANY ? acc[r][t][0][v] : acc[r][t][0][v] + acc[r][t][kSums - 1][v];
              if (WB == 1) val[v] *= sc[v];
            }
            const size_t ro = (size_t)(p.r0 + row);
            if (MODE == kGateUp) {
              typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
              float h[2];
#pragma unroll
              for (int v = 0; v < 2; ++v) h[v] = val[v] / (1.f + __expf(-val[v])) * val[2 + v];
              *reinterpret_cast<bf16x2*>(static_cast<uint16_t*>(G.out) + ro * G.N + n0 + 2 * q) = bf16x2{(__bf16)h[0], (__bf16)h[1]};
            } else {
              *reinterpret_cast<f32x4*>(static_cast<float*>(G.out) + ro * a.H + n0 + 4 * q) = f32x4{val[0], val[1], val[2], val[3]};
            }
          }
        }
      }
    }
    MM_WAIT_VM(0);
    lds_barrier();                             // before the next panels' token rows
  }
}

template <int MODE, int WB, bool MANY, int RT>
int launch_panels_typed(const StreamArgs& a, const StepDispatch& d, hipStream_t s) {
  if (a.T > kPanelsMaxT) return fail(MOE_E_UNSUPPORTED, "stream_panel_kernel: T=%d", a.T);
  const long items = item_upper_bound((StreamMode)MODE, a, 32);
  if (items <= 0) return MOE_OK;
  long grid = device_cu_count();                          // 158 KB of LDS: one workgroup per CU
  if (grid > items) grid = items;
  hipLaunchKernelGGL((stream_panel_kernel<MODE, WB, MANY, RT>), dim3((unsigned)grid), dim3(kThreadsP), 0, s, a, d);
  return hip_fail(hipGetLastError(), "stream_panel_kernel launch");
}
template <int MODE, int WB>
int launch_panels(const StreamArgs& a, const StepDispatch& d, hipStream_t s) {
  const bool many = a.T >= kTiledMinT;
  if constexpr (WB != 2)                       // bf16 weights: never faster (ffn_route)
    if (a.wide_panels) return many ? launch_panels_typed<MODE, WB, true, 2>(a, d, s) : launch_panels_typed<MODE, WB, false, 2>(a, d, s);
  return many ? launch_panels_typed<MODE, WB, true, 1>(a, d, s) : launch_panels_typed<MODE, WB, false, 1>(a, d, s);
}
template <int MODE>
int launch_panels_of(int weight_format, const StreamArgs& a, const StepDispatch& d, hipStream_t s) {
  if (weight_format == 2) return launch_panels<MODE, 2>(a, d, s);
  if (weight_format == 1) return launch_panels<MODE, 1>(a, d, s);
  return launch_panels<MODE, 0>(a, d, s);
}

}  // namespace

int launch_stream_panels(StreamMode mode, int weight_format, const StreamArgs& a, hipStream_t s) {
  const StepDispatch none = {};
  return mode == kGateUp ? launch_panels_of<kGateUp>(weight_format, a, none, s) : launch_panels_of<kDown>(weight_format, a, none, s);
}

int launch_dispatch_gate_up(int weight_format, const StreamArgs& a, const StepDispatch& d, hipStream_t s) {
  if (a.T <= 0 || a.T >= kTiledMinT || !d.on || a.n_routed != a.E || a.max_pairs != a.T * d.k_big || d.k_big > MOE_MAX_TOPK)
    return fail(MOE_E_UNSUPPORTED, "dispatch beside gate/up: T=%d", a.T);
  return launch_panels_of<kGateUp>(weight_format, a, d, s);
}

}  // namespace mm
