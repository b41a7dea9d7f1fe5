// Grouped expert GEMM for prefill steps with large groups: bf16 MFMA on 256 x 256 tiles (same
// operation, groups and operand roles as ffn_tiled.hip).
//
// What bounds it: a 128 x 256 tile moves 36 KB through LDS (24 KB of fragment reads, 12 KB of loads
// landing) per 256 cycles of MFMAs, more than the 128 bytes a cycle that LDS delivers.  A 256 x 256
// tile on four waves of 128 x 128 needs 48 KB per 512 cycles.  Its 256 accumulators, the fragments of
// two k-steps (64) and the tile list take 468 of the 512 registers that a wave can have, so there is
// one wave per SIMD, no room for waves that only load, and nothing that would hide a stall: every
// k-step is one asm block in which the MFMAs, the fragment reads of the next k-step and the loads
// into LDS alternate, and which ends with the wait for its own reads.  (About 100 scalars live in lanes of
// vector registers; they are fetched where a tile begins and ends, not between the blocks.)
//
//   * 4 waves, one workgroup per CU.  Tiles of more than 128 tokens: waves in a 2 x 2 grid, each up to 4
//     blocks of 32 tokens x 4 of 32 weight rows.  Smaller tiles: the waves split the weight rows
//     four ways and share the tokens, so that no SIMD idles.  For gate/up the weight rows are 128 rows
//     of W_gate and the same 128 of W_up, and a wave holds gate and up of the same outputs.
//   * LDS (all 160 KB): two slots of 64 k for the token rows, three for the weight rows, which come from
//     further away.  Period kt (behind the barrier that says that chunk kt has landed and chunk kt - 1
//     has been read) loads token chunk kt + 1, then weight chunk kt + 2, spread evenly over four
//     k-steps (bunching them behind the barrier costs 5 %); the newest weight chunk stays in flight
//     across the barrier.  Slots, row swizzle and out-of-range handling as in ffn_tiled.hip.
//   * The chunks of all tiles of a workgroup form one stream: load cursors run ahead into the next tile,
//     whose rows were looked up one tile earlier, and the epilogue's stores drain under its MFMAs.
//   * Groups are split into token tiles of nearly equal height: the tiles of a weight panel run side
//     by side on one XCD, and tiles of equal length keep step, so that the panel is fetched once for all
//     of them.  (8 experts of 14336, 4096 tokens, gate+up, on one card: whole tiles first and the remainders
//     last 1152 us, remainder next to the whole tiles 1057, even heights 1045; ffn_tiled.hip 1137.)
//
// Measured, ffn_tiled.hip -> this kernel, us (gate+up / down), in turn on another card: 8 experts of 14336, 4096
// tokens 1160 / 638 -> 1079 / 589, 2048 tokens 669 / 416 -> 630 / 314; 60 experts of 1408 + 5632 shared, 4096
// tokens 389 / 261 -> 339 / 206; 64 of 1408 + 2 shared, 3300 tokens 279 / 175 -> 254 / 166.  The MFMAs alone
// (no loads, no fragment reads) of the first take 747 us.
#include <atomic>
#include <type_traits>

#include "internal.h"
#include "groups.h"
#include "dispatch_device.h"
#include "wide_layout.h"

namespace mm {
namespace {

using namespace wide;

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef uint16_t S;

constexpr int kThreadsW = 256;
constexpr int kBuckets = 7;             // groups by their token rows, most first
constexpr int kGrpC = (kMaxGroups + 63) / 64;
constexpr int kOutCols(int mode) { return mode == kGateUp ? 128 : 256; }
static_assert(kOutCols(kGateUp) == kTiledPanel && kSlotRows == kWideRows, "tiles of the dispatch rules");
constexpr int kA = 8, kB = 8;           // loads of a wave per token / weight chunk
constexpr int kLoads = (kA + kB) / 4;   // ... per k-step
constexpr int kLdsBytes = (SA + SB) * kSlotB;
constexpr int VM = kB + (SA - 2) * (kA + kB);   // loads in flight behind the awaited chunk
static_assert(SB > SA && kLdsBytes <= 163840, "ring");

template <typename T> __device__ __forceinline__ T sload(const void* p) {
  return *(const __attribute__((address_space(4))) T*)(uint64_t)p;
}

// ---- one k-step: MFMAs on the current fragments, reads of the next ones, loads into LDS.  c: accumulators,
// a / b: fragments of the k-step, na / nb: of the next, at the LDS addresses pa / pb ----
struct Loads { i32x4 rs[4]; unsigned vo[4]; int so[4]; int md[4]; };

#define MF(i, j) "v_mfma_f32_32x32x16_bf16 %[c" #i #j "], %[a" #i "], %[b" #j "], %[c" #i #j "]\n\t"
#define RA(i) "ds_read_b128 %[na" #i "], %[pa] offset:%[oa" #i "]\n\t"
#define RB(j) "ds_read_b128 %[nb" #j "], %[pb] offset:%[ob" #j "]\n\t"
#define RQ(j) "ds_read_b128 %[nb" #j "], %[q" #j "] offset:%[ob" #j "]\n\t"
#define LD(l) "s_mov_b32 m0, %[md" #l "]\n\ts_nop 0\n\tbuffer_load_dwordx4 %[vo" #l "], %[rs" #l "], %[so" #l "] offen lds\n\t"
#define BAR "s_waitcnt vmcnt(%[vm])\n\ts_barrier\n\t"
// the compiler does not see what the block holds: wait states between its vector instructions and the
// matrix instructions (2), and between its scalar results and the loads that use them (5)
#define START "s_nop 4\n\t"
#define END "s_waitcnt lgkmcnt(0)"
#define C1(i, j) [c##i##j] "+a"(c[i][j])
#define C4(i) C1(i, 0), C1(i, 1), C1(i, 2), C1(i, 3)
#define NA(i) [na##i] "=&v"(na[i])
#define NB_(j) [nb##j] "=&v"(nb[j])
#define IA(i) [a##i] "v"(fa[i])
#define IB(j) [b##j] "v"(fb[j])
#define LOADS4 [rs0] "s"(L.rs[0]), [rs1] "s"(L.rs[1]), [rs2] "s"(L.rs[2]), [rs3] "s"(L.rs[3]), \
  [vo0] "v"(L.vo[0]), [vo1] "v"(L.vo[1]), [vo2] "v"(L.vo[2]), [vo3] "v"(L.vo[3]), \
  [so0] "s"(L.so[0]), [so1] "s"(L.so[1]), [so2] "s"(L.so[2]), [so3] "s"(L.so[3]), \
  [md0] "s"(L.md[0]), [md1] "s"(L.md[1]), [md2] "s"(L.md[2]), [md3] "s"(L.md[3])
#define OFFS [oa0] "n"(0), [oa1] "n"(kBlock * kRowB), [oa2] "n"(2 * kBlock * kRowB), [oa3] "n"(3 * kBlock * kRowB)
#define OB(j) [ob##j] "n"(b_frag_row(GU, j) * kRowB)
#define OFFB OB(0), OB(1), OB(2), OB(3)
// addresses of the weight fragments of the next tile's first k-step: pq for those that a narrow tile has no use for
#define QB(j) [q##j] "v"(j == 0 || j == second_frag(GU) ? pb : pq)
#define NEXT QB(0), QB(1), QB(2), QB(3), [vm] "n"(VM)
#define NALL NA(0), NA(1), NA(2), NA(3), NB_(0), NB_(1), NB_(2), NB_(3)
#define IN4 IA(0), IA(1), IA(2), IA(3), IB(0), IB(1), IB(2), IB(3)
#define REST [pa] "v"(pa), [pb] "v"(pb), LOADS4, OFFS, OFFB
// the reads behind the barrier fetch all eight fragments, whatever shape the next tile has (b_row_of)
#define RDALL RQ(0) RQ(1) RQ(2) RQ(3) RA(0) RA(1) RA(2) RA(3)

#define C2J(i, J) C1(i, 0), C1(i, J)
#define NARROW_STEPS(J)                                                                                                  \
  if constexpr (NB == 4) {                                                                                               \
    if constexpr (!BARRIER)                                                                                              \
      asm volatile(START MF(0,0) RB(0) RB(J) MF(0,J) RA(0) LD(0) MF(1,0) RA(1) RA(2) MF(1,J) RA(3) LD(1) MF(2,0) MF(2,J) LD(2) MF(3,0) LD(3) MF(3,J) END \
                   : C2J(0, J), C2J(1, J), C2J(2, J), C2J(3, J), NA(0), NA(1), NA(2), NA(3), NB_(0), NB_(J)                \
                   : IA(0), IA(1), IA(2), IA(3), IB(0), IB(J), REST : "memory");                                          \
    else                                                                                                                 \
      asm volatile(START MF(0,0) MF(0,J) BAR MF(1,0) RDALL MF(1,J) LD(0) MF(2,0) LD(1) MF(2,J) LD(2) MF(3,0) LD(3) MF(3,J) END \
                   : C2J(0, J), C2J(1, J), C2J(2, J), C2J(3, J), NALL                                                     \
                   : IA(0), IA(1), IA(2), IA(3), IB(0), IB(J), REST, NEXT : "memory");                            \
  } else if constexpr (NB == 3) {                                                                                        \
    if constexpr (!BARRIER)                                                                                              \
      asm volatile(START MF(0,0) RB(0) RB(J) MF(0,J) RA(0) LD(0) MF(1,0) RA(1) RA(2) MF(1,J) LD(1) MF(2,0) LD(2) LD(3) MF(2,J) END \
                   : C2J(0, J), C2J(1, J), C2J(2, J), NA(0), NA(1), NA(2), NB_(0), NB_(J)                                  \
                   : IA(0), IA(1), IA(2), IB(0), IB(J), REST : "memory");                                                 \
    else                                                                                                                 \
      asm volatile(START MF(0,0) MF(0,J) BAR MF(1,0) RDALL MF(1,J) LD(0) LD(1) MF(2,0) LD(2) LD(3) MF(2,J) END           \
                   : C2J(0, J), C2J(1, J), C2J(2, J), NALL                                                                \
                   : IA(0), IA(1), IA(2), IB(0), IB(J), REST, NEXT : "memory");                                   \
  } else if constexpr (NB == 2) {                                                                                        \
    if constexpr (!BARRIER)                                                                                              \
      asm volatile(START MF(0,0) RB(0) RB(J) MF(0,J) RA(0) RA(1) LD(0) MF(1,0) LD(1) LD(2) MF(1,J) LD(3) END             \
                   : C2J(0, J), C2J(1, J), NA(0), NA(1), NB_(0), NB_(J)                                                   \
                   : IA(0), IA(1), IB(0), IB(J), REST : "memory");                                                        \
    else                                                                                                                 \
      asm volatile(START MF(0,0) MF(0,J) BAR MF(1,0) RDALL MF(1,J) LD(0) LD(1) LD(2) LD(3) END                           \
                   : C2J(0, J), C2J(1, J), NALL                                                                           \
                   : IA(0), IA(1), IB(0), IB(J), REST, NEXT : "memory");                                          \
  } else {                                                                                                               \
    if constexpr (!BARRIER)                                                                                              \
      asm volatile(START MF(0,0) RB(0) RB(J) RA(0) MF(0,J) LD(0) LD(1) LD(2) LD(3) END                                   \
                   : C2J(0, J), NA(0), NB_(0), NB_(J)                                                                     \
                   : IA(0), IB(0), IB(J), REST : "memory");                                                               \
    else                                                                                                                 \
      asm volatile(START MF(0,0) MF(0,J) BAR RDALL LD(0) LD(1) LD(2) LD(3) END                                           \
                   : C2J(0, J), NALL                                                                                      \
                   : IA(0), IB(0), IB(J), REST, NEXT : "memory");                                                 \
  }

// GU: gate/up.  Tiles of more than 128 tokens: waves in a 2 x 2 grid, NB x 4 matrix tiles each.  Narrower
// ones: the waves split the weight rows four ways, NB x 2 tiles each (weight fragments 0 and
// second_frag).  pq: as pb, from the row b_row_of of the other two fragments on.
template <bool TALL, int NB, bool GU, bool BARRIER>
__device__ __forceinline__ void kstep(f32x16 (&c)[4][4], const bf16x8 (&fa)[4], const bf16x8 (&fb)[4], bf16x8 (&na)[4],
                                      bf16x8 (&nb)[4], unsigned pa, unsigned pb, unsigned pq, const Loads& L) {
  if constexpr (TALL && NB == 4) {
    if constexpr (!BARRIER)
      asm volatile(START MF(0,0) RB(0) MF(0,1) RB(1) MF(0,2) RB(2) LD(0) MF(0,3) RB(3) MF(1,0) RA(0) MF(1,1) RA(1) LD(1) MF(1,2) RA(2) MF(1,3) RA(3)
                   MF(2,0) LD(2) MF(2,1) MF(2,2) MF(2,3) MF(3,0) LD(3) MF(3,1) MF(3,2) MF(3,3) END
                   : C4(0), C4(1), C4(2), C4(3), NALL : IN4, REST : "memory");
    else
      asm volatile(START MF(0,0) MF(0,1) MF(0,2) MF(0,3) BAR MF(1,0) RQ(0) RQ(1) MF(1,1) RQ(2) RQ(3) MF(1,2) RA(0) RA(1) MF(1,3) RA(2) RA(3)
                   MF(2,0) LD(0) MF(2,1) MF(2,2) LD(1) MF(2,3) MF(3,0) LD(2) MF(3,1) MF(3,2) LD(3) MF(3,3) END
                   : C4(0), C4(1), C4(2), C4(3), NALL : IN4, REST, NEXT : "memory");
  } else if constexpr (TALL && NB == 3) {
    if constexpr (!BARRIER)
      asm volatile(START MF(0,0) RB(0) MF(0,1) RB(1) MF(0,2) RB(2) LD(0) MF(0,3) RB(3) MF(1,0) RA(0) MF(1,1) RA(1) LD(1) MF(1,2) RA(2) MF(1,3)
                   MF(2,0) LD(2) MF(2,1) MF(2,2) LD(3) MF(2,3) END
                   : C4(0), C4(1), C4(2), NA(0), NA(1), NA(2), NB_(0), NB_(1), NB_(2), NB_(3)
                   : IA(0), IA(1), IA(2), IB(0), IB(1), IB(2), IB(3), REST : "memory");
    else
      asm volatile(START MF(0,0) MF(0,1) MF(0,2) MF(0,3) BAR MF(1,0) RQ(0) RQ(1) MF(1,1) RQ(2) RQ(3) MF(1,2) RA(0) RA(1) MF(1,3) RA(2) RA(3)
                   MF(2,0) LD(0) MF(2,1) LD(1) MF(2,2) LD(2) MF(2,3) LD(3) END
                   : C4(0), C4(1), C4(2), NALL : IA(0), IA(1), IA(2), IB(0), IB(1), IB(2), IB(3), REST, NEXT : "memory");
  } else if constexpr (second_frag(GU) == 2) {
    NARROW_STEPS(2)
  } else {
    NARROW_STEPS(1)
  }
}
#undef NARROW_STEPS

// first fragments: nothing to multiply yet
template <bool GU>
__device__ __forceinline__ void first_frags(bf16x8 (&na)[4], bf16x8 (&nb)[4], unsigned pa, unsigned pb, unsigned pq) {
  asm volatile(BAR RDALL END : NALL : [pa] "v"(pa), OFFS, OFFB, NEXT : "memory");
}
__device__ __forceinline__ void load_one(i32x4 rs, unsigned vo, int so, int md) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 4\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" :: "v"(vo), "s"(rs), "s"(so), "s"(md) : "memory");
}

__device__ __forceinline__ i32x4 rsrc4(const void* p, unsigned bytes) {
  const uint64_t v = (uint64_t)p;
  return i32x4{uniform((int)(unsigned)v), uniform((int)(unsigned)(v >> 32)), uniform((int)bytes), 0x00020000};
}

// one accumulator out of the matrix registers: read where it is used, so that no more than the
// few values being stored sit in ordinary registers
__device__ __forceinline__ float acc_read(const f32x16& c, int v) {
  float x;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(c[v]));
  return x;
}

struct Tile {
  int valid, tall, nb;                // tall: 2 x 2 waves; nb: 32-row blocks per wave
  int m0, m, n0, N, K, row0, gather;
  unsigned ldb;                       // bytes between rows of both operands
  const void* w0; const void* b; void* out;
  unsigned wbytes, bbytes;
};

// rows of a group's token tiles: as even as 32-row blocks allow, so that the tiles of a panel, which
// share its weights through L2, keep step
__device__ __forceinline__ int tile_height(int m, int tiles) { return (((m + 31) >> 5) + tiles - 1) / tiles * 32; }
// relative time of a tile: in proportion to the rows while the matrix cores set the pace, flat where
// the weights do
__device__ __forceinline__ int tile_cost(int rows) {
  const int b = (rows + 31) >> 5;
  return b > 6 ? 32 : (b > 4 ? 26 : 6 + 4 * b);
}

template <int MODE>
__global__ __launch_bounds__(kThreadsW) __attribute__((amdgpu_waves_per_eu(1, 1))) void wide_kernel(const StreamArgs args) {
  // read in place: a copy would live in scratch, where the arrays' dynamic indexes lose their uniformity
  const StreamArgs& a = *(const StreamArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __attribute__((aligned(1024))) char s_ring[];
  constexpr int kOut = kOutCols(MODE);
  fetch_arguments<sizeof(StreamArgs)>();
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const unsigned lds0 = (unsigned)(size_t)s_ring;
  const int n_sh = MODE == kDown ? a.n_slabs : a.n_shared;
  const int n_groups = a.n_routed + n_sh;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, nslots = gridDim.x >> 3;
  const bool by_rows = uniform(a.by_rows) != 0;
  const int workers = by_rows ? nslots : 8 * nslots;        // workgroups that share a tile list

  // Two orders of the tiles.  By rows: panel n (kOut output columns) of group g belongs to XCD (n + g) % 8 and
  // each XCD has a list of its own; otherwise one list by groups, cut into 8 contiguous ranges.  Tile height: 256 rows use
  // LDS best, but a few large tiles can leave the last round half empty (8 experts of 614 rows,
  // down: 48 tiles of 224 rows on 32 CUs take 632 us, 64 of 160 rows 570); the height with the
  // smallest estimate of the list's time is taken.
  int gm[kGrpC], gp[kGrpC];
  int R = 256;
  {
    int best = 0x7fffffff;
#pragma unroll
    for (int c = 0; c < kGrpC; ++c) {
      gm[c] = gp[c] = 0;
      if (c * 64 < n_groups) {
        const int g = c * 64 + lane;
        if (g < n_groups) {
          const GroupSrc s = load_group_src<MODE>(a, g);
          const int N = MODE == kDown ? a.H : (g < n_sh ? a.shared_I[g] : a.I);
          const int nt = (N + kOut - 1) / kOut, first = (xcd - g) & 7;
          gm[c] = s.m;
          gp[c] = !by_rows ? nt : (nt > first ? (nt - first + 7) >> 3 : 0);
        }
      }
    }
    for (int r = 256; r >= 128; r -= 64) {
      int sum = 0, top = 0, n_top = 0;
#pragma unroll
      for (int c = 0; c < kGrpC; ++c)
        if (c * 64 < n_groups && gm[c] > 0 && gp[c] > 0) {
          const int tiles = (gm[c] + r - 1) / r, cost = tile_cost(tile_height(gm[c], tiles));
          sum += tiles * gp[c] * cost;
          top = max(top, cost);
        }
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) { sum += __shfl_xor(sum, d); top = max(top, __shfl_xor(top, d)); }
#pragma unroll
      for (int c = 0; c < kGrpC; ++c)
        if (c * 64 < n_groups && gm[c] > 0 && gp[c] > 0) {
          const int tiles = (gm[c] + r - 1) / r;
          if (tile_cost(tile_height(gm[c], tiles)) == top) n_top += tiles * gp[c];
        }
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) n_top += __shfl_xor(n_top, d);
      const int est = uniform(max(sum / workers, (n_top + workers - 1) / workers * top));
      if (est < best) { best = est; R = r; }
    }
  }
  // Tile list: inclusive prefix over the groups c * 64 + lane, by rows the groups with many rows first;
  // the token tiles of a panel are adjacent, so that they run side by side.
  int pref[kBuckets][kGrpC], tot[kBuckets];
#pragma unroll
  for (int k = 0; k < kBuckets; ++k) tot[k] = 0;
#pragma unroll
  for (int c = 0; c < kGrpC; ++c) {
    const int v = (gm[c] + R - 1) / R * gp[c], m = gm[c];
    const int bk = m > 256 || !by_rows ? 0 : (m > 192 ? 1 : (m > 128 ? 2 : 6 - ((m - 1) >> 5)));
#pragma unroll
    for (int k = 0; k < kBuckets; ++k) {
      pref[k][c] = 0x7fffffff;
      if (c * 64 < n_groups) {
        pref[k][c] = wave_scan(m > 0 && bk == k ? v : 0) + tot[k];
        tot[k] = uniform(__shfl(pref[k][c], 63));
      }
    }
  }
  int total = 0;
#pragma unroll
  for (int k = 0; k < kBuckets; ++k) total += tot[k];
  // first tile and number of tiles of this XCD, then the tiles of this workgroup
  const int first_tile = by_rows ? 0 : (int)((long)total * xcd / 8);
  const int xcd_tiles = by_rows ? total : (int)((long)total * (xcd + 1) / 8) - first_tile;
  const int mine = xcd_tiles > slot ? (xcd_tiles - slot - 1) / nslots + 1 : 0;

  // ---- this workgroup's i-th tile.  Half of the workgroups take theirs from the back, so that tiles bound
  // by their weights and tiles bound by the matrix cores run at the same time (64 experts of
  // 1024, 2048 skewed tokens, gate+up: 163 -> 153 us) ----
  auto tile_at = [&](int i) -> Tile {
    Tile T = {};
    T.valid = i < mine;
    if (!T.valid) return T;
    if (by_rows && 2 * slot >= nslots) i = mine - 1 - i;
    int v = first_tile + i * nslots + slot;
    int bk = -1, g = 0, ex = 0;
#pragma unroll
    for (int k = 0; k < kBuckets; ++k) {
      if (bk < 0) {
        if (v < tot[k]) {
          bk = k;
#pragma unroll
          for (int c = 0; c < kGrpC; ++c) if (c * 64 < n_groups) g += __popcll(__ballot(pref[k][c] <= v));
#pragma unroll
          for (int c = 0; c < kGrpC; ++c) if (g > 0 && ((g - 1) >> 6) == c) ex = __builtin_amdgcn_readlane(pref[k][c], (g - 1) & 63);
        } else {
          v -= tot[k];
        }
      }
    }
    g = uniform(g);
    GroupSrc src;
    src.row0 = 0;
    if (g < n_sh) {
      src.m = a.T;
      src.blob = a.shared_w[MODE == kDown ? a.slab_shared[g] : g];
    } else {
      const int e = g - n_sh;
      const int b0 = clampi(sload<int>(a.offsets + e), 0, a.max_pairs);
      const int b1 = clampi(sload<int>(a.offsets + e + 1), b0, a.max_pairs);
      src.blob = sload<const void*>(a.expert_w + e);
      src.m = min(b1 - b0, a.T);
      src.row0 = b0;
    }
    src.m = uniform(src.m); src.row0 = uniform(src.row0); src.blob = uniform(src.blob);
    const Group G = make_group<S, MODE, 2>(a, g, src);
    const int local = uniform(v - ex), per = uniform((int)((unsigned)(G.m + R - 1) / (unsigned)R));
    const int panel = uniform((int)((unsigned)local / (unsigned)per));
    const int rt = tile_height(G.m, per);
    T.m0 = (local - panel * per) * rt;
    const int rows = min(G.m - T.m0, rt);
    T.m = T.m0 + rows;
    T.tall = rows > 128;
    T.nb = rows > 192 ? 4 : (rows > 128 ? 3 : (rows + 31) >> 5);
    T.n0 = (by_rows ? ((xcd - g) & 7) + 8 * panel : panel) * kOut;
    T.N = G.N; T.K = G.K; T.row0 = G.row0; T.gather = G.gather;
    T.ldb = (unsigned)G.ldw * 2u;
    T.w0 = G.w0; T.b = G.b; T.out = G.out; T.wbytes = G.wbytes; T.bbytes = G.bbytes;
    return T;
  };

  // this lane's row number of the tile's token rows (64 rows per wave)
  auto row_ids = [&](const Tile& T) -> int {
    const int rl = wave * 64 + lane, r = T.m0 + rl;
    const bool val = T.valid && r < T.m;
    int id = val ? r : -1;
    if (T.valid && T.gather) id = val ? clampi(a.sorted_token[T.row0 + r], 0, a.T - 1) : -1;
    return id;
  };
  int ord = 0;
  Tile cur = tile_at(ord++);
  if (!cur.valid) return;
  const int h = lane >> 5;
  const unsigned fkey = (unsigned)((lane & 31) >> 1) & 7u;
  constexpr bool GU = MODE == kGateUp;

  Tile nx = tile_at(ord++);
  int ids_nx = row_ids(nx);

  // ---- load cursors ----
  i32x4 rsA, rsB;
  unsigned aoff[8], boff[8];
  int ka = 0, kb = 0, na_left = 0, nb_left = 0, Ka = 0, Kb = 0;
  int slA = 0, slB = 0;                                    // slots of the next token / weight chunk
  const int pc = lane & 7, sub = lane >> 3;
  auto tail_a = [&]() {
#pragma unroll
    for (int p = 0; p < kA; ++p) {
      const int col = (pc ^ (((p & 1) * 4 + (lane >> 4)) & 7)) * 8;
      aoff[p] |= (unsigned)((ka >> 1) + col >= Ka) << 31;   // kOob is the top bit
    }
  };
  auto tail_b = [&]() {
#pragma unroll
    for (int p = 0; p < kB; ++p) {
      const int col = (pc ^ (((p & 1) * 4 + (lane >> 4)) & 7)) * 8;
      boff[p] |= (unsigned)((kb >> 1) + col >= Kb) << 31;
    }
  };
  auto open_a = [&](const Tile& T, int ids) {
    rsA = rsrc4(T.valid ? T.b : a.x, buffer_bytes(T.valid ? T.bbytes : 0u));
    const unsigned closed = T.valid ? 0u : kOob;           // no such tile: nothing is read
    ka = 0; Ka = uniform(T.K); na_left = T.valid ? tile_chunks(T.K) : 0x7fffffff;
#pragma unroll
    for (int p = 0; p < kA; ++p) {
      const int id = __shfl(ids, 8 * p + sub);
      const unsigned col = (unsigned)(pc ^ (((p & 1) * 4 + (lane >> 4)) & 7));
      aoff[p] = ((unsigned)max(id, 0) * T.ldb + col * 16u) | ((unsigned)(id < 0) << 31) | closed;
    }
    if (Ka < 64) tail_a();
  };
  auto open_b = [&](const Tile& T) {
    rsB = rsrc4(T.valid ? T.w0 : a.x, buffer_bytes(T.valid ? T.wbytes : 0u));
    const unsigned closed = T.valid ? 0u : kOob;
    kb = 0; Kb = uniform(T.K); nb_left = T.valid ? tile_chunks(T.K) : 0x7fffffff;
#pragma unroll
    for (int p = 0; p < kB; ++p) {
      int n;
      unsigned extra = 0;
      if (MODE == kGateUp) {
        n = T.n0 + (wave & 1) * 64 + 8 * p + sub;
        if (wave >= 2) extra = (unsigned)T.N * T.ldb;
      } else {
        n = T.n0 + wave * 64 + 8 * p + sub;
      }
      const unsigned col = (unsigned)(pc ^ (((p & 1) * 4 + (lane >> 4)) & 7));
      boff[p] = ((unsigned)min(n, max(T.N - 1, 0)) * T.ldb + extra + col * 16u) | ((unsigned)(n >= T.N) << 31) | closed;
    }
    if (Kb < 64) tail_b();
  };
  auto step_a = [&]() {
    slA = slA + 1 == SA ? 0 : slA + 1;
    na_left = uniform(na_left - 1);
    if (na_left == 0) open_a(nx, ids_nx);
    else { ka = uniform(ka + kRowB); if (uniform(Ka - (ka >> 1)) < 64) tail_a(); }
  };
  auto step_b = [&]() {
    slB = slB + 1 == SB ? 0 : slB + 1;
    nb_left = uniform(nb_left - 1);
    if (nb_left == 0) open_b(nx);
    else { kb = uniform(kb + kRowB); if (uniform(Kb - (kb >> 1)) < 64) tail_b(); }
  };
  const int ldsA = uniform((int)lds0 + wave * kA * 1024), ldsB = uniform((int)lds0 + SA * kSlotB + wave * kB * 1024);
  // load l of a period: the token chunk's first, then the weight chunk's
  auto put = [&](Loads& L, int d, int l) {
    if (l < kA) { L.rs[d] = rsA; L.vo[d] = aoff[l]; L.so[d] = uniform(ka); L.md[d] = uniform(ldsA + slA * kSlotB + l * 1024); }
    else { L.rs[d] = rsB; L.vo[d] = boff[l - kA]; L.so[d] = uniform(kb); L.md[d] = uniform(ldsB + slB * kSlotB + (l - kA) * 1024); }
  };
  open_a(cur, row_ids(cur));
  open_b(cur);
  // ---- fill: periods 1 - SB .. -1 ----
#pragma unroll
  for (int i = 1 - SB; i < 0; ++i) {
    if (i - 1 + SA >= 0) {
#pragma unroll
      for (int l = 0; l < kA; ++l) load_one(rsA, aoff[l], ka, ldsA + slA * kSlotB + l * 1024);
      step_a();
    }
#pragma unroll
    for (int l = 0; l < kB; ++l) load_one(rsB, boff[l], kb, ldsB + slB * kSlotB + l * 1024);
    step_b();
  }

  // ---- fragment addresses: a lane's 16 bytes of k-step k, without the slot and the wave's rows ----
  unsigned col[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) col[k] = lds0 + (unsigned)((lane & 31) * kRowB) + ((unsigned)(2 * k + h) ^ fkey) * 16u;
  // bytes from a slot's start to a wave's first token row and first weight rows
  auto a_at = [&](const Tile& T) { return uniform(a_row(T.tall, T.nb, wave) * kRowB); };
  auto b_at = [&](const Tile& T) { return uniform(SA * kSlotB + b_row(GU, T.tall, wave) * kRowB); };
  auto q_at = [&](const Tile& T) { return uniform(SA * kSlotB + b_row_of(GU, T.tall, wave, 3) * kRowB); };
  bf16x8 fa[2][4], fb[2][4];
  f32x16 acc[4][4];
  int cA = 0, cB = 0;                                      // slots of the chunk being multiplied
  int arow = a_at(cur), brow = b_at(cur), qrow = q_at(cur);
  first_frags<GU>(fa[0], fb[0], col[0] + arow, col[0] + brow, col[0] + qrow);
  // loads 0 .. kLoads-1 of period 0
#pragma unroll
  for (int l = 0; l < kLoads; ++l) load_one(rsA, aoff[l], ka, ldsA + slA * kSlotB + l * 1024);

  auto run_tile = [&](auto tall_tag, auto nb_tag) {
    constexpr bool TALL = decltype(tall_tag)::value;
    constexpr int NB = decltype(nb_tag)::value, TN = TALL ? 4 : 2;
    constexpr int JS = TALL ? 1 : second_frag(GU);                       // weight fragments 0, JS, ..
    const int wm = TALL ? wave >> 1 : 0, wn = TALL ? wave & 1 : wave;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j * JS][v] = 0.f;
    const int nk = uniform(tile_chunks(cur.K));
    for (int kt = 0; kt < nk; ++kt) {
      const unsigned oA = (unsigned)(cA * kSlotB + arow), oB = (unsigned)(cB * kSlotB + brow);
      Loads L;
#pragma unroll
      for (int d = 0; d < kLoads; ++d) put(L, d, kLoads + d);
      kstep<TALL, NB, GU, false>(acc, fa[0], fb[0], fa[1], fb[1], col[1] + oA, col[1] + oB, 0u, L);
#pragma unroll
      for (int d = 0; d < kLoads; ++d) put(L, d, 2 * kLoads + d);
      kstep<TALL, NB, GU, false>(acc, fa[1], fb[1], fa[0], fb[0], col[2] + oA, col[2] + oB, 0u, L);
      step_a();
#pragma unroll
      for (int d = 0; d < kLoads; ++d) put(L, d, 3 * kLoads + d);
      kstep<TALL, NB, GU, false>(acc, fa[0], fb[0], fa[1], fb[1], col[3] + oA, col[3] + oB, 0u, L);
      step_b();
      cA = cA + 1 == SA ? 0 : cA + 1;
      cB = cB + 1 == SB ? 0 : cB + 1;
      if (kt + 1 == nk) { arow = a_at(nx); brow = b_at(nx); qrow = q_at(nx); }   // the next chunk is the next tile's first
#pragma unroll
      for (int d = 0; d < kLoads; ++d) put(L, d, d);
      kstep<TALL, NB, GU, true>(acc, fa[1], fb[1], fa[0], fb[0], col[0] + (unsigned)(cA * kSlotB + arow),
                                col[0] + (unsigned)(cB * kSlotB + brow), col[0] + (unsigned)(cB * kSlotB + qrow), L);
    }
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");      // matrix results are readable
    // ---- epilogue: accumulator v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32.  The buffer
    // ends behind the tile's last row and a column that does not exist is out of range: no branches.
    constexpr unsigned kEsz = MODE == kGateUp ? 2u : 4u;
    const unsigned ldo = (unsigned)cur.N * kEsz;
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(static_cast<char*>(cur.out) + (size_t)cur.m0 * ldo,
                                                (unsigned)min(cur.m - cur.m0, 256) * ldo);
    constexpr int kCols = MODE == kGateUp ? TN / 2 : TN;
    unsigned co[kCols];
#pragma unroll
    for (int j = 0; j < kCols; ++j) {
      const int col = cur.n0 + wn * kCols * 32 + j * 32 + (lane & 31);
      co[j] = ((unsigned)(wm * NB * 32 + 4 * h) * ldo + (unsigned)col * kEsz) | ((unsigned)(col >= cur.N) << 31);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        __builtin_amdgcn_sched_barrier(0);
        const unsigned ro_off = (unsigned)(i * 32 + 8 * (v >> 2) + (v & 3)) * ldo;
#pragma unroll
        for (int j = 0; j < kCols; ++j) {
          if constexpr (MODE == kGateUp) {
            const float gte = acc_read(acc[i][j], v);
            const float hv = gte / (1.f + __expf(-gte)) * acc_read(acc[i][j + 2], v);
            __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, (__bf16)hv), ro, (int)(co[j] + ro_off), 0, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, acc_read(acc[i][j * JS], v)), ro, (int)(co[j] + ro_off), 0, 0);
          }
        }
      }
  };

  for (;;) {
    using std::integral_constant;
    if (cur.tall) {
      if (cur.nb == 4) run_tile(std::true_type{}, integral_constant<int, 4>{});
      else run_tile(std::true_type{}, integral_constant<int, 3>{});
    } else {
      if (cur.nb == 4) run_tile(std::false_type{}, integral_constant<int, 4>{});
      else if (cur.nb == 3) run_tile(std::false_type{}, integral_constant<int, 3>{});
      else if (cur.nb == 2) run_tile(std::false_type{}, integral_constant<int, 2>{});
      else run_tile(std::false_type{}, integral_constant<int, 1>{});
    }
    cur = nx;
    if (!cur.valid) break;
    nx = tile_at(ord++);
    ids_nx = row_ids(nx);
  }
  // the loads behind the last chunk only fill LDS with zeros; they end before the workgroup does
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int MODE>
int launch_wide_mode(const StreamArgs& a, hipStream_t s) {
  static std::atomic<int> ready{0};
  if (!ready.load(std::memory_order_relaxed)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&wide_kernel<MODE>), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess)
      return hip_fail(hipGetLastError(), "wide_kernel: LDS size attribute");
    ready.store(1, std::memory_order_relaxed);
  }
  int grid = device_cu_count() / 8 * 8;
  if (grid < 8) grid = 8;                                   // a multiple of the 8 XCDs
  hipLaunchKernelGGL(wide_kernel<MODE>, dim3((unsigned)grid), dim3(kThreadsW), kLdsBytes, s, a);
  return hip_fail(hipGetLastError(), "wide_kernel launch");
}

}  // namespace

int launch_wide(StreamMode mode, const StreamArgs& a, hipStream_t s) {
  return mode == kGateUp ? launch_wide_mode<kGateUp>(a, s) : launch_wide_mode<kDown>(a, s);
}

}  // namespace mm
