#include "ffn_route.h"

namespace mm {
namespace {

long long ceil_div(long long n, int per) { return (n + per - 1) / per; }

struct Work {
  long long weight_rows;             // gate rows of all weights of the layer
  long long rows;                    // token rows x weight rows, with the mean of the two expert counts per token
  long long expert_rows;             // token rows of an expert, on average
};
Work layer_work(const moe_config& c) {
  long long sh = 0;
  for (int s = 0; s < c.n_shared; ++s) sh += c.shared_I[s];
  const long long pairs = (long long)c.T * (c.k_big + c.k_little) / 2;
  return {(long long)c.E * c.I + sh, pairs * c.I + (long long)c.T * sh, ceil_div(pairs, c.E)};
}
// bf16 bytes of the layer's weights, and the sizes that the rules tell apart
constexpr long long kLargeLayer = 6ll << 27;         // 8 x 4096 x 4096 or 64 x 1024 x 2048, gate, up and down
constexpr int kScanExperts = 64;                     // one for each lane of a wave
constexpr long long kMediumLayer = 384ll << 20;      // what cannot stay in the 256 MB behind the L2s
long long layer_bytes(const moe_config& c) { return 6ll * c.H * layer_work(c).weight_rows; }

// Gate/up tiles of a step, `rows` token rows each; every expert taken for hit
long long gate_up_tiles(const moe_config& c, int rows) {
  long long n = c.E * ceil_div(c.I, kTiledPanel) * ceil_div(layer_work(c).expert_rows, rows);
  for (int s = 0; s < c.n_shared; ++s) n += ceil_div(c.shared_I[s], kTiledPanel) * ceil_div(c.T, rows);
  return n;
}

// Down tiles of a step on the 128 x 256 kernel: 256 output columns of an expert or of a K chunk of a shared expert
long long down_tiles(const moe_config& c) {
  const long long across = ceil_div(c.H, 2 * kTiledPanel);
  long long n = c.E * across * ceil_div(layer_work(c).expert_rows, kTiledRows);
  const int chunk = c.I > 1024 ? c.I : 1024;
  for (int s = 0; s < c.n_shared; ++s) n += across * ceil_div(c.shared_I[s], chunk) * ceil_div(c.T, kTiledRows);
  return n;
}

// Whole bf16 steps whose weight rows meet this many token rows on average run on 256 x 256 tiles
// (ffn_wide.hip), smaller ones on 128 x 256 (ffn_tiled.hip), whose two extra waves per SIMD hide the
// loads of short tiles better.  Many experts are hit unevenly, so that half of them still have short
// tiles at a mean where few experts have none; the full groups of shared experts come in between.
// gate+up + down, us, 128 x 256 / 256 x 256: 8 experts of 14336, 192 rows 700 / 711, 215 rows 708 / 698,
// 384 rows 1066 / 936; 64 of 1024, 281 rows 280 / 313, 384 rows 368 / 358; 64 of 1408 + 2 shared, 246
// rows 379 / 373, 266 rows 409 / 408, 325 rows 435 / 389; 60 of 1408 + 5632 shared, 229 rows 363 / 375,
// 241 rows 383 / 379, 273 rows 410 / 404, 448 rows 656 / 561; 64 of 1536 + 3072 shared, hidden 4096, 295 rows 852 / 773; 160 of
// them, hidden 5120, 241 rows 2530 / 2056.
// That holds for large layers.  In smaller ones there are so few wide tiles per CU that the last round decides, or
// K is too short for a pipeline that one wave per SIMD has to hide: 8 of 512, hidden 512, 768 rows 38 / 50;
// 32 of 512, hidden 1024, 384 rows 71 / 77; 8 of 2048 + 2048 shared, 225 rows 101 / 109; 16 of 1408, 562 rows 166 / 186, 768
// rows 224 / 247, 1125 rows 311 / 280; 64 of 1024, hidden 512, 384 rows 128 / 130; 12 of 4096, 312 rows 228 / 264, 512 rows
// 316 / 293, 750 rows 397 / 456; 24 of 2048, 375 rows 278 / 293.  And with few experts, fewer than five tiles
// per CU want full ones: 8 of 4096, hidden 4096, 281 rows 229 / 241, 412 rows 315 / 293; 8 of 8192, 281 rows 269 / 280.
bool wide_whole(const moe_config& c, int cus) {
  const Work w = layer_work(c);
  if (layer_bytes(c) < kLargeLayer) return false;
  if (c.E > kFewExperts) return w.rows >= (c.n_shared > 0 ? 240 : 352) * w.weight_rows;
  return w.rows >= (gate_up_tiles(c, kWideRows) >= 5ll * cus ? 208 : 400) * w.weight_rows;
}

// The shared experts alone are one or two groups of T rows: the wide tiles pay once there are 1.5 of them per
// CU.  us, 128 x 256 / 256 x 256 (wide gate/up tiles): one of 5632, 1024 tokens (176) 95 / 105, 2200
// (396) 200 / 190, 2800 (484) 218 / 199, 4096 (704) 340 / 278; two of 1408, 2048 tokens (176) 94 / 110,
// 2500 (220) 110 / 112, 3500 (308) 144 / 147, 4096 (352) 160 / 158.  Short rows want five of them: one of 4096, hidden
// 512, 4096 tokens (512) 86 / 100, hidden 1024 140 / 140; one of 14336, hidden 1024, 2048 tokens (896) 203 / 215,
// 3000 tokens (1344) 324 / 288.
bool wide_shared(const moe_config& c, int cus) {
  long long tiles = 0;
  for (int s = 0; s < c.n_shared; ++s) tiles += ceil_div(c.shared_I[s], kTiledPanel) * ceil_div(c.T, kWideRows);
  return 2 * tiles >= (c.H >= 2048 ? 3ll : 10ll) * cus;
}

// Order of the wide kernel's tiles in a whole step.  Contiguous ranges keep a group's token rows in one L2
// and its weights in one range of memory; the order by rows gives every XCD the same mix of tile heights. With few experts
// a range lies in one or two groups and its tiles are alike; with many, heights differ by the skew of the selection, and by the shared
// experts' full groups until the experts have about as many rows as a tile.  gate+up + down, us, mean of six random
// layers, contiguous / by rows (rows per expert): 8 experts of 14336, 1150 tokens 698 / 722, 2048 tokens
// 952 / 957, 4096 tokens 1697 / 1715; 64 of 1024, 3000 tokens 300 / 296, 4096 tokens 356 / 352; 64 of
// 1408 + 2 shared, 2500 (176) 398 / 389, 3000 (211) 400 / 433, 4096 (288) 504 / 516; 60 of 1408 + 5632
// shared, 2500 (125) 474 / 415, 4096 (205) 559 / 539.  Ranges of equal estimated time instead of equal tile
// counts: the last 531, but 2500 434 and the 64 experts 388.  Shared experts alone: one of 5632, 2800
// tokens 199 / 217, 4096 tokens 278 / 286.
constexpr long long kContiguousMinRows = 208;
bool wide_by_rows(const moe_config& c) {
  if (c.E <= kFewExperts) return false;
  return c.n_shared == 0 || (long long)c.T * (c.k_big + c.k_little) < 2 * kContiguousMinRows * c.E;
}

// Order of the 128 x 256 tiles.  By rows pays for narrow weights in steps of few rows and few tiles per workgroup where tiles differ: beside shared
// experts, whose groups are full, and where the selection is skewed.  Contiguous order's time / the time by rows, gate/up, down, geometric mean of
// four selections, at sizes that do not run in panels: 60 of 1408 + 5632 shared, 8-bit, 770 tokens 1.17, 1.25, 810 tokens (88 rows) 1.18, 1.25, 1000
// tokens 264 / 239 us, MXFP4 1.12, 1.09, 1.13, 1.09, 203 / 202 us; 64 of 1408 + 2 shared, 8-bit, 870 tokens 1.15, 1.18, 900 tokens 246 / 217 us, MXFP4
// 1.08, 1.01, 183 / 178 us; 32 of 1024 + 2048, 8-bit, 256 tokens 1.04, 1.04, 400 tokens 1.17, 1.22, 580 tokens 1.14, 1.14, MXFP4 1.04, 1.04, 1.07, 1.07,
// 1.08, 1.04; 32 of 2048 + 4096, hidden 4096, 8-bit, 580 tokens 1.14, 1.19; 60 of 1024 + 1024, skewed, 8-bit, 700 tokens 1.12, 1.22.  Alone, 64 of 1024,
// 8-bit, skewed, 420 .. 1000 tokens 1.08 .. 1.12, 1.10 .. 1.17, 2000 tokens 1.04, 1.06, unskewed 0.95 .. 0.99, 0.94 .. 0.97.  Alike tiles of MXFP4, which
// are the shortest, lose, gate+up + down, us: 32 of 2048, 256 tokens 85 / 89, 16 of 1024, hidden 4096, 800 tokens 80 / 85.  So do small
// layers: 32 of 512, hidden 1024, 400 tokens, 8-bit 37 / 39, 24 of 2048, 800 tokens, 8-bit 117 / 121.  With bf16 weights, twice the bytes per tile,
// mixing the two kinds of tiles over the XCDs is worth more (60 experts, 1000 tokens 286 / 312), and with more panels than three per CU the balance
// is there already.  In a part of a step the tiles are alike.  8-bit experts alone take the order there too, for which the reason has gone: with 2 x 2
// waves and chunks of weights the fallback passes of 64 of 1024 took 125 / 120 at 1200 tokens and 137 / 128 at 2048, now 92 / 101 and 101 / 109, 8 of
// 14336 384 / 391.
bool tiled_by_rows(const moe_config& c, bool run_routed, bool run_shared, int cus) {
  if (c.dtype != MOE_BF16_W8 && c.dtype != MOE_BF16_MXFP4) return false;
  const bool alone = c.n_shared == 0;
  if (!run_routed || (!run_shared && !alone)) return false;
  if (alone ? c.dtype != MOE_BF16_W8 || layer_bytes(c) < kLargeLayer : layer_bytes(c) < kMediumLayer) return false;
  const Work w = layer_work(c);
  return w.rows < (alone ? 208 : 88) * w.weight_rows && w.weight_rows < 3ll * kTiledPanel * cus;
}

// Token tiles per computer of the streaming kernel (stream_lds.hip) in a whole step.  bf16 has the registers for two
// (110 of a computer's 128); the narrower formats, at 114 and 125 with one, have not.  Two pay where groups have more
// than 32 rows, whose weights then pass once per 64; elsewhere they cost: the token rows of 33 .. 64 rows, whose
// loads queue behind the weight stream, are fetched by one workgroup instead of two, and a small layer has half the
// items for its CUs.  gate+up + down, us, one / two:
//   * large layers of few experts, which the weight stream bounds (from 20 rows per expert on they run in panels): 8 of 14336, 65
//     tokens 453 / 456, 100 tokens 464 / 464, half of them with all ranks 553 / 511.  Large layers of many run in panels wherever
//     their groups have that many rows.
//   * smaller ones (experts' rows): 8 of 1024, hidden 1024, 170 tokens (32) 26 / 27, 220 tokens (41) 32 / 30; 8 of 2048 + 2048,
//     170 tokens (32) 82 / 85, 220 tokens (41) 100 / 88; 16 of 1408, 128 tokens (24) 69 / 70, 220 tokens (41) 98 / 82;
//     16 of 1024, hidden 4096, 255 tokens (24) 87 / 89.  Below 32 MB never: 8 of 512, hidden 512, 170 tokens (32)
//     18.5 / 19.8, 16 of 256 + 512, 220 tokens (21) 22.5 / 25.0, 64 of 264 + 1000, hidden 520, 255 tokens (18) 40 / 42.
// Parts of a step have few rows or few groups: fallback passes, 60 experts, 65 tokens 84 / 87, 255 tokens 148 / 148;
// 64 of 1024, 100 tokens 90 / 92; the shared expert of 5632 alone, 65 tokens 53 / 61, 200 tokens 93 / 97, 255 tokens 105 / 98.
bool two_tiles(const moe_config& c) {
  if (c.dtype != MOE_BF16) return false;
  if (layer_bytes(c) >= kLargeLayer) return c.E <= kFewExperts && c.T > 64;
  return layer_bytes(c) >= 32ll << 20 && layer_work(c).expert_rows >= 36;
}

// The streaming kernel whose waves stream rows of their own (stream_panels.hip) instead of the one with loader waves
// (stream_lds.hip), for each launch by itself.  Setting its panels up takes a microsecond longer, which a small layer does not
// bring back; its waves want a tile of rows each, and a group of several token tiles passes its weights once where the other
// kernel's items fetch them again.  Rates below: stream_lds' time / stream_panels', geometric mean of four or five selections;
// layers as experts of I (+ shared), hidden 2048 unless named.  Held against other layers, drawn at random, both launches of a call (whole
// steps and fallback passes), the time on stream_lds / by these rules: bf16, 1582 calls, 1.02 in the mean, of the 1249 over 18 us 43 below 0.97,
// 0.90 at worst; narrow formats, 680 calls, 1.13, 10 of 517, 0.87.
//   * Size: bf16, 8 of 512, hidden 512, 33 tokens 0.85, 16 of 1024, hidden 4096 (403 MB), 65 tokens 0.96; 8-bit, 64 of 256 + 1024, hidden
//     512, 130 tokens 0.89, 8 of 2048 + 2048 (226 MB), 65 tokens 0.94.
//   * Narrow formats (gate/up, down): 60 of 1408 + 5632, 8-bit 1.03 .. 1.16, 1.02 .. 1.20, MXFP4 1.08 .. 1.24, 1.09 .. 1.18; 8 of 14336 0.99
//     .. 1.8, 0.99 .. 1.8.  8-bit layers of up to 64 experts of up to 1024 with short rows lose while an expert has about half a
//     token tile, some of them more than one: 64 of 1024, 64 tokens 0.96, 0.97, 96 tokens 0.95, 0.97, but 48 tokens 1.01, 1.00, 160 tokens 1.04,
//     1.03; 32 of 1024 + 2048, 64 tokens 0.92, 0.96, 128 tokens 0.89, 0.95, 32 tokens 1.07, 1.09, 160 tokens 1.00, 1.05; hidden 4096, 16 of
//     1024, 64 tokens 1.03, 1.06.  8-bit down projections of few columns: 72 of 2880 + 2880, hidden 512, 54 .. 201 tokens 0.69.
//   * Many experts have to be looked through: 256 of 512 + 512, 8-bit, 3 tokens 0.95, fallback passes of 8 tokens 0.98, 0.86, 16 tokens
//     0.95, 0.89, 32 tokens 1.05, 0.94, 64 tokens 1.07, 0.99; 128 of 768 + 768, 8 tokens 1.03, 0.94, 16 tokens 1.10, 0.98.
bool narrow_panels(const moe_config& c, bool run_shared, bool gate_up) {
  if (layer_bytes(c) < kMediumLayer) return false;
  const bool w8 = c.dtype == MOE_BF16_W8;
  if (w8 && !gate_up && c.H < 768) return false;
  if (c.E > kScanExperts) return c.T >= (run_shared ? 8 : c.E > 2 * kScanExperts ? 32 : 16);
  const long long rows = layer_work(c).expert_rows;
  return !(w8 && run_shared && c.E > kFewExperts && c.I <= 1024 && c.H <= 2048 && rows >= 5 && rows < 14);
}
//   * bf16, whole steps, gate/up.  Less than half a panel of 64 columns per CU (three quarters with rows of more than 2048) leaves the waves'
//     tiles empty, by the columns of the mean selection: 64 of 1408, two ranks, 2 tokens (3 x 1408) 0.84; 64 of 1024, 1 token (6 x 1024) 0.96;
//     60 of 512, hidden 6144, 2 tokens 0.87; 32 of 2048 + 4096, hidden 4096, 1 token (5 x 2048) 0.89; 60 of 1408 + 5632, 1 token (7 x 1408) 1.15;
//     24 of 4096, hidden 4096, 1 token (3 x 4096) 1.00.  60 of 1408 + 5632 1.03 .. 1.16; 64 of 1408 + 2 shared 1 .. 8 tokens 1.02 .. 1.16, above 1.00 .. 1.04; 48 of
//     1408 + 2816 0.99 .. 1.21.  Without shared experts, or with rows of 4096, only while few experts are hit, or again where groups
//     are of several token tiles: 64 of 1024, skewed, 3 tokens 1.12, 8 tokens 1.05, 32 tokens 1.01, 64 tokens 0.96, 128 tokens
//     1.08; 64 of 1408 alone, 3 tokens 1.11, 6 tokens 0.97, 16 .. 128 tokens 0.95 .. 0.99; 64 of 1536 + 3072, hidden 4096, 8 tokens
//     1.04, 24 tokens 0.97, 65 tokens 1.01, 128 tokens 1.04; 32 of 2048 + 4096, hidden 4096, 24 tokens 0.97, 48 tokens 1.13, 128
//     tokens 1.05; 24 of 4096, hidden 4096, 4 tokens 0.97, 64 tokens 0.95.  Long groups of short rows gain: 20 and 32 of 4096, 2 .. 128 tokens
//     1.03 .. 1.24.  Many experts lose until their shared ones weigh, long groups aside: 128 of 768 + 768, 16 .. 128 tokens 0.95 .. 0.99, 256 of 512 +
//     512 0.94 .. 0.99, 160 of 1408 + 2 shared, 32 tokens 0.95, 128 tokens 0.99, but 128 of 4096 + 8192, hidden 640, 123 tokens 1.40, 128
//     of 2048 + 2048, hidden 512, 8 tokens 1.15.
//   * bf16, whole steps, down.  Few rows of weights hit (mean selection x hidden + shared; 128 make a panel): 64 of 1024, 1 token (6 x 2048) 0.90;
//     20 of 4096, 4 tokens (6 x 2048) 0.85, 6 tokens (9 x 2048) 1.01; 24 of 4096, hidden 4096, 1 token (3 x 4096) 0.88; 64 of 1408, 1
//     token (4 x 2048) 0.90, 2 tokens (9 x 2048) 1.00; random layers 13000 .. 20000 0.97, 20000 .. 30000 1.04.  Beside shared experts, little ranks and all:
//     48 of 1408 + 2816, 1 token (5 x 2048) 0.88, 1.00, 2 tokens (8 x 2048) 1.00, 1.13; hidden 2560, 40 of 1792 + 1792, 1 token (4 x 2560) 0.84, 0.97, 2
//     tokens (7 x 2560) 0.97, 1.07; 64 of 1408 + 2 shared, 1 token (6 x 2048) 1.04, 1.03; 60 of 1408 + 5632, 1 token (7 x 2048) 0.98, 1.00, 2 tokens 1.01,
//     1.06; 64 of 1024 + 1024, 1 token (7 x 2048) 0.99, 1.13; hidden 3072, 32 of 1536 + 2 shared, 1 token (5 x 3072) 0.97, 1.12.  Few columns:
//     64 of 14336, hidden 512, 31 .. 55 tokens 0.46 .. 0.65; 96 of 2048, hidden 768, 55 tokens 0.84; 256 of 920, hidden 1024, 133 tokens 0.87; random
//     layers, hidden 900 .. 1200 0.96, 1200 .. 1600 1.02.  Above: 60 of 1408 + 5632 1.02 .. 1.15; 64 of 1408 + 2 shared 1.00
//     .. 1.13; 64 of 1024 0.97 .. 1.06; 24 of 4096, hidden 4096 1.12 .. 1.24; 256 of 512 + 512 1.06 .. 1.12.  32 of 2048 + 4096, hidden 4096, loses
//     at 6 .. 48 tokens, 0.94 .. 0.97.
//   * bf16, few experts: long groups stream as well through stream_lds.hip, whose loads are 512 bytes of a row, while they have few
//     rows: 8 of 14336, gate/up, down, 65 tokens 0.98, 0.94, 96 tokens (18 rows) 1.01, 0.97, 128 tokens (24) 1.06, 1.02, 255 tokens 1.33,
//     1.26; 8 of 8192 + 8192, 65 tokens 1.27, 1.14.
//   * bf16, fallback passes (20 % of the tokens), whose rows the host does not know.  gate/up (k_big x tokens x I in thousands): 60 of 1408, 8 tokens
//     (45) 0.99, 12 tokens (68) 1.08, 12 .. 64 tokens 1.01 .. 1.15, 128 tokens 0.97; 64 of 1024, 8 tokens (66) 0.97, 12 .. 96 tokens 1.03 .. 1.14,
//     160 tokens 0.98; 64 of 1408, 8 tokens (68) 1.04, 12 tokens 1.15, 24 .. 96 tokens 0.97 .. 1.02; 32 of 2048, hidden 4096, 8 tokens (66) 0.89, 16
//     tokens 1.04; 48 of 2048, hidden 4096, 9 tokens (147) 0.84; 60 of 512, hidden 6144, 16 tokens (16) 0.90; more than 64 experts with rows of more
//     than 2048 0.93 .. 0.98 below 48 tokens, 1.02 .. 1.05 above; 20 and 32 of 4096, 8 .. 255 tokens 1.00 .. 1.21; 128 of 768, 16 tokens 1.11, 64
//     tokens 1.00, 96 tokens 0.97; 256 of 512 0.92 .. 0.99; 8 of 14336 0.97; 8 of 8192 0.95.  down: 60 of 1408, 16 tokens (k_big x tokens = 64) 0.97,
//     24 tokens 1.07; 20 of 4096, 24 tokens (48) 0.97, 64 tokens 1.14; 64 of 1024, 8 tokens (64) 0.93, 16 tokens 1.05; 256 of 512, 16 tokens (128)
//     0.95, 32 tokens 1.01; random layers 65 .. 130 0.99, hidden below 1300 65 .. 300 0.95, above 1.03; hidden 4096, 32 of 2048 0.91 .. 0.96, 64 of
//     1536 0.97 .. 1.00; 8 of 14336 0.95 .. 0.98.
bool bf16_panels(const moe_config& c, bool run_shared, bool gate_up) {
  if (layer_bytes(c) < kLargeLayer) return false;
  const bool many = c.E > kScanExperts, short_rows = c.H <= 2048, long_groups = c.I >= 2 * c.H, few_columns = c.H < 1280;
  const Work w = layer_work(c);
  const long long sh = w.weight_rows - (long long)c.E * c.I;
  if (!run_shared) {
    if (c.E <= kFewExperts) return false;
    if (!gate_up) return short_rows && c.T * c.k_big >= (few_columns ? 300 : many ? 130 : 100);
    if (long_groups) return c.T >= 8;
    if (c.T < (short_rows ? 8 : 12) || (long long)c.T * c.k_big * c.I < 66000) return false;
    return !many ? c.T < 128 : short_rows ? c.T >= 16 && c.T <= 64 && c.I >= 768 : c.T >= 48;
  }
  if (c.E <= kFewExperts) return c.T > 64 && (sh > 0 || w.expert_rows >= 20);
  if (many && c.T < 8) return false;
  const long long pairs = (long long)c.T * (c.k_big + c.k_little) / 2, hit = (pairs < c.E ? pairs : c.E) + sh / c.I;
  if (!gate_up) return !few_columns && (c.T > 64 || hit * c.H >= (sh > 0 ? 12000 : 20000));
  if (hit * c.I < (short_rows ? 8192 : 12288)) return false;
  // token tiles of 16 rows that the weight rows meet, in sixteenths
  const long long tiles = c.E * (long long)c.I * (w.expert_rows > 16 ? w.expert_rows : 16) + 16 * sh * ceil_div(c.T, 16);
  if (100 * tiles >= 16 * w.weight_rows * (many ? 115 : 110)) return true;
  if (many) return long_groups;
  return (short_rows && (sh > 0 || w.expert_rows >= 12)) || long_groups || 4 * pairs <= 3 * c.E;
}
bool stream_panels(const moe_config& c, bool run_routed, bool run_shared, bool gate_up) {
  if (!run_routed) return false;       // the shared experts alone: few rows per wave
  return c.dtype == MOE_BF16 ? bf16_panels(c, run_shared, gate_up) : narrow_panels(c, run_shared, gate_up);
}

// The same kernel for prefill of few rows per expert, where the tiled kernels' blocks of 128 token rows are mostly
// padding: narrow weights that meet fewer token rows on average than `most` (there is as little to set up in proportion
// that layers of any size gain), bf16 weights of up to kFewExperts experts.  Above, a panel's passes of 64 token rows over its
// weights are more and the tiled kernels' 128 are full.  Each launch by itself: the down projection, with half the columns and
// thus fewer tiles for the CUs, gains longer than gate/up.  Rates: the tiled kernel's time / the panels' (two tiles per wave where
// the next rule wants them), gate/up, down, geometric mean of four selections; token rows per weight row in brackets.  Held against
// other layers, drawn at random, with the tiles of then: narrow formats, 1434 calls, 1.15 in the mean, of the 1344 over 18 us 5 below 0.97, 0.82 at
// worst; bf16, 716 calls, 1.01, 3 of 699, 0.96.
// The lines were drawn while the tiles of narrow weights took up to 25 % (MXFP4) and 10 % (8-bit) longer, the figures are from the present ones: below 1
// on the panels' side of a line is what the line gives away since, in MXFP4 from about 50 rows on and in gate/up of skewed 8-bit experts.
//   * few experts, alike: 8 of 14336, 8-bit, 256 tokens (48) 1.00, 1.38, 340 tokens (64) 0.94, 1.23, 420 tokens (79) 0.77, 0.73; MXFP4, 256
//     tokens 1.23, 1.40, 380 tokens (71) 0.89, 1.38, 500 tokens (94) 0.69, 0.92; 8 of 512, hidden 512, 256 tokens, 8-bit 1.36, 1.50, MXFP4
//     1.10, 1.11.  Where the panels fill one round of the CUs, but not two, a second block of 64 rows is another round, which the faster
//     MXFP4 tiles do not lose: 16 of 1408, 560 tokens (52) 0.90, 0.91, 620 tokens (58) 0.75, 0.91, 8-bit 1.00, 1.32, 740 tokens (69) 1.01, 1.13.
//   * many: 60 of 1408 + 5632, 8-bit, 256 tokens (28) 1.00, 1.32, 740 tokens (81) 0.97, 0.96, 900 tokens (98) 0.93, 1.07; MXFP4 1.13, 1.35, 0.90,
//     0.81, 0.83, 0.83; 64 of 1408 + 2 shared, 8-bit, 800 tokens (79) 1.11, 1.13, MXFP4 0.89, 0.87; 20 of 4096, 400 tokens (30), 8-bit 1.27, 1.12, MXFP4
//     1.28, 1.29, 900 tokens (68) 1.10, 1.06, 0.89, 0.80.  With fewer of
//     them the rows are more alike: 24 of 4096 + 2 shared, hidden 1792, 8-bit, 582 tokens (78) 1.15, 0.84, 32 of 3456, hidden 7168, 873 tokens (82) 0.70, 0.80, 17
//     of 8192 + 16384, 299 tokens (79) 0.92, 0.89; MXFP4, 40 of 2048 + 2 shared, hidden 2816, 380 tokens (72) 0.65, 1.07, 440 tokens (84) 0.58, 0.93.
//   * many of up to 1024, with a selection skewed as by gate biases of a standard deviation of 0 / 1 / 2: 64 of 1024, 8-bit, gate/up, 300
//     tokens (28) 1.15 / 1.09 / 1.08, 380 tokens (36) 1.15 / 0.92 / 1.00, 460 tokens (43) 1.11 / 0.82 / 0.93, 620 tokens (58) 1.14 / 0.82 / 0.82, 680
//     tokens (64) 1.00 / 0.95 / 0.83, 740 tokens (69) 0.85 / 1.07 / 0.84, down 1.0 .. 1.35 throughout; MXFP4, gate/up, 300 tokens 1.25 / 0.93 / 1.10, 500
//     tokens (47) 0.89 / 0.95 / 0.94, 620 tokens 0.76 / 0.75 / 0.96, 740 tokens 0.78 / 1.02 / 0.75, down 1.17 / 1.02 / 1.14, 0.92 / 1.04 / 1.04, 0.80 / 0.86 /
//     1.02, 0.82 / 1.12 / 0.84.  What gate/up
//     loses at 36 .. 61 rows (8-bit) and from 56 on (MXFP4) it loses by its rounds: 1024 panels are four of 256 CUs exactly, so that
//     every expert with a second block makes a fifth.  Where the last round has room it gains as before: 8-bit, 96 of 768 (4.5
//     rounds), 800 tokens (38) 1.27, 128 of 768 + 768 (6.5), 740 tokens (40) 1.27, 64 of 1024 + 1024, hidden 4096 (4.4), 340 tokens (37) 1.19,
//     560 tokens (60) 1.05, MXFP4 0.99, 680 tokens (73) 0.87.
//     Smaller layers of them: 32 of 1024, 8-bit, 340 tokens (32) 1.02, 1.06, 740 tokens (69) 0.67, 0.85; MXFP4, 380 tokens (36) 1.14, 1.01, 460 tokens
//     (43) 0.85, 0.89; 64 of 512, hidden 1024, MXFP4, 380 tokens (36) 0.90, 0.92, 460 tokens (43) 0.78, 0.87.
//   * bf16, where the tiles leave part of the CUs idle in their rounds: 8 of 14336, 256 tokens (48), gate/up (896 tiles, 3.5 rounds) 1.05, down
//     (128 tiles) 1.12, 319 tokens (60) 1.04, 1.09, 380 tokens (71) 0.96, 0.80; 16 of 1024, hidden 4096, 256 tokens, gate/up (128) 1.11, down (256) 1.05, 560
//     tokens (52) 1.03, 0.96; beside shared experts, whose groups are full, and with many it loses: 60 of 1408 + 5632, 256 tokens (28) 0.96, 0.89, 8 of
//     4096 + 4096, hidden 4096, 300 tokens 0.81, 0.77.  16 of 4096, hidden 4096, 300 tokens 1.03, 1.08 and 20 of 4096, 420 tokens (32) 1.12, 1.06 stay on tiles.
//   * fallback passes (20 % of the tokens) gain more: 60 of 1408, 8-bit 1.14 .. 1.36, 1.09 .. 1.23, MXFP4 1.7 .. 2.1, 1.46 .. 1.63; 64 of 1024, 8-bit 1.10 .. 1.12,
//     1.18 .. 1.21, MXFP4 1.55 .. 1.66, 1.39 .. 1.47; bf16, 8 of 14336 1.06, 1.14, 16 of 4096 1.10, 1.16.  The lines by rows are
//     those of the whole step all the same, for a part may have all of its rows; second blocks are rare in it.
bool prefill_panels(const moe_config& c, bool run_routed, bool run_shared, bool gate_up, int cus) {
  if (!run_routed || c.T > kPanelsMaxT) return false;
  const Work w = layer_work(c);
  const bool w8 = c.dtype == MOE_BF16_W8, few = c.E <= kFewExperts, large = layer_bytes(c) >= kLargeLayer;
  auto fewer_rows = [&](int than) { return w.rows < than * w.weight_rows; };
  if (c.dtype == MOE_BF16) {
    if (!few || layer_bytes(c) < kMediumLayer || !fewer_rows(60)) return false;
    const long long tiles = gate_up ? gate_up_tiles(c, kTiledRows) : down_tiles(c);
    return !run_shared || (c.n_shared == 0 && 8 * tiles <= 7 * cus * ceil_div(tiles, cus));
  }
  if (!w8 && c.dtype != MOE_BF16_MXFP4) return false;
  int most = few ? (w8 ? 70 : 76) : c.I > 1024 ? (c.E < 48 ? 76 : 84) : large ? 76 : 36;
  if (!w8 && !few && c.I > 1024 && c.E < 48 && gate_up && run_shared) most = 70;
  if (!fewer_rows(most)) return false;
  if (!gate_up || !run_shared) return true;
  constexpr int kColumns = 64, kPanelRows = 64;      // of a panel of one tile per wave
  long long panels = c.E * ceil_div(c.I, kColumns);
  for (int s = 0; s < c.n_shared; ++s) panels += ceil_div(c.shared_I[s], kColumns) * ceil_div(c.T, kPanelRows);
  if (few) return w8 || large || fewer_rows(56) || 2 * panels <= cus;
  const bool full_rounds = 16 * (cus * ceil_div(panels, cus) - panels) < panels;
  if (c.I > 1024 || !full_rounds) return true;
  return w8 ? fewer_rows(36) || !fewer_rows(62) : fewer_rows(56);
}

// Two tiles of weight rows per wave, which share the token rows' fragments, instead of one.  A tile of narrow weights
// is computed from LDS slower than it comes from HBM once it meets several tiles of token rows, and half of the reads are
// the token rows'.  With fewer rows the larger panels leave more of the last round empty.  gate+up + down, us, one / two:
//   * MXFP4, 60 of 1408 + 5632, 200 tokens (22 rows per weight row) 103 / 105, 255 tokens (28) 119 / 112; 64 of 1408 + 2 shared,
//     255 tokens (25) 108 / 112; 8 of 14336, 128 tokens (24) 191 / 198, 200 tokens (38) 235 / 232.
//     Above 255 tokens, 20 % of the tokens with all ranks: 60 of 1408 + 5632, 256 tokens (28) 116 / 115, 420 tokens (46) 146 / 151; 64 of 1408 + 2
//     shared, 420 tokens (41) 136 / 129; 64 of 1024, 300 tokens (28) 74 / 72; 8 of 14336, 256 tokens (48) 316 / 284, 400 tokens (75) 407 / 372.
//   * 8-bit, likewise: 60 of 1408 + 5632, 256 tokens (28) 144 / 145, 420 tokens (46) 174 / 161; 64 of 1408 + 2 shared, 420 tokens (41) 152 / 153, 540
//     tokens (53) 178 / 163; 64 of 1024, 540 tokens (51) 106 / 102, with half of the tokens 132 / 126, with all 167 / 169; 8 of 14336, 256 tokens (48)
//     298 / 312, 278 tokens (52) 307 / 318, 360 / 353, 508 / 457, 370 tokens (69) 389 / 362, 502 / 447, 576 / 493.
//   * Parts of a step have fewer rows than that: 60 of 1408, fallback pass, 420 tokens, 8-bit 91 / 95, MXFP4 63 / 68.  There they pay where they make one
//     round over the CUs of two: 64 of 272, hidden 528, 256 tokens 27.1 / 25.0.  bf16 weights: 8 of 14336, 256 tokens 484 / 494.
bool wide_panels(const moe_config& c, bool run_shared, int cus) {
  if (c.dtype != MOE_BF16_W8 && c.dtype != MOE_BF16_MXFP4) return false;
  if (!run_shared) {
    constexpr int kColumns = 64;       // gate/up columns of a panel of one tile per wave
    return c.T >= kTiledMinT && c.E * ceil_div(c.I, kColumns) > cus && c.E * ceil_div(c.I, 2 * kColumns) <= cus;
  }
  const Work w = layer_work(c);
  return w.rows >= (c.dtype == MOE_BF16_W8 ? 52 : 27) * w.weight_rows;
}

// bf16 weights that are read once in a launch need no place in the caches, which then hold the token rows longer.
// gate+up + down, us, through the caches / past them: 64 of 1024, 300 tokens 146 / 133, 777 tokens 208 / 200, 16 of
// 1024, hidden 4096 (403 MB), 600 tokens 119 / 111, 24 of 2048 (604 MB), 1200 tokens 179 / 171, 32 of 1024 + 2048 (428 MB),
// 256 tokens 142 / 129.  A layer that can stay in the 256 MB behind the L2s from one step to the next loses, though one that
// has left them in between gains (second pair): 32 of 512, hidden 1024 (101 MB), 256 tokens 34 / 41, 41 / 39, 8 of
// 2048 + 2048 (226 MB), 256 tokens 66 / 81, 84 / 75, 16 of 1408 (277 MB), 600 tokens 87 / 94, 93 / 91.  A chunk has to be a
// cache line: of rows that are not whole lines its pieces share lines with the next chunk's, which then come twice (64 of
// 1968 + 2064, hidden 3256, 3424 tokens 894 / 1064, 64 of 1864, hidden 3104, fallback pass of 273 tokens 436 / 502), and
// a chunk of narrow weights is half a line and less (MXFP4, 60 experts, 600 tokens, gate+up 123 / 147; whole_lines has its own).
constexpr int kLineWeights = 64;                     // bf16 weights in a cache line of 128 bytes
bool weights_once(const moe_config& c) {
  bool lines = c.H % kLineWeights == 0 && c.I % kLineWeights == 0;
  for (int s = 0; s < c.n_shared; ++s) lines = lines && c.shared_I[s] % kLineWeights == 0;
  return c.dtype == MOE_BF16 && lines && layer_bytes(c) >= kMediumLayer;
}

// Gate/up of a whole step of 129 .. 255 tokens on the tiled kernel, past the caches, whose blocks of 128 token rows pass half as often over the
// weights of the large groups: of the shared experts and of few experts.  At 128 tokens and less the shared experts' blocks are as many as the
// panels', and with many experts so is everything that counts.  stream_lds' time / panels' / tiles', geometric mean of five selections: 60 of 1408 +
// 5632, 128 tokens 1.15 / 1.03, 129 tokens 1.02 / 1.18, 255 tokens 1.11 / 1.36; 64 of 1408 + 2 shared 1.04 / 1.00, 1.03 / 1.10, 1.08 / 1.22; 48 of
// 1408 + 2816 1.03 / 0.97, 1.04 / 1.05, 1.20 / 1.23; 8 of 14336 1.06 / 1.13, 1.06 / 1.14, 1.33 / 1.42; 8 of 8192 + 8192 1.16 / 1.12, 1.22 / 1.41,
// 1.43 / 1.90; hidden 4096, 64 of 1536 + 3072 1.04 / 0.97, 1.06 / 1.07, 1.10 / 1.17, 32 of 2048 + 4096 1.05 / 0.96, 1.11 / 1.14, 1.16 / 1.30. Alone,
// either may win: 64 of 1408 0.96 / 1.03 at all three, 64 of 1024 1.08 / 1.10, 1.08 / 1.10, 1.19 / 1.29, 20 of 4096 1.08 / 1.14, 1.08 / 1.14, 1.10 /
// 1.20, 40 of 1280, hidden 4096, 186 tokens 1.00 / 0.88, 12 of 2880, hidden 7168, 150 tokens (19 rows each) 1.10 / 0.92, 64 of 2880, hidden 3312, 157
// tokens 1.05 / 0.88, 60 of 4096, hidden 1024, 150 tokens 1.12 / 1.06, 28 random ones 1.08 / 1.02. Many: 160 of 1408 + 2 shared, 129 tokens 0.99 /
// 0.99, 255 tokens 1.03 / 1.03; 128 of 768 + 768 0.92 / 0.99, 0.96 / 0.97; 256 of 512 + 512 0.96 / 0.93, 0.96 / 0.97.  The down projection has half
// as many columns and more of K: on the tiles of 256 rows, which have one sum, it gained only in 8 of 8192 + 8192 and 32 of 2048 + 4096 (255 tokens
// 132 / 115 us).
bool tiled_gate_up(const moe_config& c) {
  const bool large_groups = c.n_shared > 0 ? c.E <= kScanExperts : c.E <= kFewExperts && layer_work(c).expert_rows >= 20;
  return c.T > kTiledRows && large_groups && layer_bytes(c) >= kLargeLayer && weights_once(c);
}

// Narrow weights in whole lines (ffn_tiled.hip, with figures of the layers that gain): a tile waits for a line before its first chunk, which
// layers of little time per tile feel (us, MXFP4, chunks / lines: 64 experts of 256, hidden 512, 900 tokens 17.0 + 13.5 / 18.5 + 14.5; 32
// of 1024, hidden 1024 (201 MB in bf16) 24.8 + 22.9 / 27.1 + 23.1; 16 of 1024, hidden 4096 (403 MB) 67.5 + 26.5 / 62.0 + 24.1), and 8-bit
// ones whose matrix cores set the pace (8 bits, 64 of 1024, 2500 tokens 173 + 130 / 175 + 131; 8 of 14336, 1400 tokens 474 + 210 / 477 + 209,
// 900 tokens 422 + 203 / 418 + 186) or whose rows are not whole lines (64 of 1968 + 2064, hidden 3264, 600 tokens 243 + 160 / 247 + 176;
// 24 of 1872, hidden 3120, 121 + 83 / 117 + 80).  MXFP4 gains there too (64 of 1920, hidden 3200, 600 tokens 184 + 110 / 175 + 106).
// A line of a panel of one token tile goes past the caches, which MXFP4 layers of up to twice the 384 MB feel in fallback passes where they would
// stay in the 256 MB behind the L2s, i.e. where no other layer runs in between (two layers in turn / six): 24 of 768 + 2 shared, hidden 4096, 500 tokens,
// the pass 84 / 90 and 96 / 90, 16 of 1024, hidden 4096, 900 tokens 74 / 80 and 90 / 80, 24 of 2048, 700 tokens 95 / 90 and 99 / 90.
bool whole_lines(const moe_config& c) {
  const Work w = layer_work(c);
  if (c.dtype == MOE_BF16 || layer_bytes(c) < 384ll << 20) return false;
  if (c.dtype != MOE_BF16_W8) return true;
  bool lines = c.H % 128 == 0 && c.I % 128 == 0;
  for (int s = 0; s < c.n_shared; ++s) lines = lines && c.shared_I[s] % 128 == 0;
  return lines && w.rows < 200 * w.weight_rows;
}

// bf16 tiles of a width that fills their last round over the CUs, which the kernel chooses where that round has room (ffn_tiled.hip, with
// figures).  With so many rows that the matrix cores set the pace of gate/up (rows per weight row: 8 of 14336, 131, 350 / 360 us, 225, 521 / 538) or
// have no room left in the down projection (20 of 4096, 150, 87 / 88; but 8 of 14336, 131, 252 / 218) it only costs.  Below, launches whose rounds have no
// room lose at most a microsecond or two where others gain 5 to 25 % (8 of 14336, 450 tokens, gate/up (84) 350 / 350, down 232 / 185; 64 of 1024, 450
// tokens, gate/up 99.7 / 95.0, down 56.9 / 57.8; 40 of 1280, hidden 4096, 500 tokens, gate/up 142.7 / 145.3, down 92.3 / 88.4).  A small layer
// has no rounds to speak of (8 of 512, hidden 512, 1000 tokens 18.0 + 16.6 / 18.7 + 17.1; 8 of 1408 + 1408, hidden 1024 (78 MB), 700 tokens 30.2 / 26.2).
bool even_tiles(const moe_config& c, bool gate_up) {
  const Work w = layer_work(c);
  return c.dtype == MOE_BF16 && layer_bytes(c) >= 64ll << 20 && w.rows < (gate_up ? 96 : 150) * w.weight_rows;
}

}  // namespace

// A call that runs the routed part alone is taken for a part of a step: a fallback pass (some ranks of the
// rejected tokens), or the experts of one wave of an offloaded layer.  Its rows are known to the
// device only, and by the layer's own sizes they would be overrated: it stays on the smaller tiles.  (Fallback pass,
// 20 % of the tokens, gate+up + down, us, 128 x 256 / 256 x 256: 60 experts of 1408, 2500 tokens 213 / 245,
// 4096 tokens 219 / 251, 50 % of them 232 / 272; 64 of 1408, 3000 tokens 222 / 245; 8 of 14336, 1200 tokens
// 549 / 598, 4000 tokens 639 / 664.  All pairs of 60 experts of 1408 without the shared one, 4096 tokens 342 / 338.)
FfnRoute ffn_route(const moe_config& c, bool run_routed, bool run_shared, int cus) {
  const bool whole = run_routed && run_shared;
  FfnRoute r = {};
  if (c.dtype == MOE_FP32) return r;
  if (c.T < kTiledMinT) {
    auto kernel = [&](bool gate_up) { return stream_panels(c, run_routed, run_shared, gate_up) ? kFfnPanels : kFfnStream; };
    r.gate_up = kernel(true); r.down = kernel(false);
    if (whole && tiled_gate_up(c)) r.gate_up = kFfnTiled;
  } else if (c.dtype == MOE_BF16 && (whole ? wide_whole(c, cus) : !run_routed && wide_shared(c, cus))) {
    r.gate_up = r.down = kFfnWide;
    r.by_rows_gate_up = r.by_rows_down = whole && wide_by_rows(c);
  } else {
    auto kernel = [&](bool gate_up) { return prefill_panels(c, run_routed, run_shared, gate_up, cus) ? kFfnPanels : kFfnTiled; };
    r.gate_up = kernel(true); r.down = kernel(false);
    const bool by_rows = tiled_by_rows(c, run_routed, run_shared, cus);
    r.by_rows_down = r.down == kFfnTiled && by_rows;
    r.by_rows_gate_up = r.gate_up == kFfnTiled && by_rows;
    r.even_gate_up = r.gate_up == kFfnTiled && even_tiles(c, true);
    r.even_down = r.down == kFfnTiled && even_tiles(c, false);
  }
  auto any = [&](FfnKernel k) { return r.gate_up == k || r.down == k; };
  r.two_tiles = any(kFfnStream) && whole && two_tiles(c);
  r.wide_panels = any(kFfnPanels) && wide_panels(c, run_shared, cus);
  r.weights_once = any(kFfnTiled) && weights_once(c);
  r.lines = any(kFfnTiled) && whole_lines(c);
  return r;
}

// Decode batches take one launch.  Every workgroup of it reads the whole gate matrix for its one token, and its
// waves the experts one after the other, so above 64 tokens only while there are few experts and the reads
// of all tokens together stay small (the GEMV's four-token blocks read a matrix a quarter as often, on as
// many waves as there are experts).  us, two launches / one, on a card that launches fast: bf16, 8 x 4096, 256
// tokens 10.8 / 8.3, 60 x 2048, 200 tokens 10.7 / 8.3, 64 x 2048, 256 tokens (64 MB) 10.7 / 9.1, 64 x 4096,
// 200 tokens (100 MB) 11.9 / 11.8, 256 tokens (128 MB) 11.8 / 12.4, 32 x 8192, 128 tokens (64 MB) 12.1 / 10.4;
// fp32, 60 x 2048, 128 tokens (60 MB) 10.7 / 9.4, 200 tokens (94 MB) 10.6 / 10.5, 64 x 2048, 128 tokens (64
// MB) 10.8 / 11.0.  Many experts, on a slower one: 128 x 2048, 65 tokens, bf16 11.8 / 11.8, fp32 11.8 /
// 15.1, 256 x 256 bf16 12.1 / 16.9.
RouterKernel router_kernel(const moe_config& c) {
  constexpr int kOneLaunchMaxT = 64, kGemvMaxT = 256, kOneLaunchExperts = 64;
  if (c.T <= kOneLaunchMaxT) return kRouterOneLaunch;
  if (c.T > kGemvMaxT) return kRouterGemm;
  const bool fp32 = c.dtype == MOE_FP32;
  const long long reads = (long long)c.T * c.E * c.H * (fp32 ? 4 : 2), limit = (fp32 ? 60ll : 100ll) << 20;
  return c.E <= kOneLaunchExperts && reads <= limit ? kRouterOneLaunch : kRouterGemv;
}

// Counting in the selection saves a launch, and every workgroup of the dispatch then adds up a row per 16 tokens instead of one per 128, eight times
// the table, which grows with T^2 E.  us per step, counted by the selection / by a launch of its own, hidden 2048: 8 experts of 2048, 8192 tokens 325 /
// 328, 16384 tokens 629 / 629; 16 of 1024, 8192 tokens 219 / 221, 12000 tokens 295 / 294; 32 of 512, 4096 tokens 157 / 158, 8192 tokens 254 / 252; 64
// of 256, 300 tokens 70 / 73, 2048 tokens 123 / 124, 4096 tokens 200 / 200, 8192 tokens 345 / 341, 16384 tokens 684 / 671; 128 of 128, 1024 tokens
// 96 / 97, 2048 tokens 124 / 123, 16384 tokens 627 / 599; 256 of 128, 512 tokens 125 / 126, 1024 tokens 137 / 136, 16384 tokens 759 / 703.
bool selection_counts(const moe_config& c) {
  constexpr int kMaxT = 8192, kMaxTable = 128 << 10;
  return c.T > kSmallDispatchT && c.T <= kMaxT && c.T * c.E <= kMaxTable && router_kernel(c) == kRouterGemm;
}

}  // namespace mm
