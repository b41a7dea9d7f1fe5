// Which kernel a call of moe_route, moe_expert_ffn or moe_layer_step runs on, and in which order its tiles: plain host C++ (no
// HIP), from sizes alone, so that the rules can be checked without a GPU.
#pragma once

#include "mobile_moe.h"

namespace mm {

// Steps of this many tokens and more run the LDS-tiled kernels (bf16 activations) where the experts see
// enough rows for MFMA tiles.  Below that the weights are streamed once through a skinny kernel.
constexpr int kTiledMinT = 256;
constexpr int kPanelsMaxT = 65535;   // tokens that stream_panels.hip can number
constexpr int kTiledPanel = 128;     // gate/up output columns of a tile of either tiled kernel
constexpr int kTiledRows = 128;      // token rows of a tile of the 128 x 256 kernel
constexpr int kWideRows = 256;       // token rows of a tile of the wide kernel
constexpr int kFewExperts = 16;      // up to here one of eight ranges of tiles lies in one or two experts

// stream_gemm.hip and stream_lds.hip; ffn_tiled.hip; ffn_wide.hip; stream_panels.hip
enum FfnKernel { kFfnStream = 0, kFfnTiled = 1, kFfnWide = 2, kFfnPanels = 3 };
// Which kernel a launch runs on does not show in its results: below kTiledMinT tokens all have two sums per output, from there on one.
struct FfnRoute {
  FfnKernel gate_up, down;
  // false where no launch runs on the kernel in question
  bool wide_panels;                  // StreamArgs::wide_panels (stream_panels.hip)
  bool two_tiles;                    // StreamArgs::two_tiles (stream_lds.hip)
  bool weights_once;                 // StreamArgs::weights_once (ffn_tiled.hip)
  bool lines;                        // StreamArgs::lines (ffn_tiled.hip)
  bool even_gate_up, even_down;      // StreamArgs::even_tiles of the two launches (ffn_tiled.hip)
  bool by_rows_gate_up, by_rows_down;   // StreamArgs::by_rows of the two launches (ffn_tiled.hip, ffn_wide.hip)
};

// run_routed, run_shared: as moe_expert_ffn gets them, also where the layer has no shared experts;
// cus: compute units of the device (only used from kTiledMinT tokens on).
FfnRoute ffn_route(const moe_config& c, bool run_routed, bool run_shared, int cus);

// Router logits of a step.  kRouterOneLaunch: logits and selection of a token in one workgroup; kRouterGemv:
// plain-FMA GEMV over many waves, then the selection; kRouterGemm: MFMA tiles (gate_mfma_kernel), then the selection.
enum RouterKernel { kRouterOneLaunch = 0, kRouterGemv = 1, kRouterGemm = 2 };
RouterKernel router_kernel(const moe_config& c);

constexpr int kSmallDispatchT = 256; // tokens that one workgroup of the dispatch places without counting
// A step of one call: the selection counts the pairs of each expert for the dispatch, per 16 tokens.
bool selection_counts(const moe_config& c);

}  // namespace mm
