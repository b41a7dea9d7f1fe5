// Prints whether a call of moe_expert_ffn streams its weights in panels (csrc/ffn_route.cpp, no HIP).
//
// stdin:   dtype T H E I k_big k_little n_shared shared_I_0 ... run_routed run_shared     (one line per call)
// stdout:  kernel panels wide_panels tiled_gate_up
#include <stdio.h>

#include "ffn_route.h"

int main() {
  moe_config c = {};
  while (scanf("%d %d %d %d %d %d %d %d", &c.dtype, &c.T, &c.H, &c.E, &c.I, &c.k_big, &c.k_little, &c.n_shared) == 8) {
    int routed, shared;
    for (int s = 0; s < c.n_shared; ++s)
      if (s >= MOE_MAX_SHARED || scanf("%d", &c.shared_I[s]) != 1) return 2;
    if (scanf("%d %d", &routed, &shared) != 2) return 2;
    const mm::FfnRoute r = mm::ffn_route(c, routed != 0, shared != 0, 256);
    printf("%d %d %d %d\n", (int)r.kernel, (int)r.panels, (int)r.wide_panels, (int)r.tiled_gate_up);
  }
}
