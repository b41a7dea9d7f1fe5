// Prints what ffn_route, router_kernel and selection_counts (csrc/ffn_route.cpp, no HIP) decide.
//
// stdin:   dtype T H E I k_big k_little n_shared shared_I_0 ... run_routed run_shared cus     (one line per call)
// stdout:  gate_up down by_rows_gate_up by_rows_down two_tiles wide_panels weights_once router even_gate_up even_down lines selection_counts
#include <stdio.h>

#include "ffn_route.h"

int main() {
  moe_config c = {};
  while (scanf("%d %d %d %d %d %d %d %d", &c.dtype, &c.T, &c.H, &c.E, &c.I, &c.k_big, &c.k_little, &c.n_shared) == 8) {
    int routed, shared, cus;
    for (int s = 0; s < c.n_shared; ++s)
      if (s >= MOE_MAX_SHARED || scanf("%d", &c.shared_I[s]) != 1) return 2;
    if (scanf("%d %d %d", &routed, &shared, &cus) != 3) return 2;
    const mm::FfnRoute r = mm::ffn_route(c, routed != 0, shared != 0, cus);
    printf("%d %d %d %d %d %d %d %d %d %d %d %d\n", (int)r.gate_up, (int)r.down, (int)r.by_rows_gate_up, (int)r.by_rows_down, (int)r.two_tiles,
           (int)r.wide_panels, (int)r.weights_once, (int)mm::router_kernel(c), (int)r.even_gate_up, (int)r.even_down, (int)r.lines,
           (int)mm::selection_counts(c));
  }
}
