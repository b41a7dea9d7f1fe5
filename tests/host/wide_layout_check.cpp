// Prints every fragment read of the 256 x 256 kernel behind its barrier: mode, tall, blocks per wave (0: no
// next tile), wave, operand, fragment, first row in the slot, first byte in LDS from the slots' start for
// the operand's last slot.  Then the load cursors.
#include <cstdio>

#include "wide_layout.h"

using namespace mm::wide;

int main() {
  std::printf("%d %d\n", kSlotRows, (SA + SB) * kSlotB);
  for (int gate_up = 0; gate_up < 2; ++gate_up)
    for (int tall = 0; tall < 2; ++tall)
      for (int nb = tall ? 3 : 0; nb <= 4; ++nb)
        for (int wave = 0; wave < 4; ++wave)
          for (int f = 0; f < kFrags; ++f) {
            const int a = a_row(tall, nb, wave) + f * kBlock, b = b_row_of(gate_up, tall, wave, f) + b_frag_row(gate_up, f);
            std::printf("%d %d %d %d a %d %d %d\n", gate_up, tall, nb, wave, f, a, (SA - 1) * kSlotB + a * kRowB);
            std::printf("%d %d %d %d b %d %d %d\n", gate_up, tall, nb, wave, f, b, (SA + SB - 1) * kSlotB + b * kRowB);
          }
  // load cursors on a tensor of one row of K values, K = 0: no tile: chunks, size that the descriptor states
  for (int K = 0; K <= 328; K += 8) std::printf("k %d %d %u\n", K, tile_chunks(K), buffer_bytes(2u * K));
}
