// Which rows of the LDS slots the waves of the 256 x 256 kernel (ffn_wide.hip) read as fragments.  Plain
// C++ without HIP, so that the bounds are checked where there is no GPU.
#pragma once

namespace mm {
namespace wide {

constexpr int kRowB = 128;              // bytes of a tile row in LDS (64 k)
constexpr int kSlotRows = 256;
constexpr int kSlotB = kSlotRows * kRowB;
constexpr int SA = 2, SB = 3;           // token slots, then weight slots: all of the CU's LDS
constexpr int kBlock = 32;              // rows of a fragment
constexpr int kFrags = 4;               // fragments of a wave and k-step, of either operand

// Tiles of more than 128 tokens (tall): waves in a 2 x 2 grid, nb blocks of token rows and four weight
// fragments each.  Narrower ones: every wave has all nb blocks of token rows and two weight fragments.
// Weight fragments 0 and 1 are neighbours, 2 and 3 lie half_rows behind them (gate/up: the up rows).
constexpr int half_rows(bool gate_up) { return gate_up ? 128 : 64; }
constexpr int b_frag_row(bool gate_up, int j) { return (j >> 1) * half_rows(gate_up) + (j & 1) * kBlock; }
constexpr int second_frag(bool gate_up) { return gate_up ? 2 : 1; }    // beside 0, of a narrow tile's wave

constexpr int a_row(bool tall, int nb, int wave) { return tall ? (wave >> 1) * nb * kBlock : 0; }
constexpr int b_row(bool gate_up, bool tall, int wave) {
  const int narrow = gate_up ? kBlock : 2 * kBlock;        // rows of a narrow tile's wave in (the gate half of) a slot
  return tall ? (wave & 1) * 2 * narrow : wave * narrow;
}
// The reads behind the barrier fetch all four weight fragments, whatever the next tile is.  The two that a
// narrow tile's wave has no use for are read from the slot's first rows: from its own row on they would
// end behind the slot, and in the last slot behind the CU's LDS.
constexpr int b_row_of(bool gate_up, bool tall, int wave, int j) {
  return tall || j == 0 || j == second_frag(gate_up) ? b_row(gate_up, tall, wave) : 0;
}

// Chunks of a tile that the load cursors step through: at least SB, so that they never run past the next tile.
constexpr int tile_chunks(int K) { return (K + 63) >> 6 < SB ? SB : (K + 63) >> 6; }
// Size that a buffer descriptor states.  A cursor's scalar offset goes on behind the row where K is shorter
// than SB chunks, and by up to SB chunks where there is no next tile.  All lanes are at kOob by then, but the
// hardware takes the scalar offset from the stated size before it compares, and that difference must not
// go below zero.  Lanes with data lie inside the tensor by themselves (rows and columns are checked), so
// stating more than a short tensor has lets nothing through.
constexpr unsigned buffer_bytes(unsigned bytes) { return bytes < (unsigned)(SB * kRowB) ? (unsigned)(SB * kRowB) : bytes; }

}  // namespace wide
}  // namespace mm
