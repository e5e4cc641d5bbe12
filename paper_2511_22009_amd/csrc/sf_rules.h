// Rules of the kernels and of the host code that launches them which need no GPU, so that
// CPU tests compile and run them too. Plain C++.
#pragma once
#include <cstdint>

namespace sf {

// Row whose addresses an epilogue item reads when its own row m lies outside the matrix of M
// rows (or its column outside the tile): its loads are unconditional, so they need a row that
// exists. m0 is the first row of the item's pass over the tile, itself past the end where
// the matrix ends in an earlier pass.
constexpr int loaded_row(bool in, int m, int m0, int M) { return in ? m : m0 < M ? m0 : M - 1; }

// Whether a step of the online softmax has to look at its scores before its probabilities
// 2^(s - offset) can stand: `top` is a lane's largest one, rounded to bf16, with its pattern
// in the high half. True whenever a score passes the offset by more than 64 or, at the first
// step, the lane's largest lies more than 64 below it; rounding to bf16 moves 2^-64 (1 - d)
// up to 2^-64 and 2^64 (1 - d) up to 2^64, so both edges belong to it, and the scores decide.
constexpr bool softmax_looks(uint32_t top, bool first) {
  constexpr uint32_t k2p64 = 0x5F800000u, k2m64 = 0x1F800000u;
  return top >= k2p64 || (first && top < k2m64 + 0x10000u);
}

}  // namespace sf
