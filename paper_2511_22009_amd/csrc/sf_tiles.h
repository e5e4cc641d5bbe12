// Tile arithmetic of the projections that needs no GPU: shared by the kernels, the host
// code that launches them and the CPU tests. Plain C++.
#pragma once

namespace sf {

// Row whose addresses an epilogue item reads when its own row m lies outside the matrix of M
// rows (or its column outside the tile): its loads are unconditional, so they need a row that
// exists. m0 is the first row of the item's pass over the tile, itself past the end where
// the matrix ends in an earlier pass.
constexpr int loaded_row(bool in, int m, int m0, int M) { return in ? m : m0 < M ? m0 : M - 1; }

}  // namespace sf
