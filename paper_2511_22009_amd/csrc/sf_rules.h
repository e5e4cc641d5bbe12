// Rules of the kernels and of the host code that launches them which need no GPU, so that
// CPU tests compile and run them too. Plain C++.
#pragma once
#include <cstdint>

namespace sf {

// Epilogues of the projections.
enum EpiKind {
  EPI_QKV = 0,       // + bias, scatter to head-major q / k and transposed v
  EPI_RES_GATE = 1,  // h += gate[slot][n] * (acc + bias)
  EPI_GELU = 2,      // out = GELU_tanh(acc + bias)
  EPI_RES = 3,       // h += acc + bias
  EPI_RES_GATE_MLP = 4, // EPI_RES_GATE for the MLP down-projection (a separate kernel
                        // symbol, so profiles tell it from the attention projection)
  EPI_KVX = 5           // + bias, the context keys / transposed values of every block:
                        // column n is block (n / D) / 2, key if (n / D) even else value
};

// Tiles of the bf16 projections; what each is stands at its kernel.
enum GemmTile {
  kTile128, kTile128x288, kTile256x192,                                   // register-staged
  kHalf128x96, kHalf128, kHalf64,                                         // K slice split over wavefronts
  kPipe128x192, kPipe128, kPipe64, kPipeHalf128x192, kPipeHalf128        // fragments a K step ahead
};

// Whether the sums over K take the two halves of every 64-wide slice apart and add them at
// the end. It follows from N alone, as a row's result must not depend on how many rows are
// in the batch: outputs up to 768 wide that are whole multiples of 96 or 128 (the attention
// output and MLP down-projections of the narrower networks). All tiles of one family give the
// same bits, and M may choose among them.
constexpr bool sums_halves(int N) { return N <= 768 && (N % 96 == 0 || N % 128 == 0); }

// Whether a tile of the table is ever chosen for an epilogue (only these are compiled).
constexpr bool gemm_tile_used(GemmTile tile, EpiKind kind) {
  return tile == kTile256x192 ? kind == EPI_GELU : tile != kPipe128 || kind != EPI_GELU;
}

// What a pair of workgroups of a tile costs that a CU runs side by side, in about ns: so much
// per 64-wide slice of K, and so much once, by what the epilogue does (residual, QKV of whole
// groups of 16 tokens, QKV of other token counts, GELU). `alone` is what a last one that has
// the CU for itself takes of that, in percent.
struct TileCost {
  GemmTile tile;
  int bm, bn, slice, alone;
  int once[4];
};

// Which tile: the one with the least work on its busiest CU. A CU gets k = tiles / 256 of
// them, rounded up. Two run side by side, so they cost so much per pair and, where k is odd, a
// last one. That one is dear where only the other workgroup hides the loads: 128 x 128 with the
// fragments ahead takes 0.85 to 0.98 of the register-staged one's time at even k and 1.03 to
// 1.24 at odd k. (Where the LDS leaves room for one workgroup per CU `alone` is near 50.)
// The share that does not grow with K is twice as large for 128 x 192 as for 128 x 128, so
// below about ten slices the register-staged 128 x 128 wins where their work over K is level.
//
// The costs are fitted to launches of all four projections of one-block networks, 3832 of
// them: 25 widths from 192 to 2048, K from 192 to 8192, at 256 to 26754 rows of 256, 1023
// and 2058 tokens. The rule's choice takes 1.003 of the fastest tile's time on average, 1.19
// in the worst case; without K and the kind of epilogue it took 1.007, most of it at the two odd
// token counts (QKV 1.017). 128 x 128 throughout (outputs summed in one go) takes 1.095. Some
// times (us per launch, rows x N x K):
//   * 64 x 64: 2048 x 1024 x 4096 26.6, the next best 34.8 (128 x 128); 2048 x 896 x 896 11.8
//     and 15.3; 1024 x 2304 x 768, more than two per CU, 13.1 and 11.1.
//   * 128 x 128, register-staged, against fragments ahead: 12288 x 1024 x 4096 (k = 3) 107.6
//     and 121.4, 8192 x 1024 x 1024 (k = 2) 33.4 and 28.4. Not the latter for the GELU
//     epilogue: 12288 x 2304 x 576 45.7 and 51.0.
//   * 128 x 192 against 128 x 128: 16384 x 2304 x 768 63.4 and 70.8, 16384 x 4608 x 1152 171
//     and 182, 8192 x 1152 x 1152 35.8 and 39.3. Below K = 600 the GELU epilogue
//     weighs more: 16384 x 1792 x 448 44.0 and, 128 x 128, 40.0. (256 x 192 with the fragments
//     ahead: 69.8 and 182, at 4096 rows 22.1 against 22.3 at N 2304; not kept.)
//   * 128 x 288 and, for the GELU epilogue, 256 x 192, both register-staged with one workgroup
//     per CU, where one round of them holds everything. 128 x 288 against 128 x 192: 4096 x
//     2304 x 768 22.2 and 22.3 (in the four-slot step 21.9 and 22.7), 8192 x 1152 x 384 16.2
//     and 16.6, 4096 x 2112 x 704 20.4 and 21.1, 8192 x 1152 x 4608 88.7 and 91.2, but 2048 x
//     4608 x 1536 35.4 and 34.6. 256 x 192: 4096 x 3072 x 768 25.1, 3072 x 3840 x 960 27.5,
//     2048 x 6144 x 1536 39.2 and 40.4.
//   * halves: 64 x 64 up to two per CU: 2048 x 768 x 768 9.7 and, 128 x 96, 11.3; 4096 x 512 x
//     512 9.2 and 10.6. Beyond, 128 x 96 4096 x 768 x 3072 24.8, the next 25.8 (128 x 128
//     split); 128 x 192 with both halves in a wavefront 8192 x 768 x 768 21.6 and, 128 x 96,
//     23.2, but 12288 x 768 x 768 (1.5 rounds of it) 33.8 and 32.2; 128 x 128 12288 x 576 x 576
//     21.7 with both halves in a wavefront, 22.8 split, 25.5 with 128 x 96, 29.8 with 128 x 192.
inline GemmTile choose_gemm_tile(int M, int N, int K, int ntok, EpiKind kind) {
  constexpr long kCUs = 256;
  constexpr TileCost kHalves[] = {{kHalf64, 64, 64, 696, 58, {1052, 1052, 1052, 1052}},
                                  {kHalf128x96, 128, 96, 1852, 50, {2883, 2883, 2883, 2883}},
                                  {kHalf128, 128, 128, 1950, 54, {4247, 4247, 4247, 4247}},
                                  {kPipeHalf128x192, 128, 192, 2933, 51, {3557, 3557, 3557, 3557}},
                                  {kPipeHalf128, 128, 128, 1530, 97, {3266, 3266, 3266, 3266}}};
  constexpr TileCost kWhole[] = {{kPipe64, 64, 64, 640, 69, {861, 1915, 2171, 1299}},
                                 {kTile128, 128, 128, 1303, 59, {2126, 2573, 2614, 1921}},
                                 {kPipe128, 128, 128, 1249, 88, {2640, 2842, 3187, 2542}},
                                 {kPipe128x192, 128, 192, 1636, 76, {5692, 4018, 4433, 4841}},
                                 {kTile128x288, 128, 288, 1565, 94, {2655, 2962, 2476, 2639}},
                                 {kTile256x192, 256, 192, 1570, 100, {4650, 4650, 4650, 4650}}};
  const bool halves = sums_halves(N);
  const int epi = kind == EPI_GELU ? 3 : kind == EPI_QKV || kind == EPI_KVX ? 1 + (ntok % 16 != 0) : 0;
  const long slices = ((long)K + 63) / 64;
  long least = -1;
  GemmTile best = kTile128;
  auto take = [&](const TileCost& t) {
    if (!gemm_tile_used(t.tile, kind)) return;
    const long tiles = ((long)M + t.bm - 1) / t.bm * (((long)N + t.bn - 1) / t.bn);
    const long k = (tiles + kCUs - 1) / kCUs;
    // one per CU by its LDS (its costs are one workgroup's), and only where one round of it holds
    // everything: slower than pairs of smaller ones beyond
    if ((t.tile == kTile128x288 || t.tile == kTile256x192) && k > 1) return;
    const long pair = t.slice * slices + t.once[epi];
    const long cost = k / 2 * pair * 100 + k % 2 * pair * t.alone;
    if (least < 0 || cost < least) {
      best = t.tile;
      least = cost;
    }
  };
  if (halves)
    for (const TileCost& t : kHalves) take(t);
  else
    for (const TileCost& t : kWhole) take(t);
  return best;
}

// fp32 tiles: 64 x 64 (0) where it gives at least two workgroups per CU, 32 x 32 (1) below,
// where it spreads the rows over more of the chip. All tiles sum K in one order.
inline int choose_gemm_f32_tile(int M, int N) {
  return (((long)M + 63) / 64) * (((long)N + 63) / 64) >= 512 ? 0 : 1;
}

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
