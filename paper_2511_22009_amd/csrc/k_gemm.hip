// K3: the velocity network's dense projections, C[M][N] = A[M][K] . B[N][K]^T (both
// operands K-contiguous, weights stored [out][in]) with the epilogue fused:
//   QKV      + bias, scattered to head-major q, k and transposed v (the layout the
//            attention kernel consumes without a transpose);
//   RES_GATE h += gate[sample][n] * (acc + bias), the gate row picked by the token's
//            sample, i.e. each sample's own timestep (adaLN gate);
//   GELU     out = GELU_tanh(acc + bias);
//   RES      h += acc + bias;
//   KVX      + bias, the cross-attention keys and transposed values of every block at
//            once (one context entry per network row).
//
// bf16 path: v_mfma_f32_32x32x16_bf16 on BM x BN workgroup tiles over 64-wide K slices
// (table at the end, choice in sf_rules.h), each wavefront owning a 64x64, 64x96, 32x96 or
// 32x32 sub-tile. Operand slices reach LDS directly in a swizzled layout or, for three tiles,
// through registers into a padded one; fragment reads are free of bank conflicts in both. The
// MFMAs take the weight fragment as the first operand, so each lane ends up holding four
// adjacent output columns of one row, which the epilogues move in 8- and 16-byte pieces. fp32
// path: v_mfma_f32_16x16x4_f32 on directly staged tiles.
#include <cmath>

#include "sf_device.h"
#include "sf_rules.h"

namespace sf {

// Destination of a projection column in part `part` (= n / D) of network row r: QKV
// part which_base + part (0 q, 1 k, 2 v) of row r; KVX the key (even part) or value of
// block part / 2, stored as row r * L + block of the [rows][heads][...] layouts.
template <EpiKind KIND>
__device__ __forceinline__ void qkv_dest(const GemmArgs& a, int part, int r, int& which, int& rr) {
  if constexpr (KIND == EPI_KVX) {
    which = 1 + (part & 1);
    rr = r * a.kv_blocks + (part >> 1);
  } else {
    which = a.which_base + part;
    rr = r;
  }
}

// True when the tile of rows m0 .. m0 + BM - 1 holds a row whose entry is live (or no
// liveness is given): the caller skips the whole tile otherwise.
template <EpiKind KIND, int BM>
__device__ __forceinline__ bool tile_live(const GemmArgs& a, int m0) {
  if constexpr (KIND != EPI_KVX) return true;
  if (!a.row_live) return true;
  const int r0 = (int)fdiv((uint32_t)m0, a.div_ntok);
  const int r1 = (int)fdiv((uint32_t)(min(m0 + BM, a.M) - 1), a.div_ntok);
  for (int r = r0; r <= r1; ++r)
    if (a.row_live[r]) return true;
  return false;
}

// ------------------------------------------------------------------ bf16 / MFMA

// Largest divisor of n that is at most cap: the number of epilogue items a thread
// handles per batch.
constexpr int batch_of(int n, int cap) {
  for (int u = cap; u > 1; --u)
    if (n % u == 0) return u;
  return 1;
}

// Epilogue of the fp32 residual projections (h += gate[sample] * (acc + bias) and
// h += acc + bias) over the C tile staged in LDS (fp32, row pitch CP), four adjacent
// outputs of a row per item. Items are processed in batches: every load of a batch (C
// from LDS, bias, gate, residual) is issued before any of its results is used, with
// out-of-tile items reading a clamped in-range address, so a batch pays one memory
// latency instead of one per item. Only the stores are predicated. m0 is the first row of the
// pass, which may lie past the matrix (loaded_row).
template <EpiKind KIND, int BM, int BN, int NT>
__device__ __forceinline__ void staged_epilogue(const GemmArgs& a, const float* Cs, int CP, int m0, int n0,
                                                int tid) {
  static_assert(KIND == EPI_RES || KIND == EPI_RES_GATE || KIND == EPI_RES_GATE_MLP, "residual epilogues only");
  constexpr bool kGate = KIND == EPI_RES_GATE || KIND == EPI_RES_GATE_MLP;
  constexpr int C4 = BN / 4;
  constexpr int TOTAL = BM * C4;
  constexpr int IT = (TOTAL + NT - 1) / NT;
  constexpr int U = batch_of(IT, kGate && NT > 256 ? 4 : 8);  // four live float4 loads per gated item
  for (int i0 = 0; i0 < IT; i0 += U) {
    float4 cv[U], bv[U], hv[U], gv[U];
    int mm[U], nn[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = tid + (i0 + u) * NT;
      const int row = c / C4, c4 = c - row * C4;
      const int m = m0 + row, n = n0 + c4 * 4;
      ok[u] = (TOTAL % NT == 0 || c < TOTAL) && m < a.M && n < a.N;
      mm[u] = loaded_row(ok[u], m, m0, a.M);
      nn[u] = ok[u] ? n : 0;
      cv[u] = *(const float4*)&Cs[(ok[u] ? row : 0) * CP + (ok[u] ? c4 * 4 : 0)];
      bv[u] = *(const float4*)(a.bias + nn[u]);
      hv[u] = *(const float4*)(a.h + (size_t)mm[u] * a.ldh + nn[u]);
      if constexpr (kGate) {
        const int r = (int)fdiv((uint32_t)mm[u], a.div_ntok);
        const int slot = r < a.n_slots ? r : r - a.n_slots;
        gv[u] = *(const float4*)(a.table + (size_t)slot * a.ldt + a.gate_off + nn[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = mm[u], n = nn[u];
      const float v0 = cv[u].x + bv[u].x, v1 = cv[u].y + bv[u].y, v2 = cv[u].z + bv[u].z, v3 = cv[u].w + bv[u].w;
      float4 h = hv[u];
      if constexpr (kGate) {
        h.x += gv[u].x * v0; h.y += gv[u].y * v1; h.z += gv[u].z * v2; h.w += gv[u].w * v3;
      } else {
        h.x += v0; h.y += v1; h.z += v2; h.w += v3;
      }
      if (ok[u]) *(float4*)(a.h + (size_t)m * a.ldh + n) = h;
    }
  }
}

// The same residual epilogue with its global operands loaded ahead of time: load()
// issues, for one pass of RP tile rows, the bias, gate-row and residual loads of a
// thread's items (clamped in-range addresses for items outside the tile), so their
// latency can pass under other work; apply() combines them with the C tile staged in
// LDS, with the arithmetic of staged_epilogue, and stores.
template <EpiKind KIND, int RP, int BN, int NT>
struct ResItems {
  static_assert(KIND == EPI_RES || KIND == EPI_RES_GATE || KIND == EPI_RES_GATE_MLP || KIND == EPI_GELU ||
                    KIND == EPI_QKV || KIND == EPI_KVX,
                "epilogue kind");
  static constexpr bool kGate = KIND == EPI_RES_GATE || KIND == EPI_RES_GATE_MLP;
  static constexpr int C4 = BN / 4;
  static constexpr int TOTAL = RP * C4;
  static constexpr int IT = (TOTAL + NT - 1) / NT;
  float4 b[IT], h[IT], g[IT];

  __device__ __forceinline__ static bool item(const GemmArgs& a, int m0, int n0, int tid, int u, int& row, int& c4,
                                              int& m, int& n) {
    const int c = tid + u * NT;
    row = c / C4;
    c4 = c - row * C4;
    m = m0 + row;
    n = n0 + c4 * 4;
    return (TOTAL % NT == 0 || c < TOTAL) && m < a.M && n < a.N;
  }
  __device__ __forceinline__ void load(const GemmArgs& a, int m0, int n0, int tid) {
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      int row, c4, m, n;
      const bool ok = item(a, m0, n0, tid, u, row, c4, m, n);
      const int mm = loaded_row(ok, m, m0, a.M), nn = ok ? n : 0;
      b[u] = *(const float4*)(a.bias + nn);
      h[u] = *(const float4*)(a.h + (size_t)mm * a.ldh + nn);
      if constexpr (kGate) {
        const int r = (int)fdiv((uint32_t)mm, a.div_ntok);
        const int slot = r < a.n_slots ? r : r - a.n_slots;
        g[u] = *(const float4*)(a.table + (size_t)slot * a.ldt + a.gate_off + nn);
      }
    }
  }
  __device__ __forceinline__ void apply(const GemmArgs& a, const float* Cs, int CP, int m0, int n0, int tid) const {
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      int row, c4, m, n;
      const bool ok = item(a, m0, n0, tid, u, row, c4, m, n);
      const float4 cv = *(const float4*)&Cs[(ok ? row : 0) * CP + (ok ? c4 * 4 : 0)];
      const float v0 = cv.x + b[u].x, v1 = cv.y + b[u].y, v2 = cv.z + b[u].z, v3 = cv.w + b[u].w;
      float4 hh = h[u];
      if constexpr (kGate) {
        hh.x += g[u].x * v0; hh.y += g[u].y * v1; hh.z += g[u].z * v2; hh.w += g[u].w * v3;
      } else {
        hh.x += v0; hh.y += v1; hh.z += v2; hh.w += v3;
      }
      if (ok) *(float4*)(a.h + (size_t)m * a.ldh + n) = hh;
    }
  }
};

// Epilogue of the bf16-output projections (GELU for the MLP up-projection, the head
// split for QKV). Bias and activation are applied in registers, where every lane holds
// four adjacent columns of one row; the bf16 results are staged in LDS (8-byte writes)
// and leave in 16-byte chunks: 8 adjacent columns of a row for the GELU output and for
// q / k (a chunk never straddles a head since the head width is a multiple of 8), and 8
// adjacent tokens of one column for the transposed v.
constexpr int kEpiPad = 8;  // bf16 row pad of the staged tile (16 bytes)

template <EpiKind KIND, int BM, int BN, int TM, int TN, int NT>
__device__ __forceinline__ void bf16_epilogue(const GemmArgs& a, const f32x16 (&acc)[TM][TN], bf16* Cs,
                                              const float* bias_s, int m0, int n0, int wm, int wn, int l32, int g,
                                              bool owner, int tid) {
  constexpr int CPB = BN + kEpiPad;
  f32x4 bias[TN][4];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[j][q] = *(const f32x4*)&bias_s[(wn * TN + j) * 32 + q * 8 + g * 4];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (!owner) break;
    const int row = (wm * TM + i) * 32 + l32;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = acc[i][j][4 * q + e] + bias[j][q][e];
          if constexpr (KIND == EPI_GELU) v[e] = gelu_tanh(v[e]);
        }
        const bf16x4 o = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
        *(bf16x4*)&Cs[row * CPB + (wn * TN + j) * 32 + q * 8 + g * 4] = o;
      }
  }
  __syncthreads();
  // row-major 16-byte chunks: the whole GELU tile; the q and k columns of QKV
  constexpr int C8 = BN / 8;
  constexpr int TOTAL = BM * C8;
  constexpr int IT = (TOTAL + NT - 1) / NT;
  constexpr int U = batch_of(IT, 8);
  for (int i0 = 0; i0 < IT; i0 += U) {
    u32x4 val[U];
    int mm[U], nn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = tid + (i0 + u) * NT;
      const int row = c / C8, c8 = c - row * C8;
      const bool in = TOTAL % NT == 0 || c < TOTAL;
      mm[u] = in ? m0 + row : a.M;
      nn[u] = n0 + c8 * 8;
      val[u] = *(const u32x4*)&Cs[(in ? row : 0) * CPB + c8 * 8];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = mm[u], n = nn[u];
      if (m >= a.M || n >= a.N) continue;
      if constexpr (KIND == EPI_GELU) {
        *(u32x4*)((bf16*)a.out + (size_t)m * a.ldo + n) = val[u];
      } else {
        const int part = (int)fdiv((uint32_t)n, a.div_D);
        const int rem = n - part * a.D;
        const int head = (int)fdiv((uint32_t)rem, a.div_dh);
        const int d = rem - head * a.dh;
        const int r0 = (int)fdiv((uint32_t)m, a.div_ntok);
        const int tok = m - r0 * a.ntok;
        int which, r;
        qkv_dest<KIND>(a, part, r0, which, r);
        bf16* base = (bf16*)(which == 0 ? a.q : a.k);
        if (which < 2) *(u32x4*)(base + (((size_t)r * a.heads + head) * a.ntok + tok) * a.dh + d) = val[u];
      }
    }
  }
  if constexpr (KIND == EPI_QKV || KIND == EPI_KVX) {
    // transposed v, skipped unless the tile reaches the v columns. Plain layout: item =
    // (column, 8 consecutive rows), one 16-byte store. Items that end a network row early
    // or start unaligned go element-wise.
    if (KIND == EPI_QKV && a.which_base + (int)fdiv((uint32_t)min(n0 + BN, a.N) - 1, a.div_D) < 2) return;
    auto v_items = [&]() {
      constexpr int RG = 8;
      constexpr int VT = BM / RG * BN;
      constexpr int VIT = (VT + NT - 1) / NT;
      for (int it = 0; it < VIT; ++it) {
        const int c = tid + it * NT;
        const int rb = c / BN, col = c - rb * BN;  // adjacent lanes: adjacent columns
        const int n = n0 + col, m = m0 + rb * RG;
        if ((VT % NT != 0 && c >= VT) || n >= a.N || m >= a.M) continue;
        const int part = (int)fdiv((uint32_t)n, a.div_D);
        const int rem = n - part * a.D;
        const int head = (int)fdiv((uint32_t)rem, a.div_dh);
        const int d = rem - head * a.dh;
        const int r0 = (int)fdiv((uint32_t)m, a.div_ntok);
        const int tok = m - r0 * a.ntok;
        int which, r;
        qkv_dest<KIND>(a, part, r0, which, r);
        if (which < 2) continue;
        const bf16* cp = Cs + (rb * RG) * CPB + col;
        bf16* vt = (bf16*)a.vT + (((size_t)r * a.heads + head) * a.dh + d) * a.ldv;
        if (tok + RG <= a.ntok && m + RG <= a.M && (tok & (RG - 1)) == 0) {
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = cp[e * CPB];
          *(bf16x8*)(vt + tok) = o;
        } else {
          for (int e = 0; e < RG && m + e < a.M; ++e) {
            const int me = m + e;
            const int re0 = (int)fdiv((uint32_t)me, a.div_ntok);
            const int te = me - re0 * a.ntok;
            int we, re;
            qkv_dest<KIND>(a, part, re0, we, re);
            ((bf16*)a.vT)[(((size_t)re * a.heads + head) * a.dh + d) * a.ldv + te] =
                cp[e * CPB];
          }
        }
      }
    };
    // permuted layout: item = (8 adjacent columns, 16 consecutive rows). The 16 rows come
    // from LDS as one 16-byte read each and are transposed in registers (two bf16 per
    // v_perm); each column leaves as two 16-byte stores in the permuted key order.
    auto v_items_perm = [&]() {
      constexpr int CG = BN / 8;
      constexpr int VT = BM / 16 * CG;
      constexpr int VIT = (VT + NT - 1) / NT;
      for (int it = 0; it < VIT; ++it) {
        const int c = tid + it * NT;
        const int rb = c / CG, cg = c - rb * CG;  // adjacent lanes: adjacent column groups
        const int n = n0 + cg * 8, m = m0 + rb * 16;
        if ((VT % NT != 0 && c >= VT) || n >= a.N || m >= a.M) continue;
        const int part = (int)fdiv((uint32_t)n, a.div_D);
        const int rem = n - part * a.D;
        const int head = (int)fdiv((uint32_t)rem, a.div_dh);
        const int d0 = rem - head * a.dh;  // the 8 columns are dims d0.. of one head (dh % 8 == 0)
        const int r0 = (int)fdiv((uint32_t)m, a.div_ntok);
        const int tok = m - r0 * a.ntok;
        int which, r;
        qkv_dest<KIND>(a, part, r0, which, r);
        if (which < 2) continue;
        if (tok + 16 <= a.ntok && m + 16 <= a.M && (tok & 15) == 0) {
          u32x4 rows[16];
#pragma unroll
          for (int e = 0; e < 16; ++e) rows[e] = *(const u32x4*)&Cs[(rb * 16 + e) * CPB + cg * 8];
          bf16* vt = (bf16*)a.vT + (((size_t)r * a.heads + head) * a.dh + d0) * a.ldv + tok;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            // column j: bf16 j of every row; a word packs tokens (t0, t1) low to high
            const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
            auto pk = [&](int t0, int t1) { return __builtin_amdgcn_perm(rows[t1][j >> 1], rows[t0][j >> 1], sel); };
            // key columns tok..tok+7 hold keys 0-3, 8-11; tok+8..tok+15 keys 4-7, 12-15
            *(u32x4*)(vt + (size_t)j * a.ldv) = u32x4{pk(0, 1), pk(2, 3), pk(8, 9), pk(10, 11)};
            *(u32x4*)(vt + (size_t)j * a.ldv + 8) = u32x4{pk(4, 5), pk(6, 7), pk(12, 13), pk(14, 15)};
          }
        } else {
          // Other rows: four tokens of a network row from a multiple of 4 on stay adjacent in
          // the permuted order and leave as one 8-byte store per column, by the item that
          // holds the first of them (the others may lie in the next item, not in the next
          // tile). Tokens of a group that the tile or the network row holds in part go singly.
          // Single stores for every token count that is no multiple of 4 bounded the launch:
          // at 2058 tokens 4116 x 1008 x 336 25.6 us with them and 14.2 so, 8232 x 2880 x 960
          // 82.2 and 57.8.
          const int m_end = min(m0 + BM, a.M);
          int r0e = r0, te = tok;
          for (int e = 0; e < 16 && m + e < m_end;) {
            const int q = te & 3, first = m + e - q;
            const bool whole = first >= m0 && first + 4 <= m_end && te - q + 4 <= a.ntok;
            const int step = whole ? 4 - q : 1;
            int we, re;
            qkv_dest<KIND>(a, part, r0e, we, re);
            bf16* vt = (bf16*)a.vT + (((size_t)re * a.heads + head) * a.dh + d0) * a.ldv + vt_pos(te);
            const bf16* cp = Cs + (rb * 16 + e) * CPB + cg * 8;
            if (!whole) {
              for (int j = 0; j < 8; ++j) vt[(size_t)j * a.ldv] = cp[j];
            } else if (q == 0) {
              u32x4 rows[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) rows[u] = *(const u32x4*)&cp[u * CPB];
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
                const uint2 w = {__builtin_amdgcn_perm(rows[1][j >> 1], rows[0][j >> 1], sel),
                                 __builtin_amdgcn_perm(rows[3][j >> 1], rows[2][j >> 1], sel)};
                *(uint2*)(vt + (size_t)j * a.ldv) = w;
              }
            }
            e += step;
            te += step;
            if (te >= a.ntok) {
              te = 0;
              ++r0e;
            }
          }
        }
      }
    };
    if (a.vperm)
      v_items_perm();
    else
      v_items();
  }
}

// Block -> tile map. The hardware hands workgroup b to XCD b % 8 and each XCD has its
// own L2, so each XCD gets a contiguous range of logical tiles; inside it tiles go in
// groups of GM tile rows, M fastest, so the A rows and B columns a group touches are
// reused from one L2. Bijective for any tile count and group size. Eight rows, but four
// where that measured faster: the register-staged tiles of the QKV projection on grids of
// at least 64 tile rows or at most 8 tile columns and of the MLP up-projection on at least
// 64; the directly staged tiles whose K slice is split over wavefronts, other than for the
// MLP down-projection, on at least 64; and 128 x 192 with the fragments ahead on at least 64 tile
// rows and 10 tile columns (16384 x 2304 x 768 68.0 us with eight, 63.4 with four, 16384 x 4608 x
// 1152 174.8 and 171.3, 8192 x 2048 x 2048 103.2 and 90.4; with six columns, 16384 x 1152 x 4608,
// 167.4 and 175.5). 128 x 128 with the fragments ahead is level (0.98 to 1.02).
constexpr int kXcds = 8;
constexpr int kGroupM = 8;
__device__ __forceinline__ void tile_coords(int nbm, int nbn, int& mt, int& nt, int GM = kGroupM) {
  const int T = nbm * nbn;
  const int b = blockIdx.x;
  const int xcd = b % kXcds, local = b / kXcds;
  const int base = T / kXcds, rem = T % kXcds;
  const int logical = xcd * base + min(xcd, rem) + local;
  const int per_group = GM * nbn;
  const int group = logical / per_group;
  const int first_m = group * GM;
  const int gsize = min(GM, nbm - first_m);
  const int in = logical - group * per_group;
  mt = first_m + in % gsize;
  nt = in / gsize;
}

// The bf16 GEMM with an explicitly interleaved main loop. Operand tiles come in through
// raw buffer loads (rows past M or N and columns past K get an out-of-range offset and
// read as zeros, so the loads carry no branches). Each K step is one straight
// block: the matrix-core instructions of tile k are interleaved (sched_group_barrier)
// with the LDS fragment reads of tile k, the LDS writes of tile k+1 (already in
// registers) and the buffer loads of tile k+2, so memory work issues under the MFMAs
// instead of in stalls between them. Loader chunks past the tile (when the chunk count
// is not a multiple of the thread count) read zeros and land in a spare LDS slot, so
// the block stays branch-free.
template <int BM, int BN, int BK, int WM, int WN, EpiKind KIND>
__global__ __launch_bounds__(WM * WN * 64) void gemm_bf16_sched_kernel(GemmArgs a) {
  constexpr int NT = WM * WN * 64;
  constexpr int LDK = BK + 8;  // LDS row pitch in bf16 (a 16-byte pad)
  constexpr int TM = BM / WM / 32;
  constexpr int TN = BN / WN / 32;
  static_assert(TM * WM * 32 == BM && TN * WN * 32 == BN, "wave grid must tile the block");
  constexpr int CPR = BK / 8;
  constexpr int ATOT = BM * CPR, BTOT = BN * CPR;
  constexpr int ACH = (ATOT + NT - 1) / NT;
  constexpr int BCH = (BTOT + NT - 1) / NT;
  constexpr int AB_BYTES = 2 * (BM + BN) * LDK * 2 + 16;  // + spare slot
  constexpr bool kBf16Out = KIND == EPI_GELU || KIND == EPI_QKV || KIND == EPI_KVX;
  constexpr int CP = BN + 4;
  constexpr int C_BYTES = kBf16Out ? 0 : BM * CP * 4;  // the fp32 tile of the residual epilogues
  constexpr int SMEM = AB_BYTES > C_BYTES ? AB_BYTES : C_BYTES;
  static_assert(SMEM <= 160 * 1024, "tile does not fit in LDS");
  static_assert(BM * (BN + kEpiPad) * 2 <= SMEM, "staged bf16 tile does not fit in LDS");
  constexpr int KS = BK / 16;                 // MFMA K steps per tile
  constexpr int NMFMA = TM * TN * KS;
  constexpr int NDSR = (TM + TN) * KS;
  constexpr int NDSW = ACH + BCH;
  constexpr int NVMEM = ACH + BCH;
  __shared__ __attribute__((aligned(16))) char smem[SMEM];
  bf16* As = (bf16*)smem;
  bf16* Bs = As + 2 * BM * LDK;
  constexpr int SPARE = 2 * (BM + BN) * LDK;  // bf16 index of the spare slot

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, g = lane >> 5;
  int mt, nt;
  {
    const int nbm = (a.M + BM - 1) / BM, nbn = (a.N + BN - 1) / BN;
    tile_coords(nbm, nbn, mt, nt,
                (KIND == EPI_QKV && (nbm >= 64 || nbn <= 8)) || (KIND == EPI_GELU && nbm >= 64) ? 4 : kGroupM);
  }
  const int m0 = mt * BM, n0 = nt * BN;
  if (!tile_live<KIND, BM>(a, m0)) return;  // uniform across the workgroup
  // the tile's bias columns go to LDS now, so the epilogue does not wait on them
  __shared__ __attribute__((aligned(16))) float bias_s[kBf16Out ? BN : 4];
  if constexpr (kBf16Out) {
    for (int c = tid; c < BN / 4; c += NT) {
      const int n = n0 + 4 * c;
      *(f32x4*)&bias_s[4 * c] = n < a.N ? *(const f32x4*)(a.bias + n) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }

  const __amdgpu_buffer_rsrc_t ra_src = buffer_rsrc(a.A, (uint32_t)a.M * a.lda * 2);
  const __amdgpu_buffer_rsrc_t rb_src = buffer_rsrc(a.B, (uint32_t)a.N * a.ldb * 2);
  // per chunk: global byte offset at k = 0 (or out of range), K column, and LDS index
  // relative to the buffer base (the spare slot minus the buffer base for chunks past
  // the tile, so `buffer base + index` always lands in the spare slot)
  int a_off[ACH], b_off[BCH], a_kc[ACH], b_kc[BCH], a_lds[ACH], b_lds[BCH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    const int c = tid + i * NT, row = c / CPR;
    const bool in = c < ATOT;
    a_kc[i] = (c % CPR) * 8;
    a_lds[i] = in ? row * LDK + a_kc[i] : -1;
    a_off[i] = (in && m0 + row < a.M) ? ((m0 + row) * a.lda + a_kc[i]) * 2 : kOffOOB;
  }
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int c = tid + i * NT, row = c / CPR;
    const bool in = c < BTOT;
    b_kc[i] = (c % CPR) * 8;
    b_lds[i] = in ? row * LDK + b_kc[i] : -1;
    b_off[i] = (in && n0 + row < a.N) ? ((n0 + row) * a.ldb + b_kc[i]) * 2 : kOffOOB;
  }
  u32x4 ra[ACH], rb[BCH];
  // FAST (K a multiple of BK): every slice lies wholly inside K or wholly past it, so
  // the loads go through resources based at the slice's first column and each thread's
  // offsets are the fixed ones of k = 0 (rows past M keep the out-of-range offset); a
  // slice past K gets empty resources and reads zeros. The main loop is compiled once
  // per form and chosen by K, so neither carries a per-slice branch.
  auto gload = [&](auto fastc, int kt) {
    const int k0 = kt * BK;
    if constexpr (decltype(fastc)::value) {
      const bool live = k0 < a.K;
      const __amdgpu_buffer_rsrc_t ra1 =
          buffer_rsrc((const char*)a.A + 2 * (size_t)k0, live ? (uint32_t)a.M * a.lda * 2 - 2 * k0 : 0u);
      const __amdgpu_buffer_rsrc_t rb1 =
          buffer_rsrc((const char*)a.B + 2 * (size_t)k0, live ? (uint32_t)a.N * a.ldb * 2 - 2 * k0 : 0u);
#pragma unroll
      for (int i = 0; i < ACH; ++i) ra[i] = buffer_load16(ra1, a_off[i]);
#pragma unroll
      for (int i = 0; i < BCH; ++i) rb[i] = buffer_load16(rb1, b_off[i]);
      return;
    }
#pragma unroll
    for (int i = 0; i < ACH; ++i)
      ra[i] = buffer_load16(ra_src, (k0 + a_kc[i] < a.K && a_off[i] != kOffOOB) ? a_off[i] + 2 * k0 : kOffOOB);
#pragma unroll
    for (int i = 0; i < BCH; ++i)
      rb[i] = buffer_load16(rb_src, (k0 + b_kc[i] < a.K && b_off[i] != kOffOOB) ? b_off[i] + 2 * k0 : kOffOOB);
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      const int idx = (ATOT % NT == 0 || a_lds[i] >= 0) ? buf * BM * LDK + a_lds[i] : SPARE;
      *(u32x4*)&As[idx] = ra[i];
    }
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
      const int idx = (BTOT % NT == 0 || b_lds[i] >= 0) ? buf * BN * LDK + b_lds[i] : SPARE - 2 * BM * LDK;
      *(u32x4*)&Bs[idx] = rb[i];
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  auto step = [&](auto fastc, int cur, int kt, bool write_next, bool load_next) {
    const bf16* Ab = As + cur * BM * LDK + (wm * TM * 32 + l32) * LDK + g * 8;
    const bf16* Bb = Bs + cur * BN * LDK + (wn * TN * 32 + l32) * LDK + g * 8;
    bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) af[0][i] = *(const bf16x8*)(Ab + i * 32 * LDK);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[0][j] = *(const bf16x8*)(Bb + j * 32 * LDK);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const int cb = kk & 1;
      if (kk + 1 < KS) {
#pragma unroll
        for (int i = 0; i < TM; ++i) af[cb ^ 1][i] = *(const bf16x8*)(Ab + i * 32 * LDK + (kk + 1) * 16);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[cb ^ 1][j] = *(const bf16x8*)(Bb + j * 32 * LDK + (kk + 1) * 16);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[cb][j], af[cb][i], acc[i][j], 0, 0, 0);
    }
    if (write_next) lstore(cur ^ 1);
    if (load_next) gload(fastc, kt + 2);
    // interleave: the fragment reads ahead of their MFMAs over the first half of the
    // MFMAs, the LDS writes and global loads over the second half
    constexpr int H1 = NMFMA / 2, H2 = NMFMA - NMFMA / 2;
#pragma unroll
    for (int i = 0; i < H1; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, (NDSR + H1 - 1) / H1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < H2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x200, (NDSW + H2 - 1) / H2, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, (NVMEM + H2 - 1) / H2, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  };

  const int nk = (a.K + BK - 1) / BK;
  auto main_loop = [&](auto fastc) {
    gload(fastc, 0);
    lstore(0);
    if (nk > 1) gload(fastc, 1);
    __syncthreads();
    int kt = 0;
    for (; kt + 2 < nk; ++kt) {
      step(fastc, kt & 1, kt, true, true);
      __syncthreads();
    }
    if (kt + 1 < nk) {
      step(fastc, kt & 1, kt, true, false);
      __syncthreads();
      ++kt;
    }
    step(fastc, kt & 1, kt, false, false);
    __syncthreads();
  };
  if (a.K % BK == 0)
    main_loop(std::true_type{});
  else
    main_loop(std::false_type{});

  // The MFMAs compute C^T blocks (weights as the first operand), so in acc[i][j]
  // lane (l32, g) holds row (wm*TM + i)*32 + l32 of the tile and, in registers
  // 4q..4q+3, the four adjacent columns (wn*TN + j)*32 + 8q + 4g + 0..3.
  if constexpr (kBf16Out) {
    bf16_epilogue<KIND, BM, BN, TM, TN, NT>(a, acc, (bf16*)smem, bias_s, m0, n0, wm, wn, l32, g, true, tid);
  } else {
    float* Cs = (float*)smem;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *(f32x4*)&Cs[((wm * TM + i) * 32 + l32) * CP + (wn * TN + j) * 32 + q * 8 + g * 4] = v;
        }
    __syncthreads();
    staged_epilogue<KIND, BM, BN, NT>(a, Cs, CP, m0, n0, tid);
  }
}

// ------------------------------------------------- bf16 / MFMA, direct LDS staging
//
// The same tile computation with operand slices moved by buffer_load ... lds straight
// from global memory into a ring of STAGES LDS buffers (no VGPR round trip, no LDS
// write instructions), fetched STAGES - 1 slices ahead.
//
// Each stage is its own __shared__ variable and the main loop is unrolled by STAGES, so
// every LDS access names one variable: the compiler then tells the in-flight loads into
// other stages apart from the stage being read and waits only for the right ones.
// The loop's barrier is a bare s_barrier (ordered by compiler-only fences) after an
// explicit wait for this slice's loads: the workgroup-scope release fence of
// __syncthreads would wait for every outstanding LDS-bound load, i.e. for all stages.
//
// Stage layout: rows of BK bf16 without padding, 16-byte chunks swizzled by dma_swz.

template <int BM, int BN, int BK, int WM, int WN, int KSPLIT, int STAGES, EpiKind KIND>
__global__ __launch_bounds__(WM * WN * KSPLIT * 64) void gemm_bf16_dma_kernel(GemmArgs a) {
  constexpr int NT = WM * WN * KSPLIT * 64;
  constexpr int TM = BM / WM / 32;
  constexpr int TN = BN / WN / 32;
  static_assert(TM * WM * 32 == BM && TN * WN * 32 == BN, "wave grid must tile the block");
  constexpr int CPR = BK / 8;
  constexpr int ATOT = BM * CPR, BTOT = BN * CPR;
  static_assert(ATOT % 64 == 0 && BTOT % 64 == 0, "whole wavefronts of 16-byte chunks per slice");
  constexpr int ACH = (ATOT + NT - 1) / NT, BCH = (BTOT + NT - 1) / NT, LPT = ACH + BCH;
  constexpr int KS = BK / 16 / KSPLIT;  // MFMA K steps per slice and wavefront
  static_assert(KS * 16 * KSPLIT == BK, "K split must divide the K slice");
  static_assert(STAGES == 3 || STAGES == 4, "three or four stages");
  constexpr bool kBf16Out = KIND == EPI_GELU || KIND == EPI_QKV || KIND == EPI_KVX;
  // each stage buffer also holds, after the main loop, one row block of the K-split
  // partial sums, one half of the fp32 output tile, or the whole bf16 output tile
  constexpr int CP = BN + 4;
  constexpr int RP = BM / 2;
  constexpr int SLICE = (BM + BN) * BK * 2;
  // K-split partials: MFMA block b = i * TN + j of every first-set wavefront (4 KB each)
  // goes to stage b % STAGES at block slot b / STAGES
  constexpr int PBLK = WM * WN * 16 * 64 * 4;
  constexpr int PART = KSPLIT == 2 ? (TM * TN + STAGES - 1) / STAGES * PBLK : 0;
  constexpr int EPI = kBf16Out ? BM * (BN + kEpiPad) * 2 : RP * CP * 4;
  constexpr int SBA = SLICE > PART ? (SLICE > EPI ? SLICE : EPI) : (PART > EPI ? PART : EPI);
  static_assert(KSPLIT == 1 || KSPLIT == 2, "K split of one or two");
  static_assert(STAGES * SBA + (kBf16Out ? BN * 4 : 16) <= 160 * 1024, "stages do not fit in LDS");
  constexpr int NMFMA = TM * TN * KS;
  constexpr int NDSR = (TM + TN) * KS;
  __shared__ __attribute__((aligned(16))) char st0[SBA];
  __shared__ __attribute__((aligned(16))) char st1[SBA];
  __shared__ __attribute__((aligned(16))) char st2[SBA];
  __shared__ __attribute__((aligned(16))) char st3[STAGES > 3 ? SBA : 16];
  // destination of the loads of wavefronts whose chunk round lies past the tile (they
  // read zeros; nothing reads this back)
  constexpr bool kSpare = ATOT % NT != 0 || BTOT % NT != 0;
  __shared__ __attribute__((aligned(16))) char spare[kSpare ? 1024 : 16];
  auto stage = [&](auto s) -> char* {
    constexpr int S = decltype(s)::value % STAGES;
    if constexpr (S == 0) return st0;
    else if constexpr (S == 1) return st1;
    else if constexpr (S == 2) return st2;
    else return st3;
  };

  const int tid = threadIdx.x;
  // the wavefront index is uniform: kept scalar, so the LDS destinations of the direct
  // loads (M0) need no readfirstlane
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / (WM * WN), wmn = wave - kg * (WM * WN);
  const int wm = wmn / WN, wn = wmn % WN;
  const int l32 = lane & 31, g = lane >> 5;
  int mt, nt;
  {
    const int nbm = (a.M + BM - 1) / BM, nbn = (a.N + BN - 1) / BN;
    tile_coords(nbm, nbn, mt, nt, nbm >= 64 && KIND != EPI_RES_GATE_MLP ? 4 : kGroupM);
  }
  const int m0 = mt * BM, n0 = nt * BN;
  if (!tile_live<KIND, BM>(a, m0)) return;  // uniform across the workgroup
  __shared__ __attribute__((aligned(16))) float bias_s[kBf16Out ? BN : 4];
  if constexpr (kBf16Out) {
    for (int c = tid; c < BN / 4; c += NT) {
      const int n = n0 + 4 * c;
      *(f32x4*)&bias_s[4 * c] = n < a.N ? *(const f32x4*)(a.bias + n) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }

  const __amdgpu_buffer_rsrc_t ra_src = buffer_rsrc(a.A, (uint32_t)a.M * a.lda * 2);
  const __amdgpu_buffer_rsrc_t rb_src = buffer_rsrc(a.B, (uint32_t)a.N * a.ldb * 2);
  // load i of a thread fills LDS chunk position i * NT + tid of the A (or B) part of a
  // stage, i.e. tile row p / CPR at chunk position p % CPR, which holds K chunk
  // (p % CPR) ^ swz(row); per load: that K column and the byte offset at k = 0
  int a_off[ACH], b_off[BCH], a_kc[ACH], b_kc[BCH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    const int p = tid + i * NT, row = p / CPR;
    a_kc[i] = ((p % CPR) ^ dma_swz<CPR>(row)) * 8;
    a_off[i] = p < ATOT && m0 + row < a.M ? ((m0 + row) * a.lda + a_kc[i]) * 2 : kOffOOB;
  }
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int p = tid + i * NT, row = p / CPR;
    b_kc[i] = ((p % CPR) ^ dma_swz<CPR>(row)) * 8;
    b_off[i] = p < BTOT && n0 + row < a.N ? ((n0 + row) * a.ldb + b_kc[i]) * 2 : kOffOOB;
  }
  // slice kt into stage buffer sb: every thread issues exactly LPT loads (past the end
  // of K they read zeros), each wavefront's 64 lanes filling one contiguous kilobyte
  // FAST (K a multiple of BK): every slice lies wholly inside K or wholly past it, so
  // the loads go through resources based at the slice's first column and each thread's
  // offsets are the fixed ones of k = 0 (rows past M keep the out-of-range offset); a
  // slice past K gets empty resources and reads zeros without touching memory
  auto issue = [&](auto fast, char* sb, int kt) {
    const int k0 = kt * BK;
    if constexpr (decltype(fast)::value) {
      const bool live = k0 < a.K;
      const __amdgpu_buffer_rsrc_t ra =
          buffer_rsrc((const char*)a.A + 2 * (size_t)k0, live ? (uint32_t)a.M * a.lda * 2 - 2 * k0 : 0u);
      const __amdgpu_buffer_rsrc_t rb =
          buffer_rsrc((const char*)a.B + 2 * (size_t)k0, live ? (uint32_t)a.N * a.ldb * 2 - 2 * k0 : 0u);
#pragma unroll
      for (int i = 0; i < ACH; ++i) {
        const bool in = ATOT % NT == 0 || i * NT + wave * 64 < ATOT;
        buffer_load16_lds(ra, in ? sb + (i * NT + wave * 64) * 16 : spare, a_off[i]);
      }
#pragma unroll
      for (int i = 0; i < BCH; ++i) {
        const bool in = BTOT % NT == 0 || i * NT + wave * 64 < BTOT;
        buffer_load16_lds(rb, in ? sb + ATOT * 16 + (i * NT + wave * 64) * 16 : spare, b_off[i]);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      const bool in = ATOT % NT == 0 || i * NT + wave * 64 < ATOT;
      buffer_load16_lds(ra_src, in ? sb + (i * NT + wave * 64) * 16 : spare,
                        (k0 + a_kc[i] < a.K && a_off[i] != kOffOOB) ? a_off[i] + 2 * k0 : kOffOOB);
    }
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
      const bool in = BTOT % NT == 0 || i * NT + wave * 64 < BTOT;
      buffer_load16_lds(rb_src, in ? sb + ATOT * 16 + (i * NT + wave * 64) * 16 : spare,
                        (k0 + b_kc[i] < a.K && b_off[i] != kOffOOB) ? b_off[i] + 2 * k0 : kOffOOB);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // this lane's rows all have the swizzle of row l32 (row blocks are 32 apart); its
  // fragment of MFMA K step kk is K chunk c0 + 2 kk
  const int sw = dma_swz<CPR>(l32);
  const int c0 = 2 * kg * KS + g;
  const int a_row = (wm * TM * 32 + l32) * CPR;
  const int b_row = ATOT + (wn * TN * 32 + l32) * CPR;
  // one K slice: wait for this slice's loads (the later slices' STAGES - 2 stay in
  // flight) and for this thread's LDS accesses, barrier, then the MFMAs on stage S
  // interleaved with the fragment reads and with the loads of slice kt + STAGES - 1
  // into the stage read in the previous step
  constexpr int kWait = waitcnt_vm_lgkm0<(STAGES - 2) * LPT>();
  auto step = [&](auto fast, auto s, int kt) {
    constexpr int S = decltype(s)::value;
    __builtin_amdgcn_s_waitcnt(kWait);
    bare_barrier();
    const char* cur = stage(std::integral_constant<int, S>{});
    bf16x8 af[2][TM], bfr[2][TN];
    auto frag = [&](int row_base, int blk, int kk) {
      return *(const bf16x8*)(cur + (row_base + blk * 32 * CPR + ((c0 + 2 * kk) ^ sw)) * 16);
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) af[0][i] = frag(a_row, i, 0);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[0][j] = frag(b_row, j, 0);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const int cb = kk & 1;
      if (kk + 1 < KS) {
#pragma unroll
        for (int i = 0; i < TM; ++i) af[cb ^ 1][i] = frag(a_row, i, kk + 1);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[cb ^ 1][j] = frag(b_row, j, kk + 1);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[cb][j], af[cb][i], acc[i][j], 0, 0, 0);
    }
    issue(fast, stage(std::integral_constant<int, S + STAGES - 1>{}), kt + STAGES - 1);
    constexpr int H1 = NMFMA / 2, H2 = NMFMA - NMFMA / 2;
#pragma unroll
    for (int i = 0; i < H1; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, (NDSR + H1 - 1) / H1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < H2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x020, (LPT + H2 - 1) / H2, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  };

  const int nk = (a.K + BK - 1) / BK;
  auto main_loop = [&](auto fast) {
    issue(fast, stage(std::integral_constant<int, 0>{}), 0);
    issue(fast, stage(std::integral_constant<int, 1>{}), 1);
    if constexpr (STAGES > 3) issue(fast, stage(std::integral_constant<int, 2>{}), 2);
    // whole rounds of STAGES steps in a loop with one exit (early exits inside the round
    // would give the loop header a path on which the stage it reads was just issued),
    // then the remaining steps
    int kt = 0;
    for (; kt + STAGES <= nk; kt += STAGES) {
      step(fast, std::integral_constant<int, 0>{}, kt);
      step(fast, std::integral_constant<int, 1>{}, kt + 1);
      step(fast, std::integral_constant<int, 2>{}, kt + 2);
      if constexpr (STAGES > 3) step(fast, std::integral_constant<int, 3>{}, kt + 3);
    }
    if (kt < nk) step(fast, std::integral_constant<int, 0>{}, kt);
    if (kt + 1 < nk) step(fast, std::integral_constant<int, 1>{}, kt + 1);
    if constexpr (STAGES > 3)
      if (kt + 2 < nk) step(fast, std::integral_constant<int, 2>{}, kt + 2);
  };
  if (a.K % BK == 0)
    main_loop(std::true_type{});
  else
    main_loop(std::false_type{});
  // the zero-filling loads past K land before the buffers are reused
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // the residual epilogues' global operands (bias, gate row, residual) for both row
  // halves are loaded now: their latency passes under the K-split merge and the staging
  ResItems<KIND, RP, BN, NT> pre[2];
  if constexpr (!kBf16Out) {
    pre[0].load(a, m0, n0, tid);
    pre[1].load(a, m0 + RP, n0, tid);
  }

  if constexpr (KSPLIT == 2) {
    // the second K half's partial sums go through LDS (lane-major, so each lane reads
    // back exactly what its partner wrote) to the first half's wavefronts: one fixed
    // order (first half + second half) for every element
    auto part = [&](int i, int j, int q) -> f32x4* {
      const int b = i * TN + j;
      const int st = b % STAGES;
      char* base = st == 0 ? st0 : st == 1 ? st1 : st == 2 ? st2 : st3;
      return (f32x4*)(base + (b / STAGES) * PBLK) + (wmn * 4 + q) * 64 + lane;
    };
    if (kg == 1) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *part(i, j, q) = f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = *part(i, j, q);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
          }
    }
    __syncthreads();
  }
  if constexpr (kBf16Out) {
    bf16_epilogue<KIND, BM, BN, TM, TN, NT>(a, acc, (bf16*)st0, bias_s, m0, n0, wm, wn, l32, g, kg == 0, tid);
  } else {
    // the two row halves of the tile staged in stages 0 and 1 under one barrier
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      float* Cs = (float*)(p == 0 ? st0 : st1);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int rb0 = (wm * TM + i) * 32;
        if (kg != 0 || rb0 < p * RP || rb0 >= (p + 1) * RP) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            *(f32x4*)&Cs[(rb0 - p * RP + l32) * CP + (wn * TN + j) * 32 + q * 8 + g * 4] = v;
          }
      }
    }
    __syncthreads();
    pre[0].apply(a, (const float*)st0, CP, m0, n0, tid);
    pre[1].apply(a, (const float*)st1, CP, m0 + RP, n0, tid);
  }
}

// ---------------------------------------- bf16 / MFMA, direct staging, fragments ahead
//
// The directly staged tile computation with every wavefront owning a sub-tile over the
// whole K slice (64x96, 64x64 or 32x96) and its fragments read one K step ahead, across
// the slice boundary too. The last K step of a slice has its operands in registers when
// the workgroup meets at the slice's one barrier, so that barrier frees the stage just
// read: its refill (STAGES slices ahead) and the reads of the next slice's first
// fragments go out under that step's MFMAs, and no MFMA waits for an LDS round trip.
//
// What bounds it: with the loads left out a 16384 x 1152 x 4608 launch of 128 x 192 tiles
// takes 126 us (1380 TFLOP/s), with the MFMAs left out 170, with both 184; with every load
// an L2 hit 153. So operand loads past L2 bind, and fewer operand bytes per output or more
// workgroups per CU help while the order of the loop does not. A prefetch of the next
// slices into L2 was worth 4 % on one shape and cost 5 % on others: not kept.
//
// HALVES: the two halves of every K slice accumulate apart and are added at the end, the
// order of gemm_bf16_dma_kernel with a K split of two, so both give the same bits.
template <int BM, int BN, int WM, int WN, int STAGES, int MINW, bool HALVES, EpiKind KIND>
__global__ __launch_bounds__(WM * WN * 64, MINW) void gemm_bf16_pipe_kernel(GemmArgs a) {
  constexpr int NT = WM * WN * 64, BK = 64, CPR = 8, KS = 4;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  static_assert(TM * WM * 32 == BM && TN * WN * 32 == BN, "wave grid must tile the block");
  constexpr int ATOT = BM * CPR, BTOT = BN * CPR;
  static_assert(ATOT % NT == 0 && BTOT % NT == 0, "whole rounds of chunks per slice");
  constexpr int ACH = ATOT / NT, BCH = BTOT / NT, LPT = ACH + BCH;
  static_assert(STAGES == 2 || STAGES == 3 || STAGES == 4, "two to four stages");
  constexpr bool kBf16Out = KIND == EPI_GELU || KIND == EPI_QKV || KIND == EPI_KVX;
  constexpr int SLICE = (ATOT + BTOT) * 16;
  // after the main loop a stage buffer holds one half of the bf16 tile, or as many rows of
  // the fp32 tile as fit
  constexpr int HB = WM > 1 ? 2 : 1;  // bf16 halves
  constexpr int EPIT = BM / HB * (BN + kEpiPad) * 2;
  constexpr int EPIB = EPIT + BN * 4;  // and, in the first one, the tile's bias
  constexpr int CP = BN + 4;
  // fp32: one 32-row block of WPP wavefront rows per pass
  constexpr int WFIT = SLICE / (32 * CP * 4);
  constexpr int WPP = WFIT >= WM ? WM : WFIT >= 2 && WM % 2 == 0 ? 2 : 1;
  constexpr int EPIF = WPP * 32 * CP * 4;
  constexpr int EPI = kBf16Out ? EPIB : EPIF;
  constexpr int SBA = SLICE > EPI ? SLICE : EPI;
  static_assert(STAGES * SBA <= 160 * 1024, "stages do not fit in LDS");
  __shared__ __attribute__((aligned(16))) char st0[SBA];
  __shared__ __attribute__((aligned(16))) char st1[SBA];
  __shared__ __attribute__((aligned(16))) char st2[STAGES > 2 ? SBA : 16];
  __shared__ __attribute__((aligned(16))) char st3[STAGES > 3 ? SBA : 16];
  auto stage = [&](auto s) -> char* {
    constexpr int S = decltype(s)::value % STAGES;
    if constexpr (S == 0) return st0;
    else if constexpr (S == 1) return st1;
    else if constexpr (S == 2) return st2;
    else return st3;
  };
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, g = lane >> 5;
  int mt, nt;
  {
    const int nbm = (a.M + BM - 1) / BM, nbn = (a.N + BN - 1) / BN;
    tile_coords(nbm, nbn, mt, nt, BN == 192 && !HALVES && nbm >= 64 && nbn >= 10 ? 4 : kGroupM);
  }
  const int m0 = mt * BM, n0 = nt * BN;
  if (!tile_live<KIND, BM>(a, m0)) return;  // uniform across the workgroup
  // the tile's bias columns are fetched now and put into LDS after the main loop
  static_assert(BN / 4 <= NT, "one bias load per thread");
  f32x4 bias_v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (kBf16Out) {
    if (tid < BN / 4 && n0 + 4 * tid < a.N) bias_v = *(const f32x4*)(a.bias + n0 + 4 * tid);
  }
  int a_off[ACH], b_off[BCH], a_kc[ACH], b_kc[BCH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    const int p = tid + i * NT, row = p / CPR;
    a_kc[i] = ((p % CPR) ^ dma_swz<CPR>(row)) * 8;
    a_off[i] = m0 + row < a.M ? ((m0 + row) * a.lda + a_kc[i]) * 2 : kOffOOB;
  }
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int p = tid + i * NT, row = p / CPR;
    b_kc[i] = ((p % CPR) ^ dma_swz<CPR>(row)) * 8;
    b_off[i] = n0 + row < a.N ? ((n0 + row) * a.ldb + b_kc[i]) * 2 : kOffOOB;
  }
  auto issue = [&](auto fast, char* sb, int kt) __attribute__((always_inline)) {
    const int k0 = kt * BK;
    const bool live = k0 < a.K;
    const __amdgpu_buffer_rsrc_t ra =
        buffer_rsrc((const char*)a.A + 2 * (size_t)k0, live ? (uint32_t)a.M * a.lda * 2 - 2 * k0 : 0u);
    const __amdgpu_buffer_rsrc_t rb =
        buffer_rsrc((const char*)a.B + 2 * (size_t)k0, live ? (uint32_t)a.N * a.ldb * 2 - 2 * k0 : 0u);
    constexpr bool F = decltype(fast)::value;
#pragma unroll
    for (int i = 0; i < ACH; ++i)
      buffer_load16_lds(ra, sb + (i * NT + wave * 64) * 16, F || k0 + a_kc[i] < a.K ? a_off[i] : kOffOOB);
#pragma unroll
    for (int i = 0; i < BCH; ++i)
      buffer_load16_lds(rb, sb + (ATOT + i * NT + wave * 64) * 16, F || k0 + b_kc[i] < a.K ? b_off[i] : kOffOOB);
  };

  constexpr int NH = HALVES ? 2 : 1;
  f32x16 accs[NH][TM][TN];
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) accs[h][i][j][r] = 0.0f;
  const int sw = dma_swz<CPR>(l32);
  const int a_row = (wm * TM * 32 + l32) * CPR;
  const int b_row = ATOT + (wn * TN * 32 + l32) * CPR;
  bf16x8 af[2][TM], bfr[2][TN];
  auto frags = [&](const char* cur, int buf, int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i) af[buf][i] = *(const bf16x8*)(cur + (a_row + i * 32 * CPR + ((g + 2 * kk) ^ sw)) * 16);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[buf][j] = *(const bf16x8*)(cur + (b_row + j * 32 * CPR + ((g + 2 * kk) ^ sw)) * 16);
  };
  auto mfmas = [&](int buf, int kk) __attribute__((always_inline)) {
    const int h = HALVES ? kk / 2 : 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        accs[h][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[buf][j], af[buf][i], accs[h][i][j], 0, 0, 0);
  };
  constexpr int NM = TM * TN, ND = TM + TN;
  auto step = [&](auto fast, auto s, int kt) __attribute__((always_inline)) {
    constexpr int S = decltype(s)::value;
    const char* cur = stage(std::integral_constant<int, S>{});
#pragma unroll
    for (int kk = 0; kk + 1 < KS; ++kk) {
      frags(cur, (kk + 1) & 1, kk + 1);
      mfmas(kk & 1, kk);
    }
    // reads spread ahead of the MFMAs of their step
#pragma unroll
    for (int i = 0; i < (KS - 1) * ND; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, NM >= ND ? NM / ND : 1, 0);
    }
    // the last K step's operands are in registers: once every wavefront is here the stage
    // can be refilled, and the next slice's first operands are read under this K step's MFMAs
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0<(STAGES - 2) * LPT>());
    bare_barrier();
    issue(fast, stage(std::integral_constant<int, S>{}), kt + STAGES);
    frags(stage(std::integral_constant<int, S + 1>{}), 0, 0);
    mfmas((KS - 1) & 1, KS - 1);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, (ND + NM - 1) / NM, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, (LPT + NM - 1) / NM, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  };
  const int nk = (a.K + BK - 1) / BK;
  auto main_loop = [&](auto fast) __attribute__((always_inline)) {
    issue(fast, stage(std::integral_constant<int, 0>{}), 0);
    issue(fast, stage(std::integral_constant<int, 1>{}), 1);
    if constexpr (STAGES > 2) issue(fast, stage(std::integral_constant<int, 2>{}), 2);
    if constexpr (STAGES > 3) issue(fast, stage(std::integral_constant<int, 3>{}), 3);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0<(STAGES - 1) * LPT>());
    bare_barrier();
    frags(stage(std::integral_constant<int, 0>{}), 0, 0);
    int kt = 0;
    for (; kt + STAGES <= nk; kt += STAGES) {
      step(fast, std::integral_constant<int, 0>{}, kt);
      step(fast, std::integral_constant<int, 1>{}, kt + 1);
      if constexpr (STAGES > 2) step(fast, std::integral_constant<int, 2>{}, kt + 2);
      if constexpr (STAGES > 3) step(fast, std::integral_constant<int, 3>{}, kt + 3);
    }
    if (kt < nk) step(fast, std::integral_constant<int, 0>{}, kt);
    if constexpr (STAGES > 2)
      if (kt + 1 < nk) step(fast, std::integral_constant<int, 1>{}, kt + 1);
    if constexpr (STAGES > 3)
      if (kt + 2 < nk) step(fast, std::integral_constant<int, 2>{}, kt + 2);
  };
  if (a.K % BK == 0)
    main_loop(std::true_type{});
  else
    main_loop(std::false_type{});
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  f32x16(&acc)[TM][TN] = accs[0];
  if constexpr (HALVES) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += accs[1][i][j][r];
  }
  if constexpr (kBf16Out) {
    float* bias_s = (float*)(st0 + EPIT);
    if (tid < BN / 4) *(f32x4*)&bias_s[4 * tid] = bias_v;
    __syncthreads();
#pragma unroll
    for (int h = 0; h < HB; ++h)
      bf16_epilogue<KIND, BM / HB, BN, TM, TN, NT>(a, acc, (bf16*)(h == 0 ? st0 : st1), bias_s, m0 + h * (BM / HB), n0,
                                                   wm - h * (WM / HB), wn, l32, g, wm / (WM / HB) == h, tid);
  } else {
#pragma unroll
    for (int p = 0; p < TM * (WM / WPP); ++p) {
      const int i = p / (WM / WPP), w0 = p % (WM / WPP) * WPP;
      float* Cs = (float*)(p % 2 == 0 ? st0 : st1);
      if (wm >= w0 && wm < w0 + WPP) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            *(f32x4*)&Cs[((wm - w0) * 32 + l32) * CP + (wn * TN + j) * 32 + q * 8 + g * 4] = v;
          }
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < WPP; ++w)
        staged_epilogue<KIND, 32, BN, NT>(a, Cs + w * 32 * CP, CP, m0 + ((w0 + w) * TM + i) * 32, n0, tid);
    }
  }
}

// ------------------------------------------------------------------ fp32 / MFMA
//
// fp32 projections on v_mfma_f32_16x16x4_f32 (fp32 operands and sums). Operand
// slices of 32 columns go global -> LDS directly into a ring of three stages, two slices
// ahead, in the layout of the bf16 kernel above (rows of eight 16-byte chunks, swizzled).
// An MFMA contracts four values, one per lane group g = lane / 16; a lane reads whole
// chunks (chunk 4 kk + g of its row) and feeds MFMA (kk, e) their element e, so that MFMA
// sums columns 16 kk + 4 g + e of the slice. The four elements e have sums of their own, added
// at the end: a quarter of the chain's length and so less rounding (velocity of two 512^2
// blocks 2.4e-7 off 64 bits, 3.1e-7 to 3.7e-7 in one chain, for 1.5 % of the call's time).
// Every tile shape sums K in this one order, so the choice of a tile, by M too, changes no
// result bit.
//
// The weights are the first operand: lane (l16, g) ends up with four adjacent output
// columns 4 g .. 4 g + 3 of row l16 of each 16 x 16 block, which leave as 16-byte accesses
// straight from registers (single stores for the transposed v, whose lanes hold adjacent
// tokens). The matrix cores bound it: 64 FLOP per cycle and SIMD against 16 B/clk of
// operand loads per CU for the 64 x 64 tile. 4096 x 768 x 3072: 152 us, 127 TFLOP/s of the
// 153 that a large product reaches, against 396 us for a 64 x 64 tile of vector FMAs;
// 420 x 192 x 768: 8.1 against 77 us.
template <EpiKind KIND>
__device__ __forceinline__ void f32_epilogue4(const GemmArgs& a, int m, int n, const f32x4& acc) {
  const f32x4 b = *(const f32x4*)(a.bias + n);
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = acc[e] + b[e];
  if constexpr (KIND == EPI_QKV || KIND == EPI_KVX) {
    // the four columns belong to one head (head widths are multiples of eight)
    const int part = (int)fdiv((uint32_t)n, a.div_D);
    const int rem = n - part * a.D;
    const int head = (int)fdiv((uint32_t)rem, a.div_dh);
    const int d = rem - head * a.dh;
    const int r0 = (int)fdiv((uint32_t)m, a.div_ntok);
    const int tok = m - r0 * a.ntok;
    int which, r;
    qkv_dest<KIND>(a, part, r0, which, r);
    const size_t bh = (size_t)r * a.heads + head;
    if (which < 2) *(f32x4*)((float*)(which == 0 ? a.q : a.k) + (bh * a.ntok + tok) * a.dh + d) = v;
    if (which >= 2) {
      float* vt = (float*)a.vT + (bh * a.dh + d) * a.ldv + tok;
#pragma unroll
      for (int e = 0; e < 4; ++e) vt[(size_t)e * a.ldv] = v[e];
    }
  } else if constexpr (KIND == EPI_GELU) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
    *(f32x4*)((float*)a.out + (size_t)m * a.ldo + n) = v;
  } else {
    f32x4* hp = (f32x4*)(a.h + (size_t)m * a.ldh + n);
    f32x4 h = *hp;
    if constexpr (KIND == EPI_RES_GATE || KIND == EPI_RES_GATE_MLP) {
      const int r = (int)fdiv((uint32_t)m, a.div_ntok);
      const int slot = r < a.n_slots ? r : r - a.n_slots;
      const f32x4 g = *(const f32x4*)(a.table + (size_t)slot * a.ldt + a.gate_off + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] += g[e] * v[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] += v[e];
    }
    *hp = h;
  }
}

template <int BM, int BN, int WM, int WN, EpiKind KIND>
__global__ __launch_bounds__(WM * WN * 64) void gemm_f32_kernel(GemmArgs a) {
  constexpr int NT = WM * WN * 64, BK = 32, CPR = 8, STAGES = 3;
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  static_assert(TM * WM * 16 == BM && TN * WN * 16 == BN, "wave grid must tile the block");
  constexpr int ATOT = BM * CPR, BTOT = BN * CPR;
  static_assert(ATOT % NT == 0 && BTOT % NT == 0, "whole rounds of chunks per slice");
  constexpr int ACH = ATOT / NT, BCH = BTOT / NT, LPT = ACH + BCH;
  __shared__ __attribute__((aligned(16))) char st0[(ATOT + BTOT) * 16];
  __shared__ __attribute__((aligned(16))) char st1[(ATOT + BTOT) * 16];
  __shared__ __attribute__((aligned(16))) char st2[(ATOT + BTOT) * 16];
  auto stage = [&](auto s) -> char* {
    constexpr int S = decltype(s)::value % STAGES;
    if constexpr (S == 0) return st0;
    else if constexpr (S == 1) return st1;
    else return st2;
  };
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l16 = lane & 15, g = lane >> 4;
  int mt, nt;
  tile_coords((a.M + BM - 1) / BM, (a.N + BN - 1) / BN, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  if (!tile_live<KIND, BM>(a, m0)) return;  // uniform across the workgroup

  // load i of a thread fills chunk position i * NT + tid of the A (or B) part of a stage.
  // The resources are based at the tile's first row and the slice's first column, so 32-bit
  // offsets reach any operand; rows past M or N lie past the resource's end
  int a_off[ACH], b_off[BCH], a_kc[ACH], b_kc[BCH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    const int p = tid + i * NT, row = p / CPR;
    a_kc[i] = ((p % CPR) ^ dma_swz<CPR>(row)) * 4;
    a_off[i] = (row * a.lda + a_kc[i]) * 4;
  }
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int p = tid + i * NT, row = p / CPR;
    b_kc[i] = ((p % CPR) ^ dma_swz<CPR>(row)) * 4;
    b_off[i] = (row * a.ldb + b_kc[i]) * 4;
  }
  const float* const A0 = (const float*)a.A + (size_t)m0 * a.lda;
  const float* const B0 = (const float*)a.B + (size_t)n0 * a.ldb;
  const int a_rows = min(a.M - m0, BM), b_rows = min(a.N - n0, BN);
  auto issue = [&](char* sb, int kt) {
    const int k0 = kt * BK;
    const bool live = k0 < a.K;
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(A0 + k0, live ? (uint32_t)(a_rows * a.lda - k0) * 4 : 0u);
    const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(B0 + k0, live ? (uint32_t)(b_rows * a.ldb - k0) * 4 : 0u);
#pragma unroll
    for (int i = 0; i < ACH; ++i)
      buffer_load16_lds(ra, sb + (i * NT + wave * 64) * 16, k0 + a_kc[i] < a.K ? a_off[i] : kOffOOB);
#pragma unroll
    for (int i = 0; i < BCH; ++i)
      buffer_load16_lds(rb, sb + (ATOT + i * NT + wave * 64) * 16, k0 + b_kc[i] < a.K ? b_off[i] : kOffOOB);
  };

  f32x4 accs[4][TM][TN];  // one sum per element of a chunk
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) accs[e][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int sw = dma_swz<CPR>(l16);  // row blocks are 16 apart: every row of a lane shares it
  const int a_row = (wm * TM * 16 + l16) * CPR, b_row = ATOT + (wn * TN * 16 + l16) * CPR;

  constexpr int kWait = waitcnt_vm_lgkm0<(STAGES - 2) * LPT>();
  auto step = [&](auto s, int kt) {
    constexpr int S = decltype(s)::value;
    __builtin_amdgcn_s_waitcnt(kWait);
    bare_barrier();
    issue(stage(std::integral_constant<int, S + STAGES - 1>{}), kt + STAGES - 1);
    const char* cur = stage(std::integral_constant<int, S>{});
    f32x4 af[2][TM], bf[2][TN];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[kk][i] = *(const f32x4*)(cur + (a_row + i * 16 * CPR + ((kk * 4 + g) ^ sw)) * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[kk][j] = *(const f32x4*)(cur + (b_row + j * 16 * CPR + ((kk * 4 + g) ^ sw)) * 16);
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            accs[e][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[kk][j][e], af[kk][i][e], accs[e][i][j], 0, 0, 0);
  };

  const int nk = (a.K + BK - 1) / BK;
  issue(stage(std::integral_constant<int, 0>{}), 0);
  issue(stage(std::integral_constant<int, 1>{}), 1);
  int kt = 0;
  for (; kt + STAGES <= nk; kt += STAGES) {
    step(std::integral_constant<int, 0>{}, kt);
    step(std::integral_constant<int, 1>{}, kt + 1);
    step(std::integral_constant<int, 2>{}, kt + 2);
  }
  if (kt < nk) step(std::integral_constant<int, 0>{}, kt);
  if (kt + 1 < nk) step(std::integral_constant<int, 1>{}, kt + 1);
  __builtin_amdgcn_s_waitcnt(0);  // the loads past K land before the LDS is given up

#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + (wm * TM + i) * 16 + l16;
    if (m >= a.M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + (wn * TN + j) * 16 + g * 4;
      f32x4 acc;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        acc[c] = (accs[0][i][j][c] + accs[1][i][j][c]) + (accs[2][i][j][c] + accs[3][i][j][c]);
      if (n < a.N) f32_epilogue4<KIND>(a, m, n, acc);
    }
  }
}

// fp32 tiles (BM x BN, wave grid): 64 x 64 where it gives at least two workgroups per CU,
// 32 x 32 below, where it spreads the rows over more of the chip (4096 x 3072 x 768: 161 us
// with 64 x 64, 170 with 32 x 32; 1024 x 768 x 768: 19.0 and 14.6; 420 x 192 x 768: 17.6
// and 8.1; 1024 x 2304 x 768, 576 tiles, 43.6 and 37.8: the line costs that one). 128 x 64 and
// 128 x 128 tiles, with one sum per output, were no faster (4096 x 768 x 768 54 us with the
// first against 47).
#define SF_GEMM_F32_TILES(X) \
  X(0, 64, 64, 2, 2)         \
  X(1, 32, 32, 2, 2)

// bf16 tiles (BM x BN, wave grid WM x WN). A CU spreads a workgroup's wavefronts
// round-robin over its four SIMDs, so a wavefront count that is a multiple of four keeps
// them evenly loaded.
//
// Register-staged (64-wide K slices).
#define SF_GEMM_TILES(X)              \
  X(kTile128, 128, 128, 64, 2, 2)     \
  X(kTile128x288, 128, 288, 64, 4, 3) \
  X(kTile256x192, 256, 192, 64, 4, 2)

// Directly staged, the K slice split over two sets of wavefronts (number of LDS stages).
#define SF_GEMM_DMA_TILES(X)                \
  X(kHalf128x96, 128, 96, 64, 4, 1, 2, 4)   \
  X(kHalf128, 128, 128, 64, 2, 2, 2, 3)     \
  X(kHalf64, 64, 64, 64, 2, 2, 2, 4)

// Directly staged with the fragments read a K step ahead (LDS stages, wavefronts per
// SIMD, both halves of a K slice summed apart).
#define SF_GEMM_PIPE_TILES(X)                             \
  X(kPipe128x192, 128, 192, 2, 2, 2, 2, false)            \
  X(kPipe128, 128, 128, 2, 2, 2, 2, false)                \
  X(kPipe64, 64, 64, 2, 2, 4, 2, false)                   \
  X(kPipeHalf128x192, 128, 192, 4, 2, 3, 2, true)         \
  X(kPipeHalf128, 128, 128, 2, 2, 2, 2, true)

template <EpiKind KIND>
static hipError_t launch_bf16_tile(GemmTile tile, const GemmArgs& a, hipStream_t s) {
#define SF_LAUNCH(kernel, bm, bn, waves) \
  launch(kernel, dim3(((a.N + bn - 1) / bn) * ((a.M + bm - 1) / bm)), dim3((waves)*64), 0, s, a)
  switch (tile) {
#define SF_TILE_CASE(id, bm, bn, bk, wm, wn)                                                         \
  case id:                                                                                           \
    if constexpr (gemm_tile_used(id, KIND))                                                          \
      SF_LAUNCH((gemm_bf16_sched_kernel<bm, bn, bk, wm, wn, KIND>), bm, bn, wm* wn);                 \
    else                                                                                             \
      return hipErrorInvalidValue;                                                                   \
    break;
    SF_GEMM_TILES(SF_TILE_CASE)
#undef SF_TILE_CASE
#define SF_DMA_TILE_CASE(id, bm, bn, bk, wm, wn, ks, st)                                             \
  case id:                                                                                           \
    SF_LAUNCH((gemm_bf16_dma_kernel<bm, bn, bk, wm, wn, ks, st, KIND>), bm, bn, wm* wn* ks);         \
    break;
    SF_GEMM_DMA_TILES(SF_DMA_TILE_CASE)
#undef SF_DMA_TILE_CASE
#define SF_PIPE_TILE_CASE(id, bm, bn, wm, wn, st, mw, hv)                                        \
  case id:                                                                                           \
    if constexpr (gemm_tile_used(id, KIND))                                                          \
      SF_LAUNCH((gemm_bf16_pipe_kernel<bm, bn, wm, wn, st, mw, hv, KIND>), bm, bn, wm* wn);      \
    else                                                                                             \
      return hipErrorInvalidValue;                                                                   \
    break;
    SF_GEMM_PIPE_TILES(SF_PIPE_TILE_CASE)
#undef SF_PIPE_TILE_CASE
    default:
      return hipErrorInvalidValue;
  }
#undef SF_LAUNCH
  return hipGetLastError();
}

template <EpiKind KIND>
static hipError_t launch_f32_tile(int tile, const GemmArgs& a, hipStream_t s) {
  switch (tile) {
#define SF_F32_TILE_CASE(id, bm, bn, wm, wn)                                                  \
  case id:                                                                                    \
    launch((gemm_f32_kernel<bm, bn, wm, wn, KIND>),                                           \
           dim3(((a.N + bn - 1) / bn) * ((a.M + bm - 1) / bm)), dim3(wm * wn * 64), 0, s, a); \
    break;
    SF_GEMM_F32_TILES(SF_F32_TILE_CASE)
#undef SF_F32_TILE_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <EpiKind KIND>
static hipError_t launch_kind(bool use_bf16, const GemmArgs& a, hipStream_t s) {
  if (use_bf16) return launch_bf16_tile<KIND>(choose_gemm_tile(a.M, a.N, a.K, a.ntok, KIND), a, s);
  return launch_f32_tile<KIND>(choose_gemm_f32_tile(a.M, a.N), a, s);
}

hipError_t launch_gemm(bool use_bf16, EpiKind kind, const GemmArgs& a, hipStream_t s) {
  switch (kind) {
    case EPI_QKV: return launch_kind<EPI_QKV>(use_bf16, a, s);
    case EPI_RES_GATE: return launch_kind<EPI_RES_GATE>(use_bf16, a, s);
    case EPI_GELU: return launch_kind<EPI_GELU>(use_bf16, a, s);
    case EPI_RES: return launch_kind<EPI_RES>(use_bf16, a, s);
    case EPI_RES_GATE_MLP: return launch_kind<EPI_RES_GATE_MLP>(use_bf16, a, s);
    case EPI_KVX: return launch_kind<EPI_KVX>(use_bf16, a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace sf
