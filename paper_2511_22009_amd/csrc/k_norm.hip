// Row kernels over the fp32 residual stream:
//  * K5: LayerNorm (biased variance, eps 1e-6, no affine) followed by the per-sample
//    adaLN modulate LN(h) (1 + scale) + shift, where the row's sample selects its own
//    row of the modulation table, so each sample is conditioned on its own t;
//  * K7: the same LN + modulate with the final layer's table entries, the linear map
//    D -> p*p*C, and unpatchify into the velocity latent.
#include "sf_device.h"

namespace sf {

constexpr float kLnEps = 1e-6f;
template <typename OT> struct Store4;
template <> struct Store4<float> {
  __device__ static void run(float* p, float a, float b, float c, float d) {
    *(float4*)p = make_float4(a, b, c, d);
  }
};
template <> struct Store4<bf16> {
  __device__ static void run(bf16* p, float a, float b, float c, float d) {
    bf16x4 o = {(bf16)a, (bf16)b, (bf16)c, (bf16)d};
    *(bf16x4*)p = o;
  }
};

// RPW rows per wavefront, NV float4 per lane per row (D <= 256 NV). Every load of
// the wavefront's rows and of their table entries (shift and scale) is issued before
// the first reduction, so the kernel pays one memory latency per row group. The loads
// are unconditional, at in-bounds indices (chunk 0 stands in for chunks past the row's
// end; a plain LN reads its unused shift and scale from the row itself), and the zeros
// of the chunks past the end are selected once all loads are issued: a load under a
// lane condition makes the compiler wait for it before the other path writes the same
// registers, which would cost one memory latency per chunk.
template <typename OT, int NV, int RPW>
__global__ __launch_bounds__(256) void ln_mod_kernel(LnArgs a) {
  const int lane = threadIdx.x & 63;
  const int mb = (blockIdx.x * 4 + (threadIdx.x >> 6)) * RPW;
  if (mb >= a.M) return;
  const int nv = a.D >> 2;
  float4 v[RPW][NV], sc[RPW][NV], sh[RPW][NV];
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int m = min(mb + r, a.M - 1);
    const float4* row = (const float4*)(a.h + (size_t)m * a.D);
    const float* tsh = (const float*)row;
    const float* tsc = (const float*)row;
    if (a.table) {
      const int q = (int)fdiv((uint32_t)m, a.tok);
      const int slot = q < a.n_slots ? q : q - a.n_slots;
      tsh = a.table + (size_t)slot * a.ldt + a.shift_off;
      tsc = a.table + (size_t)slot * a.ldt + a.scale_off;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = lane + i * 64;
      const int cc = c < nv ? c : 0;
      v[r][i] = row[cc];
      sc[r][i] = *(const float4*)(tsc + 4 * cc);
      sh[r][i] = *(const float4*)(tsh + 4 * cc);
    }
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r)
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (lane + i * 64 >= nv) v[r][i] = make_float4(0.f, 0.f, 0.f, 0.f);
  float mean[RPW], rstd[RPW];
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) s += (v[r][i].x + v[r][i].y) + (v[r][i].z + v[r][i].w);
    mean[r] = wave_sum(s) / (float)a.D;
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    float q = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (lane + i * 64 < nv) {
        float d;
        d = v[r][i].x - mean[r]; q += d * d; d = v[r][i].y - mean[r]; q += d * d;
        d = v[r][i].z - mean[r]; q += d * d; d = v[r][i].w - mean[r]; q += d * d;
      }
    }
    rstd[r] = 1.0f / sqrtf(wave_sum(q) / (float)a.D + kLnEps);
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int m = mb + r;
    if (m >= a.M) break;
    OT* out = (OT*)a.out + (size_t)m * a.D;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = lane + i * 64;
      if (c < nv) {
        float y0 = (v[r][i].x - mean[r]) * rstd[r], y1 = (v[r][i].y - mean[r]) * rstd[r];
        float y2 = (v[r][i].z - mean[r]) * rstd[r], y3 = (v[r][i].w - mean[r]) * rstd[r];
        if (a.table) {
          y0 = y0 * (1.0f + sc[r][i].x) + sh[r][i].x;
          y1 = y1 * (1.0f + sc[r][i].y) + sh[r][i].y;
          y2 = y2 * (1.0f + sc[r][i].z) + sh[r][i].z;
          y3 = y3 * (1.0f + sc[r][i].w) + sh[r][i].w;
        }
        Store4<OT>::run(out + 4 * c, y0, y1, y2, y3);
      }
    }
  }
}

template <typename OT, int NV>
static void launch_ln_nv(const LnArgs& a, hipStream_t s) {
  // one row per wavefront: more wavefronts in flight beat more rows per wavefront
  // (4096 x 768: 4.5 us against 5.1 us with two rows)
  constexpr int RPW = 1;
  const int grid = (a.M + 4 * RPW - 1) / (4 * RPW);
  launch((ln_mod_kernel<OT, NV, RPW>), dim3(grid), dim3(256), 0, s, a);
}

template <typename OT>
static hipError_t launch_ln_t(const LnArgs& a, hipStream_t s) {
  switch ((a.D + 255) / 256) {
    case 1: launch_ln_nv<OT, 1>(a, s); break;
    case 2: launch_ln_nv<OT, 2>(a, s); break;
    case 3: launch_ln_nv<OT, 3>(a, s); break;
    case 4: launch_ln_nv<OT, 4>(a, s); break;
    case 5: launch_ln_nv<OT, 5>(a, s); break;
    case 6: launch_ln_nv<OT, 6>(a, s); break;
    case 7: launch_ln_nv<OT, 7>(a, s); break;
    case 8: launch_ln_nv<OT, 8>(a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_ln(bool out_bf16, const LnArgs& a, hipStream_t s) {
  return out_bf16 ? launch_ln_t<bf16>(a, s) : launch_ln_t<float>(a, s);
}

// A workgroup takes 16 token rows, its four wavefronts a quarter of the columns each (16-wide
// chunks 4 i + wave), held in registers in the operand layout of v_mfma_f32_16x16x4_f32: lane
// (l16, g) (g = lane / 16) has columns 4 g .. 4 g + 3 of every chunk of row l16. The row
// sums are lane-local plus two lane exchanges and one pass through LDS; then the modulated
// rows feed the linear map D -> P as they stand, MFMA (i, e) contracting columns 16 (4 i +
// wave) + 4 g + e against the same columns of 16 W_f rows (exact fp32 products and sums, four
// running sums per output and wavefront), and the wavefronts' results meet in LDS. Each value
// goes straight to its unpatchified position. Every row's arithmetic is the same wherever
// it sits in its group. Loading the rows bounds it; with the map as dot products on the
// vector ALU, four rows per wavefront, it was bound by the chains of a lone wavefront per
// SIMD: 16384 rows x 1152 57.6 us, 29.6 so; 4096 x 1152 16.6 and 10.6; 1024 x 768 9.4 and 6.6.
// (The weight rows loaded after the row sums, for fewer registers: 28.0 and 10.5, but 10.3
// at 1024 x 768, where their latency is not covered.)
template <int NI>  // 64-wide column steps: D <= 64 NI
__global__ __launch_bounds__(256) void head_kernel(HeadArgs a) {
  __shared__ float red[2][4][16];
  __shared__ f32x4 part[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int M = a.rows * a.N;
  const int m0 = blockIdx.x * 16;
  const int m = min(m0 + l16, M - 1);
  const int c0 = 16 * wave + 4 * g;  // this lane's first column
  // unconditional loads at in-bounds columns, zeros selected after all are issued
  auto col = [&](int i) { return c0 + 64 * i < a.D ? c0 + 64 * i : 0; };
  f32x4 v[NI], w[NI];
  const float* row = a.h + (size_t)m * a.D;
#pragma unroll
  for (int i = 0; i < NI; ++i) v[i] = *(const f32x4*)(row + col(i));
  auto load_w = [&](int f0) {
    const float* wr = a.W_f + (size_t)min(f0 + l16, a.P - 1) * a.D;
#pragma unroll
    for (int i = 0; i < NI; ++i) w[i] = *(const f32x4*)(wr + col(i));
  };
  load_w(0);
  const int q = (int)fdiv((uint32_t)m, a.tok);
  const int slot = q < a.n_slots ? q : q - a.n_slots;
  const float* tsh = a.table + (size_t)slot * a.ldt + a.shift_off;
  const float* tsc = a.table + (size_t)slot * a.ldt + a.scale_off;
  auto row_sum = [&](int which, float s) {
    s = pair32_sum(pair16_sum(s));
    if (g == 0) red[which][wave][l16] = s;
    __syncthreads();
    return (red[which][0][l16] + red[which][1][l16]) + (red[which][2][l16] + red[which][3][l16]);
  };
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (c0 + 64 * i >= a.D) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
  }
  const float mean = row_sum(0, s) / (float)a.D;
  float sq = 0.0f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (c0 + 64 * i < a.D) {
      const float d0 = v[i][0] - mean, d1 = v[i][1] - mean, d2 = v[i][2] - mean, d3 = v[i][3] - mean;
      sq += (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
    }
  }
  const float rstd = 1.0f / sqrtf(row_sum(1, sq) / (float)a.D + kLnEps);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const f32x4 sc = *(const f32x4*)(tsc + col(i)), sh = *(const f32x4*)(tsh + col(i));
    const bool in = c0 + 64 * i < a.D;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[i][e] = in ? (v[i][e] - mean) * rstd * (1.0f + sc[e]) + sh[e] : 0.0f;
  }
  const int gwn = a.W / a.p;
  for (int f0 = 0; f0 < a.P; f0 += 16) {
    if (f0 > 0) {
      __syncthreads();  // the previous outputs were read
      load_w(f0);
    }
    f32x4 acc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][e], w[i][e], acc[e], 0, 0, 0);
    f32x4 t;
#pragma unroll
    for (int r = 0; r < 4; ++r) t[r] = (acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r]);
    part[wave][lane] = t;
    __syncthreads();
    // lane (l16, g) holds output f0 + l16 of rows 4 g .. 4 g + 3: wavefront w writes row 4 g + w
    const int mo = m0 + 4 * g + wave, f = f0 + l16;
    if (mo < M && f < a.P) {
      const float y = (part[0][lane][wave] + part[1][lane][wave]) + (part[2][lane][wave] + part[3][lane][wave]);
      const int r = (int)fdiv((uint32_t)mo, a.tok);
      const int n = mo - r * a.N;
      const int gh = n / gwn, gw = n - gh * gwn;
      const int c = f % a.C, ij = f / a.C;
      const int i = ij / a.p, j = ij - i * a.p;
      a.v[(((size_t)r * a.C + c) * a.H + gh * a.p + i) * a.W + gw * a.p + j] = y + a.b_f[f];
    }
  }
}

hipError_t launch_head(const HeadArgs& a, hipStream_t s) {
  const dim3 grid((a.rows * a.N + 15) / 16);
  const int ni = (a.D + 63) / 64;
  if (ni <= 2) launch(head_kernel<2>, grid, dim3(256), 0, s, a);
  else if (ni <= 4) launch(head_kernel<4>, grid, dim3(256), 0, s, a);
  else if (ni <= 8) launch(head_kernel<8>, grid, dim3(256), 0, s, a);
  else if (ni <= 12) launch(head_kernel<12>, grid, dim3(256), 0, s, a);
  else if (ni <= 18) launch(head_kernel<18>, grid, dim3(256), 0, s, a);
  else if (ni <= 24) launch(head_kernel<24>, grid, dim3(256), 0, s, a);
  else if (ni <= 32) launch(head_kernel<32>, grid, dim3(256), 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace sf
