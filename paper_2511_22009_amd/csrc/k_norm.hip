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

// A workgroup takes four token rows. Each wavefront normalises and modulates one of them (lane
// l holds 16-byte chunks l + 64 i) and leaves it in LDS; then wavefront w applies outputs
// 4 w .. 4 w + 3 (and every 16th group of four after them) of the linear map D -> P to all four
// rows: its slice of four W_f rows, loaded with the rows at the start, stays in registers
// while outputs last, and the 16 row x output sums leave through one butterfly reduction. Each
// value goes straight to its unpatchified position.
//
// One order of sums for every output, spelled out with fmaf so that no compilation changes it:
// per chunk fma(x, wx, y wy) + fma(z, wz, w ww), a lane's chunks in turn, then the lanes by
// xor 32, 16, 8, 4, 2, 1. In a stream step the head's last bits enter the queue and, through
// the bf16 roundings of later steps, the fourth digit of its latents, so another order is
// another trajectory (on v_mfma_f32_16x16x4_f32, sixteen rows per workgroup, a second 512^2
// step differed by 1e-4, a guided one by 7e-4, at the same error against 64 bits).
//
// The vector ALU bounds it: six instructions per four products in this order. us for 1024 x
// 768 / 4096 x 768 / 16384 x 768 / 16384 x 1152 rows x width: 4.8 / 8.5 / 24.0 / 37.7; the
// same order with four rows and all outputs per wavefront (lone wavefronts, bound by their
// chains) 10.2 / 11.0 / 28.6 / 54.2; on the matrix cores 7.5 / 8.2 / 20.4 / 30.1. Two rows per
// wavefront: 6.2 / 8.2 / 25.5 / 53.2; a loop over row groups that keeps the weights 5.4 /
// 9.3 / 26.5 / 54.4.
template <int NV>  // 256 (NV - 1) < D <= 256 NV
__global__ __launch_bounds__(256) void head_kernel(HeadArgs a) {
  __shared__ float4 rows[4][NV * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int M = a.rows * a.N;
  const int m0 = blockIdx.x * 4;
  const int nv = a.D >> 2;
  // unconditional loads at in-bounds chunks (only a row's last chunk can lie past its end),
  // zeros selected after all are issued
  auto in = [&](int i) { return i + 1 < NV || lane + i * 64 < nv; };
  auto col = [&](int i) { return in(i) ? lane + i * 64 : 0; };
  float4 w[4][NV];
  auto load_w = [&](int o0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4* wr = (const float4*)(a.W_f + (size_t)min(o0 + q, a.P - 1) * a.D);
#pragma unroll
      for (int i = 0; i < NV; ++i) w[q][i] = wr[col(i)];
    }
  };
  {
    const int m = min(m0 + wave, M - 1);
    const float4* row = (const float4*)(a.h + (size_t)m * a.D);
    const int r = (int)fdiv((uint32_t)m, a.tok);
    const int slot = r < a.n_slots ? r : r - a.n_slots;
    const float4* tsh = (const float4*)(a.table + (size_t)slot * a.ldt + a.shift_off);
    const float4* tsc = (const float4*)(a.table + (size_t)slot * a.ldt + a.scale_off);
    float4 v[NV], sc[NV], sh[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i] = row[col(i)];
      sc[i] = tsc[col(i)];
      sh[i] = tsh[col(i)];
    }
    load_w(4 * wave);
    if (!in(NV - 1)) v[NV - 1] = make_float4(0.f, 0.f, 0.f, 0.f);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    const float mean = wave_sum(s) / (float)a.D;
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const float d0 = v[i].x - mean, d1 = v[i].y - mean, d2 = v[i].z - mean, d3 = v[i].w - mean;
      const float d = fmaf(d0, d0, d1 * d1) + fmaf(d2, d2, d3 * d3);
      sq = in(i) ? sq + d : sq;
    }
    const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)a.D + kLnEps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      float4 y;
      y.x = in(i) ? fmaf((v[i].x - mean) * rstd, 1.0f + sc[i].x, sh[i].x) : 0.0f;
      y.y = in(i) ? fmaf((v[i].y - mean) * rstd, 1.0f + sc[i].y, sh[i].y) : 0.0f;
      y.z = in(i) ? fmaf((v[i].z - mean) * rstd, 1.0f + sc[i].z, sh[i].z) : 0.0f;
      y.w = in(i) ? fmaf((v[i].w - mean) * rstd, 1.0f + sc[i].w, sh[i].w) : 0.0f;
      rows[wave][lane + i * 64] = y;
    }
  }
  __syncthreads();
  for (int o0 = 4 * wave; o0 < a.P; o0 += 16) {
    if (o0 >= 16) load_w(o0);
    float acc[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float4 x = rows[r][lane + i * 64];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc[r * 4 + q] += fmaf(x.x, w[q][i].x, x.y * w[q][i].y) + fmaf(x.z, w[q][i].z, x.w * w[q][i].w);
      }
    const float tot = wave_reduce16(acc);
    const int idx = (lane >> 2) & 15;
    const int m = m0 + (idx >> 2), f = o0 + (idx & 3);
    if ((lane & 3) == 0 && f < a.P && m < M) {
      const int r = (int)fdiv((uint32_t)m, a.tok);
      const int n = m - r * a.N;
      const int gh = (int)fdiv((uint32_t)n, a.div_gw), gw = n - gh * (int)a.div_gw.d;
      const int ij = (int)fdiv((uint32_t)f, a.div_c), c = f - ij * a.C;
      const int i = (int)fdiv((uint32_t)ij, a.div_p), j = ij - i * a.p;
      a.v[(((size_t)r * a.C + c) * a.H + gh * a.p + i) * a.W + gw * a.p + j] = tot + a.b_f[f];
    }
  }
}

hipError_t launch_head(const HeadArgs& a, hipStream_t s) {
  const dim3 grid((a.rows * a.N + 3) / 4);
  switch ((a.D + 255) / 256) {
    case 1: launch(head_kernel<1>, grid, dim3(256), 0, s, a); break;
    case 2: launch(head_kernel<2>, grid, dim3(256), 0, s, a); break;
    case 3: launch(head_kernel<3>, grid, dim3(256), 0, s, a); break;
    case 4: launch(head_kernel<4>, grid, dim3(256), 0, s, a); break;
    case 5: launch(head_kernel<5>, grid, dim3(256), 0, s, a); break;
    case 6: launch(head_kernel<6>, grid, dim3(256), 0, s, a); break;
    case 7: launch(head_kernel<7>, grid, dim3(256), 0, s, a); break;
    case 8: launch(head_kernel<8>, grid, dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace sf
