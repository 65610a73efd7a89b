// Device code shared by the attention kernels: operand splitting and one 64-key chunk of
// block-causal attention on bf16 MFMA for 16 query rows (head_dim 64).
#pragma once
#include "xsm_device.h"

namespace xsm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// 2^x on the hardware's exponential instruction alone (1 ulp; results below the normal range come
// out as zero, which is what a softmax weight that small is worth)
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ uint32_t pack2(float a, float b) { return f2bf_pair(a, b); }

// (a, b) -> packed bf16 pair of the rounded values and of what the rounding dropped
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& lo) {
  hi = pack2(a, b);
  lo = pack2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}

// the lane's 16 query values (dims g*8.. and 32 + g*8..) -> operand halves, each as bf16 hi and lo parts
__device__ __forceinline__ void split_queries(const float4 (&x)[4], bf16x8 (&qh)[2], bf16x8 (&ql)[2]) {
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const float4 x0 = x[half * 2], x1 = x[half * 2 + 1];
    uint32_t hw[4], lw[4];
    split2(x0.x, x0.y, hw[0], lw[0]); split2(x0.z, x0.w, hw[1], lw[1]);
    split2(x1.x, x1.y, hw[2], lw[2]); split2(x1.z, x1.w, hw[3], lw[3]);
    qh[half] = __builtin_bit_cast(bf16x8, uint4{hw[0], hw[1], hw[2], hw[3]});
    ql[half] = __builtin_bit_cast(bf16x8, uint4{lw[0], lw[1], lw[2], lw[3]});
  }
}

// One 64-key chunk (keys key0..key0+63, fragments kf / vf as the cache loads deliver them) for the
// wavefront's 16 queries: scores, online softmax (base 2), second product.  Query r sees keys
// below lim; below first_masked every live query sees the key; keys at or past Ltot may hold
// garbage (their values are zeroed so that 0 x garbage cannot become NaN).
__device__ __forceinline__ void attn_chunk(const uint4 (&kf)[4][2], uint4 (&vf)[4][2], const bf16x8 (&qh)[2],
                                           const bf16x8 (&ql)[2], int key0, int g, bool qlive, int lim,
                                           int first_masked, int Ltot, float scale_log2, float& m_run,
                                           float& l_run, f32x4 (&o)[4]) {
  f32x4 sc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const bf16x8 kk = __builtin_bit_cast(bf16x8, kf[t][half]);
      sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, ql[half], sc[t], 0, 0, 0);
      sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, qh[half], sc[t], 0, 0, 0);
    }
  }
  // this lane's 16 scores belong to keys key0 + g*16 + t*4 + i
  const int kbase = key0 + g * 16;
  const bool edge = key0 + 64 > first_masked || !qlive;
  float cmax = -INFINITY;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v = sc[t][i] * scale_log2;
      if (edge && kbase + t * 4 + i >= lim) v = -INFINITY;
      sc[t][i] = v;
      cmax = fmaxf(cmax, v);
    }
  cmax = fmaxf(cmax, lane_xor<16>(cmax));
  cmax = fmaxf(cmax, lane_xor<32>(cmax));
  const float m_new = fmaxf(m_run, cmax);
  const float m_use = m_new == -INFINITY ? 0.f : m_new;
  const float alpha = exp2_hw(m_run - m_use);
  float psum = 0.f;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = exp2_hw(sc[t][i] - m_use);
      sc[t][i] = p;
      psum += p;
    }
  psum += lane_xor<16>(psum);
  psum += lane_xor<32>(psum);
  l_run = l_run * alpha + psum;
  m_run = m_new;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
  if (key0 + 64 > Ltot) {                         // slots past the live range hold garbage
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        uint32_t* w = reinterpret_cast<uint32_t*>(&vf[dt][jj]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (kbase + jj * 8 + e >= Ltot) w[e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
        }
      }
  }
  uint4 ph[2], pl[2];
#pragma unroll
  for (int jj = 0; jj < 2; ++jj) {
    split2(sc[2 * jj][0], sc[2 * jj][1], ph[jj].x, pl[jj].x);
    split2(sc[2 * jj][2], sc[2 * jj][3], ph[jj].y, pl[jj].y);
    split2(sc[2 * jj + 1][0], sc[2 * jj + 1][1], ph[jj].z, pl[jj].z);
    split2(sc[2 * jj + 1][2], sc[2 * jj + 1][3], ph[jj].w, pl[jj].w);
  }
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const bf16x8 vv = __builtin_bit_cast(bf16x8, vf[dt][jj]);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, __builtin_bit_cast(bf16x8, pl[jj]), o[dt], 0, 0, 0);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, __builtin_bit_cast(bf16x8, ph[jj]), o[dt], 0, 0, 0);
    }
}

}  // namespace xsm
