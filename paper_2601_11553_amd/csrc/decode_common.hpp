// Pieces that the two attention kernels of decoding steps share (decode_attention.hip, decode_stack.hip).
#pragma once

#include "percache_internal.hpp"

namespace pc {
namespace dec {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// over the four lanes (l, l + 16, l + 32, l + 48) that share a query row: the rows of 16 lanes change places in the vector pipe (a
// shuffle goes through LDS and takes a hundred clocks more)
template <class Op>
__device__ __forceinline__ float over_rows(float x, Op op) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const u32x2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float row_max(float x) {
  return over_rows(x, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float row_sum(float x) {
  return over_rows(x, [](float a, float b) { return a + b; });
}
// over all 64 lanes: the 16 of a row by data-parallel moves, then the rows
__device__ __forceinline__ float wave_sum(float x) {
#define PC_MOVE(ctrl) __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), ctrl, 0xf, 0xf, true))
  x += PC_MOVE(0xB1);    // lane ^ 1
  x += PC_MOVE(0x4E);    // lane ^ 2
  x += PC_MOVE(0x141);   // mirrored inside 8
  x += PC_MOVE(0x140);   // mirrored inside 16
#undef PC_MOVE
  return row_sum(x);
}

// E4M3 codes times a power-of-two scale -> bf16 (exact)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16x4 codes4(unsigned w, float scale) {
  union { bf16x2 p[2]; bf16x4 v; } u;
  u.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, scale, false);
  u.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, scale, true);
  return u.v;
}
__device__ __forceinline__ bf16x8 codes8(uint2 w, float scale) {
  union { bf16x4 p[2]; bf16x8 v; } u;
  u.p[0] = codes4(w.x, scale);
  u.p[1] = codes4(w.y, scale);
  return u.v;
}

// Elements 32 ks + 8 g .. +7 of one projected head row of D fp32 sums (the four lanes g share a row): load() asks for
// everything, finish() applies bias, RMSNorm over the head (gain; null: none) and RoPE and rounds to bf16 once.
template <int D>
struct RawRow {
  static constexpr int KS = D / 32;
  f32x4 x[KS][2], cs[KS / 2][4];
  bf16x8 bi[KS], gn[KS];
  __device__ __forceinline__ void load(const float *__restrict__ sums, const __bf16 *__restrict__ bias, const __bf16 *__restrict__ gain,
                                       const float2 *__restrict__ rope, int pos, int g) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      x[ks][0] = *(const f32x4 *)(sums + ks * 32 + g * 8);
      x[ks][1] = *(const f32x4 *)(sums + ks * 32 + g * 8 + 4);
    }
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
      for (int h = 0; h < 4; ++h) cs[ks][h] = *(const f32x4 *)(rope + (size_t)pos * (D / 2) + ks * 32 + g * 8 + h * 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (bias) bi[ks] = *(const bf16x8 *)(bias + ks * 32 + g * 8);
      if (gain) gn[ks] = *(const bf16x8 *)(gain + ks * 32 + g * 8);
    }
  }
  __device__ __forceinline__ void finish(bool bias, bool gain, float eps, bf16x8 (&out)[KS]) {
    if (bias) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[ks][e >> 2][e & 3] += (float)bi[ks][e];
    }
    if (gain) {
      float s = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) s += x[ks][e >> 2][e & 3] * x[ks][e >> 2][e & 3];
      const float r = 1.0f / sqrtf(row_sum(s) / (float)D + eps);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[ks][e >> 2][e & 3] *= r * (float)gn[ks][e];
    }
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float a = x[ks][e >> 2][e & 3], b = x[ks + KS / 2][e >> 2][e & 3];
        const float c = cs[ks][e >> 1][2 * (e & 1)], sn = cs[ks][e >> 1][2 * (e & 1) + 1];
        out[ks][e] = (__bf16)(a * c - b * sn);
        out[ks + KS / 2][e] = (__bf16)(b * c + a * sn);
      }
  }
};

}  // namespace dec
}  // namespace pc
