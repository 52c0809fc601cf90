// Projections of few token rows (decoding steps, the fresh part of a short query): Y[m][n] = sum_k X[m][k] W[n][k].
//
// What bounds them is the latency of one pass over the weights and, from a few dozen rows on, what a CU takes in from L2;
// the arithmetic is nothing.  So a launch needs about as many workgroups as there are CUs, every one of them with many
// bytes in flight from its first instruction on, and no second kernel behind it: a workgroup owns 16 NF weight rows x
// 16 NT token rows over the WHOLE contraction, each of its wavefronts takes a slice of the contraction through a PRIVATE
// ring of LDS stages (direct global->LDS loads, no barrier on the way), and the partial tiles meet once, in LDS, where
// the epilogue is applied to the fp32 sums.  Against slices of the contraction in separate workgroups + a reduce kernel
// that added them up (us per projection, weights cold, N x K):
//   1 row:    1024 x 2048  3.8 (4.8 + 4.0)     6144 x 1024  4.4 (4.8 + 2.7)     1024 x 3072  4.6 (4.8 + 4.0)
//   128 rows: 1024 x 2048  5.4 (9.9 + 4.8)     4096 x 1024  6.2 (9.8 in one pass on 128-token tiles)
// The operands straight from global memory into registers (lane = row) were also tried: 4.9 us for the first of these and
// 9.3 for the last -- neighbouring lanes then ask for different rows, which costs about 80 cycles per load instruction.
//
// An RMSNorm in front of the projection needs no kernel of its own: y = (x * gain) W^T * rsqrt(mean(x^2) + eps).  The
// operand is x * gain rounded to bf16 (one rounding, as of a stored normed row), the row's sum of squares is taken from
// the same registers, and the factor is applied to the fp32 sums.  It costs 0.7 us at one row and 2 us at 128, a kernel
// of its own 2.6 to 3.7.
//
// Layouts: a stage holds 64 k-elements (128 bytes) of every row, 16-byte chunks XOR-swizzled as in gemm_tile.hpp.  In the
// 16x16x32 product with the weights on the M side lane l reads elements 8 (l/16) .. +7 of row l%16 of both operands and
// ends up with weight rows 4 (l/16) + 0..3 of token l%16.
#pragma once

#include "gemm_tile.hpp"

namespace pc {
namespace few {

using gemm::ROW;
using gemm::swz128;
using gemm::wait_vmcnt;

// NF, NT: 16-row blocks of weights / of tokens in a workgroup's tile.  WV: wavefronts = slices of the contraction.
// XL > 0: the token rows are not loaded but put into LDS by the caller, XL steps of 64 k-elements per wavefront at most.
template <int NF, int NT, int WV, int NSTG, bool NORM, int XL = 0>
struct Tile {
  static constexpr int W_INSTR = 2 * NF, X_INSTR = XL ? 0 : 2 * NT;        // load instructions (8 rows x 128 bytes) per stage
  static constexpr int IPS = W_INSTR + X_INSTR + (NORM ? 1 : 0);           // and the 64 gains of the stage
  static constexpr int STAGE = (W_INSTR + X_INSTR) * 1024 + (NORM ? 128 : 0);
  static constexpr int X_OWN = XL * NT * 2048;                              // token rows of a wavefront's slice (XL)
  static constexpr int RING = WV * (NSTG * STAGE + X_OWN);
  static constexpr int SUMS = WV * NF * NT * 1024;                          // partial tiles (fp32), in the ring's place
  static constexpr int SS = WV * NT * 64;                                   // sums of squares
  static constexpr int LDS_BYTES = RING > SUMS + SS ? RING : SUMS + SS;
  static_assert((NSTG - 1) * IPS < 64 && NSTG >= 2 && NSTG <= 4, "vmcnt");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
};

// w_row(r) / x_row(r): the K contiguous elements of the weight row / token row that tile row r stands for.  gain: [K] (NORM
// only).  K: a multiple of 64.  after_request(x, s0, n) runs once, behind the first requests (loads for the epilogue); with
// XL it also fills x, this wavefront's LDS for the token rows of its n steps from s0 on ([step][row][64], chunk ^= swz128(row)).
// On return acc[f][t] holds this wavefront's slice of the sums, ss[t] this lane's part of its token's sum of squares.
template <int NF, int NT, int WV, int NSTG, bool NORM, int XL = 0, class WRow, class XRow, class After>
__device__ __forceinline__ void slice_product(char *lds, WRow w_row, XRow x_row, const __bf16 *__restrict__ gain, int K, int wave, int lane,
                                              After after_request, f32x4 (&acc)[NF][NT], float (&ss)[NT]) {
  using S = Tile<NF, NT, WV, NSTG, NORM, XL>;
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[f][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < NT; ++t) ss[t] = 0.f;
  const int steps = K / 64;
  const int s0 = wave * steps / WV, n = (wave + 1) * steps / WV - s0;
  char *ring = lds + wave * (NSTG * S::STAGE + S::X_OWN), *const x_own = ring + NSTG * S::STAGE;
  if (n <= 0) {
    after_request(x_own, s0, 0);
    return;
  }
  const int l16 = lane & 15, g = lane >> 4;
  const __bf16 *src[S::W_INSTR + S::X_INSTR];
#pragma unroll
  for (int i = 0; i < S::W_INSTR; ++i) {
    const int row = i * 8 + (lane >> 3);
    src[i] = w_row(row) + s0 * 64 + ((lane & 7) ^ swz128(row & 15)) * 8;
  }
#pragma unroll
  for (int i = 0; i < S::X_INSTR; ++i) {
    const int row = i * 8 + (lane >> 3);
    src[S::W_INSTR + i] = x_row(row) + s0 * 64 + ((lane & 7) ^ swz128(row & 15)) * 8;
  }
  const __bf16 *gsrc = NORM ? gain + s0 * 64 + lane * 8 : nullptr;
  auto request = [&](int s, int st) __attribute__((always_inline)) {
    char *base = ring + st * S::STAGE;
#pragma unroll
    for (int i = 0; i < S::W_INSTR; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[i] + s * 64),
                                       (__attribute__((address_space(3))) void *)(base + i * 1024), 16, 0, 2);
#pragma unroll
    for (int i = S::W_INSTR; i < S::W_INSTR + S::X_INSTR; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[i] + s * 64),
                                       (__attribute__((address_space(3))) void *)(base + i * 1024), 16, 0, 0);
    if (NORM) {
      if (lane < 8)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gsrc + s * 64),
                                         (__attribute__((address_space(3))) void *)(base + (S::W_INSTR + S::X_INSTR) * 1024), 16, 0, 0);
    }
  };
#pragma unroll
  for (int s = 0; s < NSTG; ++s)
    if (s < n) request(s, s);
  after_request(x_own, s0, n);
  int rd[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) rd[ks] = l16 * ROW + ((4 * ks + g) ^ swz128(l16)) * 16;
  int st = 0;
  for (int s = 0; s < n; ++s) {
    const int later = min(NSTG - 1, n - 1 - s);  // stages in flight behind this one
    if (later >= 3) wait_vmcnt<(NSTG > 3 ? 3 : 0) * S::IPS>();
    else if (later == 2) wait_vmcnt<(NSTG > 2 ? 2 : 0) * S::IPS>();
    else if (later == 1) wait_vmcnt<S::IPS>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const char *wb = ring + st * S::STAGE, *xb = XL ? x_own + s * (NT * 2048) : wb + S::W_INSTR * 1024, *gb = wb + (S::W_INSTR + S::X_INSTR) * 1024;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 w[NF], x[NT], gn;
#pragma unroll
      for (int f = 0; f < NF; ++f) w[f] = *(const bf16x8 *)(wb + f * 2048 + rd[ks]);
#pragma unroll
      for (int t = 0; t < NT; ++t) x[t] = *(const bf16x8 *)(xb + t * 2048 + rd[ks]);
      if (NORM) {
        gn = *(const bf16x8 *)(gb + (4 * ks + g) * 16);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float v = (float)x[t][e];
            ss[t] = __builtin_fmaf(v, v, ss[t]);
            x[t][e] = (__bf16)(v * (float)gn[e]);
          }
      }
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[f], x[t], acc[f][t], 0, 0, 0);
    }
    if (s + NSTG < n) {
      __builtin_amdgcn_s_waitcnt(0xf | (7 << 4) | (3 << 14));  // every read of the stage is in registers (lgkmcnt 0)
      asm volatile("" ::: "memory");
      request(s + NSTG, st);
    }
    st = st + 1 == NSTG ? 0 : st + 1;
  }
}

// Stores this wavefront's slice; behind the barrier every thread may take sums with tile_sum / the norm with row_factor.
template <int NF, int NT, int WV, int NSTG, bool NORM>
__device__ __forceinline__ void share_slices(char *lds, int wave, int lane, const f32x4 (&acc)[NF][NT], float (&ss)[NT]) {
  __syncthreads();  // the other wavefronts' rings end here
  f32x4 *p = (f32x4 *)lds + (size_t)wave * (NF * NT) * 64 + lane;
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int t = 0; t < NT; ++t) p[(f * NT + t) * 64] = acc[f][t];
  if (NORM) {
    float *q = (float *)(lds + Tile<NF, NT, WV, NSTG, NORM>::SUMS);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float s = ss[t];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (lane < 16) q[(wave * NT + t) * 16 + lane] = s;
    }
  }
  __syncthreads();
}
template <int NF, int NT, int WV>
__device__ __forceinline__ f32x4 tile_sum(const char *lds, int f, int t, int lane) {
  const f32x4 *p = (const f32x4 *)lds + (f * NT + t) * 64 + lane;
  f32x4 s = p[0];
#pragma unroll
  for (int w = 1; w < WV; ++w) s += p[(size_t)w * (NF * NT) * 64];
  return s;
}
// rsqrt(mean(x^2) + eps) of token t * 16 + l16
template <int NF, int NT, int WV>
__device__ __forceinline__ float row_factor(const char *lds, int t, int l16, int K, float eps) {
  const float *q = (const float *)(lds + WV * NF * NT * 1024) + t * 16 + l16;
  float s = q[0];
#pragma unroll
  for (int w = 1; w < WV; ++w) s += q[w * NT * 16];
  return 1.0f / sqrtf(s / (float)K + eps);
}

// workgroup id -> (weight tile, token tile): the token tiles of one weight tile are neighbours on ONE XCD (ids go
// round-robin over the 8), so its rows are fetched into one L2 once.  false: a surplus workgroup.
__device__ __forceinline__ bool place(int id, int n_wt, int n_tt, int &wt, int &tt) {
  const int j = id >> 3;
  wt = (j / n_tt) * 8 + (id & 7);
  tt = j % n_tt;
  return wt < n_wt;
}
inline unsigned grid_of(int n_wt, int n_tt) { return (unsigned)((n_wt + 7) / 8 * 8 * n_tt); }

// Tile of a launch over M token rows and n16 blocks of 16 weight rows: (NF, NT) with the least time, taken as rounds of
// one workgroup per CU times the rows a workgroup reads.  Measured at 128 rows x (N x K): 4096 x 1024 (2,4) 6.2, (4,4)
// 8.0, (2,2) 8.3, (1,2) 11.9 us -- costs 6, 8, 8, 12; 6144 x 1024 (4,4) 8.4, (2,4) 10.9 -- 8, 12.  min_nf: the caller's
// smallest NF.  The candidates are the tiles the kernels are instantiated for; a tie takes the first.  48-row token tiles save the
// padding of the 64-row ones at 65 to 96 rows and their like (layer of width 3072 with head norms, 80 rows: 125 us with 64-row tiles,
// 112 with these); beyond 256 rows there is little of it and they read the weights more often (width 896, 400 rows: 77 | 86).
// three: 48 weight rows x 64 token rows too (24 features of gate and up).  Where 64 weight rows leave CUs without a workgroup these fill them with 7/8
// of the bytes each: gate and up of ffn 3072 at 65 to 128 rows, 192 workgroups | 256: 28 layers of width 1024 over 128 rows 1541 | 1525 us.
struct Choice {
  int nf, nt;
  long cost;
};
inline Choice choose_tile(int n_cu, int M, int n16, int min_nf, bool three = false) {
  static const Choice cand[] = {{1, 1, 0}, {1, 2, 0}, {2, 1, 0}, {2, 2, 0}, {2, 3, 0}, {2, 4, 0}, {3, 4, 0}, {4, 3, 0}, {4, 4, 0}};
  Choice best{0, 0, 0};
  for (const Choice &c : cand) {
    if (c.nf < min_nf || n16 % c.nf || (c.nf == 3 && !three) || (c.nt == 3 && M > 256)) continue;
    const long tiles = (long)(n16 / c.nf) * ((M + 16 * c.nt - 1) / (16 * c.nt));
    const long cost = (tiles + n_cu - 1) / n_cu * (c.nf + c.nt);
    if (!best.nf || cost < best.cost) best = Choice{c.nf, c.nt, cost};
  }
  return best;
}
// Whether a projection with a norm in front (or none) is faster here than on the 128-row tiles behind a norm kernel: these read
// 64 rows of weights and of tokens per workgroup and round, so beyond two rounds of the largest tile (cost 16) the 128-row
// tiles win.  us at width 1024: gate and up projections of ffn 3072 20 in two rounds (320 rows), 29 in three (512), 55 in six (1000)
// against 14 to 21 and 5 for the norm; QKV of 4096 features 13 | 21 | 30 in one, two, three rounds (256, 512, 640 rows) against 17
// and 5; width 3072, 200 rows: gate and up (four rounds) 75 against 49 and 6, QKV (two) 38 against 49 and 6.  Up to 128 rows a
// token tile of the other kernels is mostly padding.  (The tiles of 48 weight rows change none of these answers: what costs up to 16 with them, two
// rounds, does so on the larger tiles too.)
inline bool pays(int n_cu, long M, int n16, int min_nf, long max_cost) { return M <= 128 || choose_tile(n_cu, (int)M, n16, min_nf).cost <= max_cost; }
// wavefronts and stages of a tile: what fits beside a second workgroup on the CU at one token block, else one per CU
template <int NF, int NT>
struct Form {
  static constexpr int WV = (NF == 1 || (NF == 2 && NT == 2)) ? 8 : 4;
  static constexpr int NSTG = NF == 1 && NT == 1 ? 2 : NF == 1 ? 3 : (NF == 2 && NT == 2) || NF >= 3 ? 2 : 3;
};

}  // namespace few
}  // namespace pc
