// The rest of a pre-norm transformer block around the cache-reusing attention module, on the retained (fresh)
// rows only, so that a stack of layers can be chained (App. B.1: after the attention module the computation
// goes on as in an ordinary block; the cached rows' activations are never needed again because the next layer
// crops them once more):
//   h' = h + (attention(RMSNorm(h) ...)) Wo^T,   h'' = h' + (silu(n Wgate^T) * (n Wup^T)) Wdown^T,  n = RMSNorm(h').
// Kernels: a row-wise RMSNorm, and the shared projection main loop with two epilogues (residual add; SwiGLU on a
// gate/up feature pair held by the same lane); for few token rows the same epilogues on the tiles of few_rows.hpp, which
// also take the RMSNorm in front of them.  percache_stack_reuse chains the layers; percache_kv_slice is the
// cache slicer of Sec. 4.1.1 (cuts the K/V of a prefilled sequence at chunk boundaries into slots).
#include <cstring>

#include "decode_stack.hpp"
#include "few_rows.hpp"

namespace {
using pc::f32x16;
using pc::f32x4;
using pc::u32x4;
using pc::gemm::BF;
using pc::gemm::pack4;
using pc::gemm::unpack4;

constexpr int kXcds = 8;

// ---------------------------------------------------------------------------------------------------
// y = x / sqrt(mean(x^2) + eps) * gain; one wavefront per row, fp32 arithmetic, bf16 in and out.
// ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rmsnorm_kernel(const __bf16 *__restrict__ X, const __bf16 *__restrict__ gain,
                                                      __bf16 *__restrict__ Y, int M, int H, float eps) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const u32x4 *x = (const u32x4 *)(X + (size_t)row * H);
  const u32x4 *gv = (const u32x4 *)gain;
  u32x4 *y = (u32x4 *)(Y + (size_t)row * H);
  const int nv = H / 8;
  float ss = 0.f;
  for (int v = lane; v < nv; v += 64) {
    pc::bf16x8 h = __builtin_bit_cast(pc::bf16x8, x[v]);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += (float)h[e] * (float)h[e];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  const float r = 1.0f / sqrtf(ss / (float)H + eps);
  for (int v = lane; v < nv; v += 64) {
    pc::bf16x8 h = __builtin_bit_cast(pc::bf16x8, x[v]);
    pc::bf16x8 gq = __builtin_bit_cast(pc::bf16x8, gv[v]);
    pc::bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (__bf16)((float)h[e] * r * (float)gq[e]);
    y[v] = __builtin_bit_cast(u32x4, o);
  }
}

// ---------------------------------------------------------------------------------------------------
// Y[M, N] = A[M, K] W[N, K]^T + R[M, N]   (o_proj and down projection with the residual add fused)
// ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void linear_residual_kernel(const __bf16 *__restrict__ A, const __bf16 *__restrict__ W,
                                                                 const __bf16 *__restrict__ R, __bf16 *__restrict__ Y, int M,
                                                                 int N, int K) {
  constexpr int NTB = 2;
  constexpr int BT = 64 * NTB;
  __shared__ __align__(16) char lds[pc::gemm::Shape<NTB>::LDS_BYTES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wf = wave & 1, wt = wave >> 1;
  const int l32 = lane & 31, g = lane >> 5;
  const int f0 = blockIdx.x * BF, m0 = blockIdx.y * BT;
  f32x16 acc[2][NTB];
  pc::gemm::mainloop<NTB>(lds, [&](int row) __attribute__((always_inline)) { return W + (size_t)(f0 + row) * K; }, A, K, m0, M,
                          K, 2 * wf, 2 * wf + 1, acc);
#pragma unroll
  for (int t = 0; t < NTB; ++t) {
    const int m_raw = m0 + (wt * NTB + t) * 32 + l32;
    const bool ok = m_raw < M;
    const int m = ok ? m_raw : M - 1;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const size_t at = (size_t)m * N + f0 + (2 * wf + a) * 32 + q4 * 8 + g * 4;
        float res[4];
        unpack4(*(const uint2 *)(R + at), res);
        if (ok)
          *(uint2 *)(Y + at) = pack4(acc[a][t][q4 * 4 + 0] + res[0], acc[a][t][q4 * 4 + 1] + res[1],
                                   acc[a][t][q4 * 4 + 2] + res[2], acc[a][t][q4 * 4 + 3] + res[3]);
      }
  }
}

// The same for a launch of at most one workgroup per CU, on mainloop_deep.  Consecutive tiles (features first) sit on one XCD, so
// that its L2 holds few token rows.
template <int NTB, int NSTG>
__global__ __launch_bounds__(512) void linear_residual_deep_kernel(const __bf16 *__restrict__ A, const __bf16 *__restrict__ W,
                                                                   const __bf16 *__restrict__ R, __bf16 *__restrict__ Y, int M, int N, int K) {
  constexpr int BT = 64 * NTB;
  __shared__ __align__(16) char lds[pc::gemm::DeepShape<NTB, NSTG>::LDS_BYTES];
  const int n_ft = N / BF, tile = (int)(blockIdx.x % kXcds) * (int)(gridDim.x / kXcds) + (int)(blockIdx.x / kXcds);
  if (tile >= n_ft * ((M + BT - 1) / BT)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wf = wave & 1, wt = (wave >> 1) & 1, kh = wave >> 2;
  const int l32 = lane & 31, g = lane >> 5;
  const int f0 = tile % n_ft * BF, m0 = tile / n_ft * BT;
  f32x16 sum[NTB];
  pc::gemm::mainloop_deep<NTB, NSTG>(lds, [&](int row) __attribute__((always_inline)) { return W + (size_t)(f0 + row) * K; }, A, K, m0, M, K,
                                     2 * wf, 2 * wf + 1, wt, sum);
#pragma unroll
  for (int t = 0; t < NTB; ++t) {
    const int m = m0 + (wt * NTB + t) * 32 + l32;
    if (m >= M) continue;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const size_t at = (size_t)m * N + f0 + (2 * wf + kh) * 32 + q4 * 8 + g * 4;
      float res[4];
      unpack4(*(const uint2 *)(R + at), res);
      *(uint2 *)(Y + at) = pack4(sum[t][q4 * 4 + 0] + res[0], sum[t][q4 * 4 + 1] + res[1], sum[t][q4 * 4 + 2] + res[2], sum[t][q4 * 4 + 3] + res[3]);
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// Y[M, F] = silu(A Wgate^T) * (A Wup^T).  A workgroup takes 64 gate rows and the 64 up rows of the same
// features; wavefront wf owns gate block wf and up block wf + 2, so both halves of a product sit in one lane.
// ---------------------------------------------------------------------------------------------------
template <int NTB>
__device__ __forceinline__ void swiglu_tile(char *lds, const __bf16 *__restrict__ A, const __bf16 *__restrict__ Wg, const __bf16 *__restrict__ Wu,
                                            __bf16 *__restrict__ Y, int f0, int m0, int M, int F, int K) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wf = wave & 1, wt = wave >> 1;
  const int l32 = lane & 31, g = lane >> 5;
  f32x16 acc[2][NTB];
  pc::gemm::mainloop<NTB>(
      lds, [&](int row) __attribute__((always_inline)) { return (row < 64 ? Wg : Wu) + (size_t)(f0 + (row & 63)) * K; }, A, K, m0, M, K,
      wf, wf + 2, acc);
#pragma unroll
  for (int t = 0; t < NTB; ++t) {
    const int m_raw = m0 + (wt * NTB + t) * 32 + l32;
    const bool ok = m_raw < M;
    const int m = ok ? m_raw : M - 1;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float gate = acc[0][t][q4 * 4 + e], up = acc[1][t][q4 * 4 + e];
        o[e] = gate / (1.0f + __expf(-gate)) * up;
      }
      if (ok) *(uint2 *)(Y + (size_t)m * F + f0 + wf * 32 + q4 * 8 + g * 4) = pack4(o[0], o[1], o[2], o[3]);
    }
  }
}
// Token tiles of 64 * NTB rows, the first n_tall of them 64 rows taller (swiglu_tall); dynamic LDS: Shape<NTB or NTB + 1>::LDS_BYTES.
template <int NTB, bool TALL>
__global__ __launch_bounds__(256, 2) void linear_swiglu_kernel(const __bf16 *__restrict__ A, const __bf16 *__restrict__ Wg,
                                                               const __bf16 *__restrict__ Wu, __bf16 *__restrict__ Y, int M,
                                                               int F, int K, int n_tall) {
  extern __shared__ __align__(16) char lds[];
  const int f0 = blockIdx.x * (BF / 2), y = blockIdx.y;
  if constexpr (TALL)
    if (y < n_tall) {
      swiglu_tile<NTB + 1>(lds, A, Wg, Wu, Y, f0, y * 64 * (NTB + 1), M, F, K);
      return;
    }
  swiglu_tile<NTB>(lds, A, Wg, Wu, Y, f0, 64 * (NTB * y + (TALL ? n_tall : 0)), M, F, K);
}

// ---------------------------------------------------------------------------------------------------
// Few token rows: the whole contraction in one launch, see few_rows.hpp.
// ---------------------------------------------------------------------------------------------------
// Y[M, N] = A[M, K] W[N, K]^T + R[M, N]   (o_proj and down projection)
template <int NF, int NT>
__global__ __launch_bounds__((64 * pc::few::Form<NF, NT>::WV)) void linear_residual_few_kernel(const __bf16 *__restrict__ A, const __bf16 *__restrict__ W,
                                                                                             const __bf16 *__restrict__ R, __bf16 *__restrict__ Y,
                                                                                             int M, int N, int K, int n_wt, int n_tt) {
  constexpr int WV = pc::few::Form<NF, NT>::WV, NSTG = pc::few::Form<NF, NT>::NSTG, PER = (NF * NT + WV - 1) / WV;
  __shared__ __align__(16) char lds[pc::few::Tile<NF, NT, WV, NSTG, false>::LDS_BYTES];
  int wt, tt;
  if (!pc::few::place(blockIdx.x, n_wt, n_tt, wt, tt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g = lane >> 4;
  const int n0 = wt * 16 * NF, m0 = tt * 16 * NT;
  auto at = [&](int b) __attribute__((always_inline)) { return (size_t)min(m0 + b % NT * 16 + l16, M - 1) * N + n0 + b / NT * 16 + g * 4; };
  uint2 res[PER];
  f32x4 acc[NF][NT];
  float ss[NT];
  pc::few::slice_product<NF, NT, WV, NSTG, false>(
      lds, [&](int r) __attribute__((always_inline)) { return W + (size_t)(n0 + r) * K; },
      [&](int r) __attribute__((always_inline)) { return A + (size_t)min(m0 + r, M - 1) * K; }, nullptr, K, wave, lane,
      [&](char *, int, int) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
          if (wave + j * WV < NF * NT) res[j] = *(const uint2 *)(R + at(wave + j * WV));
      },
      acc, ss);
  pc::few::share_slices<NF, NT, WV, NSTG, false>(lds, wave, lane, acc, ss);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int b = wave + j * WV;
    if (b >= NF * NT) continue;
    const f32x4 s = pc::few::tile_sum<NF, NT, WV>(lds, b / NT, b % NT, lane);
    float r[4];
    unpack4(res[j], r);
    if (m0 + b % NT * 16 + l16 < M) *(uint2 *)(Y + at(b)) = pack4(s[0] + r[0], s[1] + r[1], s[2] + r[2], s[3] + r[3]);
  }
}

// The o_proj of a decoding step of a few rows straight from the attention's split-KV partials: every wavefront merges the
// rows it contracts (its slice of the heads) into LDS under the latency of its first weights, by the rule of
// splitkv_combine_kernel (m = max m_s, weights l_s 2^(m_s - m), rounded to bf16 once), instead of a launch that merges and
// one that reads the result back.  Lanes l and l + 32 share 8 columns of a row and take every other partition.
constexpr int kMergeSteps = 8;   // steps of 64 columns per wavefront: up to 4096 columns
__global__ __launch_bounds__(512) void oproj_merge_few_kernel(const float *__restrict__ part_o, const float *__restrict__ part_ml, int n_splits, int T,
                                                              int Hkv, int G, int D, const __bf16 *__restrict__ W, const __bf16 *__restrict__ R,
                                                              __bf16 *__restrict__ Y, int M, int N, int K, int n_wt) {
  constexpr int WV = 8, NSTG = 2, CH = 10;
  __shared__ __align__(16) char lds[pc::few::Tile<1, 1, WV, NSTG, false, kMergeSteps>::LDS_BYTES];
  int wt, tt;
  if (!pc::few::place(blockIdx.x, n_wt, 1, wt, tt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g = lane >> 4;
  const int n0 = wt * 16;
  const size_t at = (size_t)min(l16, M - 1) * N + n0 + g * 4;
  uint2 res = make_uint2(0, 0);
  f32x4 acc[1][1];
  float ss[1];
  pc::few::slice_product<1, 1, WV, NSTG, false, kMergeSteps>(
      lds, [&](int r) __attribute__((always_inline)) { return W + (size_t)(n0 + r) * K; }, [](int) { return (const __bf16 *)nullptr; }, nullptr, K, wave,
      lane,
      [&](char *x, int s0, int n) __attribute__((always_inline)) {
        if (wave == 0) res = *(const uint2 *)(R + at);
        const int half = lane >> 5;
        for (int u = lane & 31; u < M * n * 8; u += 32) {
          const int c = u & 7, q = u >> 3, step = q % n, m = q / n;
          const int k = (s0 + step) * 64 + c * 8, head = k / D, b = m / T, i = m - b * T;
          const size_t prow = ((((size_t)b * Hkv + head / G) * G + head % G) * T + i) * n_splits;
          const float2 *ml = (const float2 *)part_ml + prow;
          const float *po = part_o + prow * D + (k - head * D);
          float mx = -INFINITY, wsum = 0.f, a8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          for (int r0 = 0; r0 < n_splits; r0 += 2 * CH) {
            float2 e[CH];
            f32x4 o[CH][2];
#pragma unroll
            for (int j = 0; j < CH; ++j) {
              if (r0 + 2 * j >= n_splits) break;
              const int sp = min(r0 + half + 2 * j, n_splits - 1);
              e[j] = ml[sp];
              o[j][0] = *(const f32x4 *)(po + (size_t)sp * D);
              o[j][1] = *(const f32x4 *)(po + (size_t)sp * D + 4);
            }
            float top = mx;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
              if (r0 + 2 * j >= n_splits) break;
              if (r0 + half + 2 * j >= n_splits || !(e[j].y > 0.f)) e[j] = make_float2(-INFINITY, 0.f);   // (an empty partition has weight 0)
              top = fmaxf(top, e[j].x);
            }
            const float shrink = mx == -INFINITY ? 0.f : exp2f(mx - top);
            mx = top;
            wsum *= shrink;
#pragma unroll
            for (int e8 = 0; e8 < 8; ++e8) a8[e8] *= shrink;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
              if (r0 + 2 * j >= n_splits) break;
              const float w = e[j].y > 0.f ? e[j].y * exp2f(e[j].x - top) : 0.f;
              wsum += w;
#pragma unroll
              for (int e8 = 0; e8 < 8; ++e8) a8[e8] += w * o[j][e8 >> 2][e8 & 3];
            }
          }
          const float m2 = __shfl_xor(mx, 32, 64), both = fmaxf(mx, m2);
          const float mine = mx == -INFINITY ? 0.f : exp2f(mx - both);
          wsum *= mine;
          wsum += __shfl_xor(wsum, 32, 64);
          pc::bf16x8 v;
          const float inv = wsum > 0.f ? 1.0f / wsum : 0.f;
#pragma unroll
          for (int e8 = 0; e8 < 8; ++e8) {
            const float t = a8[e8] * mine;
            v[e8] = (__bf16)((t + __shfl_xor(t, 32, 64)) * inv);
          }
          // (a store the compiler does not see: behind an ordinary one it waits for every request before each operand read)
          const unsigned addr = (unsigned)(size_t)(__attribute__((address_space(3))) char *)x + step * 2048 + m * 128 + ((c ^ pc::gemm::swz128(m)) * 16);
          if (half == 0) asm volatile("ds_write_b128 %0, %1" : : "v"(addr), "v"(v) : "memory");
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      },
      acc, ss);
  pc::few::share_slices<1, 1, WV, NSTG, false>(lds, wave, lane, acc, ss);
  if (wave != 0 || l16 >= M) return;
  const f32x4 s = pc::few::tile_sum<1, 1, WV>(lds, 0, 0, lane);
  float r[4];
  unpack4(res, r);
  *(uint2 *)(Y + at) = pack4(s[0] + r[0], s[1] + r[1], s[2] + r[2], s[3] + r[3]);
}

// Y[M, F] = silu(n Wgate^T) * (n Wup^T) with n = RMSNorm(A; gain, eps).  Weight blocks 0 .. NF/2 - 1 of a tile are gate
// rows, the others the up rows of the same features.
template <int NF, int NT>
__global__ __launch_bounds__((64 * pc::few::Form<NF, NT>::WV)) void swiglu_few_kernel(const __bf16 *__restrict__ A, const __bf16 *__restrict__ gain, float eps,
                                                                                    const __bf16 *__restrict__ Wg, const __bf16 *__restrict__ Wu,
                                                                                    __bf16 *__restrict__ Y, int M, int F, int K, int n_wt, int n_tt) {
  // a tile's weight rows: FEAT of the gate, then the up rows of the same features; four features x 16 tokens are a unit of the epilogue
  constexpr int WV = pc::few::Form<NF, NT>::WV, NSTG = pc::few::Form<NF, NT>::NSTG, FEAT = 8 * NF, QUADS = FEAT / 4;
  static_assert(QUADS * NT % 4 == 0, "units of whole wavefronts");
  __shared__ __align__(16) char lds[pc::few::Tile<NF, NT, WV, NSTG, true>::LDS_BYTES];
  int wt, tt;
  if (!pc::few::place(blockIdx.x, n_wt, n_tt, wt, tt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g = lane >> 4;
  const int f0 = wt * FEAT, m0 = tt * 16 * NT;
  f32x4 acc[NF][NT];
  float ss[NT];
  pc::few::slice_product<NF, NT, WV, NSTG, true>(
      lds, [&](int r) __attribute__((always_inline)) { return (r < FEAT ? Wg + (size_t)(f0 + r) * K : Wu + (size_t)(f0 + r - FEAT) * K); },
      [&](int r) __attribute__((always_inline)) { return A + (size_t)min(m0 + r, M - 1) * K; }, gain, K, wave, lane, [](char *, int, int) {}, acc, ss);
  pc::few::share_slices<NF, NT, WV, NSTG, true>(lds, wave, lane, acc, ss);
#pragma unroll
  for (int b = wave; b < QUADS * NT / 4; b += WV) {
    const int t = (b * 4 + g) / QUADS, q = (b * 4 + g) % QUADS, qu = q + QUADS, m = m0 + t * 16 + l16;
    const float r = pc::few::row_factor<NF, NT, WV>(lds, t, l16, K, eps);
    const f32x4 gate = pc::few::tile_sum<NF, NT, WV>(lds, q / 4, t, q % 4 * 16 + l16) * r, up = pc::few::tile_sum<NF, NT, WV>(lds, qu / 4, t, qu % 4 * 16 + l16) * r;
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = gate[e] / (1.0f + __expf(-gate[e])) * up[e];
    if (m < M) *(uint2 *)(Y + (size_t)m * F + f0 + q * 4) = pack4(o[0], o[1], o[2], o[3]);
  }
}

bool aligned16(const void *p) { return ((uintptr_t)p % 16) == 0; }

pc_status launch_rmsnorm(percache_ctx *ctx, const __bf16 *x, const __bf16 *gain, __bf16 *y, int M, int H, float eps,
                         hipStream_t s) {
  hipLaunchKernelGGL(rmsnorm_kernel, dim3((M + 3) / 4), dim3(256), 0, s, x, gain, y, M, H, eps);
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}
// Token rows per tile of linear_residual_deep_kernel where its tiles go to the CUs in one round, else 0: there the two-stage
// loop has about one workgroup per CU and waits out every stage's round trip; in several rounds its two workgroups per CU cover
// each other.  4224 rows x 1024 features, 192-token tiles (176 of them; of 128 tokens they are 264): 33 us over 2048 elements and
// 44 over 3072, where the two-stage loop took 50 on average (0.68 us a k-step, 10 TB/s of operands out of L2, is what bounds it).
int deep_tokens(int n_cu, int M, int N) {
  for (int bt = 128; bt <= 192; bt += 64)
    if (M > bt && (long)(N / BF) * ((M + bt - 1) / bt) <= n_cu) return bt;
  return 0;
}
pc_status launch_linear_residual(percache_ctx *ctx, const __bf16 *a, const __bf16 *w, const __bf16 *res, __bf16 *y, int M,
                                 int N, int K, hipStream_t s) {
  const int deep = deep_tokens(ctx->n_cu, M, N);
  if (deep) {
    const int tiles = N / BF * ((M + deep - 1) / deep);
    const dim3 grid((tiles + kXcds - 1) / kXcds * kXcds);
    if (deep == 128) hipLaunchKernelGGL((linear_residual_deep_kernel<2, 4>), grid, dim3(512), 0, s, a, w, res, y, M, N, K);
    else hipLaunchKernelGGL((linear_residual_deep_kernel<3, 4>), grid, dim3(512), 0, s, a, w, res, y, M, N, K);
    PC_HIP(ctx, hipGetLastError());
    return PC_OK;
  }
  hipLaunchKernelGGL(linear_residual_kernel, dim3(N / BF, (M + 127) / 128), dim3(256), 0, s, a, w, res, y, M, N, K);
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}
// How many of the first token tiles take 192 rows instead of 128, where that saves the launch its last round of two workgroups per CU (a
// taller tile costs the slot it is in half a tile, the round a whole one for the few tiles left over).  us a layer, 128 rows | with taller
// ones: width 1024, 1300 rows (48 feature tiles, 528 tiles) 148.5 | 142, 1900 163.4 | 160.3, 4224 (1584 tiles, 2 taller) 291 | 287; width 896,
// 1024 rows 102.6 | 99.0; width 3072, 2176 601 | 589, 4224 1187 | 1165.
int swiglu_tall(int n_cu, int M, int fx) {
  const long slots = 2L * n_cu, nb = (M + 63) / 64, rounds = ((nb + 1) / 2 * fx + slots - 1) / slots;
  const long column = (rounds - 1) * slots / fx, tall = nb - 2 * column;   // (token tiles of a feature tile that one round less has room for)
  return column > 0 && tall > 0 && tall <= column && tall * fx <= slots ? (int)tall : 0;
}
pc_status launch_linear_swiglu(percache_ctx *ctx, const __bf16 *a, const __bf16 *wg, const __bf16 *wu, __bf16 *y, int M, int F,
                               int K, hipStream_t s) {
  const int fx = F / (BF / 2);
  if (M <= 64 * 3) {
    hipLaunchKernelGGL((linear_swiglu_kernel<1, false>), dim3(fx, (M + 63) / 64), dim3(256), pc::gemm::Shape<1>::LDS_BYTES, s, a, wg, wu, y, M, F, K, 0);
  } else if (const int tall = swiglu_tall(ctx->n_cu, M, fx)) {
    constexpr int lds_bytes = pc::gemm::Shape<3>::LDS_BYTES;
    PC_HIP(ctx, hipFuncSetAttribute((const void *)linear_swiglu_kernel<2, true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
    const int rest = (M + 63) / 64 - 3 * tall;
    hipLaunchKernelGGL((linear_swiglu_kernel<2, true>), dim3(fx, tall + (rest > 0 ? (rest + 1) / 2 : 0)), dim3(256), lds_bytes, s, a, wg, wu, y, M, F, K, tall);
  } else {
    hipLaunchKernelGGL((linear_swiglu_kernel<2, false>), dim3(fx, (M + 127) / 128), dim3(256), pc::gemm::Shape<2>::LDS_BYTES, s, a, wg, wu, y, M, F, K, 0);
  }
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}

pc_status launch_residual_few(percache_ctx *ctx, const __bf16 *a, const __bf16 *w, const __bf16 *res, __bf16 *y, int M, int N, int K,
                              hipStream_t s) {
  const pc::few::Choice c = pc::few::choose_tile(ctx->n_cu, M, N / 16, 1);
  const int n_wt = N / (16 * c.nf), n_tt = (M + 16 * c.nt - 1) / (16 * c.nt);
#define PC_FEW(NF, NT)                                                                                                        \
  if (c.nf == NF && c.nt == NT)                                                                                               \
  hipLaunchKernelGGL((linear_residual_few_kernel<NF, NT>), dim3(pc::few::grid_of(n_wt, n_tt)), dim3(64 * pc::few::Form<NF, NT>::WV), 0, s, a, w, \
                     res, y, M, N, K, n_wt, n_tt)
  PC_FEW(1, 1); else PC_FEW(2, 1); else PC_FEW(1, 2); else PC_FEW(2, 2); else PC_FEW(2, 3); else PC_FEW(2, 4); else PC_FEW(4, 3); else PC_FEW(4, 4);
#undef PC_FEW
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}
// Up to how many of the attention's partials the o_proj of M rows merges itself (0: none).  A wavefront's share is M * steps * 8
// pieces of 8 columns (steps of 64 columns), 32 to a round of its lane pairs, and every workgroup reads all the partials: 30 where
// that is one round, 10 where it is two.  Layer, the o_proj merging | a merge launch of its own, us: one row of 2048 (one round) 11
// partitions 29.5 | 31.2, 25 32.4 | 33.2, 29 33.0 | 33.0, 31 32.8 | 32.6; of 896 13 29.8 | 31.0, 31 31.6 | 31.7, 61 35.4 | 34.2; two rows
// of 2048 (two rounds) 7 30.4 | 31.0, 11 31.7 | 31.9, 13 32.3 | 32.1, 16 33.2 | 32.2; one of 3072 9 54.6 | 54.7, 11 54.7 | 54.4, 19
// 56.5 | 55.1.
int oproj_merge_limit(const percache_config &c, long M) {
  const int steps = (c.n_q_heads * c.head_dim + 511) / 512;
  return steps > kMergeSteps || M * steps > 8 ? 0 : M * steps <= 4 ? 30 : 10;
}
pc_status launch_oproj_merge(percache_ctx *ctx, const float *part_o, const float *part_ml, int n_splits, int t_fresh, const __bf16 *w,
                             const __bf16 *res, __bf16 *y, int M, hipStream_t s) {
  const percache_config &c = ctx->cfg;
  const int n_wt = c.hidden / 16;
  hipLaunchKernelGGL(oproj_merge_few_kernel, dim3(pc::few::grid_of(n_wt, 1)), dim3(512), 0, s, part_o, part_ml, n_splits, t_fresh, c.n_kv_heads,
                     c.n_q_heads / c.n_kv_heads, c.head_dim, w, res, y, M, c.hidden, c.n_q_heads * c.head_dim, n_wt);
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}
pc_status launch_swiglu_few(percache_ctx *ctx, const __bf16 *a, const __bf16 *gain, float eps, const __bf16 *wg, const __bf16 *wu, __bf16 *y, int M,
                            int F, int K, hipStream_t s) {
  const pc::few::Choice c = pc::few::choose_tile(ctx->n_cu, M, 2 * F / 16, 2, true);
  const int n_wt = 2 * F / (16 * c.nf), n_tt = (M + 16 * c.nt - 1) / (16 * c.nt);
#define PC_FEW(NF, NT)                                                                                                    \
  if (c.nf == NF && c.nt == NT)                                                                                           \
  hipLaunchKernelGGL((swiglu_few_kernel<NF, NT>), dim3(pc::few::grid_of(n_wt, n_tt)), dim3(64 * pc::few::Form<NF, NT>::WV), 0, s, a, gain, eps, \
                     wg, wu, y, M, F, K, n_wt, n_tt)
  PC_FEW(2, 1); else PC_FEW(2, 2); else PC_FEW(2, 3); else PC_FEW(2, 4); else PC_FEW(3, 4); else PC_FEW(4, 3); else PC_FEW(4, 4);
#undef PC_FEW
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}

// Workspace of the stack call: the prefill workspace followed by the block's own activations.
struct StackWs {
  pc::PrefillWs pf;
  __bf16 *normed;  // [M, H]
  __bf16 *attn;    // [M, Hq*D]
  __bf16 *mid;     // [M, H]
  __bf16 *act;     // [M, F]
  void *steps;     // behind them, where there is room: of a step in one launch (decode_stack.hip)
  size_t total;    // without that
};
StackWs carve_stack_ws(const percache_ctx *ctx, void *base, int batch, int t_fresh, int max_chunks, int ffn) {
  const percache_config &c = ctx->cfg;
  StackWs w;
  w.pf = pc::carve_prefill_ws(c, ctx->n_cu, base, batch, t_fresh, max_chunks);
  size_t off = w.pf.total;
  char *p = (char *)base;
  auto take = [&](size_t bytes) { char *r = p ? p + off : nullptr; off += pc::align_up(bytes); return (__bf16 *)r; };
  const size_t M = (size_t)batch * t_fresh;
  w.normed = take(M * c.hidden * 2);
  w.attn = take(M * c.n_q_heads * c.head_dim * 2);
  w.mid = take(M * c.hidden * 2);
  w.act = take(M * ffn * 2);
  w.total = off;
  w.steps = p ? p + off : nullptr;
  return w;
}
// Bytes behind it that a step over the longest list of max_chunks chunks takes for all layers in one launch (0: no such step).
size_t steps_bytes(const percache_ctx *ctx, int batch, int t_fresh, int max_chunks, int ffn) {
  const percache_config &c = ctx->cfg;
  const long tiles = (long)max_chunks * (c.slot_capacity / pc::kKvTile);
  return pc::align_up(pc::stackdec::workspace_bytes(c, ctx->n_cu, batch, t_fresh, ffn, c.n_layers, tiles < INT32_MAX / 2 ? (int)tiles : INT32_MAX / 2));
}

}  // namespace

extern "C" {

pc_status percache_kv_slice(percache_ctx *ctx, int32_t layer, const void *k_dev, const void *v_dev, int32_t seq_len,
                            const int32_t *bounds_host, const int32_t *slots_host, int32_t n, void *stream) {
  if (!ctx) return PC_EINVAL;
  const percache_config &c = ctx->cfg;
  if (!k_dev || !v_dev || !bounds_host || !slots_host) return pc::fail(ctx, PC_EINVAL, "NULL pointer");
  if (!aligned16(k_dev) || !aligned16(v_dev)) return pc::fail(ctx, PC_EINVAL, "k_dev / v_dev must be 16-byte aligned");
  if (n < 1 || seq_len < 1) return pc::fail(ctx, PC_EINVAL, "n and seq_len must be positive");
  if (layer < 0 || layer >= c.n_layers) return pc::fail(ctx, PC_ESLOT, "layer %d out of range [0,%d)", layer, c.n_layers);
  for (int j = 0; j < n; ++j) {
    const int lo = bounds_host[j], hi = bounds_host[j + 1];
    if (lo < 0 || hi > seq_len || hi <= lo) return pc::fail(ctx, PC_ELEN, "chunk %d: bounds [%d,%d) not inside [0,%d)", j, lo, hi, seq_len);
    if (slots_host[j] < 0) continue;
    if (hi - lo > c.slot_capacity) return pc::fail(ctx, PC_ELEN, "chunk %d: %d tokens exceed the slot capacity %d", j, hi - lo, c.slot_capacity);
    if (slots_host[j] >= c.n_slots) return pc::fail(ctx, PC_ESLOT, "chunk %d: slot %d out of range [0,%d)", j, slots_host[j], c.n_slots);
    for (int i = 0; i < j; ++i)
      if (slots_host[i] == slots_host[j]) return pc::fail(ctx, PC_EINVAL, "slot %d appears twice", slots_host[j]);
  }
  const pc_status st = pc::launch_kv_slices(ctx, layer, slots_host, bounds_host, n, 1, (const __bf16 *)k_dev, (const __bf16 *)v_dev, seq_len,
                                            (hipStream_t)stream);
  if (st != PC_OK) return st;
  for (int j = 0; j < n; ++j)
    if (slots_host[j] >= 0) ctx->slot_len[(size_t)layer * c.n_slots + slots_host[j]] = bounds_host[j + 1] - bounds_host[j];
  return PC_OK;
}

size_t percache_stack_workspace_bytes(const percache_ctx *ctx, int32_t batch, int32_t t_fresh, int32_t max_chunks, int32_t ffn) {
  if (!ctx || batch < 1 || t_fresh < 1 || max_chunks < 0 || ffn < 1) return 0;
  return carve_stack_ws(ctx, nullptr, batch, t_fresh, max_chunks, ffn).total + steps_bytes(ctx, batch, t_fresh, max_chunks, ffn);
}

static pc_status run_stack(percache_ctx *ctx, const percache_block_weights *layers_host, int32_t n_layers, int32_t ffn,
                           float eps, const void *h_in_dev, int32_t batch, int32_t t_fresh,
                           const int32_t *slot_ids_host, const int32_t *used_len_host, const int32_t *n_chunks_host,
                           int32_t max_chunks, const int32_t *save_bounds_host, const int32_t *save_slots_host,
                           int32_t n_save, const int32_t *append_slots_host, void *h_out_dev, void *workspace_dev,
                           size_t workspace_bytes, void *stream, const int32_t *table_dev = nullptr,
                           const pc_table_shadow *shadow = nullptr) {
  if (!ctx) return PC_EINVAL;
  const percache_config &c = ctx->cfg;
  if (append_slots_host && batch >= 1 && t_fresh >= 1) {
    for (int b = 0; b < batch; ++b) {
      const int slot = append_slots_host[b];
      if (slot < 0) continue;
      if (slot >= c.n_slots) return pc::fail(ctx, PC_ESLOT, "append slot %d out of range [0,%d)", slot, c.n_slots);
      for (int bb = 0; bb < b; ++bb)
        if (append_slots_host[bb] == slot) return pc::fail(ctx, PC_EINVAL, "append slot %d appears twice", slot);
      for (int l = 0; l < n_layers && l < c.n_layers; ++l) {
        const int have = ctx->slot_len[(size_t)l * c.n_slots + slot];
        if (have != ctx->slot_len[slot]) return pc::fail(ctx, PC_ELEN, "append slot %d holds different lengths in layers 0 and %d", slot, l);
        if (have + t_fresh > c.slot_capacity)
          return pc::fail(ctx, PC_ELEN, "append slot %d holds %d tokens: %d more do not fit the capacity %d", slot, have, t_fresh, c.slot_capacity);
      }
    }
  }
  if (!layers_host || !h_in_dev || !h_out_dev) return pc::fail(ctx, PC_EINVAL, "NULL pointer");
  if (n_layers < 1 || n_layers > c.n_layers) return pc::fail(ctx, PC_ESHAPE, "n_layers %d outside [1,%d]", n_layers, c.n_layers);
  if (ffn < 64 || ffn % 64) return pc::fail(ctx, PC_ESHAPE, "ffn %d must be a positive multiple of 64", ffn);
  if (c.hidden % BF) return pc::fail(ctx, PC_ESHAPE, "hidden %d must be a multiple of %d for the block projections", c.hidden, BF);
  if (!(eps > 0.f)) return pc::fail(ctx, PC_EINVAL, "eps must be positive");
  if (!aligned16(h_in_dev) || !aligned16(h_out_dev)) return pc::fail(ctx, PC_EINVAL, "tensor pointers must be 16-byte aligned");
  if (n_save < 0 || (n_save > 0 && (!save_bounds_host || !save_slots_host))) return pc::fail(ctx, PC_EINVAL, "bad save arguments");
  for (int l = 0; l < n_layers; ++l) {
    const percache_block_weights &w = layers_host[l];
    const void *ptrs[7] = {w.gain1, w.wqkv, w.wo, w.gain2, w.w_gate, w.w_up, w.w_down};
    for (const void *p : ptrs)
      if (!p || !aligned16(p)) return pc::fail(ctx, PC_EINVAL, "layer %d: NULL or misaligned weight pointer", l);
    const void *opt[3] = {w.qkv_bias, w.q_norm, w.k_norm};
    for (const void *p : opt)
      if (p && !aligned16(p)) return pc::fail(ctx, PC_EINVAL, "layer %d: misaligned optional weight pointer", l);
  }
  // chunk tables of every layer (the slot table is per layer): all must agree, so that one upload serves the stack
  std::vector<int32_t> rows, rows_l;
  pc_status st = pc::build_chunk_table(ctx, 0, batch, t_fresh, slot_ids_host, used_len_host, n_chunks_host, max_chunks, rows);
  if (st != PC_OK) return st;
  for (int l = 1; l < n_layers; ++l) {
    st = pc::build_chunk_table(ctx, l, batch, t_fresh, slot_ids_host, used_len_host, n_chunks_host, max_chunks, rows_l);
    if (st != PC_OK) return st;
    if (rows_l != rows) return pc::fail(ctx, PC_ELEN, "the chunks' stored lengths differ between layer 0 and layer %d", l);
  }
  if (shadow && rows != shadow->rows)
    return pc::fail(ctx, PC_ELEN, "the slots' formats or lengths no longer match the device chunk table: put it again");
  const int formats = pc::table_formats(rows, pc::tbl_stride(max_chunks), batch);
  const long M = (long)batch * t_fresh;
  if (M * (long)(ffn > c.hidden ? ffn : c.hidden) >= (1L << 31)) return pc::fail(ctx, PC_ESHAPE, "activation larger than 2^31 elements");
  if ((long)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim * c.hidden >= (1L << 31)) return pc::fail(ctx, PC_ESHAPE, "operand larger than 2^31 elements");
  for (int b = 0; b < batch && n_save > 0; ++b) {
    for (int j = 0; j < n_save; ++j) {
      const int lo = save_bounds_host[j], hi = save_bounds_host[j + 1], slot = save_slots_host[(size_t)b * n_save + j];
      if (lo < 0 || hi > t_fresh || hi <= lo) return pc::fail(ctx, PC_ELEN, "save chunk %d: bounds [%d,%d) not inside [0,%d)", j, lo, hi, t_fresh);
      if (slot < 0) continue;
      if (hi - lo > c.slot_capacity) return pc::fail(ctx, PC_ELEN, "save chunk %d: %d tokens exceed the slot capacity %d", j, hi - lo, c.slot_capacity);
      if (slot >= c.n_slots) return pc::fail(ctx, PC_ESLOT, "save chunk %d: slot %d out of range [0,%d)", j, slot, c.n_slots);
      // a slot being read by this very call must not be overwritten by it
      for (int bb = 0; bb < batch; ++bb)
        for (int ci = 0; ci < n_chunks_host[bb]; ++ci)
          if (slot_ids_host[(size_t)bb * max_chunks + ci] == slot) return pc::fail(ctx, PC_EINVAL, "save slot %d is also read by this call", slot);
      for (int k = 0; k < b * n_save + j; ++k)
        if (save_slots_host[k] == slot) return pc::fail(ctx, PC_EINVAL, "save slot %d appears twice", slot);
    }
  }
  StackWs ws = carve_stack_ws(ctx, workspace_dev, batch, t_fresh, max_chunks, ffn);
  if (!workspace_dev || workspace_bytes < ws.total) return pc::fail(ctx, PC_ENOMEM, "stack workspace has %zu bytes, need %zu", workspace_bytes, ws.total);
  if ((uintptr_t)workspace_dev % pc::kAlign) return pc::fail(ctx, PC_EINVAL, "workspace must be 256-byte aligned");
  const int stride = pc::tbl_stride(max_chunks);
  int min_tiles = INT32_MAX, max_cached = 0;
  for (int b = 0; b < batch; ++b) {
    int tiles = rows[(size_t)b * stride + 2] + (t_fresh + pc::kKvTile - 1) / pc::kKvTile;
    if (tiles < min_tiles) min_tiles = tiles;
    if (rows[(size_t)b * stride + 2] > max_cached) max_cached = rows[(size_t)b * stride + 2];
  }
  hipStream_t s = (hipStream_t)stream;
  // a decoding step of few rows: the attention kernel finishes q, k and v from the projection's sums and appends the fresh
  // K/V to bf16 slots itself; (slot, tokens it holds) of every query go to the device behind the chunk lists
  const bool decode = pc::decode_rows(c, t_fresh);
  bool raw_qkv = decode;  // (the sums of every layer)
  for (int l = 0; l < n_layers; ++l) raw_qkv = raw_qkv && pc::few_rows_qkv(ctx, M, layers_host[l].q_norm || layers_host[l].k_norm);
  bool append_kernel = append_slots_host != nullptr;  // some append is left to a kernel of its own
  if (raw_qkv && append_slots_host && !table_dev) {
    append_kernel = false;
    for (int b = 0; b < batch; ++b) {
      const int slot = append_slots_host[b];
      const bool here = slot >= 0 && !ctx->is8(slot);
      if (slot >= 0 && !here) append_kernel = true;
      rows.push_back(here ? slot : -1);
      rows.push_back(here ? ctx->slot_len[slot] : 0);
    }
  }
  if (table_dev) ws.pf.table = const_cast<int32_t *>(table_dev);  // the list is on the device already: nothing to copy
  // (the kernels whose timing was asked for are launched one by one, and so are those of a call whose workspace, one sized for another call,
  // has no room for the hand-over)
  if (raw_qkv && !(ctx->prof_mask & 6) && pc::stackdec::takes(c, ctx->n_cu, batch, t_fresh, ffn, n_layers, max_cached) &&
      workspace_bytes - ws.total >= pc::stackdec::workspace_bytes(c, ctx->n_cu, batch, t_fresh, ffn, n_layers, max_cached)) {
    const __bf16 *k, *v;
    size_t dense;
    st = pc::stackdec::launch(ctx, layers_host, n_layers, ffn, eps, (const __bf16 *)h_in_dev, batch, t_fresh, table_dev ? nullptr : &rows, ws.pf.table,
                              stride, append_slots_host && !table_dev, max_cached, formats, (__bf16 *)h_out_dev, ws.steps, &k, &v, &dense, s);
    if (st != PC_OK) return st;
    for (int l = 0; l < n_layers; ++l) {
      if (n_save > 0) {
        st = pc::launch_kv_slices(ctx, l, save_slots_host, save_bounds_host, n_save, batch, k + l * dense, v + l * dense, t_fresh, s);
        if (st != PC_OK) return st;
        for (int i = 0; i < batch * n_save; ++i)
          if (save_slots_host[i] >= 0)
            ctx->slot_len[(size_t)l * c.n_slots + save_slots_host[i]] = save_bounds_host[i % n_save + 1] - save_bounds_host[i % n_save];
      }
      if (append_kernel) {
        st = pc::launch_kv_append(ctx, l, append_slots_host, batch, true, k + l * dense, v + l * dense, t_fresh, s);
        if (st != PC_OK) return st;
      }
      for (int b = 0; b < batch && append_slots_host; ++b)
        if (append_slots_host[b] >= 0) ctx->slot_len[(size_t)l * c.n_slots + append_slots_host[b]] += t_fresh;
    }
    return PC_OK;
  }
  if (!table_dev) {
    st = pc::upload_table(ctx, rows, ws.pf.table, s);
    if (st != PC_OK) return st;
  }
  const int H = c.hidden, A = c.n_q_heads * c.head_dim;
  const __bf16 *h_cur = (const __bf16 *)h_in_dev;
  __bf16 *h_out = (__bf16 *)h_out_dev;
  for (int l = 0; l < n_layers; ++l) {
    const percache_block_weights &w = layers_host[l];
#define PC_TRY(call) do { st = (call); if (st != PC_OK) return st; } while (0)
    // few token rows: one launch per projection, the RMSNorms folded into the projections behind them
    const bool few = pc::few_rows(c, M), few_qkv = pc::few_rows_qkv(ctx, M, w.q_norm || w.k_norm);
    if (!few_qkv) PC_TRY(launch_rmsnorm(ctx, h_cur, (const __bf16 *)w.gain1, ws.normed, (int)M, H, eps, s));
    pc::QkvExtras extras;
    extras.bias = (const __bf16 *)w.qkv_bias;
    extras.q_norm = (const __bf16 *)w.q_norm;
    extras.k_norm = (const __bf16 *)w.k_norm;
    extras.eps = eps;
    extras.pre_norm = few_qkv ? (const __bf16 *)w.gain1 : nullptr;
    pc::RawQkv raw;
    int left_splits = oproj_merge_limit(c, M);  // most partials, then those that the attention left, for the o_proj to merge
    if (raw_qkv) {
      raw.sums = ws.pf.qkv_raw;
      raw.ex = extras;
      raw.rope = (const float2 *)ctx->rope;
      raw.k_out = ws.pf.k;
      raw.v_out = ws.pf.v;
      if (append_slots_host) raw.append = ws.pf.table + (size_t)batch * stride;
      raw.k_slots = ctx->k_store + (size_t)l * ctx->layer_stride;
      raw.v_slots = ctx->v_store + (size_t)l * ctx->layer_stride;
      PC_TRY(pc::launch_qkv_raw(ctx, h_cur, (const __bf16 *)w.wqkv, (int)M, extras, ws.pf.qkv_raw, s));
    } else {
      bool v_blocked = decode;  // (in a decoding step nobody reads V as blocks)
      PC_TRY(pc::launch_qkv_rope(ctx, few_qkv ? h_cur : ws.normed, (const __bf16 *)w.wqkv, batch, t_fresh, ws.pf.table, stride, ws.pf.q, ws.pf.k,
                                 ws.pf.v, s, extras, decode ? nullptr : ws.pf.v_blk, decode ? nullptr : &v_blocked, ws.pf.qkv_raw));
      if (!v_blocked) PC_TRY(pc::launch_v_repack(ctx, ws.pf.v, ws.pf.v_blk, batch, t_fresh, s));
    }
    PC_TRY(pc::launch_attention(ctx, l, ws.pf.q, ws.pf.k, ws.pf.v, ws.pf.v_blk, raw_qkv ? &raw : nullptr, batch, t_fresh, ws.pf.table, stride,
                                min_tiles, 0, ws.attn, ws.pf.part_o, ws.pf.part_ml, s, formats, decode && left_splits > 0 ? &left_splits : nullptr));
    if (n_save > 0) {
      PC_TRY(pc::launch_kv_slices(ctx, l, save_slots_host, save_bounds_host, n_save, batch, ws.pf.k, ws.pf.v, t_fresh, s));
      for (int i = 0; i < batch * n_save; ++i)
        if (save_slots_host[i] >= 0)
          ctx->slot_len[(size_t)l * c.n_slots + save_slots_host[i]] = save_bounds_host[i % n_save + 1] - save_bounds_host[i % n_save];
    }
    if (append_kernel) {
      // after the attention launch in stream order: the keys it gathered from these slots are the older ones
      PC_TRY(pc::launch_kv_append(ctx, l, append_slots_host, batch, raw_qkv, ws.pf.k, ws.pf.v, t_fresh, s));
    }
    for (int b = 0; b < batch && append_slots_host; ++b)
      if (append_slots_host[b] >= 0) ctx->slot_len[(size_t)l * c.n_slots + append_slots_host[b]] += t_fresh;
    if (few) {
      if (decode && left_splits > 1) PC_TRY(launch_oproj_merge(ctx, (const float *)ws.pf.part_o, ws.pf.part_ml, left_splits, t_fresh, (const __bf16 *)w.wo, h_cur, ws.mid, (int)M, s));
      else PC_TRY(launch_residual_few(ctx, ws.attn, (const __bf16 *)w.wo, h_cur, ws.mid, (int)M, H, A, s));
    } else {
      PC_TRY(launch_linear_residual(ctx, ws.attn, (const __bf16 *)w.wo, h_cur, ws.mid, (int)M, H, A, s));
    }
    if (few && pc::few::pays(ctx->n_cu, M, 2 * ffn / 16, 2, 16)) {
      PC_TRY(launch_swiglu_few(ctx, ws.mid, (const __bf16 *)w.gain2, eps, (const __bf16 *)w.w_gate, (const __bf16 *)w.w_up, ws.act, (int)M, ffn, H, s));
    } else {
      PC_TRY(launch_rmsnorm(ctx, ws.mid, (const __bf16 *)w.gain2, ws.normed, (int)M, H, eps, s));
      PC_TRY(launch_linear_swiglu(ctx, ws.normed, (const __bf16 *)w.w_gate, (const __bf16 *)w.w_up, ws.act, (int)M, ffn, H, s));
    }
    if (few) PC_TRY(launch_residual_few(ctx, ws.act, (const __bf16 *)w.w_down, ws.mid, h_out, (int)M, H, ffn, s));
    else PC_TRY(launch_linear_residual(ctx, ws.act, (const __bf16 *)w.w_down, ws.mid, h_out, (int)M, H, ffn, s));
#undef PC_TRY
    h_cur = h_out;
  }
  return PC_OK;
}

pc_status percache_stack_reuse(percache_ctx *ctx, const percache_block_weights *layers_host, int32_t n_layers, int32_t ffn,
                               float eps, const void *h_in_dev, int32_t batch, int32_t t_fresh,
                               const int32_t *slot_ids_host, const int32_t *used_len_host, const int32_t *n_chunks_host,
                               int32_t max_chunks, const int32_t *save_bounds_host, const int32_t *save_slots_host,
                               int32_t n_save, void *h_out_dev, void *workspace_dev, size_t workspace_bytes, void *stream) {
  return run_stack(ctx, layers_host, n_layers, ffn, eps, h_in_dev, batch, t_fresh, slot_ids_host, used_len_host, n_chunks_host,
                   max_chunks, save_bounds_host, save_slots_host, n_save, nullptr, h_out_dev, workspace_dev, workspace_bytes, stream);
}

pc_status percache_stack_reuse_table(percache_ctx *ctx, const percache_block_weights *layers_host, int32_t n_layers,
                                     int32_t ffn, float eps, const void *h_in_dev, int32_t batch, int32_t t_fresh,
                                     const void *table_dev, void *h_out_dev, void *workspace_dev, size_t workspace_bytes,
                                     void *stream) {
  if (!ctx) return PC_EINVAL;
  const pc_table_shadow *sh = pc::find_table(ctx, table_dev, batch);
  if (!sh) return PC_EINVAL;
  return run_stack(ctx, layers_host, n_layers, ffn, eps, h_in_dev, batch, t_fresh, sh->ids.data(), sh->used.data(),
                   sh->n_chunks.data(), sh->max_chunks, nullptr, nullptr, 0, nullptr, h_out_dev, workspace_dev, workspace_bytes,
                   stream, (const int32_t *)table_dev, sh);
}

pc_status percache_stack_decode(percache_ctx *ctx, const percache_block_weights *layers_host, int32_t n_layers, int32_t ffn,
                                float eps, const void *h_in_dev, int32_t batch, int32_t n_new,
                                const int32_t *slot_ids_host, const int32_t *used_len_host, const int32_t *n_chunks_host,
                                int32_t max_chunks, const int32_t *append_slots_host, void *h_out_dev, void *workspace_dev,
                                size_t workspace_bytes, void *stream) {
  if (!ctx) return PC_EINVAL;
  if (!append_slots_host) return pc::fail(ctx, PC_EINVAL, "append_slots_host is NULL");
  return run_stack(ctx, layers_host, n_layers, ffn, eps, h_in_dev, batch, n_new, slot_ids_host, used_len_host, n_chunks_host,
                   max_chunks, nullptr, nullptr, 0, append_slots_host, h_out_dev, workspace_dev, workspace_bytes, stream);
}

}  // extern "C"
