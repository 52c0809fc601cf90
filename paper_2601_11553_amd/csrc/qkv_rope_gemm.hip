// Fresh-token Q/K/V projection with the RoPE of App. B.1 fused into the epilogue.
//
// Only the retained suffix of each query is projected (Sec. 4.2.2): Y = X W^T, X [M = B*T_f, H] bf16,
// W [(Hq+2Hkv)*D, H] bf16, fp32 accumulation on the bf16 matrix cores.  The position of fresh token i of
// query b is L_pre[b] + i: the position counter is advanced by the cached length before the sine/cosine
// table is read.  q and k are rotated on the fp32 accumulators and rounded to bf16 once.
//
// Tiling: the shared projection main loop (gemm_tile.hpp): a workgroup of 4 wavefronts computes 128 output
// features x (64 or 128) tokens, and each wavefront owns a feature block together with its rotation partner
// (m, m + D/2), so RoPE needs no cross-lane traffic.
#include "few_rows.hpp"

namespace {
using pc::f32x16;
using pc::f32x4;
using pc::gemm::BF;
using pc::gemm::pack4;

// NTB: 32-token blocks per wavefront (1 -> 64-token tile, 2 -> 128-token tile, 3 -> 192-token tile: 80 KB of LDS,
// still two workgroups per CU).
// EXTRA: the bias / head-norm variants (see QkvExtras) are compiled in.
// WIDE: 8 wavefronts on two heads (256 features) x the same token tile, one workgroup per CU (D = 128, no EXTRA).
template <int D, int NTB, bool EXTRA, bool WIDE = false>
__global__ __launch_bounds__(WIDE ? 512 : 256, WIDE ? 1 : 2) void qkv_rope_kernel(const __bf16 *__restrict__ X, const __bf16 *__restrict__ W, int M,
                                                          int H, int t_fresh, int Hq, int Hkv,
                                                          const int32_t *__restrict__ table, int tbl_stride,
                                                          const float2 *__restrict__ rope, __bf16 *__restrict__ Q,
                                                          __bf16 *__restrict__ K, __bf16 *__restrict__ V, pc::QkvExtras ex,
                                                          __bf16 *__restrict__ V_blk) {
  constexpr int BT = 64 * NTB;
  extern __shared__ __align__(16) char lds[];  // Shape<NTB>::LDS_BYTES

  static_assert(!WIDE || (D == 128 && !EXTRA), "the wide tile is built for head size 128 without the variants");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wf = wave & 1, wt = (wave >> 1) & 1, half = wave >> 2;  // (half: which of the tile's two heads; 0 unless WIDE)
  const int l32 = lane & 31, g = lane >> 5;
  int bx = blockIdx.x, by = blockIdx.y;
  if constexpr (WIDE) {
    // One tile per CU: give each XCD (workgroup ids go round-robin over the 8) a compact patch of the tile grid, so
    // that the weight and token rows its tiles share are fetched into its L2 once.  Ids of one XCD become consecutive
    // positions, and positions walk strips of `sw` feature tiles, token tile by token tile.
    const int nx = gridDim.x, ny = gridDim.y, total = nx * ny;
    const int id = blockIdx.y * nx + blockIdx.x, xcd = id & 7;
    const int pos = xcd * (total >> 3) + min(xcd, total & 7) + (id >> 3);
    const int sw = nx % 5 == 0 ? 5 : nx % 4 == 0 ? 4 : nx % 3 == 0 ? 3 : nx % 2 == 0 ? 2 : 1;
    const int strip = pos / (sw * ny), within = pos - strip * (sw * ny);
    by = within / sw;
    bx = strip * sw + (within - by * sw);
  }
  const int f0 = bx * (WIDE ? 2 * BF : BF);  // first feature of the tile
  const int m0 = by * BT;                     // first token row of the tile

  // feature blocks (of 32) this wavefront owns: the low half of a rotation pair and its partner
  const int fb_lo = (D == 128) ? 4 * half + wf : 2 * wf;
  const int fb_hi = (D == 128) ? 4 * half + wf + 2 : 2 * wf + 1;

  f32x16 acc[2][NTB];
  if constexpr (WIDE)
    pc::gemm::mainloop_wide<NTB>(lds, [&](int row) __attribute__((always_inline)) { return W + (size_t)(f0 + row) * H; }, X, H, m0, M, H, fb_lo, fb_hi, wt, acc);
  else
    pc::gemm::mainloop<NTB>(lds, [&](int row) __attribute__((always_inline)) { return W + (size_t)(f0 + row) * H; }, X, H, m0, M, H, fb_lo, fb_hi, acc);

  // ---- epilogue: RoPE at position L_pre[b] + i on fp32, one rounding to bf16, head-major stores
  const int head = WIDE ? 2 * bx + half : (D == 128) ? bx : 2 * bx + wf;
  const int m_base = (D == 128) ? wf * 32 : 0;  // index of the low element inside the head
  __bf16 *dst;
  int hh, n_heads;
  bool rotate = true;
  if (head < Hq) { dst = Q; hh = head; n_heads = Hq; }
  else if (head < Hq + Hkv) { dst = K; hh = head - Hq; n_heads = Hkv; }
  else { dst = V; hh = head - Hq - Hkv; n_heads = Hkv; rotate = false; }
  if constexpr (EXTRA) {
    // bias on the accumulators; then, for q and k heads, RMSNorm over the head dimension: a token's head is spread over
    // the two lanes (l, l+32) and, at D = 128, over the wavefront pair (wf = 0, 1), which meet through LDS
    if (ex.bias) {
      const __bf16 *bl = ex.bias + (size_t)head * D + m_base + g * 4;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float b_lo = (float)bl[q4 * 8 + e], b_hi = (float)bl[q4 * 8 + e + D / 2];
#pragma unroll
          for (int t = 0; t < NTB; ++t) { acc[0][t][q4 * 4 + e] += b_lo; acc[1][t][q4 * 4 + e] += b_hi; }
        }
    }
    const __bf16 *gain = head < Hq ? ex.q_norm : (head < Hq + Hkv ? ex.k_norm : nullptr);
    float ss[NTB];
#pragma unroll
    for (int t = 0; t < NTB; ++t) {
      ss[t] = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) ss[t] += acc[0][t][r] * acc[0][t][r] + acc[1][t][r] * acc[1][t][r];
      ss[t] += __shfl_xor(ss[t], 32, 64);
    }
    if (D == 128) {
      float *red = (float *)lds;  // [wt][NTB][32 tokens][wf]; the main loop is done with LDS (it ends in a barrier)
#pragma unroll
      for (int t = 0; t < NTB; ++t)
        if (g == 0) red[((wt * NTB + t) * 32 + l32) * 2 + wf] = ss[t];
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NTB; ++t) ss[t] = red[((wt * NTB + t) * 32 + l32) * 2] + red[((wt * NTB + t) * 32 + l32) * 2 + 1];
    }
    if (gain) {
      const __bf16 *gl = gain + m_base + g * 4;
#pragma unroll
      for (int t = 0; t < NTB; ++t) {
        const float r = 1.0f / sqrtf(ss[t] / (float)D + ex.eps);
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[0][t][q4 * 4 + e] *= r * (float)gl[q4 * 8 + e];
            acc[1][t][q4 * 4 + e] *= r * (float)gl[q4 * 8 + e + D / 2];
          }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NTB; ++t) {
    const int m_raw = m0 + (wt * NTB + t) * 32 + l32;
    const bool m_ok = m_raw < M;
    const int m = m_ok ? m_raw : M - 1;
    const int b = m / t_fresh, i = m - b * t_fresh;
    const int pos = table[(size_t)b * tbl_stride + 1] + i;
    __bf16 *row = dst + (((size_t)b * n_heads + hh) * t_fresh + i) * D;
    // all sixteen (cos, sin) pairs of this lane's token first (eight 16-byte loads in flight), then the math
    float4 cs[4][2];
    if (rotate) {
      const float4 *csp = (const float4 *)(rope + (size_t)pos * (D / 2) + m_base + g * 4);
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        cs[q4][0] = csp[q4 * 4];      // pairs mm, mm+1
        cs[q4][1] = csp[q4 * 4 + 1];  // pairs mm+2, mm+3
      }
    }
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const int mm = m_base + q4 * 8 + g * 4;  // first of 4 consecutive pair indices
      float lo[4], hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float a = acc[0][t][q4 * 4 + e], c = acc[1][t][q4 * 4 + e];
        if (rotate) {
          const float4 w4 = cs[q4][e >> 1];
          const float wc = (e & 1) ? w4.z : w4.x, ws = (e & 1) ? w4.w : w4.y;
          lo[e] = a * wc - c * ws;
          hi[e] = c * wc + a * ws;
        } else {
          lo[e] = a;
          hi[e] = c;
        }
      }
      if (m_ok) {
        *(uint2 *)(row + mm) = pack4(lo[0], lo[1], lo[2], lo[3]);
        *(uint2 *)(row + mm + D / 2) = pack4(hi[0], hi[1], hi[2], hi[3]);
        if (V_blk && !rotate) {
          // also as the 64-key blocks [D][64] the attention kernel reads for the fresh part (t_fresh is a multiple of
          // 64 here: no padding to write); the 32 lanes of a half wavefront hold 32 consecutive tokens of one feature
          const int tin = i & 63;
          __bf16 *vb = V_blk + ((((size_t)b * n_heads + hh) * (t_fresh >> 6) + (i >> 6)) * D) * 64 + (tin & ~15) + pc::blocked_key(tin & 15);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vb[(size_t)(mm + e) * 64] = (__bf16)lo[e];
            vb[(size_t)(mm + e + D / 2) * 64] = (__bf16)hi[e];
          }
        }
      }
    }
  }
}

// Few token rows: the whole projection in one launch (few_rows.hpp), the RMSNorm of the input rows folded in (NORM).
// A tile holds 8 NF (8 at NF = 1) rotation pairs of one head: tile rows r and r + PAIRS are features m and m + D/2.  At
// NF >= 2 a lane finds both in accumulator blocks f and f + NF/2, at NF = 1 the high half sits in lane + 32.
// (No head norm: a tile that holds a whole head would leave 32 workgroups at 32 heads -- such a projection goes through its
// sums, see finish_rope_kernel.)
template <int D, int NF, int NT, bool NORM>
__global__ __launch_bounds__((64 * pc::few::Form<NF, NT>::WV)) void qkv_rope_few_kernel(
    const __bf16 *__restrict__ X, const __bf16 *__restrict__ W, int M, int H, int t_fresh, int Hq, int Hkv, const int32_t *__restrict__ table,
    int tbl_stride, const float2 *__restrict__ rope, __bf16 *__restrict__ Q, __bf16 *__restrict__ K, __bf16 *__restrict__ V, pc::QkvExtras ex,
    __bf16 *__restrict__ V_blk, int n_wt, int n_tt) {
  constexpr int WV = pc::few::Form<NF, NT>::WV, NSTG = pc::few::Form<NF, NT>::NSTG;
  constexpr int PAIRS = NF == 1 ? 8 : 8 * NF, TPH = D / 2 / PAIRS, NFP = NF == 1 ? 1 : NF / 2, PER = (NFP * NT + WV - 1) / WV;
  __shared__ __align__(16) char lds[pc::few::Tile<NF, NT, WV, NSTG, NORM>::LDS_BYTES];
  int wt, tt;
  if (!pc::few::place(blockIdx.x, n_wt, n_tt, wt, tt)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4;
  const int head = wt / TPH, sub = wt % TPH, m0 = tt * 16 * NT;
  __bf16 *dst;
  int hh, n_heads;
  bool rotate = true;
  if (head < Hq) { dst = Q; hh = head; n_heads = Hq; }
  else if (head < Hq + Hkv) { dst = K; hh = head - Hq; n_heads = Hkv; }
  else { dst = V; hh = head - Hq - Hkv; n_heads = Hkv; rotate = false; }

  // what the epilogue needs of this wavefront's (pair block, token block) units: the cached length is asked for before the
  // first requests, the (cos, sin) rows behind them
  int q_b[PER], q_i[PER], l_pre[PER], first[PER];
  float4 cs[PER][2];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int b = min(wave + j * WV, NFP * NT - 1), m = min(m0 + b % NT * 16 + l16, M - 1);
    q_b[j] = m / t_fresh;
    q_i[j] = m - q_b[j] * t_fresh;
    first[j] = sub * PAIRS + (NF == 1 ? 4 * (g & 1) : b / NT * 16 + 4 * g);  // first of this lane's 4 consecutive pairs
    l_pre[j] = rotate ? table[(size_t)q_b[j] * tbl_stride + 1] : 0;
  }
  f32x4 acc[NF][NT];
  float ss[NT];
  pc::few::slice_product<NF, NT, WV, NSTG, NORM>(
      lds,
      [&](int r) __attribute__((always_inline)) {
        return W + (size_t)(head * D + sub * PAIRS + (r < PAIRS ? r : D / 2 + r - PAIRS)) * H;
      },
      [&](int r) __attribute__((always_inline)) { return X + (size_t)min(m0 + r, M - 1) * H; }, ex.pre_norm, H, wave, lane,
      [&](char *, int, int) __attribute__((always_inline)) {
        if (!rotate) return;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
          const float4 *p = (const float4 *)(rope + (size_t)(l_pre[j] + q_i[j]) * (D / 2) + first[j]);
          cs[j][0] = p[0];
          cs[j][1] = p[1];
        }
      },
      acc, ss);
  pc::few::share_slices<NF, NT, WV, NSTG, NORM>(lds, wave, lane, acc, ss);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int b = wave + j * WV;
    if (b >= NFP * NT) continue;
    const int t = b % NT, mm = first[j];
    float lo[4], hi[4];
    const float r = NORM ? pc::few::row_factor<NF, NT, WV>(lds, t, l16, H, ex.eps) : 1.f;
    f32x4 sl = pc::few::tile_sum<NF, NT, WV>(lds, NF == 1 ? 0 : b / NT, t, lane), sh;
    if constexpr (NF == 1) {
#pragma unroll
      for (int e = 0; e < 4; ++e) sh[e] = __shfl_xor(sl[e], 32, 64);
    } else {
      sh = pc::few::tile_sum<NF, NT, WV>(lds, b / NT + NFP, t, lane);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[e] = sl[e] * r;
      hi[e] = sh[e] * r;
    }
    if (ex.bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo[e] += (float)ex.bias[(size_t)head * D + mm + e];
        hi[e] += (float)ex.bias[(size_t)head * D + mm + e + D / 2];
      }
    }
    if (rotate) {
      const float wc[4] = {cs[j][0].x, cs[j][0].z, cs[j][1].x, cs[j][1].z}, ws[4] = {cs[j][0].y, cs[j][0].w, cs[j][1].y, cs[j][1].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = lo[e], c = hi[e];
        lo[e] = a * wc[e] - c * ws[e];
        hi[e] = c * wc[e] + a * ws[e];
      }
    }
    if (m0 + t * 16 + l16 >= M || (NF == 1 && g >= 2)) continue;
    const int i = q_i[j];
    __bf16 *row = dst + (((size_t)q_b[j] * n_heads + hh) * t_fresh + i) * D;
    *(uint2 *)(row + mm) = pack4(lo[0], lo[1], lo[2], lo[3]);
    *(uint2 *)(row + mm + D / 2) = pack4(hi[0], hi[1], hi[2], hi[3]);
    if (V_blk && !rotate) {  // also as the 64-key blocks [D][64] the attention kernel reads for the fresh part
      const int tin = i & 63;
      __bf16 *vb = V_blk + ((((size_t)q_b[j] * n_heads + hh) * ((t_fresh + 63) >> 6) + (i >> 6)) * D) * 64 + (tin & ~15) + pc::blocked_key(tin & 15);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vb[(size_t)(mm + e) * 64] = (__bf16)lo[e];
        vb[(size_t)(mm + e + D / 2) * 64] = (__bf16)hi[e];
      }
    }
  }
  if (V_blk && !rotate && t_fresh & 63) {
    // zeros behind the last token of every query that ends in this tile (masked probabilities multiply them), 8 keys at a
    // time: chunk c of a row holds keys 16 (c/2) + 4 (c%2) + {0-3, 8-11}
    const int m_end = min(m0 + 16 * NT, M), tail = t_fresh & 63, blocks = (t_fresh + 63) >> 6;
    for (int b = m0 / t_fresh; (b + 1) * t_fresh <= m_end; ++b) {
      if ((b + 1) * t_fresh <= m0) continue;
      __bf16 *vb = V_blk + (((size_t)b * n_heads + hh) * blocks + blocks - 1) * D * 64;
      for (int u = tid; u < 2 * PAIRS * 8; u += 64 * WV) {
        const int r = u >> 3, c = u & 7, feat = sub * PAIRS + (r < PAIRS ? r : D / 2 + r - PAIRS), k0 = 16 * (c >> 1) + 4 * (c & 1);
        if (k0 + 11 < tail) continue;
        __bf16 *at = vb + (size_t)feat * 64 + c * 8;
        if (k0 >= tail) {
          *(uint4 *)at = make_uint4(0, 0, 0, 0);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (k0 + (e & 3) + 8 * (e >> 2) >= tail) at[e] = (__bf16)0.f;
        }
      }
    }
  }
}

// From the projection's sums [M][F] to q, k and v: bias, RMSNorm over the head (gains q_norm, k_norm), RoPE, one rounding.
// One thread per (token, head, 4 consecutive rotation pairs), the D / 8 threads of a head side by side in a wavefront.  Where V
// is also laid out in 64-key blocks, a query's tokens are counted up to whole blocks (rows) and the surplus ones write zeros.
// Against a projection tile that holds a whole head (32 workgroups x 256 KB of weights at 32 heads of 1024): 11.8 us at 100
// rows, where the sums take 9.4 and this kernel 4.3; with more rows the whole-head tiles, 16 rows wide, run in rounds (272 of them at
// 264 rows of 16 heads).
template <int D>
__global__ __launch_bounds__(256) void finish_rope_kernel(const float *__restrict__ sums, int batch, int t_fresh, int rows, int Hq, int Hkv,
                                                          const int32_t *__restrict__ table, int tbl_stride, const float2 *__restrict__ rope,
                                                          __bf16 *__restrict__ Q, __bf16 *__restrict__ K, __bf16 *__restrict__ V, pc::QkvExtras ex,
                                                          __bf16 *__restrict__ V_blk) {
  constexpr int QUADS = D / 8;
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int n_all = Hq + 2 * Hkv;
  if (gid >= (long)batch * rows * n_all * QUADS) return;
  const int mm = (int)(gid % QUADS) * 4, head = (int)(gid / QUADS % n_all), row_id = (int)(gid / QUADS / n_all);
  const int b = row_id / rows, i = row_id - b * rows;
  const bool real = i < t_fresh;
  if (!real && head < Hq + Hkv) return;
  const float *src = sums + ((size_t)(b * t_fresh + min(i, t_fresh - 1)) * n_all + head) * D + mm;
  f32x4 lo = *(const f32x4 *)src, hi = *(const f32x4 *)(src + D / 2);
  __bf16 *dst;
  int hh, n_heads;
  bool rotate = true;
  if (head < Hq) { dst = Q; hh = head; n_heads = Hq; }
  else if (head < Hq + Hkv) { dst = K; hh = head - Hq; n_heads = Hkv; }
  else { dst = V; hh = head - Hq - Hkv; n_heads = Hkv; rotate = false; }
  if (ex.bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[e] += (float)ex.bias[(size_t)head * D + mm + e];
      hi[e] += (float)ex.bias[(size_t)head * D + mm + e + D / 2];
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) ss += lo[e] * lo[e] + hi[e] * hi[e];
#pragma unroll
  for (int o = 1; o < QUADS; o <<= 1) ss += __shfl_xor(ss, o, 64);
  const __bf16 *gain = head < Hq ? ex.q_norm : (head < Hq + Hkv ? ex.k_norm : nullptr);
  if (gain) {
    const float r = 1.0f / sqrtf(ss / (float)D + ex.eps);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[e] *= r * (float)gain[mm + e];
      hi[e] *= r * (float)gain[mm + e + D / 2];
    }
  }
  if (rotate) {
    const f32x4 *p = (const f32x4 *)(rope + (size_t)(table[(size_t)b * tbl_stride + 1] + i) * (D / 2) + mm);
    const f32x4 c01 = p[0], c23 = p[1];  // (cos, sin) of pairs mm, mm+1 and mm+2, mm+3
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float c = e < 2 ? c01[2 * e] : c23[2 * e - 4], sn = e < 2 ? c01[2 * e + 1] : c23[2 * e - 3], x = lo[e], y = hi[e];
      lo[e] = x * c - y * sn;
      hi[e] = y * c + x * sn;
    }
  }
  if (real) {
    __bf16 *row = dst + (((size_t)b * n_heads + hh) * t_fresh + i) * D;
    *(uint2 *)(row + mm) = pack4(lo[0], lo[1], lo[2], lo[3]);
    *(uint2 *)(row + mm + D / 2) = pack4(hi[0], hi[1], hi[2], hi[3]);
  }
  if (V_blk && !rotate) {
    __bf16 *vb = V_blk + (((size_t)b * n_heads + hh) * (rows >> 6) + (i >> 6)) * D * 64 + (i & 48) + pc::blocked_key(i & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vb[(size_t)(mm + e) * 64] = (__bf16)(real ? lo[e] : 0.f);
      vb[(size_t)(mm + e + D / 2) * 64] = (__bf16)(real ? hi[e] : 0.f);
    }
  }
}

// The bare sums of few token rows, fp32 [M][N] (see RawQkv).
template <int NF, int NT, bool NORM>
__global__ __launch_bounds__((64 * pc::few::Form<NF, NT>::WV)) void qkv_raw_few_kernel(const __bf16 *__restrict__ X, const __bf16 *__restrict__ W,
                                                                                      const __bf16 *__restrict__ gain, float eps, float *__restrict__ Y,
                                                                                      int M, int N, int K, int n_wt, int n_tt) {
  constexpr int WV = pc::few::Form<NF, NT>::WV, NSTG = pc::few::Form<NF, NT>::NSTG;
  __shared__ __align__(16) char lds[pc::few::Tile<NF, NT, WV, NSTG, NORM>::LDS_BYTES];
  int wt, tt;
  if (!pc::few::place(blockIdx.x, n_wt, n_tt, wt, tt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g = lane >> 4;
  const int n0 = wt * 16 * NF, m0 = tt * 16 * NT;
  f32x4 acc[NF][NT];
  float ss[NT];
  pc::few::slice_product<NF, NT, WV, NSTG, NORM>(
      lds, [&](int r) __attribute__((always_inline)) { return W + (size_t)(n0 + r) * K; },
      [&](int r) __attribute__((always_inline)) { return X + (size_t)min(m0 + r, M - 1) * K; }, gain, K, wave, lane, [](char *, int, int) {}, acc, ss);
  pc::few::share_slices<NF, NT, WV, NSTG, NORM>(lds, wave, lane, acc, ss);
#pragma unroll
  for (int b = wave; b < NF * NT; b += WV) {
    const int f = b / NT, t = b % NT, m = m0 + t * 16 + l16;
    f32x4 s = pc::few::tile_sum<NF, NT, WV>(lds, f, t, lane);
    if (NORM) s *= pc::few::row_factor<NF, NT, WV>(lds, t, l16, K, eps);
    if (m < M) *(f32x4 *)(Y + (size_t)m * N + n0 + f * 16 + g * 4) = s;
  }
}

}  // namespace

namespace pc {

// With a head norm finish_rope_kernel comes on top, which at width 1024 the second round no longer pays for (4096 features, us:
// 11 and 6 at 256 rows, 20 and 9 at 512, against 17 and 5 for the norm in front); from width 1536 on it does (2048 features, 640
// rows: 24 and 6 against 28 and 5).
bool few_rows_qkv(const percache_ctx *ctx, long M, bool head_norm) {
  const percache_config &c = ctx->cfg;
  return few_rows(c, M) && few::pays(ctx->n_cu, M, (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim / 16, 1, head_norm && c.hidden < 1536 ? 8 : 16);
}

// (no timing events: the callers bracket the whole projection)
static pc_status launch_sums(percache_ctx *ctx, const __bf16 *x, const __bf16 *w, int M, const QkvExtras &extras, float *sums, hipStream_t stream) {
  const percache_config &c = ctx->cfg;
  const int N = (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim, K = c.hidden;
  const few::Choice ch = few::choose_tile(ctx->n_cu, M, N / 16, 1);
  const int n_wt = N / (16 * ch.nf), n_tt = (M + 16 * ch.nt - 1) / (16 * ch.nt);
#define PC_FEW_K(NF, NT, NN)                                                                                                        \
  hipLaunchKernelGGL((qkv_raw_few_kernel<NF, NT, NN>), dim3(few::grid_of(n_wt, n_tt)), dim3(64 * few::Form<NF, NT>::WV), 0, stream, x, w, \
                     extras.pre_norm, extras.eps, sums, M, N, K, n_wt, n_tt)
#define PC_FEW(NF, NT)                                                                            \
  if (ch.nf == NF && ch.nt == NT) {                                                               \
    if (extras.pre_norm) PC_FEW_K(NF, NT, true); else PC_FEW_K(NF, NT, false);                     \
  }
  PC_FEW(1, 1) else PC_FEW(2, 1) else PC_FEW(1, 2) else PC_FEW(2, 2) else PC_FEW(2, 3) else PC_FEW(2, 4) else PC_FEW(4, 3) else PC_FEW(4, 4)
#undef PC_FEW
#undef PC_FEW_K
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}
pc_status launch_qkv_raw(percache_ctx *ctx, const __bf16 *x, const __bf16 *w, int M, const QkvExtras &extras, float *sums, hipStream_t stream) {
  prof_begin(ctx, PC_KERNEL_QKV_ROPE, stream);
  const pc_status st = launch_sums(ctx, x, w, M, extras, sums, stream);
  if (st == PC_OK) prof_end(ctx, PC_KERNEL_QKV_ROPE, stream);
  return st;
}

pc_status launch_qkv_rope(percache_ctx *ctx, const __bf16 *x, const __bf16 *w, int batch, int t_fresh,
                          const int32_t *table_dev, int tbl_stride, __bf16 *q, __bf16 *k, __bf16 *v,
                          hipStream_t stream, const QkvExtras &extras, __bf16 *v_blk, bool *v_blk_done, float *raw) {
  if (v_blk_done) *v_blk_done = false;
  const percache_config &c = ctx->cfg;
  const int M = batch * t_fresh;
  const int F = (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  if (F % BF) return fail(ctx, PC_ESHAPE, "(Hq + 2 Hkv) * D = %d must be a multiple of %d", F, BF);
  if ((long)F * c.hidden >= (1L << 31) || (long)M * c.hidden >= (1L << 31))
    return fail(ctx, PC_ESHAPE, "operand larger than 2^31 elements");
  const float2 *rope = (const float2 *)ctx->rope;
  if (few_rows_qkv(ctx, M, extras.q_norm || extras.k_norm)) {
    __bf16 *vb = v_blk && v_blk_done ? v_blk : nullptr;
    if (vb) *v_blk_done = true;
    if (extras.q_norm || extras.k_norm) {  // the sums, then one small kernel over whole heads
      prof_begin(ctx, PC_KERNEL_QKV_ROPE, stream);
      const pc_status st = launch_sums(ctx, x, w, M, extras, raw, stream);
      if (st != PC_OK) return st;
      const int rows = vb ? (t_fresh + 63) / 64 * 64 : t_fresh;
      const long threads = (long)batch * rows * (c.n_q_heads + 2 * c.n_kv_heads) * (c.head_dim / 8);
#define PC_FINISH(DD)                                                                                                                   \
  hipLaunchKernelGGL(finish_rope_kernel<DD>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream, raw, batch, t_fresh, rows, c.n_q_heads, \
                     c.n_kv_heads, table_dev, tbl_stride, rope, q, k, v, extras, vb)
      if (c.head_dim == 128) PC_FINISH(128); else PC_FINISH(64);
#undef PC_FINISH
      prof_end(ctx, PC_KERNEL_QKV_ROPE, stream);
      PC_HIP(ctx, hipGetLastError());
      return PC_OK;
    }
    const few::Choice ch = few::choose_tile(ctx->n_cu, M, F / 16, 1);
    const int n_wt = F / (16 * ch.nf), n_tt = (M + 16 * ch.nt - 1) / (16 * ch.nt);
    prof_begin(ctx, PC_KERNEL_QKV_ROPE, stream);
#define PC_FEW_K(DD, NF, NT, NN)                                                                                                \
  hipLaunchKernelGGL((qkv_rope_few_kernel<DD, NF, NT, NN>), dim3(few::grid_of(n_wt, n_tt)), dim3(64 * few::Form<NF, NT>::WV), 0, stream, x, w, \
                     M, c.hidden, t_fresh, c.n_q_heads, c.n_kv_heads, table_dev, tbl_stride, rope, q, k, v, extras, vb, n_wt, n_tt)
#define PC_FEW(DD, NF, NT)                                                                          \
  if (ch.nf == NF && ch.nt == NT) {                                                                 \
    if (extras.pre_norm) PC_FEW_K(DD, NF, NT, true); else PC_FEW_K(DD, NF, NT, false);               \
  }
#define PC_FEW_D(DD) PC_FEW(DD, 1, 1) else PC_FEW(DD, 2, 1) else PC_FEW(DD, 1, 2) else PC_FEW(DD, 2, 2) else PC_FEW(DD, 2, 3) else PC_FEW(DD, 2, 4) else PC_FEW(DD, 4, 3) else PC_FEW(DD, 4, 4)
    if (c.head_dim == 128) { PC_FEW_D(128) } else { PC_FEW_D(64) }
#undef PC_FEW_D
#undef PC_FEW
#undef PC_FEW_K
    prof_end(ctx, PC_KERNEL_QKV_ROPE, stream);
    PC_HIP(ctx, hipGetLastError());
    return PC_OK;
  }
  // Token tile: two workgroups share a CU, so a launch runs in rounds of 2 * n_cu tiles and a tile's time grows with
  // its token blocks; take the width with the fewest block-rounds (the wider one on a tie: fewer operand reads per
  // MFMA).  64-token tiles while there are too few rows to fill wider ones.
  int ntb = 1;
  if (M > 64 * 3) {
    long best = -1;
    for (int cand = 3; cand >= 2; --cand) {
      const long tiles = (long)(F / BF) * ((M + 64 * cand - 1) / (64 * cand));
      const long cost = (tiles + 2L * ctx->n_cu - 1) / (2L * ctx->n_cu) * cand;
      if (best < 0 || cost < best) { best = cost; ntb = cand; }
    }
  }
  // Two heads per workgroup (8 wavefronts, one workgroup per CU) while all its tiles fit one round: the token rows are
  // brought into LDS once for twice the features.  The narrowest of 192, 256 and 320 tokens that does it; against the
  // tiles above (one head, up to 192 tokens, rounds of 2 * n_cu), us a launch:
  //   4096 features, K = 1024: 3700 rows 46 | 49, 4096 rows 48 | 51, 4224 rows 52.3 | 54.1, 5120 rows 55.5 | 65.0
  //   5120 features, K = 3072: 2560 rows 85 | 101, 3072 rows 94 | 108, 3800 rows 112 | 142
  // 320 tokens take 252 registers a lane of the 256, and 147 KB of LDS: there is no wider one.  Narrow contractions are bound by the ends of the
  // tiles, which the smaller ones hide behind each other, and so do tiles that leave a quarter of the CUs idle:
  //   256 tokens, 24 heads over 8, 2560 rows: K = 128 22.9 | 21.3, 512 32.0 | 31.0, 768 37.2 | 38.6; 32 over 8, 2048 rows (192 tiles), K = 1024 42.9 | 41.1
  //   320 tokens, 16 heads over 8, 4600 rows: K = 128 28.7 | 26.5, 384 35.2 | 34.7, 512 38.8 | 39.0, 768 46.0 | 48.0
  const int n_heads_all = c.n_q_heads + 2 * c.n_kv_heads;
  __bf16 *vb_large = (v_blk && v_blk_done && t_fresh % 64 == 0) ? v_blk : nullptr;  // the large tiles lay V out for the attention kernel too
  if (vb_large) *v_blk_done = true;
  int wide = 0;   // its 64-token blocks
  if (c.head_dim == 128 && !extras.any() && n_heads_all % 2 == 0 && M >= 1024)
    for (int cand = 3; cand <= 5; ++cand) {
      const long tiles = (long)(n_heads_all / 2) * ((M + 64 * cand - 1) / (64 * cand));
      if (tiles > ctx->n_cu) continue;
      if (cand == 3 || (tiles * 4 > ctx->n_cu * 3L && c.hidden >= (cand == 4 ? 768 : 512))) wide = cand;
      break;
    }
  if (wide) {
#define PC_WIDE(NN)                                                                                                                                  \
  do {                                                                                                                                               \
    constexpr int lds_bytes = pc::gemm::WideShape<NN>::LDS_BYTES;                                                                                     \
    PC_HIP(ctx, hipFuncSetAttribute((const void *)qkv_rope_kernel<128, NN, false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));      \
    prof_begin(ctx, PC_KERNEL_QKV_ROPE, stream);                                                                                                     \
    hipLaunchKernelGGL((qkv_rope_kernel<128, NN, false, true>), dim3(n_heads_all / 2, (M + 64 * NN - 1) / (64 * NN)), dim3(512), lds_bytes, stream, x, w, \
                       M, c.hidden, t_fresh, c.n_q_heads, c.n_kv_heads, table_dev, tbl_stride, rope, q, k, v, extras, vb_large);                       \
  } while (0)
    if (wide == 3) PC_WIDE(3); else if (wide == 4) PC_WIDE(4); else PC_WIDE(5);
#undef PC_WIDE
    prof_end(ctx, PC_KERNEL_QKV_ROPE, stream);
    PC_HIP(ctx, hipGetLastError());
    return PC_OK;
  }
  dim3 grid(F / BF, (M + 64 * ntb - 1) / (64 * ntb));
#define PC_LAUNCH_E(DD, NN, EE)                                                                                        \
  do {                                                                                                                \
    constexpr int lds_bytes = pc::gemm::Shape<NN>::LDS_BYTES;                                                         \
    if (lds_bytes > 64 * 1024) /* above the default limit: opt in */                                                  \
      PC_HIP(ctx, hipFuncSetAttribute((const void *)qkv_rope_kernel<DD, NN, EE>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes)); \
    hipLaunchKernelGGL((qkv_rope_kernel<DD, NN, EE>), grid, dim3(256), lds_bytes, stream, x, w, M, c.hidden, t_fresh,  \
                       c.n_q_heads, c.n_kv_heads, table_dev, tbl_stride, rope, q, k, v, extras, vb_large);            \
  } while (0)
#define PC_LAUNCH(DD, NN)                                                                                             \
  do {                                                                                                                \
    if (extras.any()) PC_LAUNCH_E(DD, NN, true); else PC_LAUNCH_E(DD, NN, false);                                      \
  } while (0)
  prof_begin(ctx, PC_KERNEL_QKV_ROPE, stream);
  if (c.head_dim == 128) {
    if (ntb == 3) PC_LAUNCH(128, 3); else if (ntb == 2) PC_LAUNCH(128, 2); else PC_LAUNCH(128, 1);
  } else {
    if (ntb == 3) PC_LAUNCH(64, 3); else if (ntb == 2) PC_LAUNCH(64, 2); else PC_LAUNCH(64, 1);
  }
#undef PC_LAUNCH
#undef PC_LAUNCH_E
  prof_end(ctx, PC_KERNEL_QKV_ROPE, stream);
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}

}  // namespace pc
