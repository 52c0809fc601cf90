// Attention of very few query rows per kv head (decoding steps: G heads x a token or a handful) over [cached chunk K/V
// gathered by slot id ; fresh K/V].  Same arithmetic and layouts as reuse_attention.hip, another split of the work.
//
// What bounds it: the K/V stream when many queries decode at once, else the latency of one pass -- with one query a kv
// head has a few dozen 64-key tiles in all, and a workgroup that walks several of them one after the other, three of its
// four wavefronts only loading because 32-row tiles are the unit of work, spends its time waiting.  Here:
//   - the key range is cut finely: a workgroup gets about two tiles when the call is small, and all of them are requested
//     at once (a ring of four stages, direct global->LDS loads by all four wavefronts); a long call counts on two workgroups per
//     CU where two rings fit its LDS;
//   - the wavefronts share the tile by KEYS: wavefront w takes keys 16 w .. 16 w + 15 for all rows (scores by the
//     16x16x32 product with the keys on the M side, values by the 16x16x16 one, whose B operand is exactly the layout the
//     scores come out in), each with its own running maximum, sum and output; they merge once, through LDS;
//   - the few fresh keys need no V blocks: their probabilities are applied to the V rows as they were projected, in the
//     merge.
// One query, 8 kv heads, 38 tiles (bf16, D = 128): 8.6 us with q, k and v finished here, 7.1 from finished ones (the general
// kernel 13.6, behind a V repack of 2.4 and in front of an append launch of 2.8 per query); 8 queries x 8 kv heads x 256 tiles:
// 87 us of bf16 slots (6.2 TB/s of keys and values), 53 of 8-bit ones (5.1; the general kernel 62), 70 of mixed ones (73).
#include "decode_common.hpp"

namespace {
using pc::bf16x4;
using pc::bf16x8;
using pc::f32x4;
using pc::kKvTile;
using pc::kTblHeader;
using pc::dec::codes4;
using pc::dec::codes8;
using pc::dec::fast_exp2;
using pc::dec::RawRow;
using pc::dec::row_max;
using pc::dec::row_sum;

constexpr int TK = kKvTile, NW = 4;
constexpr float kSumLimit = 4.f * 256.f;  // 4 probabilities of a lane and tile, each at most 2^8 against the reference

#define PC_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xf) | (7 << 4) | (15 << 8) | ((((n) >> 4) & 3) << 14))

// FMT: 0 every cached chunk of the call sits in a bf16 slot, 1 in an 8-bit slot, 2 some of each.  NR: blocks of 16 rows.
// TWO: the form of long calls in which two workgroups share a CU (see launch_decode_attention).
template <int D, int FMT, int NR, bool TWO>
struct Lds {
  static constexpr int NSTG = TWO && FMT == 2 ? 2 : 4;                   // stages of the ring
  static constexpr int K16 = TK * D * 2, V16 = K16, K8 = TK * D, V8 = K8;
  static constexpr int STAGE = FMT == 1 ? K8 + V8 : K16 + V16;
  static constexpr int O_ROW = D + 4;                                    // floats per output row of a wavefront (padded)
  static constexpr int MERGE = NW * NR * 16 * (O_ROW + 2) * 4 + NR * 16 * 32 * 4 + 32 * D * 2;  // outputs, (m, l), fresh probabilities, fresh V
  static constexpr int BYTES = NSTG * STAGE > MERGE ? NSTG * STAGE : MERGE;
};

// RAW: q and the fresh k, v come as the projection's fp32 sums (raw.sums) and are finished here -- by every workgroup for
// its query rows, under the latency of its first K/V tiles, and by the one with the fresh keys for k and v, which it also
// writes: dense (k_out, v_out) and, where the query has a bf16 slot to append to, behind the tokens that slot holds.  The
// keys of that slot read by this launch, for this query or another, are the older ones: lengths come from the chunk list, K rows
// past the end are not read and V positions past it are cleared after the read (compute), which may see the new ones.
template <int D, int FMT, int NR, bool RAW, bool TWO>
__global__ __launch_bounds__(256, (FMT == 1 && (NR == 1 || !RAW)) || TWO ? 2 : 1) void decode_attention_kernel(
    const __bf16 *__restrict__ Q, const __bf16 *__restrict__ Kf, const __bf16 *__restrict__ Vf, pc::RawQkv raw, const __bf16 *k16,
    const __bf16 *v16, const uint8_t *__restrict__ k8, const uint8_t *__restrict__ v8, const float *__restrict__ k_scale,
    const float *__restrict__ v_scale, int n_slots16, const int32_t *__restrict__ table, int tbl_stride, int T, int Hq, int Hkv, int C,
    int n_splits, float scale_log2e, __bf16 *__restrict__ out, float *__restrict__ part_o, float *__restrict__ part_ml) {
  using L = Lds<D, FMT, NR, TWO>;
  constexpr int KS = D / 32, DB = D / 16, NSTG = L::NSTG;
  __shared__ __align__(16) char lds[L::BYTES];
  const int split = blockIdx.x % n_splits, bg = blockIdx.x / n_splits, gkv = bg % Hkv, b = bg / Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4;
  const int G = Hq / Hkv, R = G * T;

  // chunk list: lane c keeps (slot, used length) of chunk c for the first 64 chunks, later ones are read when met
  const int32_t *trow = table + (size_t)b * tbl_stride;
  int my_slot = 0, my_used = 0;
  if (lane < (tbl_stride - kTblHeader) / 2) {
    const int2 e = *(const int2 *)(trow + kTblHeader + 2 * lane);
    my_slot = e.x;
    my_used = e.y;
  }
  const int n_chunks = trow[0], n_tiles = trow[2];
  // the fresh keys (and what comes with them) count as two tiles of the last partition
  const int tile_begin = min((int)((long)split * (n_tiles + 2) / n_splits), n_tiles), tile_end = min((int)((long)(split + 1) * (n_tiles + 2) / n_splits), n_tiles);
  const int n = tile_end - tile_begin;
  const bool with_fresh = split == n_splits - 1;   // this workgroup also takes the fresh keys

  // this lane's query rows (columns of the products) and their Q operands: elements 32 ks + 8 g .. +7; the fresh keys
  // 16 wave .. +15 likewise.  RAW: everything these take is asked for here, before the tiles, and finished behind them.
  const int F = (Hq + 2 * Hkv) * D;   // (RAW) width of a row of sums: q heads, k heads, v heads
  const bool fresh_mine = with_fresh && wave * 16 < T;
  int my_i[NR];
  bf16x8 q[NR][KS], kf[KS];
  RawRow<D> rq[TWO ? 1 : NR], rk;   // (TWO: one row block at a time, the others behind the first tiles: half the registers)
  f32x4 rv[2];       // (RAW) sums and bias of 8 elements of a fresh V row: the first of this thread's units (row, 8 elements)
  bf16x8 rv_bias;
  int app_slot = -1, app_have = 0;
  constexpr int VPR = D / 8;
  const float *const row0 = raw.sums + (size_t)b * T * F;
  const int v_at = (Hq + Hkv + gkv) * D;
  auto load_q = [&](RawRow<D> &x, int r) __attribute__((always_inline)) {
    const int head = gkv * G + min(r * 16 + l16, R - 1) / T;
    x.load(row0 + (size_t)my_i[r] * F + head * D, raw.ex.bias ? raw.ex.bias + head * D : nullptr, raw.ex.q_norm, raw.rope, trow[1] + my_i[r], g);
  };
  auto load_k = [&](RawRow<D> &x) __attribute__((always_inline)) {
    const int t = min(wave * 16 + l16, T - 1), head = Hq + gkv;
    x.load(row0 + (size_t)t * F + head * D, raw.ex.bias ? raw.ex.bias + head * D : nullptr, raw.ex.k_norm, raw.rope, trow[1] + t, g);
  };
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int row = min(r * 16 + l16, R - 1), hg = row / T, head = gkv * G + hg;
    my_i[r] = row - hg * T;
    if constexpr (RAW) {
      if (!TWO || r == 0) load_q(rq[TWO ? 0 : r], r);
    } else {
      const __bf16 *p = Q + (((size_t)b * Hq + head) * T + my_i[r]) * D + g * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) q[r][ks] = *(const bf16x8 *)(p + ks * 32);
    }
  }
  if (with_fresh) {
    if constexpr (RAW) {
      if (!TWO) load_k(rk);
      const int u = min(tid, T * VPR - 1);
      const float *p = row0 + (size_t)(u / VPR) * F + v_at + u % VPR * 8;
      if (!TWO) rv[0] = *(const f32x4 *)p;
      if (!TWO) rv[1] = *(const f32x4 *)(p + 4);
      if (!TWO && raw.ex.bias) rv_bias = *(const bf16x8 *)(raw.ex.bias + v_at + u % VPR * 8);
      if (raw.append) {
        app_slot = raw.append[2 * b];
        app_have = raw.append[2 * b + 1];
      }
    } else if (fresh_mine) {
      const int t = min(wave * 16 + l16, T - 1);
      const __bf16 *p = Kf + (((size_t)b * Hkv + gkv) * T + t) * D + g * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[ks] = *(const bf16x8 *)(p + ks * 32);
    }
  }
  if (lane >= n_chunks) my_used = 0;
  const unsigned long long live = __ballot(my_used > 0);

  f32x4 o[DB][NR];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < NR; ++r) o[db][r] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref[NR], l_run[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) { m_ref[r] = -INFINITY; l_run[r] = 0.f; }

  // ---- walk over the cached tiles of the range
  struct Cursor { int chunk, off, slot, used; };
  auto enter_chunk = [&](Cursor &c) __attribute__((always_inline)) {
    if (c.chunk < 64) {  // skip unused chunks
      const unsigned long long rest = live >> c.chunk;
      c.chunk = rest ? c.chunk + __builtin_ctzll(rest) : min(n_chunks, 64);
    }
    while (c.chunk >= 64 && c.chunk < n_chunks && trow[kTblHeader + 2 * c.chunk + 1] == 0) ++c.chunk;
    if (c.chunk < min(n_chunks, 64)) {
      const int ch = __builtin_amdgcn_readfirstlane(c.chunk);
      c.slot = __builtin_amdgcn_readlane(my_slot, ch);
      c.used = __builtin_amdgcn_readlane(my_used, ch);
    } else if (c.chunk < n_chunks) {
      c.slot = trow[kTblHeader + 2 * c.chunk];
      c.used = trow[kTblHeader + 2 * c.chunk + 1];
    }
  };
  auto advance = [&](Cursor &c) __attribute__((always_inline)) {
    ++c.off;
    if (c.off * TK >= c.used) {
      c.off = 0;
      ++c.chunk;
      enter_chunk(c);
    }
  };
  Cursor cur = {0, 0, 0, 0};
  {
    const int my_tiles = (my_used + TK - 1) / TK;
    int incl = my_tiles;
#pragma unroll
    for (int sh = 1; sh < 64; sh <<= 1) {
      const int up = __shfl_up(incl, sh, 64);
      if (lane >= sh) incl += up;
    }
    cur.chunk = __popcll(__ballot(incl <= tile_begin && lane < n_chunks));
    int rem;
    if (cur.chunk < min(n_chunks, 64)) {
      rem = tile_begin - __builtin_amdgcn_readlane(incl - my_tiles, __builtin_amdgcn_readfirstlane(cur.chunk));
    } else {
      rem = tile_begin - __builtin_amdgcn_readlane(incl, 63);
      while (cur.chunk < n_chunks) {
        const int ntc = (trow[kTblHeader + 2 * cur.chunk + 1] + TK - 1) / TK;
        if (rem < ntc) break;
        rem -= ntc;
        ++cur.chunk;
      }
    }
    cur.off = rem;
    enter_chunk(cur);
  }
  Cursor cmp = cur;   // the tile being computed
  auto is8 = [&](const Cursor &c) __attribute__((always_inline)) { return FMT == 1 || (FMT == 2 && c.slot >= n_slots16); };

  // ---- requests: instruction i of a tile half fills its bytes [1024 i, +1024); 16-byte chunks XOR-swizzled inside rows of
  // 256 bytes by row & 15, of 128 bytes by (row >> 1) & 7, of 64 bytes by (row >> 2) & 3
  auto swz = [](int row_bytes, int row) __attribute__((always_inline)) { return row_bytes == 256 ? (row & 15) : row_bytes == 128 ? ((row >> 1) & 7) : ((row >> 2) & 3); };
  constexpr int I16 = L::K16 / 1024 / NW, I8 = L::K8 / 1024 / NW;   // instructions per wavefront, K or V half
  static_assert(I8 >= 1, "a tile half has an instruction for every wavefront");
  auto half = [&](const char *src, char *dst, auto row_bytes_c, int instr, int last_row) __attribute__((always_inline)) {
    constexpr int RB = decltype(row_bytes_c)::value;
#pragma unroll
    for (int k = 0; k < I16; ++k) {
      if (k >= instr) break;
      const int byte = (wave + k * NW) * 1024 + lane * 16, row = byte / RB, pc = (byte % RB) / 16;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (unsigned)(min(row, last_row) * RB + (pc ^ swz(RB, row)) * 16)),
                                       (__attribute__((address_space(3))) void *)(dst + (wave + k * NW) * 1024), 16, 0, 2);
    }
  };
  auto request = [&](int st) __attribute__((always_inline)) {   // the cursor's tile into stage st; steps the cursor
    char *dst = lds + st * L::STAGE;
    const int last = min(TK, cur.used - cur.off * TK) - 1;       // rows past a ragged end repeat the last valid row (masked later)
    if (FMT != 0 && is8(cur)) {
      const size_t base = (((size_t)(cur.slot - n_slots16) * Hkv + gkv) * C + (size_t)cur.off * TK) * D;
      half((const char *)k8 + base, dst, std::integral_constant<int, D>{}, I8, last);
      half((const char *)v8 + base, dst + L::K8, std::integral_constant<int, TK>{}, I8, D - 1);
    } else if (FMT != 1) {
      const size_t base = (((size_t)cur.slot * Hkv + gkv) * C + (size_t)cur.off * TK) * D;
      half((const char *)(k16 + base), dst, std::integral_constant<int, D * 2>{}, I16, last);
      half((const char *)(v16 + base), dst + L::K16, std::integral_constant<int, TK * 2>{}, I16, D - 1);
    }
    advance(cur);
  };

  // ---- softmax of 16 keys x 16 rows (scores in s, keys 4 g + 0..3 of the block per lane) against the lazily refreshed
  // reference exponent; returns the probabilities
  auto soften = [&](f32x4 &s, int r) __attribute__((always_inline)) {
    f32x4 p;
    auto exponentials = [&](float neg_m) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = fast_exp2(__builtin_fmaf(s[e], scale_log2e, neg_m));
      return (p[0] + p[1]) + (p[2] + p[3]);
    };
    float sum = 0.f;
    bool refresh = __builtin_amdgcn_ballot_w64(m_ref[r] == -INFINITY) != 0;   // a row that has seen no key yet
    if (!refresh) {
      sum = exponentials(-m_ref[r]);
      refresh = __builtin_amdgcn_ballot_w64(!(sum <= kSumLimit)) != 0;        // also catches inf / nan
    }
    if (refresh) {
      const float mc = row_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))) * scale_log2e;
      const bool upd = mc > m_ref[r];   // (false for a row whose keys are all masked: mc = -inf)
      const float alpha = upd ? fast_exp2(m_ref[r] - mc) : 1.0f;
      m_ref[r] = upd ? mc : m_ref[r];
      l_run[r] *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db][r] *= alpha;
      sum = exponentials(m_ref[r] == -INFINITY ? 0.f : -m_ref[r]);
    }
    l_run[r] += sum;
    return p;
  };

  // ---- one tile: this wavefront's 16 keys
  const int k_row = wave * 16 + l16;
  auto compute = [&](int st, int valid, bool b8, float ks8, float vs8) __attribute__((always_inline)) {
    if (wave * 16 >= valid) return;
    const char *kb = lds + st * L::STAGE;
    f32x4 s[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) s[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x4 vop[DB];
    if (FMT == 1 || (FMT == 2 && b8)) {
      const char *vb = kb + L::K8;
      uint2 raw[KS];
      unsigned vraw[DB];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) raw[ks] = *(const uint2 *)(kb + k_row * D + (((2 * ks + (g >> 1)) ^ swz(D, k_row)) * 16) + (g & 1) * 8);
      // byte p = 32 J + 16 a + 8 j + 4 c + e of a V row holds key 32 J + 16 j + 8 c + 4 a + e (blocked_key8)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const int row = db * 16 + l16;
        vraw[db] = *(const unsigned *)(vb + row * TK + (((2 * (wave >> 1) + (g & 1)) ^ swz(TK, row)) * 16) + 8 * (wave & 1) + 4 * (g >> 1));
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 a = codes8(raw[ks], ks8);
#pragma unroll
        for (int r = 0; r < NR; ++r) s[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, q[r][ks], s[r], 0, 0, 0);
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) vop[db] = codes4(vraw[db], vs8);
    } else {
      const char *vb = kb + L::K16;
      bf16x8 kop[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kop[ks] = *(const bf16x8 *)(kb + k_row * (D * 2) + (((4 * ks + g) ^ swz(D * 2, k_row)) * 16));
      // position p of a group of 16 keys holds key blocked_key(p): keys 4 g .. 4 g + 3 sit at 8 (g & 1) + 4 (g >> 1)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const int row = db * 16 + l16;
        vop[db] = *(const bf16x4 *)(vb + row * (TK * 2) + (((2 * wave + (g & 1)) ^ swz(TK * 2, row)) * 16) + 8 * (g >> 1));
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int r = 0; r < NR; ++r) s[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[ks], q[r][ks], s[r], 0, 0, 0);
    }
    if (valid < TK) {
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[r][e] = wave * 16 + g * 4 + e < valid ? s[r][e] : -INFINITY;
      // the values of keys past the end too: their probabilities are 0, but what stands there need not be finite -- the V of
      // tokens beyond the used length, or of one that another workgroup of this launch is appending
      const int left = valid - wave * 16 - g * 4;
      const uint2 keep = make_uint2((left > 0 ? 0xffffu : 0u) | (left > 1 ? 0xffff0000u : 0u), (left > 2 ? 0xffffu : 0u) | (left > 3 ? 0xffff0000u : 0u));
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const uint2 w = __builtin_bit_cast(uint2, vop[db]);
        vop[db] = __builtin_bit_cast(bf16x4, make_uint2(w.x & keep.x, w.y & keep.y));
      }
    }
    typedef short s16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const f32x4 p = soften(s[r], r);
      const bf16x4 pb = {(__bf16)p[0], (__bf16)p[1], (__bf16)p[2], (__bf16)p[3]};
#pragma unroll
      for (int db = 0; db < DB; ++db)
        o[db][r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, vop[db]), __builtin_bit_cast(s16x4, pb), o[db][r], 0, 0, 0);
    }
  };

  // ---- pipeline: tile t sits in stage t % NSTG; NSTG - 1 tiles are requested ahead.  The one barrier of an iteration says
  // that tile t has landed for every wavefront and that tile t-1 has been read, so its stage takes tile t + NSTG - 1.
#pragma unroll
  for (int k = 0; k < NSTG - 1; ++k)
    if (k < n) request(k);
  if constexpr (RAW) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (TWO && r > 0) {
        asm volatile("" ::: "memory");   // (one row block in registers at a time)
        load_q(rq[0], r);
      }
      rq[TWO ? 0 : r].finish(raw.ex.bias, raw.ex.q_norm, raw.ex.eps, q[r]);
    }
    if (with_fresh) {
      if (TWO) {
        asm volatile("" ::: "memory");
        load_k(rk);
      }
      rk.finish(raw.ex.bias, raw.ex.k_norm, raw.ex.eps, kf);
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(q[r][ks]));
  auto scales = [&](const Cursor &c, float &a, float &v) __attribute__((always_inline)) {
    a = v = 1.f;
    if (FMT != 0 && is8(c)) {
      const size_t at = ((size_t)(c.slot - n_slots16) * Hkv + gkv) * (C / TK) + c.off;
      a = k_scale[at];
      v = v_scale[at];
    }
  };
  float ks_n = 1.f, vs_n = 1.f;
  if (FMT != 0 && n > 0) scales(cmp, ks_n, vs_n);
  int st = 0;
  for (int t = 0; t < n; ++t) {
    const int valid = min(TK, cmp.used - cmp.off * TK);
    const bool b8 = is8(cmp);
    const float ks8 = ks_n, vs8 = vs_n;
    advance(cmp);
    // tiles behind this one that are in flight (mixed formats: counted as the smaller kind, which waits for more)
    constexpr int IPT = 2 * (FMT == 0 ? I16 : I8);
    const int later = min(NSTG - 2, n - 1 - t);
    if (later >= 2) PC_WAIT_VMCNT(2 * IPT); else if (later == 1) PC_WAIT_VMCNT(IPT); else PC_WAIT_VMCNT(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (t + NSTG - 1 < n) request(st == 0 ? NSTG - 1 : st - 1);
    if (FMT != 0 && t + 1 < n) scales(cmp, ks_n, vs_n);
    compute(st, valid, b8, ks8, vs8);
    st = st + 1 == NSTG ? 0 : st + 1;
  }

  // ---- the fresh keys: block `wave` of 16, causal
  f32x4 pf[NR];
  if (fresh_mine) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], q[r][ks], s, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = wave * 16 + g * 4 + e <= my_i[r] ? s[e] : -INFINITY;
      pf[r] = soften(s, r);
    }
  }

  if constexpr (RAW) {  // the fresh K as it is kept
    if (fresh_mine && wave * 16 + l16 < T) {
      const int t = wave * 16 + l16;
      __bf16 *dense = raw.k_out + (((size_t)b * Hkv + gkv) * T + t) * D + g * 8;
      __bf16 *slot = app_slot >= 0 ? raw.k_slots + (((size_t)app_slot * Hkv + gkv) * C + app_have + t) * D + g * 8 : nullptr;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        *(bf16x8 *)(dense + ks * 32) = kf[ks];
        if (slot) *(bf16x8 *)(slot + ks * 32) = kf[ks];
      }
    }
  }

  // ---- merge of the four wavefronts
  __syncthreads();
  float *om = (float *)lds;                                        // [wave][row][O_ROW]
  float *ml = om + NW * NR * 16 * L::O_ROW;                        // [wave][row][2]
  float *pl = ml + NW * NR * 16 * 2;                               // [row][32]
  __bf16 *vl = (__bf16 *)(pl + NR * 16 * 32);                      // fresh V [T][D]
  if (with_fresh) {
    // the fresh V rows: to LDS for the merge; RAW also where they are kept, dense and in the 64-key blocks of the slot
    for (int u = tid; u < T * VPR; u += 64 * NW) {
      const int t = u / VPR, dv = u - t * VPR;
      bf16x8 v;
      if constexpr (RAW) {
        if (TWO || u != tid) {
          const float *p = row0 + (size_t)t * F + v_at + dv * 8;
          rv[0] = *(const f32x4 *)p;
          rv[1] = *(const f32x4 *)(p + 4);
          if (raw.ex.bias) rv_bias = *(const bf16x8 *)(raw.ex.bias + v_at + dv * 8);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)(rv[e >> 2][e & 3] + (raw.ex.bias ? (float)rv_bias[e] : 0.f));
        *(bf16x8 *)(raw.v_out + (((size_t)b * Hkv + gkv) * T + t) * D + dv * 8) = v;
        if (app_slot >= 0) {
          const int at = app_have + t, in = at & (TK - 1);
          __bf16 *dst = raw.v_slots + (((size_t)app_slot * Hkv + gkv) * C + (at - in)) * D + (in & ~15) + pc::blocked_key(in & 15);
#pragma unroll
          for (int e = 0; e < 8; ++e) dst[(dv * 8 + e) * TK] = v[e];
        }
      } else {
        v = *(const bf16x8 *)(Vf + (((size_t)b * Hkv + gkv) * T + t) * D + dv * 8);
      }
      *(bf16x8 *)(vl + t * D + dv * 8) = v;
    }
    if constexpr (RAW) {
      // a block that these tokens open gets zeros behind the last of them (its padding stays finite)
      const int end = app_have + T, tail = end & (TK - 1);
      if (app_slot >= 0 && tail && (app_have == 0 || (end - 1) / TK > (app_have - 1) / TK)) {
        __bf16 *dst = raw.v_slots + (((size_t)app_slot * Hkv + gkv) * C + (end - tail)) * D;
        for (int u = tid; u < D * TK; u += 64 * NW) {
          const int p = u & (TK - 1);
          if ((p & ~15) + pc::blocked_key(p & 15) >= tail) dst[u] = (__bf16)0.f;
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int row = r * 16 + l16;
#pragma unroll
    for (int db = 0; db < DB; ++db) *(f32x4 *)(om + (wave * NR * 16 + row) * L::O_ROW + db * 16 + g * 4) = o[db][r];
    const float l = row_sum(l_run[r]);
    if (g == 0) {
      ml[(wave * NR * 16 + row) * 2] = m_ref[r];
      ml[(wave * NR * 16 + row) * 2 + 1] = l;
    }
    if (fresh_mine) *(f32x4 *)(pl + row * 32 + wave * 16 + g * 4) = pf[r];
  }
  __syncthreads();
  for (int u = tid; u < R * VPR; u += 64 * NW) {
    const int row = u / VPR, dv = u - row * VPR;
    float mw[NW], lw[NW], m = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      mw[w] = ml[(w * NR * 16 + row) * 2];
      lw[w] = ml[(w * NR * 16 + row) * 2 + 1];
      m = fmaxf(m, mw[w]);
    }
    float a[NW], l = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      a[w] = mw[w] == -INFINITY ? 0.f : fast_exp2(mw[w] - m);
      l += lw[w] * a[w];
      const float *src = om + (w * NR * 16 + row) * L::O_ROW + dv * 8;
      const f32x4 lo = *(const f32x4 *)src, hi = *(const f32x4 *)(src + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { acc[e] += lo[e] * a[w]; acc[4 + e] += hi[e] * a[w]; }
    }
    const int hg = row / T, i = row - hg * T;
    if (with_fresh) {
      for (int t = 0; t <= i; ++t) {
        const float p = pl[row * 32 + t] * (t < 16 ? a[0] : a[1]);
        const bf16x8 v = *(const bf16x8 *)(vl + t * D + dv * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += p * (float)v[e];
      }
    }
    const float inv = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= inv;
    if (n_splits == 1) {
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (__bf16)acc[e];
      *(bf16x8 *)(out + ((size_t)b * T + i) * ((size_t)Hq * D) + (size_t)(gkv * G + hg) * D + dv * 8) = v;
    } else {
      const size_t prow = (((size_t)b * Hkv + gkv) * R + row) * n_splits + split;
      // fp32: even a call of a few tiles is cut here, and its sums are rounded to bf16 once, behind the merge
      float *po = part_o + prow * D + dv * 8;
      *(f32x4 *)po = f32x4{acc[0], acc[1], acc[2], acc[3]};
      *(f32x4 *)(po + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
      if (dv == 0) {
        part_ml[prow * 2] = m;
        part_ml[prow * 2 + 1] = l;
      }
    }
  }
}

}  // namespace

namespace pc {

// Partitions of the key axis: two tiles per workgroup while the whole call then fits one workgroup per CU (finer ones cost the
// merge more than they give: one query over 64 8-bit tiles of a 3B-shaped layer, 61 us in 33 partitions, 58 in 16), else as many
// as make whole rounds of the `slots` workgroups that the chip holds at once with four tiles or more in each -- and, where a launch
// of its own merges them (more than merge_limit), at least one workgroup per CU: four tiles each would be half of that just past the
// line (layer of a query 16 heads / 8 kv heads over 64 tiles: 17.3 us in 16 partitions, 16.4 in 32; 8 queries over 8 tiles 16.7 |
// 15.2; 8-bit slots 16.5 | 15.3 and 16.0 | 14.7).  The o_proj that merges by itself pays more per partition than that gives (a
// step of the same query over 64 tiles 32.8 | 33.8, of two over 32 tiles 33.3 | 34.0).
static int decode_splits(int n_cu, int slots, long base_wgs, int tiles, int cap, int merge_limit) {
  const int ns = (tiles + 3) / 2 < cap ? (tiles + 3) / 2 : cap;  // (the fresh keys make a partition of their own then)
  if (base_wgs * ns <= n_cu) return ns;
  const int n = choose_splits(slots, base_wgs, tiles + 2, cap), round = (int)(n_cu / base_wgs);
  return n > merge_limit && n < round ? round : n;
}

pc_status launch_decode_attention(percache_ctx *ctx, int layer, const __bf16 *q, const __bf16 *kf, const __bf16 *vf, const RawQkv *raw, int batch, int t_fresh,
                                  const int32_t *table_dev, int tbl_stride, int tiles, int &n_splits, int merge_limit, __bf16 *out, float *part_o,
                                  float *part_ml, hipStream_t stream, int formats) {
  const percache_config &c = ctx->cfg;
  const int R = c.n_q_heads / c.n_kv_heads * t_fresh;
  const int fmt = !((formats & 1) && ctx->n_slots8 > 0) ? 0 : (formats & 2) ? 2 : 1;
  const __bf16 *k16 = ctx->k_store + (size_t)layer * ctx->layer_stride, *v16 = ctx->v_store + (size_t)layer * ctx->layer_stride;
  const uint8_t *k8 = ctx->k8_store + (size_t)layer * ctx->layer_stride8, *v8 = ctx->v8_store + (size_t)layer * ctx->layer_stride8;
  const size_t sc = (size_t)layer * ctx->n_slots8 * c.n_kv_heads * (c.slot_capacity / TK);
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)c.head_dim);
  const int cap = max_splits_for(c, ctx->n_cu, batch, t_fresh);
  // Two workgroups share a CU except over bf16 slots at D = 128, whose ring alone takes 128 KB.  The resident workgroups are what
  // keeps the stream of codes busy: 8 queries x 8 kv heads x 256 tiles of 8-bit slots 87 us with one per CU, 53 with two (3 rows;
  // 24 rows 107 | 64), of mixed slots 87 | 70 (104 | 79).
  const long base = (long)batch * c.n_kv_heads;
  const int slots = c.head_dim == 128 && fmt == 0 ? ctx->n_cu : 2 * ctx->n_cu;
  if (n_splits <= 0) n_splits = decode_splits(ctx->n_cu, slots, base, tiles, cap, merge_limit);
  if (n_splits > cap) n_splits = cap;
  const dim3 grid((unsigned)(base * n_splits));
  // the form that lets a second workgroup in, where the usual one does not (rings of mixed tiles, two row blocks finished at
  // once) and there is a second one: it asks for less ahead, which a call of few tiles would wait out
  const bool two = c.head_dim == 128 && base * n_splits > ctx->n_cu && (fmt == 2 || (fmt == 1 && raw && R > 16));
  const RawQkv rq = raw ? *raw : RawQkv{};
#define PC_DEC(DD, FF, RR, WW, TT)                                                                                                      \
  hipLaunchKernelGGL((decode_attention_kernel<DD, FF, RR, WW, TT>), grid, dim3(64 * NW), 0, stream, q, kf, vf, rq, k16, v16, k8, v8, ctx->k_scale + sc, \
                     ctx->v_scale + sc, ctx->n_slots16, table_dev, tbl_stride, t_fresh, c.n_q_heads, c.n_kv_heads, c.slot_capacity, n_splits,        \
                     scale_log2e, out, part_o, part_ml)
#define PC_DEC_F(DD, RR, WW)                                                                                                             \
  do {                                                                                                                                   \
    if constexpr (DD == 128) {                                                                                                            \
      if (two && fmt == 2) { PC_DEC(DD, 2, RR, WW, true); break; }                                                                        \
      if constexpr (RR == 2 && WW) { if (two) { PC_DEC(DD, 1, RR, WW, true); break; } }                                                         \
    }                                                                                                                                    \
    if (fmt == 0) PC_DEC(DD, 0, RR, WW, false); else if (fmt == 1) PC_DEC(DD, 1, RR, WW, false); else PC_DEC(DD, 2, RR, WW, false);       \
  } while (0)
#define PC_DEC_D(DD)                                                                                \
  do {                                                                                              \
    if (raw) { if (R <= 16) PC_DEC_F(DD, 1, true); else PC_DEC_F(DD, 2, true); }                     \
    else { if (R <= 16) PC_DEC_F(DD, 1, false); else PC_DEC_F(DD, 2, false); }                       \
  } while (0)
  if (c.head_dim == 128) PC_DEC_D(128); else PC_DEC_D(64);
#undef PC_DEC_D
#undef PC_DEC_F
#undef PC_DEC
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}

}  // namespace pc
