// A decoding step of few token rows through all layers in ONE launch (percache_stack_decode and its like).
//
// What bounds such a step is not bytes but the chain of dependent launches: five a layer of 5 to 9 us each (2 to 3 of them until the
// first load has come back, 1 until the last store is visible), where one pass over a layer's weights takes 5 us.  Here the
// workgroups stay: what one step of the chain hands to the next (2 to 16 KB) goes through memory inside the launch, and while a
// workgroup waits for it its weights or its K/V tiles are already on their way to LDS.  Handing 2 KB from 64 workgroups to 256 takes
// 1.1 to 1.3 us (a launch that does nothing: 3.1).
//
// Work is a list of items in the order of the chain -- per layer: Q sums of the QKV projection, T attention of a piece of the key axis, X
// merge of the pieces, O o_proj, G gate / up, D down projection -- and a workgroup takes the next item of the list from a counter.  An
// item waits for items in front of it only, and those have been taken by workgroups that run: whatever the number of workgroups that
// are resident at once (other streams may hold the rest of the chip), the first unfinished item never waits, so the launch ends.
//
// Hand-over: every buffer between two steps of the chain is filled with words of ones beforehand (the launch in front, which also writes
// the chunk lists), producers store whole words straight to memory (sc1: device scope), consumers ask for all their words until
// none is all ones any more.  No flag, no fence, no second round trip: a word is its own flag.  All ones is a NaN (as two bf16 or
// as fp32); a result that happens to be this NaN is stored as another one (keep()).  Every layer has buffers of its own, so nothing is
// refilled inside the launch.
#include <cstring>

#include "decode_common.hpp"
#include "few_rows.hpp"
#include "decode_stack.hpp"

namespace {
using pc::bf16x4;
using pc::bf16x8;
using pc::f32x4;
using pc::kKvTile;
using pc::kTblHeader;
using pc::u32x4;
using pc::dec::codes4;
using pc::dec::codes8;
using pc::dec::fast_exp2;
using pc::dec::row_max;
using pc::dec::row_sum;
using pc::dec::wave_sum;
using pc::gemm::pack4;
using pc::gemm::swz128;
using pc::gemm::unpack4;
using pc::gemm::wait_vmcnt;
using pc::stackdec::Args;
// the arguments as they stand in the launch's argument segment
typedef __attribute__((address_space(4))) const Args KArgs;
typedef __attribute__((address_space(4))) const pc::stackdec::LayerPtrs KLayer;
using pc::stackdec::kRing;
using pc::stackdec::kWaves;

constexpr int TK = kKvTile;
constexpr float kSumLimit = 4.f * 256.f;   // (as in decode_attention.hip)
constexpr unsigned EMPTY = 0xffffffffu;
constexpr int kSc1 = 16;                   // cache policy of a buffer access: device scope
// Tries of a wait, about a second: no wait gets there (see above).  One that does hands on what it has, words of ones, which are NaNs in the
// step's result, and takes the counter past the list, so that the launch ends all the same.
constexpr int kTries = 1 << 20;

typedef __amdgpu_buffer_rsrc_t Rsrc;
// n elements from p on; accesses past them read zeros and write nothing
template <class E>
__device__ __forceinline__ Rsrc rsrc_of(const E *p, size_t n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<E *>(p), 0, (int)(n * sizeof(E)), 0x00020000);
}
constexpr unsigned kNowhere = 0x80000000u;   // an offset past every buffer's end
__device__ __forceinline__ u32x4 ask(Rsrc r, unsigned off) { return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kSc1)); }
__device__ __forceinline__ uint2 ask2(Rsrc r, unsigned off) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kSc1));
  return make_uint2(v[0], v[1]);
}
__device__ __forceinline__ bool missing(u32x4 v) { return v[0] == EMPTY || v[1] == EMPTY || v[2] == EMPTY || v[3] == EMPTY; }
__device__ __forceinline__ bool missing(uint2 v) { return v.x == EMPTY || v.y == EMPTY; }
__device__ __forceinline__ unsigned keep(unsigned w) { return w == EMPTY ? 0x7fff7fffu : w; }
__device__ __forceinline__ void hand_over(Rsrc r, unsigned off, u32x4 v) {
  u32x4 w;
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = keep(v[i]);
  __builtin_amdgcn_raw_buffer_store_b128(w, r, off, 0, kSc1);
}
__device__ __forceinline__ void hand_over(Rsrc r, unsigned off, uint2 v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 w = {keep(v.x), keep(v.y)};
  __builtin_amdgcn_raw_buffer_store_b64(w, r, off, 0, kSc1);
}
__device__ __forceinline__ bool given_up(int tries, unsigned *ticket) {
  if (tries < kTries) return false;
  __hip_atomic_fetch_or(ticket, 0x40000000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}
// A wait costs the CU's other wavefronts what its tries take out of the memory pipe, and that serves the oldest first: eight wavefronts that ask
// for many lines at a time without a pause have kept the workgroup beside them, whose results they waited for, from storing these at all.
// So a waiting wavefront has the lower priority, asks for one load's worth until that is there, and sleeps in between (64 clocks a unit).
struct Waiting {
  __device__ __forceinline__ Waiting() { __builtin_amdgcn_s_setprio(0); }
  __device__ __forceinline__ ~Waiting() { __builtin_amdgcn_s_setprio(2); }
};
template <int N>
__device__ __forceinline__ void pause() {
  __builtin_amdgcn_s_sleep(N);
  asm volatile("" ::: "memory");
}
// Keeps a scalar where it is: without this the compiler fetches launch arguments again behind a wait, where every fetch counts.
template <class V>
__device__ __forceinline__ V pinned(V v) {
  asm volatile("" : "+s"(v));
  return v;
}
template <class E>   // (pointers: into global memory, or every access becomes a flat one, which counts as one of LDS too)
__device__ __forceinline__ E *pinned(E *p) {
  typedef __attribute__((address_space(1))) E *G;
  G q = (G)p;
  asm volatile("" : "+s"(q));
  return (E *)q;
}
// (not __syncthreads, which also waits for this wavefront's stores and the counter's answer)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// A workgroup takes its item up to a layer ahead.  Until one word of the step before the one it waits for is there (word; null: no
// gate), one lane asks for that, now and then.
__device__ __forceinline__ void gate(unsigned *ticket, const void *word, int wave) {
  if (!word) return;
  if (wave == 0) {
    Waiting w;
    const Rsrc r = rsrc_of((const unsigned *)word, 1);
    for (int tries = 0;; ++tries) {
      if ((unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, 0, 0, kSc1) != EMPTY || given_up(tries, ticket)) break;
      pause<10>();
    }
  }
  lds_barrier();
}
// (LDS stores the compiler does not see: behind an ordinary one it waits for every request before each LDS read)
__device__ __forceinline__ unsigned lds_addr(const char *p) { return (unsigned)(size_t)(__attribute__((address_space(3))) const char *)p; }
__device__ __forceinline__ void lds_put(unsigned addr, u32x4 v) { asm volatile("ds_write_b128 %0, %1" : : "v"(addr), "v"(v) : "memory"); }

// ---------------------------------------------------------------------------------------------------
// Projections: 16 NF weight rows x all token rows (at most kMaxRows) an item; as few_rows.hpp with the token rows handed over.  An RMSNorm in
// front costs nothing here: whoever makes 16 columns of a row also hands over a block of them times the gain, rounded once, and their sum
// of squares.  A block has 64 bytes of its own: a line that 32 workgroups write a word each to arrives 3 us later than one that two write to.
// ---------------------------------------------------------------------------------------------------
constexpr int kRowCols = 4096;
constexpr int kBlock = 64;   // 16 columns bf16, the sum of squares twice, padding
// w_row(r): the K elements that tile row r stands for.  x: token rows [M][K] bf16, or, normed, in blocks (kBlock below), whose sums of squares
// go to squares [M][K / 16] in LDS.  before: see gate.  waits_more, more(): what else this wavefront waits for (asks again, true: something is missing).
// On return acc holds the wavefront's slice.
template <int NF, class WRow, class More>
__device__ __forceinline__ void project(const KArgs &a, char *lds, WRow w_row, Rsrc x, bool normed, float *squares, const void *before, int K, int wave,
                                        int lane, bool waits_more, More more, f32x4 (&acc)[NF]) {
  constexpr int STAGE = 2048 * NF, NSTG = kRing / kWaves / STAGE, INSTR = 2 * NF;
  unsigned *const ticket = pinned(a.ticket);
  const int M = pinned(a.M), steps = K / 64, s0 = wave * steps / kWaves, n = (wave + 1) * steps / kWaves - s0;
  const int row_bytes = M * 128;   // LDS of a step of the token rows
  char *const ring = lds + wave * (kRing / kWaves), *const xs = lds + kRing + wave * a.x_bytes;
  const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 odd[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) odd[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  const __bf16 *src[INSTR];
#pragma unroll
  for (int i = 0; i < INSTR; ++i) {
    const int row = i * 8 + (lane >> 3);
    src[i] = w_row(row) + s0 * 64 + ((lane & 7) ^ swz128(row & 15)) * 8;
  }
  auto request = [&](int s, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < INSTR; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[i] + s * 64),
                                       (__attribute__((address_space(3))) void *)(ring + st * STAGE + i * 1024), 16, 0, 2);
  };
#pragma unroll
  for (int s = 0; s < NSTG; ++s)
    if (s < n) request(s, s);
  int rd[2], xr[2];
  const int row = min(l16, M - 1);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    rd[ks] = l16 * 128 + ((4 * ks + g) ^ swz128(l16)) * 16;
    xr[ks] = row * 128 + ((4 * ks + g) ^ swz128(row)) * 16;
  }
  if (M == 1 && K <= kRowCols) {
    // One token row: the weights go on into registers while the row is awaited, and the row needs no LDS.  Lane (l16, g) asks for its
    // elements 32 l16 + 8 g .. +7 of the slice, what lane (0, g) needs in product l16; so product i takes the row rotated by i lanes (the
    // columns of the other lanes are nobody's).  A step behind the wait took 350 to 460 clocks with weights and row out of LDS.  (Several
    // rows with the weights held as well: 5 to 10 % slower than out of LDS, the registers spill.)
    constexpr int MAXS = kRowCols / 64 / kWaves;
    bf16x8 w[NF][2 * MAXS];
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
      if (s < n) {   // (no break: these loops have to unroll)
        if (s % NSTG == 0) {
          wait_vmcnt<0>();
          asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int f = 0; f < NF; ++f) w[f][2 * s + ks] = *(const bf16x8 *)(ring + s % NSTG * STAGE + f * 2048 + rd[ks]);
        if (s % NSTG == NSTG - 1 && s + 1 < n) {
          __builtin_amdgcn_s_waitcnt(0xf | (7 << 4) | (3 << 14));   // every read of the stages is in registers (lgkmcnt 0)
          asm volatile("" ::: "memory");
#pragma unroll
          for (int j = 0; j < NSTG; ++j)
            if (s + 1 + j < n) request(s + 1 + j, j);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (here, not behind the wait)
    gate(ticket, before, wave);
    const int k = s0 * 64 + l16 * 32 + g * 8;
    const unsigned off = l16 >= 2 * n ? kNowhere : normed ? (unsigned)((k >> 4) * kBlock + ((k >> 3) & 1) * 16) : (unsigned)(k * 2);
    const unsigned off_sq = normed && lane < 4 * n ? (unsigned)((s0 * 4 + lane) * kBlock + 32) : kNowhere;
    u32x4 v;
    unsigned sq;
    {
      Waiting wt;
      for (int tries = 0;; ++tries) {
        v = ask(x, off);
        sq = normed ? (unsigned)__builtin_amdgcn_raw_buffer_load_b32(x, off_sq, 0, kSc1) : 0u;
        bool bad = waits_more && more();
        bad = bad || missing(v) || sq == EMPTY;
        if (__ballot(bad) == 0 || given_up(tries, ticket)) break;
        pause<1>();
      }
    }
    auto product = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      if (i >= 2 * n) return;
      u32x4 r = v;
      if constexpr (i > 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v[e], 0x120 + 16 - i, 0xf, 0xf, true);
      }
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        f32x4 &to = i & 1 ? odd[f] : acc[f];
        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[f][i], __builtin_bit_cast(bf16x8, r), to, 0, 0, 0);
      }
    };
#define PC_P(i) product(std::integral_constant<int, i>{});
    PC_P(0) PC_P(1) PC_P(2) PC_P(3) PC_P(4) PC_P(5) PC_P(6) PC_P(7) PC_P(8) PC_P(9) PC_P(10) PC_P(11) PC_P(12) PC_P(13) PC_P(14) PC_P(15)
#undef PC_P
    static_assert(2 * MAXS == 16, "products");
    if (normed) {
      const float s = wave_sum(off_sq == kNowhere ? 0.f : __uint_as_float(sq));
      if (lane == 0) squares[wave] = s;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] += odd[f];
    return;
  }
  gate(ticket, before, wave);
  bool first = true;
  int st = 0;
  const int per = normed ? 12 : 8, pieces = M * n * per;   // of 16 bytes; a step
  constexpr int U = 4;
  for (int u0 = 0; u0 < pieces || first; u0 += 64 * U) {   // (a wavefront without a slice still waits for more())
    const bool need_more = first && waits_more;
    unsigned off[U], at[U];
    bool sq[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int u = u0 + 64 * k + lane, q = u / per, c = u - q * per, m = M > 1 && n > 0 ? q / n : 0, step = q - m * n, s = s0 + step;
      sq[k] = c >= 8;
      const int blk = m * (K / 16) + s * 4 + (sq[k] ? c - 8 : c >> 1);
      off[k] = u >= pieces ? kNowhere : normed ? (unsigned)(blk * kBlock + (sq[k] ? 32 : (c & 1) * 16)) : (unsigned)((m * K + s * 64 + c * 8) * 2);
      at[k] = sq[k] ? lds_addr((const char *)(squares + blk)) : lds_addr(xs + step * row_bytes + m * 128 + (c ^ swz128(m)) * 16);
    }
    u32x4 v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = u32x4{EMPTY, EMPTY, EMPTY, EMPTY};
    {
      Waiting w;
      bool all = u0 + 64 >= pieces;   // one load's worth in all, or the first is there: ask for everything
      for (int tries = 0;; ++tries) {
        bool bad = false;
#pragma unroll
        for (int k = 0; k < U; ++k)
          if (u0 + 64 * k < pieces && (k == 0 || all)) v[k] = ask(x, off[k]);
        if (need_more && all) bad = more();
#pragma unroll
        for (int k = 0; k < U; ++k)
          if (u0 + 64 * k < pieces && (k == 0 || all)) bad = bad || v[k][0] == EMPTY || (!sq[k] && missing(v[k]));
        const bool there = __ballot(bad) == 0;
        if ((there && all) || given_up(tries, ticket)) break;
        if (there) all = true;
        else pause<2>();
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (off[k] == kNowhere) continue;
      if (sq[k]) asm volatile("ds_write_b32 %0, %1" : : "v"(at[k]), "v"(v[k][0]) : "memory");
      else lds_put(at[k], v[k]);
    }
    first = false;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  for (int s = 0; s < n; s += 2) {   // two steps at a time: all their operands on the way before the first product
    const bool two = s + 1 < n;
    const int last = two ? s + 1 : s, later = min(s + NSTG, n) - 1 - last;   // stages in flight behind these
    if (later >= 3) wait_vmcnt<(NSTG > 3 ? 3 : 0) * INSTR>();
    else if (later == 2) wait_vmcnt<(NSTG > 2 ? 2 : 0) * INSTR>();
    else if (later == 1) wait_vmcnt<INSTR>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const int st2 = st + 1 == NSTG ? 0 : st + 1;
    bf16x8 w[NF][4], xv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= 2 && !two) break;
      const char *wb = ring + (k < 2 ? st : st2) * STAGE, *xb = xs + (s + k / 2) * row_bytes;
      xv[k] = *(const bf16x8 *)(xb + xr[k & 1]);
#pragma unroll
      for (int f = 0; f < NF; ++f) w[f][k] = *(const bf16x8 *)(wb + f * 2048 + rd[k & 1]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= 2 && !two) break;
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        f32x4 &to = k & 1 ? odd[f] : acc[f];
        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[f][k], xv[k], to, 0, 0, 0);
      }
    }
    if (s + NSTG < n) {
      __builtin_amdgcn_s_waitcnt(0xf | (7 << 4) | (3 << 14));  // every read of the stages is in registers (lgkmcnt 0)
      asm volatile("" ::: "memory");
      request(s + NSTG, st);
      if (two && s + 1 + NSTG < n) request(s + 1 + NSTG, st2);
    }
    st = two ? (st2 + 1 == NSTG ? 0 : st2 + 1) : st2;
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] += odd[f];
}
// The next item, taken when the present one has all it waits for (but see merge): a workgroup that held a second one while it waits would keep
// that one's loads from being asked for by a workgroup that is free.  By wavefront 1, which has no results to hand over.
__device__ __forceinline__ void claim(unsigned *ticket, int wave, int lane, unsigned &next) {
  typedef __attribute__((address_space(1))) unsigned *G;
  G t = (G)ticket;
  asm volatile("" : "+v"(t));   // (an address the compiler knows to be uniform makes it wait for the answer on the spot)
  if (wave == 1 && lane == 0) next = __hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The wavefronts' slices meet in LDS, each in the place of its own ring; ends with a barrier.
template <int NF>
__device__ __forceinline__ void share(char *lds, int wave, int lane, const f32x4 (&acc)[NF]) {
  f32x4 *p = (f32x4 *)(lds + wave * (kRing / kWaves)) + lane;
#pragma unroll
  for (int f = 0; f < NF; ++f) p[f * 64] = acc[f];
  lds_barrier();
}
__device__ __forceinline__ f32x4 sum_of(const char *lds, int f, int lane) {
  f32x4 s = *((const f32x4 *)lds + f * 64 + lane);
#pragma unroll
  for (int w = 1; w < kWaves; ++w) s += *((const f32x4 *)(lds + w * (kRing / kWaves)) + f * 64 + lane);
  return s;
}
// The norm's factor of token row m (lanes g = 0..3 share the row), behind the barrier of share(): from the sums of 16 columns each, of one
// token row from those of the wavefronts.  (v_rsq_f32: 1 ulp, as a root and a division have)
__device__ __forceinline__ float norm_factor(const float *squares, int m, int M, int H, int g, float inv_h, float eps) {
  float s = 0.f;
  if (M == 1) {   // (at most kRowCols columns)
    const f32x4 a = *(const f32x4 *)squares, b = *(const f32x4 *)(squares + 4);
    s = ((a[0] + a[1]) + (a[2] + a[3])) + ((b[0] + b[1]) + (b[2] + b[3]));
  } else {
    for (int c = g; c < H / 64; c += 4) {
      const f32x4 v = *(const f32x4 *)(squares + m * (H / 16) + c * 4);
      s += (v[0] + v[1]) + (v[2] + v[3]);
    }
    s = row_sum(s);
  }
  return __builtin_amdgcn_rsqf(__builtin_fmaf(s, inv_h, eps));
}
// Four columns (lane g: n0 + 4 g) of token row m handed over as the input of the next projection: the row itself (v), and the block of
// these 16 columns for a norm in front.  Lanes in: the row's own; the lane behind them stores the sum of squares with the same instruction.
__device__ __forceinline__ void hand_over_row(uint2 v, uint2 gain, Rsrc raw, Rsrc blocks, int m, int n0, int H, int l16, int g, int M) {
  float x[4], gn[4];
  unpack4(v, x);
  const float sq = row_sum((x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]));
  unpack4(gain, gn);
  const uint2 p = pack4(x[0] * gn[0], x[1] * gn[1], x[2] * gn[2], x[3] * gn[3]);
  const unsigned blk = (unsigned)((m * (H / 16) + n0 / 16) * kBlock);
  if (l16 < M) hand_over(blocks, blk + g * 8, p);
  if (l16 < M && g == 0) hand_over(blocks, blk + 32, make_uint2(__float_as_uint(sq), __float_as_uint(sq)));
  if (l16 < M) hand_over(raw, (unsigned)((m * H + n0 + g * 4) * 2), v);
}

// ---------------------------------------------------------------------------------------------------
// T: attention of the R = G T query rows (at most 16) of one kv head over a piece of its key axis, as decode_attention_kernel; eight
// wavefronts take two 64-key tiles at a time, 16 keys each.
// ---------------------------------------------------------------------------------------------------
constexpr int kTail = 32;   // floats behind a piece's row: its maximum and sum, in a line of their own
template <int D, int FMT>
__device__ __forceinline__ void attend(const KArgs &a, char *lds, int layer, int id, int wave, int lane, unsigned &next) {
  constexpr int KS = D / 32, DB = D / 16, VPR = D / 8;
  constexpr int K16 = TK * D * 2, V16 = K16, K8 = TK * D, TILE = FMT == 1 ? 2 * K8 : K16 + V16, O_ROW = D + 4;
  static_assert(2 * TILE <= kRing, "two tiles");
  const int split = id % a.n_splits, bg = id / a.n_splits, gkv = bg % a.Hkv, b = bg / a.Hkv;
  const int tid = wave * 64 + lane, l16 = lane & 15, g = lane >> 4;
  unsigned *const ticket = pinned(a.ticket);
  const int T = pinned(a.T), Hkv = pinned(a.Hkv), Hq = pinned(a.Hq), G = Hq / Hkv, R = G * T, C = pinned(a.C), F = (Hq + 2 * Hkv) * D, n_splits = pinned(a.n_splits);
  const float scale_log2e = pinned(a.scale_log2e), eps = pinned(a.eps);
  const __bf16 *const bias = pinned(a.w[layer].qkv_bias), *const q_norm = pinned(a.w[layer].q_norm), *const k_norm = pinned(a.w[layer].k_norm);
  float *const part = pinned(a.part + layer * a.s_word);
  const size_t n_part = pinned(a.n_part);

  // chunk list: lane c keeps (slot, used length) of chunk c for the first 64 chunks
  const int32_t *trow = a.table + (size_t)b * a.tbl_stride;
  int my_slot = 0, my_used = 0;
  if (lane < (a.tbl_stride - kTblHeader) / 2) {
    const int2 e = *(const int2 *)(trow + kTblHeader + 2 * lane);
    my_slot = e.x;
    my_used = e.y;
  }
  const int n_chunks = trow[0], l_pre = trow[1], n_tiles = trow[2];
  if (lane >= n_chunks) my_used = 0;
  // the fresh keys count as two tiles of the last piece
  const int tile_begin = min((int)((long)split * (n_tiles + 2) / n_splits), n_tiles);
  const int tile_end = min((int)((long)(split + 1) * (n_tiles + 2) / n_splits), n_tiles);
  const bool with_fresh = split == n_splits - 1;
  const int my_tiles = (my_used + TK - 1) / TK;
  int incl = my_tiles;
#pragma unroll
  for (int sh = 1; sh < 64; sh <<= 1) {
    const int up = __shfl_up(incl, sh, 64);
    if (lane >= sh) incl += up;
  }
  int slot = 0, valid = 0, off = 0;   // this wavefront's tile of the round
  auto locate = [&](int tile) __attribute__((always_inline)) {
    valid = 0;
    if (tile >= tile_end) return;
    int c = __popcll(__ballot(incl <= tile && lane < n_chunks)), used;
    if (c < min(n_chunks, 64)) {
      const int cc = __builtin_amdgcn_readfirstlane(c);
      off = tile - __builtin_amdgcn_readlane(incl - my_tiles, cc);
      slot = __builtin_amdgcn_readlane(my_slot, cc);
      used = __builtin_amdgcn_readlane(my_used, cc);
    } else {   // chunks past the 64th (c == 64)
      off = tile - __builtin_amdgcn_readlane(incl, 63);
      for (;; ++c) {
        used = trow[kTblHeader + 2 * c + 1];
        const int nt = (used + TK - 1) / TK;
        if (off < nt || c + 1 >= n_chunks) break;
        off -= nt;
      }
      slot = trow[kTblHeader + 2 * c];
    }
    valid = min(TK, used - off * TK);
  };

  const int kw = wave & 3, tw = wave >> 2;   // 16-key block, tile of the round
  const __bf16 *const k16 = a.k16 + (size_t)layer * a.layer_stride, *const v16 = a.v16 + (size_t)layer * a.layer_stride;
  const uint8_t *const k8 = a.k8 + (size_t)layer * a.layer_stride8, *const v8 = a.v8 + (size_t)layer * a.layer_stride8;
  float ks8 = 1.f, vs8 = 1.f;
  auto swz = [](int row_bytes, int row) __attribute__((always_inline)) { return row_bytes == 256 ? (row & 15) : row_bytes == 128 ? ((row >> 1) & 7) : ((row >> 2) & 3); };
  auto half = [&](const char *src, char *dst, auto row_bytes_c, auto instr_c, int last_row) __attribute__((always_inline)) {
    constexpr int RB = decltype(row_bytes_c)::value;
#pragma unroll
    for (int k = 0; k < decltype(instr_c)::value; ++k) {
      const int byte = (kw + k * 4) * 1024 + lane * 16, row = byte / RB, c16 = (byte % RB) / 16;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (unsigned)(min(row, last_row) * RB + (c16 ^ swz(RB, row)) * 16)),
                                       (__attribute__((address_space(3))) void *)(dst + (kw + k * 4) * 1024), 16, 0, 2);
    }
  };
  bool b8 = false;
  auto request = [&](int tile) __attribute__((always_inline)) {
    locate(tile);
    if (valid <= 0) return;
    char *dst = lds + tw * TILE;
    b8 = FMT == 1 || (FMT == 2 && slot >= a.n_slots16);
    if (FMT != 0 && b8) {
      const size_t base = (((size_t)(slot - a.n_slots16) * Hkv + gkv) * C + (size_t)off * TK) * D;
      half((const char *)k8 + base, dst, std::integral_constant<int, D>{}, std::integral_constant<int, K8 / 4096>{}, valid - 1);
      half((const char *)v8 + base, dst + K8, std::integral_constant<int, TK>{}, std::integral_constant<int, K8 / 4096>{}, D - 1);
      const size_t at = (size_t)layer * a.scale_stride + ((size_t)(slot - a.n_slots16) * Hkv + gkv) * (C / TK) + off;
      ks8 = a.k_scale[at];
      vs8 = a.v_scale[at];
    } else if (FMT != 1) {
      const size_t base = (((size_t)slot * Hkv + gkv) * C + (size_t)off * TK) * D;
      half((const char *)(k16 + base), dst, std::integral_constant<int, D * 2>{}, std::integral_constant<int, K16 / 4096>{}, valid - 1);
      half((const char *)(v16 + base), dst + K16, std::integral_constant<int, TK * 2>{}, std::integral_constant<int, K16 / 4096>{}, D - 1);
    }
  };
  request(tile_begin + tw);

  gate(ticket, a.h_b + layer * a.s_word, wave);

  // ---- q, and in the last piece k and v of the fresh tokens, from the projection's sums: a row a wavefront, finished (bias, head
  // norm, RoPE, one rounding) into LDS.  Lane m has elements m and m + D / 2.
  __bf16 *const qs = (__bf16 *)(lds + kRing), *const ks = qs + R * D, *const vs = ks + T * D;
  int app_slot = -1, app_have = 0;
  if (with_fresh && a.append) {
    app_slot = a.append[2 * b];
    app_have = a.append[2 * b + 1];
  }
  {
    const Rsrc sums = rsrc_of(a.qsum + layer * a.s_word, a.n_qsum);
    const bool act = D == 128 || lane < 32;
    const int m = act ? lane : 0;
    for (int r = wave; r < (with_fresh ? R + 2 * T : R); r += kWaves) {
      const int kind = r < R ? 0 : r < R + T ? 1 : 2, t = kind == 0 ? r % T : kind == 1 ? r - R : r - R - T;
      const int head = kind == 0 ? gkv * G + r / T : kind == 1 ? Hq + gkv : Hq + Hkv + gkv;
      const __bf16 *const gain = kind == 0 ? q_norm : kind == 1 ? k_norm : nullptr;
      float b0 = 0.f, b1 = 0.f, g0 = 1.f, g1 = 1.f;
      float2 cs = make_float2(1.f, 0.f);
      if (bias) {
        b0 = (float)bias[head * D + m];
        b1 = (float)bias[head * D + m + D / 2];
      }
      if (gain) {
        g0 = (float)gain[m];
        g1 = (float)gain[m + D / 2];
      }
      if (kind < 2) cs = a.rope[(size_t)(l_pre + t) * (D / 2) + m];
      const unsigned at = (unsigned)(((b * T + t) * F + head * D + m) * 4);
      unsigned x0, x1;
      {
      Waiting wait;
      for (int tries = 0;; ++tries) {
        x0 = __builtin_amdgcn_raw_buffer_load_b32(sums, at, 0, kSc1);
        x1 = __builtin_amdgcn_raw_buffer_load_b32(sums, at + D * 2, 0, kSc1);
        if (__ballot(x0 == EMPTY || x1 == EMPTY) == 0 || given_up(tries, ticket)) break;
        pause<2>();
      }
      }
      float f0 = __uint_as_float(x0) + b0, f1 = __uint_as_float(x1) + b1;
      if (gain) {
        const float n = 1.0f / sqrtf(wave_sum(act ? f0 * f0 + f1 * f1 : 0.f) / (float)D + eps);
        f0 *= n * g0;
        f1 *= n * g1;
      }
      if (act) {
        qs[r * D + m] = (__bf16)(f0 * cs.x - f1 * cs.y);
        qs[r * D + m + D / 2] = (__bf16)(f1 * cs.x + f0 * cs.y);
      }
    }
  }
  wait_vmcnt<0>();   // the first tiles too
  lds_barrier();
  const int row = min(l16, R - 1), my_i = row % T;
  const bool fresh_k = with_fresh && wave == 0;
  const int vt = tid / VPR, vd = tid - vt * VPR;   // this thread's 8 elements of a fresh V row
  const bool fresh_v = with_fresh && vt < T;
  bf16x8 q[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) q[k] = *(const bf16x8 *)(qs + row * D + k * 32 + g * 8);

  f32x4 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref = -INFINITY, l_run = 0.f;
  auto soften = [&](f32x4 &s) __attribute__((always_inline)) {   // as in decode_attention.hip
    f32x4 p;
    auto exponentials = [&](float neg_m) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = fast_exp2(__builtin_fmaf(s[e], scale_log2e, neg_m));
      return (p[0] + p[1]) + (p[2] + p[3]);
    };
    float sum = 0.f;
    bool refresh = __builtin_amdgcn_ballot_w64(m_ref == -INFINITY) != 0;
    if (!refresh) {
      sum = exponentials(-m_ref);
      refresh = __builtin_amdgcn_ballot_w64(!(sum <= kSumLimit)) != 0;
    }
    if (refresh) {
      const float mc = row_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))) * scale_log2e;
      const bool upd = mc > m_ref;
      const float alpha = upd ? fast_exp2(m_ref - mc) : 1.0f;
      m_ref = upd ? mc : m_ref;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] *= alpha;
      sum = exponentials(m_ref == -INFINITY ? 0.f : -m_ref);
    }
    l_run += sum;
    return p;
  };
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  const int k_row = kw * 16 + l16;
  auto compute = [&]() __attribute__((always_inline)) {
    if (kw * 16 >= valid) return;
    const char *kb = lds + tw * TILE;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    bf16x4 vop[DB];
    if (FMT == 1 || (FMT == 2 && b8)) {
      const char *vb = kb + K8;
      uint2 raw[KS];
      unsigned vraw[DB];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) raw[ks] = *(const uint2 *)(kb + k_row * D + (((2 * ks + (g >> 1)) ^ swz(D, k_row)) * 16) + (g & 1) * 8);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const int r = db * 16 + l16;
        vraw[db] = *(const unsigned *)(vb + r * TK + (((2 * (kw >> 1) + (g & 1)) ^ swz(TK, r)) * 16) + 8 * (kw & 1) + 4 * (g >> 1));
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(codes8(raw[ks], ks8), q[ks], s, 0, 0, 0);
#pragma unroll
      for (int db = 0; db < DB; ++db) vop[db] = codes4(vraw[db], vs8);
    } else {
      const char *vb = kb + K16;
      bf16x8 kop[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kop[ks] = *(const bf16x8 *)(kb + k_row * (D * 2) + (((4 * ks + g) ^ swz(D * 2, k_row)) * 16));
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const int r = db * 16 + l16;
        vop[db] = *(const bf16x4 *)(vb + r * (TK * 2) + (((2 * kw + (g & 1)) ^ swz(TK * 2, r)) * 16) + 8 * (g >> 1));
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[ks], q[ks], s, 0, 0, 0);
    }
    if (valid < TK) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = kw * 16 + g * 4 + e < valid ? s[e] : -INFINITY;
      // what stands behind the last key need not be finite, or is being appended by this very launch
      const int left = valid - kw * 16 - g * 4;
      const uint2 mask = make_uint2((left > 0 ? 0xffffu : 0u) | (left > 1 ? 0xffff0000u : 0u), (left > 2 ? 0xffffu : 0u) | (left > 3 ? 0xffff0000u : 0u));
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const uint2 vv = __builtin_bit_cast(uint2, vop[db]);
        vop[db] = __builtin_bit_cast(bf16x4, make_uint2(vv.x & mask.x, vv.y & mask.y));
      }
    }
    const f32x4 p = soften(s);
    const bf16x4 pb = {(__bf16)p[0], (__bf16)p[1], (__bf16)p[2], (__bf16)p[3]};
#pragma unroll
    for (int db = 0; db < DB; ++db)
      o[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, vop[db]), __builtin_bit_cast(s16x4, pb), o[db], 0, 0, 0);
  };
  for (int t = tile_begin; t < tile_end; t += 2) {
    if (t > tile_begin) {
      __syncthreads();   // the tiles before have been read
      request(t + tw);
      wait_vmcnt<0>();
      __syncthreads();
    }
    compute();
  }
  f32x4 pf = {0.f, 0.f, 0.f, 0.f};
  if (fresh_k) {   // the fresh keys, causal
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    bf16x8 kf[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) kf[k] = *(const bf16x8 *)(ks + min(l16, T - 1) * D + k * 32 + g * 8);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], q[ks], s, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = g * 4 + e <= my_i ? s[e] : -INFINITY;
    pf = soften(s);
    if (l16 < T) {
      __bf16 *dense = a.k_dense + (size_t)layer * a.l_kv + (((size_t)b * Hkv + gkv) * T + l16) * D + g * 8;
      __bf16 *dst = app_slot >= 0 ? a.k16 + (size_t)layer * a.layer_stride + (((size_t)app_slot * Hkv + gkv) * C + app_have + l16) * D + g * 8 : nullptr;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        *(bf16x8 *)(dense + ks * 32) = kf[ks];
        if (dst) *(bf16x8 *)(dst + ks * 32) = kf[ks];
      }
    }
  }

  // ---- merge of the eight wavefronts
  claim(ticket, wave, lane, next);
  lds_barrier();
  float *om = (float *)lds;                    // [wave][row][O_ROW]
  float *ml = om + kWaves * R * O_ROW;         // [wave][row][2]
  float *pl = ml + kWaves * R * 2;             // [row][16] probabilities of the fresh keys
  if (fresh_v) {
    const bf16x8 v = *(const bf16x8 *)(vs + vt * D + vd * 8);
    *(bf16x8 *)(a.v_dense + (size_t)layer * a.l_kv + (((size_t)b * Hkv + gkv) * T + vt) * D + vd * 8) = v;
    if (app_slot >= 0) {
      const int at = app_have + vt, in = at & (TK - 1);
      __bf16 *dst = a.v16 + (size_t)layer * a.layer_stride + (((size_t)app_slot * Hkv + gkv) * C + (at - in)) * D + (in & ~15) + pc::blocked_key(in & 15);
#pragma unroll
      for (int e = 0; e < 8; ++e) dst[(vd * 8 + e) * TK] = v[e];
    }
  }
  if (with_fresh && app_slot >= 0) {   // a block that these tokens open gets zeros behind the last of them
    const int end = app_have + T, tail = end & (TK - 1);
    if (tail && (app_have == 0 || (end - 1) / TK > (app_have - 1) / TK)) {
      __bf16 *dst = a.v16 + (size_t)layer * a.layer_stride + (((size_t)app_slot * Hkv + gkv) * C + (end - tail)) * D;
      for (int u = tid; u < D * TK; u += 64 * kWaves) {
        const int p = u & (TK - 1);
        if ((p & ~15) + pc::blocked_key(p & 15) >= tail) dst[u] = (__bf16)0.f;
      }
    }
  }
  {
    const float l = row_sum(l_run);
    if (l16 < R) {
#pragma unroll
      for (int db = 0; db < DB; ++db) *(f32x4 *)(om + (wave * R + l16) * O_ROW + db * 16 + g * 4) = o[db];
      if (g == 0) {
        ml[(wave * R + l16) * 2] = m_ref;
        ml[(wave * R + l16) * 2 + 1] = l;
      }
      if (fresh_k) *(f32x4 *)(pl + l16 * 16 + g * 4) = pf;
    }
  }
  lds_barrier();
  const Rsrc po = rsrc_of(part, n_part);
  constexpr int UPR = D / 4;   // four columns a thread
  for (int u = tid; u < R * UPR; u += 64 * kWaves) {
    const int r = u / UPR, dv = u - r * UPR;
    float2 e[kWaves];
    f32x4 v[kWaves];
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      e[x] = *(const float2 *)(ml + (x * R + r) * 2);
      v[x] = *(const f32x4 *)(om + (x * R + r) * O_ROW + dv * 4);
    }
    float m = e[0].x;
#pragma unroll
    for (int x = 1; x < kWaves; ++x) m = fmaxf(m, e[x].x);
    float l = 0.f, a0 = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      const float f = e[x].x == -INFINITY ? 0.f : fast_exp2(e[x].x - m);
      if (x == 0) a0 = f;
      l += e[x].y * f;
      acc += v[x] * f;
    }
    if (with_fresh) {
      const int i = r % T;
      for (int t = 0; t <= i; ++t) {
        const float p = pl[r * 16 + t] * a0;
        const bf16x4 fv = *(const bf16x4 *)(vs + t * D + dv * 4);
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[x] += p * (float)fv[x];
      }
    }
    acc *= l > 0.f ? 1.0f / l : 0.f;
    const unsigned prow = (unsigned)(((b * Hkv + gkv) * R + r) * n_splits + split);
    hand_over(po, (prow * (D + kTail) + dv * 4) * 4, __builtin_bit_cast(u32x4, acc));
    if (dv == 0) hand_over(po, (prow * (D + kTail) + D) * 4, make_uint2(__float_as_uint(m), __float_as_uint(l)));
  }
}

// ---------------------------------------------------------------------------------------------------
// X: the pieces of one kv head's rows merged, by the rule of splitkv_combine_kernel.  `share` neighbouring lanes have 8 columns of a row and
// take every share-th piece.  The next item is taken before the pieces are there: behind them a layer of width 3072 is slower (12 tiles 47.8 us, behind
// them 48.4), most are as fast (width 1024, 38 tiles 23.9 either way); but where the QKV items just fill the CUs nobody else is free for the o_proj's,
// and it would be the better way (width 2048, 24 tiles 34.5 | 32.3, 1024 over 60 tiles 27.8 | 24.7).
// ---------------------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void merge(const KArgs &a, int layer, int bg, int wave, int lane, unsigned &next) {
  constexpr int VPR = D / 8, CH = 4;
  unsigned *const ticket = pinned(a.ticket);
  const int T = pinned(a.T), Hkv = pinned(a.Hkv), Hq = pinned(a.Hq), G = Hq / Hkv, R = G * T, tid = wave * 64 + lane, b = bg / Hkv, gkv = bg % Hkv, ns = pinned(a.n_splits);
  const Rsrc out = rsrc_of(pinned(a.attn + 2 * layer * a.s_word), pinned(a.n_attn));
  const int share_log2 = pinned(a.x_share_log2), n_lanes = 1 << share_log2, u = tid >> share_log2, j0 = tid & (n_lanes - 1);
  gate(ticket, a.qsum + layer * a.s_word, wave);
  claim(ticket, wave, lane, next);
  if ((wave * 64) >> share_log2 >= R * VPR) return;   // (whole wavefronts)
  const bool mine = u < R * VPR;
  const int r = mine ? u / VPR : 0, dv = u - u / VPR * VPR;
  const Rsrc po = rsrc_of(pinned(a.part + layer * a.s_word), pinned(a.n_part));
  const unsigned prow = (unsigned)((bg * R + r) * ns);
  float mx = -INFINITY, wsum = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int p0 = 0; p0 < ns; p0 += CH << share_log2) {
    uint2 e[CH];
    u32x4 o[CH][2];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      e[j] = make_uint2(EMPTY, EMPTY);
      o[j][0] = o[j][1] = u32x4{EMPTY, EMPTY, EMPTY, EMPTY};
    }
    {
      Waiting w;
      bool all = false;   // the first maxima and sums are there: ask for everything
      for (int tries = 0;; ++tries) {
        bool bad = false;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
          if (j > 0 && !all) break;
          const int p = p0 + j0 + (j << share_log2);
          const bool in = mine && p < ns;
          const unsigned row = (prow + p) * ((D + kTail) * 4);
          e[j] = ask2(po, in ? row + D * 4 : kNowhere);
          if (!all) break;
          o[j][0] = ask(po, in ? row + dv * 32 : kNowhere);
          o[j][1] = ask(po, in ? row + dv * 32 + 16 : kNowhere);
        }
#pragma unroll
        for (int j = 0; j < CH; ++j) {
          if (j > 0 && !all) break;
          bad = bad || missing(e[j]) || (all && (missing(o[j][0]) || missing(o[j][1])));
        }
        const bool there = __ballot(bad) == 0;
        if ((there && all) || given_up(tries, ticket)) break;
        if (there) all = true;
        else if (all) pause<16>();
        else pause<4>();
      }
    }
    float top = mx;
#pragma unroll
    for (int j = 0; j < CH; ++j) {   // (past the list: zeros, weight 0)
      const float l = __uint_as_float(e[j].y);
      if (l > 0.f) top = fmaxf(top, __uint_as_float(e[j].x));
    }
    const float shrink = mx == -INFINITY ? 0.f : exp2f(mx - top);
    mx = top;
    wsum *= shrink;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= shrink;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const float l = __uint_as_float(e[j].y), f = l > 0.f ? l * exp2f(__uint_as_float(e[j].x) - top) : 0.f;
      wsum += f;
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += f * __uint_as_float(i < 4 ? o[j][0][i & 3] : o[j][1][i & 3]);
    }
  }
  float top = mx;
  for (int s = 1; s < n_lanes; s <<= 1) top = fmaxf(top, __shfl_xor(top, s, 64));
  const float f = mx == -INFINITY ? 0.f : exp2f(mx - top);
  wsum *= f;
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] *= f;
  for (int s = 1; s < n_lanes; s <<= 1) {
    wsum += __shfl_xor(wsum, s, 64);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += __shfl_xor(acc[i], s, 64);
  }
  if (!mine || j0 != 0) return;
  const float inv = wsum > 0.f ? 1.0f / wsum : 0.f;
  bf16x8 v;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (__bf16)(acc[i] * inv);
  const int hg = r / T, i = r - hg * T;
  hand_over(out, (unsigned)(((b * T + i) * Hq * D + (gkv * G + hg) * D + dv * 8) * 2), __builtin_bit_cast(u32x4, v));
}

template <int D, int FMT>
__global__ __launch_bounds__(64 * kWaves, 2) void decode_stack_kernel(const Args args) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int next_s;
  __builtin_amdgcn_s_setprio(2);
  if (threadIdx.x == 0) next_s = (int)__hip_atomic_fetch_add(args.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  int item = __builtin_amdgcn_readfirstlane(next_s);
  while (item < args.n_items) {
    // (opaque: what an item derives from these stays inside it -- kept across the loop, the steps' addresses take all registers)
    const KArgs *ap = (const KArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    int tid = threadIdx.x;
    asm volatile("" : "+s"(ap), "+v"(tid));
    const KArgs &a = *ap;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4;
    const int M = pinned(a.M), H = pinned(a.H), A = pinned(a.Hq) * D, F = A + 2 * pinned(a.Hkv) * D, FF = pinned(a.ffn);
    unsigned *const ticket = pinned(a.ticket);
    const float eps = pinned(a.eps), inv_h = pinned(a.inv_h);
    unsigned next = 0;
    const int layer = item / a.per_layer;
    int id = item - layer * a.per_layer;
    const KLayer &w = a.w[layer];
    const size_t blk = layer * a.s_word;
    float *const squares = (float *)(lds + kRing + kWaves * a.x_bytes);   // [M][H / 16] sums of squares of the token rows
    const int m = min(l16, M - 1);
    if (id >= a.n_q && id < a.n_q + a.n_t) {
      attend<D, FMT>(a, lds, layer, id - a.n_q, wave, lane, next);
    } else if (id >= a.n_q + a.n_t && id < a.n_q + a.n_t + a.n_x) {
      merge<D>(a, layer, id - a.n_q - a.n_t, wave, lane, next);
    } else if (id >= a.per_layer - a.n_o - a.n_g && id < a.per_layer - a.n_o) {
      f32x4 acc[2];
      const Rsrc to = rsrc_of(pinned(a.act + 2 * blk), pinned(a.n_act));
      const int f0 = (id - (a.per_layer - a.n_o - a.n_g)) * 16;
      project<2>(a, lds, [&](int r) __attribute__((always_inline)) { return (r < 16 ? w.w_gate + (size_t)(f0 + r) * H : w.w_up + (size_t)(f0 + r - 16) * H); },
                 rsrc_of((const char *)(a.mid_b + blk), a.n_block), true, squares, a.attn + 2 * blk, H, wave, lane, false,
                 []() __attribute__((always_inline)) { return false; }, acc);
      claim(ticket, wave, lane, next);
      share<2>(lds, wave, lane, acc);
      if (wave == 0) {
        f32x4 gate = sum_of(lds, 0, lane), up = sum_of(lds, 1, lane);
        const float r = norm_factor(squares, m, M, H, g, inv_h, eps);
        gate *= r;
        up *= r;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = gate[e] / (1.0f + __expf(-gate[e])) * up[e];
        if (l16 < M) hand_over(to, (unsigned)((l16 * FF + f0 + g * 4) * 2), pack4(o[0], o[1], o[2], o[3]));
      }
    } else {
      // QKV, o_proj, down projection: one loop, three sets of operands
      const int kind = id < a.n_q ? 0 : id < a.per_layer - a.n_o ? 1 : 2;
      const int n0 = (kind == 0 ? id : kind == 1 ? id - (a.n_q + a.n_t + a.n_x) : id - (a.per_layer - a.n_o)) * 16, K = kind == 0 ? H : kind == 1 ? A : FF;
      const __bf16 *const w0 = (kind == 0 ? w.wqkv : kind == 1 ? w.wo : w.w_down) + (size_t)n0 * K;
      const Rsrc x = kind == 0 ? rsrc_of((const __bf16 *)(a.h_b + blk), a.n_block / 2) : kind == 1 ? rsrc_of(a.attn + 2 * blk, a.n_attn) : rsrc_of(a.act + 2 * blk, a.n_act);
      const void *const before = kind == 0 ? (layer > 0 ? a.act + 2 * (blk - a.s_word) : nullptr) : kind == 1 ? (void *)(a.part + blk) : a.mid_b + blk;
      const Rsrc res = rsrc_of((kind == 1 ? a.h : a.mid) + 2 * blk, a.n_h);
      const unsigned out = (unsigned)((m * H + n0 + g * 4) * 2);
      const size_t nb = blk + a.s_word;
      const bool ends = kind == 2 && layer == a.out_layer;
      char *const to = pinned(kind == 0 ? (char *)(a.qsum + blk) : kind == 1 ? (char *)(a.mid + 2 * blk) : ends ? (char *)a.h_out : (char *)(a.h + 2 * nb));
      const char *const to_b = pinned(kind == 1 ? (const char *)(a.mid_b + blk) : (const char *)(a.h_b + nb));
      const size_t n_to = pinned(kind == 0 ? a.n_qsum * 4 : a.n_h * 2), n_block = pinned(a.n_block);
      f32x4 acc[1];
      uint2 rw = make_uint2(0, 0), gain = rw;
      const __bf16 *const gains = kind == 1 ? w.gain2 : layer + 1 < a.n_layers ? a.w[layer + 1].gain1 : a.gain_after;
      if (kind != 0 && wave == 0 && gains) gain = *(const uint2 *)(gains + n0 + g * 4);
      project<1>(a, lds, [&](int r) __attribute__((always_inline)) { return w0 + (size_t)r * K; }, x, kind == 0, squares, before, K, wave, lane, kind != 0 && wave == 0,
                 [&]() __attribute__((always_inline)) {
                   rw = ask2(res, out);
                   return missing(rw);
                 }, acc);
      claim(ticket, wave, lane, next);
      share<1>(lds, wave, lane, acc);
      if (wave == 0) {
        f32x4 s = sum_of(lds, 0, lane);
        if (kind == 0) {
          s *= norm_factor(squares, m, M, H, g, inv_h, eps);
          if (l16 < M) hand_over(rsrc_of(to, n_to), (unsigned)((l16 * F + n0 + g * 4) * 4), __builtin_bit_cast(u32x4, s));
        } else {
          float r[4];
          unpack4(rw, r);
          const uint2 v = pack4(s[0] + r[0], s[1] + r[1], s[2] + r[2], s[3] + r[3]);
          if (!ends) hand_over_row(v, gain, rsrc_of(to, n_to), rsrc_of(to_b, n_block), m, n0, H, l16, g, M);
          else if (l16 < M) *(uint2 *)(to + out) = v;
        }
      }
    }
    __syncthreads();   // the item's LDS is free
    if (tid == 64) next_s = (int)next;
    __syncthreads();
    item = __builtin_amdgcn_readfirstlane(next_s);
  }
}

// What a step needs before its first launch: the buffers of the hand-over filled with ones, the counters at zero, the chunk lists, and
// the first layer's input handed over (workgroup m: row m).
__global__ __launch_bounds__(256) void decode_stack_begin_kernel(u32x4 *fill, size_t n_fill, unsigned *tickets, int n_tickets, int32_t *table, int n_list,
                                                                 const __bf16 *__restrict__ h_in, const __bf16 *__restrict__ gain, int M, int H, __bf16 *h,
                                                                 float *h_b, const pc::ListWords lists) {
  const u32x4 ones = {EMPTY, EMPTY, EMPTY, EMPTY};
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_fill; i += (size_t)gridDim.x * 256) fill[i] = ones;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < n_tickets; i += 256) tickets[i] = 0;
    for (int i = threadIdx.x; i < n_list; i += 256) table[i] = lists.v[i];
  }
  const int m = blockIdx.x;
  if (m >= M) return;
  for (int c = threadIdx.x; c < H / 4; c += 256) {   // (four neighbouring lanes have 16 columns; H is a multiple of 128)
    const uint2 v = *(const uint2 *)(h_in + (size_t)m * H + c * 4);
    float x[4], gn[4];
    unpack4(v, x);
    unpack4(*(const uint2 *)(gain + c * 4), gn);
    float sq = (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
    sq += __shfl_xor(sq, 1, 64);
    sq += __shfl_xor(sq, 2, 64);
    const uint2 p = pack4(x[0] * gn[0], x[1] * gn[1], x[2] * gn[2], x[3] * gn[3]);
    *(uint2 *)(h + (size_t)m * H + c * 4) = make_uint2(keep(v.x), keep(v.y));
    char *const blk = (char *)h_b + (size_t)(m * (H / 16) + c / 4) * kBlock;
    *(uint2 *)(blk + (c & 3) * 8) = make_uint2(keep(p.x), keep(p.y));
    if ((c & 3) == 0) *(uint2 *)(blk + 32) = make_uint2(keep(__float_as_uint(sq)), keep(__float_as_uint(sq)));
  }
}

}  // namespace

namespace pc {
namespace stackdec {

// The blocks of a layer that are handed over, in words of 4 bytes, for n_splits pieces of the key axis; the layer's input in front.
struct Blocks {
  size_t h, block, qsum, part, attn, act, total;
  size_t head() const { return h + block; }
};
static Blocks blocks_of(const percache_config &c, int M, int ffn, int n_splits) {
  auto up = [](size_t w) { return align_up(w, 64); };
  const size_t A = (size_t)c.n_q_heads * c.head_dim, rows = (size_t)M * c.n_q_heads;
  Blocks b;
  b.h = up((size_t)M * c.hidden / 2);
  b.block = up((size_t)M * (c.hidden / 16) * (kBlock / 4));
  b.qsum = up((size_t)M * (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim);
  b.part = up(rows * n_splits * (c.head_dim + kTail));
  b.attn = up(M * A / 2);
  b.act = up((size_t)M * ffn / 2);
  b.total = 2 * b.head() + b.qsum + b.part + b.attn + b.act;
  return b;
}
// one counter a launch
static size_t ticket_bytes(int n_layers) { return align_up((size_t)((n_layers + kMaxLayers - 1) / kMaxLayers) * sizeof(unsigned)); }
static size_t dense_elems(const percache_config &c, int M) { return align_up((size_t)M * c.n_kv_heads * c.head_dim, 128); }

// Which steps take this path.  The chain of launches costs 6 to 8 us a layer more than the items, a step's beginning (the fill, the loads of a
// cold launch) 6.5 once; what takes the gain away is rows that every workgroup polls and reads out of LDS, items that leave a round of workgroups
// half empty, and pieces of the key axis past a round of them (takes).  us a layer, launch by launch | here, two cached tiles a query unless said:
//   layers: one row of width 1024, one layer 24.6 | 23.9, at 24 tiles 26.7 | 26.7, at 60 29.0 | 31.1; two layers 25.1 | 21.5, eight 25.6 | 19.8; of width
//   896, one layer 24.8 | 26.1, two 25.3 | 23.6; four rows of width 1024, two layers 27.3 | 27.0, four 27.6 | 25.7; two of width 512, one 18.4 | 20.8,
//   two 19.1 | 18.0, four 19.6 | 16.7; one row of width 4096, 38 tiles, two layers 85.3 | 86.9, four 86.0 | 85.5.
//   width, one row, eight layers: 3072 51.0 | 44.5, 4096 82.6 | 78.9, 5120 (320 items on 256 CUs) 107 | 115, 8192 280 | 276; between gate/up and down
//   14 336 columns gain (width 4096), 18 944 do not (3584) 86.5 | 88.2.  Two rows of 2048, two layers 37.0 | 38.0.
//   rows times the widest contraction: 9216 (three rows of width 1024) four layers 27.6 | 25.2, 9728 (two tokens of a query, width 896) four layers 25.9 |
//   26.3, eight 26.2 | 25.6, 12 288 (three rows of width 1280) eight layers 29.6 | 25.8, 14 592 (three of width 896) four layers 27.0 | 26.9, 17 920 (two
//   of width 1536) eight layers 39.8 | 40.0.
constexpr int kMaxWidth = 4096, kMaxContraction = 16384;
static bool shape_fits(const percache_config &c, int32_t batch, int32_t t_fresh, int32_t ffn, int n_layers) {
  const long R = (long)(c.n_q_heads / c.n_kv_heads) * t_fresh, M = (long)batch * t_fresh, A = (long)c.n_q_heads * c.head_dim;
  if (R > kMaxQueryRows || M > kMaxRows || M * c.hidden > kMaxWidth) return false;
  if (M * (ffn > A ? ffn : A) > (M == 1 ? kMaxContraction : n_layers < 8 ? 9216 : 12288)) return false;
  if (n_layers < (M == 1 && c.hidden <= 3072 ? 2 : 4)) return false;
  // the merge of the wavefronts' outputs, in the ring's place
  return (size_t)kWaves * R * (c.head_dim + 6) * 4 + R * 64 <= (size_t)kRing;
}
static int splits_for(const percache_config &c, int n_cu, int32_t batch, int32_t t_fresh, int max_tiles) {
  const int cap = max_splits_for(c, n_cu, batch, t_fresh), want = (max_tiles + 3) / 2;
  return want < cap ? want : cap;
}

size_t workspace_bytes(const percache_config &c, int n_cu, int32_t batch, int32_t t_fresh, int32_t ffn, int n_layers, int max_tiles) {
  if (!shape_fits(c, batch, t_fresh, ffn, n_layers)) return 0;
  const int M = batch * t_fresh;
  const Blocks b = blocks_of(c, M, ffn, splits_for(c, n_cu, batch, t_fresh, max_tiles));
  return ticket_bytes(n_layers) + (n_layers * b.total + b.head()) * 4 + (size_t)n_layers * 2 * dense_elems(c, M) * 2;
}

// At most four tiles, two rounds, to a piece: more of them want the ring of decode_attention_kernel.  The pieces of a layer hold the workgroups
// that should have its o_proj and gate/up weights on their way, and the merge of a kv head's pieces is one workgroup's.  us a layer, launch by
// launch | here, 256 CUs:
//   pieces, one row, four layers: width 1024, 248 30.5 | 27.9, 408 32.5 | 30.0, 512 33.6 | 33.6, 16 heads of 64, 320 27.1 | 26.3, 496 28.7 | 28.9; width
//   2048, 248 40.7 | 37.9, 408 43.0 | 42.6, 512 44.2 | 46.0; width 2560, 160 55.8 | 53.3, 248 56.7 | 56.8, 328 57.9 | 59.8; width 3072, 248 54.1 |
//   50.6, 408 56.0 | 55.3, 512 57.0 | 60.3; width 4096, 248 86.6 | 87.2, 328 87.9 | 89.8.
//   two layers: width 1024, 160 28.2 | 24.9, 408 32.2 | 31.2, 512 33.4 | 35.0; width 2560, 160 55.3 | 55.1, 248 56.4 | 58.6.
//   several rows, four layers, width 1024: two rows, 160 28.8 | 26.2, three 168 29.0 | 28.3, three tokens of a query, 104 29.0 | 27.8, 160 30.1 | 30.4, two
//   over 16 heads of 64, 64 24.9 | 24.1, 160 26.1 | 27.0; three rows over nothing cached 24.4 | 24.6.
//   floats that a merge reads (rows x head size x pieces of a kv head), four layers: one row, 48 000 51.5 | 50.3, 55 000 38.1 | 33.8, 63 000 52.4 | 54.0, 73 000
//   39.3 | 37.9, 91 000 39.8 | 39.5; several, 26 000 31.3 | 30.3, 38 000 32.2 | 32.1, 40 000 31.4 | 32.5.
bool takes(const percache_config &c, int n_cu, int32_t batch, int32_t t_fresh, int32_t ffn, int n_layers, int max_tiles) {
  if (!shape_fits(c, batch, t_fresh, ffn, n_layers)) return false;
  const int M = batch * t_fresh, ns = splits_for(c, n_cu, batch, t_fresh, max_tiles);
  const long pieces = (long)batch * c.n_kv_heads * ns, merge = (long)(c.n_q_heads / c.n_kv_heads) * t_fresh * c.head_dim * ns;
  if (max_tiles + 2 > 4 * ns) return false;
  if (M > 1) return max_tiles > 0 && pieces * 8 <= n_cu * 5L && merge <= 32768;
  const int eighths = n_layers < 4 ? 5 : c.hidden <= 1024 ? 14 : 8;   // of n_cu
  return pieces * 8 <= (long)n_cu * eighths && merge <= 57344;
}

template <int D>
static pc_status launch_kernel(percache_ctx *ctx, int fmt, dim3 grid, size_t lds, hipStream_t s, const Args &a) {
  void (*const kernel)(Args) = fmt == 0 ? decode_stack_kernel<D, 0> : fmt == 1 ? decode_stack_kernel<D, 1> : decode_stack_kernel<D, 2>;
  PC_HIP(ctx, hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));   // (above 64 KB it must be opted into)
  hipLaunchKernelGGL(kernel, grid, dim3(64 * kWaves), lds, s, a);
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}

pc_status launch(percache_ctx *ctx, const percache_block_weights *layers, int n_layers, int ffn, float eps, const __bf16 *h_in, int batch, int t_fresh,
                 const std::vector<int32_t> *rows, int32_t *table, int tbl_stride, bool append, int max_tiles, int formats, __bf16 *h_out, void *ws,
                 const __bf16 **k_dense, const __bf16 **v_dense, size_t *dense_stride, hipStream_t stream) {
  const percache_config &c = ctx->cfg;
  const int M = batch * t_fresh, R = c.n_q_heads / c.n_kv_heads * t_fresh, D = c.head_dim, A = c.n_q_heads * D;
  const int ns = splits_for(c, ctx->n_cu, batch, t_fresh, max_tiles);
  const Blocks b = blocks_of(c, M, ffn, ns);
  unsigned *const tickets = (unsigned *)ws;
  char *p = (char *)ws + ticket_bytes(n_layers);
  Args a;
  memset(&a, 0, sizeof a);
  float *words = (float *)p;
  // layer after layer, a layer's blocks one behind the other; behind the last layer the input of one more (never written by the last
  // launch, between two launches as between two layers)
  const size_t total = ((size_t)n_layers * b.total + b.head()) * 4;
  a.h = (__bf16 *)words;
  a.h_b = (float *)(a.h + 2 * b.h);
  a.qsum = a.h_b + b.block;
  a.part = a.qsum + b.qsum;
  a.attn = (__bf16 *)(a.part + b.part);
  a.mid = a.attn + 2 * b.attn;
  a.mid_b = (float *)(a.mid + 2 * b.h);
  a.act = (__bf16 *)(a.mid_b + b.block);
  a.s_word = b.total;
  a.n_h = 2 * b.h;
  a.n_block = b.block * 4;
  a.n_qsum = b.qsum;
  a.n_part = b.part;
  a.n_attn = 2 * b.attn;
  a.n_act = 2 * b.act;
  const size_t dense = dense_elems(c, M);
  a.k_dense = (__bf16 *)(p + total);
  a.v_dense = a.k_dense + (size_t)n_layers * dense;
  a.l_kv = dense;
  *k_dense = a.k_dense;
  *v_dense = a.v_dense;
  *dense_stride = dense;
  a.table = table;
  a.append = append ? table + (size_t)batch * tbl_stride : nullptr;
  a.rope = (const float2 *)ctx->rope;
  a.n_slots16 = ctx->n_slots16;
  a.layer_stride = ctx->layer_stride;
  a.layer_stride8 = ctx->layer_stride8;
  a.scale_stride = (size_t)ctx->n_slots8 * c.n_kv_heads * (c.slot_capacity / kKvTile);
  a.eps = eps;
  a.inv_h = 1.0f / (float)c.hidden;
  a.scale_log2e = 1.4426950408889634f / sqrtf((float)D);
  a.M = M;
  a.T = t_fresh;
  a.H = c.hidden;
  a.Hq = c.n_q_heads;
  a.Hkv = c.n_kv_heads;
  a.ffn = ffn;
  a.C = c.slot_capacity;
  a.tbl_stride = tbl_stride;
  a.n_splits = ns;
  a.n_q = (A + 2 * c.n_kv_heads * D) / 16;
  a.n_t = batch * c.n_kv_heads * ns;
  a.n_x = batch * c.n_kv_heads;
  a.n_o = c.hidden / 16;
  a.n_g = ffn / 16;
  a.per_layer = a.n_q + a.n_t + a.n_x + 2 * a.n_o + a.n_g;
  while ((64 * kWaves >> (a.x_share_log2 + 1)) >= R * (D / 8) && a.x_share_log2 < 5 && (1 << a.x_share_log2) < ns) ++a.x_share_log2;
  // LDS: the ring and the token rows of the widest contraction; one workgroup a CU (two, which reach further ahead but wait in twice the
  // number: width 1024, one row 24.5 us a layer against 23.5, four rows 33.4 against 31.3)
  const int widest = c.hidden > ffn ? (c.hidden > A ? c.hidden : A) : (ffn > A ? ffn : A), sq = M * (c.hidden / 16) * 4 + 32;
  static_assert(kRing + kMaxContraction * 2 + kWaves * kMaxRows * 128 + kMaxWidth / 4 + 512 <= 160 * 1024 && kMaxWidth <= kRowCols, "LDS of the rows");
  a.x_bytes = (widest / 64 + kWaves - 1) / kWaves * M * 128;
  const size_t rows_lds = (size_t)kWaves * a.x_bytes, qkv_lds = (size_t)(R + 2 * t_fresh) * D * 2;   // (q, k and v of an attention item stand there too)
  const size_t lds = kRing + (rows_lds + sq > qkv_lds ? rows_lds + sq : qkv_lds);

  const int n_launches = (n_layers + kMaxLayers - 1) / kMaxLayers;
  const bool inline_list = rows && rows->size() <= (size_t)kListWords;
  if (rows && !inline_list) {
    const pc_status st = upload_table(ctx, *rows, table, stream);
    if (st != PC_OK) return st;
  }
  static_assert(sizeof(ListWords) + 64 <= 4096 && sizeof(Args) <= 4096, "launch arguments");
  ListWords lists;
  const int n_list = inline_list ? (int)rows->size() : 0;
  memset(&lists, 0, sizeof lists);
  if (n_list) memcpy(lists.v, rows->data(), (size_t)n_list * 4);
  const size_t head = b.head() * 4, n16 = (total - head) / 16;
  unsigned blocks = (unsigned)((n16 + 1023) / 1024 < 2048 ? (n16 + 1023) / 1024 : 2048);
  if (blocks < (unsigned)M) blocks = (unsigned)M;
  hipLaunchKernelGGL(decode_stack_begin_kernel, dim3(blocks), dim3(256), 0, stream, (u32x4 *)(p + head), n16, tickets, n_launches, table, n_list, h_in,
                     (const __bf16 *)layers[0].gain1, M, c.hidden, a.h, a.h_b, lists);
  PC_HIP(ctx, hipGetLastError());

  const int fmt = !((formats & 1) && ctx->n_slots8 > 0) ? 0 : (formats & 2) ? 2 : 1;
  const Args base = a;
  for (int l0 = 0, k = 0; l0 < n_layers; l0 += kMaxLayers, ++k) {
    const int n = n_layers - l0 < kMaxLayers ? n_layers - l0 : kMaxLayers;
    a = base;
    for (int l = 0; l < n; ++l) {
      const percache_block_weights &w = layers[l0 + l];
      a.w[l] = LayerPtrs{(const __bf16 *)w.gain1, (const __bf16 *)w.wqkv, (const __bf16 *)w.wo, (const __bf16 *)w.gain2, (const __bf16 *)w.w_gate,
                         (const __bf16 *)w.w_up, (const __bf16 *)w.w_down, (const __bf16 *)w.qkv_bias, (const __bf16 *)w.q_norm, (const __bf16 *)w.k_norm};
    }
    const size_t skip = (size_t)l0 * b.total;
    for (float **f : {&a.h_b, &a.qsum, &a.part, &a.mid_b}) *f += skip;
    for (__bf16 **f : {&a.h, &a.attn, &a.mid, &a.act}) *f += 2 * skip;
    a.n_layers = n;
    a.gain_after = l0 + n < n_layers ? (const __bf16 *)layers[l0 + n].gain1 : nullptr;
    a.k_dense += (size_t)l0 * dense;
    a.v_dense += (size_t)l0 * dense;
    a.k16 = ctx->k_store + (size_t)l0 * a.layer_stride;
    a.v16 = ctx->v_store + (size_t)l0 * a.layer_stride;
    a.k8 = ctx->k8_store + (size_t)l0 * a.layer_stride8;
    a.v8 = ctx->v8_store + (size_t)l0 * a.layer_stride8;
    a.k_scale = ctx->k_scale + (size_t)l0 * a.scale_stride;
    a.v_scale = ctx->v_scale + (size_t)l0 * a.scale_stride;
    a.h_out = h_out;
    a.out_layer = l0 + n == n_layers ? n - 1 : -1;
    a.ticket = tickets + k;
    a.n_items = n * a.per_layer;
    const int grid = a.n_items < ctx->n_cu ? a.n_items : ctx->n_cu;
    const pc_status st = D == 128 ? launch_kernel<128>(ctx, fmt, dim3(grid), lds, stream, a) : launch_kernel<64>(ctx, fmt, dim3(grid), lds, stream, a);
    if (st != PC_OK) return st;
  }
  return PC_OK;
}

}  // namespace stackdec
}  // namespace pc
