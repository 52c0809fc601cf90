// Slot-indexed per-layer K/V store: the device-resident form of the per-chunk tensor files of
// Sec. 4.1.1 (cache slicer output).
//
// Layout per layer and (slot, kv head), chosen for the attention kernel's streams:
//   K: [token][head_dim] bf16                       -- one 64-key tile is a contiguous 16 KB run (D = 128)
//   V: [token / 64][head_dim][64 keys] bf16 blocks  -- the transposed tile the PV product consumes, also one
//      contiguous run; inside each group of 16 keys the order is pc::blocked_key (see percache_internal.hpp);
//      keys past the stored count are zero in the last block.
// percache_kv_put / percache_kv_get convert from / to the caller's dense [kv head][token][head_dim] tensors.
#include "percache_internal.hpp"

namespace {
using pc::kKvTile;

// One launch serves a list of (slot, dense block) pairs.  A dense block is a token range of a dense tensor: head g's token t
// is row  row0 + g * head_rows + t  of D elements.  Only as many entries are filled in as the launch has (grid z).  The lists are
// kernel arguments: a call of a few short chunks costs what its launch costs, so chunks that are tensors of their own travel
// as slot ids alone, and short append lists in 128 bytes (a put of one chunk 8.2 us, host bound; with 1 KB lists copied twice 8.8).
constexpr int kListMax = 64;
struct Entry {
  int32_t slot;    // slot of the format the kernel handles (kv_mixed_kernel: of the context), negative: skip the entry
  int32_t row0;
  int32_t n_tok;
  int32_t off;     // tokens the slot already holds (append; else 0)
};
struct ChunkList {   // chunks of n_tok tokens, chunk i from row i * row_step on
  int32_t slots[kListMax];
  int32_t n_tok, row_step;
  __host__ __device__ Entry at(int i) const { return {slots[i], i * row_step, n_tok, 0}; }
  void set_slot(int i, int32_t slot) { slots[i] = slot; }
};
template <int N>
struct PieceList {
  Entry entry[N];
  __host__ __device__ Entry at(int i) const { return entry[i]; }
  void set_slot(int i, int32_t slot) { entry[i].slot = slot; }
};

// 8 x 8 sixteen-bit elements: out[k] holds element k of in[0..7]
__device__ __forceinline__ void transpose8(const pc::u32x4 (&in)[8], pc::u32x4 (&out)[8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int p = 0; p < 4; ++p)
      out[k][p] = __builtin_amdgcn_perm(in[2 * p + 1][k >> 1], in[2 * p][k >> 1], (k & 1) ? 0x07060302u : 0x05040100u);
}
// Chunk c of 8 positions of a 64-key block row holds the keys chunk_key(c, FMT8) + {0, 1, 2, 3, 8, 9, 10, 11} (the lane order of
// pc::blocked_key, of pc::blocked_key8 for 8-bit slots).
template <bool FMT8>
__device__ __forceinline__ int chunk_key(int c) {
  return FMT8 ? 32 * (c >> 2) + 16 * (c & 1) + 4 * ((c >> 1) & 1) : 16 * (c >> 1) + 4 * (c & 1);
}
__device__ __forceinline__ int in_chunk(int e) { return (e & 3) + 8 * (e >> 2); }

// bf16 slots <-> dense tensors.  HBM bound.  The unit of work is a wavefront with eight 16-byte loads and eight 16-byte stores
// per lane in flight: 64 tokens x 64 head-dim elements of K (a copy) or of V, where a lane holds an 8 x 8 piece -- 8 keys of
// a 64-key block's chunk x 8 head-dim elements -- and turns it in registers (32 byte permutes).  With 2-byte accesses on the
// dense (put) or the block (get) side a get of 8 chunks of 1000 tokens, 8 heads of 128, took 21.7 us, a put 13.0 us; now
// 9.6 us and 9.9 us (6.9 TB/s read and written).
struct Store16 {
  __bf16 *k, *v;
  long slot_stride;
};
template <int D, bool kToStore>
__device__ __forceinline__ void copy_unit(const Store16 &st, __bf16 *__restrict__ dense_k, __bf16 *__restrict__ dense_v, int C, const Entry &e, int slot, int g,
                                          int unit, int head_rows) {
  constexpr int UNITS = 2 * (D / 64);  // per tile: K and V halves
  __bf16 *const __restrict__ slot_k = st.k, *const __restrict__ slot_v = st.v;
  const long slot_stride_elems = st.slot_stride;
  const int n_tok = e.n_tok;
  const int tile = unit / UNITS, part = unit % UNITS, t0 = tile * kKvTile;
  if (slot < 0 || t0 >= n_tok) return;
  const int lane = threadIdx.x & 63, hi = lane >> 3, lo = lane & 7;
  const int d0 = (part >> 1) * 64;
  const size_t drow = (size_t)e.row0 + (size_t)g * head_rows + t0;
  const size_t sbase = (size_t)slot * slot_stride_elems + ((size_t)g * C + t0) * D;
  const int last = n_tok - 1 - t0;  // last token of this tile
  if (!(part & 1)) {  // K: 8 KB of the tile's contiguous run, 1 KB per instruction
    const __bf16 *src = kToStore ? dense_k + drow * D : slot_k + sbase;
    __bf16 *dst = kToStore ? slot_k + sbase : dense_k + drow * D;
    const int at = (part >> 1) * 4096 + lane * 8, end = (min(last, kKvTile - 1) + 1) * D;
    pc::u32x4 r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = *(const pc::u32x4 *)(src + min(at + j * 512, end - 8));
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (at + j * 512 < end) *(pc::u32x4 *)(dst + at + j * 512) = r[j];
    return;
  }
  pc::u32x4 in[8], out[8];
  __bf16 *block = slot_v + sbase + (size_t)(d0 + hi * 8) * kKvTile + lo * 8;  // chunk lo of the block rows d0 + 8 hi ..
  __bf16 *rows = dense_v + drow * D + d0 + hi * 8;                             // 8 elements of token rows chunk_key(lo) + ..
  const int k0 = chunk_key<false>(lo);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int t = k0 + in_chunk(j);
    if (!kToStore) in[j] = *(const pc::u32x4 *)(block + j * kKvTile);
    else in[j] = *(const pc::u32x4 *)(rows + (size_t)min(t, last) * D);
    if (kToStore && t > last) in[j] = pc::u32x4{0, 0, 0, 0};  // (keys past the end)
  }
  transpose8(in, out);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int t = k0 + in_chunk(j);
    if (kToStore) *(pc::u32x4 *)(block + j * kKvTile) = out[j];
    else if (t <= last) *(pc::u32x4 *)(rows + (size_t)t * D) = out[j];
  }
}
template <int D, bool kToStore, class List>
__global__ __launch_bounds__(256) void kv_copy_kernel(Store16 st, __bf16 *__restrict__ dense_k, __bf16 *__restrict__ dense_v, int C, List list, int head_rows) {
  const Entry e = list.at(blockIdx.z);
  copy_unit<D, kToStore>(st, dense_k, dense_v, C, e, e.slot, blockIdx.y, blockIdx.x * 4 + (threadIdx.x >> 6), head_rows);
}

// Appends n_new tokens behind the off tokens a slot already holds; blockIdx.y selects the slot of a list (one launch for
// all queries of a decoding step).  K: rows copied to their place.  V: every position of the 64-key blocks that receive a
// token is rewritten from off on -- the new tokens, then zeros, so that the padding of the last block stays finite
// (masked probabilities multiply it).
template <class List>
__global__ __launch_bounds__(256) void kv_append_kernel(__bf16 *__restrict__ k_store, __bf16 *__restrict__ v_store,
                                                        const __bf16 *__restrict__ k_dense, const __bf16 *__restrict__ v_dense,
                                                        int n_heads, List list, int n_new, int D, int C, long slot_stride_elems) {
  const Entry ent = list.at(blockIdx.y);
  const int slot = ent.slot, off = ent.off;
  if (slot < 0) return;
  const long new_head_stride = (long)n_new * D;
  __bf16 *slot_k = k_store + (size_t)slot * slot_stride_elems, *slot_v = v_store + (size_t)slot * slot_stride_elems;
  const __bf16 *k_new = k_dense + (size_t)blockIdx.y * n_heads * new_head_stride, *v_new = v_dense + (size_t)blockIdx.y * n_heads * new_head_stride;
  const int tile0 = off / kKvTile, n_tiles = (off + n_new + kKvTile - 1) / kKvTile - tile0;
  const long stride = (long)gridDim.x * blockDim.x;
  const long tid0 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long total_k = (long)n_heads * n_new * D;
  for (long e = tid0; e < total_k; e += stride) {
    const int dd = (int)(e % D);
    const long r = e / D;
    const int t = (int)(r % n_new), g = (int)(r / n_new);
    slot_k[((size_t)g * C + off + t) * D + dd] = k_new[(size_t)g * new_head_stride + (size_t)t * D + dd];
  }
  const long total_v = (long)n_heads * n_tiles * D * kKvTile;
  for (long e = tid0; e < total_v; e += stride) {
    const int p = (int)(e % kKvTile);  // physical position inside the block
    long r = e / kKvTile;
    const int dd = (int)(r % D);
    r /= D;
    const int tile = tile0 + (int)(r % n_tiles), g = (int)(r / n_tiles);
    const int t_abs = tile * kKvTile + (p & ~15) + pc::blocked_key(p & 15);
    if (t_abs < off) continue;  // older tokens stay
    const int t = t_abs - off;
    const __bf16 val = t < n_new ? v_new[(size_t)g * new_head_stride + (size_t)t * D + dd] : (__bf16)0.f;
    slot_v[((size_t)g * C + (size_t)tile * kKvTile) * D + (size_t)dd * kKvTile + p] = val;
  }
}

// ---------------------------------------------------------------------------------------------------
// 8-bit slots.  Layout per (slot, kv head):  K [token][head_dim] bytes;  V [token / 64][head_dim][64] bytes with
// key order pc::blocked_key8 inside a block, zero codes past the stored count;  one scale 2^e per 64-token block
// for K and one for V.  One workgroup per (chunk, kv head, 64-token block).
// ---------------------------------------------------------------------------------------------------
// 2^e with e the smallest integer such that amax <= 448 * 2^e, e kept in [-110, 127] (0 for amax == 0).
// 448 = 1.75 * 2^8: with amax = 1.f * 2^k the answer is k - 8 when 1.f <= 1.75, else k - 7.
__device__ __forceinline__ int block_exponent(float amax) {
  if (amax == 0.f) return 0;
  const unsigned bits = __float_as_uint(amax);
  const int field = (int)((bits >> 23) & 0xff);
  if (field == 0) return -110;  // below 2^-126
  const int k = field - 127;
  const int e = (bits & 0x7fffffu) <= 0x600000u ? k - 8 : k - 7;
  return e < -110 ? -110 : (e > 127 ? 127 : e);
}
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }  // e in [-126, 127]

// four E4M3 codes of four floats already divided by the scale (round to nearest even in hardware; |y| <= 448)
__device__ __forceinline__ unsigned encode4(float a, float b, float c, float d) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(a, -448.f, 448.f), __builtin_amdgcn_fmed3f(b, -448.f, 448.f), 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(c, -448.f, 448.f), __builtin_amdgcn_fmed3f(d, -448.f, 448.f), w, true);
  return (unsigned)w;
}

// Entry::off: the slot already holds that many tokens and the dense tensors are the tokens that follow them (0: a put).  The
// block that was partly filled is then quantised afresh from the values its old tokens read back as plus the new
// tokens (its exponent is recomputed over all of them; old codes are re-rounded only if the exponent moves); the
// launch covers the blocks from off / 64 on (of every entry as many as the entry with the most has).
//
// A workgroup takes one (chunk, kv head, 64-token block); half of its wavefronts K, half V, a wavefront 64 head-dim elements of
// all 64 tokens, 8 x 8 elements a lane (eight 16-byte loads in flight).  V: 8 keys of a chunk of the block rows x 8 head-dim
// elements, whose codes are turned in registers.  (Codes turned through LDS byte by byte, four loads per lane behind tests:
// 14.3 us for 8 chunks of 1000 tokens, 8 heads of 128; now 13.2 us.)
struct Store8 {
  uint8_t *k, *v;
  float *k_scale, *v_scale;
  long slot_stride, scale_stride;
};
template <int D>
__device__ __forceinline__ void quant_block(const Store8 &st, const __bf16 *__restrict__ dense_k, const __bf16 *__restrict__ dense_v, int C, const Entry &ent,
                                            int slot, int g, int head_rows) {
  constexpr int HALF = D / 64;  // wavefronts of each kind
  __shared__ float red[2 * HALF];
  uint8_t *const __restrict__ slot_k = st.k, *const __restrict__ slot_v = st.v;
  float *const __restrict__ scale_k = st.k_scale, *const __restrict__ scale_v = st.v_scale;
  const long slot_stride_elems = st.slot_stride, scale_slot_stride = st.scale_stride;
  const int off = ent.off, n_new = ent.n_tok, n_tok = off + n_new;
  const int blk = blockIdx.x + off / kKvTile, t0 = blk * kKvTile;
  if (slot < 0 || t0 >= n_tok) return;  // (the whole workgroup leaves)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hi = lane >> 3, lo = lane & 7;
  const bool is_v = wave >= HALF;
  const int d = (wave % HALF) * 64 + (is_v ? hi : lo) * 8;  // first of this lane's 8 head-dim elements
  const size_t dense_at = ((size_t)ent.row0 + (size_t)g * head_rows) * D + d;
  const size_t slot_at = (size_t)slot * slot_stride_elems + ((size_t)g * C + t0) * D;
  const size_t sc = (size_t)slot * scale_slot_stride + (size_t)g * (C / kKvTile) + blk;
  const __bf16 *src = (is_v ? dense_v : dense_k) + dense_at;
  auto token = [&](int j) __attribute__((always_inline)) { return is_v ? chunk_key<true>(lo) + in_chunk(j) : hi + 8 * j; };  // inside the block
  pc::bf16x8 x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] = *(const pc::bf16x8 *)(src + (size_t)min(max(t0 + token(j) - off, 0), n_new - 1) * D);
  uint8_t *const kc = slot_k + slot_at + d, *const vc = slot_v + slot_at + (size_t)d * kKvTile + lo * 8;
  if (t0 < off) {  // (only the first block of an append) what the stored codes read back as, exact in bf16
    const float scale = (is_v ? scale_v : scale_k)[sc];
    uint2 w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = *(const uint2 *)(is_v ? vc + j * kKvTile : kc + (size_t)token(j) * D);
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) {  // K: row j holds its 8 elements; V: row d + e holds the 8 keys
        const uint2 ww = is_v ? w[e] : w[j];
        const int at = is_v ? j : e;
        const unsigned code = (at < 4 ? ww.x : ww.y) >> (8 * (at & 3));
        const float v = __builtin_amdgcn_cvt_f32_fp8((int)code, 0) * scale;
        x[j][e] = t0 + token(j) < off ? (__bf16)v : x[j][e];
      }
  }
  float amax = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool in = t0 + token(j) < n_tok;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (!in) x[j][e] = (__bf16)0.f;  // (zero codes past the stored count)
      amax = fmaxf(amax, fabsf((float)x[j][e]));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
  if (lane == 0) red[wave] = amax;
  __syncthreads();
  amax = red[is_v ? HALF : 0];
#pragma unroll
  for (int w = 1; w < HALF; ++w) amax = fmaxf(amax, red[(is_v ? HALF : 0) + w]);
  const int ex = block_exponent(amax);
  const float inv = pow2f(-ex);
  if (lane == 0 && wave % HALF == 0) (is_v ? scale_v : scale_k)[sc] = pow2f(ex);
  uint2 c[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    c[j].x = encode4((float)x[j][0] * inv, (float)x[j][1] * inv, (float)x[j][2] * inv, (float)x[j][3] * inv);
    c[j].y = encode4((float)x[j][4] * inv, (float)x[j][5] * inv, (float)x[j][6] * inv, (float)x[j][7] * inv);
  }
  if (!is_v) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (t0 + token(j) < n_tok) *(uint2 *)(kc + (size_t)token(j) * D) = c[j];
    return;
  }
  // 8 x 8 bytes: pairs of keys first, then fours
  unsigned pr[4][4];  // [key pair][d pair]: two keys of element 2 q, two of element 2 q + 1
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      pr[p][q] = __builtin_amdgcn_perm(q < 2 ? c[2 * p + 1].x : c[2 * p + 1].y, q < 2 ? c[2 * p].x : c[2 * p].y, (q & 1) ? 0x07030602u : 0x05010400u);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const unsigned sel = (e & 1) ? 0x07060302u : 0x05040100u;
    *(uint2 *)(vc + e * kKvTile) = make_uint2(__builtin_amdgcn_perm(pr[1][e >> 1], pr[0][e >> 1], sel), __builtin_amdgcn_perm(pr[3][e >> 1], pr[2][e >> 1], sel));
  }
}

template <int D, class List>
__global__ __launch_bounds__(2 * D) void kv_quant_kernel(Store8 st, const __bf16 *__restrict__ dense_k, const __bf16 *__restrict__ dense_v, int C, List list,
                                                         int head_rows) {
  const Entry e = list.at(blockIdx.z);
  quant_block<D>(st, dense_k, dense_v, C, e, e.slot, blockIdx.y, head_rows);
}

// The values an 8-bit slot holds, as dense bf16 [kv head][token][head_dim]: code * 2^e (exact).  Work split as in
// kv_copy_kernel: 8 codes per load, the 8 x 8 piece of a V block turned in registers as bf16.
template <int D>
__device__ __forceinline__ void dequant_unit(const Store8 &st, __bf16 *__restrict__ dense_k, __bf16 *__restrict__ dense_v, int C, const Entry &e, int slot, int g,
                                             int unit, int head_rows) {
  constexpr int UNITS = 2 * (D / 64);
  const uint8_t *const __restrict__ slot_k = st.k, *const __restrict__ slot_v = st.v;
  const float *const __restrict__ scale_k = st.k_scale, *const __restrict__ scale_v = st.v_scale;
  const long slot_stride_elems = st.slot_stride, scale_slot_stride = st.scale_stride;
  const int n_tok = e.n_tok;
  const int tile = unit / UNITS, part = unit % UNITS, t0 = tile * kKvTile;
  if (slot < 0 || t0 >= n_tok) return;
  const int lane = threadIdx.x & 63, hi = lane >> 3, lo = lane & 7;
  const int d0 = (part >> 1) * 64;
  const size_t drow = (size_t)e.row0 + (size_t)g * head_rows + t0;
  const size_t sbase = (size_t)slot * slot_stride_elems + ((size_t)g * C + t0) * D;
  const float scale = (part & 1 ? scale_v : scale_k)[(size_t)slot * scale_slot_stride + (size_t)g * (C / kKvTile) + tile];
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  auto widen = [&](uint2 w) __attribute__((always_inline)) {
    pc::u32x4 o;
    o[0] = __builtin_bit_cast(unsigned, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.x, scale, false));
    o[1] = __builtin_bit_cast(unsigned, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.x, scale, true));
    o[2] = __builtin_bit_cast(unsigned, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.y, scale, false));
    o[3] = __builtin_bit_cast(unsigned, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w.y, scale, true));
    return o;
  };
  uint2 raw[8];
  if (!(part & 1)) {
    const uint8_t *src = slot_k + sbase + d0 + lo * 8;
    __bf16 *dst = dense_k + drow * D + d0 + lo * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) raw[j] = *(const uint2 *)(src + (size_t)min(hi + 8 * j, n_tok - 1 - t0) * D);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (t0 + hi + 8 * j < n_tok) *(pc::u32x4 *)(dst + (size_t)(hi + 8 * j) * D) = widen(raw[j]);
    return;
  }
  const uint8_t *block = slot_v + sbase + (size_t)(d0 + hi * 8) * kKvTile + lo * 8;
  __bf16 *rows = dense_v + drow * D + d0 + hi * 8;
  pc::u32x4 in[8], out[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) raw[j] = *(const uint2 *)(block + j * kKvTile);
#pragma unroll
  for (int j = 0; j < 8; ++j) in[j] = widen(raw[j]);
  transpose8(in, out);
  const int k0 = chunk_key<true>(lo);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int t = k0 + in_chunk(j);
    if (t0 + t < n_tok) *(pc::u32x4 *)(rows + (size_t)t * D) = out[j];
  }
}

template <int D, class List>
__global__ __launch_bounds__(256) void kv_dequant_kernel(Store8 st, __bf16 *__restrict__ dense_k, __bf16 *__restrict__ dense_v, int C, List list, int head_rows) {
  const Entry e = list.at(blockIdx.z);
  dequant_unit<D>(st, dense_k, dense_v, C, e, e.slot, blockIdx.y, blockIdx.x * 4 + (threadIdx.x >> 6), head_rows);
}

// A list that names slots of both formats (ids of the context, the 8-bit ones from n_slots16 on): a workgroup takes one 64-token tile of one head, in
// whichever format its slot has.  One launch instead of one per format, and the conversions of the 8-bit slots, which alone reach 3.5 to 4 TB/s, run
// beside the copies.  16 chunks of 1000 tokens, 8 heads of 128, half of them 8-bit, put and got: a launch a format 53.0 us, one 47.5 (4.9 TB/s read and
// written, what a large copy reaches).
template <int D, bool kToStore, class List>
__global__ __launch_bounds__(2 * D) void kv_mixed_kernel(Store16 s16, Store8 s8, int n_slots16, __bf16 *__restrict__ dense_k, __bf16 *__restrict__ dense_v, int C,
                                                         List list, int head_rows) {
  const Entry e = list.at(blockIdx.z);
  const int unit = blockIdx.x * (2 * D / 64) + (threadIdx.x >> 6);
  if (e.slot < n_slots16) copy_unit<D, kToStore>(s16, dense_k, dense_v, C, e, e.slot, blockIdx.y, unit, head_rows);
  else if (kToStore) quant_block<D>(s8, dense_k, dense_v, C, e, e.slot - n_slots16, blockIdx.y, head_rows);
  else dequant_unit<D>(s8, dense_k, dense_v, C, e, e.slot - n_slots16, blockIdx.y, unit, head_rows);
}

pc_status check_slot(percache_ctx *ctx, int32_t layer, int32_t slot) {
  if (!ctx) return PC_EINVAL;
  if (layer < 0 || layer >= ctx->cfg.n_layers) return pc::fail(ctx, PC_ESLOT, "layer %d out of range [0,%d)", layer, ctx->cfg.n_layers);
  if (slot < 0 || slot >= ctx->cfg.n_slots) return pc::fail(ctx, PC_ESLOT, "slot %d out of range [0,%d)", slot, ctx->cfg.n_slots);
  return PC_OK;
}

Store16 store16(const percache_ctx *ctx, int layer) {
  const size_t off = (size_t)layer * ctx->layer_stride;
  return {ctx->k_store + off, ctx->v_store + off, (long)ctx->slot_stride};
}
Store8 store8(const percache_ctx *ctx, int layer) {
  const size_t off = (size_t)layer * ctx->layer_stride8;
  const long sc_slot = (long)ctx->cfg.n_kv_heads * (ctx->cfg.slot_capacity / kKvTile);
  const size_t sc_off = (size_t)layer * ctx->n_slots8 * sc_slot;
  return {ctx->k8_store + off, ctx->v8_store + off, ctx->k_scale + sc_off, ctx->v_scale + sc_off, (long)ctx->slot_stride, sc_slot};
}

// Copies between dense tensors and the n slots of a list (slot ids of the context), its longest entry of `longest` tokens.
template <bool kToStore, class List>
pc_status launch_copy(percache_ctx *ctx, int layer, List &list, int n, int longest, void *k_dev, void *v_dev, int head_rows, hipStream_t stream) {
  const percache_config &c = ctx->cfg;
  __bf16 *const k = (__bf16 *)k_dev, *const v = (__bf16 *)v_dev;
  int n8 = 0;
  for (int i = 0; i < n; ++i) n8 += ctx->is8(list.at(i).slot);
  const int tiles = (longest + kKvTile - 1) / kKvTile;
  auto grid = [&](int x) { return dim3(x, c.n_kv_heads, n); };
  const bool d128 = c.head_dim == 128;
  if (n8 && n8 < n) {
    if (d128) hipLaunchKernelGGL((kv_mixed_kernel<128, kToStore, List>), grid(tiles), dim3(256), 0, stream, store16(ctx, layer), store8(ctx, layer), ctx->n_slots16, k, v, c.slot_capacity, list, head_rows);
    else hipLaunchKernelGGL((kv_mixed_kernel<64, kToStore, List>), grid(tiles), dim3(128), 0, stream, store16(ctx, layer), store8(ctx, layer), ctx->n_slots16, k, v, c.slot_capacity, list, head_rows);
  } else if (n8) {
    for (int i = 0; i < n; ++i) list.set_slot(i, list.at(i).slot - ctx->n_slots16);
    const Store8 st = store8(ctx, layer);
    if (kToStore) {
      if (d128) hipLaunchKernelGGL((kv_quant_kernel<128, List>), grid(tiles), dim3(256), 0, stream, st, k, v, c.slot_capacity, list, head_rows);
      else hipLaunchKernelGGL((kv_quant_kernel<64, List>), grid(tiles), dim3(128), 0, stream, st, k, v, c.slot_capacity, list, head_rows);
    } else {
      if (d128) hipLaunchKernelGGL((kv_dequant_kernel<128, List>), grid(tiles), dim3(256), 0, stream, st, k, v, c.slot_capacity, list, head_rows);
      else hipLaunchKernelGGL((kv_dequant_kernel<64, List>), grid((tiles + 1) / 2), dim3(256), 0, stream, st, k, v, c.slot_capacity, list, head_rows);
    }
  } else {
    const Store16 st = store16(ctx, layer);
    if (d128) hipLaunchKernelGGL((kv_copy_kernel<128, kToStore, List>), grid(tiles), dim3(256), 0, stream, st, k, v, c.slot_capacity, list, head_rows);
    else hipLaunchKernelGGL((kv_copy_kernel<64, kToStore, List>), grid((tiles + 1) / 2), dim3(256), 0, stream, st, k, v, c.slot_capacity, list, head_rows);
  }
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}
// The n chunks of a list that are tensors of their own, [n][Hkv][n_tokens][D]
template <bool kToStore>
pc_status copy_chunks(percache_ctx *ctx, int layer, const int32_t *slots, int n, int n_tokens, void *k_dev, void *v_dev, hipStream_t stream) {
  ChunkList l;
  for (int i = 0; i < n; ++i) l.slots[i] = slots[i];
  l.n_tok = n_tokens;
  l.row_step = ctx->cfg.n_kv_heads * n_tokens;
  return launch_copy<kToStore>(ctx, layer, l, n, n_tokens, k_dev, v_dev, n_tokens, stream);
}

// launch_kv_append for a list of at most N slots
template <int N>
pc_status append_list(percache_ctx *ctx, int layer, const int32_t *slot_list, int n, bool only_8bit, const __bf16 *k, const __bf16 *v, int n_tokens,
                      hipStream_t stream) {
  const percache_config &c = ctx->cfg;
  PieceList<N> l16, l8;
  int n16 = 0, n8 = 0, blocks8 = 0;
  for (int i = 0; i < n; ++i) {
    const int slot = slot_list[i], off = slot < 0 ? 0 : ctx->slot_len[(size_t)layer * c.n_slots + slot];
    const bool is8 = slot >= 0 && ctx->is8(slot), is16 = slot >= 0 && !is8 && !only_8bit;
    l8.entry[i] = {is8 ? slot - ctx->n_slots16 : -1, i * c.n_kv_heads * n_tokens, n_tokens, off};
    l16.entry[i] = {is16 ? slot : -1, 0, 0, off};
    n8 += is8;
    n16 += is16;
    const int blocks = (off + n_tokens + kKvTile - 1) / kKvTile - off / kKvTile;
    if (is8 && blocks > blocks8) blocks8 = blocks;
  }
  if (n8) {
    const dim3 grid(blocks8, c.n_kv_heads, n);
    if (c.head_dim == 128) hipLaunchKernelGGL((kv_quant_kernel<128, PieceList<N>>), grid, dim3(256), 0, stream, store8(ctx, layer), k, v, c.slot_capacity, l8, n_tokens);
    else hipLaunchKernelGGL((kv_quant_kernel<64, PieceList<N>>), grid, dim3(128), 0, stream, store8(ctx, layer), k, v, c.slot_capacity, l8, n_tokens);
    PC_HIP(ctx, hipGetLastError());
  }
  if (n16) {
    const size_t at = (size_t)layer * ctx->layer_stride;
    const long work = (long)c.n_kv_heads * c.head_dim * ((n_tokens + kKvTile - 1) / kKvTile + 1) * kKvTile;
    const long blocks = (work + 255) / 256;
    hipLaunchKernelGGL((kv_append_kernel<PieceList<N>>), dim3((unsigned)(blocks > 1024 ? 1024 : blocks), n), dim3(256), 0, stream, ctx->k_store + at,
                       ctx->v_store + at, k, v, c.n_kv_heads, l16, n_tokens, c.head_dim, c.slot_capacity, (long)ctx->slot_stride);
    PC_HIP(ctx, hipGetLastError());
  }
  return PC_OK;
}

}  // namespace

namespace pc {
pc_status launch_kv_slices(percache_ctx *ctx, int layer, const int32_t *slots, const int32_t *bounds, int n_pieces, int batch, const __bf16 *k,
                           const __bf16 *v, int seq_len, hipStream_t stream) {
  const int Hkv = ctx->cfg.n_kv_heads, D = ctx->cfg.head_dim;
  PieceList<kListMax> l;
  int n = 0, first = 0, longest = 0;   // pieces collected, query of the first one (rows are counted from it), tokens of the longest
  auto flush = [&]() {
    const size_t at = (size_t)first * Hkv * seq_len * D;
    const pc_status st = n ? launch_copy<true>(ctx, layer, l, n, longest, (void *)(k + at), (void *)(v + at), seq_len, stream) : PC_OK;
    n = longest = 0;
    return st;
  };
  for (int b = 0; b < batch; ++b)
    for (int j = 0; j < n_pieces; ++j) {
      if (slots[(size_t)b * n_pieces + j] < 0) continue;
      if (n == kListMax) {
        const pc_status st = flush();
        if (st != PC_OK) return st;
      }
      if (n == 0) first = b;
      const int tokens = bounds[j + 1] - bounds[j];
      l.entry[n++] = {slots[(size_t)b * n_pieces + j], (b - first) * Hkv * seq_len + bounds[j], tokens, 0};
      if (tokens > longest) longest = tokens;
    }
  return flush();
}
pc_status launch_kv_append(percache_ctx *ctx, int layer, const int32_t *slot_list, int n, bool only_8bit, const __bf16 *k, const __bf16 *v,
                           int n_tokens, hipStream_t stream) {
  const size_t per_slot = (size_t)ctx->cfg.n_kv_heads * n_tokens * ctx->cfg.head_dim;
  for (int i0 = 0; i0 < n; i0 += kListMax) {
    const int cnt = n - i0 < kListMax ? n - i0 : kListMax;
    const pc_status st = cnt <= 8 ? append_list<8>(ctx, layer, slot_list + i0, cnt, only_8bit, k + i0 * per_slot, v + i0 * per_slot, n_tokens, stream)
                                  : append_list<kListMax>(ctx, layer, slot_list + i0, cnt, only_8bit, k + i0 * per_slot, v + i0 * per_slot, n_tokens, stream);
    if (st != PC_OK) return st;
  }
  return PC_OK;
}
}  // namespace pc

extern "C" {

pc_status percache_kv_append(percache_ctx *ctx, int32_t layer, int32_t slot, const void *k_dev, const void *v_dev,
                             int32_t n_tokens, void *stream) {
  pc_status st = check_slot(ctx, layer, slot);
  if (st != PC_OK) return st;
  if (!k_dev || !v_dev) return pc::fail(ctx, PC_EINVAL, "k_dev / v_dev is NULL");
  if (((uintptr_t)k_dev | (uintptr_t)v_dev) % 16) return pc::fail(ctx, PC_EINVAL, "k_dev / v_dev must be 16-byte aligned");
  const percache_config &c = ctx->cfg;
  const int have = ctx->slot_len[(size_t)layer * c.n_slots + slot];
  if (n_tokens < 1 || have + n_tokens > c.slot_capacity)
    return pc::fail(ctx, PC_ELEN, "slot %d holds %d tokens: %d more do not fit the capacity %d", slot, have, n_tokens, c.slot_capacity);
  st = pc::launch_kv_append(ctx, layer, &slot, 1, false, (const __bf16 *)k_dev, (const __bf16 *)v_dev, n_tokens, (hipStream_t)stream);
  if (st != PC_OK) return st;
  ctx->slot_len[(size_t)layer * c.n_slots + slot] = have + n_tokens;
  return PC_OK;
}

pc_status percache_kv_put(percache_ctx *ctx, int32_t layer, int32_t slot, const void *k_dev, const void *v_dev,
                          int32_t n_tokens, void *stream) {
  pc_status st = check_slot(ctx, layer, slot);
  if (st != PC_OK) return st;
  if (!k_dev || !v_dev) return pc::fail(ctx, PC_EINVAL, "k_dev / v_dev is NULL");
  if (((uintptr_t)k_dev | (uintptr_t)v_dev) % 16) return pc::fail(ctx, PC_EINVAL, "k_dev / v_dev must be 16-byte aligned");
  const percache_config &c = ctx->cfg;
  if (n_tokens < 1 || n_tokens > c.slot_capacity) return pc::fail(ctx, PC_ELEN, "n_tokens %d outside [1,%d]", n_tokens, c.slot_capacity);
  st = copy_chunks<true>(ctx, layer, &slot, 1, n_tokens, (void *)k_dev, (void *)v_dev, (hipStream_t)stream);
  if (st != PC_OK) return st;
  ctx->slot_len[(size_t)layer * c.n_slots + slot] = n_tokens;
  return PC_OK;
}

pc_status percache_kv_put_batch(percache_ctx *ctx, int32_t layer, const int32_t *slots_host, int32_t n, const void *k_dev,
                                const void *v_dev, int32_t n_tokens, void *stream) {
  if (!ctx) return PC_EINVAL;
  if (!slots_host || n < 1) return pc::fail(ctx, PC_EINVAL, "slots_host is NULL or n < 1");
  if (!k_dev || !v_dev) return pc::fail(ctx, PC_EINVAL, "k_dev / v_dev is NULL");
  if (((uintptr_t)k_dev | (uintptr_t)v_dev) % 16) return pc::fail(ctx, PC_EINVAL, "k_dev / v_dev must be 16-byte aligned");
  const percache_config &c = ctx->cfg;
  if (n_tokens < 1 || n_tokens > c.slot_capacity) return pc::fail(ctx, PC_ELEN, "n_tokens %d outside [1,%d]", n_tokens, c.slot_capacity);
  for (int i = 0; i < n; ++i) {
    pc_status st = check_slot(ctx, layer, slots_host[i]);
    if (st != PC_OK) return st;
    for (int j = 0; j < i; ++j)
      if (slots_host[j] == slots_host[i]) return pc::fail(ctx, PC_EINVAL, "slot %d appears twice in the batch", slots_host[i]);
  }
  const size_t per_chunk = (size_t)c.n_kv_heads * n_tokens * c.head_dim;
  for (int i0 = 0; i0 < n; i0 += kListMax) {
    const int cnt = n - i0 < kListMax ? n - i0 : kListMax;
    pc_status st = copy_chunks<true>(ctx, layer, slots_host + i0, cnt, n_tokens, (void *)((const __bf16 *)k_dev + per_chunk * i0),
                                     (void *)((const __bf16 *)v_dev + per_chunk * i0), (hipStream_t)stream);
    if (st != PC_OK) return st;
  }
  for (int i = 0; i < n; ++i) ctx->slot_len[(size_t)layer * c.n_slots + slots_host[i]] = n_tokens;
  return PC_OK;
}

pc_status percache_kv_get(percache_ctx *ctx, int32_t layer, int32_t slot, void *k_out_dev, void *v_out_dev,
                          int32_t *n_tokens_out_host, void *stream) {
  pc_status st = check_slot(ctx, layer, slot);
  if (st != PC_OK) return st;
  if (!k_out_dev || !v_out_dev) return pc::fail(ctx, PC_EINVAL, "k_out_dev / v_out_dev is NULL");
  if (((uintptr_t)k_out_dev | (uintptr_t)v_out_dev) % 16) return pc::fail(ctx, PC_EINVAL, "outputs must be 16-byte aligned");
  const percache_config &c = ctx->cfg;
  int n_tokens = ctx->slot_len[(size_t)layer * c.n_slots + slot];
  if (n_tokens <= 0) return pc::fail(ctx, PC_ESLOT, "slot %d of layer %d is empty", slot, layer);
  st = copy_chunks<false>(ctx, layer, &slot, 1, n_tokens, k_out_dev, v_out_dev, (hipStream_t)stream);
  if (st != PC_OK) return st;
  if (n_tokens_out_host) *n_tokens_out_host = n_tokens;
  return PC_OK;
}

pc_status percache_kv_get_batch(percache_ctx *ctx, int32_t layer, const int32_t *slots_host, int32_t n, void *k_out_dev,
                                void *v_out_dev, int32_t n_tokens, void *stream) {
  if (!ctx) return PC_EINVAL;
  if (!slots_host || n < 1) return pc::fail(ctx, PC_EINVAL, "slots_host is NULL or n < 1");
  if (!k_out_dev || !v_out_dev) return pc::fail(ctx, PC_EINVAL, "k_out_dev / v_out_dev is NULL");
  if (((uintptr_t)k_out_dev | (uintptr_t)v_out_dev) % 16) return pc::fail(ctx, PC_EINVAL, "outputs must be 16-byte aligned");
  const percache_config &c = ctx->cfg;
  if (n_tokens < 1 || n_tokens > c.slot_capacity) return pc::fail(ctx, PC_ELEN, "n_tokens %d outside [1,%d]", n_tokens, c.slot_capacity);
  for (int i = 0; i < n; ++i) {
    pc_status st = check_slot(ctx, layer, slots_host[i]);
    if (st != PC_OK) return st;
    const int have = ctx->slot_len[(size_t)layer * c.n_slots + slots_host[i]];
    if (have <= 0) return pc::fail(ctx, PC_ESLOT, "slot %d of layer %d is empty", slots_host[i], layer);
    if (have < n_tokens) return pc::fail(ctx, PC_ELEN, "slot %d holds %d tokens, %d asked for", slots_host[i], have, n_tokens);
  }
  const size_t per_chunk = (size_t)c.n_kv_heads * n_tokens * c.head_dim;
  for (int i0 = 0; i0 < n; i0 += kListMax) {
    const int cnt = n - i0 < kListMax ? n - i0 : kListMax;
    pc_status st = copy_chunks<false>(ctx, layer, slots_host + i0, cnt, n_tokens, (void *)((__bf16 *)k_out_dev + per_chunk * i0),
                                      (void *)((__bf16 *)v_out_dev + per_chunk * i0), (hipStream_t)stream);
    if (st != PC_OK) return st;
  }
  return PC_OK;
}

pc_status percache_kv_evict(percache_ctx *ctx, int32_t layer, int32_t slot) {
  pc_status st = check_slot(ctx, layer, slot);
  if (st != PC_OK) return st;
  ctx->slot_len[(size_t)layer * ctx->cfg.n_slots + slot] = 0;
  return PC_OK;
}

int32_t percache_kv_len(const percache_ctx *ctx, int32_t layer, int32_t slot) {
  if (!ctx) return PC_EINVAL;
  if (layer < 0 || layer >= ctx->cfg.n_layers || slot < 0 || slot >= ctx->cfg.n_slots) return PC_ESLOT;
  return ctx->slot_len[(size_t)layer * ctx->cfg.n_slots + slot];
}

}  // extern "C"
