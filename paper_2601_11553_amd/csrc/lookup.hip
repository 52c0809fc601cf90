// Query-level match (Sec. 4.2.1): cosine top-1 of probe embeddings against every row of the QA bank's
// embedding matrix, and the hit flag against tau_query.
//
// The bank is streamed from HBM exactly once per pass of up to 32 probes.  The dot products run on the
// fp16 matrix cores (16x16x32, fp32 accumulate) only because they perform the cross-lane reduction for
// free; the kernel is bound by the HBM stream of the bank, not by arithmetic.
#include <atomic>
#include <chrono>
#include <climits>
#include <cmath>

#include "gemm_tile.hpp"

namespace {
using pc::f16x8;
using pc::f32x4;
using pc::u32x4;

struct Best {
  float s;
  int idx;
};
__device__ __forceinline__ bool better(float s1, int i1, float s2, int i2) { return s1 > s2 || (s1 == s2 && i1 < i2); }

// Sorted list of the K best (similarity, row) pairs, best first; ties go to the lower row.
template <int K>
struct TopK {
  float s[K];
  int i[K];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int j = 0; j < K; ++j) { s[j] = -INFINITY; i[j] = INT_MAX; }
  }
  __device__ __forceinline__ void insert(float cs, int ci) {
    if (!better(cs, ci, s[K - 1], i[K - 1])) return;
    s[K - 1] = cs;
    i[K - 1] = ci;
#pragma unroll
    for (int j = K - 1; j > 0; --j) {
      const bool up = better(s[j], i[j], s[j - 1], i[j - 1]);
      const float ts = s[j]; const int ti = i[j];
      s[j] = up ? s[j - 1] : ts;   i[j] = up ? i[j - 1] : ti;
      s[j - 1] = up ? ts : s[j - 1]; i[j - 1] = up ? ti : i[j - 1];
    }
  }
  // drops the head if this list owns it
  __device__ __forceinline__ void pop_if(bool mine) {
#pragma unroll
    for (int j = 0; j < K - 1; ++j) { s[j] = mine ? s[j + 1] : s[j]; i[j] = mine ? i[j + 1] : i[j]; }
    s[K - 1] = mine ? -INFINITY : s[K - 1];
    i[K - 1] = mine ? INT_MAX : i[K - 1];
  }
};

// ---------------------------------------------------------------------------------------------------
// Inverse L2 norms of newly written bank rows; one wavefront per row.  Also copies the rows into the
// bank when the source is elsewhere.
// ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void bank_put_kernel(const _Float16 *__restrict__ src, _Float16 *__restrict__ dst,
                                                       float *__restrict__ inv_norm, int n, int d) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  const u32x4 *s = (const u32x4 *)(src + (size_t)row * d);
  u32x4 *t = (u32x4 *)(dst + (size_t)row * d);
  float ss = 0.f;
  for (int v = lane; v < d / 8; v += 64) {
    u32x4 raw = s[v];
    t[v] = raw;
    f16x8 h = __builtin_bit_cast(f16x8, raw);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += (float)h[e] * (float)h[e];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if (lane == 0) inv_norm[row] = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
}

// ---------------------------------------------------------------------------------------------------
// Streaming pass.  Workgroup = 4 wavefronts; workgroup b owns a contiguous range of 16-row blocks (at most
// kMaxBlocksPerWg), its wavefronts take them round-robin.  Each wavefront streams its row blocks through a
// PRIVATE ring of LDS stages with direct global->LDS loads: one stage holds 16 rows x CHB bytes (a chunk of
// CHB/2 elements per row), one load instruction brings 1 KB that is contiguous in memory (whole 128-byte
// lines, requested once), and NSTG-1 chunks are always in flight per wavefront.  No workgroup barrier is
// needed in the loop: a ring is written and read by one wavefront only.  The 16-byte chunks of a row are
// XOR-swizzled inside the stage so that the MFMA operand reads (lane (r = lane%16, g = lane/16) reads
// elements [32 step + 8 g, +8) of row r) are bank-conflict free.  The probes of the pass (NPB blocks of 16,
// zero padded) and the inverse norms of the workgroup's rows sit in LDS too.
// Result lane layout of the 16x16 product: lane holds probe (lane%16), rows 4*(lane/16) + 0..3.
// ---------------------------------------------------------------------------------------------------
// cache policy of the bank stream (aux operand of the global->LDS load): 2 = non-temporal, the rows are used once
constexpr int kBankLoadAux = 2;
constexpr int kProbePad = 32;  // bytes added to every probe row in LDS (measured: 16 leaves 4 conflict cycles per operand read, 32 none)
constexpr int kMaxBlocksPerWg = 128;  // 2048 rows: bounds the LDS copy of the inverse norms (8 KB)
#define PC_LOOKUP_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xf) | (7 << 4) | (15 << 8) | ((((n) >> 4) & 3) << 14))

// LDS stores that the compiler does not see: in front of an ordinary one it waits for every direct load to LDS that is on its way.
__device__ __forceinline__ unsigned lds_addr(const void *p) { return (unsigned)(size_t)(__attribute__((address_space(3))) const char *)(const char *)p; }
__device__ __forceinline__ void lds_put(const void *p, u32x4 v) { asm volatile("ds_write_b128 %0, %1" : : "v"(lds_addr(p)), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_put(const void *p, float v) { asm volatile("ds_write_b32 %0, %1" : : "v"(lds_addr(p)), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_barrier() {   // (not __syncthreads, which waits for these loads too)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The value of lane ^ 1 and lane ^ 2; of the mirrored lane of eight and of sixteen, which stands for the other quad and the other eight lanes where the
// lanes of a quad (of eight) agree.  Register moves: a shuffle goes through LDS.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true)); }
__device__ __forceinline__ float lane_xor1(float v) { return dpp<0xb1>(v); }              // quad_perm [1,0,3,2]
__device__ __forceinline__ float lane_xor2(float v) { return dpp<0x4e>(v); }              // quad_perm [2,3,0,1]
__device__ __forceinline__ float lane_other_quad(float v) { return dpp<0x141>(v); }       // row_half_mirror
__device__ __forceinline__ float lane_other_eight(float v) { return dpp<0x140>(v); }      // row_mirror

template <int CHB>
__device__ __forceinline__ int row_swz(int row) { return CHB >= 256 ? (row & 15) : ((row >> 1) & 7); }

// The merge of the workgroups' lists inside the launch that makes them (null marks: by lookup_finalize_kernel).  Every workgroup stores its
// lists straight to memory (device scope), then a mark, a number that no other call uses, and then looks at the marks of all: who finds them
// all there merges.  Nobody waits for another workgroup, so it does not matter in which order they were started.  The workgroup whose mark
// is the last one to reach memory finds all of them (it looks behind its own store); others that arrive with it may too, and write the same
// values.
constexpr int kInLaunchGrid = 64;   // (one lane looks at one mark)
struct InLaunch {
  unsigned long long *marks;   // [workgroups, at most kInLaunchGrid], whatever they hold
  unsigned long long mark;
  float tau;
  int k;
  int32_t *idx_out;
  float *sim_out;
  uint8_t *hit_out;
};

// Merge of the per-lane lists of one workgroup: the four lanes that share a probe (K rounds of "best head wins and
// is popped"), then the four wavefronts through LDS; the workgroup's lists go to partial[blockIdx.x][NPB*16][KL].
template <int NPB, int KL>
__device__ __forceinline__ void merge_workgroup_lists(TopK<KL> (&best)[NPB], char *smem, Best *__restrict__ partial, bool in_launch = false) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  __syncthreads();  // probes no longer needed: reuse LDS for the cross-wave step
  Best *red = (Best *)smem;  // [4 waves][NPB*16][KL]
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
#pragma unroll
    for (int j = 0; j < KL; ++j) {
      float s = best[pb].s[0];
      int i = best[pb].i[0];
#pragma unroll
      for (int o = 16; o < 64; o <<= 1) {
        float s2 = __shfl_xor(s, o, 64);
        int i2 = __shfl_xor(i, o, 64);
        if (better(s2, i2, s, i)) { s = s2; i = i2; }
      }
      best[pb].pop_if(i != INT_MAX && best[pb].i[0] == i);  // rows are unique: at most one lane owns the winner
      if (g == 0) red[(wave * (NPB * 16) + pb * 16 + r16) * KL + j] = Best{s, i};
    }
  }
  __syncthreads();
  if (tid < NPB * 16) {
    int head[4] = {0, 0, 0, 0};
    for (int j = 0; j < KL; ++j) {
      Best b = Best{-INFINITY, INT_MAX};
      int from = -1;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (head[w] >= KL) continue;
        Best o = red[(w * (NPB * 16) + tid) * KL + head[w]];
        if (o.idx != INT_MAX && better(o.s, o.idx, b.s, b.idx)) { b = o; from = w; }
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) head[w] += (w == from);
      Best *to = partial + ((size_t)blockIdx.x * (NPB * 16) + tid) * KL + j;
      if (in_launch) __hip_atomic_store((unsigned long long *)to, __builtin_bit_cast(unsigned long long, b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else *to = b;
    }
  }
}

// See InLaunch; a wavefront a probe, the sum of whose squares it brings.
template <int K>
__device__ __forceinline__ void merge_in_launch(const InLaunch &f, char *smem, const Best *partial, int stride, int n_probes, float tot) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = gridDim.x;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the lists are in memory
  __syncthreads();
  if (wave == 0) {
    if (lane == 0) __hip_atomic_store(f.marks + blockIdx.x, f.mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this one's mark too, before it looks
    const unsigned long long seen = lane < n ? __hip_atomic_load(f.marks + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : f.mark;
    if (lane == 0) *(int *)smem = 0;
    if (__ballot(seen != f.mark) == 0 && lane == 0) *(int *)smem = 1;
  }
  __syncthreads();
  if (!*(const int *)smem) return;
  const int p = wave;   // (at most kInLaunchProbes)
  if (p < n_probes) {
    TopK<K> mine;
    mine.clear();
    for (int w = lane; w < n; w += 64) {
      const unsigned long long *lst = (const unsigned long long *)(partial + ((size_t)w * stride + p) * K);
      Best b[K];
#pragma unroll
      for (int j = 0; j < K; ++j) b[j] = __builtin_bit_cast(Best, __hip_atomic_load(lst + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if (w == lane) {   // (the first list as it stands: it is sorted)
          mine.s[j] = b[j].idx != INT_MAX ? b[j].s : -INFINITY;
          mine.i[j] = b[j].idx;
        } else if (b[j].idx != INT_MAX) {
          mine.insert(b[j].s, b[j].idx);
        }
      }
    }
    const float inv = tot > 0.f ? 1.0f / sqrtf(tot) : 0.f;
    for (int j = 0; j < f.k; ++j) {
      float s = mine.s[0];
      int i = mine.i[0];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const float s2 = __shfl_xor(s, o, 64);
        const int i2 = __shfl_xor(i, o, 64);
        if (better(s2, i2, s, i)) { s = s2; i = i2; }
      }
      mine.pop_if(i != INT_MAX && mine.i[0] == i);
      if (lane == 0) {
        const float sim = i == INT_MAX ? -INFINITY : s * inv;
        f.idx_out[(size_t)p * f.k + j] = i == INT_MAX ? -1 : i;
        f.sim_out[(size_t)p * f.k + j] = sim;
        if (f.hit_out && j == 0) f.hit_out[p] = sim > f.tau ? 1 : 0;
      }
    }
  }
}

// Arguments of the per-row mode (K == 0): instead of the best rows per probe, the best PROBE per bank row is
// written (cache refresh, Sec. 4.1.3: does any new chunk enter a stored query's top-k?).
struct RowScan {
  const float *kth;        // [N] similarity a new chunk must exceed for row j (the row's current k-th best)
  float *best_sim;         // [N] out: best similarity over all new chunks so far
  int32_t *best_new;       // [N] out: index of that chunk, -1 while none has a similarity that is a number
  uint8_t *stale;          // [N] out: best_sim > kth
  int p0;                  // index of this pass's first probe
  int first;               // 1: first pass (outputs are overwritten), 0: merged with the previous passes
};

// The k best rows of a probe (k > 1) lie in the k groups of rows whose best rows are the best (of equal ones, the lower row's).  So a pass over the
// bank with K == kGroups writes for every group its best row and how good the second one is, and topk_groups_kernel picks k groups; only where
// one of these may hold two of the k rows does it look at rows again.  Sorted lists of eight in every lane, which this replaces, cost ten
// instructions an entry for nearly every row, because one of a wavefront's 64 lists takes nearly every row in.
// us a call, 8 best, lists | groups (3 best in brackets): 8 probes, 50 000 rows of width 1024 33.0 | 25.6 (25.9 | 25.3), 200 000 rows 78.9 | 71.6 (71.2 | 71.0),
// 32 probes 88.9 | 76.6; 64 probes 179 | 78 (175 | 77), 1024 probes 712 | 437 (708 | 432).
// Over a few thousand rows every row is a group (see groups_of).
// A group is what one lane or two meet in a stretch of the bank; which rows these are only Groups::first_row knows.  A workgroup has about four a
// wavefront: under many probes their bytes count, but over a small bank two of the k best rows would often share a large one.
constexpr int kGroups = -1, kRows = -2;   // (kRows: every row is a group)
struct Group {
  float best, second;   // without the probe's norm; best: a NaN where no row has a similarity that is a number
  int row, unused;
};
struct Groups {
  enum Kind { stream, wide, big, big_fine, rows };   // (rows: every row a group)
  Group *g;      // [probes][pitch] (rows: the similarities alone, four to a Group's place; a last place's rest is not a number)
  int n;         // of a probe
  int pitch;     // an odd number of 128-byte lines: 32 probes' groups go to as many places
  int p0;        // this pass's first probe
  int kind;
  int stretch;   // blocks (tiles) of a group
  int per;       // groups of a wavefront (workgroup)
  int per_wg;    // blocks of a workgroup; big: workgroups
  int blocks;    // (tiles) of the bank
  int sets;      // wide: sets of 32 rows in a block, a group of its own each

  __device__ float *of_rows(int p) const { return (float *)(g + (size_t)p * pitch); }
  __host__ Groups from_probe(int p) const {
    Groups o = *this;
    o.p0 += p;
    return o;
  }
  // A group's rows in jobs of 16 (stream) or 32 consecutive ones: how many jobs, the first row of one (negative: none), and whether row i of it counts.
  __host__ __device__ int jobs() const { return kind == big ? 2 * stretch : kind == big_fine ? 1 : stretch; }
  __host__ __device__ int first_row(int group, int job) const {
    if (kind == big_fine) return (group >> 1) * 32;
    const int j = group % per, w = group / per;   // of wavefront (workgroup) w
    if (kind == stream) {
      const int block = w % 4 + 4 * (j * stretch + job);
      return block < per_wg && w / 4 * per_wg + block < blocks ? (w / 4 * per_wg + block) * 16 : -1;
    }
    if (kind == wide) {
      const int block = j * stretch + job;
      return block < per_wg && w / sets * per_wg + block < blocks ? ((w / sets * per_wg + block) * sets + w % sets) * 32 : -1;
    }
    const int tile = big_begin(w / 4) + j * stretch + job / 2;
    return tile < big_begin(w / 4 + 1) ? tile * 256 + w % 4 * 64 + job % 2 * 32 : -1;
  }
  __host__ __device__ bool counts(int group, int i) const { return kind == big_fine ? (i >> 2 & 1) == (group & 1) : true; }
  __host__ __device__ int big_begin(int wg) const { return (int)((long)wg * blocks / per_wg); }   // a workgroup's first tile
};
// The best and the second best of numbers offered in the order of their rows.
struct Top2 {
  float m = -INFINITY, s = -INFINITY;
  int i = INT_MAX;
  __device__ __forceinline__ void add(float v, int row) {   // (a NaN changes nothing, and -infinity not i: see first)
    i = v > m ? row : i;
    s = __builtin_amdgcn_fmed3f(m, s, v);
    m = fmaxf(m, v);
  }
  __device__ __forceinline__ void first(float v, int row) { i = v == v && row < i ? row : i; }   // (where no number is above -infinity)
  __device__ __forceinline__ void merge(const Top2 &o) {
    s = fmaxf(fmaxf(s, o.s), fminf(m, o.m));
    if (better(o.m, o.i, m, i)) { m = o.m; i = o.i; }
  }
  __device__ __forceinline__ Top2 of_lane_xor(int o) const {
    Top2 t;
    t.m = __shfl_xor(m, o, 64);
    t.s = __shfl_xor(s, o, 64);
    t.i = __shfl_xor(i, o, 64);
    return t;
  }
};
__device__ __forceinline__ void write_group(Group *to, const Top2 &t) {   // (a second of +infinity: its rows are looked at again)
  *(f32x4 *)to = f32x4{t.i == INT_MAX ? __builtin_nanf("") : t.m, t.m == -INFINITY ? INFINITY : t.s, __int_as_float(t.i), 0.f};
}

template <int NPB, int CHB, int NSTG, int K>
__global__ __launch_bounds__(256) void lookup_stream_kernel(const _Float16 *__restrict__ bank,
                                                            const float *__restrict__ inv_norm, int N, int d,
                                                            const _Float16 *__restrict__ probes, int n_probes,
                                                            int per_wg, int ring_off, Best *__restrict__ partial, RowScan rs, InLaunch in_launch, Groups gm) {
  extern __shared__ __align__(16) char smem[];
  constexpr int CS = CHB / 64;           // MFMA k-steps (32 elements) per chunk
  constexpr int STG = 16 * CHB;          // bytes per stage
  constexpr int IPS = STG / 1024;        // load instructions per stage
  constexpr int LPR = CHB / 16;          // lanes (16-byte chunks) per row
  constexpr int AHEAD = NSTG - 1;
  // probe rows in LDS are padded by kProbePad = 32 bytes (a row is a multiple of 128 bytes): lane (probe r16, k-group g)
  // then reads at (32 r16 + 16 g) modulo 256.  With 16 bytes of padding -- 16 (r16 + g) modulo 256 -- the counters showed
  // four bank-conflict cycles per operand read, with 32 none
  const int row_bytes = d * 2 + kProbePad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, g = lane >> 4;

  const int n_blocks = (N + 15) / 16;
  const int rb_begin = blockIdx.x * per_wg;
  const int rb_end = min(n_blocks, rb_begin + per_wg);

  const int chunks = d * 2 / CHB;
  char *ring = smem + ring_off + wave * (NSTG * STG);
  // load instruction i of a stage: lane lands at stage byte 1024 i + 16 lane = (row, physical chunk)
  int ld_row[IPS], ld_col[IPS];
#pragma unroll
  for (int i = 0; i < IPS; ++i) {
    const int row = i * (1024 / CHB) + lane / LPR, pc = lane % LPR;
    ld_row[i] = row;
    ld_col[i] = (pc ^ row_swz<CHB>(row)) * 8;  // element offset of the logical chunk inside the row's chunk
  }
  auto issue = [&](int rb, int chunk, int st) __attribute__((always_inline)) {
    const _Float16 *base = bank + chunk * (CHB / 2);
#pragma unroll
    for (int i = 0; i < IPS; ++i) {
      const int row = min(rb * 16 + ld_row[i], N - 1);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(base + (size_t)row * d + ld_col[i]),
                                       (__attribute__((address_space(3))) void *)(ring + st * STG + i * 1024), 16, 0, kBankLoadAux);
    }
  };
  auto advance = [&](int &rb_, int &c_) __attribute__((always_inline)) {
    if (++c_ == chunks) { c_ = 0; rb_ += 4; }
  };
  // flat pipeline over this wavefront's (row block, chunk) items.  Loads are issued unconditionally (past the
  // end they re-read the last block into a stage nobody will read), so exactly AHEAD items are outstanding
  // behind the one about to be multiplied and a partial vmcnt wait is exact.
  int rb = rb_begin + wave, c = 0, prb = rb, pch = 0, ist = 0;
  const int rb_last = rb_end - 1;

  // Probes (zero rows beyond n_probes) and this workgroup's inverse norms (zero beyond N) to LDS, eight loads a thread at a time; the ring's first
  // stages are asked for behind the last of these loads, in front of the wait for them: one memory latency, not three.  us a call, one after the
  // other | like this: best of 200 000 rows of width 1024, 16 probes 67.1 | 65.2, of 50 000 22.3 | 21.4, 32 probes of 200 000 of width 384 32.5 | 30.3.
  const int vec_per_row = d / 8, n_vec = n_probes * vec_per_row;
  float *inv_lds = (float *)(smem + (size_t)NPB * 16 * row_bytes);
  float row_inv[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) row_inv[e] = inv_norm[min(rb_begin * 16 + e * 256 + tid, N - 1)];
  u32x4 val[8];
  auto fetch = [&](int v0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) val[i] = ((const u32x4 *)probes)[min(v0 + i * 256 + tid, n_vec - 1)];
  };
  auto keep = [&](int v0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int v = v0 + i * 256 + tid, p = v / vec_per_row, c = v - p * vec_per_row;
      if (p < NPB * 16) lds_put(smem + (size_t)p * row_bytes + c * 16, p < n_probes ? val[i] : u32x4{0, 0, 0, 0});
    }
  };
  int v0 = 0;
  for (; v0 + 2048 < NPB * 16 * vec_per_row; v0 += 2048) {
    fetch(v0);
    keep(v0);
  }
  fetch(v0);
  __builtin_amdgcn_sched_barrier(0);   // (in this order: the wait for these leaves the ring's loads alone)
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) {   // (also without a block of its own: rows of the bank that nobody reads)
    issue(min(prb, rb_last), pch, ist);
    advance(prb, pch);
    ist = ist + 1 == NSTG ? 0 : ist + 1;
  }
  __builtin_amdgcn_sched_barrier(0);
  PC_LOOKUP_WAIT_VMCNT(AHEAD * IPS);   // (left to itself the compiler waits for the ring as well)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = e * 256 + tid;
    if (r < per_wg * 16) lds_put(inv_lds + r, rb_begin * 16 + r < N ? row_inv[e] : 0.f);
  }
  keep(v0);
  for (int r = 1024 + tid; r < per_wg * 16; r += 256) {
    const int row = rb_begin * 16 + r;
    lds_put(inv_lds + r, row < N ? inv_norm[row] : 0.f);
  }
  lds_barrier();

  constexpr int KL = K > 0 ? K : 1;
  TopK<KL> best[NPB];  // this lane's best rows for probe pb*16 + r16 (K > 0)
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) best[pb].clear();
  // sum of squares of the probe that this wavefront merges (see InLaunch), in the order of inverse_norm
  constexpr bool CAN_MERGE = NPB == 1 && K > 0 && K <= 4;
  float merge_sum = 0.f;
  if (CAN_MERGE && in_launch.marks) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float ss = 0.f;
      for (int v = q * 64 + lane; v < vec_per_row; v += 256) {
        const f16x8 h = *(const f16x8 *)(smem + (size_t)wave * row_bytes + v * 16);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += (float)h[e] * (float)h[e];
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
      merge_sum += ss;
    }
  }
  // per-row mode: the product is taken the other way round (probes on the M side), so a lane holds ONE row (r16) and
  // the probes pb*16 + 4g + 0..3; their inverse norms (a padding probe's is a NaN, which no comparison picks), added up from LDS while the ring's
  // first stages are on their way; the norms go to the rows' padding.  A probe's squares are sixteen sums, of every sixteenth 16 bytes, in a
  // pass of 32 (eight lanes of two sums) as in one of 16 (sixteen lanes): equal embeddings of a call have equal norms whichever pass they are in.
  float pinv[NPB][4];
  if constexpr (K == 0) {
    constexpr int LP = 16 / NPB;
    const int p = tid / LP;
    float ss[NPB] = {};
    for (int v0 = tid % LP; v0 < vec_per_row; v0 += 16) {
#pragma unroll
      for (int j = 0; j < NPB; ++j) {
        const int v = v0 + j * LP;
        if (j > 0 && v >= vec_per_row) continue;   // (rows are whole multiples of 128 bytes)
        const f16x8 h = *(const f16x8 *)(smem + (size_t)p * row_bytes + v * 16);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss[j] += (float)h[e] * (float)h[e];
      }
    }
#pragma unroll
    for (int j = 0; j < NPB; ++j) {
      ss[j] += lane_xor1(ss[j]);
      ss[j] += lane_xor2(ss[j]);
      ss[j] += lane_other_quad(ss[j]);
    }
    const float tot = NPB == 1 ? ss[0] + lane_other_eight(ss[0]) : ss[0] + ss[NPB - 1];
    if (tid % LP == 0) lds_put(smem + (size_t)p * row_bytes + d * 2, p >= n_probes ? __builtin_nanf("") : tot > 0.f ? 1.0f / sqrtf(tot) : 0.f);
    lds_barrier();
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
      for (int e = 0; e < 4; ++e) pinv[pb][e] = *(const float *)(smem + (size_t)(pb * 16 + g * 4 + e) * row_bytes + d * 2);
  }

  // swizzled byte offsets of this lane's operand reads inside a stage
  int rd_off[CS];
#pragma unroll
  for (int s = 0; s < CS; ++s) rd_off[s] = r16 * CHB + (((4 * s + g) ^ row_swz<CHB>(r16)) * 16);

  Top2 top[NPB];   // (K == kGroups) of the group that this wavefront is in
  f32x4 acc[NPB];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) acc[pb] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto compute = [&](int chunk, int st) __attribute__((always_inline)) {
    const char *pbase = smem + (size_t)r16 * row_bytes + (chunk * (CHB / 2) + g * 8) * 2;
    const char *abase = ring + st * STG;
#pragma unroll
    for (int s = 0; s < CS; ++s) {
      f16x8 av = *(const f16x8 *)(abase + rd_off[s]);
#pragma unroll
      for (int pb = 0; pb < NPB; ++pb) {
        f16x8 bv = *(const f16x8 *)(pbase + (size_t)pb * 16 * row_bytes + s * 64);
        // (both operands have the same lane layout -- index lane%16, elements 8*(lane/16).. -- so swapping them
        // transposes the result: lane holds row r16 and probes 4g + 0..3)
        acc[pb] = K == 0 ? __builtin_amdgcn_mfma_f32_16x16x32_f16(bv, av, acc[pb], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, acc[pb], 0, 0, 0);
      }
    }
  };
  // scale by the rows' inverse norms and keep the running best list (the lowest row wins ties)
  auto epilogue = [&](int rb) __attribute__((always_inline)) {
    if (K > 0) {
      const f32x4 inv4 = *(const f32x4 *)(inv_lds + (rb - rb_begin) * 16 + g * 4);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = rb * 16 + g * 4 + r;
        const bool ok = row < N;
#pragma unroll
        for (int pb = 0; pb < NPB; ++pb) {
          const float s = acc[pb][r] * inv4[r];
          if (ok) best[pb].insert(s, row);
        }
      }
    } else if (K == kRows) {
      const f32x4 inv4 = *(const f32x4 *)(inv_lds + (rb - rb_begin) * 16 + g * 4);
      const int row0 = rb * 16 + g * 4;
#pragma unroll
      for (int pb = 0; pb < NPB; ++pb) {
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = row0 + r < N ? acc[pb][r] * inv4[r] : __builtin_nanf("");
        if (pb * 16 + r16 < n_probes && row0 < N) *(f32x4 *)(gm.of_rows(gm.p0 + pb * 16 + r16) + row0) = v;
      }
    } else if (K == kGroups) {
      // this lane's four rows of the block per probe; at the end of a stretch the four lanes of the probe
      const f32x4 inv4 = *(const f32x4 *)(inv_lds + (rb - rb_begin) * 16 + g * 4);
      const int nth = (rb - rb_begin) >> 2;   // of this wavefront's blocks
      const bool ends = (nth + 1) % gm.stretch == 0 || rb + 4 >= rb_end;
#pragma unroll
      for (int pb = 0; pb < NPB; ++pb) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = rb * 16 + g * 4 + r;
          v[r] = row < N ? acc[pb][r] * inv4[r] : __builtin_nanf("");
          top[pb].add(v[r], row);
        }
        if (__ballot(top[pb].i == INT_MAX)) {
          if (top[pb].i == INT_MAX)
#pragma unroll
            for (int r = 0; r < 4; ++r) top[pb].first(v[r], rb * 16 + g * 4 + r);
        }
        if (ends) {
          Top2 t = top[pb];
          t.merge(t.of_lane_xor(16));
          t.merge(t.of_lane_xor(32));
          if (g == 0 && pb * 16 + r16 < n_probes)
            write_group(gm.g + (size_t)(gm.p0 + pb * 16 + r16) * gm.pitch + (blockIdx.x * 4 + wave) * gm.per + nth / gm.stretch, t);
          top[pb] = Top2{};
        }
      }
    } else {
      // best probe of row r16: this lane's probes first (ascending, so the lowest wins ties), then the four lanes
      // that hold the row
      const int row = rb * 16 + r16;
      const float inv = inv_lds[(rb - rb_begin) * 16 + r16];
      float s = -INFINITY;
      int pi = INT_MAX;
#pragma unroll
      for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float c = acc[pb][e] * inv * pinv[pb][e];
          const int p = rs.p0 + pb * 16 + g * 4 + e;
          if (better(c, p, s, pi)) { s = c; pi = p; }
        }
#pragma unroll
      for (int o = 16; o < 64; o <<= 1) {
        const float s2 = __shfl_xor(s, o, 64);
        const int p2 = __shfl_xor(pi, o, 64);
        if (better(s2, p2, s, pi)) { s = s2; pi = p2; }
      }
      if (row < N && g == 0) {
        if (!rs.first && !better(s, pi, rs.best_sim[row], rs.best_new[row])) { s = rs.best_sim[row]; pi = rs.best_new[row]; }
        rs.best_sim[row] = s;
        rs.best_new[row] = pi == INT_MAX ? -1 : pi;
        rs.stale[row] = s > rs.kth[row] ? 1 : 0;
      }
    }
  };
  if (rb < rb_end) {
    int st = 0;
    clear();
    while (true) {
      issue(min(prb, rb_last), pch, ist);  // overwrites the stage multiplied in the previous iteration
      advance(prb, pch);
      ist = ist + 1 == NSTG ? 0 : ist + 1;
      PC_LOOKUP_WAIT_VMCNT(AHEAD * IPS);
      asm volatile("" ::: "memory");
      compute(c, st);
      if (c == chunks - 1) { epilogue(rb); clear(); }
      advance(rb, c);
      st = st + 1 == NSTG ? 0 : st + 1;
      if (rb >= rb_end) break;
    }
  }
  PC_LOOKUP_WAIT_VMCNT(0);

  if (K == kGroups) {   // groups that this wavefront has no rows for
    const int mine = rb_end > rb_begin + wave ? (rb_end - rb_begin - wave + 3) / 4 : 0;
    for (int j = (mine + gm.stretch - 1) / gm.stretch; j < gm.per; ++j)
      if (lane < n_probes && lane < NPB * 16) write_group(gm.g + (size_t)(gm.p0 + lane) * gm.pitch + (blockIdx.x * 4 + wave) * gm.per + j, Top2{});
  }
  if (K <= 0) return;  // per-row mode and groups: everything has been written
  merge_workgroup_lists<NPB, KL>(best, smem, partial, CAN_MERGE && in_launch.marks);
  if constexpr (CAN_MERGE) {
    if (in_launch.marks) merge_in_launch<KL>(in_launch, smem, partial, NPB * 16, n_probes, merge_sum);
  }
}

// The inverse norm of a probe, by the first 256 threads of a workgroup: a thread's share of the squares, to be asked for before other loads are
// waited for, then their sum (part [4] in LDS; one barrier).
__device__ __forceinline__ float probe_squares(const _Float16 *__restrict__ probe, int d, int tid) {
  float ss = 0.f;
  if (tid < 256)
    for (int v = tid; v < d / 8; v += 256) {
      const f16x8 h = __builtin_bit_cast(f16x8, ((const u32x4 *)probe)[v]);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss += (float)h[e] * (float)h[e];
    }
  return ss;
}
__device__ __forceinline__ float inverse_norm(float ss, int tid, float *part) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if (tid < 256 && (tid & 63) == 0) part[tid >> 6] = ss;
  __syncthreads();
  const float tot = ((part[0] + part[1]) + part[2]) + part[3];
  return tot > 0.f ? 1.0f / sqrtf(tot) : 0.f;
}

// ---------------------------------------------------------------------------------------------------
// Per probe: the best of the workgroups' best rows, divided by the probe's norm and compared with tau.  One workgroup
// of four wavefronts per probe.
// ---------------------------------------------------------------------------------------------------
constexpr int kFinalizeThreads = 256;
__global__ __launch_bounds__(kFinalizeThreads) void lookup_finalize_kernel(const Best *__restrict__ partial, int n_partials, int partial_stride,
                                                                           const _Float16 *__restrict__ probes, int d, float tau, int32_t *__restrict__ idx_out,
                                                                           float *__restrict__ sim_out, uint8_t *__restrict__ hit_out) {
  constexpr int NWV = kFinalizeThreads / 64;
  __shared__ float norm_part[NWV];
  __shared__ Best red[NWV];
  const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  Best b{-INFINITY, INT_MAX};
  // (the first list's row is on its way while the probe's squares are)
  Best first = b;
  if (tid < n_partials) first = partial[(size_t)tid * partial_stride + p];
  const float ss = probe_squares(probes + (size_t)p * d, d, tid);
  if (first.idx != INT_MAX && better(first.s, first.idx, b.s, b.idx)) b = first;
  for (int w = tid + kFinalizeThreads; w < n_partials; w += kFinalizeThreads) {
    const Best o = partial[(size_t)w * partial_stride + p];
    if (o.idx != INT_MAX && better(o.s, o.idx, b.s, b.idx)) b = o;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const Best c{__shfl_xor(b.s, o, 64), __shfl_xor(b.idx, o, 64)};
    if (better(c.s, c.idx, b.s, b.idx)) b = c;
  }
  if (lane == 0) red[wave] = b;
  const float inv = inverse_norm(ss, tid, norm_part);
  if (tid != 0) return;
#pragma unroll
  for (int w = 1; w < NWV; ++w)
    if (better(red[w].s, red[w].idx, b.s, b.idx)) b = red[w];
  const float sim = b.idx == INT_MAX ? -INFINITY : b.s * inv;
  idx_out[p] = b.idx == INT_MAX ? -1 : b.idx;
  sim_out[p] = sim;
  hit_out[p] = sim > tau ? 1 : 0;
}

// ---------------------------------------------------------------------------------------------------
// The k best rows of a probe out of its groups (see Group); one workgroup of eight wavefronts per probe.  The groups are dealt to 64 bins; the
// k-th best bin's largest value is a bound that k groups reach, and usually hardly any more: these few are compared with each other.  Where
// the second row of none of the k best groups comes near, their best rows are the answer.  Otherwise the rows of the groups in question are
// multiplied by the probe again, with the product and the order of the pass, so that every sum comes out as it did there.
// What bounds it is latency: of the load of the groups and of five steps that meet at a barrier.
// A call of 8 probes over 50 000 rows of width 1024 takes 3.5 us more than one for the best row; where a probe is in doubt, 4 to 10 us more.
// ---------------------------------------------------------------------------------------------------
constexpr int kMaxTopK = 8;
constexpr int kSelectThreads = 512, kSelectHeld = 8, kCandidates = 1024;
constexpr int kRowsUpTo = 8192;   // rows of the bank that may be groups of their own
// similarities as numbers that rise with them; 0: not a number
__device__ __forceinline__ unsigned ordered(float v) {
  const unsigned u = __float_as_uint(v + 0.f);   // (-0 becomes 0)
  return v != v ? 0u : u & 0x80000000u ? ~u : u | 0x80000000u;
}
// a similarity and its row in one number: the larger similarity is larger, and the lower row among equals
__device__ __forceinline__ unsigned long long key_of(unsigned v, int row) { return (unsigned long long)v << 32 | (unsigned)~row; }
__device__ __forceinline__ int row_of(unsigned long long key) { return ~(int)(unsigned)key; }
__device__ __forceinline__ float value_of(unsigned long long key) {   // (-0 comes back as 0)
  const unsigned o = (unsigned)(key >> 32);
  return __uint_as_float(o & 0x80000000u ? o & 0x7fffffffu : ~o);
}
template <bool ROWS>
__global__ __launch_bounds__(kSelectThreads, 4) void topk_groups_kernel(Groups gm, const _Float16 *__restrict__ bank, const float *__restrict__ inv_norm, int N, int d,
                                                                     const _Float16 *__restrict__ probes, int k, int32_t *__restrict__ idx_out,
                                                                     float *__restrict__ sim_out) {
  constexpr int WAVES = kSelectThreads / 64;
  __shared__ unsigned top[kSelectThreads];
  __shared__ __align__(16) unsigned long long cand[kCandidates + 8];
  __shared__ uint2 cand_more[kCandidates];   // group, ordered second
  __shared__ unsigned long long sel[kMaxTopK];
  __shared__ uint2 sel_more[kMaxTopK];
  __shared__ int bin_rank[64], n_cand, n_rows;   // (a count of their own for the rows: a late wavefront may still be reading the groups')
  __shared__ float norm_part[4];
  const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const Group *const groups = gm.g + (size_t)p * gm.pitch;
  const _Float16 *const probe = probes + (size_t)p * d;
  // the groups: the first kSelectHeld a thread stay in registers; of rows all do, four of them next to each other.  (No branch around a load: it would be
  // waited for before the next one goes out.)
  const float *const rows = gm.of_rows(p);
  auto group_at = [&](int at) __attribute__((always_inline)) {
    if (!ROWS) return groups[at];
    return Group{rows[at], 0.f, at, 0};
  };
  constexpr int HELD = ROWS ? kRowsUpTo / kSelectThreads : kSelectHeld;
  Group held[HELD];
  auto held_at = [&](int i) __attribute__((always_inline)) { return ROWS ? (i / 4 * kSelectThreads + tid) * 4 + i % 4 : i * kSelectThreads + tid; };
  if constexpr (ROWS) {
    static_assert(HELD % 4 == 0 && HELD * kSelectThreads == kRowsUpTo, "all of them");
#pragma unroll
    for (int i = 0; i < HELD; i += 4) {
      const f32x4 v = *(const f32x4 *)(rows + min(held_at(i), (gm.n - 1) & ~3));
#pragma unroll
      for (int e = 0; e < 4; ++e) held[i + e] = Group{held_at(i + e) < gm.n ? v[e] : __builtin_nanf(""), 0.f, held_at(i + e), 0};
    }
  } else {
#pragma unroll
    for (int i = 0; i < HELD; ++i) {
      held[i] = group_at(min(held_at(i), gm.n - 1));
      if (held_at(i) >= gm.n) held[i].best = __builtin_nanf("");
    }
  }
  if (tid < 64) bin_rank[tid] = 0;
  if (tid == 0) n_cand = n_rows = 0;
  const float inv = inverse_norm(probe_squares(probe, d, tid), tid, norm_part);
  unsigned best = 0;
#pragma unroll
  for (int i = 0; i < HELD; ++i) best = max(best, ordered(held[i].best));
#pragma unroll 8
  for (int at = HELD * kSelectThreads + tid; at < gm.n; at += kSelectThreads) best = max(best, ordered(group_at(at).best));
  top[tid] = best;
  __syncthreads();
  // the k-th best of 64 bins; a wavefront compares all of them with eight
  unsigned bin = top[lane];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) bin = max(bin, top[w * 64 + lane]);
  {
    int before = 0;
#pragma unroll
    for (int j = 0; j < 64 / WAVES; ++j) {
      const int o = wave * (64 / WAVES) + j;
      const unsigned v = __builtin_amdgcn_readlane(bin, o);
      before += v > bin || (v == bin && o < lane);
    }
    if (before) atomicAdd(&bin_rank[lane], before);
  }
  __syncthreads();
  const unsigned bound = max(1u, (unsigned)__builtin_amdgcn_readlane(bin, __builtin_ctzll(__ballot(bin_rank[lane] == k - 1))));
  auto offer = [&](const Group &o, int at) __attribute__((always_inline)) {
    const unsigned v = ordered(o.best);
    if (v < bound) return;
    const int to = atomicAdd(&n_cand, 1);
    if (to >= kCandidates) return;
    cand[to] = key_of(v, o.row);
    cand_more[to] = make_uint2(at, ordered(o.second));
  };
  if (best >= bound) {
#pragma unroll
    for (int i = 0; i < HELD; ++i) offer(held[i], held_at(i));
    for (int at = HELD * kSelectThreads + tid; at < gm.n; at += kSelectThreads) offer(group_at(at), at);
  }
  __syncthreads();
  int n = n_cand;
  if (n <= kCandidates) {
    for (int c = tid; c < n; c += kSelectThreads) {
      const unsigned long long mine = cand[c];
      int before = 0;
      for (int j0 = 0; j0 < n; j0 += 8) {
        unsigned long long o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = cand[j0 + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) before += j0 + j < n && o[j] > mine;
      }
      if (before < k) {
        sel[before] = mine;
        sel_more[before] = cand_more[c];
      }
    }
    n = min(n, k);
  } else {
    // very many equal groups: k times the best one behind the last one taken
    unsigned long long last = ~0ull;
    for (int j = 0; j < k; ++j) {
      unsigned long long key = 0;
      uint2 more = make_uint2(0, 0);
      for (int at = tid; at < gm.n; at += kSelectThreads) {
        const Group c = group_at(at);
        const unsigned long long o = c.best == c.best ? key_of(ordered(c.best), c.row) : 0ull;
        if (o < last && o > key) {
          key = o;
          more = make_uint2(at, ordered(c.second));
        }
      }
      unsigned long long top_key = key;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long other = __shfl_xor(top_key, o, 64);
        if (other > top_key) top_key = other;
      }
      __syncthreads();
      if (lane == 0) cand[wave] = top_key;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < WAVES; ++w)
        if (cand[w] > top_key) top_key = cand[w];
      if (key == top_key) {   // (rows differ: one thread)
        sel[j] = key;
        sel_more[j] = more;
      }
      last = top_key;
    }
    n = k;   // (more candidates than that, all of them numbers)
  }
  // the k best of the n candidates to the front, in their order
  auto keep_best = [&](int n) __attribute__((always_inline)) {
    unsigned long long key[2] = {0, 0};
    int rank[2] = {k, k};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = h * kSelectThreads + tid;
      if (c >= n) continue;
      key[h] = cand[c];
      rank[h] = 0;
      for (int j0 = 0; j0 < n; j0 += 8) {
        unsigned long long o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = cand[j0 + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) rank[h] += j0 + j < n && o[j] > key[h];
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (rank[h] < k) cand[rank[h]] = key[h];
    if (tid == 0) n_rows = min(n, k);
    __syncthreads();
  };
  __syncthreads();
  if constexpr (ROWS) {   // (perhaps fewer rows than asked for)
    if (tid < k) {
      idx_out[(size_t)p * k + tid] = tid < n ? row_of(sel[tid]) : -1;
      sim_out[(size_t)p * k + tid] = tid < n ? value_of(sel[tid]) * inv : -INFINITY;
    }
    return;
  }
  const unsigned kth = n == k ? (unsigned)(sel[k - 1] >> 32) : 1u;   // (fewer groups than rows asked for: every row that is a number)
  bool doubt = n < k;
  for (int j = 0; j < n; ++j) doubt = doubt || sel_more[j].y >= kth;
  if (!doubt) {
    if (tid < k) {
      idx_out[(size_t)p * k + tid] = row_of(sel[tid]);
      sim_out[(size_t)p * k + tid] = value_of(sel[tid]) * inv;
    }
    return;
  }
  const int best_groups = n, per = gm.jobs(), l32 = lane & 31, g2 = lane >> 5, r16 = lane & 15, g = lane >> 4;
  if (tid < best_groups && sel_more[tid].y < kth) cand[atomicAdd(&n_rows, 1)] = sel[tid];
  int doubted = 0;
  for (int s = 0; s < best_groups; ++s) doubted += sel_more[s].y >= kth;
  __syncthreads();
  const u32x4 *const b = (const u32x4 *)probe;
  auto offer_row = [&](float v, int row) __attribute__((always_inline)) {
    const unsigned o = row < N ? ordered(v) : 0u;
    if (o >= kth) cand[atomicAdd(&n_rows, 1)] = key_of(o, row);
  };
  for (int job0 = 0; job0 < doubted * per; job0 += WAVES) {
    const int job = job0 + wave;
    int s = 0;
    for (int nth = job / per; s < best_groups && (sel_more[s].y < kth || nth-- > 0); ++s) {}
    const int group = s < best_groups ? (int)sel_more[s].x : 0, row0 = s < best_groups ? gm.first_row(group, job % per) : -1;
    if (row0 >= 0) {
      constexpr int U = 8;
      if (gm.kind == Groups::stream) {
        const u32x4 *const a = (const u32x4 *)(bank + (size_t)min(row0 + r16, N - 1) * d) + g;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < d / 32; s0 += U) {
          u32x4 av[U], bv[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int at = min(s0 + u, d / 32 - 1);
            av[u] = a[at * 4];
            bv[u] = b[at * 4 + g];
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (s0 + u < d / 32) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, av[u]), __builtin_bit_cast(f16x8, bv[u]), acc, 0, 0, 0);
        }
        if (r16 == 0) {   // (every column of the product is this probe's)
#pragma unroll
          for (int e = 0; e < 4; ++e) offer_row(acc[e] * inv_norm[min(row0 + g * 4 + e, N - 1)], row0 + g * 4 + e);
        }
      } else {
        const u32x4 *const a = (const u32x4 *)(bank + (size_t)min(row0 + l32, N - 1) * d) + g2;
        pc::f32x16 acc[2];   // (lookup_wide_kernel: even and odd steps apart)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
        for (int s0 = 0; s0 < d / 16; s0 += U) {
          u32x4 av[U], bv[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int at = min(s0 + u, d / 16 - 1);
            av[u] = a[at * 2];
            bv[u] = b[at * 2 + g2];
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (s0 + u >= d / 16) continue;
            const f16x8 x = __builtin_bit_cast(f16x8, av[u]), y = __builtin_bit_cast(f16x8, bv[u]);
            if ((u & 1) && gm.kind == Groups::wide) acc[1] = pc::gemm::mma(x, y, acc[1]);
            else acc[0] = pc::gemm::mma(x, y, acc[0]);
          }
        }
        if (l32 == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = (r >> 2) * 8 + g2 * 4 + (r & 3);
            const float v = gm.kind == Groups::wide ? acc[0][r] + acc[1][r] : acc[0][r];
            if (gm.counts(group, i)) offer_row(v * inv_norm[min(row0 + i, N - 1)], row0 + i);
          }
        }
      }
    }
    __syncthreads();
    static_assert(kCandidates == 2 * kSelectThreads && kCandidates >= 2 * 32 * WAVES, "two a thread; a round of jobs has room behind the k best");
    if (job0 + WAVES < doubted * per) {   // (another round)
      const int have = n_rows;
      __syncthreads();   // (nobody adds to it before all have read it)
      if (have > kCandidates - 32 * WAVES) keep_best(have);
    }
  }
  n = n_rows;
  keep_best(n);
  if (tid < k) {   // (perhaps fewer rows than asked for)
    idx_out[(size_t)p * k + tid] = tid < n ? row_of(cand[tid]) : -1;
    sim_out[(size_t)p * k + tid] = tid < n ? value_of(cand[tid]) * inv : -INFINITY;
  }
}

// ---------------------------------------------------------------------------------------------------
// Many probes at once (more than the one-pass kernels take): the scan is a matrix product E P^T and is bound by the
// matrix cores, not by the stream of the bank.  Tiles of 256 bank rows x PT probes (256, or 128 where that pads less)
// per workgroup of 8 wavefronts, one workgroup per CU,
// which walks a group of consecutive bank tiles; the bank rows are the M side, so a lane holds, for ONE probe, 32 rows
// per tile, scales them by the rows' inverse norms and keeps its best (or the best two of a group).  A CU takes in
// at most 64 bytes per clock from L2, which a 128 x 128 tile would need for as long as its MFMAs run; at 256 x 256
// the operand bytes per flop halve.
// Wavefront (wa, wb) owns bank-row blocks 2 wa, 2 wa + 1 and probe blocks NB wb .. NB wb + NB - 1 (NB = PT / 64).
// LDS stages of 64 k-elements (128-byte rows, chunk ^= (row >> 1) & 7) in a ring of NSTG: as many as fit (two of
// 64 KB at PT = 256, three of 48 KB at PT = 128); a request has NSTG - 1 k-steps to land in.  (128-row tiles with a
// ring of five for up to 128 probes were tried: 0.104 ms against 0.097, a k-step of so little arithmetic is all
// barrier.)  One software pipeline runs over all the k-steps of all the
// workgroup's tiles: the operands of the next 16 k-elements are read from LDS while the MFMAs of the current ones
// run, and the one barrier of a k-step sits before its last quarter -- there every wavefront has read the rest of the
// current stage into registers (so the stage can be requested again, NSTG k-steps ahead) and the next stage has
// landed (its first operands are read under that last quarter's MFMAs).  The request goes out in two parts, behind the
// operand reads of that quarter and of the next one: every wavefront its share of rows and probes alike, so that no
// branch keeps the requests from between the MFMAs, and the last of them has two quarters to land in (three parts, the
// last under the quarter in front of the wait, rows and probes by different wavefronts: 1024 probes, 200 000 rows of
// width 1024, 390 us; now 381).  Tried on it: four wavefronts of 128 x 128 (a third of the LDS reads fewer, one
// instruction stream a SIMD) 433; the whole request under one quarter, or priorities that differ between the wavefronts
// of a SIMD: no change.
// ---------------------------------------------------------------------------------------------------
constexpr int kBigRows = 256;
template <int PT>
struct BigTile {
  static constexpr int A_BYTES = kBigRows * 128, B_BYTES = PT * 128, STAGE = A_BYTES + B_BYTES;
  static constexpr int NSTG = 160 * 1024 / STAGE;
  static constexpr int LDS = NSTG * STAGE;
  static constexpr int A_PER = A_BYTES / 1024 / 8, B_PER = B_BYTES / 1024 / 8;  // request instructions per wavefront and stage
  static constexpr int PER = A_PER + B_PER, PART = PER / 2;                     // requested in two parts
  static_assert((PT == 256 || PT == 128) && NSTG >= 2 && NSTG <= 5, "tile");
};

template <int PT, int K>
__global__ __launch_bounds__(512, 1) void lookup_big_kernel(const _Float16 *__restrict__ bank, const float *__restrict__ inv_norm,
                                                            int N, int d, const _Float16 *__restrict__ probes, int n_probes,
                                                            int p_pad, int n_groups, int p_tiles, Best *__restrict__ partial, Groups gm) {
  extern __shared__ __align__(16) char smem[];
  using BT = BigTile<PT>;
  constexpr int ROW = 128, RT = kBigRows, NSTG = BT::NSTG, STAGE = BT::STAGE, NA = RT / 128, NB = PT / 64;
  // the probe tiles of one bank group run next to each other on ONE XCD (workgroup ids go round-robin over the 8):
  // the group's rows come from HBM once and are re-read from that XCD's L2
  const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;
  const int group = (jj / p_tiles) * 8 + xcd, p_tile = jj % p_tiles;
  if (group >= n_groups) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wa = wave & 3, wb = wave >> 2;
  const int l32 = lane & 31, g = lane >> 5;
  const int n_tiles = (N + RT - 1) / RT;
  const int tile_begin = (int)((long)group * n_tiles / n_groups), tile_end = (int)((long)(group + 1) * n_tiles / n_groups);
  const int m0 = p_tile * PT;
  const int nk = d / 64;

  // requests: instruction i of a half-stage fills its bytes [1024 i, 1024 i + 1024), i.e. rows 8 i .. 8 i + 7; every wavefront brings
  // A_PER of the bank rows' and B_PER of the probes', from a scalar base and 32-bit lane offsets (the bank's from its tile on)
  const int my_chunk = lane & 7;
  unsigned off[BT::PER];
  int f_tile = tile_begin, f_kt = 0;  // what the next request brings
  const char *a_base = nullptr;
  auto aim = [&]() __attribute__((always_inline)) {
    a_base = (const char *)(bank + (size_t)f_tile * RT * d);
#pragma unroll
    for (int k = 0; k < BT::A_PER; ++k) {
      const int row = (wave * BT::A_PER + k) * 8 + (lane >> 3);
      off[k] = (unsigned)((min(f_tile * RT + row, N - 1) - f_tile * RT) * d + ((my_chunk ^ pc::gemm::swz128(row)) * 8)) * 2u;
    }
  };
#pragma unroll
  for (int k = 0; k < BT::B_PER; ++k) {
    const int row = (wave * BT::B_PER + k) * 8 + (lane >> 3);
    off[BT::A_PER + k] = (unsigned)((min(m0 + row, n_probes - 1) - m0) * d + ((my_chunk ^ pc::gemm::swz128(row)) * 8)) * 2u;
  }
  const char *const b_base = (const char *)(probes + (size_t)m0 * d);
  // instructions k0 .. k1 - 1 of the request for k-step (f_tile, f_kt) into ring slot `slot`
  auto request_part = [&](int slot, int k0, int k1) __attribute__((always_inline)) {
#pragma unroll
    for (int k = k0; k < k1; ++k) {
      const bool a = k < BT::A_PER;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)((a ? a_base : b_base) + (size_t)f_kt * 128 + off[k]),
                                       (__attribute__((address_space(3))) void *)(smem + slot * STAGE + (a ? (wave * BT::A_PER + k) * 1024 : BT::A_BYTES + (wave * BT::B_PER + k - BT::A_PER) * 1024)),
                                       16, 0, 0);
    }
  };
  // on to the next k-step; past the last one the cursor stays on valid rows (requests made then land in a slot that
  // nobody reads any more)
  auto advance = [&]() __attribute__((always_inline)) {
    if (++f_kt == nk) {
      f_kt = 0;
      if (f_tile + 1 < tile_end) {
        ++f_tile;
        a_base += (size_t)RT * d * 2;
        if (f_tile + 1 == n_tiles) aim();   // (rows past the end)
      }
    }
  };
  // operand reads: this lane's row inside a 32-row block is l32; k-quarter q of a stage is chunk 2 q + g
  int rd[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) rd[q] = ((2 * q + g) ^ pc::gemm::swz128(l32)) * 16;
  const int a_off = (NA * wa * 32 + l32) * ROW, b_off = BT::A_BYTES + (NB * wb * 32 + l32) * ROW;
  f16x8 oa[2][NA], ob[2][NB];  // two register sets
  auto read_ops = [&](int set, int slot, int q) __attribute__((always_inline)) {
    const char *base = smem + slot * STAGE + rd[q];
#pragma unroll
    for (int a = 0; a < NA; ++a) oa[set][a] = *(const f16x8 *)(base + a_off + a * 32 * ROW);
#pragma unroll
    for (int t = 0; t < NB; ++t) ob[set][t] = *(const f16x8 *)(base + b_off + t * 32 * ROW);
  };
  pc::f32x16 acc[NA][NB];
  auto mma_ops = [&](int set) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
      for (int a = 0; a < NA; ++a) acc[a][t] = pc::gemm::mma(oa[set][a], ob[set][t], acc[a][t]);
  };
  // one MFMA, one LDS read, ... : the reads of the next quarter go out under the MFMAs of this one, and so do
  // `loads` request instructions (a CU's 64 per k-step issued in one burst hold every wavefront in the issue queue
  // for the thousand cycles the texture path needs for them)
  auto interleave = [&](int loads) __attribute__((always_inline)) {
    constexpr int READS = NA + NB, MMAS = NA * NB;
#pragma unroll
    for (int i = 0; i < (READS < MMAS ? READS : MMAS); ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < (MMAS > READS ? MMAS - READS : 0); ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      for (int l = loads * i / (MMAS - READS); l < loads * (i + 1) / (MMAS - READS); ++l) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
  };

  Top2 top[NB];      // (K == kGroups) of the group that this wavefront is in
  TopK<1> best[NB];  // this lane's rows for probes m0 + (NB wb + t) * 32 + l32 (K == 1)
#pragma unroll
  for (int t = 0; t < NB; ++t) best[t].clear();

  if (tile_begin < tile_end) {  // the first k-step, then whole requests for the next NSTG - 2 and the first part of one more
    aim();
    request_part(0, 0, BT::PER);
    advance();
    pc::gemm::wait_vmcnt0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s2 = 1; s2 < NSTG - 1; ++s2) {
      request_part(s2, 0, BT::PER);
      advance();
    }
    request_part(NSTG - 1, 0, BT::PART);  // (the rest of it under the first quarter below)
    read_ops(0, 0, 0);
  }
  int slot = 0;  // ring slot of this k-step
  for (int tile = tile_begin; tile < tile_end; ++tile) {
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][t][r] = 0.f;
    const int row_mine = tile * RT + NA * wa * 32 + lane;
    const float inv_mine = row_mine < N && lane < NA * 32 ? inv_norm[row_mine] : __builtin_nanf("");  // (in flight under the tile's k-steps)
    for (int kt = 0; kt < nk; ++kt) {
      const int slot_prev = slot == 0 ? NSTG - 1 : slot - 1, slot_next = slot == NSTG - 1 ? 0 : slot + 1;
      // a request was begun behind the last barrier, into the slot that k-step gave up: the rest of its instructions
      read_ops(1, slot, 1);
      request_part(slot_prev, BT::PART, BT::PER);
      mma_ops(0);
      interleave(BT::PER - BT::PART);
      advance();
      read_ops(0, slot, 2);
      mma_ops(1);
      interleave(0);
      read_ops(1, slot, 3);
      mma_ops(0);
      interleave(0);
      // every read of this stage is in registers and this wavefront's part of the next stage has landed: all of its
      // requests but the NSTG - 2 latest ones, which are for later k-steps
      pc::gemm::wait_vmcnt_lds<(NSTG - 2) * BT::PER>();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      read_ops(0, slot_next, 0);      // (past the last k-step: whatever that slot holds, never multiplied)
      request_part(slot, 0, BT::PART);       // the k-step NSTG ahead (past the end: see advance())
      mma_ops(1);
      interleave(BT::PART);
      slot = slot_next;
    }
    // cosines of this tile's rows (up to the probe's own norm, which the finalize kernel divides by)
    const int r0 = tile * RT;
    if constexpr (K == 1) {
      // Lane L of the wavefront has fetched the inverse norm of the wavefront's row L (of NA * 32) while the tile was
      // multiplied -- NaN past the end of the bank, which no comparison below ever prefers -- and a lane takes the
      // ones of its own rows from there.  Its 32 rows are visited in rising order, so "greater" alone keeps the
      // lowest row among equals, within the tile and against earlier tiles.
      float ls[NB];
      int lc[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t) { ls[t] = -INFINITY; lc[t] = 0; }
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          float inv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) inv[e] = __shfl(inv_mine, a * 32 + q4 * 8 + g * 4 + e, 64);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < NB; ++t) {
              const float v = acc[a][t][q4 * 4 + e] * inv[e];
              lc[t] = v > ls[t] ? a * 16 + q4 * 4 + e : lc[t];
              ls[t] = fmaxf(ls[t], v);
            }
          __builtin_amdgcn_sched_barrier(0);  // (four exchanged norms live at a time, not thirty-two)
        }
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const int row = r0 + (NA * wa + (lc[t] >> 4)) * 32 + ((lc[t] >> 2) & 3) * 8 + g * 4 + (lc[t] & 3);
        const bool up = ls[t] > best[t].s[0];
        best[t].s[0] = up ? ls[t] : best[t].s[0];
        best[t].i[0] = up ? row : best[t].i[0];
      }
    } else if constexpr (K == kRows) {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int in = a * 32 + q4 * 8 + g * 4, row = r0 + NA * wa * 32 + in;
          float inv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) inv[e] = __shfl(inv_mine, in + e, 64);
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            const int p = m0 + (NB * wb + t) * 32 + l32;
            if (p < n_probes && row < N)
              *(f32x4 *)(gm.of_rows(gm.p0 + p) + row) = f32x4{acc[a][t][q4 * 4] * inv[0], acc[a][t][q4 * 4 + 1] * inv[1], acc[a][t][q4 * 4 + 2] * inv[2], acc[a][t][q4 * 4 + 3] * inv[3]};
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    } else {
      // lane (l32, 0) has rows 0..3, 8..11, 16..19, 24..27 of a block, lane (l32, 1) the others
      const int base = r0 + NA * wa * 32 + g * 4;
      const bool fine = gm.kind == Groups::big_fine, ends = (tile - tile_begin + 1) % gm.stretch == 0 || tile + 1 == tile_end;
      float inv[NA][16];
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) inv[a][r] = __shfl(inv_mine, a * 32 + (r >> 2) * 8 + g * 4 + (r & 3), 64);
      // (probes outside: one best and second best at a time; in the other order they spill)
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const int p = m0 + (NB * wb + t) * 32 + l32;
        Group *const to = gm.g + (size_t)(gm.p0 + p) * gm.pitch;
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          Top2 mine;
#pragma unroll
          for (int r = 0; r < 16; ++r) mine.add(acc[a][t][r] * inv[a][r], a * 32 + (r >> 2) * 8 + (r & 3));
          if (__ballot(mine.i == INT_MAX)) {
            if (mine.i == INT_MAX)
#pragma unroll
              for (int r = 0; r < 16; ++r) mine.first(acc[a][t][r] * inv[a][r], a * 32 + (r >> 2) * 8 + (r & 3));
          }
          mine.i += mine.i == INT_MAX ? 0 : base;
          if (fine) {
            if (p < n_probes) write_group(to + ((tile * 4 + wa) * NA + a) * 2 + g, mine);
          } else {
            top[t].merge(mine);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (!fine && ends) {
          Top2 both = top[t];
          both.merge(both.of_lane_xor(32));
          if (g == 0 && p < n_probes) write_group(to + (group * 4 + wa) * gm.per + (tile - tile_begin) / gm.stretch, both);
          top[t] = Top2{};
        }
      }
    }
  }
  if constexpr (K != 1) {
    pc::gemm::wait_vmcnt0();  // (the surplus requests)
    if (K == kGroups && gm.kind == Groups::big)   // groups that this wavefront has no rows for
      for (int j = (tile_end - tile_begin + gm.stretch - 1) / gm.stretch; j < gm.per; ++j)
        for (int t = 0; t < NB; ++t) {
          const int p = m0 + (NB * wb + t) * 32 + l32;
          if (g == 0 && p < n_probes) write_group(gm.g + (size_t)(gm.p0 + p) * gm.pitch + (group * 4 + wa) * gm.per + j, Top2{});
        }
    return;
  }
  // the two lanes of a probe, then the four wavefronts (wa) that hold other rows of the same probes
  __builtin_amdgcn_s_waitcnt(7 << 4);
  __syncthreads();
  Best *red = (Best *)smem;  // [wb][wa][NB * 32]
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    float s = best[t].s[0];
    int i = best[t].i[0];
    const float s2 = __shfl_xor(s, 32, 64);
    const int i2 = __shfl_xor(i, 32, 64);
    if (better(s2, i2, s, i)) { s = s2; i = i2; }
    if (g == 0) red[(wb * 4 + wa) * (NB * 32) + t * 32 + l32] = Best{s, i};
  }
  __syncthreads();
  if (tid < PT) {  // one thread per probe of the tile: probe wb2 * NB * 32 + within
    const int wb2 = tid / (NB * 32), within = tid % (NB * 32);
    Best b{-INFINITY, INT_MAX};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const Best c = red[(wb2 * 4 + w) * (NB * 32) + within];
      if (c.idx != INT_MAX && (b.idx == INT_MAX || better(c.s, c.idx, b.s, b.idx))) b = c;
    }
    partial[(size_t)group * p_pad + m0 + tid] = b;
  }
}

// ---------------------------------------------------------------------------------------------------
// Up to 128 probes in one pass of the bank (embedding widths of 512, 768 and 1024 elements).
// One workgroup per CU; wavefront w keeps ITS 32 probes in registers as the N-side operands of the 32x32x16 product
// (d/4 registers per lane: one wavefront per SIMD), and all four wavefronts multiply the same 32-row blocks of the
// bank, which stream through a ring of LDS stages shared by the workgroup (32 rows x 512 bytes per stage; every
// load instruction brings two contiguous 512-byte runs; NSTG - 1 stages in flight).  One barrier per stage: it
// publishes the stage that has landed and retires the one just multiplied.  A lane ends up with 16 rows of one
// probe per block, scales them by the rows' inverse norms and keeps its best (or the best two of a group), as in the kernel above.
// RS sets of 32 rows a block: up to 64 probes leave two of the four wavefronts without any, so these take another 32 rows (RS = 2): half the
// arithmetic a row, and half the barriers, of stages twice as large.  200 000 rows of width 1024, 64 probes: best row 90 us | 74, per-row mode 101 | 73
// (3 of them an earlier launch for the probes' norms, which the wavefronts now take from the registers that hold the probes).
// Per-row mode (K == 0, see RowScan): the operands swap sides, so a lane holds ONE row and 16 probes; the wavefronts'
// candidates of a block meet in LDS and are written out one block later, behind a barrier that is there anyway, by the
// wavefronts in turn.  The thresholds sit in LDS beside the inverse norms: a load from memory in front of the decision
// would drain the ring.
// ---------------------------------------------------------------------------------------------------
constexpr int kWideProbes = 128;
constexpr int kWideStages = 8;              // of 32 rows; half as many of 64
constexpr int kWideChunk = 512;             // bytes of a row per stage (256 where they do not divide a row)
constexpr int kWideMaxBlocksPerWg = 192;    // 6144 rows: bounds the LDS copy of the inverse norms (24 KB)
constexpr int kScanMaxBlocksPerWg = 80;     // per-row mode: of the inverse norms and the thresholds (20 KB), beside the candidates
constexpr int kScanHead = kScanMaxBlocksPerWg * 32 * 8 + 2 * 4 * 32 * (int)sizeof(Best);

template <int D_EMB, int K, int RS, int CHB = kWideChunk>
__global__ __launch_bounds__(256, 1) void lookup_wide_kernel(const _Float16 *__restrict__ bank, const float *__restrict__ inv_norm,
                                                             int N, const _Float16 *__restrict__ probes, int n_probes, int per_wg,
                                                             Best *__restrict__ partial, RowScan rs, Groups gm) {
  extern __shared__ __align__(16) char smem[];
  constexpr int NSTG = kWideStages / RS, BR = 32 * RS, NG = 4 / RS;   // rows of a block, wavefronts with probes of their own
  constexpr int CHUNKS = D_EMB * 2 / CHB;  // stages per row block
  constexpr int CS = CHB / 32;             // MFMA k-steps (16 elements) per stage
  constexpr int STG = BR * CHB;            // bytes per stage
  constexpr int IPS = STG / 1024 / 4;      // load instructions per stage and wavefront
  static_assert(D_EMB * 2 % CHB == 0, "row must be a whole number of chunks");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, g2 = lane >> 5;
  const int pg = wave % NG, set = wave / NG;   // this wavefront's probes, and its 32 rows of a block
  const int n_blocks = (N + BR - 1) / BR;
  const int rb_begin = blockIdx.x * per_wg, rb_end = min(n_blocks, rb_begin + per_wg);

  // inverse norms of this workgroup's rows (zero beyond N), then the ring
  float *inv_lds = (float *)smem;
  float *kth_lds = inv_lds + kScanMaxBlocksPerWg * 32;                  // (K == 0)
  Best *cand = (Best *)(kth_lds + kScanMaxBlocksPerWg * 32);            // (K == 0) [block parity][wavefront][row]
  char *ring = smem + (K == 0 ? kScanHead : kWideMaxBlocksPerWg * 32 * (int)sizeof(float));
  const bool idle = pg * 32 >= n_probes;  // nothing but padding: this wavefront only loads
  // load instruction i of a stage (i = wave + 4 k): stage bytes [1024 i, +1024) = whole rows
  int ld_row[IPS], ld_col[IPS];
#pragma unroll
  for (int k = 0; k < IPS; ++k) {
    const int row = (wave + 4 * k) * (1024 / CHB) + lane / (CHB / 16), pc = lane % (CHB / 16);
    ld_row[k] = row;
    ld_col[k] = (pc ^ (row & 15)) * 8;  // element offset of the logical 16-byte chunk this lane fetches
  }
  auto issue = [&](int rb, int chunk, int st) __attribute__((always_inline)) {
    const _Float16 *base = bank + chunk * (CHB / 2);
#pragma unroll
    for (int k = 0; k < IPS; ++k) {
      const int row = min(rb * BR + ld_row[k], N - 1);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(base + (size_t)row * D_EMB + ld_col[k]),
                                       (__attribute__((address_space(3))) void *)(ring + st * STG + (wave + 4 * k) * 1024), 16, 0, kBankLoadAux);
    }
  };
  // The first stages are asked for behind the probes and the norms but in front of the wait for them: all of these are one memory latency.
  // Four rows' norms a thread at a time (one by one they are a latency each).
  float row_inv[4], row_kth[4];
  auto fetch_rows = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = min(rb_begin * BR + r0 + e * 256 + tid, N - 1);
      row_inv[e] = inv_norm[row];
      if (K == 0) row_kth[e] = rs.kth[row];
    }
  };
  auto keep_rows = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = r0 + e * 256 + tid;
      if (r >= per_wg * BR) continue;
      lds_put(inv_lds + r, rb_begin * BR + r < N ? row_inv[e] : 0.f);
      if (K == 0) lds_put(kth_lds + r, rb_begin * BR + r < N ? row_kth[e] : 0.f);
    }
  };
  fetch_rows(0);
  // this lane's probe: elements [16 ks + 8 g2, +8) for every k-step (zero for a padding probe)
  f16x8 pq[D_EMB / 16];
  {
    const int p = pg * 32 + l32;
    const u32x4 *src = (const u32x4 *)(probes + (size_t)min(p, n_probes - 1) * D_EMB);
#pragma unroll
    for (int ks = 0; ks < D_EMB / 16; ++ks) pq[ks] = __builtin_bit_cast(f16x8, src[2 * ks + g2]);
  }
  const int rb_last = rb_end - 1;
  int prb = rb_begin, pch = 0, ist = 0, st = 0;
  auto advance = [&](int &rb_, int &c_) __attribute__((always_inline)) {
    if (++c_ == CHUNKS) { c_ = 0; ++rb_; }
  };
  // flat sequence of (row block, chunk) items; loads go out unconditionally (past the end they repeat the last
  // block into a stage nobody reads), so the count of loads in flight is the same at every wait
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < NSTG - 1; ++k) {
    issue(min(prb, rb_last), pch, ist);
    advance(prb, pch);
    ist = ist + 1 == NSTG ? 0 : ist + 1;
  }
  __builtin_amdgcn_sched_barrier(0);
  PC_LOOKUP_WAIT_VMCNT((NSTG - 1) * IPS);   // (left to itself the compiler waits for the ring as well, or moves a load behind it)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    asm volatile("" : "+v"(row_inv[e]));
    if (K == 0) asm volatile("" : "+v"(row_kth[e]));
  }
  keep_rows(0);
  for (int r0 = 1024; r0 < per_wg * BR; r0 += 1024) {
    fetch_rows(r0);
    keep_rows(r0);
  }
  if (pg * 32 + l32 >= n_probes) {
#pragma unroll
    for (int ks = 0; ks < D_EMB / 16; ++ks) pq[ks] = f16x8{};
  }
#pragma unroll
  for (int ks = 0; ks < D_EMB / 16; ++ks) asm volatile("" : "+v"(pq[ks]));
  // per-row mode: inverse norms of the probes this lane meets (a padding probe's is a NaN, which no comparison picks)
  float pinv[K == 0 ? 16 : 1];
  if constexpr (K == 0) {
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < D_EMB / 16; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) ss[e & 3] += (float)pq[ks][e] * (float)pq[ks][e];
    float tot = (ss[0] + ss[1]) + (ss[2] + ss[3]);
    tot += __shfl_xor(tot, 32, 64);
    const float inv = pg * 32 + l32 >= n_probes ? __builtin_nanf("") : tot > 0.f ? 1.0f / sqrtf(tot) : 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) pinv[r] = __shfl(inv, (r >> 2) * 8 + g2 * 4 + (r & 3), 64);
#pragma unroll
    for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(pinv[r]));
  }
  lds_barrier();

  int rd_off[CS];  // swizzled byte offsets of this lane's operand reads inside a stage
#pragma unroll
  for (int s = 0; s < CS; ++s) rd_off[s] = (set * 32 + l32) * CHB + (((2 * s + g2) ^ (l32 & 15)) * 16);

  Top2 top;   // (K == kGroups) of the group that this workgroup is in
  TopK<1> best;
  best.clear();
  // (K == 0) the candidates of a block whose barrier has passed: one row per lane of the wavefront whose turn it is
  auto write_rows = [&](int rb) __attribute__((always_inline)) {
    if ((rb & 3) != wave || lane >= BR) return;
    const int row = rb * BR + lane;
    Best b = cand[(rb & 1) * 128 + lane];
#pragma unroll
    for (int w = 1; w < NG; ++w) {
      const Best o = cand[(rb & 1) * 128 + w * BR + lane];
      if (better(o.s, o.idx, b.s, b.idx)) b = o;
    }
    if (row >= N) return;
    if (!rs.first) {
      const Best o{rs.best_sim[row], rs.best_new[row]};
      if (!better(b.s, b.idx, o.s, o.idx)) b = o;
    }
    rs.best_sim[row] = b.s;
    rs.best_new[row] = b.idx == INT_MAX ? -1 : b.idx;
    rs.stale[row] = b.s > kth_lds[(rb - rb_begin) * BR + lane] ? 1 : 0;
  };
  if (K == 0 && idle && g2 == 0) cand[pg * BR + set * 32 + l32] = cand[128 + pg * BR + set * 32 + l32] = Best{-INFINITY, INT_MAX};
  if (rb_begin < rb_end) {
    for (int rb = rb_begin; rb < rb_end; ++rb) {
      pc::f32x16 acc[2];  // two accumulation chains: an MFMA does not wait for the one before it
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][r] = 0.f;
#pragma unroll
      for (int c = 0; c < CHUNKS; ++c) {
        // the oldest stage in flight has landed (mine), then (barrier) everyone's; the barrier also says that the
        // stage multiplied last is free for the next load
        PC_LOOKUP_WAIT_VMCNT((NSTG - 2) * IPS);
        if (K == 0 && c == 0) asm volatile("s_waitcnt lgkmcnt(0)");  // (the last block's candidates are in LDS)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(min(prb, rb_last), pch, ist);
        advance(prb, pch);
        ist = ist + 1 == NSTG ? 0 : ist + 1;
        if (K == 0 && c == 0 && rb > rb_begin) write_rows(rb - 1);
        if (K == 0 && idle) {
          st = st + 1 == NSTG ? 0 : st + 1;
          continue;
        }
        // all of the stage's operands are asked for before its first MFMA (left to itself the compiler reads one
        // operand, waits, multiplies: one LDS latency per MFMA instead of one per stage)
        const char *abase = ring + st * STG;
        f16x8 av[CS];
#pragma unroll
        for (int s = 0; s < CS; ++s) av[s] = *(const f16x8 *)(abase + rd_off[s]);
#pragma unroll
        for (int s = 0; s < CS; ++s)
          acc[s & 1] = K == 0 ? __builtin_amdgcn_mfma_f32_32x32x16_f16(pq[c * CS + s], av[s], acc[s & 1], 0, 0, 0)
                              : __builtin_amdgcn_mfma_f32_32x32x16_f16(av[s], pq[c * CS + s], acc[s & 1], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, CS, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, CS, 0);
        st = st + 1 == NSTG ? 0 : st + 1;
      }
      if constexpr (K == 0) {
        // element r of the product: row l32 of the block, probe wave*32 + (r/4)*8 + 4*g2 + r%4 (ascending: the lowest wins ties)
        if (idle) continue;
        const float inv = inv_lds[(rb - rb_begin) * BR + set * 32 + l32];
        Best b{-INFINITY, INT_MAX};
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int p = pg * 32 + (r >> 2) * 8 + g2 * 4 + (r & 3);
          const float s = (acc[0][r] + acc[1][r]) * inv * pinv[r];
          if (better(s, rs.p0 + p, b.s, b.idx)) b = Best{s, rs.p0 + p};
        }
        const Best o{__shfl_xor(b.s, 32, 64), __shfl_xor(b.idx, 32, 64)};
        if (better(o.s, o.idx, b.s, b.idx)) b = o;
        if (g2 == 0) cand[(rb & 1) * 128 + pg * BR + set * 32 + l32] = b;
        continue;
      }
      // element r of the product: row (r/4)*8 + 4*g2 + r%4 of the block, probe wave*32 + l32
      if constexpr (K == kRows) {
        const int p = pg * 32 + l32;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int rin = set * 32 + q4 * 8 + g2 * 4, row0 = rb * BR + rin;
          const f32x4 inv4 = *(const f32x4 *)(inv_lds + (rb - rb_begin) * BR + rin);
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = row0 + e < N ? (acc[0][q4 * 4 + e] + acc[1][q4 * 4 + e]) * inv4[e] : __builtin_nanf("");
          if (p < n_probes && row0 < N) *(f32x4 *)(gm.of_rows(gm.p0 + p) + row0) = v;
        }
        continue;
      }
      if constexpr (K == kGroups) {
        float v[16];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int rin = q4 * 8 + g2 * 4;
          const f32x4 inv4 = *(const f32x4 *)(inv_lds + (rb - rb_begin) * BR + set * 32 + rin);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = q4 * 4 + e, row = rb * BR + set * 32 + rin + e;
            v[r] = row < N ? (acc[0][r] + acc[1][r]) * inv4[e] : __builtin_nanf("");
            top.add(v[r], row);
          }
        }
        if (__ballot(top.i == INT_MAX)) {
          const bool none = top.i == INT_MAX;
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (none) top.first(v[r], rb * BR + set * 32 + (r >> 2) * 8 + g2 * 4 + (r & 3));
        }
        const int nth = rb - rb_begin, p = pg * 32 + l32;
        if ((nth + 1) % gm.stretch == 0 || rb == rb_last) {
          top.merge(top.of_lane_xor(32));
          if (g2 == 0 && p < n_probes) write_group(gm.g + (size_t)(gm.p0 + p) * gm.pitch + (blockIdx.x * RS + set) * gm.per + nth / gm.stretch, top);
          top = Top2{};
        }
        continue;
      }
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int rin = q4 * 8 + g2 * 4;
        const f32x4 inv4 = *(const f32x4 *)(inv_lds + (rb - rb_begin) * BR + set * 32 + rin);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = rb * BR + set * 32 + rin + e;
          if (row < N) best.insert((acc[0][q4 * 4 + e] + acc[1][q4 * 4 + e]) * inv4[e], row);
        }
      }
    }
    if constexpr (K == 0) {
      __syncthreads();
      write_rows(rb_last);
    }
  }
  PC_LOOKUP_WAIT_VMCNT(0);
  if constexpr (K == kGroups) {   // groups that this workgroup has no rows for
    const int p = pg * 32 + l32;
    for (int j = (max(rb_end - rb_begin, 0) + gm.stretch - 1) / gm.stretch; j < gm.per; ++j)
      if (g2 == 0 && p < n_probes) write_group(gm.g + (size_t)(gm.p0 + p) * gm.pitch + (blockIdx.x * RS + set) * gm.per + j, Top2{});
  }
  if constexpr (K <= 0) return;  // per-row mode and groups: everything has been written
  // the two lanes of a probe hold different rows
  float s = best.s[0];
  int i = best.i[0];
  const float s2 = __shfl_xor(s, 32, 64);
  const int i2 = __shfl_xor(i, 32, 64);
  if (better(s2, i2, s, i)) { s = s2; i = i2; }
  if (g2 == 0) partial[((size_t)blockIdx.x * RS + set) * (NG * 32) + pg * 32 + l32] = Best{s, i};
}

__global__ void lookup_empty_kernel(int n_out, int n_probes, int32_t *idx_out, float *sim_out, uint8_t *hit_out) {
  int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n_out) { idx_out[p] = -1; sim_out[p] = -INFINITY; }
  if (hit_out && p < n_probes) hit_out[p] = 0;
}

constexpr int kPassProbes = 32;

// LDS bytes of one workgroup: probes, inverse norms, then (1 KB aligned) the four wavefront rings.
constexpr size_t kMaxLds = 160 * 1024;
struct StreamShape {
  int grid, per_wg, nstg, chb, ring_off;
  size_t lds;
};
StreamShape stream_shape(const percache_ctx *ctx, int npb, int N) {
  const int d = ctx->cfg.emb_dim;
  StreamShape s;
  s.chb = d * 2 % 512 == 0 ? 512 : d * 2 % 256 == 0 ? 256 : 128;  // widest chunk that divides a row
  const int n_blocks = (N + 15) / 16;
  s.grid = ctx->n_cu;  // the rings allow one workgroup per CU
  const int need = (n_blocks + 3) / 4;  // at least one block per wavefront
  if (s.grid > need) s.grid = need > 0 ? need : 1;
  s.per_wg = (n_blocks + s.grid - 1) / s.grid;
  if (s.per_wg > kMaxBlocksPerWg) {
    s.per_wg = kMaxBlocksPerWg;
    s.grid = (n_blocks + s.per_wg - 1) / s.per_wg;
  }
  size_t head = (size_t)npb * 16 * (d * 2 + kProbePad) + (size_t)s.per_wg * 16 * sizeof(float);
  s.ring_off = (int)((head + 1023) / 1024 * 1024);
  // three stages per wavefront for a single probe block if they fit beside the probes, else two
  s.nstg = npb == 1 && s.ring_off + (size_t)4 * 3 * 16 * s.chb <= kMaxLds ? 3 : 2;
  s.lds = s.ring_off + (size_t)4 * s.nstg * 16 * s.chb;
  return s;
}
int max_stream_grid(const percache_ctx *ctx) {
  int by_rows = (ctx->cfg.bank_capacity / 16 + kMaxBlocksPerWg) / kMaxBlocksPerWg;
  return by_rows > ctx->n_cu ? by_rows : ctx->n_cu;
}

constexpr int kBatchedFrom = 32;  // more probes than one streaming pass takes: the 128-probe pass or the matrix-product kernel
// Per-row scan: more new embeddings than one streaming pass takes go through 128-probe passes.  200k rows, streaming passes | 128-probe
// passes, us: width 384 69 | 42 at 33, 79 | 43 at 64, 161 | 67 at 128; width 1024 141 | 72 at 64, 288 | 111 at 128, 495 | 227 at 200.
constexpr int kScanWideFrom = 32;
constexpr int kWideUpTo = 128;    // one such pass; beyond it the matrix-product kernel is the faster one

// Launch shape of the 256-row kernel: probe tiles x groups of consecutive 256-row bank tiles, one workgroup per CU (a
// multiple of 8 groups, so that a group's probe tiles share an XCD), every group at least one tile.
struct BigShape {
  int p_tiles, groups;
};
BigShape big_shape(int n_cu, int N, int n_probes, int pt) {
  BigShape b;
  b.p_tiles = (n_probes + pt - 1) / pt;
  const int n_tiles = (N + kBigRows - 1) / kBigRows;
  b.groups = n_cu / b.p_tiles / 8 * 8;
  if (b.groups < 8) b.groups = 8;
  if (b.groups > n_tiles) b.groups = n_tiles;
  return b;
}
// whether 256-probe tiles are filled well enough to beat 128-probe ones (at most a third of padding)
bool big_tiles_pay(int n_probes) {
  if (n_probes <= kWideUpTo) return false;
  const long padded = (long)(n_probes + 255) / 256 * 256;
  return padded * 3 <= (long)n_probes * 4;
}

template <int NPB, int CHB, int NSTG, int K>
pc_status launch_stream(percache_ctx *ctx, const StreamShape &sh, hipStream_t st, int N, int d, const _Float16 *pp, int np,
                        Best *partial, const RowScan &rs, const InLaunch &il, const Groups &gm) {
  static bool big_lds_set = false;  // dynamic LDS above 64 KB must be opted into once per kernel
  if (!big_lds_set) {
    PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_stream_kernel<NPB, CHB, NSTG, K>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds));
    big_lds_set = true;
  }
  hipLaunchKernelGGL((lookup_stream_kernel<NPB, CHB, NSTG, K>), dim3(sh.grid), dim3(256), sh.lds, st, ctx->bank, ctx->bank_inv, N, d,
                     pp, np, sh.per_wg, sh.ring_off, partial, rs, il, gm);
  return PC_OK;
}

template <int K>
pc_status launch_one_block(percache_ctx *ctx, const StreamShape &sh, hipStream_t st, int N, int d, const _Float16 *pp, int np, Best *partial, const RowScan &rs,
                           const InLaunch &il, const Groups &gm) {
  return sh.chb == 128   ? launch_stream<1, 128, 3, K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm)
         : sh.chb == 256 ? launch_stream<1, 256, 3, K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm)
                         : launch_stream<1, 512, 3, K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm);
}
template <int K>
pc_status launch_pass(percache_ctx *ctx, const StreamShape &sh, int npb, hipStream_t st, int N, int d, const _Float16 *pp, int np,
                      Best *partial, const RowScan &rs = RowScan{}, const InLaunch &il = InLaunch{}, const Groups &gm = Groups{}) {
  if (npb == 1 && sh.nstg == 3) return launch_one_block<K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm);
  if (npb == 1) return launch_stream<1, 512, 2, K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm);  // only the widest rows (512-byte chunks) get here
  return sh.chb == 128   ? launch_stream<2, 128, 2, K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm)
         : sh.chb == 256 ? launch_stream<2, 256, 2, K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm)
                         : launch_stream<2, 512, 2, K>(ctx, sh, st, N, d, pp, np, partial, rs, il, gm);
}

// What a call of n_probes needs at least: eight rows a workgroup and probe, of which a call for the best row uses one.  A top-k call that is given no
// more than this makes its groups as large as they have to be: four a workgroup always fit.
size_t list_bytes(const percache_ctx *ctx, int32_t n_probes) {
  size_t lists = (size_t)max_stream_grid(ctx) * kPassProbes;
  if (n_probes > kBatchedFrom) {
    // the 256-row kernel: groups * p_tiles <= max(n_cu, 8 p_tiles) workgroups of at most 256 lists
    const size_t p_big = ((size_t)n_probes + 127) / 128;
    const size_t big = ((size_t)ctx->n_cu > 8 * p_big ? (size_t)ctx->n_cu : 8 * p_big) * 256;
    if (big > lists) lists = big;
    // the 128-probe pass: one list per workgroup and probe
    const size_t wide_grid = (size_t)ctx->cfg.bank_capacity / (32 * kWideMaxBlocksPerWg) + 1;
    const size_t wide = (wide_grid > (size_t)ctx->n_cu ? wide_grid : (size_t)ctx->n_cu) * kWideProbes;
    if (wide > lists) lists = wide;
  }
  return pc::align_up(lists * kMaxTopK * sizeof(Best));
}

constexpr int kInLaunchProbes = 4;   // (one wavefront of the merging workgroup each)
bool being_captured(hipStream_t st) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}
// A number for the marks of a call that no other call uses (from a start that a workspace's contents will not hold by chance).
unsigned long long next_mark() {
  static std::atomic<unsigned long long> counter{std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull | 1};
  return counter.fetch_add(2, std::memory_order_relaxed);
}


// The kernel that a pass of so many probes takes.
enum class Route { stream, wide, big };
Route route_of(const percache_ctx *ctx, int n_probes) {
  const int d = ctx->cfg.emb_dim;
  if (n_probes > kBatchedFrom && n_probes <= kWideUpTo && (d == 512 || d == 768 || d == 1024)) return Route::wide;
  return n_probes > kBatchedFrom ? Route::big : Route::stream;
}
struct WideShape {
  int sets, grid, per_wg;   // per_wg: blocks of sets x 32 rows
};
WideShape wide_shape(int n_cu, int N, int n_probes, int max_blocks = kWideMaxBlocksPerWg) {
  WideShape w;
  // us a call, one set | two: best of 200 000 rows of width 1024, 64 probes 91 | 75, 50 000 rows 33.5 | 30.1, 20 000 of width 512 14.3 | 15.2, 2000 of
  // width 768 12.1 | 13.6: under four blocks of 32 rows a CU, blocks of 64 leave CUs without one.
  w.sets = n_probes <= kWideProbes / 2 && N >= 4 * 32 * n_cu ? 2 : 1;
  const int n_blocks = (N + 32 * w.sets - 1) / (32 * w.sets);
  w.grid = n_cu < n_blocks ? n_cu : n_blocks;
  w.per_wg = (n_blocks + w.grid - 1) / w.grid;
  if (w.per_wg > max_blocks / w.sets) w.per_wg = max_blocks / w.sets;
  w.grid = (n_blocks + w.per_wg - 1) / w.per_wg;
  return w;
}
// Per-row scan of up to 128 new embeddings in one pass of the bank.
bool scan_in_wide_passes(int n_new, int d) { return n_new > kScanWideFrom && (d == 384 || d == 512 || d == 768 || d == 1024); }
pc_status launch_scan_wide(percache_ctx *ctx, hipStream_t st, int N, int d, const _Float16 *pp, int np, const RowScan &rs) {
  const WideShape w = wide_shape(ctx->n_cu, N, np, kScanMaxBlocksPerWg);
#define PC_SCAN_SETS(DD, RS, CC)                                                                                      \
  do {                                                                                                                \
    constexpr int lds = kScanHead + kWideStages * 32 * CC;                                                            \
    PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_wide_kernel<DD, 0, RS, CC>, hipFuncAttributeMaxDynamicSharedMemorySize, lds)); \
    hipLaunchKernelGGL((lookup_wide_kernel<DD, 0, RS, CC>), dim3(w.grid), dim3(256), lds, st, ctx->bank, ctx->bank_inv, N, pp, np, w.per_wg, (Best *)nullptr, rs, Groups{}); \
  } while (0)
#define PC_SCAN(DD, CC)                                                                                               \
  do {                                                                                                                \
    if (w.sets == 2) PC_SCAN_SETS(DD, 2, CC); else PC_SCAN_SETS(DD, 1, CC);                                           \
  } while (0)
  if (d == 384) PC_SCAN(384, 256); else if (d == 512) PC_SCAN(512, 512); else if (d == 768) PC_SCAN(768, 512); else PC_SCAN(1024, 512);
#undef PC_SCAN
#undef PC_SCAN_SETS
  PC_HIP(ctx, hipGetLastError());
  return PC_OK;
}

int probe_tile(int n_probes) { return big_tiles_pay(n_probes) ? 256 : 128; }
// The groups of a call of so many probes (see Groups) that has room for so many of a probe: about four a wavefront, in the matrix-product kernel at least
// 1024 in all; there, over a small bank, the 16 rows that a lane has in a block of 32.  Fewer, larger ones where there is no room for these.
// us a call, 8 best of 200 000 rows of width 1024, room for all | in the least workspace: 32 probes 83 | 88, 128 103 | 103, 512 249 | 299, 1024 455 | 643 (lists
// in every lane, which needed no more, 89, 179, 420, 723).
constexpr int kFineGroupsUpTo = 16384, kLeastGroups = 1024, kGroupsPerWave = 4, kGroupsPerWide = 8;
constexpr int kRowsUpToBig = kRowsUpTo / 2;
Groups groups_of(const percache_ctx *ctx, int n_probes, int N, size_t room) {
  Groups g{};
  int blocks, into, parts;   // the blocks of a wavefront (workgroup) into so many groups or a few less; wavefronts (workgroups)
  const Route r = route_of(ctx, n_probes);
  if (r == Route::stream) {
    const StreamShape sh = stream_shape(ctx, 1, N);
    g.kind = Groups::stream;
    g.per_wg = sh.per_wg;
    g.blocks = (N + 15) / 16;
    blocks = (sh.per_wg + 3) / 4, into = kGroupsPerWave, parts = sh.grid * 4;
  } else if (r == Route::wide) {
    const WideShape w = wide_shape(ctx->n_cu, N, n_probes);
    g.kind = Groups::wide;
    g.per_wg = w.per_wg;
    g.sets = w.sets;
    g.blocks = (N + 32 * w.sets - 1) / (32 * w.sets);
    blocks = w.per_wg, into = kGroupsPerWide / w.sets, parts = w.grid * w.sets;
  } else {
    const BigShape bg = big_shape(ctx->n_cu, N, n_probes, probe_tile(n_probes));
    g.kind = Groups::big;
    g.per_wg = bg.groups;
    g.blocks = (N + kBigRows - 1) / kBigRows;
    const int least = (kLeastGroups / 4 + bg.groups - 1) / bg.groups;
    blocks = (g.blocks + bg.groups - 1) / bg.groups, into = least > kGroupsPerWave ? least : kGroupsPerWave, parts = bg.groups * 4;
  }
  do {
    g.stretch = (blocks + into - 1) / into;
    g.per = (blocks + g.stretch - 1) / g.stretch;
    g.n = parts * g.per;
  } while ((size_t)g.n > room && into-- > 1);
  if (r == Route::big && N <= kFineGroupsUpTo && (size_t)g.blocks * 16 <= room) {
    g.kind = Groups::big_fine;
    g.n = g.blocks * 16;
  }
  // Every row a group: no probe is ever in doubt, which over so few rows one of them would nearly always be.  us a call, lists in every lane | groups | rows:
  // 9 probes, 2 best of 200 rows of width 768 11.3 | 13.1 | 9.2, 8 best of 1000 of width 1024 19.5 | 14.9 | 10.2, 3 best of 8000 of width 384 11.0 | 12.3 | 8.9; 128
  // probes, 3 best of 8000 of width 768 21.8 | (22.7) | 17.5; 1024 probes, 8 best of 200 44.2 | 66.9 | 28.2, of 2500 of width 1024 47.4 | 51.7 | 39.5, of
  // 4000 of width 768 44.8 | 42.5 | 37.0.  Under more than 128 probes the similarities' bytes weigh more: 600 probes, 3 best of 8000 of width 384
  // 35.7 | 26.9 | 30.6, so there half as many rows.
  if (N <= (r == Route::big ? kRowsUpToBig : kRowsUpTo) && (size_t)(N + 3) / 4 <= room) {
    g.kind = Groups::rows;
    g.n = N;
  }
  const int places = g.kind == Groups::rows ? (g.n + 3) / 4 : g.n, odd_lines = ((places + 7) / 8 | 1) * 8;
  g.pitch = (size_t)odd_lines <= room ? odd_lines : places;
  return g;
}
// The places of a probe's groups that a call of so many probes has a use for, over whatever the bank holds.
size_t group_places(const percache_ctx *ctx, int n_probes) {
  const int d = ctx->cfg.emb_dim, cus = ctx->n_cu;
  size_t n;
  if (n_probes <= kBatchedFrom) {
    n = (size_t)max_stream_grid(ctx) * 4 * kGroupsPerWave;
  } else if (n_probes <= kWideUpTo && (d == 512 || d == 768 || d == 1024)) {
    const size_t grid = (size_t)ctx->cfg.bank_capacity / (32 * kWideMaxBlocksPerWg) + 1;
    n = (grid > (size_t)cus ? grid : (size_t)cus) * kGroupsPerWide;
  } else {   // (no fewer tiles than that, so no more groups of them: see big_shape)
    const int tiles = (n_probes + 255) / 256, groups = cus / tiles > 8 ? cus / tiles : 8;
    n = 4 * (size_t)groups * kGroupsPerWave;
    const size_t least = kLeastGroups + 4 * (size_t)groups;
    n = n > least ? n : least;
  }
  const size_t rows = kRowsUpTo / 4;
  return (n > rows || n_probes > kWideUpTo ? n : rows) + 16;
}

// The passes over the bank: the best row of every probe and its hit flag (or, with il.marks, the k best), or (gm) the group maxima.
pc_status run_passes(percache_ctx *ctx, hipStream_t st, int N, const _Float16 *probes, int n_probes, float tau, int k, int32_t *idx_out_dev, float *sim_out_dev,
                     uint8_t *hit_out_dev, Best *partial, const InLaunch &il, const Groups *gm) {
  const int d = ctx->cfg.emb_dim;
  const Route route = route_of(ctx, n_probes);
  if (route == Route::wide) {
    // up to 128 probes: one pass of the bank
    const WideShape w = wide_shape(ctx->n_cu, N, n_probes);
    const size_t lds = (size_t)kWideMaxBlocksPerWg * 32 * sizeof(float) + (size_t)kWideStages * 32 * kWideChunk;
#define PC_WIDE_SETS(DD, KK, RS)                                                                                      \
  do {                                                                                                                \
    PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_wide_kernel<DD, KK, RS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
    hipLaunchKernelGGL((lookup_wide_kernel<DD, KK, RS>), dim3(w.grid), dim3(256), lds, st, ctx->bank, ctx->bank_inv, N, probes, n_probes, w.per_wg, partial, RowScan{}, \
                       gm ? *gm : Groups{});                                                                          \
  } while (0)
#define PC_WIDE(DD, KK)                                                                                               \
  do {                                                                                                                \
    if (w.sets == 2) PC_WIDE_SETS(DD, KK, 2); else PC_WIDE_SETS(DD, KK, 1);                                           \
  } while (0)
    pc::prof_begin(ctx, PC_KERNEL_LOOKUP, st);
    if (!gm) {
      if (d == 512) PC_WIDE(512, 1); else if (d == 768) PC_WIDE(768, 1); else PC_WIDE(1024, 1);
    } else if (gm->kind == Groups::rows) {
      if (d == 512) PC_WIDE(512, kRows); else if (d == 768) PC_WIDE(768, kRows); else PC_WIDE(1024, kRows);
    } else {
      if (d == 512) PC_WIDE(512, kGroups); else if (d == 768) PC_WIDE(768, kGroups); else PC_WIDE(1024, kGroups);
    }
    pc::prof_end(ctx, PC_KERNEL_LOOKUP, st);
    PC_HIP(ctx, hipGetLastError());
#undef PC_WIDE
#undef PC_WIDE_SETS
    if (gm) return PC_OK;
    hipLaunchKernelGGL(lookup_finalize_kernel, dim3(n_probes), dim3(kFinalizeThreads), 0, st, partial, w.grid * w.sets, kWideProbes / w.sets, probes, d, tau, idx_out_dev, sim_out_dev, hit_out_dev);
    PC_HIP(ctx, hipGetLastError());
    return PC_OK;
  }
  if (route == Route::big) {  // (d is a multiple of 64: percache_create checks it)
    // many probes: the matrix-core product on 256-row tiles, one workgroup per CU; 256-probe tiles where the probes
    // fill them to three quarters, else 128-probe tiles
    const int pt = probe_tile(n_probes);
    const BigShape bg = big_shape(ctx->n_cu, N, n_probes, pt);
    static bool big_lds_set = false;  // dynamic LDS above 64 KB must be opted into once
    if (!big_lds_set) {
      PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_big_kernel<256, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, BigTile<256>::LDS));
      PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_big_kernel<128, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, BigTile<128>::LDS));
      PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_big_kernel<256, kGroups>, hipFuncAttributeMaxDynamicSharedMemorySize, BigTile<256>::LDS));
      PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_big_kernel<128, kGroups>, hipFuncAttributeMaxDynamicSharedMemorySize, BigTile<128>::LDS));
      PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_big_kernel<256, kRows>, hipFuncAttributeMaxDynamicSharedMemorySize, BigTile<256>::LDS));
      PC_HIP(ctx, hipFuncSetAttribute((const void *)lookup_big_kernel<128, kRows>, hipFuncAttributeMaxDynamicSharedMemorySize, BigTile<128>::LDS));
      big_lds_set = true;
    }
    const dim3 grid((unsigned)((bg.groups + 7) / 8 * 8 * bg.p_tiles));
    pc::prof_begin(ctx, PC_KERNEL_LOOKUP, st);
#define PC_BIG(PP, KK)                                                                                                 \
  hipLaunchKernelGGL((lookup_big_kernel<PP, KK>), grid, dim3(512), (BigTile<PP>::LDS), st, ctx->bank, ctx->bank_inv, N, d, probes, n_probes, \
                     bg.p_tiles * pt, bg.groups, bg.p_tiles, partial, gm ? *gm : Groups{})
    if (!gm) { if (pt == 256) PC_BIG(256, 1); else PC_BIG(128, 1); }
    else if (gm->kind == Groups::rows) { if (pt == 256) PC_BIG(256, kRows); else PC_BIG(128, kRows); }
    else { if (pt == 256) PC_BIG(256, kGroups); else PC_BIG(128, kGroups); }
#undef PC_BIG
    pc::prof_end(ctx, PC_KERNEL_LOOKUP, st);
    PC_HIP(ctx, hipGetLastError());
    if (gm) return PC_OK;
    hipLaunchKernelGGL(lookup_finalize_kernel, dim3(n_probes), dim3(kFinalizeThreads), 0, st, partial, bg.groups, bg.p_tiles * pt, probes, d, tau,
                       idx_out_dev, sim_out_dev, hit_out_dev);
    PC_HIP(ctx, hipGetLastError());
    return PC_OK;
  }
  // two probe blocks per pass unless their LDS copy leaves no room for the rings (very wide embeddings)
  const int pass_probes = stream_shape(ctx, 2, N).lds <= kMaxLds ? kPassProbes : 16;
  for (int p0 = 0; p0 < n_probes; p0 += pass_probes) {
    int np = n_probes - p0 < pass_probes ? n_probes - p0 : pass_probes;
    int npb = np <= 16 ? 1 : 2;
    StreamShape sh = stream_shape(ctx, npb, N);
    const _Float16 *pp = probes + (size_t)p0 * d;
    pc::prof_begin(ctx, PC_KERNEL_LOOKUP, st);
    const Groups here = gm ? gm->from_probe(p0) : Groups{};
    // (up to four best rows in one launch: lists of four; kInLaunchProbes and 1024 elements leave room for three stages)
    pc_status ls = gm && here.kind == Groups::rows ? launch_pass<kRows>(ctx, sh, npb, st, N, d, pp, np, partial, RowScan{}, il, here)
                   : gm                             ? launch_pass<kGroups>(ctx, sh, npb, st, N, d, pp, np, partial, RowScan{}, il, here)
                   : k == 1                         ? launch_pass<1>(ctx, sh, npb, st, N, d, pp, np, partial, RowScan{}, il)
                                                    : launch_one_block<4>(ctx, sh, st, N, d, pp, np, partial, RowScan{}, il, Groups{});
    if (ls != PC_OK) return ls;
    pc::prof_end(ctx, PC_KERNEL_LOOKUP, st);
    PC_HIP(ctx, hipGetLastError());
    if (il.marks || gm) continue;
    hipLaunchKernelGGL(lookup_finalize_kernel, dim3(np), dim3(kFinalizeThreads), 0, st, partial, sh.grid, npb * 16, pp, d, tau, idx_out_dev + p0, sim_out_dev + p0,
                       hit_out_dev + p0);
    PC_HIP(ctx, hipGetLastError());
  }
  return PC_OK;
}

// k best rows per probe (k == 1: the query-level match with its hit flag; hit_out may be null otherwise)
pc_status run_lookup(percache_ctx *ctx, const void *probes_dev, int32_t n_probes, float tau, int k, int32_t *idx_out_dev,
                     float *sim_out_dev, uint8_t *hit_out_dev, void *workspace_dev, size_t workspace_bytes, void *stream) {
  if (!ctx) return PC_EINVAL;
  const percache_config &c = ctx->cfg;
  if (c.bank_capacity <= 0) return pc::fail(ctx, PC_ESHAPE, "context was created without a bank");
  if (n_probes < 0) return pc::fail(ctx, PC_EINVAL, "n_probes is negative");
  if (k < 1 || k > kMaxTopK) return pc::fail(ctx, PC_ESHAPE, "k = %d outside [1,%d]", k, kMaxTopK);
  if (n_probes == 0) return PC_OK;
  if (!probes_dev || !idx_out_dev || !sim_out_dev || (k == 1 && !hit_out_dev)) return pc::fail(ctx, PC_EINVAL, "NULL probe or output pointer");
  if ((uintptr_t)probes_dev % 16) return pc::fail(ctx, PC_EINVAL, "probes_dev must be 16-byte aligned");
  if (!(tau == tau)) return pc::fail(ctx, PC_EINVAL, "tau is NaN");
  hipStream_t st = (hipStream_t)stream;
  const int N = ctx->bank_size, d = c.emb_dim;
  if (N == 0) {
    const int n_out = n_probes * k;
    hipLaunchKernelGGL(lookup_empty_kernel, dim3((n_out + 255) / 256), dim3(256), 0, st, n_out, n_probes, idx_out_dev, sim_out_dev, hit_out_dev);
    PC_HIP(ctx, hipGetLastError());
    return PC_OK;
  }
  const size_t need = list_bytes(ctx, n_probes);
  if (!workspace_dev || workspace_bytes < need) return pc::fail(ctx, PC_ENOMEM, "lookup workspace has %zu bytes, need %zu", workspace_bytes, need);
  if ((uintptr_t)workspace_dev % 16) return pc::fail(ctx, PC_EINVAL, "workspace must be 16-byte aligned");
  Best *partial = (Best *)workspace_dev;
  const _Float16 *probes = (const _Float16 *)probes_dev;
  if (stream_shape(ctx, 1, N).lds > kMaxLds && n_probes <= kBatchedFrom)   // (checked before anything is enqueued)
    return pc::fail(ctx, PC_ESHAPE, "emb_dim %d needs %zu bytes of LDS per workgroup", d, stream_shape(ctx, 1, N).lds);
  InLaunch il{};
  if (k <= 4 && n_probes <= kInLaunchProbes && d <= 1024 && workspace_dev != ctx->static_scratch) {
    // A short pass over a small bank merges its lists itself (the marks behind the lists, which one probe block leaves room for): what it saves is a
    // launch, a third of the host's work, what it costs is 0.7 us of the GPU's and, past a probe a wavefront, a second round.  us a call, calls one after
    // the other, the merge apart | here, 2000 rows of width 768: best row of 1 probe 11.6 | 8.7, of 4 11.6 | 8.9, of 8 10.7 | 10.8, 4 best of 1 13.8 | 12.2,
    // of 8 14.0 | 16.3; 4096 rows of width 1024: best row of 1 11.7 | 9.6, 5 best of 4 17.2 | 17.6; of width 2048, where the GPU is behind the host
    // either way: best row of 1 11.7 | 12.5.  Waited for: 2000 rows of width 768, best row of 1 23.7 | 24.0, 4 best of 1 about 31 | 30.5.  A captured
    // call has paid for its launches (best row of 1 8.1 | 8.8, 4 best of 4 12.7 | 12.9), and so no mark is ever used twice.  With more lists than
    // lanes (20 000 rows, 256 lists) the merge here is the slower one from two best on, and behind a long stream the launch apart is hidden.
    const StreamShape sh = stream_shape(ctx, 1, N);
    if (sh.grid <= kInLaunchGrid && !being_captured(st))
      il = InLaunch{(unsigned long long *)(partial + (size_t)sh.grid * 16 * (k == 1 ? 1 : 4)), next_mark(), tau, k, idx_out_dev, sim_out_dev, hit_out_dev};
  }
  if (k == 1 || il.marks) return run_passes(ctx, st, N, probes, n_probes, tau, k, idx_out_dev, sim_out_dev, hit_out_dev, partial, il, nullptr);
  // A workspace with room for less than 256 groups of a probe takes the probes in turns (of equal size, 64 or more, so that none is another kernel's): 4096
  // probes, 8 best of 200 000 rows of width 1024 in the least workspace, at once 4870 us, in turns 2390 (lists in every lane 2290, room for all 1640).
  constexpr int kLeastRoom = 256, kTurnRoom = 512;
  const size_t places = workspace_bytes / sizeof(Group);
  const int per_probe = N < kTurnRoom * 16 ? (N + 15) / 16 : kTurnRoom;
  long turns = places / (size_t)n_probes >= (size_t)kLeastRoom ? 1 : (long)(((size_t)n_probes * per_probe + places - 1) / places);
  if (turns > n_probes / 64) turns = n_probes < 64 ? 1 : n_probes / 64;
  for (long t = 0; t < turns; ++t) {
    const int p0 = (int)(t * n_probes / turns), np = (int)((t + 1) * n_probes / turns) - p0;
    Groups gm = groups_of(ctx, np, N, places / (size_t)np);
    gm.g = (Group *)workspace_dev;
    const pc_status ls = run_passes(ctx, st, N, probes + (size_t)p0 * d, np, tau, k, nullptr, nullptr, nullptr, nullptr, InLaunch{}, &gm);
    if (ls != PC_OK) return ls;
    auto *const select = gm.kind == Groups::rows ? topk_groups_kernel<true> : topk_groups_kernel<false>;
    hipLaunchKernelGGL(select, dim3(np), dim3(kSelectThreads), 0, st, gm, ctx->bank, ctx->bank_inv, N, d, probes + (size_t)p0 * d, k,
                       idx_out_dev + (size_t)p0 * k, sim_out_dev + (size_t)p0 * k);
    PC_HIP(ctx, hipGetLastError());
  }
  return PC_OK;
}

}  // namespace

extern "C" {

pc_status percache_bank_put(percache_ctx *ctx, int32_t index, const void *emb_dev, int32_t n, void *stream) {
  if (!ctx) return PC_EINVAL;
  const percache_config &c = ctx->cfg;
  if (c.bank_capacity <= 0) return pc::fail(ctx, PC_ESHAPE, "context was created without a bank");
  if (!emb_dev) return pc::fail(ctx, PC_EINVAL, "emb_dev is NULL");
  if ((uintptr_t)emb_dev % 16) return pc::fail(ctx, PC_EINVAL, "emb_dev must be 16-byte aligned");
  if (n < 1) return pc::fail(ctx, PC_EINVAL, "n must be positive");
  if (index < 0 || index > ctx->bank_size) return pc::fail(ctx, PC_EINVAL, "index %d outside [0,%d] (no holes allowed)", index, ctx->bank_size);
  if ((long)index + n > c.bank_capacity) return pc::fail(ctx, PC_ENOMEM, "rows [%d,%ld) exceed bank capacity %d", index, (long)index + n, c.bank_capacity);
  hipLaunchKernelGGL(bank_put_kernel, dim3((n + 3) / 4), dim3(256), 0, (hipStream_t)stream, (const _Float16 *)emb_dev,
                     ctx->bank + (size_t)index * c.emb_dim, ctx->bank_inv + index, n, c.emb_dim);
  PC_HIP(ctx, hipGetLastError());
  if (index + n > ctx->bank_size) ctx->bank_size = index + n;
  return PC_OK;
}

size_t percache_lookup_workspace_bytes(const percache_ctx *ctx, int32_t n_probes) {
  if (!ctx || n_probes < 0) return 0;
  return list_bytes(ctx, n_probes);
}

size_t percache_lookup_topk_workspace_bytes(const percache_ctx *ctx, int32_t n_probes) {
  if (!ctx || n_probes < 0) return 0;
  // (not less for more probes, so that the workspace of a longer call is as good; past 4096 the groups are larger instead)
  size_t places = 0;
  for (const int upto : {kBatchedFrom, kWideUpTo, 256, 512, 768, 1024, 4096}) {
    const int n = n_probes < upto ? n_probes : upto;
    const size_t p = (size_t)n * group_places(ctx, n);
    places = places > p ? places : p;
  }
  const size_t bytes = places * sizeof(Group), lists = list_bytes(ctx, n_probes);
  return pc::align_up(bytes > lists ? bytes : lists);
}

pc_status percache_lookup(percache_ctx *ctx, const void *probes_dev, int32_t n_probes, float tau, int32_t *idx_out_dev,
                          float *sim_out_dev, uint8_t *hit_out_dev, void *workspace_dev, size_t workspace_bytes,
                          void *stream) {
  return run_lookup(ctx, probes_dev, n_probes, tau, 1, idx_out_dev, sim_out_dev, hit_out_dev, workspace_dev, workspace_bytes, stream);
}

pc_status percache_lookup_noalloc(percache_ctx *ctx, const void *probes_dev, int32_t n_probes, float tau,
                                  int32_t *idx_out_dev, float *sim_out_dev, uint8_t *hit_out_dev, void *stream) {
  if (!ctx) return PC_EINVAL;
  if (n_probes > kPassProbes)
    return pc::fail(ctx, PC_ESHAPE, "percache_lookup_noalloc takes at most %d probes per call, got %d", kPassProbes, n_probes);
  const size_t need = list_bytes(ctx, n_probes < 0 ? 0 : n_probes);
  if (need > pc::kStaticScratchBytes)
    return pc::fail(ctx, PC_ESHAPE, "a bank of %d rows needs %zu bytes of scratch, the library's static scratch holds %zu",
                    ctx->cfg.bank_capacity, need, pc::kStaticScratchBytes);
  if (!ctx->static_scratch) return pc::fail(ctx, PC_EHIP, "static scratch was not resolved on this device");
  // nothing in the scratch has to start at zero: every workgroup of a pass writes all of its lists before the
  // finalize kernel (next on the stream) reads exactly those
  return run_lookup(ctx, probes_dev, n_probes, tau, 1, idx_out_dev, sim_out_dev, hit_out_dev, ctx->static_scratch,
                    pc::kStaticScratchBytes, stream);
}

pc_status percache_bank_refresh_scan(percache_ctx *ctx, const void *new_emb_dev, int32_t n_new, const float *kth_sim_dev,
                                     float *best_sim_out_dev, int32_t *best_new_out_dev, uint8_t *stale_out_dev,
                                     void *workspace_dev, size_t workspace_bytes, void *stream) {
  if (!ctx) return PC_EINVAL;
  const percache_config &c = ctx->cfg;
  if (c.bank_capacity <= 0) return pc::fail(ctx, PC_ESHAPE, "context was created without a bank");
  if (n_new < 1) return pc::fail(ctx, PC_EINVAL, "n_new must be positive");
  if (!new_emb_dev || !kth_sim_dev || !best_sim_out_dev || !best_new_out_dev || !stale_out_dev) return pc::fail(ctx, PC_EINVAL, "NULL pointer");
  if ((uintptr_t)new_emb_dev % 16) return pc::fail(ctx, PC_EINVAL, "new_emb_dev must be 16-byte aligned");
  const int N = ctx->bank_size, d = c.emb_dim;
  if (N == 0) return PC_OK;  // nothing to mark
  const size_t need = list_bytes(ctx, n_new);
  if (!workspace_dev || workspace_bytes < need || (size_t)n_new * sizeof(float) > need)
    return pc::fail(ctx, PC_ENOMEM, "workspace has %zu bytes, need %zu (and at most %zu new rows per call)", workspace_bytes, need, need / sizeof(float));
  if ((uintptr_t)workspace_dev % 16) return pc::fail(ctx, PC_EINVAL, "workspace must be 16-byte aligned");
  {
    const size_t lds1 = stream_shape(ctx, 1, N).lds;
    if (lds1 > kMaxLds) return pc::fail(ctx, PC_ESHAPE, "emb_dim %d needs %zu bytes of LDS per workgroup", d, lds1);
  }
  hipStream_t st = (hipStream_t)stream;
  const _Float16 *probes = (const _Float16 *)new_emb_dev;
  int p0 = 0;
  // (one kernel for all passes of a call: equal embeddings then have equal sums, and the lower index wins)
  for (; p0 < n_new && scan_in_wide_passes(n_new, d); p0 += kWideProbes) {
    const int np = n_new - p0 < kWideProbes ? n_new - p0 : kWideProbes;
    const RowScan rs{kth_sim_dev, best_sim_out_dev, best_new_out_dev, stale_out_dev, p0, p0 == 0 ? 1 : 0};
    const pc_status ls = launch_scan_wide(ctx, st, N, d, probes + (size_t)p0 * d, np, rs);
    if (ls != PC_OK) return ls;
  }
  const int pass_probes = stream_shape(ctx, 2, N).lds <= kMaxLds ? kPassProbes : 16;
  for (; p0 < n_new; p0 += pass_probes) {
    const int np = n_new - p0 < pass_probes ? n_new - p0 : pass_probes;
    const int npb = np <= 16 ? 1 : 2;
    StreamShape sh = stream_shape(ctx, npb, N);
    RowScan rs{kth_sim_dev, best_sim_out_dev, best_new_out_dev, stale_out_dev, p0, p0 == 0 ? 1 : 0};
    pc_status ls = launch_pass<0>(ctx, sh, npb, st, N, d, probes + (size_t)p0 * d, np, nullptr, rs);
    if (ls != PC_OK) return ls;
    PC_HIP(ctx, hipGetLastError());
  }
  return PC_OK;
}

pc_status percache_lookup_topk(percache_ctx *ctx, const void *probes_dev, int32_t n_probes, int32_t k, int32_t *idx_out_dev,
                               float *sim_out_dev, void *workspace_dev, size_t workspace_bytes, void *stream) {
  return run_lookup(ctx, probes_dev, n_probes, 0.f, k, idx_out_dev, sim_out_dev, nullptr, workspace_dev, workspace_bytes, stream);
}

}  // extern "C"
