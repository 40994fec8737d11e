// prefill_sparse_attention on bf16 caches: attention for a block of prompt tokens that share key tiles.
//
// Every token of the block attends its sink and recent keys and the members of its own listed buckets (the rule of
// arXiv 2502.08246 for decoding: Section 3 "Per-head attention span", Section 4 "Beyond top-k", one list per group as in
// Section 5).  Token by token, the keys of a bucket are read once for every token that lists it (at 128 tokens with 5 % of
// 1024 buckets each: 6 times, 4.4 GB for a block whose cache holds 0.54 GB).  Here the work is turned round:
//   1. invert  per (sequence, KV head) the lists become, for every bucket, the tokens that list it, cut into tiles of
//              32 query rows (32 / G tokens with their G heads);
//   2. attend  a wave takes one (bucket, tile): scores S^T = K Q^T and values O = P V on v_mfma_f32_32x32x16_bf16, the
//              keys read once per tile; the result (maximum, sum, O) of each row goes to its token's slot for that bucket.
//              Sink and recent keys are a few more slots per token, attended from the position-ordered tensors in tiles of
//              consecutive tokens.  The four waves of a workgroup share out the key tiles of a long bucket;
//   3. merge   the slots of every (token, KV head) are combined (Algorithm 2).
// HBM-bound: the cache once, plus the slots (G * 520 bytes per token and listed bucket, written and read).  128 tokens, 32
// heads on 8, 51 of 1024 buckets of 131072 keys: 590 us token by token, here 7 + 125 + 22 (0.54 GB of keys and 0.12 GB of
// slots at 5.3 TB/s, then the slots at 5.6); 512 tokens: 2200 -> 460; 16 tokens: 91 -> 70.
//
// The matrix operands come straight from memory, without LDS.  K: lane (key, half) loads 16-byte pieces of its key's row.
// Scores leave the matrix cores with lane (query, half) holding keys 8*(r/4) + 4*half + r%4 of a 32-key tile, and the keys
// of 16 that a lane of the next product contributes are taken to be exactly those (registers 8g .. 8g+7 for group g), so
// weights need no exchange between lanes; V: lane (n, half) loads features 4n .. 4n+3 of those eight keys (whole rows per
// 32 lanes), regrouped by feature with v_perm_b32, one product per feature e of the four; column n of product e is
// feature 4n + e, so that a lane's four accumulators hold four neighbouring features.  A weight enters as two bf16 parts
// (16 significant bits), as in the decode kernels.
#include "common.h"

namespace saap {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __bf16 bf16x2v_t __attribute__((ext_vector_type(2)));

constexpr int kMaxSplits = 16;        // slots of a token's sink and recent keys, at most
constexpr int kLongRun = 384;         // keys from which a bucket is shared out over the four waves of a workgroup
constexpr int kMaxSlots = 1024;       // slots per token (the merge keeps their weights in LDS)
constexpr int kInvertThreads = 1024, kInvertParts = 8;
static_assert(kInvertThreads * kInvertParts >= SAAP_MAX_BUCKETS, "a thread per bucket");
// Counters, a cache line each.  The short tiles are dealt to kQueues queues (four tiles here, four there, so that the tiles
// of a bucket stay in one L2), a workgroup takes from the one of its number: thousands of takings from one address cost more
// than they are for (ten thousand from one: this kernel 211 us instead of 131).
constexpr int kQueues = 32, kLine = 32;
enum { kCountItems, kCountShort, kCountLong, kQueue0, kCounters = kQueue0 + kQueues };
static_assert(kCounters * kLine * sizeof(unsigned) <= SAAP_WS_HEADER_BYTES, "the header holds the counters");

struct BlockParams {
  const bf16_t *q, *K, *V, *Ks, *Vs;  // [S,Tq,Hq,d]; position-ordered [S,Hkv,Nt,d]; sorted [S,Hkv,Ncap,d]
  const int32_t *off, *len, *idx, *selected, *pos0;
  void* out;
  float* lse;
  unsigned* counters;                 // kCounters, zero on entry and on exit
  int* items;                         // [kv units * Tq * nprobe]: token << 13 | place in its list, grouped by (kv unit, bucket)
  int4* tiles;                        // [2 * kv units * Tq * nprobe]: short tiles from the front, long ones from the back; two int4 each
  float2* part_ml;                    // [units * slots][G]
  float* part_o;                      // [units * slots][G][d]
  long long n_items_all;              // kv units * Tq * nprobe
  int S, Hq, Hkv, Tq, Nt, Ncap, B, nprobe, splits, slots, n_sink, n_recent, out_bf16;
  float scale_log2;
};

// What the token at t of sequence s sees: sink keys [0, sink), recent keys [recent, end), bucket members in between.
struct Span { int sink, recent, end; };
__device__ __forceinline__ Span token_span(const BlockParams& p, int s, int t) {
  Span w;
  w.end = min(max(p.pos0[s] + t + 1, 0), p.Nt);
  w.sink = min(p.n_sink, w.end);
  w.recent = max(w.sink, w.end - p.n_recent);
  return w;
}

// ---- 1. the lists of a (sequence, KV head) by bucket ------------------------------------------------------
// A tile: {kv unit, first item, tokens, first row of the bucket} {keys, -, -, -}.
// A workgroup per kv unit and kInvertParts-th of its buckets, one bucket a thread: all of them read the unit's lists (from
// L2), and the counting in LDS, two atomics per listed bucket, is what takes the time (a workgroup per kv unit: 12.5 us for
// 128 tokens with 51 buckets each, here 7).  Where a workgroup's items and tiles
// go comes from three counters, so their order varies; no result depends on it.
template <int TT /* tokens per tile */>
__global__ void __launch_bounds__(kInvertThreads)
block_invert_kernel(BlockParams p) {
  __shared__ int s_cnt[kInvertThreads];                  // tokens of a bucket, then its next free item
  __shared__ int s_sum[3][16];
  __shared__ int s_base[3];
  const int kvu = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_items = p.Tq * p.nprobe;
  const int32_t* __restrict__ sel = p.selected + (size_t)kvu * n_items;
  const int per = (p.B + kInvertParts - 1) / kInvertParts, b0 = blockIdx.y * per, nb = min(per, p.B - b0);
  const bool mine = tid < nb;
  const int b_at = mine ? b0 + tid : 0;
  const int len = p.len[(size_t)kvu * p.B + b_at], off = p.off[(size_t)kvu * (p.B + 1) + b_at];
  s_cnt[tid] = 0;
  __syncthreads();
  // f(item, place among the workgroup's buckets) for every item of theirs, eight loads in flight
  auto for_items = [&](auto f) {
    for (int i0 = tid; i0 < n_items; i0 += 8 * kInvertThreads) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = sel[min(i0 + u * kInvertThreads, n_items - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + u * kInvertThreads, b = min(max(v[u], 0), p.B - 1) - b0;
        if (i < n_items && b >= 0 && b < nb) f(i, b);
      }
    }
  };
  for_items([&](int, int b) { atomicAdd(&s_cnt[b], 1); });
  __syncthreads();
  const int c = s_cnt[tid], kind = len > kLongRun ? 1 : 0, tiles = (c + TT - 1) / TT;
  int run[3] = {c, kind ? 0 : tiles, kind ? tiles : 0};
#pragma unroll
  for (int k = 0; k < 3; ++k) {                          // exclusive prefixes over the buckets: items, short tiles, long tiles
    const int own = run[k], incl = (int)wave_prefix_sum((unsigned)own);
    run[k] = incl - own;
    if (lane == 63) s_sum[k][wave] = incl;
  }
  __syncthreads();
  if (tid < 3) {
    int total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) total += s_sum[tid][w];
    s_base[tid] = (int)atomicAdd(p.counters + tid * kLine, (unsigned)total);
  }
#pragma unroll
  for (int w = 0; w < 15; ++w)
#pragma unroll
    for (int k = 0; k < 3; ++k) run[k] += w < wave ? s_sum[k][w] : 0;
  __syncthreads();
  const int first = min(max(off, 0), p.Ncap - 1);
  const int n = min(max(len, 0), p.Ncap - first);        // a damaged index must not turn into a read outside the cache
  run[0] += s_base[0];
  s_cnt[tid] = run[0];
  for (int k = 0; k < tiles; ++k) {
    const int at = s_base[1 + kind] + run[1 + kind] + k;
    int4* tile = p.tiles + 2 * (kind ? p.n_items_all - 1 - at : (long long)at);
    tile[0] = make_int4(kvu, run[0] + k * TT, min(TT, c - k * TT), first);
    tile[1] = make_int4(n, 0, 0, 0);
  }
  __syncthreads();
  // the tokens of a bucket in any order: a row's result does not depend on its place in the tile
  const float inv = 1.0f / (float)p.nprobe;
  for_items([&](int i, int b) {
    int t = (int)((float)i * inv), j = i - t * p.nprobe;  // i / nprobe, at most one off
    if (j < 0) { --t; j += p.nprobe; }
    if (j >= p.nprobe) { ++t; j -= p.nprobe; }
    p.items[atomicAdd(&s_cnt[b], 1)] = (t << 13) | j;
  });
}

// ---- 2. attention of one wave over the key tiles of a run ---------------------------------------------------
// The 32 query rows of a tile as the B operand, their state and their outputs (row r of an accumulator register: see
// row_of; column = lane % 32, half = lane / 32).
struct WaveTile {
  bf16x8_t q[8];
  float m, l;                         // lane (query, half): running reference and the half's sum of weights
  f32x16_t o[4];                      // register r: query row_of(r), features 4 * column + e
  __device__ __forceinline__ void clear() {
    m = kNegBig;
    l = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (f32x16_t){0};
  }
};
__device__ __forceinline__ int row_of(int r, int half) { return 8 * (r / 4) + 4 * half + (r % 4); }
// x of the lanes of the row that register r holds (`per` lanes of a row's token share it)
template <int per = 1>
__device__ __forceinline__ int row_value(int x, int r, int half) {
  const int a = __builtin_amdgcn_readlane(x, row_of(r, 0) / per * per), b = __builtin_amdgcn_readlane(x, row_of(r, 1) / per * per);
  return half ? b : a;
}
// the larger of a lane's value and that of the lane 32 away
__device__ __forceinline__ float max_halves(float x) {
  const unsigned u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
  const unsigned u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// A run of n keys as a buffer: 32-bit offsets, the tile's in a register and the lane's eight rows in the instruction, and
// rows past its end read as zeros without a comparison.
// (The address is the same in every lane; the compiler has to be told so.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t run_buffer(const bf16_t* rows, int n) {
  const unsigned long long at = reinterpret_cast<unsigned long long>(rows);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)at), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(at >> 32));
  rows = reinterpret_cast<const bf16_t*>(((unsigned long long)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(rows), 0, (unsigned)n * kD * (unsigned)sizeof(bf16_t), 0x00027000);
}

// Whether either half of a word is an infinity or a NaN.
__device__ __forceinline__ bool no_number(unsigned x) { return ((x & 0x7f80u) == 0x7f80u) | ((x & 0x7f800000u) == 0x7f800000u); }
// Infinities and NaNs among a tile's values become zeros; whether there were any.
__device__ __forceinline__ bool zero_no_numbers(u32x2_t (&vr)[16]) {
  typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
  u16x2_t top = {0, 0};                                  // the largest exponent of either half
#pragma unroll
  for (int i = 0; i < 32; ++i) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2_t, vr[i / 2][i % 2] & 0x7f807f80u));
  if (__builtin_expect(__ballot(top[0] == 0x7f80 || top[1] == 0x7f80) == 0ull, 1)) return false;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const unsigned x = vr[i / 2][i % 2];
    vr[i / 2][i % 2] = x & (((x & 0x7f80u) == 0x7f80u ? 0u : 0x0000ffffu) | ((x & 0x7f800000u) == 0x7f800000u ? 0u : 0xffff0000u));
  }
  return true;
}

// Keys [k0, k1) at K, V in tiles of 32, every `stride`-th key a tile's first.  The query of lane `col` attends the keys whose
// position (pos[k], or k itself) is in [lo, hi); keys in [safe0, safe1) are in every query's range.
constexpr int kPosRegs = kLongRun / 64;
struct Run {
  const bf16_t *K, *V;
  const int32_t* pos;
  int k0, k1, lo, hi, safe0, safe1;
};

// A key outside a query's range has weight zero, and zero times an infinity or a NaN is no zero: where a tile's queries differ
// in what they see, such values are zeroed and added afterwards, by a second walk that ordinary values never come to (taken
// inside the loop it cost the loop its registers: 128 tokens over 128k keys 193.5 -> 199.9 us, this way 193.3 -> 194.4).
// The reference m of a row moves only when one of its scores is more than 8 (2^8 in weight) above it, so that the outputs are
// rescaled (an exchange over the lanes) once or twice per run; by the row's own scores alone, whoever shares its tile.
__device__ __forceinline__ void attend_run(WaveTile& w, const Run& run, int stride, float scale_log2, float* s_w /* [32][32] */,
                                           const int* s_pos = nullptr) {
  const int k0 = __builtin_amdgcn_readfirstlane(run.k0), k1 = __builtin_amdgcn_readfirstlane(run.k1);
  const int safe0 = __builtin_amdgcn_readfirstlane(run.safe0), safe1 = __builtin_amdgcn_readfirstlane(run.safe1);
  if (k0 >= k1) return;
  constexpr int kRow = kD * (int)sizeof(bf16_t);
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const __amdgpu_buffer_rsrc_t kb = run_buffer(run.K, k1), vbuf = run_buffer(run.V, k1);
  const int k_at = col * kRow + half * 16, v_at = half * 4 * kRow + col * 8;
  u32x4_t kr[8];
  u32x2_t vr[16];
  auto load_k = [&](int t) {
#pragma unroll
    for (int st = 0; st < 8; ++st) kr[st] = __builtin_amdgcn_raw_buffer_load_b128(kb, k_at + t * kRow + st * 32, 0, 0);
  };
  auto load_v = [&](int t) {
#pragma unroll
    for (int i = 0; i < 16; ++i)       // slot i % 8 of key group i / 8
      vr[i] = __builtin_amdgcn_raw_buffer_load_b64(vbuf, v_at + t * kRow + (16 * (i / 8) + (i % 8 < 4 ? i % 8 : i % 8 + 4)) * kRow, 0, 0);
  };
  auto edge = [&](int t) { return t < safe0 || min(t + 32, k1) > safe1; };         // some key is outside some query's range
  auto position = [&](int t) {
    const int key = min(t + col, k1 - 1);
    return s_pos ? s_pos[key] : run.pos ? run.pos[key] : key;
  };
  auto mask = [&](f32x16_t& s, int t) {
    if (t + 32 > k1)                                     // the run's last tile
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = t + row_of(r, half) >= k1 ? -INFINITY : s[r];
    if (edge(t)) {
      const int pos = position(t);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int pk = row_value(pos, r, half);
        s[r] = (pk < run.lo) | (pk >= run.hi) ? -INFINITY : s[r];
      }
    }
  };
  auto highest = [&](const f32x16_t& s) {
    float top = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) top = fmaxf(top, s[r]);
    return max_halves(top);
  };
  const float m_before = w.m;
  bool no_numbers = false;
  load_k(k0);
  load_v(k0);
  for (int t = k0; t < k1; t += stride) {
    const int nxt = t + stride;                          // past the end: zeros nobody uses
    f32x16_t s = {0};
#pragma unroll
    for (int st = 0; st < 8; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kr[st]), w.q[st], s, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_k(nxt);                                         // in flight under the softmax and the value product
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] *= scale_log2;
    mask(s, t);
    const float top = highest(s);
    if (__ballot(top > w.m + 8.f) != 0ull) {
      const float mn = top > w.m + 8.f ? top : w.m, alpha = fast_exp2(w.m - mn);
      w.m = mn;
      w.l *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float a = __int_as_float(row_value(__float_as_int(alpha), r, half));
#pragma unroll
        for (int e = 0; e < 4; ++e) w.o[e][r] *= a;
      }
    }
    float add[4];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = fast_exp2(s[r] - w.m);
      add[r % 4] = r < 4 ? s[r] : add[r % 4] + s[r];
    }
    w.l += (add[0] + add[1]) + (add[2] + add[3]);
    if (edge(t)) no_numbers |= zero_no_numbers(vr);      // zero times an infinity or a NaN is no zero
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      unsigned ph[4], pl[4];                             // weights of the lane's eight keys: upper halves, and the rest rounded
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned u0 = __float_as_uint(s[8 * g + 2 * i]), u1 = __float_as_uint(s[8 * g + 2 * i + 1]);
        typedef float f32x2_t __attribute__((ext_vector_type(2)));
        const f32x2_t rest = {s[8 * g + 2 * i] - __uint_as_float(u0 & 0xffff0000u), s[8 * g + 2 * i + 1] - __uint_as_float(u1 & 0xffff0000u)};
        ph[i] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        pl[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(rest, bf16x2v_t));
      }
      const bf16x8_t a_hi = __builtin_bit_cast(bf16x8_t, (u32x4_t){ph[0], ph[1], ph[2], ph[3]});
      const bf16x8_t a_lo = __builtin_bit_cast(bf16x8_t, (u32x4_t){pl[0], pl[1], pl[2], pl[3]});
      bf16x8_t vb[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        u32x4_t b;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          b[i] = __builtin_amdgcn_perm(vr[8 * g + 2 * i + 1][e / 2], vr[8 * g + 2 * i][e / 2], e % 2 ? 0x07060302u : 0x05040100u);
        vb[e] = __builtin_bit_cast(bf16x8_t, b);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) w.o[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_hi, vb[e], w.o[e], 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) w.o[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_lo, vb[e], w.o[e], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    load_v(nxt);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (__builtin_expect(!no_numbers, 1)) return;
  // The run's edge tiles held infinities or NaNs: they are added here, to the rows that attend them and with the weights
  // that the walk above had (the same steps again), one key at a time.
  float m = m_before;
#pragma unroll 1
  for (int t = k0; t < k1; t += stride) {
    load_k(t);
    f32x16_t s = {0};
#pragma unroll
    for (int st = 0; st < 8; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kr[st]), w.q[st], s, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] *= scale_log2;
    mask(s, t);
    const float top = highest(s);
    m = top > m + 8.f ? top : m;
    if (!edge(t)) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) s_w[row_of(r, half) * 32 + col] = fast_exp2(s[r] - m);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int pos = position(t);
#pragma unroll 1
    for (int key = 0; key < min(32, k1 - t); ++key) {
      const int pk = __builtin_amdgcn_readlane(pos, key);
      const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(vbuf, (t + key) * kRow + col * 8, 0, 0);
      if (__ballot(no_number(v[0]) | no_number(v[1])) == 0ull) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float wt = s_w[key * 32 + row_of(r, half)], hi = __uint_as_float(__float_as_uint(wt) & 0xffff0000u);
        const bool in = pk >= row_value(run.lo, r, half) && pk < row_value(run.hi, r, half);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = e % 2 ? bf16_hi(v[e / 2]) : bf16_lo(v[e / 2]);
          if (in && !(fabsf(x) < INFINITY)) w.o[e][r] += x * hi + x * (wt - hi);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// Four waves that attended parts of the same rows: their states and outputs end up, combined, in wave 0.
__device__ __forceinline__ void combine_waves(WaveTile& w, float* s_ml /* [2][4][32] */, float* s_o /* [2][32 * d] */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  w.l = sum_halves(w.l);
  __syncthreads();
  if (half == 0) {
    s_ml[wave * 32 + col] = w.m;
    s_ml[128 + wave * 32 + col] = w.l;
  }
  __syncthreads();
  auto top_of = [&](int row) { return fmaxf(fmaxf(s_ml[row], s_ml[32 + row]), fmaxf(s_ml[64 + row], s_ml[96 + row])); };
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = row_of(r, half);
    const float a = fast_exp2(s_ml[wave * 32 + row] - top_of(row));
#pragma unroll
    for (int e = 0; e < 4; ++e) w.o[e][r] *= a;
  }
  const float M = top_of(col);
  float L = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) L = fmaf(fast_exp2(s_ml[i * 32 + col] - M), s_ml[128 + i * 32 + col], L);
  w.m = M;
  w.l = half == 0 ? L : 0.f;                             // wave 0's lanes hand it on as the sum over the halves
  // waves 2 and 3 to 0 and 1, then 1 to 0
#pragma unroll
  for (int step = 2; step > 0; step >>= 1) {
    if (wave >= step && wave < 2 * step) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        *reinterpret_cast<float4*>(s_o + (wave - step) * 32 * kD + row_of(r, half) * kD + col * 4) = make_float4(w.o[0][r], w.o[1][r], w.o[2][r], w.o[3][r]);
    }
    __syncthreads();
    if (wave < step) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float4 v = *reinterpret_cast<const float4*>(s_o + wave * 32 * kD + row_of(r, half) * kD + col * 4);
        w.o[0][r] += v.x; w.o[1][r] += v.y; w.o[2][r] += v.z; w.o[3][r] += v.w;
      }
    }
    __syncthreads();
  }
}

// A bucket's tile as the kernels read it: the same in every lane.
struct BucketTile { int kvu, item0, tokens, row, n; };
__device__ __forceinline__ BucketTile read_tile(const BlockParams& p, long long at) {
  const int4 a = p.tiles[2 * at];
  const int n = p.tiles[2 * at + 1].x;
  return BucketTile{__builtin_amdgcn_readfirstlane(a.x), __builtin_amdgcn_readfirstlane(a.y), __builtin_amdgcn_readfirstlane(a.z),
                    __builtin_amdgcn_readfirstlane(a.w), __builtin_amdgcn_readfirstlane(n)};
}

// Members are stored in ascending position: those some query of the tile attends are [k_lo, k_hi), those every query attends
// [s_lo, s_hi).  What a token sees moves up with its place, so the first and the last token of the tile bound both.
struct Bounds {
  Span sp, lo, hi;                    // the lane's query; the tile's first and last token
  int k_lo, s_lo, s_hi, k_hi;
  __device__ __forceinline__ Bounds(const BlockParams& p, int s, int t) {
    sp = token_span(p, s, t);
    lo = token_span(p, s, -(int)wave_max(-(float)t));
    hi = token_span(p, s, (int)wave_max((float)t));
    k_lo = s_lo = s_hi = k_hi = 0;
  }
  __device__ __forceinline__ void count(int position) {  // one key a lane
    k_lo += __popcll(__ballot(position < lo.sink));
    s_lo += __popcll(__ballot(position < hi.sink));
    s_hi += __popcll(__ballot(position < lo.recent));
    k_hi += __popcll(__ballot(position < hi.recent));
  }
};

template <int G>
__device__ __forceinline__ void load_queries(WaveTile& w, const BlockParams& p, int s, int h, int item) {
  const int lane = threadIdx.x & 63;
  const bf16_t* qr = p.q + ((size_t)(s * p.Tq + (item >> 13)) * p.Hq + h * G + (lane & 31) % G) * kD + (lane >> 5) * 8;
#pragma unroll
  for (int st = 0; st < 8; ++st) w.q[st] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(qr + st * 16));
}

template <int G>
__device__ __forceinline__ void store_slots(const WaveTile& w, const BlockParams& p, int s, int h, int item, int tokens) {
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  auto at = [&](int it) { return ((size_t)((s * p.Tq + (it >> 13)) * p.Hkv + h) * p.slots + (it & 8191)) * G; };
  const float L = sum_halves(w.l);
  if (half == 0 && col / G < tokens) p.part_ml[at(item) + col % G] = make_float2(w.m, L);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = row_of(r, half);
    const int it = row_value<G>(item, r, half);
    if (row / G < tokens)
      *reinterpret_cast<float4*>(p.part_o + (at(it) + row % G) * kD + col * 4) = make_float4(w.o[0][r], w.o[1][r], w.o[2][r], w.o[3][r]);
  }
}

template <int G>
__global__ void __launch_bounds__(256, 2)
block_attend_kernel(BlockParams p) {
  constexpr int TT = 32 / G;                             // tokens per tile; rows beyond them repeat the last one and are not stored
  __shared__ __align__(16) float s_o[2 * 32 * kD];
  __shared__ float s_ml[256];
  __shared__ int s_pos[4][kLongRun];                     // positions of the keys of a wave's bucket
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31;
  const int n_kv = p.S * p.Hkv, t_tiles = (p.Tq + TT - 1) / TT, n_dense = n_kv * t_tiles * p.splits;
  const int n_short = (int)p.counters[kCountShort * kLine], n_long = (int)p.counters[kCountLong * kLine];
  WaveTile w;
  float* s_w = s_o + wave * 32 * 32;                     // of attend_run: combine_waves uses s_o between its barriers

  // sink and recent keys: a wave takes a tile of consecutive tokens and a split of their recent keys, the waves of a
  // workgroup neighbouring tiles (the same keys, from the compute unit's L1)
  for (int task = blockIdx.x * 4 + wave; task < n_dense; task += gridDim.x * 4) {
    const int tile = task % t_tiles, rest = task / t_tiles, split = rest % p.splits, kvu = rest / p.splits;
    const int s = kvu / p.Hkv, t0 = tile * TT, tokens = min(TT, p.Tq - t0);
    const int t = t0 + min(col / G, tokens - 1), item = (t << 13) | (p.nprobe + split);
    const Span sp = token_span(p, s, t), sp0 = token_span(p, s, t0), sp1 = token_span(p, s, t0 + tokens - 1);
    const size_t base = (size_t)kvu * p.Nt * kD;
    // the tile's recent keys are [first token's begin, last token's end); a split takes whole tiles of them
    const int n_tiles = (sp1.end - sp0.recent + 31) / 32, per = (n_tiles + p.splits - 1) / p.splits * 32;
    const int r0 = sp0.recent + split * per;
    Run run{p.K + base, p.V + base, nullptr, r0, min(r0 + per, sp1.end), sp.recent, sp.end, sp1.recent, sp0.end};
    load_queries<G>(w, p, s, kvu - s * p.Hkv, item);
    w.clear();
    for (int part = 0; part < 2; ++part) {
      attend_run(w, run, 32, p.scale_log2, s_w);
      run = Run{p.K + base, p.V + base, nullptr, 0, split == 0 ? sp1.sink : 0, 0, sp.sink, 0, sp0.sink};
    }
    store_slots<G>(w, p, s, kvu - s * p.Hkv, item, tokens);
  }

  // long buckets: the four waves take the key tiles in turn
  for (int task = blockIdx.x; task < n_long; task += gridDim.x) {
    const BucketTile tile = read_tile(p, p.n_items_all - 1 - task);
    const int kvu = tile.kvu, s = kvu / p.Hkv, item = p.items[tile.item0 + min(col / G, tile.tokens - 1)];
    Bounds b(p, s, item >> 13);
    const int32_t* pos = p.idx + (size_t)kvu * p.Ncap + tile.row;
    for (int i = 0; i < tile.n; i += 64) b.count(i + lane < tile.n ? pos[i + lane] : 0x7fffffff);
    const size_t base = ((size_t)kvu * p.Ncap + tile.row) * kD;
    // whole tiles from the bucket's first row, dealt alike: a row's sums must not depend on who shares its tile
    const Run run{p.Ks + base, p.Vs + base, pos, (b.k_lo & ~127) + wave * 32, b.k_hi, b.sp.sink, b.sp.recent, b.s_lo, b.s_hi};
    load_queries<G>(w, p, s, kvu - s * p.Hkv, item);
    w.clear();
    attend_run(w, run, 128, p.scale_log2, s_w);
    combine_waves(w, s_ml, s_o);
    if (wave == 0) store_slots<G>(w, p, s, kvu - s * p.Hkv, item, tile.tokens);
    __syncthreads();                                     // this task's LDS is free
  }

  // short buckets, one a wave.  Two tiles ahead a wave takes its number, one ahead it reads the tile, and the tile's items and
  // positions are on their way under the stores of the tile before it.
  auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  const int queues = min(kQueues, (int)gridDim.x), queue = ((int)gridDim.x - 1 - (int)blockIdx.x) % queues;
  const int waves = 4 * (((int)gridDim.x - queue + queues - 1) / queues);          // that take from this queue: their first two are given
  auto tile_of = [&](int k) { return (k / 4 * queues + queue) * 4 + k % 4; };
  auto take = [&]() {
    unsigned v = 0;
    if (lane == 0) v = atomicAdd(p.counters + (kQueue0 + queue) * kLine, 1u);
    return (int)v;
  };
  // (counted from the last workgroup, which had the least of the dense pieces)
  const int first = uniform(((int)gridDim.x - 1 - (int)blockIdx.x) / queues * 4 + wave);
  int at = tile_of(first), next = tile_of(first + waves), item, pos[kPosRegs];
  if (at >= n_short) return;
  BucketTile tile = read_tile(p, at);
  auto fetch = [&](const BucketTile& b) {
    item = p.items[b.item0 + min(col / G, b.tokens - 1)];
    const int32_t* rows = p.idx + (size_t)b.kvu * p.Ncap + b.row;
#pragma unroll
    for (int i = 0; i < kPosRegs; ++i) pos[i] = 64 * i + lane < b.n ? rows[64 * i + lane] : 0x7fffffff;
  };
  fetch(tile);
  while (true) {
    const int kvu = tile.kvu, s = kvu / p.Hkv, mine = item, tokens = tile.tokens;
    load_queries<G>(w, p, s, kvu - s * p.Hkv, mine);
    w.clear();
    const int after = take();
    const bool more = next < n_short;
    const int4* ahead = p.tiles + 2 * (long long)(more ? next : at);
    const int4 a = ahead[0];
    const int an = ahead[1].x;
    Bounds b(p, s, mine >> 13);
#pragma unroll
    for (int i = 0; i < kPosRegs; ++i) {
      b.count(pos[i]);
      s_pos[wave][64 * i + lane] = pos[i];
    }
    const size_t base = ((size_t)kvu * p.Ncap + tile.row) * kD;
    const Run run{p.Ks + base, p.Vs + base, nullptr, b.k_lo & ~31, b.k_hi, b.sp.sink, b.sp.recent, b.s_lo, b.s_hi};
    attend_run(w, run, 32, p.scale_log2, s_w, s_pos[wave]);
    if (more) {
      tile = BucketTile{uniform(a.x), uniform(a.y), uniform(a.z), uniform(a.w), uniform(an)};
      fetch(tile);
    }
    store_slots<G>(w, p, s, kvu - s * p.Hkv, mine, tokens);
    if (!more) break;
    at = next;
    next = tile_of(2 * waves + uniform(after));
  }
}

// ---- 3. the slots of a (token, KV head) ---------------------------------------------------------------------
// Reads the slots at 5.6 TB/s (128 tokens, 59 slots of 4 heads: 22 us).
// G * d / 4 float4 columns; the workgroup's 256 threads form 8 / G groups that take the slots in turn, eight loads in flight.
template <int G>
__global__ void __launch_bounds__(256)
block_merge_kernel(BlockParams p) {
  constexpr int kCols = G * kD / 4, kGroups = 256 / kCols, kDeep = 8;
  extern __shared__ float s_w[];                         // [slots][G] weights 2^(m_i - M), 0 for an empty slot
  __shared__ float s_M[G], s_L[G];
  __shared__ float4 s_acc[256];
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float2* ml = p.part_ml + (size_t)unit * p.slots * G;
  if (unit == 0 && tid < kCounters) p.counters[tid * kLine] = 0u;        // the queues are done with
  for (int g = wave; g < G; g += 4) {
    float M = kNegBig;
    for (int i = lane; i < p.slots; i += 64) {
      const float2 v = ml[(size_t)i * G + g];
      if (v.y != 0.f) M = fmaxf(M, v.x);
    }
    M = wave_max(M);
    float L = 0.f;
    for (int i = lane; i < p.slots; i += 64) {
      const float2 v = ml[(size_t)i * G + g];
      const float wt = v.y != 0.f ? fast_exp2(v.x - M) : 0.f;   // a sum that is no number is passed on
      s_w[i * G + g] = wt;
      L = fmaf(wt, v.y, L);
    }
    L = wave_sum(L);
    if (lane == 0) {
      s_M[g] = M;
      s_L[g] = L;
    }
  }
  __syncthreads();
  const int colx = tid % kCols, grp = tid / kCols, g = colx / (kD / 4);
  const float4* po = reinterpret_cast<const float4*>(p.part_o) + (size_t)unit * p.slots * kCols + colx;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
  for (int i0 = grp; i0 < p.slots; i0 += kGroups * kDeep) {
    float4 v[kDeep];
    float wt[kDeep];
#pragma unroll
    for (int u = 0; u < kDeep; ++u) {
      const int i = min(i0 + u * kGroups, p.slots - 1);
      v[u] = po[(size_t)i * kCols];
      wt[u] = i0 + u * kGroups < p.slots ? s_w[i * G + g] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kDeep; ++u)
      if (wt[u] > 0.f) {                                 // what an empty slot holds is not a number to multiply with
        acc.x = fmaf(wt[u], v[u].x, acc.x);
        acc.y = fmaf(wt[u], v[u].y, acc.y);
        acc.z = fmaf(wt[u], v[u].z, acc.z);
        acc.w = fmaf(wt[u], v[u].w, acc.w);
      }
  }
  s_acc[tid] = acc;
  __syncthreads();
  if (tid >= kCols) return;
#pragma unroll
  for (int i = 1; i < kGroups; ++i) {
    const float4 v = s_acc[i * kCols + tid];
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  const float L = s_L[g], inv = L > 0.f ? 1.0f / L : 0.f * L;            // no keys: zeros; a score that is no number: no numbers
  const size_t qrow = (size_t)unit * G + g;              // units are (sequence, token, KV head)
  const int e0 = colx % (kD / 4) * 4;
  if (p.out_bf16) {
    uint2 pk;
    pk.x = f32_to_bf16_bits(acc.x * inv) | (f32_to_bf16_bits(acc.y * inv) << 16);
    pk.y = f32_to_bf16_bits(acc.z * inv) | (f32_to_bf16_bits(acc.w * inv) << 16);
    *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.out) + qrow * kD + e0) = pk;
  } else {
    *reinterpret_cast<float4*>(static_cast<float*>(p.out) + qrow * kD + e0) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  }
  if (e0 == 0 && p.lse) p.lse[qrow] = L > 0.f ? (s_M[g] + __log2f(L)) * kLn2 : -INFINITY;
}

// Splits of the recent keys: a thousand pieces or so, about half of the waves of the chip (the others start on the buckets);
// more of them shorten the longest piece of a small block and cost a large one a slot each.
int dense_splits(long long S, int Tq, int Hkv, int G, int n_recent) {
  const long long tt = 32 / G, tiles = S * Hkv * ((Tq + tt - 1) / tt);
  int splits = 2;
  while (splits < kMaxSplits && splits * tiles < 1024) splits *= 2;
  const int most = (n_recent < 0 ? 0x7fffffff : n_recent) / 64 + 1;       // two key tiles each
  return splits < most ? splits : most;
}

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

template <int G>
int32_t launch_block(const BlockParams& p, hipStream_t hs) {
  const size_t lds_merge = (size_t)p.slots * G * sizeof(float);
  if (!allow_lds<block_merge_kernel<G>>(lds_merge)) return SAAP_HIP_ERROR;
  if (p.nprobe > 0)
    hipLaunchKernelGGL(block_invert_kernel<32 / G>, dim3((unsigned)(p.S * p.Hkv), kInvertParts), dim3(kInvertThreads), 0, hs, p);
  // two workgroups per compute unit (their registers' room), no more than there can be tasks
  const long long tt = 32 / G, tasks = (long long)p.S * p.Hkv * ((p.Tq + tt - 1) / tt) * p.splits / 4 + p.n_items_all / 4 + 1;
  const long long grid = tasks < 2LL * device_cus() ? tasks : 2LL * device_cus();
  hipLaunchKernelGGL(block_attend_kernel<G>, dim3((unsigned)grid), dim3(256), 0, hs, p);
  hipLaunchKernelGGL(block_merge_kernel<G>, dim3((unsigned)(p.S * p.Tq * p.Hkv)), dim3(256), lds_merge, hs, p);
  return launch_status();
}

}  // namespace

// header | items | tiles | (max, sum) pairs | outputs of the slots; 0 where the path does not apply: lists too long for the
// merge's tables, or slots beyond 1.5 GiB
size_t block_workspace_bytes(long long S, int Tq, int Hq, int Hkv, int nprobe) {
  const long long units = S * Tq * Hkv, G = Hq / Hkv, slots = nprobe + dense_splits(S, Tq, Hkv, (int)G, -1);
  const size_t outputs = (size_t)units * slots * G * kD * sizeof(float);
  if (slots > kMaxSlots || Tq > 4096 || outputs > ((size_t)3 << 29)) return 0;
  const size_t items = (size_t)units * nprobe;
  return SAAP_WS_HEADER_BYTES + align256(items * sizeof(int)) + align256(items * 2 * sizeof(int4)) +
         align256((size_t)units * slots * G * sizeof(float2)) + outputs;
}

int32_t block_attention(const void* q, const void* K, const void* V, const void* Ks, const void* Vs, const int32_t* off,
                        const int32_t* len, const int32_t* idx, const int32_t* selected, const int32_t* pos0, int nprobe,
                        int n_sink, int n_recent, float scale, void* out, int out_bf16, float* lse, int S, int Hq, int Hkv, int Tq,
                        int Nt, int Ncap, int B, void* ws, hipStream_t hs) {
  BlockParams p{};
  p.q = static_cast<const bf16_t*>(q); p.K = static_cast<const bf16_t*>(K); p.V = static_cast<const bf16_t*>(V);
  p.Ks = static_cast<const bf16_t*>(Ks); p.Vs = static_cast<const bf16_t*>(Vs);
  p.off = off; p.len = len; p.idx = idx; p.selected = selected; p.pos0 = pos0; p.out = out; p.lse = lse;
  p.S = S; p.Hq = Hq; p.Hkv = Hkv; p.Tq = Tq; p.Nt = Nt; p.Ncap = Ncap; p.B = B; p.nprobe = nprobe;
  p.splits = dense_splits(S, Tq, Hkv, Hq / Hkv, n_recent);
  p.slots = nprobe + p.splits; p.n_sink = n_sink; p.n_recent = n_recent; p.out_bf16 = out_bf16; p.scale_log2 = scale * kLog2e;
  const long long units = (long long)S * Tq * Hkv;
  const int G = Hq / Hkv;
  p.n_items_all = units * nprobe;
  char* at = static_cast<char*>(ws);
  p.counters = reinterpret_cast<unsigned*>(at);
  at += SAAP_WS_HEADER_BYTES;
  p.items = reinterpret_cast<int*>(at);
  at += align256((size_t)p.n_items_all * sizeof(int));
  p.tiles = reinterpret_cast<int4*>(at);
  at += align256((size_t)p.n_items_all * 2 * sizeof(int4));
  p.part_ml = reinterpret_cast<float2*>(at);
  at += align256((size_t)units * p.slots * G * sizeof(float2));
  p.part_o = reinterpret_cast<float*>(at);
  switch (G) {
    case 1: return launch_block<1>(p, hs);
    case 2: return launch_block<2>(p, hs);
    case 4: return launch_block<4>(p, hs);
    default: return launch_block<8>(p, hs);
  }
}

}  // namespace saap
