// assign_keys: nearest-centroid assignment of keys at prefill (Section 2, indexing step, and
// Section 4 of arXiv 2502.08246): bucket = argmax_b <x, c_b> + bias_b.
//
// The result is DEFINED on double-precision scores (in-order sum of exact products, lowest id
// on ties).  Two kernels produce exactly that:
//   * mfma kernel (bf16 inputs): scores on the matrix cores, fp32 accumulation.  A workgroup
//     holds 256 keys in registers as the B operand of v_mfma_f32_32x32x16_bf16 and streams the
//     centroids through LDS in tiles of 32 as the A operand, so one lane owns one key and its 16
//     accumulator registers are 16 different centroids.  Per key the lane tracks the best and
//     second-best score; the low 4 bits of a score carry the accumulator register number, so
//     the running argmax costs 2.5 vector instructions per score (tag; max3 and med3 + max per pair).
//   * re-scoring kernel: a key whose best two fp32 scores are closer than the accumulation error
//     bound is scored again, 32 such keys of a head at a time: one more matrix-core pass (two
//     beyond 1024 buckets) finds every centroid within the bound of the key's maximum, and only
//     those (typically two) are scored in double precision.
//   * fp32 inputs: the same with fp32 matrix instructions, close keys scored by the workgroup that found them.
// No score matrix is ever written to memory.
#include <type_traits>

#include "assign_close.h"
#include "common.h"

namespace saap {
namespace {

constexpr int kRowsPerWg = 256;   // keys per workgroup of the mfma kernel (4 waves x 64)
constexpr int kCentTile = 32;     // centroids per matrix tile
constexpr int kSlab = 64;         // centroids per LDS slab (two matrix tiles)
constexpr int kPitch = 136;       // bf16 elements per LDS row (272 bytes: conflict-free b128 reads)

// max_b |c_b| per KV head (fp32, rounded up a little).  16 lanes per centroid row.
constexpr int kNormThreads = 1024;
__global__ void __launch_bounds__(kNormThreads)
cent_norm_kernel(const bf16_t* __restrict__ cent, float* __restrict__ cmax, int B) {
  __shared__ float s_m[kNormThreads / 64];
  const int h = blockIdx.x, tid = threadIdx.x, piece = tid & 15, sub = tid >> 4;
  const bf16_t* cu = cent + (size_t)h * B * kD;
  float mx = 0.f;
  for (int b0 = 0; b0 < B; b0 += kNormThreads / 16 * 4) {
    Vec8<bf16_t> v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u].load(cu + (size_t)min(b0 + u * (kNormThreads / 16) + sub, B - 1) * kD + piece * 8);
#pragma unroll
    for (int u = 0; u < 4; ++u) mx = fmaxf(mx, sum16(v[u].dot(v[u])));
  }
  mx = max_rows(mx);
  if ((tid & 63) == 0) s_m[tid >> 6] = mx;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kNormThreads / 64; ++w) mx = fmaxf(mx, s_m[w]);
    cmax[h] = sqrtf(mx) * 1.0001f;
  }
}

// NORMS: the workgroup makes the largest norm of its head itself, from the rows on their way to LDS, and the head's first one
// leaves it in cmax (see the launch).  RAGGED: the last slab has rows past the last centroid.
template <bool HAS_BIAS, bool NORMS, bool RAGGED>
__global__ void __launch_bounds__(256, 2)
assign_mfma_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ cent, const float* __restrict__ bias,
                   float* __restrict__ cmax, int32_t* __restrict__ ids, int32_t* __restrict__ flagged,
                   unsigned* __restrict__ n_flagged, size_t list_cap, int Hkv, int N, int B, float tol) {
  __shared__ __align__(16) bf16_t s_c[2][kSlab * kPitch];
  // Biases of a slab.  They are read until the slab after the next is being stored: four in turn.
  __shared__ __align__(16) float s_bias[HAS_BIAS ? 4 : 1][HAS_BIAS ? kSlab : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int unit = blockIdx.y, h = unit % Hkv;
  const int col = lane & 31, half = lane >> 5;
  const bf16_t* cu = cent + (size_t)h * B * kD;

  // B operand: two tiles of 32 keys per wave; lane holds features 16*step + 8*half .. +7 of key `col`.
  const int row_base = blockIdx.x * kRowsPerWg + wave * 64;
  bf16x8_t xb[2][8];
  float xnorm2[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const int r = min(row_base + rt * 32 + col, N - 1);
    const bf16_t* xr = x + ((size_t)unit * N + r) * kD + half * 8;
    float s = 0.f;
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const uint4 raw = *reinterpret_cast<const uint4*>(xr + st * 16);
      xb[rt][st] = __builtin_bit_cast(bf16x8_t, raw);
      const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s = fmaf(bf16_lo(w[i]), bf16_lo(w[i]), s);
        s = fmaf(bf16_hi(w[i]), bf16_hi(w[i]), s);
      }
    }
    s += __shfl_xor(s, 32);
    xnorm2[rt] = s;
  }

  // Centroids stream through LDS in slabs of kSlab = 64 (two matrix tiles of 32), double
  // buffered: a slab is 1024 pieces of 16 bytes, four per thread, fetched into registers one
  // slab ahead (a slab's worth of matrix work covers the L2 latency) and stored mid-way through
  // the compute of the slab before.
  const int n_slabs = (B + kSlab - 1) / kSlab;
  // The staging registers must stay registers: fetch and stash run unconditionally (the last
  // pass fetches the last slab again and stores it into the idle buffer), which keeps them out of
  // control flow; behind a branch the compiler parked them in scratch memory and waited for every
  // load right after issuing it.
  // Rows past the last centroid are read as zeros (what a buffer load gives beyond the buffer's end) and do not count (track_pair).  With
  // centroid 0 in their place every key of bucket 0 had two equal best scores and was re-scored (2 heads of 2082 keys, 48 buckets:
  // re-scoring 11.5 us, 4.9 now); with a score of 0 every key that scores below zero everywhere (8 heads of 16384 such keys, 48
  // buckets: 187 us in all, 20 now).  A loop without the rows' 64-bit addresses is the faster one besides: 8 heads of 131072 keys, 1024
  // buckets, 257 -> 251 us.
  u32x4_t stage[kSlab / 16];
  float stage_bias = 0.f;
  const __amdgpu_buffer_rsrc_t rows_of_c = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(cu), 0, (int)((unsigned)B * (kD * 2)), 0x00027000);
  auto fetch = [&](int t) {
#pragma unroll
    for (int i = 0; i < kSlab / 16; ++i)
      stage[i] = __builtin_amdgcn_raw_buffer_load_b128(rows_of_c, (int)((unsigned)t * (kSlab * kD * 2) + (tid + i * 256) * 16), 0, 0);
    if constexpr (HAS_BIAS) stage_bias = bias[(size_t)h * B + min(t * kSlab + lane, B - 1)];      // (every wave the same)
  };
  float norm2 = 0.f;                             // NORMS: the largest squared norm of the rows that the thread's row of lanes has stored
  // Rows past the last centroid score the lowest finite value.  An infinite score would be a NaN with a tag in its low bits and displace
  // others: a bias of -infinity (a masked bucket) or nearly so is cut down to what leaves room for the product; keys whose best two
  // scores come from such biases find them equal and are re-scored.  That happens on the biases' way to LDS, once for a workgroup: loaded
  // by each lane for each tile they held up the ranking (8 heads of 131072 keys, 1024 buckets 414 us, 283 so, 254 without biases).
  constexpr float kLowest = -3.402823466e38f, kMostBias = 1.7e38f;
  auto stash = [&](int buf, int t) {
    if constexpr (HAS_BIAS)
      s_bias[t & 3][lane] = t * kSlab + lane < B ? __builtin_amdgcn_fmed3f(stage_bias, -kMostBias, kMostBias) : kLowest;
#pragma unroll
    for (int i = 0; i < kSlab / 16; ++i) {
      const int piece = tid + i * 256, r = piece >> 4, pc = piece & 15;
      *reinterpret_cast<u32x4_t*>(&s_c[buf][r * kPitch + pc * 8]) = stage[i];
      if constexpr (NORMS) {
        Vec8<bf16_t> v;
        v.r = make_uint4(stage[i][0], stage[i][1], stage[i][2], stage[i][3]);
        norm2 = fmaxf(norm2, sum16(v.dot(v)));
      }
    }
  };
  fetch(0);
  stash(0, 0);
  fetch(min(1, n_slabs - 1));
  __syncthreads();

  const uint32_t keep = 0xFFFFFFF0u;
  float best[2], second[2];
  int best_tile[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    best[rt] = -INFINITY;
    second[rt] = -INFINITY;
    best_tile[rt] = 0;
  }

  typedef __attribute__((ext_vector_type(16))) float f32x16_t;
  // A operand of k-step `st` of matrix tile `sub` of the slab in `buf`
  auto a_frag = [&](int buf, int sub, int st) {
    const uint4 raw = *reinterpret_cast<const uint4*>(&s_c[buf][(sub * kCentTile + col) * kPitch + st * 16 + half * 8]);
    return __builtin_bit_cast(bf16x8_t, raw);
  };
  // running best / second best over accumulator registers r, r+1 of both key tiles; register r
  // of this lane is centroid 8*(r/4) + 4*half + r%4 of matrix tile `tile` (global tile number).
  // Two scores per step: with s <= b the second largest of {b, s, x, y} is max(s, med3(b, x, y)),
  // the largest max3(b, x, y): 2.5 vector instructions per score with the tag, not 3.
  // last: the ragged tile, whose rows past the last centroid score less than any other (the lowest finite value: with a tag in
  // its place an infinity would be a NaN); one wins where no score compares, and the key is re-scored (id >= B below).
  auto track_pair = [&](auto last, const f32x16_t& c0, const f32x16_t& c1, const float (&add)[16], int tile, int r) {
    float p0[2], p1[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float s0 = c0[r + u], s1 = c1[r + u];
      if (HAS_BIAS) {
        s0 += add[r + u];
        s1 += add[r + u];
      }
      if constexpr (decltype(last)::value) {
        const int b = tile * kCentTile + 8 * ((r + u) / 4) + 4 * half + ((r + u) % 4);
        s0 = b < B ? s0 : kLowest;
        s1 = b < B ? s1 : kLowest;
      }
      p0[u] = __uint_as_float((__float_as_uint(s0) & keep) | (uint32_t)(r + u));
      p1[u] = __uint_as_float((__float_as_uint(s1) & keep) | (uint32_t)(r + u));
    }
    second[0] = fmaxf(second[0], __builtin_amdgcn_fmed3f(best[0], p0[0], p0[1]));
    best[0] = fmaxf(fmaxf(best[0], p0[0]), p0[1]);
    second[1] = fmaxf(second[1], __builtin_amdgcn_fmed3f(best[1], p1[0], p1[1]));
    best[1] = fmaxf(fmaxf(best[1], p1[0]), p1[1]);
  };
  // Software pipeline over matrix tiles: while the matrix cores work on tile (buf, sub) into
  // n0/n1, the vector pipe ranks the finished scores o0/o1 of the tile before.  One k-step (two
  // matrix instructions, 2 x 8 passes) is paired with one register pair of ranking (ten vector
  // instructions) between scheduling fences; left alone the compiler issues all sixteen matrix
  // instructions first and the two pipes run one after the other.
  auto step = [&](auto last, int buf, int sub, f32x16_t& n0, f32x16_t& n1, const f32x16_t& o0, const f32x16_t& o1,
                  int tile_old, bool has_new, bool has_old) {
    const float old0 = best[0], old1 = best[1];
    bf16x8_t a = a_frag(buf, sub, 0);
    float add[16];                               // the old tile's biases: register r's centroid is 8*(r/4) + 4*half + r%4 of it
    if (HAS_BIAS && has_old) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(&s_bias[tile_old >> 1 & 3][(tile_old & 1) * kCentTile + 8 * i + 4 * half]);
        add[4 * i] = v.x; add[4 * i + 1] = v.y; add[4 * i + 2] = v.z; add[4 * i + 3] = v.w;
      }
    }
    if (has_new) {
      n0 = (f32x16_t){0};
      n1 = (f32x16_t){0};
    }
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      __builtin_amdgcn_sched_barrier(0);
      if (has_new) {
        const bf16x8_t a_next = a_frag(buf, sub, min(st + 1, 7));
        n0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xb[0][st], n0, 0, 0, 0);
        n1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xb[1][st], n1, 0, 0, 0);
        a = a_next;
      }
      if (has_old) track_pair(last, o0, o1, add, tile_old, 2 * st);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (has_old) {
      best_tile[0] = best[0] != old0 ? tile_old : best_tile[0];
      best_tile[1] = best[1] != old1 ? tile_old : best_tile[1];
    }
  };

  const std::false_type inner;
  const std::integral_constant<bool, RAGGED && !HAS_BIAS> last;          // (biases see to it)
  f32x16_t a0, a1, b0 = {0}, b1 = {0};   // b0, b1: not read by the first step
  step(inner, 0, 0, a0, a1, b0, b1, 0, true, false);
  for (int t = 0; t < n_slabs - 1; ++t) {
    const int buf = t & 1;
    step(inner, buf, 1, b0, b1, a0, a1, t * 2 + 0, true, true);
    stash(buf ^ 1, t + 1);
    fetch(min(t + 2, n_slabs - 1));
    __syncthreads();
    step(inner, buf ^ 1, 0, a0, a1, b0, b1, t * 2 + 1, true, true);
  }
  // Of the last slab's two tiles one is ragged, and where that is the first there is no second: 8 heads of 131072 keys, 1000 buckets
  // 258 us with both looked at, 249.5 so.
  const int t_last = (n_slabs - 1) * 2, buf_last = (n_slabs - 1) & 1;
  if (!RAGGED || B > (t_last + 1) * kCentTile) {
    step(inner, buf_last, 1, b0, b1, a0, a1, t_last, true, true);
    step(last, 0, 0, a0, a1, b0, b1, t_last + 1, false, true);
  } else {
    step(last, 0, 0, b0, b1, a0, a1, t_last, false, true);
  }

  // lanes l and l+32 own the same key: merge their candidates, lower id on equal packed scores
  __shared__ unsigned s_listed, s_list_base;
  __shared__ float s_norm2[4];
  if (tid == 0) s_listed = 0u;
  if constexpr (NORMS) {
    norm2 = max_rows(norm2);
    if (lane == 0) s_norm2[wave] = norm2;
  }
  __syncthreads();
  float norm;
  if constexpr (NORMS) {
    norm = sqrtf(fmaxf(fmaxf(s_norm2[0], s_norm2[1]), fmaxf(s_norm2[2], s_norm2[3]))) * 1.0001f;
    if (tid == 0 && blockIdx.x == 0 && unit < Hkv) cmax[h] = norm;
  } else {
    norm = cmax[h];
  }
  const float tol_c = tol * norm;
  bool listed[2];
  unsigned slot[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const int r = (int)(__float_as_uint(best[rt]) & 15u);
    int id = best_tile[rt] * kCentTile + 8 * (r / 4) + 4 * half + (r % 4);
    const float ob = __shfl_xor(best[rt], 32);
    const float os = __shfl_xor(second[rt], 32);
    const int oid = __shfl_xor(id, 32);
    const float mb = best[rt], ms = second[rt];
    float nb, ns;
    if (ob > mb || (ob == mb && oid < id)) {
      nb = ob;
      ns = fmaxf(mb, os);
      id = oid;
    } else {
      nb = mb;
      ns = fmaxf(ob, ms);
    }
    const int row = row_base + rt * 32 + col;
    listed[rt] = false;
    if (half == 0 && row < N) {
      const size_t g = (size_t)unit * N + row;
      ids[g] = id;
      // error bound of the fp32 accumulation plus the 4 mantissa bits used for the register tag (of a score of zero: all that it has)
      const float from_product = tol_c * sqrtf(xnorm2[rt]);
      const float thr = from_product + 5e-6f * fabsf(nb) + 4e-36f;
      // (products near the end of fp32's range may have overflowed, with a bias or without)
      if (!(nb - ns > thr) || id >= B || !(from_product < tol * 1e38f)) {
        listed[rt] = true;
        slot[rt] = atomicAdd(&s_listed, 1u);
      }
    }
  }
  // one list per KV head (the re-scoring shares centroid loads between keys of a head); the
  // workgroup's keys are added in one piece, with one global counter update
  __syncthreads();
  if (tid == 0 && s_listed) s_list_base = atomicAdd(n_flagged + h, s_listed);
  __syncthreads();
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
    if (listed[rt])   // global row index fits in 31 bits: checked on the host
      flagged[(size_t)h * list_cap + s_list_base + slot[rt]] = (int32_t)((size_t)unit * N + row_base + rt * 32 + col);
}

// fp32 inputs, few keys: double-precision scoring of every key against every centroid (in-order sum,
// lowest id on ties).  One workgroup per key.
__global__ void __launch_bounds__(256)
assign_exact_f32_kernel(const float* __restrict__ x, const float* __restrict__ cent, const float* __restrict__ bias,
                        int32_t* __restrict__ ids, int Hkv, int N, int B) {
  __shared__ double s_x[kD];
  __shared__ double s_best[256];
  __shared__ int s_id[256];
  const int tid = threadIdx.x;
  const long long g = blockIdx.x;
  const int h = (int)((g / N) % Hkv);
  if (tid < kD) s_x[tid] = (double)x[(size_t)g * kD + tid];
  __syncthreads();
  double best = 0.0;
  int best_id = -1;
  for (int b = tid; b < B; b += blockDim.x) {
    const float* c = cent + ((size_t)h * B + b) * kD;
    double t = 0.0;
    for (int j = 0; j < kD; ++j) t = fma(s_x[j], (double)c[j], t);
    if (bias) t += (double)bias[(size_t)h * B + b];
    if (best_id < 0 || t > best) {
      best = t;
      best_id = b;
    }
  }
  s_best[tid] = best;
  s_id[tid] = best_id;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) {
      const int oid = s_id[tid + s], mid = s_id[tid];
      const double ob = s_best[tid + s];
      if (oid >= 0 && (mid < 0 || ob > s_best[tid] || (ob == s_best[tid] && oid < mid))) {
        s_best[tid] = ob;
        s_id[tid] = oid;
      }
    }
    __syncthreads();
  }
  if (tid == 0) ids[g] = s_id[0];
}

// Re-scoring of the listed keys (bf16).  The keys are listed per KV head; a workgroup takes 32
// consecutive entries of one head's list as the B operand of the matrix instruction (every wave
// holds the same 32 keys) and its eight waves share out the centroid tiles, so a centroid row is
// read once for 32 keys.
//   pass 1: fp32 scores of all centroids on the matrix cores, running maximum per key; a wave keeps
//           the scores of its first kKeepTiles tiles in registers (all of them up to 1024 buckets)
//           and has the loads of those tiles in flight together;
//   pass 2: every centroid whose score is within the error bound of the key's maximum goes into a
//           candidate list in LDS: from the kept scores, and for further tiles from the same
//           instructions run again (same results bit for bit).  Any centroid that can be the
//           double-precision argmax is among them, because both fp32 scores carry at most half the
//           bound as error; a score that does not compare (NaN) counts as a candidate;
//   pass 3: the candidates (typically two per key) in double precision, in order, one per thread;
//           the largest per key, lowest id on ties, through LDS atomics (maximum of the scores in
//           an order-preserving integer form, then minimum of the ids that reach it).
// If the list overflows (degenerate keys, e.g. all scores equal) the group's keys are scored
// against every centroid in double precision instead.
// Grid: (Hkv, workgroups per head), the head fastest, so that the few workgroups that find a group
// of keys are the first to be dispatched.  counters[h] = length of head h's list, counters[Hkv] =
// workgroups that have finished.
constexpr int kGroupKeys = 32;
constexpr int kCandCap = 2048;
constexpr int kRescoreThreads = 512, kRescoreWaves = kRescoreThreads / 64;
constexpr int kHalfPitch = kD / 2 + 8;   // bf16 elements per LDS row of half a centroid row (144 bytes: conflict-free b128 reads)
constexpr int kKeepTiles = 4;      // matrix tiles per wave whose scores stay in registers between the passes

// double-precision score of centroid row c against key row xr (in order), rows of 16-byte pieces
__device__ __forceinline__ double score_bf16_f64(const uint4* __restrict__ xr, const uint4* __restrict__ c) {
  // The loads and conversions stay inside the (rarely taken) candidate path: hoisted out of a
  // caller's loop the key's 128 doubles would hold 256 registers for the whole kernel.
  asm volatile("" ::: "memory");
  double t = 0.0;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {   // half a row of each in flight, then that half of the chain
    uint4 xw[kD / 16], cw[kD / 16];
#pragma unroll
    for (int j = 0; j < kD / 16; ++j) {
      xw[j] = xr[hh * (kD / 16) + j];
      cw[j] = c[hh * (kD / 16) + j];
    }
#pragma unroll
    for (int j = 0; j < kD / 16; ++j) {
      const uint32_t w[4] = {cw[j].x, cw[j].y, cw[j].z, cw[j].w}, v[4] = {xw[j].x, xw[j].y, xw[j].z, xw[j].w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        t = fma((double)bf16_lo(v[k]), (double)bf16_lo(w[k]), t);
        t = fma((double)bf16_hi(v[k]), (double)bf16_hi(w[k]), t);
      }
    }
  }
  return t;
}

__device__ __forceinline__ bool better(double s, int id, double best, int best_id) {
  return id >= 0 && (best_id < 0 || s > best || (s == best && id < best_id));
}

// Doubles as unsigned integers in the same order (no NaNs; -0 is turned into +0 first).
__device__ __forceinline__ unsigned long long ordered_bits(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v + 0.0);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__global__ void __launch_bounds__(kRescoreThreads)
assign_rescore_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ cent,
                      const float* __restrict__ bias, const float* __restrict__ cmax,
                      int32_t* __restrict__ ids, const int32_t* __restrict__ rows,
                      unsigned* __restrict__ counters, unsigned* __restrict__ stat, size_t list_cap, int Hkv,
                      int B, float tol) {
  typedef __attribute__((ext_vector_type(16))) float f32x16_t;
  __shared__ float s_max[kRescoreWaves][kGroupKeys];
  __shared__ float s_lim[kGroupKeys];
  __shared__ int s_key[kGroupKeys];        // global row of each key of the group
  __shared__ unsigned s_ncand;
  __shared__ int s_cand[kCandCap];         // key << 24 | centroid
  __shared__ unsigned long long s_cscore[kCandCap];   // ordered_bits of the candidate's score
  __shared__ unsigned long long s_kbest[kGroupKeys];
  __shared__ int s_kid[kGroupKeys];
  __shared__ double s_wbest[kRescoreWaves];
  __shared__ int s_wid[kRescoreWaves];
  __shared__ int s_flag;
  __shared__ __align__(16) bf16_t s_half[kRescoreWaves][kCentTile * kHalfPitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  const int h = blockIdx.x;
  const float norm = cmax[h];
  const unsigned n_rows = counters[h];
  unsigned total = 0;                                    // of all heads' lists, for the last workgroup to leave
  for (int i = tid; i < Hkv; i += kRescoreThreads) total += counters[i];
  const unsigned n_groups = (n_rows + kGroupKeys - 1) / kGroupKeys;
  rows += (size_t)h * list_cap;
  const bf16_t* cu = cent + (size_t)h * B * kD;
  const float* bu = bias ? bias + (size_t)h * B : nullptr;
  const int n_tiles = (B + kCentTile - 1) / kCentTile;

  SAAP_TRACE(0);
  for (unsigned grp = blockIdx.y; grp < n_groups; grp += gridDim.y) {
    const unsigned first = grp * kGroupKeys;
    const int n_here = (int)min((unsigned)kGroupKeys, n_rows - first);
    // B operand: lane holds features 16*step + 8*half .. +7 of key `col` (idle columns repeat the last key)
    const int gk = rows[first + min(col, n_here - 1)];
    const bf16_t* xr = x + (size_t)gk * kD + half * 8;
    bf16x8_t xb[8];
    float xnorm2 = 0.f;
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      Vec8<bf16_t> v;
      v.load(xr + st * 16);
      xb[st] = __builtin_bit_cast(bf16x8_t, v.r);
      xnorm2 += v.dot(v);
    }
    xnorm2 += __shfl_xor(xnorm2, 32);
    SAAP_TRACE(1);
    if (tid < kGroupKeys) {
      s_key[tid] = gk;
      s_kbest[tid] = 0ull;
      s_kid[tid] = 0x7fffffff;
    }
    if (tid == 0) s_ncand = 0u;

    // scores of centroid tile t for the 32 keys: register r of this lane is centroid
    // 32*t + 8*(r/4) + 4*half + r%4 against key `col`
    // Whole lines are loaded (a half row per eight lanes) and turned round in the wave's LDS: loads in the operand's layout touch
    // a line four times, and a group's 256 KB (1024 centroids) then took 9.5 us to come, 5.3 like this (8 heads of 65536 keys, a
    // few groups each: 21.1 -> 15.1 us with the candidates listed by bits).
    struct Tile { u32x4_t p[2][4]; };                    // [half of the features][rows lane / 8 + 8 i]
    auto tile_load = [&](int t, Tile& a) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bf16_t* cr = cu + (size_t)min(t * kCentTile + (lane >> 3) + 8 * i, B - 1) * kD + (lane & 7) * 8;
        a.p[0][i] = *reinterpret_cast<const u32x4_t*>(cr);
        a.p[1][i] = *reinterpret_cast<const u32x4_t*>(cr + kD / 2);
      }
    };
    auto tile_product = [&](const Tile& a) {
      bf16_t* s = s_half[wave];                          // LDS accesses of one wave run in order
      f32x16_t acc = {0};
#pragma unroll
      for (int f = 0; f < 2; ++f) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4_t*>(s + ((lane >> 3) + 8 * i) * kHalfPitch + (lane & 7) * 8) = a.p[f][i];
        __builtin_amdgcn_wave_barrier();
        bf16x8_t c[4];
#pragma unroll
        for (int st = 0; st < 4; ++st) c[st] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(s + col * kHalfPitch + st * 16 + half * 8));
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int st = 0; st < 4; ++st) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[st], xb[4 * f + st], acc, 0, 0, 0);
      }
      return acc;
    };
    auto centroid_of = [&](int t, int r) { return t * kCentTile + 8 * (r / 4) + 4 * half + (r % 4); };
    // the scores that are compared: matrix product plus the centroid's bias (one fp32 addition)
    auto add_bias = [&](f32x16_t& acc, int t) {
      if (bu) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] += bu[min(centroid_of(t, r), B - 1)];
      }
    };
    auto tile_scores = [&](int t) {
      Tile a;
      tile_load(t, a);
      f32x16_t acc = tile_product(a);
      add_bias(acc, t);
      return acc;
    };
    auto tile_max = [&](const f32x16_t& acc, int t, float mx) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (centroid_of(t, r) < B) mx = fmaxf(mx, acc[r]);
      return mx;
    };
    // bit r: the score in register r is a candidate's
    auto tile_hits = [&](const f32x16_t& acc, float lim) {
      unsigned hits = 0u;
#pragma unroll
      for (int r = 0; r < 16; ++r) hits |= !(acc[r] < lim) ? 1u << r : 0u;
      return hits;
    };
    // the candidates of two tiles, `hits` 16 bits of each (bits in turn: a branch per register costs more than the few bits set)
    auto list_candidates = [&](unsigned hits, int t_low, int t_high) {
      while (hits != 0u) {
        const int bit = __ffs((int)hits) - 1;
        hits &= hits - 1u;
        const int b = centroid_of(bit < 16 ? t_low : t_high, bit & 15);
        if (b < B && col < n_here) {
          const unsigned i = atomicAdd(&s_ncand, 1u);
          if (i < (unsigned)kCandCap) s_cand[i] = (col << 24) | b;
        }
      }
    };

    // the wave's first kKeepTiles tiles: every load goes out before the first product (tiles past
    // the end repeat the last one and are ignored below)
    f32x16_t kept[kKeepTiles];
    // the tile numbers are made opaque per group: as loop invariants the compiler computes every address of
    // every tile (centroid rows, biases) ahead of the loop and spills them
    int wave_t = wave;
    asm volatile("" : "+v"(wave_t));
    {
      Tile a[kKeepTiles];
#pragma unroll
      for (int k = 0; k < kKeepTiles; ++k) tile_load(min(wave_t + k * kRescoreWaves, n_tiles - 1), a[k]);
      __builtin_amdgcn_sched_barrier(0);     // left alone the compiler keeps three or four loads in flight
#pragma unroll
      for (int k = 0; k < kKeepTiles; ++k) {
        // a tile that is not there has no candidates (scores of zero would be listed, one by one, where all others are below zero)
        kept[k] = (f32x16_t){0} - INFINITY;
        if (wave_t + k * kRescoreWaves < n_tiles) kept[k] = tile_product(a[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < kKeepTiles; ++k) add_bias(kept[k], min(wave_t + k * kRescoreWaves, n_tiles - 1));
    float mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < kKeepTiles; ++k) {
      const int t = wave_t + k * kRescoreWaves;
      if (t < n_tiles) mx = tile_max(kept[k], t, mx);
    }
    for (int t = wave_t + kKeepTiles * kRescoreWaves; t < n_tiles; t += kRescoreWaves) mx = tile_max(tile_scores(t), t, mx);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (half == 0) s_max[wave][col] = mx;
    __syncthreads();
    SAAP_TRACE(2);
    if (tid < kGroupKeys) {
      float m = s_max[0][tid];
      for (int w = 1; w < kRescoreWaves; ++w) m = fmaxf(m, s_max[w][tid]);
      // two fp32 scores are compared: the same bound as for the first matrix pass (a maximum of +infinity may be a finite one's overflow)
      m = fminf(m, 3.402823466e38f);
      s_lim[tid] = m - (tol * norm * sqrtf(xnorm2) + 5e-6f * fabsf(m));
    }
    __syncthreads();
    const float lim = s_lim[col];
    static_assert(kKeepTiles % 2 == 0, "tiles in pairs");
#pragma unroll
    for (int k = 0; k < kKeepTiles; k += 2) {
      const int t = wave_t + k * kRescoreWaves;            // a tile past the end lists centroids past B: dropped
      list_candidates(tile_hits(kept[k], lim) | tile_hits(kept[k + 1], lim) << 16, t, t + kRescoreWaves);
    }
    for (int t = wave_t + kKeepTiles * kRescoreWaves; t < n_tiles; t += kRescoreWaves) list_candidates(tile_hits(tile_scores(t), lim), t, t);
    __syncthreads();
    SAAP_TRACE(3);
    const unsigned n_cand = s_ncand;
    if (tid == 0) SAAP_TRACE_VALUE(7, n_cand);
    if (n_cand <= (unsigned)kCandCap) {
      for (unsigned i = tid; i < n_cand; i += kRescoreThreads) {
        const int key = s_cand[i] >> 24, b = s_cand[i] & 0xffffff;
        double t = score_bf16_f64(reinterpret_cast<const uint4*>(x + (size_t)s_key[key] * kD),
                                  reinterpret_cast<const uint4*>(cu + (size_t)b * kD));
        if (bu) t += (double)bu[b];
        const unsigned long long o = ordered_bits(t);
        s_cscore[i] = o;
        atomicMax(&s_kbest[key], o);
      }
      __syncthreads();
      SAAP_TRACE(4);
      for (unsigned i = tid; i < n_cand; i += kRescoreThreads) {
        const int key = s_cand[i] >> 24, b = s_cand[i] & 0xffffff;
        if (s_cscore[i] == s_kbest[key]) atomicMin(&s_kid[key], b);
      }
      __syncthreads();
      // every key has a candidate (its fp32 maximum is within the bound of itself)
      if (tid < n_here) ids[s_key[tid]] = s_kid[tid];
      SAAP_TRACE(5);
    } else {
      // too many candidates: every key of the group against every centroid in double precision
      for (int key = 0; key < n_here; ++key) {
        const uint4* xk = reinterpret_cast<const uint4*>(x + (size_t)s_key[key] * kD);
        double best = 0.0;
        int best_id = -1;
        for (int b = tid; b < B; b += kRescoreThreads) {
          double t = score_bf16_f64(xk, reinterpret_cast<const uint4*>(cu + (size_t)b * kD));
          if (bu) t += (double)bu[b];
          if (better(t, b, best, best_id)) {
            best = t;
            best_id = b;
          }
        }
        for (int o = 1; o < 64; o <<= 1) {
          const double ob = __shfl_xor(best, o);
          const int oid = __shfl_xor(best_id, o);
          if (better(ob, oid, best, best_id)) {
            best = ob;
            best_id = oid;
          }
        }
        if (lane == 0) {
          s_wbest[wave] = best;
          s_wid[wave] = best_id;
        }
        __syncthreads();
        if (tid == 0) {
          for (int w = 1; w < kRescoreWaves; ++w)
            if (better(s_wbest[w], s_wid[w], best, best_id)) {
              best = s_wbest[w];
              best_id = s_wid[w];
            }
          ids[s_key[key]] = best_id;
        }
        __syncthreads();
      }
    }
    __syncthreads();
  }
  // Every workgroup has read its list length by now; the last one to leave keeps the total for
  // diagnostics and leaves all counters zero for the next call.
  __syncthreads();
  if (tid == 0) s_flag = atomicAdd(counters + Hkv, 1u) == gridDim.x * gridDim.y - 1 ? 1 : 0;
  __syncthreads();
  if (s_flag) {
    for (int i = tid; i < Hkv; i += kRescoreThreads) counters[i] = 0u;
    if (tid == 0) {
      *stat = 0u;
      counters[Hkv] = 0u;
    }
    __syncthreads();
    if (total) atomicAdd(stat, total);
  }
  SAAP_TRACE(6);
}

// fp32 inputs.  Scores on the fp32 matrix instructions: 128 keys to a workgroup, 32 of them in a wave's registers, centroids
// through LDS in tiles of 32 rows.  A lane has 16 scores of its key per tile and keeps the best, its id and the second best.  Keys whose two are closer
// than the scores' error take a second walk over the tiles, which lists the centroids within the error of the best; those are
// scored in double precision, one to a thread, which defines the result (in-order sums, lowest id on ties).  Keys with a score that
// does not compare, with norms out of the ordinary, or of a workgroup that lists too many, are scored against every centroid, 32 at a time
// from tiles in LDS (all keys, equal centroids: 8 heads of 3840 keys, 96 centroids 573 us with one key after the other, 108 so; 8 of
// 8192, 256: 1081, 323; one head of 8064, 240: 778, 257, which a workgroup per key did in 114: there are 63 workgroups here).
// (8 heads of 3815 keys, 96 centroids: 189 us with every key scored so, 16.5 now; one head of 8000, 240 centroids: 122,
// 31; 8 of 8192, 256: 974, 53.)
constexpr int kF32Keys = 128, kF32Pitch = kD + 4;        // floats per LDS row (conflict-free 16-byte reads)
constexpr int kF32Cand = 1024, kScanKeys = 32;
__global__ void __launch_bounds__(256, 2)
assign_f32_kernel(const float* __restrict__ x, const float* __restrict__ cent, const float* __restrict__ bias,
                  int32_t* __restrict__ ids, int Hkv, int N, int B, float tol) {
  typedef __attribute__((ext_vector_type(16))) float f32x16_t;
  __shared__ __align__(16) float s_c[2][kCentTile * kF32Pitch];
  __shared__ float s_norm2[4];
  __shared__ unsigned s_close, s_odd, s_ncand;
  __shared__ int s_list[kF32Keys];                       // keys that are scored against every centroid
  __shared__ int s_cand[kF32Cand];                       // key of the workgroup << 24 | centroid
  __shared__ unsigned long long s_cscore[kF32Cand], s_kbest[kF32Keys];
  __shared__ int s_kid[kF32Keys];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int unit = blockIdx.y, h = unit % Hkv;
  const int col = lane & 31, half = lane >> 5;
  const float* cu = cent + (size_t)h * B * kD;
  const float* bu = bias ? bias + (size_t)h * B : nullptr;
  const int row = blockIdx.x * kF32Keys + wave * 32 + col;
  // the lane's features 8 g + 4 half .. + 3 of its key: the four k of matrix instructions 4 g .. 4 g + 3
  float4 xb[16];
  {
    const float* xr = x + ((size_t)unit * N + min(row, N - 1)) * kD + 4 * half;
#pragma unroll
    for (int g = 0; g < 16; ++g) xb[g] = *reinterpret_cast<const float4*>(xr + 8 * g);
  }
  // rows past the last centroid repeat it and do not count
  float4 stage[4];
  auto fetch = [&](int t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = tid + 256 * i;
      stage[i] = *reinterpret_cast<const float4*>(cu + (size_t)min(t * kCentTile + (p >> 5), B - 1) * kD + (p & 31) * 4);
    }
  };
  auto square = [](const float4& v) { return fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, v.w * v.w))); };
  float norm2 = 0.f;
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = tid + 256 * i;
      *reinterpret_cast<float4*>(&s_c[buf][(p >> 5) * kF32Pitch + (p & 31) * 4]) = stage[i];
    }
  };
  auto stash = [&](int buf) {
    store(buf);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float q = sum16(square(stage[i]));
      norm2 = fmaxf(norm2, q + __shfl_xor(q, 16));
    }
  };
  const int n_tiles = (B + kCentTile - 1) / kCentTile;
  // f(score, centroid) for the lane's scores, tile by tile; rows past the last centroid are left out
  auto walk = [&](auto f) {
    fetch(0);
    stash(0);
    fetch(min(1, n_tiles - 1));
    __syncthreads();
    for (int t = 0; t < n_tiles; ++t) {
      f32x16_t acc = {0};
      const float* c = &s_c[t & 1][col * kF32Pitch + 4 * half];
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        const float4 a = *reinterpret_cast<const float4*>(c + 8 * g);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, xb[g].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, xb[g].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, xb[g].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, xb[g].w, acc, 0, 0, 0);
      }
      stash((t + 1) & 1);
      fetch(min(t + 2, n_tiles - 1));
      // register r: centroid 8*(r/4) + 4*half + r%4 of the tile
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int b = t * kCentTile + 8 * (r / 4) + 4 * half + (r % 4);
        if (b < B) f(bu ? acc[r] + bu[b] : acc[r], b);
      }
      __syncthreads();
    }
  };
  float xn2 = 0.f, xmax = 0.f;
#pragma unroll
  for (int g = 0; g < 16; ++g) {
    xn2 += square(xb[g]);
    xmax = fmaxf(fmaxf(xmax, fmaxf(fabsf(xb[g].x), fabsf(xb[g].y))), fmaxf(fabsf(xb[g].z), fabsf(xb[g].w)));
  }
  xn2 += __shfl_xor(xn2, 32);
  xmax = fmaxf(xmax, __shfl_xor(xmax, 32));
  if (tid == 0) s_close = s_odd = s_ncand = 0u;
  float best = -INFINITY, second = -INFINITY;
  int id = 0;
  bool bad = false;                                      // a score that is no number
  walk([&](float v, int b) {
    bad |= !(v == v);
    second = fmaxf(second, fminf(best, v));
    id = v > best ? b : id;
    best = fmaxf(best, v);
  });
  norm2 = max_rows(norm2);
  if (lane == 0) s_norm2[wave] = norm2;
  __syncthreads();
  norm2 = fmaxf(fmaxf(s_norm2[0], s_norm2[1]), fmaxf(s_norm2[2], s_norm2[3]));
  // lanes l and l+32 hold the same key
  const float ob = __shfl_xor(best, 32), os = __shfl_xor(second, 32);
  const int oid = __shfl_xor(id, 32), obad = __shfl_xor((int)bad, 32);
  second = fmaxf(fmaxf(second, os), fminf(best, ob));
  id = ob > best || (ob == best && oid < id) ? oid : id;
  best = fmaxf(best, ob);
  const KeyScores ks = decide_key(best, second, bad || obad != 0, xmax, xn2, norm2, tol, row < N);
  const int key = wave * 32 + col;
  if (B > 1 && half == 0) {
    if (ks.odd) s_list[atomicAdd(&s_odd, 1u)] = row;
    else if (ks.close) atomicAdd(&s_close, 1u);
  }
  if (row < N && half == 0) ids[(size_t)unit * N + row] = id;
  if (tid < kF32Keys) {
    s_kbest[tid] = 0ull;
    s_kid[tid] = 0x7fffffff;
  }
  __syncthreads();
  // Up to eight close keys, as most workgroups have: every centroid in double precision takes half as long as the second walk and its
  // candidates, or less (2500 keys, 256 / 1024 centroids: 53.7 / 194 us in all with it, 35 to 40 / 120 to 134 so).
  const bool few = s_close <= 8u;
  if (few) {
    if (ks.close && half == 0 && B > 1) s_list[atomicAdd(&s_odd, 1u)] = row;
    __syncthreads();
  } else if (B > 1) {
    walk([&](float v, int b) {
      if (ks.lists(v)) {
        const unsigned i = atomicAdd(&s_ncand, 1u);
        if (i < (unsigned)kF32Cand) s_cand[i] = key << 24 | b;
      }
    });
    const unsigned n_cand = s_ncand;
    if (n_cand <= (unsigned)kF32Cand) {
      for (unsigned i = tid; i < n_cand; i += 256) {
        const int c = s_cand[i], at = c >> 24;
        const float* xk = x + ((size_t)unit * N + blockIdx.x * kF32Keys + at) * kD;
        const float* ck = cu + (size_t)(c & 0xffffff) * kD;
        double t = 0.0;
        for (int q = 0; q < kD; q += 16) {
          float4 a[4], w[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            a[j] = *reinterpret_cast<const float4*>(xk + q + 4 * j);
            w[j] = *reinterpret_cast<const float4*>(ck + q + 4 * j);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            t = fma((double)a[j].x, (double)w[j].x, t);
            t = fma((double)a[j].y, (double)w[j].y, t);
            t = fma((double)a[j].z, (double)w[j].z, t);
            t = fma((double)a[j].w, (double)w[j].w, t);
          }
        }
        if (bu) t += (double)bu[c & 0xffffff];
        const unsigned long long o = ordered_bits(t);
        s_cscore[i] = o;
        atomicMax(&s_kbest[at], o);
      }
      __syncthreads();
      for (unsigned i = tid; i < n_cand; i += 256)
        if (s_cscore[i] == s_kbest[s_cand[i] >> 24]) atomicMin(&s_kid[s_cand[i] >> 24], s_cand[i] & 0xffffff);
      __syncthreads();
      if (ks.close && half == 0) ids[(size_t)unit * N + row] = s_kid[key];       // every key's best is a candidate
    } else if (ks.close && half == 0) {
      s_list[atomicAdd(&s_odd, 1u)] = row;
    }
    __syncthreads();
  }
  // One or two keys: a thread to a centroid, rows straight from memory (5 us a key and 256 centroids; 15 for up to eight keys from
  // tiles).
  const int n_listed = (int)s_odd;
  if (n_listed <= 2) {
    double* const s_x = reinterpret_cast<double*>(s_cscore);             // [kD], and the waves' best
    double* const s_wbest = s_x + kD;
    int* const s_wid = s_cand;
    static_assert(kF32Cand >= kD + 4, "room for them");
    for (int i = 0; i < n_listed; ++i) {
      const size_t g = (size_t)unit * N + s_list[i];
      if (tid < kD) s_x[tid] = (double)x[g * kD + tid];
      __syncthreads();
      double most = 0.0;
      int most_id = -1;
      auto take = [&](double o, int o_id) {
        if (better(o, o_id, most, most_id)) {
          most = o;
          most_id = o_id;
        }
      };
      for (int b = tid; b < B; b += 256) {
        asm volatile("" ::: "memory");                   // hoisted out of the loop, the key's doubles would hold 256 registers
        const float4* c = reinterpret_cast<const float4*>(cu + (size_t)b * kD);
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          float4 v[16];
#pragma unroll
          for (int j = 0; j < 16; ++j) v[j] = c[16 * q + j];
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const double* xs = s_x + 64 * q + 4 * j;
            t = fma(xs[0], (double)v[j].x, t);
            t = fma(xs[1], (double)v[j].y, t);
            t = fma(xs[2], (double)v[j].z, t);
            t = fma(xs[3], (double)v[j].w, t);
          }
        }
        if (bu) t += (double)bu[b];
        take(t, b);
      }
      for (int n = 1; n < 64; n <<= 1) take(__shfl_xor(most, n), __shfl_xor(most_id, n));
      if (lane == 0) {
        s_wbest[wave] = most;
        s_wid[wave] = most_id;
      }
      __syncthreads();
      if (tid == 0) {
        for (int w = 1; w < 4; ++w) take(s_wbest[w], s_wid[w]);
        ids[g] = most_id;
      }
      __syncthreads();
    }
    return;
  }
  // every centroid, 32 keys at a time: a thread has a centroid of the tile and four of the keys (or one, of eight)
  float* const s_keys = &s_c[1][0];                      // [kScanKeys][kD]
  static_assert(kScanKeys * kD <= kCentTile * kF32Pitch, "room for them");
  for (int first = 0; first < n_listed; first += kScanKeys) {
    const int n_here = min(kScanKeys, n_listed - first), slot = tid >> 5, c_of = tid & 31;
    for (int p = tid; p < n_here * 32; p += 256)
      *reinterpret_cast<float4*>(s_keys + p * 4) = *reinterpret_cast<const float4*>(x + ((size_t)unit * N + s_list[first + (p >> 5)]) * kD + (p & 31) * 4);
    double most[kScanKeys / 8];
    int most_id[kScanKeys / 8];
#pragma unroll
    for (int k = 0; k < kScanKeys / 8; ++k) {
      most[k] = 0.0;
      most_id[k] = -1;
    }
    fetch(0);
    for (int t = 0; t < n_tiles; ++t) {
      store(0);
      fetch(min(t + 1, n_tiles - 1));
      __syncthreads();
      double sum[kScanKeys / 8] = {0.0};
      auto score = [&](auto per) {                       // (a branch inside the loop would have every LDS read waited for)
#pragma unroll 4
        for (int q = 0; q < kD; q += 4) {
          const float4 c = *reinterpret_cast<const float4*>(&s_c[0][c_of * kF32Pitch + q]);
#pragma unroll
          for (int k = 0; k < decltype(per)::value; ++k) {
            const float4 v = *reinterpret_cast<const float4*>(s_keys + (slot + 8 * k) * kD + q);
            sum[k] = fma((double)v.x, (double)c.x, sum[k]);
            sum[k] = fma((double)v.y, (double)c.y, sum[k]);
            sum[k] = fma((double)v.z, (double)c.z, sum[k]);
            sum[k] = fma((double)v.w, (double)c.w, sum[k]);
          }
        }
      };
      if (n_here > 8) score(std::integral_constant<int, kScanKeys / 8>{});
      else score(std::integral_constant<int, 1>{});
      const int b = t * kCentTile + c_of;
      const double add = bu && b < B ? (double)bu[b] : 0.0;
#pragma unroll
      for (int k = 0; k < kScanKeys / 8; ++k) {
        if (bu) sum[k] += add;
        if (b < B && (most_id[k] < 0 || sum[k] > most[k])) {
          most[k] = sum[k];
          most_id[k] = b;
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kScanKeys / 8; ++k) {
      for (int n = 16; n > 0; n >>= 1) {
        const double o = __shfl_xor(most[k], n);
        const int o_id = __shfl_xor(most_id[k], n);
        if (better(o, o_id, most[k], most_id[k])) {
          most[k] = o;
          most_id[k] = o_id;
        }
      }
      if (c_of == 0 && slot + 8 * k < n_here) ids[(size_t)unit * N + s_list[first + slot + 8 * k]] = most_id[k];
    }
  }
}

}  // namespace

// header | cmax[<=4095 floats] + 1 word: keys re-scored by the last call (16 KiB) | flagged row list [rows] int32
size_t assign_workspace_bytes(long long rows) {
  return (size_t)SAAP_WS_HEADER_BYTES + 16384 + (size_t)rows * sizeof(int32_t);
}

}  // namespace saap

using namespace saap;

extern "C" int32_t saap_assign_keys(const void* x, const void* centroids, const float* bias,
                                    int32_t* bucket_ids, int32_t S, int32_t Hkv, int32_t N, int32_t B,
                                    int32_t d, int32_t dtype, void* ws, size_t ws_bytes, void* stream) {
  const Call call(stream);
  saap_trace_arm();
  if (!x || !centroids || !bucket_ids || !ws) return SAAP_INVALID_ARG;
  if (!aligned16(x) || !aligned16(centroids) || !aligned16(bucket_ids) || !aligned16(ws)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || N <= 0 || B <= 0) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  const long long rows = units * N;
  if (rows > 0x7fffffffLL || units > 65535 || Hkv > 4095 || B >= (1 << 24)) return SAAP_UNSUPPORTED;
  if (ws_bytes < assign_workspace_bytes(rows)) return SAAP_WORKSPACE_TOO_SMALL;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const int cus = device_cus();

  // fp32 accumulation of 128 products (exact ones of bf16 values, rounded ones of fp32 values): |error| <= 128 * 2^-24 * |x| |c| per
  // score; two scores are compared, and a factor 4 of head-room covers the matrix core's internal summation order.
  const float tol = 8.0f * 128.0f * 5.9604645e-8f;
  if (dtype == SAAP_F32) {
    // A workgroup per key that scores it exactly, or matrix instructions for 128 keys of a (sequence, head) at a time: both take a time
    // that grows with the centroids, the former with the keys (2048 keys, 64 / 256 / 1024 centroids 11.1 / 34 / 119 us), the latter with
    // the rounds of two workgroups per compute unit, however few keys they hold (10.7 / 30 / 106 us a round without close keys, 14 to
    // 17 / 35 to 40 / 120 to 134 with some).  512 sequences of 8 heads, 64 centroids: one key each 19 us exactly, 90 otherwise, four 62 and 89; 64 of 8 heads,
    // eight keys each 19 and 15 to 20.
    const long long wgs_of_unit = (N + kF32Keys - 1) / kF32Keys, rounds = (wgs_of_unit * units + 2 * cus - 1) / (2 * cus);
    if (rows <= 8ll * cus * rounds) {
      hipLaunchKernelGGL(assign_exact_f32_kernel, dim3((unsigned)rows), dim3(256), 0, hs, static_cast<const float*>(x),
                         static_cast<const float*>(centroids), bias, bucket_ids, Hkv, N, B);
      return launch_status();
    }
    hipLaunchKernelGGL(assign_f32_kernel, dim3((unsigned)((N + kF32Keys - 1) / kF32Keys), (unsigned)units), dim3(256), 0, hs,
                       static_cast<const float*>(x), static_cast<const float*>(centroids), bias, bucket_ids, Hkv, N, B, tol);
    return launch_status();
  }

  unsigned* n_flagged = reinterpret_cast<unsigned*>(ws);   // header words 0..Hkv, zero on entry: list lengths, arrivals
  const size_t list_cap = (size_t)S * N;                   // entries per head's list
  float* cmax = reinterpret_cast<float*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  int32_t* flagged = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES + 16384);
  const bf16_t* xb = static_cast<const bf16_t*>(x);
  const bf16_t* cb = static_cast<const bf16_t*>(centroids);
  const dim3 grid((unsigned)((N + kRowsPerWg - 1) / kRowsPerWg), (unsigned)units);
  // The norms take a workgroup some 0.1 us per slab of centroids and round of workgroups (two per compute unit), a launch of their
  // own 2.5 us and, behind other work, 4.7.
  const long long rounds = ((long long)grid.x * units + 2 * cus - 1) / (2 * cus);
  const bool own_norms = rounds * ((B + kSlab - 1) / kSlab) <= 16;
  if (!own_norms) hipLaunchKernelGGL(cent_norm_kernel, dim3((unsigned)Hkv), dim3(kNormThreads), 0, hs, cb, cmax, B);
  auto launch = [&](auto has_bias, auto norms, auto ragged) {
    hipLaunchKernelGGL((assign_mfma_kernel<decltype(has_bias)::value, decltype(norms)::value, decltype(ragged)::value>), grid, dim3(256), 0, hs,
                       xb, cb, bias, cmax, bucket_ids, flagged, n_flagged, list_cap, Hkv, N, B, tol);
  };
  auto as_constant = [](bool v, auto f) { v ? f(std::true_type{}) : f(std::false_type{}); };
  as_constant(bias != nullptr, [&](auto has_bias) {
    as_constant(own_norms, [&](auto norms) { as_constant(B % kSlab != 0, [&](auto ragged) { launch(has_bias, norms, ragged); }); });
  });
  unsigned* stat = reinterpret_cast<unsigned*>(cmax) + 4095;
  // workgroups per head: one per compute unit over all heads together, as many as run at once (two rounds of them, most with no
  // group to score, ended 3 us later)
  const unsigned per_head = (unsigned)((cus + Hkv - 1) / Hkv);
  hipLaunchKernelGGL(assign_rescore_kernel, dim3((unsigned)Hkv, per_head), dim3(kRescoreThreads), 0, hs, xb, cb, bias, cmax,
                     bucket_ids, flagged, n_flagged, stat, list_cap, Hkv, B, tol);
  return launch_status();
}
