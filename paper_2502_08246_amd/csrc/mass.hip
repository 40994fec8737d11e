// bucket_attention_mass: the share of a query's softmax attention that falls into each bucket,
//   mass[b] = sum over the member keys n of bucket b of softmax_n(scale * <q, k_n>)
// with the softmax taken over ALL keys of the (sequence, KV head).  This is the row of A * H_k
// that the query model f_q is trained towards (Section 4 "Learning the query assignment", Eq. 1
// of arXiv 2502.08246); summed over a selection it is the attention mass the selection captures.
//
// Two kernels over the bucket-sorted cache (only K is read, 256 bytes per bf16 key):
//   * partial: a wave takes whole buckets (contiguous runs of rows); 16 lanes read one row with
//     one 16-byte load each, eight rows per group in flight; per bucket and head it keeps the
//     maximum m of t = log2(e) * scale * <q,k> and s = sum 2^(t - m), and writes (m, s);
//   * normalise: per query head, M = max_b m_b, L = sum_b s_b 2^(m_b - M), mass_b = s_b 2^(m_b - M) / L.
#include "common.h"

namespace saap {
namespace {

constexpr int kMassThreads = 256;
constexpr int kInFlight = 8;      // rows a 16-lane group has in flight

template <typename T, int G>
__global__ void __launch_bounds__(kMassThreads)
mass_partial_kernel(const T* __restrict__ q, const T* __restrict__ K, const int32_t* __restrict__ off,
                    const int32_t* __restrict__ len, float2* __restrict__ part, long long rows, int B,
                    float scale_log2) {
  const int unit = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane & 15, grp = lane >> 4;
  Vec8<T> qv[G];
#pragma unroll
  for (int g = 0; g < G; ++g) qv[g].load(q + ((size_t)unit * G + g) * kD + sub * 8);
  const T* Kb = K + (size_t)unit * rows * kD + sub * 8;
  const int n_waves = gridDim.x * (kMassThreads / 64);
  for (int b = blockIdx.x * (kMassThreads / 64) + wave; b < B; b += n_waves) {
    const int first = off[(size_t)unit * (B + 1) + b], n = len[(size_t)unit * B + b];
    float m[G], s[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      m[g] = kNegBig;
      s[g] = 0.f;
    }
    for (int r0 = grp; r0 < n; r0 += 4 * kInFlight) {      // rows r0, r0+4, ... of this 16-lane group
      Vec8<T> kv[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) kv[u].load(Kb + (size_t)(first + min(r0 + 4 * u, n - 1)) * kD);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float t[kInFlight];
        float bm = -INFINITY;
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
          const float d = sum16(kv[u].dot(qv[g])) * scale_log2;
          t[u] = r0 + 4 * u < n ? d : -INFINITY;
          bm = fmaxf(bm, t[u]);                           // finite: row r0 is real
        }
        const float mn = fmaxf(m[g], bm);
        float acc = s[g] * fast_exp2(m[g] - mn);
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) acc += fast_exp2(t[u] - mn);
        s[g] = acc;
        m[g] = mn;
      }
    }
    // the four groups of the wave
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float M = max_rows(m[g]);
      const float S = sum_rows(s[g] * fast_exp2(m[g] - M));
      if (lane == 0) part[((size_t)unit * B + b) * G + g] = make_float2(M, S);
    }
  }
}

template <int G>
__global__ void __launch_bounds__(256)
mass_normalise_kernel(const float2* __restrict__ part, float* __restrict__ mass, float* __restrict__ lse, int B) {
  __shared__ float s_red[4];
  const int row = blockIdx.x, unit = row / G, g = row % G, tid = threadIdx.x;
  const float2* pu = part + (size_t)unit * B * G + g;
  float M = kNegBig;
  for (int b = tid; b < B; b += 256) M = fmaxf(M, pu[(size_t)b * G].x);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
  if ((tid & 63) == 0) s_red[tid >> 6] = M;
  __syncthreads();
  M = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
  __syncthreads();
  float L = 0.f;
  for (int b = tid; b < B; b += 256) {
    const float2 p = pu[(size_t)b * G];
    L = fmaf(p.y, fast_exp2(p.x - M), L);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) L += __shfl_xor(L, o);
  if ((tid & 63) == 0) s_red[tid >> 6] = L;
  __syncthreads();
  L = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
  const float inv = L > 0.f ? 1.0f / L : 0.f;
  for (int b = tid; b < B; b += 256) {
    const float2 p = pu[(size_t)b * G];
    mass[(size_t)row * B + b] = p.y * fast_exp2(p.x - M) * inv;
  }
  if (tid == 0 && lse) lse[row] = L > 0.f ? (M + __log2f(L)) * kLn2 : -INFINITY;
}

template <typename T, int G>
void launch_mass(const void* q, const void* K, const int32_t* off, const int32_t* len, float2* part, float* mass,
                 float* lse, long long units, long long rows, int B, float scale_log2, hipStream_t hs) {
  const int cus = device_cus();
  // enough workgroups per unit to fill the chip a few times, never more waves than buckets
  long long per_unit = ((long long)cus * 8 + units - 1) / units;
  const long long by_buckets = (B + kMassThreads / 64 - 1) / (kMassThreads / 64);
  if (per_unit > by_buckets) per_unit = by_buckets;
  hipLaunchKernelGGL((mass_partial_kernel<T, G>), dim3((unsigned)per_unit, (unsigned)units), dim3(kMassThreads), 0, hs,
                     static_cast<const T*>(q), static_cast<const T*>(K), off, len, part, rows, B, scale_log2);
  hipLaunchKernelGGL(mass_normalise_kernel<G>, dim3((unsigned)(units * G)), dim3(256), 0, hs, part, mass, lse, B);
}

// ---- many queries per KV head (a training batch): scores on the matrix cores -----------------------
// 32 QT queries per wave sit in registers as the B operand of v_mfma_f32_32x32x16_bf16 (one lane per query and half of
// the key rows); the keys of a bucket stream through LDS in tiles of 32 as the A operand (padded rows, whole-row loads,
// double buffered, the next tile's loads in flight), so that one lane sees 16 scores of its query per tile and keeps the
// bucket's running maximum and sum for it.  A workgroup takes every n_slices-th bucket.  part[(unit*B + b)*R + q] = (m, s).
// Per tile and 32 queries a wave issues 8 matrix instructions (256 cycles) and about 50 vector instructions, 16 of them
// exponentials at half the rate (280 cycles); the two kinds overlap only in part whatever their order (a loop of nothing else:
// 455 ns for two such tiles on random numbers, where the sum is 531), so that waves in flight decide: 128 registers, four
// workgroups per compute unit.  8 heads, 1000 queries, 131072 keys: 486 us with one key tile waited for at a time, 359 with two
// tiles of loads in flight and three workgroups, 347 now; 323 with neither masks, pairs nor barriers.  (The weights of a tile
// under the products of the next in one wave need 32 more registers: 395 to 420 us.)
constexpr int kMassPitch = 136;      // bf16 elements per LDS row (272 bytes: conflict-free b128 reads)
constexpr int kMassTile = 32;        // keys per tile
constexpr int kMassBuckets = 512;    // buckets per workgroup at most

// SIGN of the score scale: below zero the largest score is the smallest product.
template <int QT, int SIGN>
__global__ void __launch_bounds__(256, 4)
mass_mfma_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ K, const int32_t* __restrict__ off,
                 const int32_t* __restrict__ len, float2* __restrict__ part, long long rows, int B, int R,
                 float scale_log2) {
  typedef __attribute__((ext_vector_type(16))) float f32x16_t;
  __shared__ __align__(16) bf16_t s_k[2][kMassTile * kMassPitch];
  __shared__ int4 s_list[kMassBuckets];               // bucket, first row, length
  __shared__ int s_live[4], s_tiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  const int unit = blockIdx.z;
  const int q0 = (blockIdx.y * 4 + wave) * 32 * QT + col;
  // B operand: lane holds features 16*step + 8*half .. +7 of query `col` of each tile (idle columns repeat the last query)
  bf16x8_t xb[QT][8];
#pragma unroll
  for (int i = 0; i < QT; ++i) {
    const bf16_t* qr = q + ((size_t)unit * R + min(q0 + 32 * i, R - 1)) * kD + half * 8;
#pragma unroll
    for (int st = 0; st < 8; ++st) xb[i][st] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qr + st * 16));
  }
  const bf16_t* Ku = K + (size_t)unit * rows * kD;
  // The workgroup's buckets (every gridDim.x-th) that hold keys, in LDS, so that walking on to the next one is no trip to
  // memory, in ascending order: the reference below goes from bucket to bucket, so the order is part of the result's bits.
  // The pairs of a bucket without keys are written here.
  auto pair_of = [&](int b, int i) { return part + ((size_t)unit * B + b) * R + q0 + 32 * i; };
  if (tid == 0) s_tiles = 0;
  __syncthreads();
  int n_before = 0;
  for (int b0 = blockIdx.x; b0 < B; b0 += 256 * gridDim.x) {      // at most kMassBuckets: checked on the host
    const int b = b0 + tid * gridDim.x, at = min(b, B - 1);
    const int n = len[(size_t)unit * B + at], first = off[(size_t)unit * (B + 1) + at];
    const bool live = b < B && n > 0;
    const unsigned long long mask = __ballot(live);
    if (lane == 0) s_live[wave] = __popcll(mask);
    __syncthreads();
    int place = n_before + __popcll(mask & ((1ull << lane) - 1ull));
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      place += w < wave ? s_live[w] : 0;
      n_before += s_live[w];
    }
    if (live) {
      s_list[place] = make_int4(b, first, n, 0);
      atomicAdd(&s_tiles, (n + kMassTile - 1) / kMassTile);
    }
    __syncthreads();
  }
  for (int b = blockIdx.x; b < B; b += gridDim.x)
    if (half == 0 && len[(size_t)unit * B + b] <= 0)
#pragma unroll
      for (int i = 0; i < QT; ++i)
        if (q0 + 32 * i < R) *pair_of(b, i) = make_float2(kNegBig, 0.f);
  __syncthreads();
  const int n_live = __builtin_amdgcn_readfirstlane(n_before), n_tiles = __builtin_amdgcn_readfirstlane(s_tiles);
  if (n_tiles == 0) return;
  // Tiles of 32 keys, bucket by bucket; the walk is the same in all waves (scalar registers) and, past the end, comes back
  // to the last bucket (valid loads that nobody uses).
  struct Tile { int j, b, first, n, t0; };
  auto enter = [&](int j) {
    const int4 e = s_list[j];
    return Tile{j, __builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y), __builtin_amdgcn_readfirstlane(e.z), 0};
  };
  auto after = [&](const Tile& t) {
    const bool same = t.t0 + kMassTile < t.n;
    Tile r = enter(same ? t.j : min(t.j + 1, n_live - 1));
    r.t0 = same ? t.t0 + kMassTile : 0;
    return r;
  };

  struct Staged { u32x4_t p[2]; };        // native vectors: a uint4 here ends up in scratch memory
  // 32 rows x 16 pieces of 16 bytes, two per thread; rows past the bucket repeat its last key
  auto fetch = [&](Staged& g, const Tile& t) {
    const char* rows_at = reinterpret_cast<const char*>(Ku + (size_t)(t.first + t.t0) * kD);      // the whole workgroup's
    const unsigned last = t.n - 1 - t.t0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned pi = tid + 256 * i, r = pi >> 4, pc = pi & 15;
      g.p[i] = *reinterpret_cast<const u32x4_t*>(rows_at + (min(r, last) * (kD * 2) + pc * 16));
    }
  };
  auto stash = [&](const Staged& g, int buf) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int pi = tid + 256 * i, r = pi >> 4, pc = pi & 15;
      *reinterpret_cast<u32x4_t*>(&s_k[buf][r * kMassPitch + pc * 8]) = g.p[i];
    }
  };
  // Sums are kept relative to a reference m (base-2 logits) that stays over the buckets and moves only when a tile's sum
  // says that scores lie far above it, so that no maximum is taken over a tile's scores: within 2^64 above the
  // reference a sum loses nothing, and a key so far below it that its weight vanishes is as far below the largest key.
  constexpr float kFarAbove = 1.8446744e19f;             // 2^64
  float m[QT], s[QT];
#pragma unroll
  for (int i = 0; i < QT; ++i) {
    m[i] = kNegBig;
    s[i] = 0.f;
  }
  auto compute = [&](int buf, const Tile& t) {
    f32x16_t acc[QT];
#pragma unroll
    for (int i = 0; i < QT; ++i) acc[i] = (f32x16_t){0};
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const bf16x8_t a = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(&s_k[buf][col * kMassPitch + st * 16 + half * 8]));
#pragma unroll
      for (int i = 0; i < QT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xb[i][st], acc[i], 0, 0, 0);
    }
    // register r of this lane: key t0 + 8*(r/4) + 4*half + r%4 against query `col`
    float to_log2 = scale_log2;
    if (t.t0 + kMassTile > t.n) {                        // the bucket's last tile: rows past its end do not count
      if (SIGN == 0) to_log2 = 1.f;                      // scaled here: zero times the mask would be no number
      const int left = t.n - t.t0 - 4 * half;
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int i = 0; i < QT; ++i) {
          const bool in = 8 * (r / 4) + (r % 4) < left;
          acc[i][r] = !in ? (SIGN < 0 ? INFINITY : -INFINITY) : SIGN == 0 ? acc[i][r] * 0.f : acc[i][r];
        }
    }
    auto weights = [&](const f32x16_t& c, float ref) {
      float add[4];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float w = fast_exp2(fmaf(c[r], to_log2, -ref));
        add[r % 4] = r < 4 ? w : add[r % 4] + w;
      }
      return (add[0] + add[1]) + (add[2] + add[3]);
    };
#pragma unroll
    for (int i = 0; i < QT; ++i) {
      float add = weights(acc[i], m[i]);
      if (__builtin_expect(__ballot(!(add < kFarAbove)) != 0ull, 0)) {      // the first tile, and rarely after it
        float best = acc[i][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) best = SIGN < 0 ? fminf(best, acc[i][r]) : fmaxf(best, acc[i][r]);
        const float mn = fmaxf(m[i], best * to_log2);   // stays where this half holds no key above it
        add = weights(acc[i], mn);
        s[i] *= fast_exp2(m[i] - mn);
        m[i] = mn;
      }
      s[i] += add;
    }
    if (t.t0 + kMassTile >= t.n) {                       // the bucket is complete; lanes l and l+32 hold the same query
      float2* const pairs = part + ((size_t)unit * B + t.b) * R;
#pragma unroll
      for (int i = 0; i < QT; ++i) {
        const float mo = other_half(m[i]), so = other_half(s[i]);
        const float M = fmaxf(m[i], mo);
        const float S = s[i] * fast_exp2(m[i] - M) + so * fast_exp2(mo - M);
        if (half == 0 && q0 + 32 * i < R) pairs[(unsigned)(q0 + 32 * i)] = make_float2(M, S);
        s[i] = 0.f;
        m[i] = m[i] < INFINITY ? m[i] : kNegBig;         // no reference for the buckets that follow
      }
    }
  };
  Tile t0 = enter(0), t1 = after(t0);
  Staged st;
  fetch(st, t0);
  stash(st, 0);
  fetch(st, t1);
  __syncthreads();
  for (int c = 0; c < n_tiles; ++c) {
    stash(st, (c + 1) & 1);
    const Tile t2 = after(t1);
    fetch(st, t2);
    compute(c & 1, t0);
    __syncthreads();
    t0 = t1;
    t1 = t2;
  }
}

// mass[(unit*R + q)*B + b] = s_b 2^(m_b - M) / L for 32 queries per workgroup: thread (query, bucket group).  Two passes
// over the pairs, eight loads in flight per thread: maximum and sum in one (the sum rescaled when the maximum moves), then
// the masses, in tiles of 32 queries x 64 buckets through LDS so that the rows of `mass` are written in whole lines
// (three passes, one load at a time: 130 us for 8 x 1000 queries and 1024 buckets, 32 us now).
__global__ void __launch_bounds__(256)
mass_normalise_batch_kernel(const float2* __restrict__ part, float* __restrict__ mass, float* __restrict__ lse, int B,
                            int R) {
  constexpr int kDeep = 8;
  __shared__ float s_m[8][32], s_l[8][32];
  __shared__ float s_tile[32][65];
  const int tid = threadIdx.x, ql = tid & 31, bg = tid >> 5;
  const int unit = blockIdx.y, q0 = blockIdx.x * 32;
  const int qi = min(q0 + ql, R - 1);
  const float2* pu = part + (size_t)unit * B * R + qi;
  float M = kNegBig, L = 0.f;
  for (int b0 = bg; b0 < B; b0 += 8 * kDeep) {
    float2 p[kDeep];
#pragma unroll
    for (int u = 0; u < kDeep; ++u) p[u] = pu[(size_t)min(b0 + 8 * u, B - 1) * R];
    float bm = M;
#pragma unroll
    for (int u = 0; u < kDeep; ++u) bm = fmaxf(bm, p[u].x);
    L *= fast_exp2(M - bm);
    M = bm;
#pragma unroll
    for (int u = 0; u < kDeep; ++u)
      if (b0 + 8 * u < B) L = fmaf(p[u].y, fast_exp2(p[u].x - M), L);
  }
  s_m[bg][ql] = M;
  s_l[bg][ql] = L;
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 8; ++g) M = fmaxf(M, s_m[g][ql]);
  L = 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g) L = fmaf(s_l[g][ql], fast_exp2(s_m[g][ql] - M), L);      // fixed order
  const float inv = L > 0.f ? 1.0f / L : 0.f;
  if (bg == 0 && q0 + ql < R && lse) lse[(size_t)unit * R + q0 + ql] = L > 0.f ? (M + __log2f(L)) * kLn2 : -INFINITY;
  for (int bt = 0; bt < B; bt += 8 * kDeep) {
    float2 p[kDeep];
#pragma unroll
    for (int u = 0; u < kDeep; ++u) p[u] = pu[(size_t)min(bt + bg + 8 * u, B - 1) * R];
    __syncthreads();                                     // the tile before has been written out
#pragma unroll
    for (int u = 0; u < kDeep; ++u) s_tile[ql][bg + 8 * u] = p[u].y * fast_exp2(p[u].x - M) * inv;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = (tid >> 6) + 4 * i, b = bt + (tid & 63);
      if (q0 + row < R && b < B) mass[((size_t)unit * R + q0 + row) * B + b] = s_tile[row][tid & 63];
    }
  }
}

// The same for up to 32 PER buckets: 32 threads to a query, each holding its pairs, which are read once and all in flight together
// (8 x 1000 queries and 1024 buckets: 32.7 us in the kernel above, 22.6 here, 98 MB).
template <int PER>
__global__ void __launch_bounds__(1024)
mass_normalise_held_kernel(const float2* __restrict__ part, float* __restrict__ mass, float* __restrict__ lse, int B, int R) {
  constexpr int kGroups = 32, kTile = 256;               // buckets per tile on the way out
  __shared__ float s_m[kGroups][32], s_l[kGroups][32];
  __shared__ float s_tile[32][kTile + 1];
  const int tid = threadIdx.x, ql = tid & 31, bg = tid >> 5;
  const int unit = blockIdx.y, q0 = blockIdx.x * 32;
  const float2* pu = part + (size_t)unit * B * R + min(q0 + ql, R - 1);
  float2 p[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) p[u] = pu[(size_t)min(bg + kGroups * u, B - 1) * R];
  float M = kNegBig, L = 0.f;
#pragma unroll
  for (int u = 0; u < PER; ++u) M = fmaxf(M, p[u].x);
  s_m[bg][ql] = M;
  __syncthreads();
#pragma unroll
  for (int g = 0; g < kGroups; ++g) M = fmaxf(M, s_m[g][ql]);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    p[u].y *= fast_exp2(p[u].x - M);
    if (bg + kGroups * u < B) L += p[u].y;
  }
  s_l[bg][ql] = L;
  __syncthreads();
  L = 0.f;
#pragma unroll
  for (int g = 0; g < kGroups; ++g) L += s_l[g][ql];      // fixed order
  const float inv = L > 0.f ? 1.0f / L : 0.f;
  if (bg == 0 && q0 + ql < R && lse) lse[(size_t)unit * R + q0 + ql] = L > 0.f ? (M + __log2f(L)) * kLn2 : -INFINITY;
#pragma unroll
  for (int t = 0; t < PER * kGroups / kTile; ++t) {
    if (t * kTile >= B) break;
    if (t > 0) __syncthreads();                          // the tile before has been written out
#pragma unroll
    for (int u = 0; u < kTile / kGroups; ++u) s_tile[ql][bg + kGroups * u] = p[t * (kTile / kGroups) + u].y * inv;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32 * kTile / 1024; ++i) {
      const int row = (tid >> 8) + 4 * i, b = t * kTile + (tid & 255);
      if (q0 + row < R && b < B) mass[((size_t)unit * R + q0 + row) * B + b] = s_tile[row][tid & 255];
    }
  }
}

}  // namespace

size_t mass_batch_workspace_bytes(long long units, long long R, int B) {
  return (size_t)SAAP_WS_HEADER_BYTES + (size_t)units * R * B * sizeof(float2);
}

size_t mass_workspace_bytes(long long units, int G, int B) {
  return (size_t)SAAP_WS_HEADER_BYTES + (size_t)units * B * G * sizeof(float2);
}

}  // namespace saap

using namespace saap;

extern "C" int32_t saap_bucket_attention_mass(const void* q, const void* Ksorted, const int32_t* off,
                                              const int32_t* len, float scale, float* mass, float* lse, int32_t S,
                                              int32_t Hq, int32_t Hkv, int32_t Ncap, int32_t B, int32_t d,
                                              int32_t dtype, void* ws, size_t ws_bytes, void* stream) {
  const Call call(stream);
  if (!q || !Ksorted || !off || !len || !mass || !ws) return SAAP_INVALID_ARG;
  if (!aligned16(q) || !aligned16(Ksorted) || !aligned16(ws)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0 || Ncap <= 0 || B <= 0) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD) return SAAP_UNSUPPORTED;
  const int G = Hq / Hkv;
  if (G != 1 && G != 2 && G != 4 && G != 8) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535) return SAAP_UNSUPPORTED;
  if (ws_bytes < mass_workspace_bytes(units, G, B)) return SAAP_WORKSPACE_TOO_SMALL;
  float2* part = reinterpret_cast<float2*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const float sl2 = scale * kLog2e;
#define SAAP_CASE(TT, GG) launch_mass<TT, GG>(q, Ksorted, off, len, part, mass, lse, units, Ncap, B, sl2, hs); break
  if (dtype == SAAP_BF16) {
    switch (G) {
      case 1: SAAP_CASE(bf16_t, 1);
      case 2: SAAP_CASE(bf16_t, 2);
      case 4: SAAP_CASE(bf16_t, 4);
      case 8: SAAP_CASE(bf16_t, 8);
    }
  } else {
    switch (G) {
      case 1: SAAP_CASE(float, 1);
      case 2: SAAP_CASE(float, 2);
      case 4: SAAP_CASE(float, 4);
      case 8: SAAP_CASE(float, 8);
    }
  }
#undef SAAP_CASE
  return launch_status();
}

extern "C" int32_t saap_bucket_attention_mass_batch(const void* q, const void* Ksorted, const int32_t* off,
                                                    const int32_t* len, float scale, float* mass, float* lse,
                                                    int32_t S, int32_t Hkv, int32_t R, int32_t Ncap, int32_t B,
                                                    int32_t d, int32_t dtype, void* ws, size_t ws_bytes,
                                                    void* stream) {
  const Call call(stream);
  if (!q || !Ksorted || !off || !len || !mass || !ws) return SAAP_INVALID_ARG;
  if (!aligned16(q) || !aligned16(Ksorted) || !aligned16(mass) || !aligned16(ws)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || R <= 0 || Ncap <= 0 || B <= 0) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD || dtype != SAAP_BF16) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535 || (R + 127) / 128 > 65535) return SAAP_UNSUPPORTED;
  if (ws_bytes < mass_batch_workspace_bytes(units, R, B)) return SAAP_WORKSPACE_TOO_SMALL;
  float2* part = reinterpret_cast<float2*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  hipStream_t hs = static_cast<hipStream_t>(stream);
  // 256 queries per workgroup (two tiles per wave share the key operand's LDS reads) unless 128 leave fewer idle
  const int qt = (R + 255) / 256 * 256 <= (R + 127) / 128 * 128 ? 2 : 1;
  const int qblocks = (R + 128 * qt - 1) / (128 * qt);
  // bucket slices: enough workgroups to fill the chip a few times (buckets differ in size), never more than buckets
  long long slices = ((long long)device_cus() * 8 + units * qblocks - 1) / (units * qblocks);
  if (slices > B) slices = B;
  if (slices < 1) slices = 1;
  if (slices < (B + kMassBuckets - 1) / kMassBuckets) slices = (B + kMassBuckets - 1) / kMassBuckets;
  const float scale_log2 = scale * kLog2e;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)slices, (unsigned)qblocks, (unsigned)units), dim3(256), 0, hs, static_cast<const bf16_t*>(q),
                       static_cast<const bf16_t*>(Ksorted), off, len, part, (long long)Ncap, B, R, scale_log2);
  };
  if (scale_log2 < 0.f) qt == 2 ? launch(mass_mfma_kernel<2, -1>) : launch(mass_mfma_kernel<1, -1>);
  else if (scale_log2 == 0.f) qt == 2 ? launch(mass_mfma_kernel<2, 0>) : launch(mass_mfma_kernel<1, 0>);
  else qt == 2 ? launch(mass_mfma_kernel<2, 1>) : launch(mass_mfma_kernel<1, 1>);
  // Pairs held in registers where their 32 threads a query each have more than four (up to 128 buckets the smaller workgroups are as
  // fast: 8 x 64 rows of 128 4.4 us, 4.7 held), in as few registers as do (288 buckets, 1000 rows: 11.4 us read twice, 11.8 with 32
  // pairs a thread, 9.9 with 16); those of more than 1024 buckets do not fit.
  const dim3 grid((unsigned)((R + 31) / 32), (unsigned)units);
  if (B <= 128) hipLaunchKernelGGL(mass_normalise_batch_kernel, grid, dim3(256), 0, hs, part, mass, lse, B, R);
  else if (B <= 256) hipLaunchKernelGGL(mass_normalise_held_kernel<8>, grid, dim3(1024), 0, hs, part, mass, lse, B, R);
  else if (B <= 512) hipLaunchKernelGGL(mass_normalise_held_kernel<16>, grid, dim3(1024), 0, hs, part, mass, lse, B, R);
  else if (B <= 1024) hipLaunchKernelGGL(mass_normalise_held_kernel<32>, grid, dim3(1024), 0, hs, part, mass, lse, B, R);
  else hipLaunchKernelGGL(mass_normalise_batch_kernel, grid, dim3(256), 0, hs, part, mass, lse, B, R);
  return launch_status();
}
