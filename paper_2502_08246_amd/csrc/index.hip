// build_bucket_index and append_keys: the CSR index of Appendix F (tensors Off, Idx) of
// arXiv 2502.08246 plus the bucket-sorted copy of K and V, and the slot append used during
// generation.
//
// The sort is a stable counting sort, deterministic by construction (no atomics decide an
// order):
//   1. hist      every workgroup counts the bucket ids of its slice of positions
//   2. colscan   per bucket, exclusive scan of the slice counts over slices -> len, slice bases
//   3. scatter   exclusive scan of (len + slack) over the buckets -> off; one workgroup per slice; every wave walks
//                its part of the slice in order, 64 positions at a time; the rank of a position among equal ids
//                inside the 64 comes from ballots, the waves' and the buckets' running positions are kept in LDS -> idx
//   4. permute   rows of K and V are copied to their slot, 16 bytes per lane, whole rows
// A short context takes one launch: order_direct does steps 1 to 3.
//
// With a resident block (attention sink + recent keys, Section 3 "Per-head attention span")
// only the positions [lo, hi) go through steps 1-3; the resident positions are placed by
// their slot rule into one more run behind the B buckets, and window_push moves one key per
// decode step from that run into its bucket.
#include <algorithm>

#include "common.h"

namespace saap {
namespace {

constexpr int kSlice = 2048;   // positions per slice (one workgroup of the histogram and of the scatter each)

__global__ void __launch_bounds__(256)
hist_kernel(const int32_t* __restrict__ ids, int32_t* __restrict__ slice_hist, int N, int B, int n_slices,
            int lo, int hi) {
  extern __shared__ int s_cnt[];
  const int slice = blockIdx.x, unit = blockIdx.y;
  for (int b = threadIdx.x; b < B; b += blockDim.x) s_cnt[b] = 0;
  __syncthreads();
  const int n0 = slice * kSlice, n1 = min(n0 + kSlice, N);
  const int32_t* idu = ids + (size_t)unit * N;
  int mine[kSlice / 256];
#pragma unroll
  for (int k = 0; k < kSlice / 256; ++k) {
    const int n = n0 + threadIdx.x + k * 256;
    mine[k] = n < n1 && n >= lo && n < hi ? idu[n] : -1;
  }
#pragma unroll
  for (int k = 0; k < kSlice / 256; ++k)
    if (mine[k] >= 0 && mine[k] < B) atomicAdd(&s_cnt[mine[k]], 1);
  __syncthreads();
  int32_t* out = slice_hist + ((size_t)unit * n_slices + slice) * B;
  for (int b = threadIdx.x; b < B; b += blockDim.x) out[b] = s_cnt[b];
}

// One thread per (unit, bucket): counts of the slices -> exclusive bases, total -> len.
__global__ void __launch_bounds__(256)
colscan_kernel(int32_t* __restrict__ slice_hist, int32_t* __restrict__ len, int B, int n_slices, int lstride) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x, unit = blockIdx.y;
  if (b >= B) return;
  int32_t* col = slice_hist + (size_t)unit * n_slices * B + b;
  int run = 0;
  int s = 0;
  for (; s + 8 <= n_slices; s += 8) {
    int c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = col[(size_t)(s + i) * B];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      col[(size_t)(s + i) * B] = run;
      run += c[i];
    }
  }
  for (; s < n_slices; ++s) {
    const int c = col[(size_t)s * B];
    col[(size_t)s * B] = run;
    run += c;
  }
  len[(size_t)unit * lstride + b] = run;
}

// Resident key j of a unit (j-th resident position in ascending order): its place in the resident run, its id kept
// for the later move; slots that stay empty (context shorter than the run) are marked.
__device__ __forceinline__ void place_resident(int j, const int32_t* __restrict__ ids, int32_t* __restrict__ idx,
                                               int32_t* __restrict__ rid, int base, int N, int n_sink, int n_recent, int n_res) {
  const int W = n_sink + n_recent;
  if (j >= n_res) {              // slot r(p) = p while the block is not full: slots n_res.. are empty
    rid[j] = -1;
    idx[base + j] = -1;
    return;
  }
  const int p = (N <= W || j < n_sink) ? j : N - n_recent + (j - n_sink);
  const int r = p < n_sink ? p : n_sink + (p - n_sink) % n_recent;
  idx[base + r] = p;
  rid[r] = ids[p];
}

__global__ void __launch_bounds__(256)
resident_kernel(const int32_t* __restrict__ ids, const int32_t* __restrict__ off, int32_t* __restrict__ idx,
                int32_t* __restrict__ res_ids, int N, int Ncap, int B, int n_sink, int n_recent, int n_res) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x, unit = blockIdx.y;
  const int W = n_sink + n_recent;
  if (j >= W) return;
  place_resident(j, ids + (size_t)unit * N, idx + (size_t)unit * Ncap, res_ids + (size_t)unit * W, off[(size_t)unit * (B + 2) + B], N,
                 n_sink, n_recent, n_res);
}

__global__ void __launch_bounds__(256) fill_i32_kernel(int32_t* p, size_t n, int32_t v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Counters of the waves of a workgroup, 16 bits per (wave, bucket), two buckets to a word.
__device__ __forceinline__ void wave_count_add(unsigned* cnt, int b, unsigned n) { atomicAdd(&cnt[b >> 1], n << (16 * (b & 1))); }
__device__ __forceinline__ unsigned wave_count(const unsigned* cnt, int b) { return (cnt[b >> 1] >> (16 * (b & 1))) & 0xffffu; }

// The position in `b` (-1: none) of each of the wave's 64 lanes goes to its slot.  next[b]: first slot of bucket b of
// this slice; mine: the wave's counters, holding what the waves before it (and its own earlier rounds) have placed.
__device__ __forceinline__ void place_round(int b, int n, int id_bits, const int* next, unsigned* mine, int32_t* __restrict__ ix) {
  const int lane = threadIdx.x & 63;
  const unsigned long long below = (1ull << lane) - 1ull;
  const bool ok = b >= 0;
  unsigned long long eq = __ballot(ok);
  for (int i = 0; i < id_bits; ++i) {
    const bool bit = (b >> i) & 1;
    const unsigned long long m = __ballot(bit);
    eq &= bit ? m : ~m;
  }
  if (ok) {
    const int rank = __popcll(eq & below);
    ix[next[b] + (int)wave_count(mine, b) + rank] = n;
    // one update per id, by the last of its lanes; lanes of two ids may share a word, hence an atomic
    if ((eq & ~below) == (1ull << lane)) wave_count_add(mine, b, (unsigned)__popcll(eq));
  }
  // one wave: its LDS accesses execute in order, so the update is seen by the next 64 positions.  No barrier:
  // a barrier also waits for the index store above, one memory round trip per 64 positions
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// One workgroup of four waves per slice of 2048 positions, 512 of them to a wave.  The waves count their parts first, so
// that each knows what the others before it place: eight rounds one after the other, where one wave per slice had 32
// (8 units of 65536 positions: 22 -> 9.6 us).  The unit is the fastest grid dimension: with a multiple of 8 units all slices
// of one share an L2, where the 4-byte stores of many slices to a line of idx meet (64 units of 131072 positions: 105 -> 58 us;
// 8 of 65536: 9.6 -> 7.9).  The workgroup also marks the free slots of every n_slices-th bucket and its share of those
// behind the last run: every entry of idx is written, and the row copy reads them all.
// KW: 64 KW runs to a wave, B <= 256 KW; their lengths and earlier slices' counts are loaded with the ids, all in flight together.
// Scan and scatter, 8 units of 500000 positions, 4096 / 8192 buckets: 48 / 146 us with the scan in a launch of its own, 84 / 275 with
// 16 / 32 neighbouring runs a thread and an array more in LDS, 41 / 110 now; 64 units of 131072, 1024 / 4096 buckets: 56 / 106, 53 / 178
// and 52 / 91.
constexpr int kScatterThreads = 256, kScatterWaves = kScatterThreads / 64;
template <int KW>
__global__ void __launch_bounds__(kScatterThreads)
scatter_kernel(const int32_t* __restrict__ ids, const int32_t* __restrict__ slice_base, int32_t* __restrict__ len,
               int32_t* __restrict__ off, int32_t* __restrict__ idx, int N, int Ncap, int B,
               int n_slices, int id_bits, int lo, int hi, int slack, int W, int n_res) {
  // Runs' starts for this slice [B, to a multiple of four] | counters [waves][words]
  extern __shared__ __align__(16) int s_next[];
  __shared__ int s_wsum[kScatterWaves];
  const int unit = blockIdx.x, slice = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int words = (B + 1) / 2, padded = (B + 3) & ~3;
  unsigned* s_cnt = reinterpret_cast<unsigned*>(s_next + padded);
  const int32_t* base = slice_base + ((size_t)unit * n_slices + slice) * B;
  const int lstride = W >= 0 ? B + 1 : B;
  int32_t* l = len + (size_t)unit * lstride;
  int32_t* o = off + (size_t)unit * (lstride + 1);
  int32_t* ix = idx + (size_t)unit * Ncap;
  const int32_t* idu = ids + (size_t)unit * N;
  constexpr int kRounds = kSlice / kScatterThreads;      // of 64 positions per wave
  const int n0 = slice * kSlice + wave * (kSlice / kScatterWaves);
  int mine[kRounds];                                     // the wave's ids, loaded up front
#pragma unroll
  for (int k = 0; k < kRounds; ++k) {
    const int n = n0 + k * 64 + lane;
    mine[k] = n >= lo && n < hi ? idu[n] : -1;           // hi <= N
  }
  // the wave's share of the runs, [w0, w1): their lengths, and what earlier slices place in them
  const int w0 = wave * 64 * KW, w1 = min(w0 + 64 * KW, B);
  int run[KW], earlier[KW];
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int b = min(w0 + k * 64 + lane, B - 1);
    run[k] = l[b];
    earlier[k] = base[b];
  }
  for (int i = tid; i < kScatterWaves * words; i += kScatterThreads) s_cnt[i] = 0u;
  // Every slice scans the runs of its unit for itself: a launch between the column scan and this one takes 4.6 us (10.8 at 8192
  // buckets).  Each wave turns its runs round in the place of their starts, four neighbouring ones to a lane: no bank conflicts,
  // and no more LDS than without the scan.
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int b = w0 + k * 64 + lane;
    if (b < padded) s_next[b] = b < B ? run[k] + slack : 0;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the wave's own writes, in other lanes
  int4 four[KW / 4];
  int total = 0;
#pragma unroll
  for (int k = 0; k < KW / 4; ++k) {
    const int b = w0 + k * 256 + 4 * lane;
    four[k] = b < B ? *reinterpret_cast<const int4*>(s_next + b) : make_int4(0, 0, 0, 0);
    total += (four[k].x + four[k].y) + (four[k].z + four[k].w);
  }
  total = (int)wave_prefix_sum((unsigned)total);
  if (lane == 63) s_wsum[wave] = total;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRounds; ++k) {
    if (mine[k] >= B) mine[k] = -1;
    if (mine[k] >= 0) wave_count_add(s_cnt + wave * words, mine[k], 1u);
  }
  int at = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kScatterWaves; ++w) {
    at += w < wave ? s_wsum[w] : 0;
    all += s_wsum[w];
  }
#pragma unroll
  for (int k = 0; k < KW / 4; ++k) {
    const int4 v = four[k];
    const int sum = (v.x + v.y) + (v.z + v.w), incl = (int)wave_prefix_sum((unsigned)sum), first = at + incl - sum;
    const int b = w0 + k * 256 + 4 * lane;
    if (b < B) *reinterpret_cast<int4*>(s_next + b) = make_int4(first, first + v.x, first + v.x + v.y, first + v.x + v.y + v.z);
    at += __builtin_amdgcn_readlane(incl, 63);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int b = w0 + k * 64 + lane;
    if (b < B) s_next[b] += earlier[k];
  }
  __syncthreads();
  // exclusive prefix of the counters over the waves; at most 2048 per half word, no carry between the two
  for (int i = tid; i < words; i += kScatterThreads) {
    unsigned run = 0u;
#pragma unroll
    for (int w = 0; w < kScatterWaves; ++w) {
      const unsigned c = s_cnt[w * words + i];
      s_cnt[w * words + i] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRounds; ++k) place_round(mine[k], n0 + k * 64 + lane, id_bits, s_next, s_cnt + wave * words, ix);
  // free slots: those of the wave's runs slice, slice + n_slices, ...; a run ends where the next starts
  const int first_marked = w0 + (slice + n_slices - w0 % n_slices) % n_slices;
  for (int m0 = first_marked; slack > 0 && m0 < w1; m0 += 64 * n_slices) {
    const int next = m0 + lane * n_slices + 1;
    const int ends = next < w1 ? s_next[next] - base[next] : at;
    const int n_marked = min(64, (w1 - m0 + n_slices - 1) / n_slices);
    for (int i = 0; i < n_marked; ++i) {
      const int end = __builtin_amdgcn_readlane(ends, i);
      for (int j = lane; j < slack; j += 64) ix[end - slack + j] = -1;
    }
  }
  // the unit's off (no slice is earlier than the first); with a resident block (W >= 0) one more run of W slots closes it, n_res
  // of them in use
  if (slice == 0) {
    for (int b = tid; b < B; b += kScatterThreads) o[b] = s_next[b];
    if (tid == 0) {
      o[B] = all;
      if (W >= 0) {
        o[B + 1] = all + W;
        l[B] = n_res;
      }
    }
  }
  // keys with ids outside [0,B) are dropped: as many slots stay empty behind the last run
  for (int j = all + max(W, 0) + slice * kScatterThreads + tid; j < Ncap; j += n_slices * kScatterThreads) ix[j] = -1;
}

// Steps 1 to 3 in one launch for contexts of up to kDirectKeys positions and kDirectBuckets buckets: workgroups of 16 waves take 1024
// ROUNDS positions each, hold their ids, and where a unit has several workgroups each counts the others' ids for itself (the L2
// serves them; a position takes an LDS addition).  A whole build, 8 heads: 16000 keys 35 us with one workgroup for 16384 positions,
// 30 now; with three launches 20000 keys 40, 37.5 now, 30000 49.5, 47.5, and 49000 69 either way; where half of the ids are the same 43 and
// 44.5 at 24000, and if all are 44 and 45.5 (57 with an addition for each).
constexpr int kDirectKeys = 32768, kDirectBuckets = 2048, kDirectThreads = 1024, kDirectWaves = kDirectThreads / 64;
template <int ROUNDS>
__global__ void __launch_bounds__(kDirectThreads, 8)      // two workgroups to a compute unit
order_direct_kernel(const int32_t* __restrict__ ids, int32_t* __restrict__ len, int32_t* __restrict__ off, int32_t* __restrict__ idx,
                    int32_t* __restrict__ res_ids, int N, int Ncap, int B, int id_bits, int lo, int hi, int slack, int W, int n_sink,
                    int n_recent, int n_res) {
  // first slots of this part [B] | counters [waves][words] | with several parts: ids before this part [B], after it [B]
  extern __shared__ int s_next[];
  __shared__ int s_wsum[kDirectWaves], s_end;
  const int unit = blockIdx.x, part = blockIdx.y, n_parts = gridDim.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int words = (B + 1) / 2;
  unsigned* s_cnt = reinterpret_cast<unsigned*>(s_next + B);
  unsigned* cnt = s_cnt + wave * words;
  int* s_before = reinterpret_cast<int*>(s_cnt + kDirectWaves * words);
  int* s_after = s_before + B;
  const int32_t* idu = ids + (size_t)unit * N;
  int32_t* ix = idx + (size_t)unit * Ncap;
  const int lstride = W >= 0 ? B + 1 : B;
  int32_t* l = len + (size_t)unit * lstride;
  int32_t* o = off + (size_t)unit * (lstride + 1);
  constexpr int kPart = kDirectThreads * ROUNDS;
  const int p0 = lo + part * kPart, p1 = min(p0 + kPart, hi);
  const int per = ((p1 - p0 + kDirectWaves - 1) / kDirectWaves + 63) & ~63;      // positions per wave, at most 64 ROUNDS
  const int n0 = p0 + wave * per, n1 = min(n0 + per, p1);
  int v[ROUNDS];
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k) v[k] = idu[min(n0 + k * 64 + lane, N - 1)];
  for (int i = tid; i < kDirectWaves * words + (n_parts > 1 ? 2 * B : 0); i += kDirectThreads) s_cnt[i] = 0u;
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k)
    if (n0 + k * 64 + lane >= n1 || v[k] < 0 || v[k] >= B) v[k] = -1;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k)
    if (v[k] >= 0) wave_count_add(cnt, v[k], 1u);
  if (n_parts > 1) {
    constexpr int kDeep = 8;                             // loads of a thread in flight
    // The additions of a wave to one address wait for each other: an id that the wave meets often, in the first 64 of 512, is counted
    // apart.
    constexpr int kNone = -2, kOften = 8;
    auto count_others = [&](int from, int to, int* s) {
      int hot = kNone, n_hot = 0;
      auto leave_hot = [&] {
        if (n_hot > 0 && lane == 0) atomicAdd(&s[hot], n_hot);
        n_hot = 0;
      };
      for (int n = from + wave * 64; n < to; n += kDeep * kDirectThreads) {
        int u[kDeep];
#pragma unroll
        for (int k = 0; k < kDeep; ++k) u[k] = idu[min(n + lane + k * kDirectThreads, N - 1)];
#pragma unroll
        for (int k = 0; k < kDeep; ++k)
          if (n + lane + k * kDirectThreads >= to || u[k] >= B) u[k] = -1;
        // (the most frequent of the one so far and those of two lanes)
        int most = max(hot == kNone ? 0 : (int)__popcll(__ballot(u[0] == hot)), kOften - 1), next = kNone;
        if (hot != kNone && most >= kOften) next = hot;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int f = __builtin_amdgcn_readlane(u[0], 32 * i), c = (int)__popcll(__ballot(u[0] == f));
          if (f >= 0 && c > most) {
            most = c;
            next = f;
          }
        }
        if (next != hot) {
          leave_hot();
          hot = next;
        }
        if (hot == kNone) {                              // as a rule: nothing more than the additions
#pragma unroll
          for (int k = 0; k < kDeep; ++k)
            if (u[k] >= 0) atomicAdd(&s[u[k]], 1);
          continue;
        }
#pragma unroll
        for (int k = 0; k < kDeep; ++k) {
          n_hot += (int)__popcll(__ballot(u[k] == hot));
          if (u[k] >= 0 && u[k] != hot) atomicAdd(&s[u[k]], 1);
        }
      }
      leave_hot();
    };
    count_others(lo, p0, s_before);
    count_others(p1, hi, s_after);
  }
  __syncthreads();
  // exclusive prefix over the waves (at most 16384 per half word), totals, and the buckets' offsets
  static_assert(kDirectBuckets / 2 == kDirectThreads, "one pair of buckets per thread");
  unsigned tot = 0u;
  if (tid < words) {
    unsigned c[kDirectWaves];                            // read before the first is written: one LDS latency
#pragma unroll
    for (int w = 0; w < kDirectWaves; ++w) c[w] = s_cnt[w * words + tid];
#pragma unroll
    for (int w = 0; w < kDirectWaves; ++w) {
      s_cnt[w * words + tid] = tot;
      tot += c[w];
    }
  }
  const int b0 = 2 * tid;
  int lens[2] = {(int)(tot & 0xffffu), (int)(tot >> 16)}, before[2] = {0, 0};
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (n_parts > 1 && b0 + i < B) {
      before[i] = s_before[b0 + i];
      lens[i] += before[i] + s_after[b0 + i];
    }
  const int mine = (b0 < B ? lens[0] + slack : 0) + (b0 + 1 < B ? lens[1] + slack : 0);
  const int incl = (int)wave_prefix_sum((unsigned)mine);
  if (lane == 63) s_wsum[wave] = incl;
  __syncthreads();
  int run = incl - mine;
  for (int w = 0; w < wave; ++w) run += s_wsum[w];
  if (tid == 0 && part == 0) o[0] = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int b = b0 + i;
    if (b < B) {
      s_next[b] = run + before[i];
      run += lens[i] + slack;
      if (part == 0) {
        l[b] = lens[i];
        o[b + 1] = run;
      }
      if (b == B - 1) {
        s_end = run;
        if (W >= 0 && part == 0) {
          o[B + 1] = run + W;
          l[B] = n_res;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k)
    if (n0 + k * 64 < n1) place_round(v[k], n0 + k * 64 + lane, id_bits, s_next, cnt, ix);
  // free slots: the end of a bucket is the start of the next
  const int all = s_end, step = n_parts * kDirectThreads, first = part * kDirectThreads + tid;
  for (int i = first; i < B * slack; i += step) {
    const int b = i / slack;
    const int end = b + 1 < B ? s_next[b + 1] - (n_parts > 1 ? s_before[b + 1] : 0) : all;
    ix[end - slack + (i - b * slack)] = -1;
  }
  for (int j = all + max(W, 0) + first; j < Ncap; j += step) ix[j] = -1;       // behind the last run: dropped keys
  if (W > 0)
    for (int j = first; j < W; j += step) place_resident(j, idu, ix, res_ids + (size_t)unit * W, all, N, n_sink, n_recent, n_res);
}

// Copy rows into their slots: out[slot] = in[idx[slot]] for member slots (0 <= idx[slot] < N).  ZERO: free slots are set
// to zero (here they cost their own bytes once; a fill of the whole cache ahead of the copy writes every member slot twice).
template <int CHUNKS /* 16-byte pieces per row */, bool ZERO>
__global__ void __launch_bounds__(256)
permute_kernel(const uint4* __restrict__ K, const uint4* __restrict__ V, const int32_t* __restrict__ idx,
               uint4* __restrict__ Ks, uint4* __restrict__ Vs, int N, int Ncap) {
  constexpr int kRowsPerThread = 4;
  const int unit = blockIdx.y, piece = threadIdx.x % CHUNKS;
  const int first = (int)((blockIdx.x * 256u + threadIdx.x) / CHUNKS) * kRowsPerThread;
  const int32_t* ix = idx + (size_t)unit * Ncap;
  const uint4* Ku = K + (size_t)unit * N * CHUNKS + piece;
  const uint4* Vu = V + (size_t)unit * N * CHUNKS + piece;
  uint4* Ko = Ks + (size_t)unit * Ncap * CHUNKS + piece;
  uint4* Vo = Vs + (size_t)unit * Ncap * CHUNKS + piece;
  int src[kRowsPerThread];
#pragma unroll
  for (int r = 0; r < kRowsPerThread; ++r) src[r] = first + r < Ncap ? ix[first + r] : -1;
  uint4 kv[kRowsPerThread], vv[kRowsPerThread];
#pragma unroll
  for (int r = 0; r < kRowsPerThread; ++r) {
    kv[r] = vv[r] = make_uint4(0u, 0u, 0u, 0u);
    if ((unsigned)src[r] < (unsigned)N) {
      kv[r] = stream_load16(Ku + (size_t)src[r] * CHUNKS);
      vv[r] = stream_load16(Vu + (size_t)src[r] * CHUNKS);
    }
  }
#pragma unroll
  for (int r = 0; r < kRowsPerThread; ++r) {
    if ((unsigned)src[r] < (unsigned)N || (ZERO && first + r < Ncap)) {
      stream_store16(Ko + (size_t)(first + r) * CHUNKS, kv[r]);
      stream_store16(Vo + (size_t)(first + r) * CHUNKS, vv[r]);
    }
  }
}

// ---- append ------------------------------------------------------------------------------

template <typename T> __device__ __forceinline__ double to_f64(T v);
template <> __device__ __forceinline__ double to_f64<float>(float v) { return (double)v; }
template <> __device__ __forceinline__ double to_f64<bf16_t>(bf16_t v) {
  return (double)__uint_as_float((uint32_t)v << 16);
}


// Eight bf16 elements (one 16-byte piece of a row) -> double.
__device__ __forceinline__ void widen8(const uint4& u, double* o) {
  o[0] = (double)bf16_lo(u.x); o[1] = (double)bf16_hi(u.x); o[2] = (double)bf16_lo(u.y); o[3] = (double)bf16_hi(u.y);
  o[4] = (double)bf16_lo(u.z); o[5] = (double)bf16_hi(u.z); o[6] = (double)bf16_lo(u.w); o[7] = (double)bf16_hi(u.w);
}

// Score of one centroid row against the key in s_x: the in-order double-precision sum of the
// exact products.  All 16-byte loads of the row (of half a row for fp32) are issued before the
// dependent chain of 128 fused multiply-adds starts.
// Eight features of the key are read from LDS while the eight before them are multiplied (left alone the compiler reads two at a time and
// waits for each: 100 sequences of 8 heads, 303 buckets, some keys with two candidates 12.5 us, 11.1).
template <typename T>
__device__ __forceinline__ double score_row(const T* __restrict__ c, const double* __restrict__ s_x);
__device__ __forceinline__ double add_products(double t, const double (&w)[8], double (&x)[8], const double* __restrict__ next) {
  double ahead[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) ahead[e] = next[e];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < 8; ++e) t = fma(x[e], w[e], t);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = ahead[e];
  return t;
}
template <>
__device__ __forceinline__ double score_row<bf16_t>(const bf16_t* __restrict__ c, const double* __restrict__ s_x) {
  uint4 u[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) u[i] = reinterpret_cast<const uint4*>(c)[i];
  double t = 0.0, x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = s_x[e];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    double w[8];
    widen8(u[i], w);
    t = add_products(t, w, x, s_x + 8 * min(i + 1, 15));
  }
  return t;
}
template <>
__device__ __forceinline__ double score_row<float>(const float* __restrict__ c, const double* __restrict__ s_x) {
  double t = 0.0, x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = s_x[e];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {   // half a row (sixteen pieces) at a time
    float4 u[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) u[i] = reinterpret_cast<const float4*>(c)[hh * 16 + i];
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      const double w[8] = {(double)u[i].x, (double)u[i].y, (double)u[i].z, (double)u[i].w,
                           (double)u[i + 1].x, (double)u[i + 1].y, (double)u[i + 1].z, (double)u[i + 1].w};
      t = add_products(t, w, x, s_x + 8 * min(hh * 8 + i / 2 + 1, 15));
    }
  }
  return t;
}

// (score, id) candidates: o beats m if it exists and is larger, or equal with the lower id.
__device__ __forceinline__ void take_better(double& best, int& best_id, double ob, int oid) {
  if (oid >= 0 && (best_id < 0 || ob > best || (ob == best && oid < best_id))) {
    best = ob;
    best_id = oid;
  }
}
// Best candidate of the wave, in every lane.  Inside the rows of 16 lanes the partners' candidates come over the
// data-parallel primitives (three register moves per step), between the rows over the row-swap instructions: no
// step goes through the LDS crossbar.  All 64 lanes must be active.
template <int CTRL>
__device__ __forceinline__ void take_better_dpp(double& best, int& best_id) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(best);
  const unsigned long long lo = dpp_u32<CTRL>((unsigned)u), hi = dpp_u32<CTRL>((unsigned)(u >> 32));
  const int oid = (int)dpp_u32<CTRL>((unsigned)best_id);
  take_better(best, best_id, __longlong_as_double((long long)((hi << 32) | lo)), oid);
}
__device__ __forceinline__ void wave_best(double& best, int& best_id) {
  take_better_dpp<kDppXor1>(best, best_id);
  take_better_dpp<kDppXor2>(best, best_id);
  take_better_dpp<kDppHalfMirror>(best, best_id);
  take_better_dpp<kDppMirror>(best, best_id);
  // between the rows: the row-swap instructions hand every lane its own candidate and that of the same lane one
  // row (then two rows) away, in an order that is the same for the three words
  {
    const unsigned long long u = (unsigned long long)__double_as_longlong(best);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    const auto id = __builtin_amdgcn_permlane16_swap((unsigned)best_id, (unsigned)best_id, false, false);
    best = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    best_id = (int)id[0];
    take_better(best, best_id, __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1])), (int)id[1]);
  }
  {
    const unsigned long long u = (unsigned long long)__double_as_longlong(best);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    const auto id = __builtin_amdgcn_permlane32_swap((unsigned)best_id, (unsigned)best_id, false, false);
    best = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    best_id = (int)id[0];
    take_better(best, best_id, __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1])), (int)id[1]);
  }
}

// A slab's centroids that may be the key's, as exchanged between the workgroups of a unit: the largest lower bound of an exact
// score, the n centroids whose upper bound reaches it, lower id first.  n = 3: the best of the slab by exact scores.
struct PushPartial {
  float lo, hi0;
  union {
    struct { float hi1; int id0; } bounds;
    double exact;
  };
  int id, n;                                     // id of the second, or of the exact best
};

// window_push: P workgroups per (sequence, KV head), each with a slab of the centroids; the last to arrive picks the bucket and does
// the bookkeeping.  Scores are fp32 first, whole rows of 16 lanes each, with bounds on how far the exact one can be: as a rule
// one centroid's upper bound reaches the largest lower bound of all, and that is the bucket, as double-precision scores define
// it.  Otherwise those that do are scored exactly; where more than two of a slab do, the slab's workgroup scores all of its
// centroids before it reports (equal rows, a key of zeros: 12 us a call; left to the last workgroup they took 34 us at 64 units of 1024
// centroids, 117 at 8 of 4096).
// Which key is displaced and where it goes does not depend on the new key's bucket: every
// workgroup reads that state up front (the loads overlap the scoring), slab 0 copies the displaced
// row to its bucket, and the last workgroup, which runs after all of these reads, writes the new
// row and the updated counts.
// C: element type of the cache.  C = T stores the new rows as they are; C = fp8_t (an 8-bit cache,
// T = bf16) stores x / scale of the (sequence, head) rounded to E4M3, saturated at +-448.
template <typename C, typename T>
__device__ __forceinline__ C to_cache(T v, float inv_scale) {
  if constexpr (sizeof(C) == sizeof(T)) {
    return v;
  } else {
    const float f = fminf(fmaxf(Vec8<T>::widen(v) * inv_scale, -448.f), 448.f);
    return (C)(__builtin_amdgcn_cvt_pk_fp8_f32(f, f, 0, false) & 0xff);
  }
}

constexpr int kPushThreads = 256, kPushRows = 8 /* of a 16-lane group in flight */, kPushSlab = kPushRows * kPushThreads / 16;

template <typename T, typename C = T>
__global__ void __launch_bounds__(kPushThreads)
window_push_kernel(const T* __restrict__ x_new, const T* __restrict__ k_new, const T* __restrict__ v_new,
                   const int32_t* __restrict__ pos_new, const T* __restrict__ cent, const float* __restrict__ bias,
                   const int32_t* __restrict__ off, int32_t* __restrict__ len, int32_t* __restrict__ idx,
                   C* __restrict__ Ks, C* __restrict__ Vs, const float* __restrict__ kscale,
                   const float* __restrict__ vscale, int32_t* __restrict__ res_ids,
                   int32_t* __restrict__ new_ids, int32_t* __restrict__ overflow, PushPartial* __restrict__ part,
                   unsigned* __restrict__ counters, int Hkv, int Ncap, int B, int runs, int n_sink, int n_recent,
                   int P, int cpl /* kPushSlab * cpl centroids to a workgroup */) {
  // runs = B + 1: index with a resident run.  runs = B: plain index (append_keys): W = 0, every key
  // goes straight into its bucket, res_ids is not touched and pos_new may be null (idx gets -2).
  __shared__ double s_x[kD];
  __shared__ __align__(16) T s_xt[kD];
  __shared__ float s_lo[kPushThreads / 64], s_hi[2];
  __shared__ double s_best[kPushThreads / 64];
  __shared__ int s_n, s_id[2], s_state[6], s_list[2 * 64], s_best_id[kPushThreads / 64];
  const int slab = blockIdx.x, unit = blockIdx.y, h = unit % Hkv, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = tid & 15, grp = tid >> 4;
  SAAP_TRACE(0);
  const int W = n_sink + n_recent;
  const int32_t* o = off + (size_t)unit * (runs + 1);
  int32_t* l = len + (size_t)unit * runs;
  int32_t* ix = idx + (size_t)unit * Ncap;
  int32_t* rid = res_ids + (size_t)unit * W;
  C* Ku = Ks + (size_t)unit * Ncap * kD;
  C* Vu = Vs + (size_t)unit * Ncap * kD;
  const T* cu = cent + (size_t)h * B * kD;
  const float* bu = bias ? bias + (size_t)h * B : nullptr;

  // ---- the loads that wait for nothing: the new key, its position, the first centroids ----
  const T xe = x_new[(size_t)unit * kD + (tid & (kD - 1))];
  const int pos = pos_new ? pos_new[unit / Hkv] : 0x7fffffff;
  const int res_base = o[B];
  const int row0 = slab * kPushSlab * cpl;
  Vec8<T> c[kPushRows];
  auto load_rows = [&](int it) {
#pragma unroll
    for (int i = 0; i < kPushRows; ++i) c[i].load(cu + (size_t)min(row0 + it * kPushSlab + grp + 16 * i, B - 1) * kD + sub * 8);
  };
  load_rows(0);
  T k0 = T(0), k1 = T(0), v0 = T(0), v1 = T(0);
  float k_inv = 1.f, v_inv = 1.f;                // powers of two
  if (wave == 0) {
    k0 = k_new[(size_t)unit * kD + lane], k1 = k_new[(size_t)unit * kD + 64 + lane];
    v0 = v_new[(size_t)unit * kD + lane], v1 = v_new[(size_t)unit * kD + 64 + lane];
    if (kscale) k_inv = 1.0f / kscale[unit];
    if (vscale) v_inv = 1.0f / vscale[unit];
  }
  // ---- what can be decided without the bucket, by the last wave (same values in every lane) ----
  // -1: refused   0: slot of a run that is still filling   1: ring slot, a key is displaced   2: no ring
  const int kind = pos < 0 ? -1 : pos < W ? 0 : n_recent > 0 ? 1 : 2;
  if (wave == kPushThreads / 64 - 1) {
    int slot = -1, dst = -1, e = -1, cur = 0, moved_pos = -1;
    bool refused = kind < 0;
    if (kind == 0) {
      slot = res_base + pos;                     // r(pos) = pos while the run is not full
    } else if (kind == 1) {
      const int r = n_sink + (pos - n_sink) % n_recent;
      const int from = res_base + r;
      e = rid[r];
      moved_pos = ix[from];
      const C a0 = Ku[(size_t)from * kD + lane], a1 = Ku[(size_t)from * kD + 64 + lane];
      const C b0 = Vu[(size_t)from * kD + lane], b1 = Vu[(size_t)from * kD + 64 + lane];
      // e outside [0,B) means the caller broke the protocol (pushes out of order, foreign state):
      // refuse like a full bucket instead of indexing with it
      const bool ok = e >= 0 && e < B;
      cur = ok ? l[e] : 0;
      if (ok && o[e] + cur < o[e + 1]) {
        slot = from;
        dst = o[e] + cur;
        if (slab == 0) {                         // the displaced row: ring slot -> its bucket
          Ku[(size_t)dst * kD + lane] = a0;
          Ku[(size_t)dst * kD + 64 + lane] = a1;
          Vu[(size_t)dst * kD + lane] = b0;
          Vu[(size_t)dst * kD + 64 + lane] = b1;
        }
      } else {
        refused = true;
      }
    }
    if (lane == 0) {
      s_state[0] = slot; s_state[1] = dst; s_state[2] = e; s_state[3] = cur; s_state[4] = moved_pos; s_state[5] = refused;
    }
  }
  if (tid < kD) {
    s_x[tid] = to_f64<T>(xe);
    s_xt[tid] = xe;
  }
  if (tid == 0) s_n = 0;
  __syncthreads();
  SAAP_TRACE(1);

  // ---- this slab's centroids: lane `sub` < 8 of a group keeps row grp + 16 sub of every round ----
  Vec8<T> xv;
  xv.load(s_xt + sub * 8);
  const float xn2 = sum16(xv.dot(xv));
  // |fp32 score - exact score| <= 128 2^-24 |x| |c|, with head-room of four for the order of the sum, and the addition of the bias.
  // Products and sums below the smallest normal fp32 number (1.2e-38, 128 of each) may be lost, from scores and from the squares of
  // norms.
  constexpr float kTol = 4.0f * 128.0f * 5.9604645e-8f, kLost = 4e-36f;
  const float x_bound = kTol * __builtin_amdgcn_sqrtf(xn2 + kLost);      // (one unit in the last place off is within the head-room)
  float lo = -INFINITY, top[3] = {-INFINITY, -INFINITY, -INFINITY};
  int top_id[2] = {-1, -1};
  for (int it = 0; it < cpl; ++it) {
    float score = 0.f, n2 = 0.f;
#pragma unroll
    for (int i = 0; i < kPushRows; ++i) {
      const float d = sum16(c[i].dot(xv)), q = sum16(c[i].dot(c[i]));
      score = sub == i ? d : score;
      n2 = sub == i ? q : n2;
    }
    if (it + 1 < cpl) load_rows(it + 1);
    const int b = row0 + it * kPushSlab + grp + 16 * sub;
    if (sub < kPushRows && b < B) {
      const float add = bu ? bu[b] : 0.f;
      const bool never = add == -INFINITY && fabsf(score) < INFINITY;      // whatever the product is exactly
      score += add;
      const float err = x_bound * __builtin_amdgcn_sqrtf(n2 + kLost) + 2.5e-7f * fabsf(score) + kLost;
      const bool known = fabsf(score) < INFINITY && err < INFINITY;        // infinities and NaN: nothing is known
      const float up = known ? score + err : never ? -INFINITY : INFINITY, down = known ? score - err : -INFINITY;
      lo = fmaxf(lo, down);
      if (up > top[0]) {
        top[2] = top[1];
        top[1] = top[0];
        top_id[1] = top_id[0];
        top[0] = up;
        top_id[0] = b;
      } else if (up > top[1]) {
        top[2] = top[1];
        top[1] = up;
        top_id[1] = b;
      } else {
        top[2] = fmaxf(top[2], up);
      }
    }
  }
  SAAP_TRACE(2);
  {
    const float wave_lo = wave_max(lo);
    if (lane == 0) s_lo[wave] = wave_lo;
  }
  __syncthreads();
  lo = fmaxf(fmaxf(s_lo[0], s_lo[1]), fmaxf(s_lo[2], s_lo[3]));
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (top_id[i] >= 0 && top[i] >= lo) {
      const int at = atomicAdd(&s_n, 1);
      if (at < 2) {
        s_id[at] = top_id[i];
        s_hi[at] = top[i];
      }
    }
  if (top_id[1] >= 0 && top[2] >= lo && top[2] > -INFINITY) atomicAdd(&s_n, 1);
  __syncthreads();
  const int n_slab = min(s_n, 3);
  double best = 0.0;                             // of the exact scores
  int best_id = -1;
  if (n_slab > 2) {
    for (int i = tid; i < kPushSlab * cpl && row0 + i < B; i += kPushThreads) {
      asm volatile("" ::: "memory");             // hoisted out of the loop, the key's doubles would hold 256 registers
      double t = score_row<T>(cu + (size_t)(row0 + i) * kD, s_x);
      if (bu) t += (double)bu[row0 + i];
      take_better(best, best_id, t, row0 + i);
    }
    wave_best(best, best_id);
    if (lane == 0) {
      s_best[wave] = best;
      s_best_id[wave] = best_id;
    }
    __syncthreads();
  }
  if (wave != 0) return;
  SAAP_TRACE(3);
  int n_cand = n_slab;                           // listed, not scored yet
  unsigned long long scored = 0;                 // slabs (lanes) with an exact best
  if (n_slab > 2) {
    n_cand = 0;
    scored = 1ull;
#pragma unroll
    for (int w = 1; w < kPushThreads / 64; ++w) take_better(best, best_id, s_best[w], s_best_id[w]);
  }
  // two candidates in the order of their ids, whichever came first: a score that is no number has the same outcome every time
  const int at0 = n_cand == 2 && s_id[1] < s_id[0] ? 1 : 0;
  int id0 = n_cand > 0 ? s_id[at0] : -1;
  const int id1 = n_cand > 1 ? s_id[at0 ^ 1] : -1;
  if (P > 1) {
    if (lane == 0) {
      const float hi0 = n_cand > 0 ? s_hi[at0] : -INFINITY, hi1 = n_cand > 1 ? s_hi[at0 ^ 1] : -INFINITY;
      auto pair = [](unsigned a, unsigned b) { return (unsigned long long)b << 32 | a; };
      unsigned long long* mine = reinterpret_cast<unsigned long long*>(part + (size_t)unit * P + slab);
      const unsigned long long middle = n_slab > 2 ? (unsigned long long)__double_as_longlong(best) : pair(__float_as_uint(hi1), (unsigned)id0);
      __hip_atomic_store(mine, pair(__float_as_uint(lo), __float_as_uint(hi0)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(mine + 1, middle, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(mine + 2, pair((unsigned)(n_slab > 2 ? best_id : id1), (unsigned)n_slab), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // every load above has returned and every store has been acknowledged before the arrival counts
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    unsigned old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(&counters[unit], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = (unsigned)__builtin_amdgcn_readfirstlane((int)old);
    SAAP_TRACE(4);
    if (old != (unsigned)(P - 1)) return;
    // every partial was stored through to the device's coherent level and acknowledged before its arrival was
    // counted: loads of the same scope see it, and no cache has to be invalidated for them
    unsigned long long* q = reinterpret_cast<unsigned long long*>(part + (size_t)unit * P + min(lane, P - 1));      // P <= 64
    const unsigned long long q0 = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long q1 = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long q2 = __hip_atomic_load(q + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool mine = lane < P;
    const float hi0 = __uint_as_float((unsigned)(q0 >> 32)), hi1 = __uint_as_float((unsigned)q1);
    const int n = mine ? (int)(q2 >> 32) : 0;
    lo = wave_max(mine ? __uint_as_float((unsigned)q0) : -INFINITY);
    scored = __ballot(n > 2);
    best = __longlong_as_double((long long)q1);
    best_id = n > 2 ? (int)(unsigned)q2 : -1;
    const bool one = (n == 1 || n == 2) && hi0 >= lo, two = n == 2 && hi1 >= lo;
    const unsigned long long first = __ballot(one), second = __ballot(two), below = (1ull << lane) - 1ull;
    n_cand = __popcll(first) + __popcll(second);
    if (one) s_list[__popcll(first & below)] = (int)(q1 >> 32);
    if (two) s_list[__popcll(first) + __popcll(second & below)] = (int)(unsigned)q2;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    id0 = s_list[0];
    SAAP_TRACE(5);
    if (lane == 0) __hip_atomic_store(&counters[unit], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (lane == 0) {
    s_list[0] = id0;
    s_list[1] = id1;
  }
  if (scored == 0 && n_cand < 2) {
    best_id = n_cand ? id0 : 0;                  // none: every score is -infinity, the lowest id of equal ones
  } else {                                       // more than one may be the largest
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    for (int i = lane; i < n_cand; i += 64) {
      asm volatile("" ::: "memory");
      const int bc = s_list[i];
      double t = score_row<T>(cu + (size_t)bc * kD, s_x);
      if (bu) t += (double)bu[bc];
      take_better(best, best_id, t, bc);
    }
    wave_best(best, best_id);
  }
  best_id = __builtin_amdgcn_readfirstlane(best_id);
  int slot = s_state[0];
  const int dst = s_state[1], e = s_state[2], moved_pos = s_state[4];
  int cur = s_state[3];
  bool refused = s_state[5] != 0;

  // ---- bookkeeping, by the one workgroup that knows the bucket ----
  const int b = best_id;
  if (kind == 2) {                             // no ring: the new key goes straight into its bucket
    const int c2 = l[b];
    if (o[b] + c2 < o[b + 1]) slot = o[b] + c2; else refused = true;
    cur = c2;
  }
  if (lane == 0) {
    new_ids[unit] = b;
    if (refused) {
      *overflow = 1;
    } else {
      if (kind == 0) {
        l[B] += 1;
        rid[pos] = b;
      } else if (kind == 1) {
        l[e] = cur + 1;
        ix[dst] = moved_pos;
        rid[slot - res_base] = b;
      } else {
        l[b] = cur + 1;
      }
      ix[slot] = pos_new ? pos : -2;
    }
  }
  if (!refused) {
    Ku[(size_t)slot * kD + lane] = to_cache<C, T>(k0, k_inv);
    Ku[(size_t)slot * kD + 64 + lane] = to_cache<C, T>(k1, k_inv);
    Vu[(size_t)slot * kD + lane] = to_cache<C, T>(v0, v_inv);
    Vu[(size_t)slot * kD + 64 + lane] = to_cache<C, T>(v1, v_inv);
  }
  SAAP_TRACE(6);
}

// ---- recompact: fresh slack behind every bucket without assigning the keys again ---------------
// One workgroup per unit: new offsets from the current lengths.  `runs` = B, or B + 1 with a
// resident run, which keeps its fixed number of slots.
__global__ void __launch_bounds__(1024)
reoffset_kernel(const int32_t* __restrict__ len, const int32_t* __restrict__ off, int32_t* __restrict__ off_new,
                int runs, int B, int slack, int Ncap_new, int32_t* __restrict__ overflow) {
  __shared__ int s_wsum[16];
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (B + blockDim.x - 1) / blockDim.x;
  const int b0 = tid * per, b1 = min(b0 + per, B);
  const int32_t* l = len + (size_t)unit * runs;
  const int32_t* o = off + (size_t)unit * (runs + 1);
  int32_t* on = off_new + (size_t)unit * (runs + 1);
  int mine = 0;
  for (int b = b0; b < b1; ++b) mine += l[b] + slack;
  const int incl = (int)wave_prefix_sum((unsigned)mine);
  if (lane == 63) s_wsum[wave] = incl;
  __syncthreads();
  int run = incl - mine;
  for (int w = 0; w < wave; ++w) run += s_wsum[w];
  if (tid == 0) on[0] = 0;
  for (int b = b0; b < b1; ++b) {
    run += l[b] + slack;
    on[b + 1] = run;
    if (b == B - 1) {
      int end = run;
      if (runs > B) {
        end += o[B + 1] - o[B];
        on[B + 1] = end;
      }
      if (end > Ncap_new) *overflow = 1;
    }
  }
}

// One workgroup per (run, unit): the run's member slots move to their place in the new cache.
template <int CHUNKS /* 16-byte pieces per row */>
__global__ void __launch_bounds__(256)
recopy_kernel(const int32_t* __restrict__ off, const int32_t* __restrict__ len, const int32_t* __restrict__ off_new,
              const int32_t* __restrict__ idx, int32_t* __restrict__ idx_new, const uint4* __restrict__ Ks,
              const uint4* __restrict__ Vs, uint4* __restrict__ Kn, uint4* __restrict__ Vn, int runs, int Ncap,
              int Ncap_new, const int32_t* __restrict__ overflow) {
  if (*overflow) return;                       // the new cache is too small: nothing is moved
  const int b = blockIdx.x, unit = blockIdx.y, tid = threadIdx.x;
  const int first = off[(size_t)unit * (runs + 1) + b], dst = off_new[(size_t)unit * (runs + 1) + b];
  // a resident run is a ring: every slot up to its length moves, whatever position it holds
  const int n = len[(size_t)unit * runs + b];
  for (int r = tid; r < n; r += 256) idx_new[(size_t)unit * Ncap_new + dst + r] = idx[(size_t)unit * Ncap + first + r];
  constexpr int kRowsPerPass = 256 / CHUNKS;
  const int piece = tid % CHUNKS;
  for (int r = tid / CHUNKS; r < n; r += kRowsPerPass) {
    const size_t src = ((size_t)unit * Ncap + first + r) * CHUNKS + piece;
    const size_t out = ((size_t)unit * Ncap_new + dst + r) * CHUNKS + piece;
    stream_store16(Kn + out, stream_load16(Ks + src));
    stream_store16(Vn + out, stream_load16(Vs + src));
  }
}

}  // namespace

size_t push_workspace_bytes(long long units, int B) {
  static_assert(SAAP_MAX_BUCKETS <= 64 * kPushSlab, "a lane per workgroup of a unit");
  // 24 bytes for every 128 centroids, of units with more than one workgroup, are never more than this
  static_assert(sizeof(PushPartial) == 24 && kPushSlab == 128, "as stated");
  return (size_t)SAAP_WS_HEADER_BYTES + (size_t)units * ((B + 63) / 64) * 16;
}

// Rounds of the scoring workgroups: one when few units leave the device empty, more
// when there are enough units to fill it anyway (about two workgroups per compute unit in all).
static int push_rounds(long long units, int B) {
  const long long slabs = (B + kPushSlab - 1) / kPushSlab;
  long long want = 2LL * device_cus() / units;                // workgroups per unit
  if (want < 1) want = 1;
  long long cpl = (slabs + want - 1) / want;
  if (cpl < 1) cpl = 1;
  if (cpl > 8) cpl = 8;
  return (int)cpl;
}

size_t build_workspace_bytes(long long units, int N, int B) {
  const long long n_slices = (N + kSlice - 1) / kSlice;
  return (size_t)SAAP_WS_HEADER_BYTES + (size_t)units * n_slices * B * sizeof(int32_t);
}

}  // namespace saap

using namespace saap;

// off, len and idx of the index (steps 1 to 3).  W < 0: plain index (B runs); otherwise the index with a resident run of
// W slots behind the B buckets and its ids in res_ids.  slice_hist: scratch of units * slices * B counters.
void saap::order_keys(const int32_t* bucket_ids, int32_t* off, int32_t* len, int32_t* idx, int32_t* res_ids, int32_t* slice_hist,
                      long long units, int N, int Ncap, int B, int slack, int W, int n_sink, int n_recent, hipStream_t hs) {
  const bool windowed = W >= 0;
  const int n_res = windowed ? (N < W ? N : W) : 0;
  int id_bits = 1;
  while ((1 << id_bits) < B) ++id_bits;
  // positions [lo, hi) go into the buckets
  const int lo = windowed ? (N <= W ? 0 : n_sink) : 0;
  const int hi = windowed ? (N <= W ? 0 : N - n_recent) : N;
  const size_t next_bytes = (size_t)B * sizeof(int), wave_bytes = (size_t)(B + 1) / 2 * sizeof(unsigned);
  // One launch where it has room for a workgroup per compute unit at most, or two where each holds as much as it can.
  if (N <= kDirectKeys && B <= kDirectBuckets) {
    auto direct = [&](auto rounds, int most) {
      constexpr int R = decltype(rounds)::value;
      const long long parts = std::max(1, (hi - lo + kDirectThreads * R - 1) / (kDirectThreads * R));
      const size_t lds = next_bytes + kDirectWaves * wave_bytes + (parts > 1 ? 2 * next_bytes : 0);
      if ((parts > 1 && units * parts > most) || !allow_lds<order_direct_kernel<R>>(lds)) return false;
      hipLaunchKernelGGL(order_direct_kernel<R>, dim3((unsigned)units, (unsigned)parts), dim3(kDirectThreads), lds, hs, bucket_ids, len, off,
                         idx, res_ids, N, Ncap, B, id_bits, lo, hi, slack, W, n_sink, n_recent, n_res);
      return true;
    };
    const int cus = device_cus();
    if (hi - lo <= kDirectThreads * 4 && direct(std::integral_constant<int, 4>{}, cus)) return;
    if (direct(std::integral_constant<int, 8>{}, cus) || direct(std::integral_constant<int, 16>{}, 2 * cus)) return;
  }
  const int n_slices = (N + kSlice - 1) / kSlice, lstride = windowed ? B + 1 : B;
  hipLaunchKernelGGL(hist_kernel, dim3(n_slices, (unsigned)units), dim3(256), next_bytes, hs, bucket_ids, slice_hist, N, B, n_slices,
                     lo, hi);
  hipLaunchKernelGGL(colscan_kernel, dim3((B + 255) / 256, (unsigned)units), dim3(256), 0, hs, slice_hist, len, B, n_slices, lstride);
  const size_t lds = (size_t)((B + 3) & ~3) * sizeof(int) + kScatterWaves * wave_bytes;
  auto scatter = [&](auto runs) {
    constexpr int KW = decltype(runs)::value;
    (void)allow_lds<scatter_kernel<KW>>(lds);
    hipLaunchKernelGGL(scatter_kernel<KW>, dim3((unsigned)units, n_slices), dim3(kScatterThreads), lds, hs, bucket_ids, slice_hist, len,
                       off, idx, N, Ncap, B, n_slices, id_bits, lo, hi, slack, W, n_res);
  };
  static_assert(SAAP_MAX_BUCKETS <= 256 * 32, "runs of a scatter workgroup");
  if (B <= 1024) scatter(std::integral_constant<int, 4>{});
  else if (B <= 2048) scatter(std::integral_constant<int, 8>{});
  else if (B <= 4096) scatter(std::integral_constant<int, 16>{});
  else scatter(std::integral_constant<int, 32>{});
  if (W > 0)
    hipLaunchKernelGGL(resident_kernel, dim3((unsigned)((W + 255) / 256), (unsigned)units), dim3(256), 0, hs, bucket_ids, off, idx,
                       res_ids, N, Ncap, B, n_sink, n_recent, n_res);
}

template <int CHUNKS>
static void permute(const void* K, const void* V, const int32_t* idx, void* Ks, void* Vs, long long units, int N, int Ncap, bool zero,
                    hipStream_t hs) {
  const dim3 grid((unsigned)(((long long)(Ncap + 3) / 4 * CHUNKS + 255) / 256), (unsigned)units);
  const auto *k = static_cast<const uint4*>(K), *v = static_cast<const uint4*>(V);
  auto *ko = static_cast<uint4*>(Ks), *vo = static_cast<uint4*>(Vs);
  if (zero) hipLaunchKernelGGL((permute_kernel<CHUNKS, true>), grid, dim3(256), 0, hs, k, v, idx, ko, vo, N, Ncap);
  else hipLaunchKernelGGL((permute_kernel<CHUNKS, false>), grid, dim3(256), 0, hs, k, v, idx, ko, vo, N, Ncap);
}

// Shared body of the build calls.  res_ids == nullptr: plain index (B runs); otherwise the
// index with a resident run of W = n_sink + n_recent slots behind the B buckets.  zero: free slots are set to zero.
static int32_t build_index(const int32_t* bucket_ids, const void* K, const void* V, int32_t* off, int32_t* len,
                           int32_t* idx, void* Ksorted, void* Vsorted, int32_t* res_ids, int32_t S, int32_t Hkv,
                           int32_t N, int32_t Ncap, int32_t B, int32_t d, int32_t dtype, int32_t slack,
                           int32_t n_sink, int32_t n_recent, bool zero, void* ws, size_t ws_bytes, void* stream) {
  const bool windowed = res_ids != nullptr;
  if (!bucket_ids || !K || !V || !off || !len || !idx || !Ksorted || !Vsorted || !ws) return SAAP_INVALID_ARG;
  const void* ptrs[] = {bucket_ids, K, V, off, len, idx, Ksorted, Vsorted, ws, res_ids};
  for (const void* p : ptrs)
    if (!aligned16(p)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || N <= 0 || B <= 0 || slack < 0 || n_sink < 0 || n_recent < 0) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  const long long W = (long long)n_sink + n_recent;
  if (W > 0x3fffffff) return SAAP_INVALID_ARG;
  const long long n_res = windowed ? (N < W ? N : W) : 0;
  if ((long long)Ncap != (long long)N - n_res + (long long)B * slack + (windowed ? W : 0)) return SAAP_INVALID_ARG;
  if (d != kD || B > SAAP_MAX_BUCKETS) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535) return SAAP_UNSUPPORTED;
  if (ws_bytes < build_workspace_bytes(units, N, B)) return SAAP_WORKSPACE_TOO_SMALL;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  int32_t* slice_hist = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  order_keys(bucket_ids, off, len, idx, res_ids, slice_hist, units, N, Ncap, B, slack, windowed ? (int)W : -1, n_sink, n_recent, hs);
  if (dtype == SAAP_BF16) permute<16>(K, V, idx, Ksorted, Vsorted, units, N, Ncap, zero, hs);
  else permute<32>(K, V, idx, Ksorted, Vsorted, units, N, Ncap, zero, hs);
  return launch_status();
}

extern "C" int32_t saap_build_bucket_index(const int32_t* bucket_ids, const void* K, const void* V,
                                           int32_t* off, int32_t* len, int32_t* idx, void* Ksorted,
                                           void* Vsorted, int32_t S, int32_t Hkv, int32_t N, int32_t Ncap,
                                           int32_t B, int32_t d, int32_t dtype, int32_t slack, void* ws,
                                           size_t ws_bytes, void* stream) {
  const Call call(stream);
  return build_index(bucket_ids, K, V, off, len, idx, Ksorted, Vsorted, nullptr, S, Hkv, N, Ncap, B, d, dtype, slack,
                     0, 0, false, ws, ws_bytes, stream);
}

extern "C" int32_t saap_build_bucket_index_zeroed(const int32_t* bucket_ids, const void* K, const void* V,
                                                  int32_t* off, int32_t* len, int32_t* idx, void* Ksorted,
                                                  void* Vsorted, int32_t S, int32_t Hkv, int32_t N, int32_t Ncap,
                                                  int32_t B, int32_t d, int32_t dtype, int32_t slack, void* ws,
                                                  size_t ws_bytes, void* stream) {
  const Call call(stream);
  return build_index(bucket_ids, K, V, off, len, idx, Ksorted, Vsorted, nullptr, S, Hkv, N, Ncap, B, d, dtype, slack,
                     0, 0, true, ws, ws_bytes, stream);
}

extern "C" int32_t saap_build_windowed_index(const int32_t* bucket_ids, const void* K, const void* V,
                                             int32_t* off, int32_t* len, int32_t* idx, void* Ksorted,
                                             void* Vsorted, int32_t* resident_ids, int32_t S, int32_t Hkv,
                                             int32_t N, int32_t Ncap, int32_t B, int32_t d, int32_t dtype,
                                             int32_t slack, int32_t n_sink, int32_t n_recent, void* ws,
                                             size_t ws_bytes, void* stream) {
  const Call call(stream);
  if (!resident_ids) return SAAP_INVALID_ARG;
  return build_index(bucket_ids, K, V, off, len, idx, Ksorted, Vsorted, resident_ids, S, Hkv, N, Ncap, B, d, dtype,
                     slack, n_sink, n_recent, false, ws, ws_bytes, stream);
}

extern "C" int32_t saap_build_windowed_index_zeroed(const int32_t* bucket_ids, const void* K, const void* V,
                                                    int32_t* off, int32_t* len, int32_t* idx, void* Ksorted,
                                                    void* Vsorted, int32_t* resident_ids, int32_t S, int32_t Hkv,
                                                    int32_t N, int32_t Ncap, int32_t B, int32_t d, int32_t dtype,
                                                    int32_t slack, int32_t n_sink, int32_t n_recent, void* ws,
                                                    size_t ws_bytes, void* stream) {
  const Call call(stream);
  if (!resident_ids) return SAAP_INVALID_ARG;
  return build_index(bucket_ids, K, V, off, len, idx, Ksorted, Vsorted, resident_ids, S, Hkv, N, Ncap, B, d, dtype,
                     slack, n_sink, n_recent, true, ws, ws_bytes, stream);
}

extern "C" int32_t saap_window_push(const void* x_new, const void* k_new, const void* v_new,
                                    const int32_t* pos_new, const void* centroids, const float* bias,
                                    const int32_t* off, int32_t* len, int32_t* idx, void* Ksorted,
                                    void* Vsorted, int32_t* resident_ids, int32_t* new_bucket_ids,
                                    int32_t* overflow_flag, int32_t S, int32_t Hkv, int32_t Ncap, int32_t B,
                                    int32_t d, int32_t dtype, int32_t n_sink, int32_t n_recent, void* ws,
                                    size_t ws_bytes, void* stream) {
  const Call call(stream);
  if (!x_new || !k_new || !v_new || !pos_new || !centroids || !off || !len || !idx || !Ksorted || !Vsorted ||
      !resident_ids || !new_bucket_ids || !overflow_flag || !ws)
    return SAAP_INVALID_ARG;
  if (!aligned16(centroids) || !aligned16(ws)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || Ncap <= 0 || B <= 0 || n_sink < 0 || n_recent < 0) return SAAP_INVALID_ARG;
  if ((long long)n_sink + n_recent > Ncap) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD || B > SAAP_MAX_BUCKETS) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535 || units * sizeof(unsigned) > SAAP_WS_HEADER_BYTES) return SAAP_UNSUPPORTED;
  if (ws_bytes < push_workspace_bytes(units, B)) return SAAP_WORKSPACE_TOO_SMALL;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const int cpl = push_rounds(units, B);
  const int P = (B + kPushSlab * cpl - 1) / (kPushSlab * cpl);
  unsigned* counters = static_cast<unsigned*>(ws);
  PushPartial* part = reinterpret_cast<PushPartial*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  const dim3 grid((unsigned)P, (unsigned)units);
  if (dtype == SAAP_BF16)
    hipLaunchKernelGGL(window_push_kernel<bf16_t>, grid, dim3(kPushThreads), 0, hs, static_cast<const bf16_t*>(x_new),
                       static_cast<const bf16_t*>(k_new), static_cast<const bf16_t*>(v_new), pos_new,
                       static_cast<const bf16_t*>(centroids), bias, off, len, idx, static_cast<bf16_t*>(Ksorted),
                       static_cast<bf16_t*>(Vsorted), nullptr, nullptr, resident_ids, new_bucket_ids, overflow_flag, part, counters,
                       Hkv, Ncap, B, B + 1, n_sink, n_recent, P, cpl);
  else
    hipLaunchKernelGGL(window_push_kernel<float>, grid, dim3(kPushThreads), 0, hs, static_cast<const float*>(x_new),
                       static_cast<const float*>(k_new), static_cast<const float*>(v_new), pos_new,
                       static_cast<const float*>(centroids), bias, off, len, idx, static_cast<float*>(Ksorted),
                       static_cast<float*>(Vsorted), nullptr, nullptr, resident_ids, new_bucket_ids, overflow_flag, part, counters,
                       Hkv, Ncap, B, B + 1, n_sink, n_recent, P, cpl);
  return launch_status();
}

extern "C" int32_t saap_append_keys(const void* x_new, const void* k_new, const void* v_new,
                                    const int32_t* pos_new, const void* centroids, const float* bias,
                                    const int32_t* off, int32_t* len, int32_t* idx, void* Ksorted,
                                    void* Vsorted, int32_t* new_bucket_ids, int32_t* overflow_flag, int32_t S,
                                    int32_t Hkv, int32_t Ncap, int32_t B, int32_t d, int32_t dtype, void* ws,
                                    size_t ws_bytes, void* stream) {
  const Call call(stream);
  saap_trace_arm();
  if (!x_new || !k_new || !v_new || !centroids || !off || !len || !idx || !Ksorted || !Vsorted ||
      !new_bucket_ids || !overflow_flag || !ws)
    return SAAP_INVALID_ARG;
  if (!aligned16(centroids) || !aligned16(ws)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || Ncap <= 0 || B <= 0) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD || B > SAAP_MAX_BUCKETS) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535 || units * sizeof(unsigned) > SAAP_WS_HEADER_BYTES) return SAAP_UNSUPPORTED;
  if (ws_bytes < push_workspace_bytes(units, B)) return SAAP_WORKSPACE_TOO_SMALL;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const int cpl = push_rounds(units, B);
  const int P = (B + kPushSlab * cpl - 1) / (kPushSlab * cpl);
  unsigned* counters = static_cast<unsigned*>(ws);
  PushPartial* part = reinterpret_cast<PushPartial*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  const dim3 grid((unsigned)P, (unsigned)units);
  int32_t* no_resident = nullptr;
  // the push kernel on a plain index: no resident run, the key goes straight into its bucket
  if (dtype == SAAP_BF16)
    hipLaunchKernelGGL(window_push_kernel<bf16_t>, grid, dim3(kPushThreads), 0, hs, static_cast<const bf16_t*>(x_new),
                       static_cast<const bf16_t*>(k_new), static_cast<const bf16_t*>(v_new), pos_new,
                       static_cast<const bf16_t*>(centroids), bias, off, len, idx, static_cast<bf16_t*>(Ksorted),
                       static_cast<bf16_t*>(Vsorted), nullptr, nullptr, no_resident, new_bucket_ids, overflow_flag, part, counters, Hkv,
                       Ncap, B, B, 0, 0, P, cpl);
  else
    hipLaunchKernelGGL(window_push_kernel<float>, grid, dim3(kPushThreads), 0, hs, static_cast<const float*>(x_new),
                       static_cast<const float*>(k_new), static_cast<const float*>(v_new), pos_new,
                       static_cast<const float*>(centroids), bias, off, len, idx, static_cast<float*>(Ksorted),
                       static_cast<float*>(Vsorted), nullptr, nullptr, no_resident, new_bucket_ids, overflow_flag, part, counters, Hkv,
                       Ncap, B, B, 0, 0, P, cpl);
  return launch_status();
}

// The push kernel on an 8-bit cache (bf16 features and new rows, E4M3 rows in the cache).
// res_ids == nullptr: plain index (append), else the index with a resident run.
static int32_t push_fp8(const void* x_new, const void* k_new, const void* v_new, const int32_t* pos_new,
                        const void* centroids, const float* bias, const int32_t* off, int32_t* len, int32_t* idx,
                        uint8_t* K8, uint8_t* V8, const float* kscale, const float* vscale, int32_t* res_ids,
                        int32_t* new_bucket_ids, int32_t* overflow_flag, int32_t S, int32_t Hkv, int32_t Ncap,
                        int32_t B, int32_t d, int32_t n_sink, int32_t n_recent, void* ws, size_t ws_bytes,
                        void* stream) {
  if (!x_new || !k_new || !v_new || !centroids || !off || !len || !idx || !K8 || !V8 || !kscale || !vscale ||
      !new_bucket_ids || !overflow_flag || !ws)
    return SAAP_INVALID_ARG;
  if (!aligned16(centroids) || !aligned16(ws)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || Ncap <= 0 || B <= 0 || n_sink < 0 || n_recent < 0) return SAAP_INVALID_ARG;
  if (res_ids && (!pos_new || (long long)n_sink + n_recent > Ncap)) return SAAP_INVALID_ARG;
  if (d != kD || B > SAAP_MAX_BUCKETS) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535 || units * sizeof(unsigned) > SAAP_WS_HEADER_BYTES) return SAAP_UNSUPPORTED;
  if (ws_bytes < push_workspace_bytes(units, B)) return SAAP_WORKSPACE_TOO_SMALL;
  const int cpl = push_rounds(units, B);
  const int P = (B + kPushSlab * cpl - 1) / (kPushSlab * cpl);
  unsigned* counters = static_cast<unsigned*>(ws);
  PushPartial* part = reinterpret_cast<PushPartial*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  hipLaunchKernelGGL((window_push_kernel<bf16_t, fp8_t>), dim3((unsigned)P, (unsigned)units), dim3(kPushThreads), 0,
                     static_cast<hipStream_t>(stream), static_cast<const bf16_t*>(x_new),
                     static_cast<const bf16_t*>(k_new), static_cast<const bf16_t*>(v_new), pos_new,
                     static_cast<const bf16_t*>(centroids), bias, off, len, idx, K8, V8, kscale, vscale, res_ids,
                     new_bucket_ids, overflow_flag, part, counters, Hkv, Ncap, B, res_ids ? B + 1 : B, n_sink, n_recent,
                     P, cpl);
  return launch_status();
}

extern "C" int32_t saap_append_keys_fp8(const void* x_new, const void* k_new, const void* v_new,
                                        const int32_t* pos_new, const void* centroids, const float* bias,
                                        const int32_t* off, int32_t* len, int32_t* idx, uint8_t* K8, uint8_t* V8,
                                        const float* kscale, const float* vscale, int32_t* new_bucket_ids,
                                        int32_t* overflow_flag, int32_t S, int32_t Hkv, int32_t Ncap, int32_t B,
                                        int32_t d, void* ws, size_t ws_bytes, void* stream) {
  const Call call(stream);
  return push_fp8(x_new, k_new, v_new, pos_new, centroids, bias, off, len, idx, K8, V8, kscale, vscale, nullptr,
                  new_bucket_ids, overflow_flag, S, Hkv, Ncap, B, d, 0, 0, ws, ws_bytes, stream);
}

extern "C" int32_t saap_window_push_fp8(const void* x_new, const void* k_new, const void* v_new,
                                        const int32_t* pos_new, const void* centroids, const float* bias,
                                        const int32_t* off, int32_t* len, int32_t* idx, uint8_t* K8, uint8_t* V8,
                                        const float* kscale, const float* vscale, int32_t* resident_ids,
                                        int32_t* new_bucket_ids, int32_t* overflow_flag, int32_t S, int32_t Hkv,
                                        int32_t Ncap, int32_t B, int32_t d, int32_t n_sink, int32_t n_recent,
                                        void* ws, size_t ws_bytes, void* stream) {
  const Call call(stream);
  if (!resident_ids) return SAAP_INVALID_ARG;
  return push_fp8(x_new, k_new, v_new, pos_new, centroids, bias, off, len, idx, K8, V8, kscale, vscale, resident_ids,
                  new_bucket_ids, overflow_flag, S, Hkv, Ncap, B, d, n_sink, n_recent, ws, ws_bytes, stream);
}

extern "C" int32_t saap_recompact_index(const int32_t* off, const int32_t* len, const int32_t* idx,
                                        const void* Ksorted, const void* Vsorted, int32_t* off_new,
                                        int32_t* idx_new, void* Ksorted_new, void* Vsorted_new,
                                        int32_t* overflow_flag, int32_t S, int32_t Hkv, int32_t Ncap,
                                        int32_t Ncap_new, int32_t B, int32_t resident, int32_t d, int32_t dtype,
                                        int32_t slack_new, void* stream) {
  const Call call(stream);
  if (!off || !len || !idx || !Ksorted || !Vsorted || !off_new || !idx_new || !Ksorted_new || !Vsorted_new ||
      !overflow_flag)
    return SAAP_INVALID_ARG;
  const void* ptrs[] = {idx, Ksorted, Vsorted, idx_new, Ksorted_new, Vsorted_new};
  for (const void* p : ptrs)
    if (!aligned16(p)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || Ncap <= 0 || Ncap_new <= 0 || B <= 0 || slack_new < 0) return SAAP_INVALID_ARG;
  if (resident != 0 && resident != 1) return SAAP_INVALID_ARG;
  if (Ksorted == Ksorted_new || Vsorted == Vsorted_new || idx == idx_new || off == off_new) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD || B > SAAP_MAX_BUCKETS) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535) return SAAP_UNSUPPORTED;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const int runs = B + resident;
  hipLaunchKernelGGL(reoffset_kernel, dim3((unsigned)units), dim3(1024), 0, hs, len, off, off_new, runs, B, slack_new,
                     Ncap_new, overflow_flag);
  const size_t n_idx = (size_t)units * Ncap_new;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n_idx + 255) / 256)), dim3(256), 0, hs, idx_new, n_idx, -1);
  const dim3 grid((unsigned)runs, (unsigned)units);
  if (dtype == SAAP_BF16)
    hipLaunchKernelGGL(recopy_kernel<16>, grid, dim3(256), 0, hs, off, len, off_new, idx, idx_new,
                       static_cast<const uint4*>(Ksorted), static_cast<const uint4*>(Vsorted),
                       static_cast<uint4*>(Ksorted_new), static_cast<uint4*>(Vsorted_new), runs, Ncap, Ncap_new,
                       overflow_flag);
  else
    hipLaunchKernelGGL(recopy_kernel<32>, grid, dim3(256), 0, hs, off, len, off_new, idx, idx_new,
                       static_cast<const uint4*>(Ksorted), static_cast<const uint4*>(Vsorted),
                       static_cast<uint4*>(Ksorted_new), static_cast<uint4*>(Vsorted_new), runs, Ncap, Ncap_new,
                       overflow_flag);
  return launch_status();
}
