// Training of the query model f_q (Section 4 "Query assignment function", Eq. 1 of arXiv
// 2502.08246; Appendix "Training details": Adam):
//   z = W2 relu(W1 x + b1) + b2,  f_q(x) = softmax(z),
//   L = 1/R sum_r sum_b T[r,b] (log T[r,b] - log f_q(x_r)[b])       (T: bucket attention mass, rows of A*H_k)
// With batch normalisation (the model of Section 6.1) the hidden layer is
//   relu(gamma * (a - mean_r a) / sqrt(var_r a + eps) + beta),  a = W1 x + b1,
// and fold_batch_norm turns the trained layer into plain W1, b1 for inference.
// query_model_loss_grads computes L and the gradients of all four parameter tensors for a batch,
// adam_update applies one Adam step to a tensor; a training step is the first call followed by
// the second on each tensor.  All arithmetic is fp32 or, in the large products, as exact as fp32 (below); every sum is
// taken by one thread or one workgroup in a fixed order (no atomics), so a step is reproducible bit for bit.
//
// The five matrix products run on the matrix cores.  fp32 matrix instructions reach 154 TFLOP/s in a large product on this card
// and take the vector units' time; bfloat16 ones do 16 times the work in the same cycles.  So the operands of a large product
// are split into three bfloat16 each on their way to LDS (nothing is lost: 3 x 8 bits, the values scaled up before the split so
// that the last bits of the smallest ones are bfloat16 values too) and six products of those make one fp32 product, the five
// small ones summed apart: the gradients' error against float64 is 0.6 to 1.0 times that of fp32 matrix instructions (8 x 1000
// rows, 512 hidden units, 1024 buckets: dW1 3.8e-7 instead of 6.2e-7, dW2 3.2e-7 instead of 4.7e-7).  A sum of one term only,
// where nothing averages out, is 1.03 times as far off: the products of planes left out are up to 2^-26 of it.
// Operands whose scaled values a bfloat16 does not hold (infinities, NaN, from 2^104 on) make the tile not finite, and so do sums
// from 2^80 on; it is then done again with fp32 instructions.  The first product stays in fp32, and so do results of few tiles
// (gemm_split_kernel).
// Features in bfloat16 are read as they are: one plane in the last product, widened on their way to LDS in the first (a launch of its
// own that widened them took 5 us).
// Bounds are free (R, B, hidden; rows that are no multiple of 16 bytes are read element by element).  The bias gradients are the
// column sums of an operand of a weight gradient: the workgroups of the first tile column add them up as they load it.
// 8 weight sets, 1000 rows, 128 -> 512 -> 1024: the three large products 93 us each with fp32 instructions, 49 to 53 now, the scaling
// included (1.0 PFLOP/s of bfloat16 products; a loop of nothing but these instructions on such data runs at 1.8 GHz: 27 us).  What is
// left is the start and the stores of a product, 12 us that nothing covers (all tiles of a product run at once), and the slices'
// barriers.
#include <algorithm>

#include "common.h"

namespace saap {
namespace {

constexpr int kGemmThreads = 256;

enum { EPI_NONE = 0, EPI_BIAS = 1, EPI_BIAS_RELU = 2, EPI_MASK = 3 };

struct GemmArgs {
  const void* A;       // TA ? [K,M] : [M,K]   (EA: float, or bf16_t for features that come as such)
  const void* B;       // TB ? [N,K] : [K,N]   (EB)
  float* C;            // [M,N]
  const float* bias;   // [N]   (EPI_BIAS, EPI_BIAS_RELU)
  const float* aux;    // [M,N] (EPI_MASK: C = aux > 0 ? acc : 0)
  int M, N, K;
  long long sA, sB, sC, sBias, sAux;   // strides between the weight sets (blockIdx.x), in elements
  float* colsum;       // [M] per weight set or null: sums of A' over k (TA only), strides sColsum
  long long sColsum;
  int m_first, n_first;                // gemm_split_kernel: where the launch's first tile starts
};

// fp32 values as sums of three bfloat16 each, to 24 bits and more: the nearest one, the nearest to what that leaves, and the
// nearest to what is left then.  This takes the values' next plane, as pairs, and leaves the rest.
// An fp32 value is a multiple of 2^-149, the smallest normal bfloat16 is 2^-126: scaled by 2^24 (exact) a value of any size keeps
// its 24 bits.  (Unscaled, the third plane of values below 2^-110 and then the second fall below the smallest bfloat16: 9e-6 of
// products of operands near 2^-118, which fp32 instructions have to 5e-7.  The multiplication takes 4 to 6 % of a product's time:
// 57 to 59 us without it, 60 to 63 with.)
constexpr float kUp = 16777216.f, kDown = 1.f / (kUp * kUp);
template <int E>
__device__ __forceinline__ void take_plane(float* rest, uint32_t* u) {
#pragma unroll
  for (int e = 0; e < E / 2; ++e) {
    u[e] = pack_bf16(rest[2 * e], rest[2 * e + 1]);
    rest[2 * e] -= bf16_lo(u[e]);
    rest[2 * e + 1] -= bf16_hi(u[e]);
  }
}
// The six products of planes that make a product of fp32 values, the smallest first; those of planes 1 and 2, and of 2 and 2,
// are below 2^-26 of the whole.
constexpr int kPlaneA[6] = {2, 0, 1, 1, 0, 0}, kPlaneB[6] = {0, 2, 1, 0, 1, 0};

// One thread's share of a slice of an operand, R rows by 16 values of k, on its way to LDS.  LDS holds the
// three planes, each [k / 8][row][k % 8]; a lane of the matrix cores takes eight values of k.  KC: the
// operand's contiguous dimension is k (VEC: rows start on 16 bytes), else it is the row dimension (a wave loads 64 neighbouring
// rows at one k).  The pitches keep reads and writes free of bank conflicts.
constexpr int kSlice = 16;
// (rows x K values from p on, fewer than 2^29; no load relies on the buffer's bounds)
template <typename E>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_buffer(const E* p, int rows, int K) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<E*>(p), 0, rows * K * (int)sizeof(E), 0x00027000);
}
// T: float, or bf16_t: one plane holds the value.
template <bool KC, bool VEC, int R, int THREADS, typename T>
struct PlaneLoader {
  static constexpr int kPlanes = sizeof(T) == 4 ? 3 : 1;
  static_assert(sizeof(T) == 4 || !KC, "bfloat16 operands that are contiguous along k: not needed");
  static constexpr int E = R * kSlice / THREADS;          // consecutive values of k of one row: 8 or 4
  static constexpr int kPitch = R + (KC ? 4 : 0), kPlane = kSlice / 8 * kPitch, kUnits = kPlanes * kPlane;   // units of 16 bytes
  static_assert(E == 8 || E == 4, "whole pieces of a row's values");
  float r[E];
  static __device__ __forceinline__ int tid() { return threadIdx.x % THREADS; }          // THREADS threads share an operand's slice
  static __device__ __forceinline__ int row() { return KC ? tid() / (kSlice / E) : tid() % R; }
  static __device__ __forceinline__ int first_k() { return E * (KC ? tid() % (kSlice / E) : tid() / R); }
  // Byte offset of the thread's values from the slice's first: all that a lane adds to an address that the whole workgroup
  // shares.  Rows past the end repeat the last one and are not stored.
  static __device__ __forceinline__ int offset(int t0, int n_t, int K) {
    const int t = min(t0 + row(), n_t - 1);
    return (int)sizeof(T) * (KC ? t * K + first_k() : first_k() * n_t + t);
  }
  // The slice from k0 on, or the last 16 values of k where it would reach past the end.
  __device__ __forceinline__ void fetch(__amdgpu_buffer_rsrc_t x, int at, int k0, int n_t, int K) {
    k0 = min(k0, K - kSlice);
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int e = 0; e < E; ++e) r[e] = __uint_as_float((unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(x, at, 2 * (k0 + e) * n_t, 0) << 16);
    } else if constexpr (KC && VEC) {
#pragma unroll
      for (int e = 0; e < E; e += 4) {
        const u32x4_t u = __builtin_amdgcn_raw_buffer_load_b128(x, at + 4 * e, 4 * k0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) r[e + j] = __uint_as_float(u[j]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e)
        r[e] = __uint_as_float(KC ? __builtin_amdgcn_raw_buffer_load_b32(x, at + 4 * e, 4 * k0, 0)
                                  : __builtin_amdgcn_raw_buffer_load_b32(x, at, 4 * (k0 + e) * n_t, 0));
    }
  }
  __device__ __forceinline__ void clear_from(int k) {
#pragma unroll
    for (int e = 0; e < E; ++e) r[e] = first_k() + e < k ? r[e] : 0.f;
  }
  // up: kUp, or 0 for a slice that does not count
  __device__ __forceinline__ void stash(uint4* s, float up) const {
    float rest[E];
#pragma unroll
    for (int e = 0; e < E; ++e) rest[e] = r[e] * up;
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
      uint32_t u[E / 2];
      take_plane<E>(rest, u);
      uint4* at = s + p * kPlane + first_k() / 8 * kPitch + row();
      if constexpr (E == 8) *at = make_uint4(u[0], u[1], u[2], u[3]);
      else reinterpret_cast<uint2*>(at)[first_k() / 4 % 2] = make_uint2(u[0], u[1]);
    }
  }
  __device__ __forceinline__ float sum() const {
    float t = (r[0] + r[1]) + (r[2] + r[3]);
    if constexpr (E == 8) t += (r[4] + r[5]) + (r[6] + r[7]);
    return t;
  }
  static __device__ __forceinline__ bf16x8_t read(const uint4* s, int plane, int row, int kg) {
    return __builtin_bit_cast(bf16x8_t, s[plane * kPlane + kg * kPitch + row]);
  }
};

// Four neighbouring values (VEC: they start on a multiple of four).
template <bool VEC>
__device__ __forceinline__ float4 four_of(const float* p) {
  if constexpr (VEC) return *reinterpret_cast<const float4*>(p);
  return make_float4(p[0], p[1], p[2], p[3]);
}
template <bool VEC>
__device__ __forceinline__ float4 four_of(const bf16_t* p) {
  if constexpr (VEC) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    return make_float4(bf16_lo(u.x), bf16_hi(u.x), bf16_lo(u.y), bf16_hi(u.y));
  }
  return make_float4(Vec8<bf16_t>::widen(p[0]), Vec8<bf16_t>::widen(p[1]), Vec8<bf16_t>::widen(p[2]), Vec8<bf16_t>::widen(p[3]));
}

// The same in fp32 for operands whose contiguous dimension is k: R rows by SL values of k, four a piece.  LDS holds [row][k], a
// lane reads four k at a time; product (g, j) of a slice sums k = 8 g + 4 (lane / 32) + j.
template <bool VEC, int R, int SL, typename T>
struct SliceLoader {
  static constexpr int kPieces = R * SL / 4 / kGemmThreads, kPitch = SL + 4, kFloats = R * kPitch;
  float4 r[kPieces];
  // piece i of this thread: row t, four values from k on
  static __device__ __forceinline__ void place(int i, int& t, int& k) {
    const int q = threadIdx.x + i * kGemmThreads;
    k = q % (SL / 4) * 4;
    t = q / (SL / 4);
  }
  // (fp32 matrix products and ordinary vector instructions take the same units by turns: address arithmetic per slice cost a
  // fifth of the products' time.)
  struct Offsets { unsigned at[kPieces]; };
  static __device__ __forceinline__ Offsets offsets(int t0, int n_t, int K) {
    Offsets o;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      int t, k;
      place(i, t, k);
      o.at[i] = (unsigned)sizeof(T) * (unsigned)(min(t0 + t, n_t - 1) * K + k);
    }
    return o;
  }
  // The slice from k0 on; where it would reach past the end of k, the last SL values instead, of which stash() clears those
  // before k0.  (Cleared here, they would be waited for here.)
  __device__ __forceinline__ void fetch(const T* X, const Offsets& o, int k0, int K) {
    const char* x = reinterpret_cast<const char*>(X + min(k0, K - SL));
#pragma unroll
    for (int i = 0; i < kPieces; ++i) r[i] = four_of<VEC>(reinterpret_cast<const T*>(x + o.at[i]));
  }
  __device__ __forceinline__ void stash(float* s, int k0, int K) {
    const int before = k0 - min(k0, K - SL);              // values of the slice that belong to the one before it
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      int t, k;
      place(i, t, k);
      if (before > 0) {
        r[i].x = k >= before ? r[i].x : 0.f;
        r[i].y = k + 1 >= before ? r[i].y : 0.f;
        r[i].z = k + 2 >= before ? r[i].z : 0.f;
        r[i].w = k + 3 >= before ? r[i].w : 0.f;
      }
      *reinterpret_cast<float4*>(s + t * kPitch + k) = r[i];
    }
  }
  // the lane's four values of k of group g, of row `row`
  static __device__ __forceinline__ float4 read(const float* s, int row, int g, int half) {
    return *reinterpret_cast<const float4*>(s + row * kPitch + 8 * g + 4 * half);
  }
};

typedef __attribute__((ext_vector_type(16))) float f32x16_t;

// Registers r of a lane hold rows m0 + 8*(r/4) + 4*half + r%4 of column n.
template <int EPI, int REGS, typename V>
__device__ __forceinline__ void store_tile(const GemmArgs& g, int w, int m0, int n, int half, const V& acc) {
  if (n >= g.N) return;
  float bias = 0.f;
  if (EPI == EPI_BIAS || EPI == EPI_BIAS_RELU) bias = g.bias[(size_t)w * g.sBias + n];
  auto row = [&](int r) { return m0 + 8 * (r / 4) + 4 * half + (r % 4); };
  float aux[REGS];
  if (EPI == EPI_MASK) {
#pragma unroll
    for (int r = 0; r < REGS; ++r) aux[r] = g.aux[(size_t)w * g.sAux + (size_t)min(row(r), g.M - 1) * g.N + n];
  }
  float* C = g.C + (size_t)w * g.sC + n;
#pragma unroll
  for (int r = 0; r < REGS; ++r) {
    float v = acc[r];
    if (EPI == EPI_BIAS || EPI == EPI_BIAS_RELU) v += bias;
    if (EPI == EPI_BIAS_RELU) v = fmaxf(v, 0.f);
    if (EPI == EPI_MASK) v = aux[r] > 0.f ? v : 0.f;
    if (row(r) < g.M) C[(size_t)row(r) * g.N] = v;
  }
}

constexpr int kDirect = 32;
template <bool KC, bool VEC, typename T>
struct DirectOperand {
  float r[4][4];                                         // [g][j]: k = k0 + 8 g + 4 (lane / 32) + j, the same for both operands
  __device__ __forceinline__ void fetch(const T* X, int t0, int k0, int n_t, int K) {
    const int lane = threadIdx.x & 63, half = lane >> 5, t = min(t0 + (lane & 31), n_t - 1);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int k = k0 + 8 * g + 4 * half;
      if constexpr (KC && VEC) {
        const float4 v = four_of<true>(X + (size_t)t * K + min(k, K - 4));
        r[g][0] = v.x; r[g][1] = v.y; r[g][2] = v.z; r[g][3] = v.w;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) r[g][j] = Vec8<T>::widen(KC ? X[(size_t)t * K + min(k + j, K - 1)] : X[(size_t)min(k + j, K - 1) * n_t + t]);
      }
    }
  }
  __device__ __forceinline__ void clear(int k0, int K) {
    const int half = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) r[g][j] = k0 + 8 * g + 4 * half + j < K ? r[g][j] : 0.f;
  }
};

// A matrix tile of the product in fp32, operands straight from memory (a lane loads what the matrix cores take from it).
template <bool TA, bool TB, bool VEC, typename EA, typename EB>
__device__ __forceinline__ f32x16_t fp32_tile(const GemmArgs& g, const EA* A, const EB* B, int m0, int n0) {
  f32x16_t acc = {0};
  DirectOperand<!TA, VEC, EA> a;
  DirectOperand<TB, VEC, EB> b;
#pragma unroll 1
  for (int k0 = 0; k0 < g.K; k0 += kDirect) {
    a.fetch(A, m0, k0, g.M, g.K);
    b.fetch(B, n0, k0, g.N, g.K);
    if (k0 + kDirect > g.K) {
      a.clear(k0, g.K);
      b.clear(k0, g.K);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.r[q][j], b.r[q][j], acc, 0, 0, 0);
  }
  return acc;
}

// Whether the wave's tile holds numbers only.  (x - x is 0 for a number and NaN otherwise.)
__device__ __forceinline__ bool all_finite(const f32x16_t& v) {
  float d = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) d += v[r] - v[r];
  return __ballot(d != 0.f) == 0;
}

// C = A B^T in fp32 (the first product).  A workgroup of two by two waves owns a tile of 64 TM x 64, a wave TM matrix tiles of 32.
template <int EPI, bool VEC, int TM, int SL, typename EA>
__global__ void __launch_bounds__(kGemmThreads, 4)
gemm_f32_kernel(GemmArgs g) {
  constexpr int BM = 64 * TM, BN = 64;
  typedef SliceLoader<VEC, BM, SL, EA> LoadA;
  typedef SliceLoader<VEC, BN, SL, float> LoadB;
  __shared__ __align__(16) float s_ab[2][LoadA::kFloats + LoadB::kFloats];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w = blockIdx.x, n0 = blockIdx.y * BN, m0 = blockIdx.z * BM;
  const EA* A = static_cast<const EA*>(g.A) + (size_t)w * g.sA;
  const float* B = static_cast<const float*>(g.B) + (size_t)w * g.sB;
  const int wm = (wave >> 1) * 32 * TM, wn = (wave & 1) * 32;
  const int col = lane & 31, half = lane >> 5;
  f32x16_t acc[TM];
#pragma unroll
  for (int a = 0; a < TM; ++a) acc[a] = (f32x16_t){0};

  const typename LoadA::Offsets oa = LoadA::offsets(m0, g.M, g.K);
  const typename LoadB::Offsets ob = LoadB::offsets(n0, g.N, g.K);
  struct Staged { LoadA a; LoadB b; };
  auto fetch = [&](Staged& st, int k0) {
    st.a.fetch(A, oa, k0, g.K);
    st.b.fetch(B, ob, k0, g.K);
    __builtin_amdgcn_sched_barrier(0);                          // left alone the compiler moves the loads behind the products
  };
  auto stash = [&](Staged& st, int buf, int k0) {
    st.a.stash(s_ab[buf], k0, g.K);
    st.b.stash(s_ab[buf] + LoadA::kFloats, k0, g.K);
  };
  auto compute = [&](int buf) {
    const float* sa = s_ab[buf];
    const float* sb = s_ab[buf] + LoadA::kFloats;
#pragma unroll
    for (int q = 0; q < SL / 8; ++q) {
      const float4 b = LoadB::read(sb, wn + col, q, half);
      float4 a[TM];
#pragma unroll
      for (int t = 0; t < TM; ++t) a[t] = LoadA::read(sa, wm + 32 * t + col, q, half);
#pragma unroll
      for (int t = 0; t < TM; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t].x, b.x, acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < TM; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t].y, b.y, acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < TM; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t].z, b.z, acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < TM; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t].w, b.w, acc[t], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int n_slices = (g.K + SL - 1) / SL;
  Staged even, odd;
  fetch(even, 0);
  fetch(odd, SL);
  stash(even, 0, 0);
  __syncthreads();
  for (int c = 0; c < n_slices; c += 2) {
    fetch(even, (c + 2) * SL);
    compute(0);
    stash(odd, 1, (c + 1) * SL);
    __syncthreads();
    fetch(odd, (c + 3) * SL);
    if (c + 1 < n_slices) compute(1);
    stash(even, 0, (c + 2) * SL);
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < TM; ++t) store_tile<EPI, 16>(g, w, m0 + wm + 32 * t, n0 + wn + col, half, acc[t]);
}

// C = A' B'; A' is M x K, B' is K x N.  Two by WN waves own a tile of 64 TM x 32 WN, a wave TM matrix tiles of 32.  KS: the
// workgroup has as many such groups of waves, which share out k and add up at the end.
template <bool TA, bool TB, int EPI, bool VEC, typename EB, int TM, int WN, int KS>
__global__ void __launch_bounds__(128 * WN * KS, KS > 2 ? 1 : 2)
gemm_kernel(GemmArgs g) {
  constexpr int kThreads = 128 * WN, BM = 64 * TM, BN = 32 * WN;
  typedef PlaneLoader<!TA, VEC, BM, kThreads, float> LoadA;
  typedef PlaneLoader<TB, VEC, BN, kThreads, EB> LoadB;
  constexpr int kUnits = LoadA::kUnits + LoadB::kUnits;
  __shared__ uint4 s_all[KS * 2 * kUnits];
  const int lane = threadIdx.x & 63, wave = threadIdx.x % kThreads >> 6;
  const int part = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads) : 0;       // of k
  const int w = blockIdx.x, n0 = blockIdx.y * BN, m0 = blockIdx.z * BM;
  const float* A = static_cast<const float*>(g.A) + (size_t)w * g.sA;
  const EB* B = static_cast<const EB*>(g.B) + (size_t)w * g.sB;
  const int wm = wave / WN * 32 * TM, wn = wave % WN * 32;
  const int col = lane & 31, half = lane >> 5;
  uint4* const s_ab = s_all + part * 2 * kUnits;
  const bool sums = TA && g.colsum != nullptr && blockIdx.y == 0;
  float csum = 0.f;                                             // of the thread's row of A' (TA: it is always the same)
  f32x16_t acc[TM], low[TM];                                    // the sums of the products of planes 0, and of the others
#pragma unroll
  for (int t = 0; t < TM; ++t) acc[t] = low[t] = (f32x16_t){0};

  const int oa = LoadA::offset(m0, g.M, g.K), ob = LoadB::offset(n0, g.N, g.K);
  const __amdgpu_buffer_rsrc_t ra = operand_buffer(A, g.M, g.K), rb = operand_buffer(B, g.N, g.K);
  struct Staged { LoadA a; LoadB b; };
  Staged even, odd;
  auto fetch = [&](Staged& st, int k0) {
    st.a.fetch(ra, oa, k0, g.M, g.K);
    st.b.fetch(rb, ob, k0, g.N, g.K);
  };
  auto stash = [&](const Staged& st, int buf, bool live) {
    st.a.stash(s_ab + buf * kUnits, KS > 1 && !live ? 0.f : kUp);
    st.b.stash(s_ab + buf * kUnits + LoadA::kUnits, kUp);
    if (TA) csum += __int_as_float(__float_as_int(st.a.sum()) & -(int)live);    // (a select would become a branch)
  };
  // the slice in buffer `buf`; the split of the next one runs under its products
  auto step = [&](Staged& st, int buf, int k0_next, int end) {
    const uint4* sa = s_ab + buf * kUnits;
    const uint4* sb = sa + LoadA::kUnits;
    bf16x8_t a[TM][3], b[LoadB::kPlanes];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (p < LoadB::kPlanes) b[p] = LoadB::read(sb, p, wn + col, half);
#pragma unroll
      for (int t = 0; t < TM; ++t) a[t][p] = LoadA::read(sa, p, wm + 32 * t + col, half);
    }
    stash(st, buf ^ 1, k0_next < end);
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        if (kPlaneB[i] >= LoadB::kPlanes) continue;
        f32x16_t& sum = i < 5 ? low[t] : acc[t];
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t][kPlaneA[i]], b[kPlaneB[i]], sum, 0, 0, 0);
      }
    // moved up, the loads would get other registers than the values that they replace, and be waited for when copied over
    __builtin_amdgcn_sched_barrier(0);
    fetch(st, k0_next + 2 * kSlice);
    __syncthreads();
  };
  // The first slice of all is the one that may be short: the values of one operand past its end are taken out (an infinity or NaN
  // of the other there spoils the tile, which is then done again, and so does one of a slice that counts for another part only).
  const int n_slices = (g.K + kSlice - 1) / kSlice, short_by = n_slices * kSlice - g.K;
  const int per = (n_slices + KS - 1) / KS;                     // slices of a part; one that has fewer goes through the motions
  const int i0 = part * per, end = KS > 1 ? min(g.K, (i0 + per) * kSlice - short_by) : g.K;
  auto start = [&](int i) { return i * kSlice - short_by; };    // of slice i >= 1, and where the values after slice 0 start
  fetch(even, max(start(i0), 0));
  fetch(odd, start(i0 + 1));
  if (i0 == 0) even.a.clear_from(kSlice - short_by);
  stash(even, 0, max(start(i0), 0) < end);
  fetch(even, start(i0 + 2));
  __syncthreads();
  int k0 = start(i0 + 1);
  int pairs = per / 2;
  do {
    step(odd, 0, k0, end);
    step(even, 1, k0 + kSlice, end);
    k0 += 2 * kSlice;
  } while (--pairs > 0);
  if (per & 1) step(odd, 0, k0, end);
  if (TA && sums) {
    // the threads that loaded the same row add up in a fixed order
    constexpr int kGroups = KS * kThreads / BM;
    float* s = reinterpret_cast<float*>(s_all);                 // [kGroups][BM]
    s[threadIdx.x] = csum;
    __syncthreads();
    if (threadIdx.x < BM && m0 + (int)threadIdx.x < g.M) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < kGroups; ++i) t += s[i * BM + threadIdx.x];
      g.colsum[(size_t)w * g.sColsum + m0 + threadIdx.x] = t;
    }
    if (KS > 1) __syncthreads();
  }
  // not a number, infinite, or too large for a scaled bfloat16: as fp32 products have it
  if constexpr (KS == 1) {
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int tm = m0 + wm + 32 * t, tn = n0 + wn;
      acc[t] = (acc[t] + low[t]) * kDown;
      if (!all_finite(acc[t])) acc[t] = fp32_tile<TA, TB, VEC>(g, A, B, tm, tn);
      store_tile<EPI, 16>(g, w, tm, tn + col, half, acc[t]);
    }
  } else {
    // part i adds up registers 16 / KS * i and on of all parts, in order
    static_assert(TM == 1 && (KS == 2 || KS == 4), "a matrix tile per wave");
    constexpr int kWaves = kThreads / 64, kQuads = 4 / KS;
    static_assert(KS * kWaves * 4 * 64 <= KS * 2 * kUnits, "the parts' sums take the operands' place");
    float4* s = reinterpret_cast<float4*>(s_all);               // [part][wave][four registers][lane]
    const f32x16_t mine = acc[0] + low[0];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      s[((part * kWaves + wave) * 4 + q) * 64 + lane] = make_float4(mine[4 * q], mine[4 * q + 1], mine[4 * q + 2], mine[4 * q + 3]);
    __syncthreads();
    const int tm = m0 + wm, tn = n0 + wn;
    f32x4_t sum[kQuads];
    float d = 0.f;
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
      sum[q] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        const float4 v = s[((i * kWaves + wave) * 4 + part * kQuads + q) * 64 + lane];
        sum[q] += (f32x4_t){v.x, v.y, v.z, v.w};
      }
      sum[q] *= kDown;
#pragma unroll
      for (int r = 0; r < 4; ++r) d += sum[q][r] - sum[q][r];
    }
    if (__ballot(d != 0.f) != 0) {
      const f32x16_t all = fp32_tile<TA, TB, VEC>(g, A, B, tm, tn);
#pragma unroll
      for (int i = 0; i < KS; ++i)
        if (i == part)
#pragma unroll
          for (int q = 0; q < kQuads; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[q][r] = all[4 * (i * kQuads + q) + r];
    }
#pragma unroll
    for (int q = 0; q < kQuads; ++q) store_tile<EPI, 4>(g, w, tm + 8 * (part * kQuads + q), tn + col, half, sum[q]);
  }
}

// C = A' B' in fp32 for results of few tiles: a workgroup owns one matrix tile, its four waves a quarter of the k each, operands straight
// from memory (a lane loads what the matrix cores take from it), the next slice's loads in flight.
template <bool TA, bool TB, int EPI, bool VEC, typename EA, typename EB>
__global__ void __launch_bounds__(kGemmThreads, !VEC ? 2 : sizeof(EB) == 2 ? 3 : 4)
gemm_split_kernel(GemmArgs g) {
  constexpr int kStep = 4 * kDirect;
  __shared__ float4 s_red[4 * 4 * 64];                   // [wave][four registers][lane]
  __shared__ float s_sum[4 * 32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
  const int w = blockIdx.x, n0 = g.n_first + (int)blockIdx.y * 32, m0 = g.m_first + (int)blockIdx.z * 32;
  const EA* A = static_cast<const EA*>(g.A) + (size_t)w * g.sA;
  const EB* B = static_cast<const EB*>(g.B) + (size_t)w * g.sB;
  const bool sums = TA && g.colsum != nullptr && n0 == 0;
  float csum = 0.f;                                      // of the lane's column of A, this half's k
  f32x16_t acc = {0};
  struct Staged { DirectOperand<!TA, VEC, EA> a; DirectOperand<TB, VEC, EB> b; };
  auto fetch = [&](Staged& st, int k0) {
    st.a.fetch(A, m0, k0, g.M, g.K);
    st.b.fetch(B, n0, k0, g.N, g.K);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&](Staged& st, int k0) {
    if (k0 + kDirect > g.K) {
      st.a.clear(k0, g.K);
      st.b.clear(k0, g.K);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(st.a.r[q][j], st.b.r[q][j], acc, 0, 0, 0);
        if (TA && sums) csum += st.a.r[q][j];
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  Staged even, odd;
  fetch(even, wave * kDirect);
  for (int k0 = wave * kDirect; k0 < g.K; k0 += 2 * kStep) {
    fetch(odd, k0 + kStep);                              // past the end: the last values again, not used
    compute(even, k0);
    fetch(even, k0 + 2 * kStep);
    if (k0 + kStep < g.K) compute(odd, k0 + kStep);
  }
  // wave i adds up registers 4 i .. 4 i + 3 of the four
#pragma unroll
  for (int i = 0; i < 4; ++i) s_red[(wave * 4 + i) * 64 + lane] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
  csum += __shfl_xor(csum, 32);
  if (half == 0) s_sum[wave * 32 + col] = csum;
  __syncthreads();
  float4 t = s_red[wave * 64 + lane];
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    const float4 v = s_red[(i * 4 + wave) * 64 + lane];
    t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
  }
  const f32x4_t part = {t.x, t.y, t.z, t.w};
  store_tile<EPI, 4>(g, w, m0 + 8 * wave, n0 + col, half, part);
  if (sums && threadIdx.x < 32 && m0 + col < g.M)
    g.colsum[(size_t)w * g.sColsum + m0 + col] = (s_sum[col] + s_sum[32 + col]) + (s_sum[64 + col] + s_sum[96 + col]);
}

// Products of planes: 128 x 128 tiles of eight waves where every compute unit has one (8 sets, 1000 rows, 512 x 1024: 49 to 53 us a
// product; 62 to 68 with 128 x 64 and four waves, which split twice as many values for a matrix instruction and read their operands
// from LDS no slower than that takes), unless half of the last column stays empty and there are few of them (8192 rows, 64 columns:
// 64 us with 128 x 64, 87; 192: 45 and 49; 576: 40 either way).  64 x 64 with more than two workgroups per compute unit.  Below that a
// slice's chain (operands from LDS, split, products, barrier: 0.7 us) is what takes the time, so that more waves share out k: two
// groups (4 sets, 1000 rows, 512 x 1024: 42 -> 37 us; 8 sets, 96 x 1024: 32 -> 24), four where every compute unit has one workgroup
// at most (20 of those 24; 1 set, 512 x 1024: 20 -> 16).
// With fewer than 512 matrix tiles, or 640 where k is short, a tile's k is shared out over four waves in fp32 (8 sets, 1024 rows, 192 x
// 128: 9 us, 17; 4 sets, 100 rows, 512 x 256: 6.5 us, 8.0), and so it is where k is too short to be shared out or an operand too large
// for offsets of 32 bits; that one takes several launches where a grid dimension has no room for its smaller tiles.
constexpr long long kMostTiles = 65535;
template <bool TA, bool TB, int EPI, bool VEC, bool F32, typename EA, typename EB>
void gemm_sized(const GemmArgs& g, int Hw, hipStream_t hs) {
  auto grid = [&](int bm, int bn) { return dim3((unsigned)Hw, (unsigned)((g.N + bn - 1) / bn), (unsigned)((g.M + bm - 1) / bm)); };
  auto count = [&](int bm, int bn) { const dim3 d = grid(bm, bn); return (long long)d.x * d.y * d.z; };
  const bool tiled = g.K >= 32 && (long long)g.M * g.K < (1ll << 29) && (long long)g.N * g.K < (1ll << 29) && g.N <= kMostTiles * 64;
  if constexpr (F32) {
    static_assert(!TA && TB && sizeof(EB) == 4, "rows of both operands along k");
    // 128 x 64 tiles where they give every compute unit the four workgroups it has room for, or else 64 x 64 with slices twice as
    // long for the same LDS
    if (tiled && count(128, 64) >= 4LL * device_cus()) {
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, VEC, 2, 16, EA>), grid(128, 64), dim3(kGemmThreads), 0, hs, g);
      return;
    }
    if (tiled && count(64, 64) >= device_cus()) {
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, VEC, 1, 32, EA>), grid(64, 64), dim3(kGemmThreads), 0, hs, g);
      return;
    }
  } else {
    static_assert(sizeof(EA) == 4, "three planes");
    auto launch = [&](auto kernel, int bm, int bn, int threads) { hipLaunchKernelGGL(kernel, grid(bm, bn), dim3(threads), 0, hs, g); };
    const int columns = (g.N + 63) / 64;
    const bool half_empty = columns < 7 && columns % 2 == 1;      // the last tile of 128 columns, and it counts
    if (tiled && half_empty && count(128, 64) >= 2LL * device_cus()) return launch(gemm_kernel<TA, TB, EPI, VEC, EB, 2, 2, 1>, 128, 64, 256);
    if (tiled && !half_empty && count(128, 128) >= device_cus()) return launch(gemm_kernel<TA, TB, EPI, VEC, EB, 2, 4, 1>, 128, 128, 512);
    if (tiled && count(64, 64) > 2LL * device_cus()) return launch(gemm_kernel<TA, TB, EPI, VEC, EB, 1, 2, 1>, 64, 64, 256);
    if (tiled && g.K >= 128 && count(64, 64) <= device_cus() && count(32, 32) >= 2LL * device_cus())
      return launch(gemm_kernel<TA, TB, EPI, VEC, EB, 1, 2, 4>, 64, 64, 1024);
    if (tiled && g.K >= 64 && 2 * count(32, 32) >= 5LL * device_cus()) return launch(gemm_kernel<TA, TB, EPI, VEC, EB, 1, 2, 2>, 64, 64, 512);
    if (tiled && count(64, 64) >= device_cus()) return launch(gemm_kernel<TA, TB, EPI, VEC, EB, 1, 2, 1>, 64, 64, 256);
  }
  for (long long m = 0; m < g.M; m += kMostTiles * 32)
    for (long long n = 0; n < g.N; n += kMostTiles * 32) {
      GemmArgs part = g;
      part.m_first = (int)m;
      part.n_first = (int)n;
      auto tiles = [](long long left) { return (unsigned)std::min((left + 31) / 32, kMostTiles); };
      hipLaunchKernelGGL((gemm_split_kernel<TA, TB, EPI, VEC, EA, EB>), dim3((unsigned)Hw, tiles(g.N - n), tiles(g.M - m)), dim3(kGemmThreads),
                         0, hs, part);
    }
}

// F32: every product and sum in fp32, for the first product: a hidden unit's sign decides which gradients flow through it, and
// a unit that another rounding moves across zero moves them by far more than a rounding.
template <bool TA, bool TB, int EPI, bool F32 = false, typename EA = float, typename EB = float>
void gemm(const GemmArgs& g, int Hw, hipStream_t hs) {
  // loads of four values need rows of both operands that start on a multiple of four
  auto rows_aligned = [](const void* p, int ld, long long stride) { return aligned16(p) && ld % 4 == 0 && stride % 4 == 0; };
  if (rows_aligned(g.A, TA ? g.M : g.K, g.sA) && rows_aligned(g.B, TB ? g.K : g.N, g.sB)) gemm_sized<TA, TB, EPI, true, F32, EA, EB>(g, Hw, hs);
  else gemm_sized<TA, TB, EPI, false, F32, EA, EB>(g, Hw, hs);
}

// Sum of a workgroup's values, in a fixed order; every thread gets it.  s_red: 256/64 + 1 floats.
__device__ __forceinline__ float block_sum(float v, float* s_red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}
__device__ __forceinline__ float block_max(float v, float* s_red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
}

// One workgroup per row: logits z -> the row's loss and, in place, the gradient with respect to
// the logits: ((sum_b T) * softmax(z) - T) / R.
// PER > 0: rows of at most 256 PER buckets, read once, all loads in flight together (8 x 1000 rows of 1024: 29 us with three
// passes over a row, and 8 us less in a training iteration now; its 98 MB take 21 at the rate of a copy).  PER = 0: rows of any
// length, three passes.
template <int PER>
__global__ void __launch_bounds__(256)
softmax_kl_kernel(float* __restrict__ z, const float* __restrict__ T, float* __restrict__ loss_rows, int R, int B) {
  __shared__ float s_red[4];
  const size_t row = (size_t)blockIdx.y * R + blockIdx.x;
  float* zr = z + row * B;
  const float* tr = T + row * B;
  float zv[PER > 0 ? PER : 1], tv[PER > 0 ? PER : 1];
  if constexpr (PER > 0) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int b = min((int)threadIdx.x + 256 * i, B - 1);
      zv[i] = zr[b];
      tv[i] = tr[b];
    }
  }
  // f(b, z, t) for the thread's buckets, in ascending order
  auto each = [&](auto f) {
    if constexpr (PER > 0) {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int b = threadIdx.x + 256 * i;
        if (b < B) f(b, zv[i], tv[i]);
      }
    } else {
      for (int b = threadIdx.x; b < B; b += 256) f(b, zr[b], tr[b]);
    }
  };
  float mx = -INFINITY, tsum = 0.f;
  each([&](int, float zb, float t) {
    mx = fmaxf(mx, zb);
    tsum += t;
  });
  mx = block_max(mx, s_red);
  tsum = block_sum(tsum, s_red);
  float se = 0.f;
  each([&](int, float zb, float) { se += __expf(zb - mx); });
  se = block_sum(se, s_red);
  const float lse = mx + __logf(se), inv_r = 1.0f / (float)R;
  float l = 0.f;
  each([&](int b, float zb, float t) {
    const float logp = zb - lse;
    if (t > 0.f) l += t * (__logf(t) - logp);
    zr[b] = (tsum * __expf(logp) - t) * inv_r;
  });
  l = block_sum(l, s_red);
  if (threadIdx.x == 0) loss_rows[row] = l;
}

// loss[w] = mean over the R rows, summed in a fixed order by one workgroup
__global__ void __launch_bounds__(256)
loss_mean_kernel(const float* __restrict__ loss_rows, float* __restrict__ loss, int R) {
  __shared__ float s_red[4];
  float v = 0.f;
  for (int r = threadIdx.x; r < R; r += 256) v += loss_rows[(size_t)blockIdx.x * R + r];
  v = block_sum(v, s_red);
  if (threadIdx.x == 0) loss[blockIdx.x] = v / (float)R;
}

// Column sums in a fixed order.  A workgroup owns 64 columns; its 16 waves each take a contiguous slice of
// the rows (a wave reads 64 neighbouring columns of one row at a time) and the 16 slice sums are added in
// slice order, so the result does not depend on timing.
constexpr int kBnCols = 64, kBnSlices = 16, kBnThreads = kBnCols * kBnSlices;

// sum over the slices of v, in slice order; every thread of a column gets the same bits
__device__ __forceinline__ float slice_sum(float v, float (*s_part)[kBnCols], int col, int slice) {
  __syncthreads();
  s_part[slice][col] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < kBnSlices; ++i) t += s_part[i][col];
  return t;
}

// Batch normalisation of the hidden pre-activations a [rows, n_cols] (Section 6.1 names the layer).
// Columns and rows are dealt as above.  The batch mean, then the variance about it (divisor rows).
// stats [4, n_cols] per weight set: mean, 1/sqrt(var + eps), and room for the two backward sums.
// Running statistics (optional) follow run = (1 - momentum) run + momentum batch, the variance with
// divisor rows - 1.
__global__ void __launch_bounds__(kBnThreads)
bn_stats_kernel(const float* __restrict__ A, float* __restrict__ stats, float* __restrict__ run_mean,
                float* __restrict__ run_var, int rows, int n_cols, float eps, float momentum) {
  __shared__ float s_part[kBnSlices][kBnCols];
  const int col = threadIdx.x % kBnCols, slice = threadIdx.x / kBnCols;
  const int c = blockIdx.x * kBnCols + col;
  const bool live = c < n_cols;
  const int per = (rows + kBnSlices - 1) / kBnSlices, r0 = slice * per, r1 = min(r0 + per, rows);
  const float* a = A + (size_t)blockIdx.y * rows * n_cols + (live ? c : 0);
  float sum = 0.f;
  if (live)
    for (int r = r0; r < r1; ++r) sum += a[(size_t)r * n_cols];
  const float mean = slice_sum(sum, s_part, col, slice) / (float)rows;
  float sq = 0.f;
  if (live)
    for (int r = r0; r < r1; ++r) {
      const float dlt = a[(size_t)r * n_cols] - mean;
      sq += dlt * dlt;
    }
  sq = slice_sum(sq, s_part, col, slice);
  if (!live || slice != 0) return;
  float* st = stats + (size_t)blockIdx.y * 4 * n_cols;
  st[c] = mean;
  st[n_cols + c] = 1.0f / sqrtf(sq / (float)rows + eps);
  if (run_mean) {
    const size_t i = (size_t)blockIdx.y * n_cols + c;
    run_mean[i] = (1.0f - momentum) * run_mean[i] + momentum * mean;
    run_var[i] = (1.0f - momentum) * run_var[i] + momentum * (sq / (float)(rows - 1));
  }
}

// h = relu(gamma * ahat + beta), ahat = (a - mean) * rstd
__global__ void __launch_bounds__(256)
bn_relu_kernel(const float* __restrict__ A, const float* __restrict__ stats, const float* __restrict__ gamma,
               const float* __restrict__ beta, float* __restrict__ H, int rows, int n_cols) {
  const size_t per_set = (size_t)rows * n_cols;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= per_set) return;
  const int c = (int)(i % n_cols), w = blockIdx.y;
  const float* st = stats + (size_t)w * 4 * n_cols;
  const float ahat = (A[w * per_set + i] - st[c]) * st[n_cols + c];
  H[w * per_set + i] = fmaxf(gamma[(size_t)w * n_cols + c] * ahat + beta[(size_t)w * n_cols + c], 0.f);
}

// Backward sums per column, rows sliced as in bn_stats_kernel: dbeta = sum dy, dgamma = sum dy * ahat.
__global__ void __launch_bounds__(kBnThreads)
bn_backward_sums_kernel(const float* __restrict__ A, const float* __restrict__ DY, float* __restrict__ stats,
                        float* __restrict__ dgamma, float* __restrict__ dbeta, int rows, int n_cols) {
  __shared__ float s_part[kBnSlices][kBnCols];
  const int col = threadIdx.x % kBnCols, slice = threadIdx.x / kBnCols;
  const int c = blockIdx.x * kBnCols + col;
  const bool live = c < n_cols;
  const int per = (rows + kBnSlices - 1) / kBnSlices, r0 = slice * per, r1 = min(r0 + per, rows);
  const size_t base = (size_t)blockIdx.y * rows * n_cols + (live ? c : 0);
  float* st = stats + (size_t)blockIdx.y * 4 * n_cols;
  const float mean = live ? st[c] : 0.f, rstd = live ? st[n_cols + c] : 0.f;
  float sb = 0.f, sg = 0.f;
  if (live)
    for (int r = r0; r < r1; ++r) {
      const float dy = DY[base + (size_t)r * n_cols];
      sb += dy;
      sg += dy * ((A[base + (size_t)r * n_cols] - mean) * rstd);
    }
  sb = slice_sum(sb, s_part, col, slice);
  sg = slice_sum(sg, s_part, col, slice);
  if (!live || slice != 0) return;
  st[2 * n_cols + c] = sb;
  st[3 * n_cols + c] = sg;
  dbeta[(size_t)blockIdx.y * n_cols + c] = sb;
  dgamma[(size_t)blockIdx.y * n_cols + c] = sg;
}

// In place: dy -> da = gamma * rstd * (dy - dbeta / rows - ahat * dgamma / rows)
__global__ void __launch_bounds__(256)
bn_backward_kernel(const float* __restrict__ A, float* __restrict__ DY, const float* __restrict__ stats,
                   const float* __restrict__ gamma, int rows, int n_cols) {
  const size_t per_set = (size_t)rows * n_cols;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= per_set) return;
  const int c = (int)(i % n_cols), w = blockIdx.y;
  const float* st = stats + (size_t)w * 4 * n_cols;
  const float rstd = st[n_cols + c], inv_rows = 1.0f / (float)rows;
  const float ahat = (A[w * per_set + i] - st[c]) * rstd;
  const float dy = DY[w * per_set + i];
  DY[w * per_set + i] = gamma[(size_t)w * n_cols + c] * rstd * (dy - st[2 * n_cols + c] * inv_rows - ahat * st[3 * n_cols + c] * inv_rows);
}

// W1' = s W1 (row-wise), b1' = (b1 - mean) s + beta with s = gamma / sqrt(var + eps); one thread per row of W1
template <typename TO>
__global__ void __launch_bounds__(256)
bn_fold_kernel(const float* __restrict__ W1, const float* __restrict__ b1, const float* __restrict__ gamma,
               const float* __restrict__ beta, const float* __restrict__ mean, const float* __restrict__ var, float eps,
               TO* __restrict__ W1o, float* __restrict__ b1o, size_t rows_total, int d) {
  const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= rows_total) return;
  const float s = gamma[j] / sqrtf(var[j] + eps);
  b1o[j] = (b1[j] - mean[j]) * s + beta[j];
  for (int k = 0; k < d; ++k) {
    const float v = W1[j * d + k] * s;
    if constexpr (sizeof(TO) == 4) {
      W1o[j * d + k] = v;
    } else {
      W1o[j * d + k] = Vec8<bf16_t>::narrow(v);
    }
  }
}

__global__ void __launch_bounds__(256)
adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v, size_t n,
            float lr, float beta1, float beta2, float eps, float c1, float c2) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
  const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

}  // namespace

// header | h [Hw,R,hidden] | z then dL/dz [Hw,R,B] | dL/da [Hw,R,hidden] | row losses [Hw,R]
//        | batch-norm variant: pre-activations a [Hw,R,hidden] | column statistics [Hw,4,hidden] | [Hw,R,d], not used: the size is part
//        of the interface
size_t train_workspace_bytes(long long Hw, long long R, int d, int hidden, int B) {
  return (size_t)SAAP_WS_HEADER_BYTES + (size_t)Hw * R * ((size_t)d + 3 * (size_t)hidden + B + 1) * sizeof(float) +
         (size_t)Hw * 4 * hidden * sizeof(float);
}

}  // namespace saap

using namespace saap;

// bn == nullptr: the plain model.
static int32_t loss_grads(const void* x, const float* target, const saap_mlp_f32* params, const saap_mlp_f32* grads,
                          const saap_batch_norm_f32* bn, float* loss, int32_t Hw, int32_t R, int32_t d, int32_t hidden,
                          int32_t B, int32_t x_dtype, void* ws, size_t ws_bytes, void* stream) {
  if (!x || !target || !params || !grads || !loss || !ws) return SAAP_INVALID_ARG;
  if (bn) {
    if (!bn->gamma || !bn->beta || !bn->grad_gamma || !bn->grad_beta) return SAAP_INVALID_ARG;
    if ((bn->running_mean == nullptr) != (bn->running_var == nullptr)) return SAAP_INVALID_ARG;
    if (!(bn->eps > 0.f) || !(bn->momentum >= 0.f && bn->momentum <= 1.f)) return SAAP_INVALID_ARG;
    if (R < 2) return SAAP_INVALID_ARG;   // no variance estimate from one row
  }
  if (!params->W1 || !params->b1 || !params->W2 || !params->b2 || !grads->W1 || !grads->b1 || !grads->W2 || !grads->b2)
    return SAAP_INVALID_ARG;
  if (!aligned16(x) || !aligned16(ws)) return SAAP_INVALID_ARG;
  if (Hw <= 0 || R <= 0 || d <= 0 || hidden <= 0 || B <= 0) return SAAP_INVALID_ARG;
  if (x_dtype != SAAP_F32 && x_dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (Hw > 65535 || R > 65535 * 64) return SAAP_UNSUPPORTED;
  if (ws_bytes < train_workspace_bytes(Hw, R, d, hidden, B)) return SAAP_WORKSPACE_TOO_SMALL;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  float* h = reinterpret_cast<float*>(static_cast<char*>(ws) + SAAP_WS_HEADER_BYTES);
  float* z = h + (size_t)Hw * R * hidden;
  float* da = z + (size_t)Hw * R * B;
  float* loss_rows = da + (size_t)Hw * R * hidden;
  const bool narrow = x_dtype == SAAP_BF16;
  const long long sx = (long long)R * d, sh = (long long)R * hidden, sz = (long long)R * B;
  const long long sW1 = (long long)hidden * d, sW2 = (long long)B * hidden;
  float* pre = loss_rows + (size_t)Hw * R;          // batch-norm variant only
  float* stats = pre + (size_t)Hw * R * hidden;
  const dim3 per_col((unsigned)((hidden + kBnCols - 1) / kBnCols), (unsigned)Hw);
  const dim3 per_elem((unsigned)(((size_t)R * hidden + 255) / 256), (unsigned)Hw);
  if (!bn) {
    // h = relu(x W1^T + b1)
    const GemmArgs g = {x, params->W1, h, params->b1, nullptr, R, hidden, d, sx, sW1, sh, hidden, 0, nullptr, 0, 0, 0};
    narrow ? gemm<false, true, EPI_BIAS_RELU, true, bf16_t>(g, Hw, hs) : gemm<false, true, EPI_BIAS_RELU, true>(g, Hw, hs);
  } else {
    // a = x W1^T + b1;  h = relu(gamma * normalised(a) + beta)
    const GemmArgs g = {x, params->W1, pre, params->b1, nullptr, R, hidden, d, sx, sW1, sh, hidden, 0, nullptr, 0, 0, 0};
    narrow ? gemm<false, true, EPI_BIAS, true, bf16_t>(g, Hw, hs) : gemm<false, true, EPI_BIAS, true>(g, Hw, hs);
    hipLaunchKernelGGL(bn_stats_kernel, per_col, dim3(kBnThreads), 0, hs, pre, stats, bn->running_mean, bn->running_var, R, hidden,
                       bn->eps, bn->momentum);
    hipLaunchKernelGGL(bn_relu_kernel, per_elem, dim3(256), 0, hs, pre, stats, bn->gamma, bn->beta, h, R, hidden);
  }
  // z = h W2^T + b2
  gemm<false, true, EPI_BIAS>({h, params->W2, z, params->b2, nullptr, R, B, hidden, sh, sW2, sz, B, 0, nullptr, 0, 0, 0}, Hw, hs);
  // row losses; z becomes dL/dz
  auto softmax_kl = B <= 1024 ? softmax_kl_kernel<4> : B <= 2048 ? softmax_kl_kernel<8> : softmax_kl_kernel<0>;
  hipLaunchKernelGGL(softmax_kl, dim3((unsigned)R, (unsigned)Hw), dim3(256), 0, hs, z, target, loss_rows, R, B);
  hipLaunchKernelGGL(loss_mean_kernel, dim3((unsigned)Hw), dim3(256), 0, hs, loss_rows, loss, R);
  // dW2 = dz^T h, db2 = column sums of dz
  gemm<true, false, EPI_NONE>({z, h, grads->W2, nullptr, nullptr, B, hidden, R, sz, sh, sW2, 0, 0, grads->b2, B, 0, 0}, Hw, hs);
  // da = (dz W2) where h > 0
  gemm<false, false, EPI_MASK>({z, params->W2, da, nullptr, h, R, hidden, B, sz, sW2, sh, 0, sh, nullptr, 0, 0, 0}, Hw, hs);
  if (bn) {
    // through the normalisation: da holds dL/dy on entry and dL/da on exit
    hipLaunchKernelGGL(bn_backward_sums_kernel, per_col, dim3(kBnThreads), 0, hs, pre, da, stats, bn->grad_gamma, bn->grad_beta, R,
                       hidden);
    hipLaunchKernelGGL(bn_backward_kernel, per_elem, dim3(256), 0, hs, pre, da, stats, bn->gamma, R, hidden);
  }
  // dW1 = da^T x, db1 = column sums of da
  const GemmArgs g = {da, x, grads->W1, nullptr, nullptr, hidden, d, R, sh, sx, sW1, 0, 0, grads->b1, hidden, 0, 0};
  narrow ? gemm<true, false, EPI_NONE, false, float, bf16_t>(g, Hw, hs) : gemm<true, false, EPI_NONE>(g, Hw, hs);
  return launch_status();
}

extern "C" int32_t saap_query_model_loss_grads(const void* x, const float* target, const saap_mlp_f32* params,
                                               const saap_mlp_f32* grads, float* loss, int32_t Hw, int32_t R,
                                               int32_t d, int32_t hidden, int32_t B, int32_t x_dtype, void* ws,
                                               size_t ws_bytes, void* stream) {
  const Call call(stream);
  return loss_grads(x, target, params, grads, nullptr, loss, Hw, R, d, hidden, B, x_dtype, ws, ws_bytes, stream);
}

extern "C" int32_t saap_query_model_bn_loss_grads(const void* x, const float* target, const saap_mlp_f32* params,
                                                  const saap_mlp_f32* grads, const saap_batch_norm_f32* bn, float* loss,
                                                  int32_t Hw, int32_t R, int32_t d, int32_t hidden, int32_t B,
                                                  int32_t x_dtype, void* ws, size_t ws_bytes, void* stream) {
  const Call call(stream);
  if (!bn) return SAAP_INVALID_ARG;
  return loss_grads(x, target, params, grads, bn, loss, Hw, R, d, hidden, B, x_dtype, ws, ws_bytes, stream);
}

extern "C" int32_t saap_fold_batch_norm(const float* W1, const float* b1, const float* gamma, const float* beta,
                                        const float* running_mean, const float* running_var, float eps, void* W1_out,
                                        float* b1_out, int32_t Hw, int32_t hidden, int32_t d, int32_t out_dtype,
                                        void* stream) {
  const Call call(stream);
  if (!W1 || !b1 || !gamma || !beta || !running_mean || !running_var || !W1_out || !b1_out) return SAAP_INVALID_ARG;
  if (Hw <= 0 || hidden <= 0 || d <= 0 || !(eps > 0.f)) return SAAP_INVALID_ARG;
  if (out_dtype != SAAP_F32 && out_dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  const size_t rows = (size_t)Hw * hidden;
  const dim3 grid((unsigned)((rows + 255) / 256));
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (out_dtype == SAAP_F32)
    hipLaunchKernelGGL(bn_fold_kernel<float>, grid, dim3(256), 0, hs, W1, b1, gamma, beta, running_mean, running_var, eps,
                       static_cast<float*>(W1_out), b1_out, rows, d);
  else
    hipLaunchKernelGGL(bn_fold_kernel<bf16_t>, grid, dim3(256), 0, hs, W1, b1, gamma, beta, running_mean, running_var, eps,
                       static_cast<bf16_t*>(W1_out), b1_out, rows, d);
  return launch_status();
}

extern "C" int32_t saap_adam_update(float* param, const float* grad, float* m, float* v, size_t n, int32_t step,
                                    float lr, float beta1, float beta2, float eps, void* stream) {
  const Call call(stream);
  if (!param || !grad || !m || !v) return SAAP_INVALID_ARG;
  if (n == 0 || step < 1 || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f)) return SAAP_INVALID_ARG;
  // bias corrections 1 / (1 - beta^t), evaluated in double on the host
  const float c1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
  const float c2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream), param,
                     grad, m, v, n, lr, beta1, beta2, eps, c1, c2);
  return launch_status();
}
