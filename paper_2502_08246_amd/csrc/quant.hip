// quantize_kv: 8-bit storage of a bucket-sorted K/V cache.  The paper names compression of the
// cached vectors as complementary to the partition (Section 2, related work on vector
// compression) without fixing a format; this build uses OCP FP8 E4M3 (bias 7, largest finite
// value 448) with one power-of-two scale per (sequence, KV head) and tensor, which halves the
// bytes the decode attention reads per key.
//   scale = 2^e, e the smallest integer with max|x| <= 448 * 2^e (1 for an all-zero unit)
//   code  = round-to-nearest-even of x / scale (the chip's v_cvt_pk_fp8_f32)
// Two launches for K and V together: per-unit maxima (atomic max on the bit pattern, which orders non-negative floats, one per
// workgroup), and the conversion, whose last workgroup of a unit clears its maximum again (a third launch with more than 512 units).
#include <algorithm>

#include "common.h"

namespace saap {
namespace {

constexpr int kQThreads = 256;
constexpr int kQSlices = 64;      // workgroups per (tensor, unit) in both passes (gridDim.x): fewer of short units, more of a few long ones
constexpr int kQUnroll = 4;       // 16-byte (bf16) loads a thread has in flight

template <typename T>
__global__ void __launch_bounds__(kQThreads)
absmax_kernel(const T* __restrict__ K, const T* __restrict__ V, unsigned* __restrict__ amax_bits, size_t pieces,
              int units, int stride) {
  __shared__ float s_m[kQThreads / 64];
  const int unit = blockIdx.y, tensor = blockIdx.z;
  const T* x = (tensor ? V : K) + (size_t)unit * pieces * 8;
  float m = 0.f;
  // four loads in flight per thread (a piece past the end reads the last one again: the maximum does not change)
  const size_t step = (size_t)gridDim.x * kQThreads;
  for (size_t i = (size_t)blockIdx.x * kQThreads + threadIdx.x; i < pieces; i += kQUnroll * step) {
    Vec8<T> v[kQUnroll];
#pragma unroll
    for (int u = 0; u < kQUnroll; ++u) v[u].load_stream(x + min(i + u * step, pieces - 1) * 8);
#pragma unroll
    for (int u = 0; u < kQUnroll; ++u) {
      float f[8];
      v[u].to_float(f);
#pragma unroll
      for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(f[e]));
    }
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
  __syncthreads();
  // A line of its own for every unit, where there is room, and one update per workgroup: updates of a line wait for each other
  // (2 units of 2466 rows: 14.0 us with one per wave in neighbouring words, 3.4 now; 8 of 6027: 51, 6.5).
  if (threadIdx.x == 0)
    atomicMax(&amax_bits[(size_t)(tensor * units + unit) * stride], __float_as_uint(fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]))));
}

// 2^e with the smallest e such that amax <= 448 * 2^e; 448 = 0.875 * 2^9
__device__ __forceinline__ int unit_exponent(float amax) {
  int ex;
  const float f = frexpf(amax, &ex);
  const int e = f <= 0.875f ? ex - 9 : ex - 8;
  return min(max(e, -100), 100);
}

template <typename T>
__global__ void __launch_bounds__(kQThreads)
quantize_kernel(const T* __restrict__ K, const T* __restrict__ V, uint8_t* __restrict__ K8, uint8_t* __restrict__ V8,
                unsigned* __restrict__ amax_bits, float* __restrict__ kscale, float* __restrict__ vscale,
                size_t pieces, int units, int stride) {
  const int unit = blockIdx.y, tensor = blockIdx.z;
  const T* x = (tensor ? V : K) + (size_t)unit * pieces * 8;
  uint2* y = reinterpret_cast<uint2*>((tensor ? V8 : K8) + (size_t)unit * pieces * 8);
  unsigned* const word = amax_bits + (size_t)(tensor * units + unit) * stride;       // the maximum, and workgroups that have read it
  __shared__ float s_amax;
  const size_t step = (size_t)gridDim.x * kQThreads, first = (size_t)blockIdx.x * kQThreads + threadIdx.x;
  Vec8<T> v[kQUnroll];
  auto load = [&](size_t i) {
#pragma unroll
    for (int u = 0; u < kQUnroll; ++u) v[u].load_stream(x + min(i + u * step, pieces - 1) * 8);
  };
  // One thread reads the maximum, for all of them, while the first rows are on their way, and counts the workgroup; the answer is not
  // waited for until the rows are done.  The last workgroup of the unit to have read it clears it for the next call (a launch that
  // clears takes 4 us).
  if (threadIdx.x == 0) s_amax = __uint_as_float(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  load(first);
  __syncthreads();
  const float amax = s_amax;
  unsigned before = 0u;
  if (stride > 1 && threadIdx.x == 0) before = __hip_atomic_fetch_add(word + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int e = amax > 0.f ? unit_exponent(amax) : 0;
  const float inv = ldexpf(1.f, -e);
  if (blockIdx.x == 0 && threadIdx.x == 0) (tensor ? vscale : kscale)[unit] = ldexpf(1.f, e);
  for (size_t i = first; i < pieces; i += kQUnroll * step) {
    if (i != first) load(i);
#pragma unroll
    for (int u = 0; u < kQUnroll; ++u) {
      float f[8];
      v[u].to_float(f);
      int lo = 0, hi = 0;
      lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[0] * inv, f[1] * inv, lo, false);
      lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[2] * inv, f[3] * inv, lo, true);
      hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[4] * inv, f[5] * inv, hi, false);
      hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[6] * inv, f[7] * inv, hi, true);
      if (i + u * step < pieces) y[i + u * step] = make_uint2((unsigned)lo, (unsigned)hi);
    }
  }
  if (stride > 1 && threadIdx.x == 0 && before == gridDim.x - 1) {
    __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(word + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__global__ void clear_words_kernel(unsigned* w, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = 0u;
}

}  // namespace
}  // namespace saap

using namespace saap;

extern "C" int32_t saap_quantize_kv(const void* Ksorted, const void* Vsorted, uint8_t* K8, uint8_t* V8, float* kscale,
                                    float* vscale, int32_t S, int32_t Hkv, int32_t Ncap, int32_t d, int32_t dtype,
                                    void* ws, size_t ws_bytes, void* stream) {
  const Call call(stream);
  if (!Ksorted || !Vsorted || !K8 || !V8 || !kscale || !vscale || !ws) return SAAP_INVALID_ARG;
  if (!aligned16(Ksorted) || !aligned16(Vsorted) || !aligned16(K8) || !aligned16(V8) || !aligned16(ws))
    return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || Ncap <= 0) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD) return SAAP_UNSUPPORTED;
  const long long units = (long long)S * Hkv;
  if (units > 65535 || 2 * units * sizeof(unsigned) > SAAP_WS_HEADER_BYTES) return SAAP_UNSUPPORTED;
  if (ws_bytes < SAAP_WS_HEADER_BYTES) return SAAP_WORKSPACE_TOO_SMALL;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  unsigned* amax_bits = reinterpret_cast<unsigned*>(ws);   // header words, zero on entry and on exit
  // Words between the maxima of two units: a line of 64 bytes (the maximum and the count of its readers); with more units than there are
  // lines the maxima alone, cleared by a launch of 4 us.  (Counts that share lines wait for each other: 1000 units of 1500 rows 1149 us,
  // 365 without; 336 with fewer workgroups as well.)
  const int stride = 2 * units * 64 <= (long long)SAAP_WS_HEADER_BYTES ? 16 : 1;
  const size_t pieces = (size_t)Ncap * kD / 8;
  // Up to three workgroups per compute unit where a few units have five rounds of rows for them: one head of 139264 rows 69 us with 64
  // workgroups to a tensor, 33 with 384, 43 with 512; of 34756 rows 13.0 with 64, 11.2 with 128, 21.7 with 512, whose updates of the
  // unit's line wait for each other.
  const long long filling = 3LL * device_cus() / (2 * units), with_work = (long long)(pieces / (5 * kQThreads * kQUnroll));
  // No more than have rows: a workgroup without any would read the maximum and count itself for nothing (2048 units of 54 rows: 1669 us
  // with 64 each, 26 with two).  Many units have workgroups enough with all of their loads used.
  const long long per_wg = stride > 1 ? kQThreads : kQThreads * kQUnroll, most = ((long long)pieces + per_wg - 1) / per_wg;
  const dim3 grid((unsigned)std::min(most, std::max<long long>(kQSlices, std::min(filling, with_work))), (unsigned)units, 2);
  if (dtype == SAAP_BF16) {
    hipLaunchKernelGGL(absmax_kernel<bf16_t>, grid, dim3(kQThreads), 0, hs, static_cast<const bf16_t*>(Ksorted),
                       static_cast<const bf16_t*>(Vsorted), amax_bits, pieces, (int)units, stride);
    hipLaunchKernelGGL(quantize_kernel<bf16_t>, grid, dim3(kQThreads), 0, hs, static_cast<const bf16_t*>(Ksorted),
                       static_cast<const bf16_t*>(Vsorted), K8, V8, amax_bits, kscale, vscale, pieces, (int)units, stride);
  } else {
    hipLaunchKernelGGL(absmax_kernel<float>, grid, dim3(kQThreads), 0, hs, static_cast<const float*>(Ksorted),
                       static_cast<const float*>(Vsorted), amax_bits, pieces, (int)units, stride);
    hipLaunchKernelGGL(quantize_kernel<float>, grid, dim3(kQThreads), 0, hs, static_cast<const float*>(Ksorted),
                       static_cast<const float*>(Vsorted), K8, V8, amax_bits, kscale, vscale, pieces, (int)units, stride);
  }
  if (stride == 1)
    hipLaunchKernelGGL(clear_words_kernel, dim3((unsigned)((2 * units + 255) / 256)), dim3(256), 0, hs, amax_bits,
                     (int)(2 * units));
  return launch_status();
}
