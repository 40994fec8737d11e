// update_centroids: the centroid step of the k-means that defines the buckets of arXiv 2502.08246
// (Section 4, "Learning the key assignment": k-means on keys; Section 3 uses the spherical
// variant; Appendix A gives the training set-up).  With saap_assign_keys (assignment step) and
// saap_build_bucket_index (grouping the features by bucket) it makes one Lloyd iteration on the
// GPU, so that centroids for any head can be produced without leaving the device.
//
// One workgroup per (KV head, bucket).  The bucket's member rows are one contiguous run per
// sequence of the grouped features; 16 lanes read one row (16 or 32 bytes each), 16 rows are in
// flight per pass, every lane adds up its 8 features over its rows in fp32 in a fixed order, the
// 16 row groups are then added in order through LDS.  Sums are therefore reproducible from run to run.
#include "common.h"

namespace saap {
namespace {

// idx: null (x grouped by bucket) or [S,Hkv,Ncap], the row of each slot.
// DEEP rows of a 16-lane group in flight: four where a bucket is a round or two of them (eight workgroups per compute unit: 8 heads of
// 65536 keys, 1024 buckets, 27 us; 30 with eight), eight for longer ones, whose places are then looked up a round ahead (4 heads
// of 120000 keys, 512 buckets: 52 us with four and a look-up and the rows' loads one after the other, 36 now;
// 8 of 4736, 16 buckets: 13.5, 9.0; 8 of 65536, 656 buckets: 27.7, 25.4).
template <typename T, bool GATHER, int DEEP>
__global__ void __launch_bounds__(256, DEEP > 4 ? 4 : 8)
centroid_update_kernel(const T* __restrict__ x, const int32_t* __restrict__ idx, const int32_t* __restrict__ off, const int32_t* __restrict__ len,
                       const T* __restrict__ cent_old, T* __restrict__ cent_new, int S, int Hkv, int Ncap, int B,
                       int normalize) {
  __shared__ float s_part[16][kD];
  __shared__ float s_sq[2];
  const int b = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = tid & 15, grp = tid >> 4;            // 16 lanes per row, 16 row groups
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  long long count = 0;
  for (int s = 0; s < S; ++s) {
    const size_t unit = (size_t)s * Hkv + h;
    const int first = off[unit * (B + 1) + b], n = len[unit * B + b];
    count += n;
    const T* rows = x + (GATHER ? unit * Ncap : unit * Ncap + first) * kD + sub * 8;
    const int32_t* ix = GATHER ? idx + unit * Ncap + first : nullptr;
    int at[DEEP];
    auto look_up = [&](int r) {
#pragma unroll
      for (int u = 0; u < DEEP; ++u) {
        at[u] = min(r + 16 * u, n - 1);
        if constexpr (GATHER) at[u] = ix[at[u]];
      }
    };
    if (DEEP > 4 && n > 0) look_up(grp);
    for (int r = grp; r < n; r += 16 * DEEP) {
      if (DEEP == 4) look_up(r);
      Vec8<T> v[DEEP];
#pragma unroll
      for (int u = 0; u < DEEP; ++u) v[u].load(rows + (size_t)at[u] * kD);
      if (DEEP > 4) look_up(r + 16 * DEEP);
#pragma unroll
      for (int u = 0; u < DEEP; ++u) {
        float f[8];
        v[u].to_float(f);
        const bool in = r + 16 * u < n;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += in ? f[e] : 0.f;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) s_part[grp][sub * 8 + e] = acc[e];
  __syncthreads();
  const size_t crow = ((size_t)h * B + b) * kD;
  float mean = 0.f;
  if (tid < kD) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) t += s_part[g][tid];
    mean = count > 0 ? t / (float)count : 0.f;
    // squared norm of the mean: 64 lanes on DPP and row swaps, then the two waves in order
    const float sq = sum_rows(sum16(mean * mean));
    if (lane == 0) s_sq[wave] = sq;
  }
  __syncthreads();
  if (tid < kD) {
    float v;
    if (count == 0) {
      v = Vec8<T>::widen(cent_old[crow + tid]);         // a bucket without members keeps its centroid
    } else {
      v = mean;
      if (normalize) {
        const float nrm = sqrtf(s_sq[0] + s_sq[1]);
        v = nrm > 0.f ? mean / nrm : mean;
      }
    }
    cent_new[crow + tid] = Vec8<T>::narrow(v);
  }
}

template <typename T, bool GATHER>
void launch_update(const void* x, const int32_t* idx, const int32_t* off, const int32_t* len, const void* cent_old, void* cent_new,
                   int S, int Hkv, int Ncap, int B, int normalize, hipStream_t hs) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)B, (unsigned)Hkv), dim3(256), 0, hs, static_cast<const T*>(x), idx, off, len,
                       static_cast<const T*>(cent_old), static_cast<T*>(cent_new), S, Hkv, Ncap, B, normalize);
  };
  if (sizeof(T) == 2 && Ncap >= 96ll * B) launch(centroid_update_kernel<T, GATHER, sizeof(T) == 2 ? 8 : 4>);
  else launch(centroid_update_kernel<T, GATHER, 4>);
}

size_t align16(size_t n) { return (n + 15) & ~(size_t)15; }

}  // namespace

// header | the slices' counters of the sort | off [units,B+1] | len [units,B] | idx [units,N]
size_t update_from_ids_workspace_bytes(long long units, int N, int B) {
  return align16(build_workspace_bytes(units, N, B)) + align16((size_t)units * (B + 1) * 4) + align16((size_t)units * B * 4) +
         (size_t)units * N * 4;
}

}  // namespace saap

using namespace saap;

static int32_t check_update(const void* x, const void* cent_old, const void* cent_new, int32_t S, int32_t Hkv, int32_t N, int32_t B,
                            int32_t d, int32_t dtype) {
  if (!x || !cent_old || !cent_new) return SAAP_INVALID_ARG;
  if (!aligned16(x) || !aligned16(cent_old) || !aligned16(cent_new)) return SAAP_INVALID_ARG;
  if (S <= 0 || Hkv <= 0 || N <= 0 || B <= 0) return SAAP_INVALID_ARG;
  if (dtype != SAAP_F32 && dtype != SAAP_BF16) return SAAP_INVALID_ARG;
  if (d != kD || B > SAAP_MAX_BUCKETS || Hkv > 65535) return SAAP_UNSUPPORTED;
  return SAAP_OK;
}

extern "C" int32_t saap_update_centroids(const void* x_sorted, const int32_t* off, const int32_t* len,
                                         const void* centroids_old, void* centroids_new, int32_t S, int32_t Hkv,
                                         int32_t Ncap, int32_t B, int32_t d, int32_t dtype, int32_t normalize,
                                         void* stream) {
  const Call call(stream);
  if (!off || !len) return SAAP_INVALID_ARG;
  const int32_t st = check_update(x_sorted, centroids_old, centroids_new, S, Hkv, Ncap, B, d, dtype);
  if (st != SAAP_OK) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (dtype == SAAP_BF16)
    launch_update<bf16_t, false>(x_sorted, nullptr, off, len, centroids_old, centroids_new, S, Hkv, Ncap, B, normalize, hs);
  else
    launch_update<float, false>(x_sorted, nullptr, off, len, centroids_old, centroids_new, S, Hkv, Ncap, B, normalize, hs);
  return launch_status();
}

extern "C" int32_t saap_update_centroids_from_ids(const void* x, const int32_t* bucket_ids, const void* centroids_old,
                                                  void* centroids_new, int32_t S, int32_t Hkv, int32_t N, int32_t B,
                                                  int32_t d, int32_t dtype, int32_t normalize, void* ws, size_t ws_bytes,
                                                  void* stream) {
  const Call call(stream);
  if (!bucket_ids || !ws || !aligned16(ws)) return SAAP_INVALID_ARG;
  const int32_t st = check_update(x, centroids_old, centroids_new, S, Hkv, N, B, d, dtype);
  if (st != SAAP_OK) return st;
  const long long units = (long long)S * Hkv;
  if (units > 65535) return SAAP_UNSUPPORTED;
  if (ws_bytes < update_from_ids_workspace_bytes(units, N, B)) return SAAP_WORKSPACE_TOO_SMALL;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  char* p = static_cast<char*>(ws);
  int32_t* slice_hist = reinterpret_cast<int32_t*>(p + SAAP_WS_HEADER_BYTES);
  p += align16(build_workspace_bytes(units, N, B));
  int32_t* off = reinterpret_cast<int32_t*>(p);
  p += align16((size_t)units * (B + 1) * 4);
  int32_t* len = reinterpret_cast<int32_t*>(p);
  p += align16((size_t)units * B * 4);
  int32_t* idx = reinterpret_cast<int32_t*>(p);
  order_keys(bucket_ids, off, len, idx, nullptr, slice_hist, units, N, N, B, 0, -1, 0, 0, hs);
  if (dtype == SAAP_BF16)
    launch_update<bf16_t, true>(x, idx, off, len, centroids_old, centroids_new, S, Hkv, N, B, normalize, hs);
  else
    launch_update<float, true>(x, idx, off, len, centroids_old, centroids_new, S, Hkv, N, B, normalize, hs);
  return launch_status();
}
