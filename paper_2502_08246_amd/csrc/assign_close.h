// What the fp32 scores of a key say about its bucket (assign_f32_kernel).  Plain arithmetic, for the host as well.
#pragma once
#include <cmath>

#ifdef __HIPCC__
#define SAAP_EVERYWHERE __host__ __device__ inline
#else
#define SAAP_EVERYWHERE inline
#endif

namespace saap {

struct KeyScores {
  bool odd;      // nothing is known: to be scored against every centroid
  bool close;    // the best is not known: the centroids that score `limit` at least may be it
  float limit;
  // A flag decides which keys take part, no value of the limit does: a score may be +infinity.  The lanes behind the last key hold a
  // copy of it, and what they listed would be read behind the last row.
  SAAP_EVERYWHERE bool lists(float score) const { return close && score >= limit; }
};

// best, second: of the key's scores; nan: a score that is no number; xmax, xn2: of the key's features, the largest magnitude and the sum
// of squares; norm2: the largest of the centroids'; in_range: there is such a key.
SAAP_EVERYWHERE KeyScores decide_key(float best, float second, bool nan, float xmax, float xn2, float norm2, float tol, bool in_range) {
  // both scores' errors (tol), the additions of their biases, products below the smallest fp32 number
  const float thr = tol * sqrtf(norm2) * sqrtf(xn2) + 5e-7f * fabsf(best) + 4e-36f;
  // norms next to nothing bound nothing; but a key of zeros has its biases for scores, exactly; scores near the end of fp32's range
  // (biases of infinity) may have overflowed, and no limit can be taken from them
  constexpr float kTiny = 1e-30f, kHuge = 1e37f;
  const bool known = !nan && xn2 < INFINITY && norm2 < INFINITY && (!(xmax > 0.f) || (norm2 > kTiny && xn2 > kTiny && fabsf(best) < kHuge));
  return {in_range && !known, in_range && known && xmax > 0.f && !(best - second > thr), best - thr};
}

}  // namespace saap
