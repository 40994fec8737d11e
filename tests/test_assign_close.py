"""Which centroids the second walk of the fp32 key assignment lists, as a host program over the kernel's own rule: a workgroup's 128 lanes,
of which the last ones hold copies of the last key."""
from test_host_sync import run_program


def test_only_close_keys_of_the_tensor_list_centroids(tmp_path):
    """Close keys beside keys whose scores are infinite, overflow, are no numbers or next to nothing, in any place; and, as the
    last one, behind it."""
    run_program(tmp_path, r"""
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "assign_close.h"
constexpr int kKeys = 128, kD = 128, B = 16;
int main() {
  const float inf = INFINITY, nan = NAN, tol = 8.0f * 128.0f * 5.9604645e-8f;
  std::mt19937 rng(1);
  std::normal_distribution<float> normal;
  std::vector<float> c(B * kD);
  for (auto& v : c) v = normal(rng);
  std::copy_n(c.begin(), kD, c.begin() + 5 * kD);                        // every key's best two may be equal
  int listed_by_close = 0;
  for (float special : {inf, -inf, nan, 3e38f, 1e30f, 1e-30f, 0.f})
    for (int n : {24, 127, 128, 1})
      for (int at : {n - 1, 0, n / 2}) {
        std::vector<float> x(kKeys * kD);
        for (int k = 0; k < n; ++k)
          for (int i = 0; i < kD; ++i) x[k * kD + i] = c[i] + 0.1f * normal(rng);
        if (special == inf || special == -inf || special == nan) x[at * kD + 7] = special;
        else for (int i = 0; i < kD; ++i) x[at * kD + i] = special * (c[i] < 0 ? -1.f : 1.f);
        if (special != special) x[at * kD + 7] = nan;
        for (int k = 0; k < kKeys; ++k) {
          const float* xk = &x[std::min(k, n - 1) * kD];
          float best = -inf, second = -inf, xn2 = 0, xmax = 0, norm2 = 0, score[B];
          double exact[B];
          bool bad = false;
          for (int i = 0; i < kD; ++i) xn2 += xk[i] * xk[i], xmax = fmaxf(xmax, fabsf(xk[i]));
          for (int b = 0; b < B; ++b) {
            float s = 0, q = 0;
            exact[b] = 0;
            for (int i = 0; i < kD; ++i) s += xk[i] * c[b * kD + i], q += c[b * kD + i] * c[b * kD + i], exact[b] += (double)xk[i] * c[b * kD + i];
            score[b] = s;
            norm2 = fmaxf(norm2, q);
            bad |= s != s;
            second = fmaxf(second, fminf(best, s));
            best = fmaxf(best, s);
          }
          const saap::KeyScores ks = saap::decide_key(best, second, bad, xmax, xn2, norm2, tol, k < n);
          if (ks.odd && ks.close) return printf("key %d of %d: both\n", k, n), 1;
          const double most = *std::max_element(exact, exact + B);
          for (int b = 0; b < B; ++b) {
            if (ks.lists(score[b]) && (k >= n || ks.odd)) return printf("special %g, key %d of %d lists centroid %d\n", special, k, n, b), 1;
            if (k < n && ks.close && exact[b] == most && !ks.lists(score[b])) return printf("key %d of %d misses centroid %d\n", k, n, b), 1;
            listed_by_close += ks.lists(score[b]);
          }
        }
      }
  return listed_by_close > 1000 ? 0 : 2;
}
""")
