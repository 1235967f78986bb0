// Host build of the nonlocal-means kernel's shape rules, for their test.
// Build: g++ -O2 -std=c++17 -fPIC -shared
#include "../../paper_1807_08084_amd/csrc/nlm_shape.hpp"

extern "C" {
// rows * 10 + waves
int host_nlm_shape(int f64, int kl, int64_t height, int64_t width, int r) {
  const polsar_host::NlmShape s =
      f64 ? polsar_host::nlm_shape_f64(kl, height, width, r) : polsar_host::nlm_shape(false, kl, height, width);
  return s.rows * 10 + s.waves;
}
}
