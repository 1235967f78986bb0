// Output rows per lane and waves per tile of the nonlocal-means kernel.  Plain
// C++: also compiled for the host by its test.
#pragma once

#include <algorithm>
#include <cstdint>

namespace polsar_host {

struct NlmShape {
  int rows, waves;
};

inline int64_t nlm_blocks(int64_t height, int64_t width, int rows) {
  return ((width + 63) / 64) * ((height + rows - 1) / rows);
}

// By the number of two-row tiles (1024 SIMDs to fill).  KL in FP32 as (rows,
// waves): 256x256, r = 11 (512 tiles): 39 us (2, 8), 49 (2, 4), 151 (2, 1);
// 450x600, r = 5 (2250 tiles): 46 us (2, 4), 54 (2, 8), 62 (2, 1); 1024x1024, r =
// 11 (8192): 445 us (2, 4), 436 (3, 4), 490 (3, 1); 1200x1200, r = 5 (11400): 181
// us (3, 1), 183 (2, 4); 2048x2048, r = 11: 1607 us (3, 1), 1705 (2, 4).  Three
// rows only there: B in FP32, with the inverse before it, takes 1062 us with two
// and 1088 with three (2048x2048, r = 7; 450x600, r = 5: 51 and 57), FP64 has no
// registers for three.
inline NlmShape nlm_shape(bool f64, bool kl, int64_t height, int64_t width) {
  const int64_t tiles = nlm_blocks(height, width, 2);
  if (tiles < 1024) return {2, 8};
  if (tiles < 9216) return {2, 4};
  return {!f64 && kl ? 3 : 2, 1};
}

// FP64 runs two or three waves per SIMD, and its pairs saturate them: what
// counts is the work of the busiest SIMD.  In units of a pair: a neighbour costs
// its rows' pairs and, for KL, about one more for its 18 LDS reads; staging a row
// six; joining a tile's waves five a row.  Waves that split a small window
// unevenly wait for the longest, and one or two waves per SIMD hide less latency.
// A shape is taken over the one by tile counts where it is a tenth less.  us by
// tile counts, by this rule, and with four-wave blocks of one row a wave (the
// kernel before): B: 550x173, r = 1: 31, 14, 15; 173x585, r = 5: 122, 80, 106;
// 256x256, r = 5: 67, 49, 69; 768x768, r = 2: 118, 98, 94; r = 8: 793, 793, 825;
// KL: 128x128, r = 5: 20, 15, 51; 173x585, r = 5: 69, 47, 66; 768x768, r = 2: 92,
// 75, 83.
inline double nlm_cost_f64(NlmShape s, bool kl, int64_t height, int64_t width, int r) {
  constexpr int64_t cus = 256, simds = 4 * cus;
  const int64_t blocks = nlm_blocks(height, width, s.rows);
  const double row = (2 * r + 1) * (s.rows + (kl ? 1.0 : 0.0)) + 6.0;
  const int rows = 2 * r + s.rows, most = s.rows == 1 && !(kl && s.waves > 1) ? 3 : 2;  // waves per SIMD
  const double waves = (double)(blocks * s.waves) / simds, held = std::min<double>(most, waves);
  double per, n;
  if (s.waves == 1) {
    n = (double)((blocks + simds - 1) / simds);
    per = rows * row;
  } else {
    n = (double)((blocks + cus - 1) / cus) * (s.waves / 4);
    const bool alone = s.waves == 8 || blocks <= cus;  // no other block fills the wait
    per = (alone ? (double)((rows + s.waves - 1) / s.waves) : (double)rows / s.waves) * row + 5.0 * s.rows;
  }
  const double eff = held <= 1 ? 0.6 : held <= 2 ? 0.6 + 0.3 * (held - 1) : 0.9 + 0.1 * (held - 2);
  return n * per / eff;
}

inline NlmShape nlm_shape_f64(bool kl, int64_t height, int64_t width, int r) {
  NlmShape best = nlm_shape(true, kl, height, width);
  double limit = 0.9 * nlm_cost_f64(best, kl, height, width, r);
  for (const NlmShape s : {NlmShape{1, 1}, NlmShape{2, 1}, NlmShape{1, 4}, NlmShape{2, 4}}) {
    const double t = nlm_cost_f64(s, kl, height, width, r);
    if (t < limit) {
      limit = t;
      best = s;
    }
  }
  return best;
}

}  // namespace polsar_host
