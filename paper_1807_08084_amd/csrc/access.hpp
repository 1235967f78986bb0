// Which accesses of the inverse and the Wishart pass stream (non-temporal) and
// which go through the 256 MB memory-side cache, by sizes and alignment.
// Plain C++: the rules are also compiled for the host by their test.
#pragma once

#include <cstddef>
#include <cstdint>

namespace polsar_host {

// Which accesses of a kernel are non-temporal.
enum : int { LOADS_NT = 1, STORES_NT = 2 };

constexpr int64_t MB = int64_t(1) << 20;

// Whether planes start off 128-byte lines: two waves then share a line at each
// of their seams.
inline bool off_lines(const void* p, int64_t pitch, size_t es) {
  return (uintptr_t)p % 128 || pitch * (int64_t)es % 128;
}

// The inverse.  Input lines that two waves read meet in the cache: off-line
// planes are loaded through it, us with streaming and with cached loads over six
// images in turn, FP32: 1398101 pixels 23.0, 22.4; 5475897: 75.5, 73.2; 12000369:
// 159.6, 154.3; 22369621: 303, 297; from 2^25 pixels on, where 16-byte accesses
// leave fewer seams, 34952533: 454, 460.  Aligned planes while several images fit:
// 1165085 pixels 18.0, 16.2 (over one, read before: 15.1, 14.4); 1398101: 21.1,
// 21.7 (18.0, 16.7); 4194304: 63.4, 64.9.
inline int inv_det_access(int64_t n, size_t es, bool off) {
  const bool cached = off ? n < (int64_t(1) << 25) : 9 * n * (int64_t)es <= 48 * MB;
  return cached ? STORES_NT : LOADS_NT | STORES_NT;
}

// The Wishart pass.  A pass without a gradient streams (cached loads: FP32,
// 6553601 pixels in plain planes, 87 -> 103 us).  With one, by the bytes of sigma
// and Z together; backward alone, FP32, us with streaming accesses, cached loads
// and both cached, over three inputs in turn (and over twelve):
// * Inputs off lines: cached loads at every size, 96 MB: 38.9, 36.2 (39.5, 38.0);
//   320 MB: 105.8, 102.3 (106.6, 102.6).
// * Aligned inputs up to 80 MB: cached loads, 32 MB: 12.1, 11.6 (12.8, 13.3); 80
//   MB: 26.0, 22.5 (26.4, 27.4): more where an input comes back soon or was just
//   written than it costs where none does.  Past that both lose, 128 MB: 37.3, 39.3
//   (38.1, 39.6); fused 41.5, 43.8.
// * A gradient off lines, where two waves' stores into a line are two partial
//   writes unless they meet in the cache: both cached from 80 to 176 MB, aligned
//   inputs, 96 MB: 34.8, 34.4, 35.1 (35.7, 36.5, 35.1), over one 34.3, 26.2, 26.1;
//   160 MB: 54.3, 56.1, 54.8 (55.0, 56.1, 54.6), over one 53.3, 42.1, 41.6; inputs
//   off lines, 128 MB: 47.1, 45.9, 45.2 (47.9, 46.1, 45.3).  Below, cached stores
//   push the inputs out: 64 MB 24.6, 19.0, 23.7; past it 256 MB 79.0, 81.3, 80.3.
inline int wishart_access(int64_t n, size_t es, bool bwd, bool off_in, bool off_grad) {
  const int64_t in = 18 * n * (int64_t)es;
  const bool small = in <= 80 * MB, middle = off_grad && !small && in <= 176 * MB;
  if (!bwd) return LOADS_NT | STORES_NT;
  return (off_in || small || middle ? 0 : LOADS_NT) | (middle ? 0 : STORES_NT);
}

}  // namespace polsar_host
