// The launch table: default shapes, the entries that callers set, and the shape
// of each kind of call.  Plain C++: also compiled for the host by its test.
#pragma once

#include <algorithm>
#include <cstdint>
#include <map>
#include <mutex>
#include <tuple>

#include "../../include/polsar.h"

namespace polsar_host {

// Defaults from a sweep of all launch shapes on MI355X (4096x4096 image):
// one 128-lane tile per block, one 128-bit vector per lane per plane,
// non-temporal (streaming) loads and stores.
// The Wishart kernel in FP64 with 16-byte accesses needs all 256 VGPRs (one
// wave per SIMD); with 8-byte accesses it runs at three waves per SIMD and
// 20% faster.  blocks_per_cu caps the resident blocks: with 4-5 waves per CU
// the 19 concurrent plane streams of a 3x3 inverse reach ~82% of HBM peak,
// with more they contend.
// Images below this many pixels take the Wishart kernel's launch from op 5
// of the table instead of op 1: on 2048x2048 (2^22 pixels) 8-byte accesses
// in 128-lane blocks, at most 5 per CU, ran the FP32 fused forward+backward
// 9-16% faster than the 4096x4096 image's shape, which is 4% faster there.
constexpr int64_t WISHART_SMALL = int64_t(1) << 23;
// Images of at least this many pixels take the inverse kernel's launch from
// op 6 of the table instead of op 0.  FP32 compensated on 8192x8192: 16-byte
// accesses in 128-lane blocks, at most 4 per CU: 846 us with a quarter of the
// pixels past the quick form, 841 with almost none (8-byte accesses, at most 6
// per CU: 866 and 845; on 4096x4096 images those take 204 us against 209).
// The Cholesky forms and the FP32-I/O FP64
// adjugate take the joint best of both 8192x8192 images (1-2% over their
// op-0 shapes); the other forms keep their op-0 shapes.
constexpr int64_t INV_DET_LARGE = int64_t(1) << 25;

inline int wishart_op(int64_t n) { return n < WISHART_SMALL ? 5 : 1; }
inline int inv_det_op(int64_t n) { return n >= INV_DET_LARGE ? 6 : 0; }

inline polsar_launch default_launch(int op, int dtype, int method, int prec) {
  const bool f64 = dtype == POLSAR_F64, chol = method == POLSAR_CHOLESKY;
  switch (op) {
    case 1:  // FP32: 8-byte accesses, at most 4 blocks per CU (4096^2: 0.774 of HBM against 0.763 with
             // 16-byte accesses and no cap; 8192^2: 0.738 against 0.684).  FP64 shapes with 256-lane blocks
             // reach 0.78 on 4096^2 but fall to 0.58 on 8192^2; 128 lanes, 4 per CU: 0.754 and 0.685
      return f64 ? polsar_launch{128, 1, 0, 1, 8, 4} : polsar_launch{256, 1, 0, 1, 8, 4};
    case 5:  // the Wishart kernel below WISHART_SMALL pixels: more, smaller tiles (FP64 on 2048^2: 5 blocks
             // per CU 0.757 of HBM, the Wishart tuner's pick in every bench run, against 0.689 with 4)
      return f64 ? polsar_launch{128, 1, 0, 1, 8, 5} : polsar_launch{128, 1, 0, 1, 8, 5};
    case 2:  // FP32 compensated: 8-byte accesses, at most 6 blocks of 128 lanes per CU (four-look 4096x4096
             // image: 357 us, 370 with 8 blocks of 256 lanes)
      if (!f64 && !chol && prec == POLSAR_COMPENSATED) return polsar_launch{128, 1, 0, 1, 8, 6};
      return f64 ? polsar_launch{256, 1, 0, 1, 8, 4} : polsar_launch{128, 1, 0, 1, 16, 0};
    case 3:  // one block of 128 lanes per tile, 8-byte accesses.  FP32, 12 images of 128..2048 and of 1024..2048
             // a side: 219 and 614 us at 6 blocks per CU, 221 and 624 without a cap.  FP64, 12 images of 128..1024
             // and of 1024 a side: 156 and 697 us at 5, 154 and 748 at 6; a persistent grid of 2 blocks of 256
             // lanes, 169 and 844
      return f64 ? polsar_launch{128, 1, 0, 1, 8, 5} : polsar_launch{128, 1, 0, 1, 8, 6};
    case 4:  // copy probe: few waves in flight stream best
      return polsar_launch{64, 1, 0, 1, 16, 5};
    case 6:  // the inverse kernel on images of at least INV_DET_LARGE pixels
      if (f64) break;
      if (!chol && prec == POLSAR_COMPENSATED) return polsar_launch{128, 1, 0, 1, 16, 4};
      if (!chol && prec == POLSAR_WIDE) return polsar_launch{64, 1, 0, 1, 16, 5};
      if (chol && prec == POLSAR_PLAIN) return polsar_launch{128, 1, 0, 1, 16, 3};
      if (chol && prec == POLSAR_COMPENSATED) return polsar_launch{128, 1, 0, 1, 16, 8};
      break;
    default:
      break;
  }
  // op 0: winners of the autotuner on 4096x4096 and 8192x8192 images of the
  // same recipe, taken together.  FP32 compensated, 4096x4096: 204-207 us with
  // at most 6 blocks of 128 lanes of 8-byte accesses, without and with
  // statuses, 210 and 211 with 8.  The FP64 adjugate runs 11%
  // faster on 8192x8192 with 16-byte accesses and 6 single-wave blocks per
  // CU than with 12 waves of 8-byte accesses (1% slower on 4096x4096).
  if (!chol && prec == POLSAR_COMPENSATED) return f64 ? polsar_launch{64, 1, 0, 1, 16, 6} : polsar_launch{128, 1, 0, 1, 8, 6};
  if (chol && prec == POLSAR_PLAIN) return f64 ? polsar_launch{64, 1, 0, 1, 16, 5} : polsar_launch{256, 1, 0, 1, 8, 3};
  if (!chol && prec == POLSAR_PLAIN) return f64 ? polsar_launch{64, 1, 0, 1, 16, 6} : polsar_launch{64, 1, 0, 1, 16, 5};
  if (chol && prec == POLSAR_WIDE) return polsar_launch{64, 2, 0, 1, 16, 0};
  if (chol) return polsar_launch{64, 1, 0, 1, 16, 0};
  return polsar_launch{128, 1, 0, 1, 8, 0};  // adjugate, FP32 storage with FP64 arithmetic
}

inline bool valid_launch(const polsar_launch& c, int op) {
  if (c.block != 64 && c.block != 128 && c.block != 256) return false;
  if (c.unroll != 1 && c.unroll != 2 && !((op == 0 || op == 6) && c.unroll == 4)) return false;
  if ((op == 2 || op == 3 || op == 4) && c.unroll != 1) return false;
  if (op == 4 && c.grid_per_cu != 0) return false;
  if (c.grid_per_cu < 0 || c.grid_per_cu > 64) return false;
  if (c.nontemporal != 0 && c.nontemporal != 1) return false;
  if (c.vector_bytes != 16 && c.vector_bytes != 8) return false;
  if (c.blocks_per_cu < 0 || c.blocks_per_cu > 64) return false;
  return true;
}

inline bool same_launch(const polsar_launch& a, const polsar_launch& b) {
  return a.block == b.block && a.unroll == b.unroll && a.grid_per_cu == b.grid_per_cu &&
         a.nontemporal == b.nontemporal && a.vector_bytes == b.vector_bytes && a.blocks_per_cu == b.blocks_per_cu;
}

// The entries set by callers and tuners.  A default shape set again is the
// default (a caller that restores what it read before leaves the table as it was).
class LaunchTable {
 public:
  void set(int op, int dtype, int method, int prec, const polsar_launch& c) {
    std::lock_guard<std::mutex> g(mu_);
    if (same_launch(c, default_launch(op, dtype, method, prec))) set_.erase({op, dtype, method, prec});
    else set_[{op, dtype, method, prec}] = c;
  }
  // is_default: whether no caller has set another shape
  polsar_launch get(int op, int dtype, int method, int prec, bool* is_default = nullptr) const {
    std::lock_guard<std::mutex> g(mu_);
    const auto it = set_.find({op, dtype, method, prec});
    if (is_default) *is_default = it == set_.end();
    return it == set_.end() ? default_launch(op, dtype, method, prec) : it->second;
  }

  // The launches of calls whose best cap depends on more than the table's key:
  // the default is adjusted, an entry that was set runs as it was set.

  // The inverse's launch.  An FP32 compensated call on a large image that wants
  // statuses (op 6) runs twice the resident blocks of the table: the FP32
  // evaluations of its ill-conditioned pixels need the waves (8192x8192 with
  // eigenvalues down to 1e-8: 858 us at 8 blocks per CU, 915 at 5), without
  // them fewer stream better (846 us at 4, 912 at 8).  Between 2^20 and 2^22
  // pixels one block more does (us at 6 and 7, three images in turn, eigenvalues
  // down to 1e-8: 1600x1600 41.5, 39.3, 1801x1799 52.0, 49.4; well conditioned
  // 34.8, 35.2 and 43.5, 43.9); from there on it costs more than it gives where
  // pixels are well conditioned (2048x2048 65.8, 67.9; 1024x1024 16.2, 16.9).
  polsar_launch inv_det(int64_t n, int dtype, int method, int prec, bool want_st) const {
    const int op = inv_det_op(n);
    bool standard;
    polsar_launch c = get(op, dtype, method, prec, &standard);
    if (standard && want_st && dtype == POLSAR_F32 && method == POLSAR_ADJUGATE && prec == POLSAR_COMPENSATED) {
      if (op == 6) c.blocks_per_cu = std::min(2 * c.blocks_per_cu, 64);
      else if (n > int64_t(1) << 20 && n < int64_t(1) << 22) ++c.blocks_per_cu;
    }
    return c;
  }

  // The multilook's launch.  FP32 compensated with Z stored too: one block per CU
  // fewer than the table's for its 9 more write streams, from four looks on
  // (3000x3001, four looks: 272 us at 5, 277 at 6; 4096x4096: 464 and 470; nine
  // looks of 2000x2000: 204 and 207), below which the looks' loads are too few to
  // hide the arithmetic (two of 2000x2000: 100 and 94).
  polsar_launch multilook(int dtype, int method, int prec, int n_looks, bool want_z) const {
    bool standard;
    polsar_launch c = get(2, dtype, method, prec, &standard);
    if (standard && want_z && n_looks >= 4 && dtype == POLSAR_F32 && method == POLSAR_ADJUGATE && prec == POLSAR_COMPENSATED &&
        c.blocks_per_cu > 1)
      --c.blocks_per_cu;
    return c;
  }

  // The Wishart kernel's launch.  A pass that writes no gradient runs twice the
  // resident blocks of the table: the cap is there for the nine write streams,
  // and a pass without them is bound by its reads in flight (forward alone,
  // FP32 2048x2048: 57 us, 65 with the table's 5; FP64 4096x4096: 359 with 8,
  // 428 with 4).  The tiles stay those of the table, so the partial sums and the
  // loss have the same bits as the fused pass's.
  polsar_launch wishart(int64_t n, int dtype, bool bwd) const {
    bool standard;
    polsar_launch c = get(wishart_op(n), dtype, 0, 0, &standard);
    if (standard && !bwd) c.blocks_per_cu = std::min(2 * c.blocks_per_cu, 64);
    return c;
  }

  // The batch's launch.  A plan that writes neither inverses nor gradients runs
  // twice the blocks, as the Wishart kernel does (likelihoods alone, us at the
  // table's cap and at twice: FP32 20 images of 300x301 30.5, 27.9; 8 of 1024x1024
  // 115.9, 110.4; FP64 55.0, 45.3 and 224.9, 209.2).
  polsar_launch batch(int dtype, int method, int prec, bool writes) const {
    bool standard;
    polsar_launch c = get(3, dtype, method, prec, &standard);
    if (standard && !writes) c.blocks_per_cu = std::min(2 * c.blocks_per_cu, 64);
    return c;
  }

 private:
  mutable std::mutex mu_;
  std::map<std::tuple<int, int, int, int>, polsar_launch> set_;
};

}  // namespace polsar_host
