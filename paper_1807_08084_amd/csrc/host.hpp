// Argument checks shared by the entry points.
#pragma once

#include <cstddef>
#include <cstdint>

#include "../../include/polsar.h"
#include "common.hpp"

namespace polsar_host {
using namespace polsar_dev;

inline size_t esize(int dtype) { return dtype == POLSAR_F64 ? 8 : 4; }

// Byte range [lo, hi) spanned by `planes` planes of n elements at `pitch`.
struct Range {
  uintptr_t lo, hi;
};
inline Range span(const void* p, int planes, int64_t pitch, int64_t n, size_t es) {
  uintptr_t lo = (uintptr_t)p;
  return Range{lo, lo + (uintptr_t)(((planes - 1) * pitch + n) * (int64_t)es)};
}
inline bool overlap(Range a, Range b) { return a.lo < b.hi && b.lo < a.hi; }

inline int check_planes(const void* p, int64_t pitch, int64_t n, size_t es) {
  if (!p) return n == 0 ? POLSAR_OK : POLSAR_E_ARG;  // an empty batch may pass null planes
  if (pitch < n || pitch > ((int64_t)1 << 40)) return POLSAR_E_ARG;
  if ((uintptr_t)p % es) return POLSAR_E_ALIGN;
  return POLSAR_OK;
}

inline bool vec_ok(const void* p, int64_t pitch, size_t es) {
  return p == nullptr || (((uintptr_t)p % 16) == 0 && ((pitch * (int64_t)es) % 16) == 0);
}

inline int op_code(int method, int prec) {
  if (method == POLSAR_ADJUGATE) return prec == POLSAR_PLAIN ? ADJ_PLAIN : prec == POLSAR_COMPENSATED ? ADJ_COMP : ADJ_WIDE;
  return prec == POLSAR_PLAIN ? CHOL_PLAIN : prec == POLSAR_COMPENSATED ? CHOL_COMP : CHOL_WIDE;
}

// Valid (dtype, method, precision) combination?
inline int check_mode(int dtype, int method, int prec) {
  if (dtype != POLSAR_F32 && dtype != POLSAR_F64) return POLSAR_E_ARG;
  if (method != POLSAR_ADJUGATE && method != POLSAR_CHOLESKY) return POLSAR_E_ARG;
  if (prec != POLSAR_PLAIN && prec != POLSAR_COMPENSATED && prec != POLSAR_WIDE) return POLSAR_E_ARG;
  if (dtype == POLSAR_F64 && prec == POLSAR_WIDE) return POLSAR_E_UNSUPPORTED;
  if (dtype == POLSAR_F64 && method == POLSAR_CHOLESKY && prec != POLSAR_PLAIN) return POLSAR_E_UNSUPPORTED;
  return POLSAR_OK;
}

}  // namespace polsar_host
