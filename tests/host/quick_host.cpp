// Host build of the FP32 compensated form's parts (pixel.hpp), for tests: the
// quick form and what it claims, the FP32 evaluation against its unsplit
// steps, and the two error-free forms against each other.
// Build: g++ -O2 -std=c++17 -fPIC -shared -fopenmp -ffp-contract=off
#include <cstdint>
#include <cstring>

#include "../../paper_1807_08084_amd/csrc/pixel.hpp"

extern "C" {

// quick: QUICK_*; ok: whether the FP32 evaluation carries the pixel; st: the
// error-free form's status.  Returns the pixels where the FP32 evaluation
// differs from cofactors_comp and det_comp, or the error-free forms differ.
int64_t host_quick(int64_t n, const float* z, float* inv, float* det, uint8_t* quick, uint8_t* ok, uint8_t* st,
                   int threads) {
  int64_t bad = 0;
#pragma omp parallel for num_threads(threads) schedule(static) reduction(+ : bad)
  for (int64_t i = 0; i < n; ++i) {
    float zz[9], x[9], y[9], d, e, bound, bound2;
    for (int k = 0; k < 9; ++k) zz[k] = z[k * n + i];
    quick[i] = (uint8_t)px::adjugate_comp_quick(zz, x, d);
    for (int k = 0; k < 9; ++k) inv[k * n + i] = x[k];
    det[i] = d;
    ok[i] = px::adjugate_comp_try(zz, &bound);
    px::DW<float> c[9];
    float rerr[9];
    bool ordered = true;
    px::cofactors_comp(zz, c, rerr, &ordered);
    const float dc = px::det_comp(zz, c, rerr, bound2);
    const float t = 1.0f / dc;
    const bool ok2 = ordered && dc > 0.0f && px::finite_(dc) && px::finite_(t) && !(bound2 > px::REROUTE_REL * dc) &&
                     zz[0] > 0.0f && c[2].hi + c[2].lo > 0.0f;
    const int s = px::adjugate_comp_reroute(zz, x, d), s2 = px::adjugate_comp_reroute_small(zz, y, e);
    st[i] = (uint8_t)s;
    bool same = ok2 == (bool)ok[i] && s == s2 && (bound == bound2 || (bound != bound && bound2 != bound2));
    same = same && (d == e || (d != d && e != e));
    for (int k = 0; k < 9; ++k) same = same && (x[k] == y[k] || (x[k] != x[k] && y[k] != y[k]));
    bad += !same;
  }
  return bad;
}

}  // extern "C"
