// Host build of the rules that choose streaming or cached accesses, for their
// test.  Build: g++ -O2 -std=c++17 -fPIC -shared
#include "../../paper_1807_08084_amd/csrc/access.hpp"

extern "C" {
int host_inv_det_access(int64_t n, int es, int off) { return polsar_host::inv_det_access(n, es, off); }
int host_wishart_access(int64_t n, int es, int bwd, int off_in, int off_grad) {
  return polsar_host::wishart_access(n, es, bwd, off_in, off_grad);
}
int host_off_lines(uint64_t p, int64_t pitch, int es) { return polsar_host::off_lines((const void*)p, pitch, es); }
}
