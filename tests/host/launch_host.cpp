// Host build of the launch table, for its test.
// Build: g++ -O2 -std=c++17 -fPIC -shared
#include "../../paper_1807_08084_amd/csrc/launch.hpp"

namespace {
polsar_host::LaunchTable table;
}

extern "C" {
void host_set(int op, int dtype, int method, int prec, const polsar_launch* c) { table.set(op, dtype, method, prec, *c); }
void host_get(int op, int dtype, int method, int prec, polsar_launch* c) { *c = table.get(op, dtype, method, prec); }
void host_inv_det(int64_t n, int dtype, int method, int prec, int want_st, polsar_launch* c) {
  *c = table.inv_det(n, dtype, method, prec, want_st);
}
void host_multilook(int dtype, int method, int prec, int looks, int want_z, polsar_launch* c) {
  *c = table.multilook(dtype, method, prec, looks, want_z);
}
void host_batch(int dtype, int method, int prec, int writes, polsar_launch* c) {
  *c = table.batch(dtype, method, prec, writes);
}
void host_wishart(int64_t n, int dtype, int bwd, polsar_launch* c) { *c = table.wishart(n, dtype, bwd); }
}
