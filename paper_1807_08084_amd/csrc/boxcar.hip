// Spatial (boxcar) multilook of a single-look image, fused with the
// per-pixel inverse and determinant.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/polsar.h"
#include "common.hpp"
#include "host.hpp"

namespace {
using namespace polsar_dev;
using namespace polsar_host;

// Spatial multilook fused with the inverse: Eq. (ZN) with the looks of pixel
// (y, x) taken from its (2R+1) x (2R+1) neighbourhood in a single-look
// image, clipped at the border,
//   Z(y, x) = (1/|W|) sum_{(y', x') in W(y, x)} S(y', x') S(y', x')^H.
// A block (one wave) owns BOX_TW output columns of a strip of rows and walks
// down it one input row at a time: the row's single-look
// pixels (with an R-pixel halo each side, zeros outside the image, which add
// nothing) are staged in LDS in FP64, double-buffered, while the next row is
// being loaded; each lane forms the sum of its K = 2R+1 horizontal
// neighbours' outer products in FP64 (exact products for FP32 input) and
// adds K consecutive row sums for its output.  Each output is scaled by the
// reciprocal of the clipped window size (within an FP64 ulp of the
// quotient), rounded to the storage type (optionally stored) and inverted
// with the per-pixel function of the per-call kernel.
//
// The vertical sums without subtraction (so every window keeps the error
// bound of a plain sum of its own terms): a lane keeps the sums of the last
// 1, 2, .. K-1 rows' row sums.  A new row's sum added to the longest is the
// next output's window, added to each of the others it makes the next longer
// one: K-1 additions of nine components, in ascending row order, and no copy
// of the K row sums from slot to slot (4096x4096, 5x5 windows: 320 -> 280 us).
//
// Bound by FP64 latency at two (7x7) or three waves per SIMD, 130 to 207
// registers a lane: a row takes a lone wave about 2900 cycles and a SIMD
// with several 2150 (3x3) to 2850 (7x7), for 306 vector instructions (3x3).
// More registers than 168 at 5x5 cost the third wave, 20%; a fourth wave at
// 3x3, bought with three spilled registers, 12%.
constexpr int BOX_TW = 64, BOX_MAX_R = 3;

struct BoxArgs {
  const void* s;
  int64_t sp;
  void* z;
  int64_t zp;
  void* inv;
  int64_t ip;
  void* det;
  uint8_t* status;
  unsigned long long* counters;
  int64_t H, W;
  int64_t nbx;  // blocks across the image
  int strip;    // rows per block
};

// The block's strip and this lane's column.
template <int R>
struct BoxStrip {
  int64_t x0, ys, y_first, y_last, gx, cols;
  double rcp;  // 1 / pixels of a window with all its rows
  __device__ BoxStrip(const BoxArgs& a) {
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t bx = t % a.nbx, by = t / a.nbx;
    x0 = bx * BOX_TW;
    ys = by * a.strip;
    const int64_t ye = ys + a.strip < a.H ? ys + a.strip : a.H;
    y_first = ys - R;  // rows staged (outside the image: zeros)
    y_last = ye - 1 + R;
    gx = x0 + threadIdx.x;
    cols = (gx + R < a.W ? gx + R : a.W - 1) - (gx - R > 0 ? gx - R : 0) + 1;
    rcp = 1.0 / (double)((2 * R + 1) * cols);
  }
};

// The staged pixels of input row y this lane loads.  Pixels outside the
// image load pixel 0 instead (every load is in bounds and unconditional, so
// the loads stay in flight while the current row is summed) and are staged
// as zeros, which add nothing.
template <class T, int R, int P>
__device__ __forceinline__ void box_load_row(const BoxArgs& a, int64_t x0, int64_t y, T (&v)[P][6], bool (&ok)[P]) {
  constexpr int SW = BOX_TW + 2 * R;
  const T* __restrict__ S = (const T*)a.s;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int col = threadIdx.x + p * BOX_TW;
    const int64_t x = x0 - R + col;
    ok[p] = col < SW && y >= 0 && y < a.H && x >= 0 && x < a.W;
    const int64_t i = ok[p] ? y * a.W + x : 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) v[p][k] = S[k * a.sp + i];
  }
}

// Stage the loaded row in an LDS row buffer, in FP64.
template <class T, int R, int P>
__device__ __forceinline__ void box_stage(double (*row)[BOX_TW + 2 * R], const T (&v)[P][6], const bool (&ok)[P]) {
  constexpr int SW = BOX_TW + 2 * R;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int col = threadIdx.x + p * BOX_TW;
    if (col < SW)
#pragma unroll
      for (int k = 0; k < 6; ++k) row[k][col] = ok[p] ? (double)v[p][k] : 0.0;
  }
}

// This lane's row sum of the staged row: its K horizontal neighbours.
template <int R>
__device__ __forceinline__ void box_row_sum(double (*row)[BOX_TW + 2 * R], double (&sum)[9]) {
  double s6[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) s6[k] = row[k][threadIdx.x];
  px::look_first(s6, sum);
#pragma unroll
  for (int dx = 1; dx < 2 * R + 1; ++dx) {
#pragma unroll
    for (int k = 0; k < 6; ++k) s6[k] = row[k][threadIdx.x + dx];
    px::look_accumulate_chained(s6, sum);
  }
}

// Output row yo of this lane from its window sum: Z, inverse, det, status.
template <class T, int OP, int R, bool NT>
__device__ __forceinline__ void box_output(const BoxArgs& a, const BoxStrip<R>& b, int64_t yo, const double (&w)[9],
                                           unsigned& c0, unsigned& c1, unsigned& c2) {
  // (at 5x5 the kept reciprocal's registers would cost a wave)
  double rcp = b.rcp;
  if (R == 2 || yo < R || yo + R >= a.H) {  // the same for every lane of the block
    const int64_t rows = (yo + R < a.H ? yo + R : a.H - 1) - (yo - R > 0 ? yo - R : 0) + 1;
    rcp = 1.0 / (double)(rows * b.cols);
  }
  T zz[9], xx[9], dt;
#pragma unroll
  for (int c = 0; c < 9; ++c) zz[c] = (T)(w[c] * rcp);
  const int64_t i = yo * a.W + b.gx;
  auto put = [&](T* p, T v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
  };
  if (a.z)
#pragma unroll
    for (int c = 0; c < 9; ++c) put((T*)a.z + c * a.zp + i, zz[c]);
  const int st_px = run_pixel<T, OP>(zz, xx, dt, a.status || a.counters);
  tally(st_px, c0, c1, c2);
  if (a.inv)
#pragma unroll
    for (int c = 0; c < 9; ++c) put((T*)a.inv + c * a.ip + i, xx[c]);
  if (a.det) put((T*)a.det + i, dt);
  if (a.status) a.status[i] = (uint8_t)st_px;
}

template <class T, int OP, int R, bool NT>
__global__ __launch_bounds__(BOX_TW, R == 2 ? 3 : 1) void k_boxcar(BoxArgs a) {
  constexpr int K = 2 * R + 1, SW = BOX_TW + 2 * R;
  constexpr int P = (SW + BOX_TW - 1) / BOX_TW;  // staged pixels per lane and row
  __shared__ double row[2][6][SW];
  const BoxStrip<R> b(a);
  // part[m]: the sum of the last m + 1 rows' row sums
  double part[K > 1 ? K - 1 : 1][9];
#pragma unroll
  for (int m = 0; m < K - 1; ++m)
#pragma unroll
    for (int c = 0; c < 9; ++c) part[m][c] = 0.0;
  T pre[P][6];
  bool pok[P];
  unsigned c0 = 0, c1 = 0, c2 = 0;
  box_load_row<T, R, P>(a, b.x0, b.y_first, pre, pok);
#pragma unroll 1
  for (int64_t y = b.y_first; y <= b.y_last; ++y) {  // the same for every lane of the block
    const int buf = (int)((y - b.y_first) & 1);
    box_stage<T, R, P>(row[buf], pre, pok);
    wave_sync();
    if (y + 1 <= b.y_last) box_load_row<T, R, P>(a, b.x0, y + 1, pre, pok);  // in flight while this row is summed
    double sum[9], w[9];
    box_row_sum<R>(row[buf], sum);
    // output row y - R: window rows y - 2R .. y
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      w[c] = K > 1 ? part[K > 1 ? K - 2 : 0][c] + sum[c] : sum[c];
#pragma unroll
      for (int m = K - 2; m > 0; --m) part[m][c] = part[m - 1][c] + sum[c];
      part[0][c] = sum[c];
    }
    const int64_t yo = y - R;
    if (yo >= b.ys && b.gx < a.W) box_output<T, OP, R, NT>(a, b, yo, w, c0, c1, c2);
  }
  if (a.counters) flush_counters(a.counters, c0, c1, c2);
}

// ---- boxcar launch: one block (one wave) per BOX_TW columns x strip rows, a
// 1-D grid; the radius is a template parameter (the sums are indexed at
// compile time)

// Rows per block: a block re-forms its 2R halo rows' sums, so tall strips do
// less, and short ones fill the chip and end together.  The rows a SIMD walks
// are (strip + 2R) times its waves, and about 1.2 strips more for the end.
// Measured (FP32, us at 64, 32, 16, 8 rows): 450x600, 3x3: 80, 43, 26, 18;
// 1024x1024: 79, 45, 25, 21; 2048x2048: 84, 61, 59, 62; 2999x3001: 167, 163,
// 149, 152; 4096x4096: 268, 243, 245, 259; 7x7 with Z, 2999x3001: 364, 302,
// 278, 304; 7x7, 4096x4096: 331, 344, 368, 430 (32 is taken).
int box_strip(const BoxArgs& a, int R) {
  int cus = 256;
  (void)polsar_device_compute_units(&cus);
  int best = 64;
  double best_t = 1e300;
  for (int strip : {64, 32, 24, 16, 8, 4}) {
    const double waves = (double)(a.nbx * ((a.H + strip - 1) / strip)) / (4.0 * cus);  // per SIMD
    const double t = (strip + 2 * R) * (waves + 1.2);
    if (t < best_t) { best_t = t; best = strip; }
  }
  return best;
}

// Streaming stores where every row of every output plane starts on a 128-byte
// line, so that a wave's store fills whole lines (FP64 3x3 on 2048x2048: 120
// -> 94 us, FP32 3x3 with Z on 4096x4096: 379 -> 361); elsewhere the lines two
// waves share have to meet in the cache (2999x3001, 3x3: 150 us against 184).
bool box_nontemporal(const BoxArgs& a, size_t es) {
  auto whole = [&](const void* p, int64_t pitch) { return !p || ((uintptr_t)p % 128 == 0 && pitch * es % 128 == 0); };
  return a.W * es % 128 == 0 && whole(a.z, a.zp) && whole(a.inv, a.ip) && whole(a.det, 0);
}

template <class T, int OP, int R>
hipError_t go_boxcar_r(BoxArgs& a, hipStream_t s) {
  a.nbx = (a.W + BOX_TW - 1) / BOX_TW;
  a.strip = box_strip(a, R);
  const int64_t nby = (a.H + a.strip - 1) / a.strip;
  const dim3 grid((unsigned)(a.nbx * nby));
  if (box_nontemporal(a, sizeof(T))) hipLaunchKernelGGL((k_boxcar<T, OP, R, true>), grid, dim3(BOX_TW), 0, s, a);
  else hipLaunchKernelGGL((k_boxcar<T, OP, R, false>), grid, dim3(BOX_TW), 0, s, a);
  return hipGetLastError();
}

template <class T, int OP>
hipError_t go_boxcar(BoxArgs& a, int r, hipStream_t s) {
  switch (r) {
    case 0: return go_boxcar_r<T, OP, 0>(a, s);
    case 1: return go_boxcar_r<T, OP, 1>(a, s);
    case 2: return go_boxcar_r<T, OP, 2>(a, s);
    default: return go_boxcar_r<T, OP, 3>(a, s);
  }
}

hipError_t launch_boxcar(int dtype, int op, BoxArgs& a, int r, hipStream_t s) {
  if (dtype == POLSAR_F32) {
    switch (op) {
      case ADJ_PLAIN: return go_boxcar<float, ADJ_PLAIN>(a, r, s);
      case ADJ_COMP: return go_boxcar<float, ADJ_COMP>(a, r, s);
      case ADJ_WIDE: return go_boxcar<float, ADJ_WIDE>(a, r, s);
      case CHOL_PLAIN: return go_boxcar<float, CHOL_PLAIN>(a, r, s);
      case CHOL_COMP: return go_boxcar<float, CHOL_COMP>(a, r, s);
      default: return go_boxcar<float, CHOL_WIDE>(a, r, s);
    }
  }
  switch (op) {
    case ADJ_PLAIN: return go_boxcar<double, ADJ_PLAIN>(a, r, s);
    case ADJ_COMP: return go_boxcar<double, ADJ_COMP>(a, r, s);
    default: return go_boxcar<double, CHOL_PLAIN>(a, r, s);
  }
}

}  // namespace

extern "C" {

int polsar_boxcar_inv_det(int dtype, int method, int precision, int64_t height, int64_t width, int radius,
                          const void* s, int64_t s_pitch, void* z, int64_t z_pitch, void* inv, int64_t inv_pitch,
                          void* det, uint8_t* status, unsigned long long* counters, void* stream) {
  int r = check_mode(dtype, method, precision);
  if (r) return r;
  if (height < 0 || width < 0 || radius < 0 || radius > BOX_MAX_R) return POLSAR_E_ARG;
  if (height > ((int64_t)1 << 24) || width > ((int64_t)1 << 24)) return POLSAR_E_ARG;
  const int64_t n = height * width;
  // one 64-lane block per 64 columns of a strip of at least 4 rows: at most
  // 2^26 blocks (single columns), a 1-D grid
  if (n > ((int64_t)1 << 32)) return POLSAR_E_ARG;
  const size_t es = esize(dtype);
  if ((r = check_planes(s, s_pitch, n, es))) return r;
  if (z && (r = check_planes(z, z_pitch, n, es))) return r;
  if (inv && (r = check_planes(inv, inv_pitch, n, es))) return r;
  if (det && ((uintptr_t)det % es)) return POLSAR_E_ALIGN;
  if (counters && ((uintptr_t)counters % 8)) return POLSAR_E_ALIGN;
  if (!z && !inv && !det && !status && !counters) return POLSAR_E_ARG;
  if (n > 0) {
    const Range rl = span(s, 6, s_pitch, n, es);
    const Range rz = z ? span(z, 9, z_pitch, n, es) : Range{0, 0};
    const Range ri = inv ? span(inv, 9, inv_pitch, n, es) : Range{0, 0};
    const Range rd = det ? span(det, 1, n, n, es) : Range{0, 0};
    const Range rs = status ? span(status, 1, n, n, 1) : Range{0, 0};
    const Range all[5] = {rl, rz, ri, rd, rs};
    for (int p = 0; p < 5; ++p)
      for (int q = p + 1; q < 5; ++q)
        if (all[p].hi > all[p].lo && all[q].hi > all[q].lo && overlap(all[p], all[q])) return POLSAR_E_ALIAS;
  }
  if (n == 0) return POLSAR_OK;
  BoxArgs a{s, s_pitch, z, z_pitch, inv, inv_pitch, det, status, counters, height, width, 0, 0};
  if (launch_boxcar(dtype, op_code(method, precision), a, radius, (hipStream_t)stream) != hipSuccess)
    return POLSAR_E_HIP;
  return POLSAR_OK;
}

}  // extern "C"
