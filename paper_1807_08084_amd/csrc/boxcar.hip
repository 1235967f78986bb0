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
// A wave owns 64 columns of a strip of rows, or 128 (FP32 compensated 3x3:
// two a lane, side by side), and walks down it one input row at a time: the row's
// single-look pixels (with an R-pixel halo each side, zeros outside the image,
// which add nothing) are staged in LDS in FP64, double-buffered, while the next
// row is being loaded; each lane forms the sum of its K = 2R+1 horizontal
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
// Bound by FP64 issue and latency at two or three waves per SIMD (139 to 247
// registers a lane) and, with the stores of 10 or 19 planes, by memory: FP32 3x3
// on 4096x4096 takes 187 us with the determinant alone and 217 with all ten
// planes (170 at the copy rate).  Two columns a lane at 3x3 share their windows'
// two inner columns, 36 FP64 operations per column's row sum instead of 54, and
// halve the accesses: 239 -> 217 us.  5x5 and 7x7 have no registers for that, nor
// do the other forms' inverses twice (plain, 225 us at one column, 360 at two).
// A bound of 168 registers (three waves) spills at 5x5: 315 us against 283 with
// two waves and none.
constexpr int BOX_TW = 64, BOX_MAX_R = 3, BOX_MIN_STRIP = 4;

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

// This lane of its wave.
__device__ __forceinline__ int box_lane() { return threadIdx.x % BOX_TW; }

// The wave's strip and this lane's columns (C of them, side by side).
template <int R, int C>
struct BoxStrip {
  static constexpr int TW = BOX_TW * C;
  int64_t x0, ys, y_first, y_last, gx, cols[C];
  double rcp[C];  // 1 / pixels of a window with all its rows
  __device__ BoxStrip(const BoxArgs& a, int waves, int wave) {
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t bx = t % a.nbx, by = t / a.nbx;
    x0 = (bx * waves + wave) * TW;
    ys = by * a.strip;
    const int64_t ye = ys + a.strip < a.H ? ys + a.strip : a.H;
    y_first = ys - R;  // rows staged (outside the image: zeros)
    y_last = ye - 1 + R;
    gx = x0 + box_lane() * C;
#pragma unroll
    for (int l = 0; l < C; ++l) {
      const int64_t x = gx + l;
      cols[l] = (x + R < a.W ? x + R : a.W - 1) - (x - R > 0 ? x - R : 0) + 1;
      rcp[l] = 1.0 / (double)((2 * R + 1) * cols[l]);
    }
  }
};

// The next input row's pixels on their way to LDS: this lane's columns of the
// six planes, and one value of the R halo columns on either side (12R of them,
// a lane each).  The addresses are a row's, uniform, plus the lane's offset.
// Pixels outside the image load one inside instead (every load is in bounds
// and unconditional, so the loads stay in flight while the current row is
// summed) and are staged as zeros, which add nothing.
template <class T, int R, int C>
struct BoxLoad {
  static constexpr int HALO = 12 * R, TW = BOX_TW * C;
  static_assert(HALO <= BOX_TW, "a lane per halo value");
  typedef typename VecOf<T, C>::type VT;
  uint32_t off[C], hoff;  // in bytes, from the row's start (and the halo value's plane)
  int64_t hplane;
  bool ok[C], hok, inner;
  T v[6][C], h;
  __device__ BoxLoad(const BoxArgs& a, const BoxStrip<R, C>& b) {
    const int hk = R && box_lane() < HALO ? box_lane() / (2 * R) : 0, hc = R ? box_lane() % (2 * R) : 0;
    const int64_t hx = b.x0 + (hc < R ? hc - R : hc - R + TW);
    inner = b.x0 + TW <= a.W;
#pragma unroll
    for (int l = 0; l < C; ++l) {
      ok[l] = b.gx + l < a.W;
      off[l] = (uint32_t)((ok[l] ? b.gx + l : 0) * sizeof(T));
    }
    hok = hx >= 0 && hx < a.W;
    hoff = (uint32_t)((hok ? hx : 0) * sizeof(T));
    hplane = hk * a.sp;
  }
  __device__ __forceinline__ void load(const BoxArgs& a, int64_t y) {
    const int64_t yc = y < 0 ? 0 : y < a.H ? y : a.H - 1;
    const T* __restrict__ S = (const T*)a.s + yc * a.W;
    auto at = [](const T* p, uint32_t o) { return (const T*)((const char*)p + o); };
    if (C == 1 || !inner) {
#pragma unroll
      for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int l = 0; l < C; ++l) v[k][l] = *at(S + k * a.sp, off[l]);
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k) load_v<T, C, false>(at(S + k * a.sp, off[0]), v[k]);
    }
    if constexpr (R > 0) h = *at(S + hplane, hoff);
  }
  // Stage the loaded row y in an LDS row buffer, in FP64.
  __device__ __forceinline__ void stage(const BoxArgs& a, int64_t y, double (*row)[TW + 2 * R]) const {
    const bool oky = y >= 0 && y < a.H;
    if (inner && oky) {
#pragma unroll
      for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int l = 0; l < C; ++l) row[k][box_lane() * C + R + l] = (double)v[k][l];
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int l = 0; l < C; ++l) row[k][box_lane() * C + R + l] = ok[l] && oky ? (double)v[k][l] : 0.0;
    }
    if constexpr (R > 0)
      if (box_lane() < HALO) {
        const int hc = box_lane() % (2 * R);
        row[box_lane() / (2 * R)][hc < R ? hc : hc + TW] = hok && oky ? (double)h : 0.0;
      }
  }
};

// This lane's row sums of the staged row: the K horizontal neighbours of each
// of its columns.  Two columns' windows share all but their outer columns,
// whose products are added to the shared sum last.
template <int R, int C>
__device__ __forceinline__ void box_row_sum(double (*row)[BOX_TW * C + 2 * R], double (&sum)[C][9]) {
  const int j = box_lane() * C;
  if constexpr (C == 1) {
    double s6[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) s6[k] = row[k][j];
    px::look_first(s6, sum[0]);
#pragma unroll
    for (int dx = 1; dx < 2 * R + 1; ++dx) {
#pragma unroll
      for (int k = 0; k < 6; ++k) s6[k] = row[k][j + dx];
      px::look_accumulate_chained(s6, sum[0]);
    }
  } else {
    static_assert(C == 2 && R > 0, "two columns with a common neighbour");
    typedef double V2 __attribute__((ext_vector_type(2)));
    double left[6], right[6], shared[9];
#pragma unroll
    for (int m = 0; m <= R; ++m) {
      double p[6], q[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const V2 v = *(const V2*)&row[k][j + 2 * m];  // rows of an even length: 16-byte aligned
        p[k] = v.x;
        q[k] = v.y;
      }
      if (m == 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) left[k] = p[k];
        px::look_first(q, shared);
      } else {
        px::look_accumulate_chained(p, shared);
        if (m < R) px::look_accumulate_chained(q, shared);
        else
#pragma unroll
          for (int k = 0; k < 6; ++k) right[k] = q[k];
      }
    }
#pragma unroll
    for (int c = 0; c < 9; ++c) sum[0][c] = sum[1][c] = shared[c];
    px::look_accumulate_chained(left, sum[0]);
    px::look_accumulate_chained(right, sum[1]);
  }
}

// Output row yo of this lane from its window sums: Z, inverse, det, status.
template <class T, int R, int C>
struct BoxOut {
  T zz[C][9], xx[C][9], dt[C];
  int st[C];
  template <int OP>
  __device__ __forceinline__ void compute(const BoxArgs& a, const BoxStrip<R, C>& b, int64_t yo,
                                          const double (&w)[C][9]) {
#pragma unroll
    for (int l = 0; l < C; ++l) {
      double rcp = b.rcp[l];
      if (yo < R || yo + R >= a.H) {  // the same for every lane of the block
        const int64_t rows = (yo + R < a.H ? yo + R : a.H - 1) - (yo - R > 0 ? yo - R : 0) + 1;
        rcp = 1.0 / (double)(rows * b.cols[l]);
      }
#pragma unroll
      for (int c = 0; c < 9; ++c) zz[l][c] = (T)(w[l][c] * rcp);
    }
    const bool want_st = a.status || a.counters;
    if constexpr (C == 2 && OP == ADJ_COMP && sizeof(T) == 4) {
      // what the quick form leaves over goes through one copy of the rest
      int quick[C];
#pragma unroll
      for (int l = 0; l < C; ++l) {
        quick[l] = px::adjugate_comp_quick(zz[l], xx[l], dt[l]);
        st[l] = px::ST_OK;
      }
      if (quick[0] != px::QUICK_ALL || quick[1] != px::QUICK_ALL) {
#pragma unroll 1
        for (int l = 0; l < C; ++l) {
          const int ql = l ? quick[1] : quick[0];
          if (ql == px::QUICK_ALL) continue;
          T zl[9], xl[9], dl = l ? dt[1] : dt[0];
#pragma unroll
          for (int c = 0; c < 9; ++c) {
            zl[c] = l ? zz[1][c] : zz[0][c];
            xl[c] = l ? xx[1][c] : xx[0][c];
          }
          const int sl = px::adjugate_comp_rest(zl, xl, dl, ql, want_st);
#pragma unroll
          for (int c = 0; c < 9; ++c) {
            xx[0][c] = l ? xx[0][c] : xl[c];
            xx[1][c] = l ? xl[c] : xx[1][c];
          }
          dt[0] = l ? dt[0] : dl;
          dt[1] = l ? dl : dt[1];
          st[0] = l ? st[0] : sl;
          st[1] = l ? sl : st[1];
        }
      }
    } else {
#pragma unroll
      for (int l = 0; l < C; ++l) st[l] = run_pixel<T, OP>(zz[l], xx[l], dt[l], want_st);
    }
  }
  template <bool NT>
  __device__ __forceinline__ void store(const BoxArgs& a, const BoxStrip<R, C>& b, int64_t yo) const {
    const int64_t i = yo * a.W + b.x0;  // uniform; the lane's offset is its own
    const bool whole = C == 1 || b.x0 + BoxStrip<R, C>::TW <= a.W;
    const int j = box_lane() * C;
    auto put = [&](T* p, const T (&v)[C]) {
      if (whole) store_v<T, C, NT>(p + j, v);
      else
#pragma unroll
        for (int l = 0; l < C; ++l)
          if (b.gx + l < a.W) p[j + l] = v[l];
    };
    auto planes = [&](void* base, int64_t pitch, const T (&v)[C][9]) {
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        T o[C];
#pragma unroll
        for (int l = 0; l < C; ++l) o[l] = v[l][c];
        put((T*)base + c * pitch + i, o);
      }
    };
    if (a.z) planes(a.z, a.zp, zz);
    if (a.inv) planes(a.inv, a.ip, xx);
    if (a.det) put((T*)a.det + i, dt);
    if (a.status)
#pragma unroll
      for (int l = 0; l < C; ++l)
        if (l == 0 || b.gx + l < a.W) (a.status + i)[j + l] = (uint8_t)st[l];
  }
};

template <class T, int OP, int R, int C, bool NT, int NW>
__global__ __launch_bounds__(BOX_TW * NW, C == 2 ? 2 : 1) void k_boxcar(BoxArgs a) {
  constexpr int K = 2 * R + 1, SW = BOX_TW * C + 2 * R;
  __shared__ __align__(16) double rows[NW][2][6][SW];
  const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / BOX_TW);
  double (*row)[6][SW] = rows[wave];
  const BoxStrip<R, C> b(a, NW, wave);
  if (NW > 1 && b.x0 >= a.W) return;  // no barrier waits for a wave that has ended
  // part[m]: the sum of the last m + 1 rows' row sums
  double part[K > 1 ? K - 1 : 1][C][9];
#pragma unroll
  for (int m = 0; m < K - 1; ++m)
#pragma unroll
    for (int l = 0; l < C; ++l)
#pragma unroll
      for (int c = 0; c < 9; ++c) part[m][l][c] = 0.0;
  unsigned c0 = 0, c1 = 0, c2 = 0;
  BoxLoad<T, R, C> next(a, b);
  next.load(a, b.y_first);
  next.stage(a, b.y_first, row[0]);
#pragma unroll 1
  for (int64_t y = b.y_first; y <= b.y_last; ++y) {  // the same for every lane of the block
    const int buf = (int)((y - b.y_first) & 1);
    wave_sync();
    if (y < b.y_last) next.load(a, y + 1);  // in flight while this row is summed and inverted
    double sum[C][9], w[C][9];
    box_row_sum<R, C>(row[buf], sum);
    // output row y - R: window rows y - 2R .. y
#pragma unroll
    for (int l = 0; l < C; ++l)
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        w[l][c] = K > 1 ? part[K > 1 ? K - 2 : 0][l][c] + sum[l][c] : sum[l][c];
#pragma unroll
        for (int m = K - 2; m > 0; --m) part[m][l][c] = part[m - 1][l][c] + sum[l][c];
        part[0][l][c] = sum[l][c];
      }
    const int64_t yo = y - R;
    const bool mine = yo >= b.ys && b.gx < a.W;
    BoxOut<T, R, C> out;
    if (mine) {
      out.template compute<OP>(a, b, yo, w);
#pragma unroll
      for (int l = 0; l < C; ++l)
        if (l == 0 || b.gx + l < a.W) tally(out.st[l], c0, c1, c2);
    }
    // the next row is staged before this one's outputs leave: waiting for its
    // loads after the stores would wait for the stores too
    if (y < b.y_last) next.stage(a, y + 1, row[buf ^ 1]);
    if (NW > 1) __builtin_amdgcn_s_barrier();  // keeps step; nothing is exchanged
    if (mine) out.template store<NT>(a, b, yo);
  }
  if (a.counters) flush_counters(a.counters, c0, c1, c2);
}

// ---- boxcar launch: one block per NW waves' columns x strip rows, a 1-D grid;
// the radius is a template parameter (the sums are indexed at compile time)

// Rows per block.  Blocks of one launch take the same time, so they end in
// rounds of as many as are resident at once; a round takes its rows, the 2R
// halo rows whose sums a strip re-forms among them, times the waves per SIMD
// and about 1.2 more.  The strips that just fill a number of rounds are among
// those tried; several rounds even out pixels of different cost, for which
// each of them counts 8% over their number less.  FP32 3x3 on 4096x4096 (2048
// waves a round), rows: us: 64: 217, 32: 219, 16: 227, 24 (2.7 rounds): 235, 48
// (1.3): 270; FP32 7x7 with Z on 2999x3008, 70 rows (one round): 180, 24 (2.9):
// 203; on 3072x3072, 70 (1.01 rounds): 243; FP32 3x3 on 450x600, 4 rows: 13, 8:
// 18, 16: 30.
int box_strip(const BoxArgs& a, int R, int waves, int resident) {
  int cus = 256;
  (void)polsar_device_compute_units(&cus);
  const int64_t slots = (int64_t)resident * cus;
  int64_t best = BOX_MIN_STRIP;
  double best_t = 1e300;
  auto consider = [&](int64_t rows) {
    rows = std::max<int64_t>(BOX_MIN_STRIP, std::min<int64_t>(rows, a.H));
    const int64_t blocks = a.nbx * ((a.H + rows - 1) / rows), full = blocks / slots, rest = blocks % slots;
    auto round = [&](int64_t n) { return n ? (double)(n * waves) / (4.0 * cus) + 1.2 : 0.0; };
    const double t = (double)(rows + 2 * R) * ((double)full * round(slots) + round(rest)) *
                     (1.0 + 0.08 / std::max(1.0, (double)blocks / (double)slots));
    if (t < best_t) { best_t = t; best = rows; }
  };
  for (int64_t rounds = 1; rounds <= 16; ++rounds) {
    const int64_t strips = std::max<int64_t>(1, rounds * slots / a.nbx);
    consider((a.H + strips - 1) / strips);
  }
  for (int64_t rows : {64, 32, 24, 16, 8, 4}) consider(rows);
  return (int)best;
}

// Streaming stores where every row of every output plane starts on a 128-byte
// line, so that a wave's store fills whole lines (FP64 3x3 on 2048x2048: 120
// -> 94 us, FP32 3x3 with Z on 4096x4096: 379 -> 361); elsewhere the lines two
// waves share have to meet in the cache (2999x3001, 3x3: 150 us against 184).
bool box_nontemporal(const BoxArgs& a, size_t es) {
  auto whole = [&](const void* p, int64_t pitch) { return !p || ((uintptr_t)p % 128 == 0 && pitch * es % 128 == 0); };
  return a.W * es % 128 == 0 && whole(a.z, a.zp) && whole(a.inv, a.ip) && whole(a.det, 0);
}

template <class T, int OP, int R, int C, bool NT, int NW>
hipError_t go_boxcar_nw(BoxArgs& a, hipStream_t s) {
  static const int resident = [] {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_boxcar<T, OP, R, C, NT, NW>, BOX_TW * NW, 0);
    return e == hipSuccess && n > 0 ? n : 1;
  }();
  constexpr int cols = BOX_TW * C * NW;
  a.nbx = (a.W + cols - 1) / cols;
  a.strip = box_strip(a, R, NW, resident);
  const int64_t nby = (a.H + a.strip - 1) / a.strip;
  hipLaunchKernelGGL((k_boxcar<T, OP, R, C, NT, NW>), dim3((unsigned)(a.nbx * nby)), dim3(BOX_TW * NW), 0, s, a);
  return hipGetLastError();
}

// Waves per block, side by side in the same strip and kept in step by a barrier
// a row, where rows do not start on lines: the line two waves share then is
// whole in the cache before it is evicted, and memory sees no partial writes
// (with Z, 256 waves of an XCD write 1.2 MB a row into its 4 MB of cache).
// 2999x3001, us at 1, 4 and 8 waves: FP32 7x7 with Z 277, 249, 222, without 182,
// 186, 185; FP32 3x3 with Z 248, 220, 204, without 142, 132, 142.  Outputs that
// fit in the 256 MB memory-side cache do not need it (1001x999, 7x7 with Z: 34.6,
// 35.8, 36.7; 450x600, 3x3 with Z: 17.9, 17.8, 21.0).
// A block with more than a quarter of its waves past the image's last column
// takes fewer.
template <class T, int OP, int R, int C>
hipError_t go_boxcar_c(BoxArgs& a, hipStream_t s) {
  if (box_nontemporal(a, sizeof(T))) return go_boxcar_nw<T, OP, R, C, true, 1>(a, s);
  const int64_t tiles = (a.W + BOX_TW * C - 1) / (BOX_TW * C);
  auto filled = [&](int waves) { return tiles * 4 >= (tiles + waves - 1) / waves * waves * 3; };
  const bool large = a.H * a.W * 19 * (int64_t)sizeof(T) > (int64_t)256 << 20;
  if (a.z && large && filled(8)) return go_boxcar_nw<T, OP, R, C, false, 8>(a, s);
  if (C == 2 && filled(4)) return go_boxcar_nw<T, OP, R, C, false, C == 2 ? 4 : 1>(a, s);
  return go_boxcar_nw<T, OP, R, C, false, 1>(a, s);
}

// Two columns a lane, but not where an odd tile of 64 columns would leave a
// third or more of the lanes idle (5000x64, 3x3: 14 us against 18).
template <class T, int OP, int R>
hipError_t go_boxcar_r(BoxArgs& a, hipStream_t s) {
  if constexpr (sizeof(T) == 4 && R == 1 && OP == ADJ_COMP) {
    const int64_t tiles = (a.W + BOX_TW - 1) / BOX_TW;
    if (tiles % 2 == 0 || tiles > 3) return go_boxcar_c<T, OP, R, 2>(a, s);
  }
  return go_boxcar_c<T, OP, R, 1>(a, s);
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
  // a block of at most 512 lanes takes at least 64 columns of a strip of at
  // least 4 rows: a little over 2^24 blocks, a 1-D grid
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
