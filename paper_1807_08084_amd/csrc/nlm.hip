// Nonlocal-means filtering of a PolSAR covariance image with stochastic
// distances between Wishart laws, the consumer the Introduction motivates:
// every pixel compares its covariance with each pixel of a (2r+1)^2 search
// window, which needs the inverse (symmetrized Kullback-Leibler distance) or
// the determinant (Bhattacharyya distance) of every covariance, and the
// filtered covariance is the weighted mean
//     out_p = sum_q w_pq Z_q / sum_q w_pq,   w_pq = exp(-d(Z_p, Z_q) / h).
// Distances between complex Wishart laws of N looks (Frery, Nascimento and
// Cintra, IEEE Trans. Geosci. Remote Sens. 52(2), 2014; the Sigma-free
// terms cancel):
//   KL: d = N/2 (tr(Z_p^-1 Z_q) + tr(Z_q^-1 Z_p)) - 3N
//   B:  d = N (ln det((Z_p + Z_q)/2) - (ln det Z_p + ln det Z_q)/2)
// with tr(AB) = a_A a_B + d_A d_B + f_A f_B + 2 (Re/Im products of b, c, e)
// for Hermitian A, B, and det of the pair mean by the row-0 real-part
// expansion (Eq. detr).  Windows are clipped at the image border.
//
// A wave owns TW columns of G output rows, a lane one column of them.  It
// walks down the G + 2r input rows its outputs' windows cover: a row's TW + 2r
// columns (covariance, and what the distance needs beside it) are staged in
// LDS, and every lane then sweeps its 2r + 1 neighbours there, each neighbour
// read once for the lane's G outputs.  Where an image has too few tiles to fill
// the chip, the S waves of a block share one tile: each takes a run of its
// input rows, and their sums are added in row order at the end.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "../../include/polsar.h"
#include "common.hpp"
#include "nlm_shape.hpp"

namespace {
using polsar_dev::wave_sync;
using polsar_dev::xcd_tile;

constexpr int TW = 64, MAX_R = 16;

struct NlmArgs {
  const void* z;
  int64_t zp;
  const void* aux;  // KL: 9 inverse planes; B: det plane
  int64_t ap;
  void* out;
  int64_t op;
  void* wsum;
  int64_t H, W;
  int r;
  double n_looks, h;
};

template <class T> __device__ __forceinline__ T exp2_(T x);
// FP32: the hardware's base-2 exponential (within 1 ulp; results below the
// normal range flush, which only drops weights under 2^-126 of the largest)
template <> __device__ __forceinline__ float exp2_(float x) { return __builtin_amdgcn_exp2f(x); }
template <> __device__ __forceinline__ double exp2_(double x) { return exp2(x); }
template <class T> __device__ __forceinline__ T log2_(T x);
// (log2f, not the bare hardware logarithm: determinants of images with tiny
// entries can be subnormal, which log2f scales first)
template <> __device__ __forceinline__ float log2_(float x) { return log2f(x); }
template <> __device__ __forceinline__ double log2_(double x) { return log2(x); }

// DIST 0: symmetrized Kullback-Leibler, one chain of 18 FMAs over Z and Z^-1
// of both pixels.  DIST 1: Bhattacharyya, the determinant of the pair's sum by
// the sum's own cofactors of row 0, in the storage type.
//
// Bound by VALU issue: two waves of a SIMD issue FP32 operations in
// alternation, so a neighbour costs about 2.5 cycles per operation and wave
// against 30 (KL) operations, an exponential (8 cycles) and its share of the
// LDS reads, 20 words in five 128-bit reads over the lane's G outputs.  G
// outputs per lane divide the LDS reads and the rows staged per output by G;
// single-wave tiles need no barrier.  KL in FP32, 2048x2048, r = 11: 1.61 ms
// at G = 3 (127 registers, four waves per SIMD), 1.74 at G = 2, 2.12 at G = 1,
// 1.96 at G = 4 (two waves), against 2.18 ms for four-wave blocks over a ring
// of rows with two columns per lane.  FP32 matrix instructions (4x4x1) for
// both contractions gave the same bits at 2.40 ms: they share the vector
// units' rate.
template <class T, int DIST, int G, int S>
__global__ __launch_bounds__(TW * S) void k_nlm(NlmArgs a) {
  // staged values per pixel: Z, then Z^-1 (KL) or the logarithm of det Z (B);
  // and the features an output keeps
  constexpr int F = DIST == 0 ? 18 : 10, NP = DIST == 0 ? 18 : 9;
  constexpr bool BARE = DIST == 1 && std::is_same<T, float>::value;  // the hardware's logarithm, below
  constexpr int E = 16 / sizeof(T), FQ = (F + E - 1) / E;  // values per 16-byte LDS access
  typedef T VT __attribute__((ext_vector_type(E)));
  // a compile-time row length keeps every access at a fixed offset from one
  // address per lane; afterwards a band holds its wave's sums
  constexpr int BW = TW + 2 * MAX_R;
  constexpr int BAND = FQ * BW * E > 10 * G * TW ? FQ * BW * E : 10 * G * TW;
  __shared__ __align__(16) T bands[S][BAND];
  const T* __restrict__ Z = (const T*)a.z;
  const T* __restrict__ A = (const T*)a.aux;
  const int lane = threadIdx.x % TW, part = threadIdx.x / TW;
  VT* band = (VT*)bands[part];
  const unsigned tile = xcd_tile((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x,
                                 gridDim.x * gridDim.y * gridDim.z);
  const int64_t x0 = (int64_t)(tile % gridDim.x) * TW, y0 = (int64_t)(tile / gridDim.x) * G;
  if (y0 >= a.H) return;  // the grid's rows past the last tile row
  const int64_t px = x0 + lane;
  const int r = a.r, nc = TW + 2 * r;
  const T N = (T)a.n_looks;
  const T log2e = (T)1.4426950408889634;
  // w = exp2(alpha * s + beta): KL s = the two traces; B s = log2 det(Zp + Zq) - (lp + lq)/2
  const T alpha = DIST == 0 ? -N * log2e / (T(2) * (T)a.h) : -N / (T)a.h;
  const T beta = DIST == 0 ? T(3) * N * log2e / (T)a.h : T(3) * N / (T)a.h;

  // the outputs' features: KL: Z_p with the off-diagonal doubled (for
  // tr(Q^-1 P)), then Z_p^-1 likewise; B: Z_p, and log2 det Z_p in lp
  T P[G][NP], lp[G], acc[G][9], ws[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    ws[g] = lp[g] = T(0);
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[g][k] = T(0);
#pragma unroll
    for (int k = 0; k < NP; ++k) P[g][k] = T(0);
    if (px < a.W && y0 + g < a.H) {
      const int64_t i = (y0 + g) * a.W + px;
#pragma unroll
      for (int k = 0; k < 9; ++k) P[g][k] = Z[k * a.zp + i] * (DIST == 1 || k < 3 ? T(1) : T(2));
      if constexpr (DIST == 0) {
#pragma unroll
        for (int k = 0; k < 9; ++k) P[g][9 + k] = A[k * a.ap + i] * (k < 3 ? T(1) : T(2));
      } else {
        lp[g] = log2_(A[i]);
      }
    }
  }
  // this lane's window of staged columns, clipped at the image's sides; none
  // past the last column
  int dlo = px < r ? r - (int)px : 0;
  const int64_t right = a.W - 1 - px;
  int dhi = right < r ? (int)right + r : 2 * r;
  if (px >= a.W) { dlo = 1; dhi = 0; }
  const bool inner = x0 >= r && x0 + TW - 1 + r < a.W;  // no lane's window is clipped

  auto read = [&](int col, T (&q)[F]) {
#pragma unroll
    for (int k = 0; k < FQ; ++k) {
      const VT v = band[k * BW + col];
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (k * E + e < F) q[k * E + e < F ? k * E + e : 0] = v[e];
    }
  };
  // the distance's sum over the pair's components
  auto score = [&](int g, const T (&q)[F]) -> T {
    if constexpr (DIST == 0) {
      T tt = P[g][9] * q[0];
      tt = fma(q[9], P[g][0], tt);
#pragma unroll
      for (int k = 1; k < 9; ++k) {
        tt = fma(P[g][9 + k], q[k], tt);
        tt = fma(q[9 + k], P[g][k], tt);
      }
      return tt;
    } else {
      T mm[9], cf[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) mm[k] = P[g][k] + q[k];
      px::cofactors_plain(mm, cf);
      return px::det_from_cofactors(mm, cf);
    }
  };
  // tt: the score, in FP32 B its logarithm
  auto accumulate = [&](int g, T tt, const T (&q)[F]) {
    T w;
    if constexpr (DIST == 0) w = exp2_(alpha * tt + beta);
    else w = exp2_(alpha * ((BARE ? tt : log2_(tt)) - T(0.5) * (lp[g] + q[9])) + beta);
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[g][k] += w * q[k];
    ws[g] += w;
  };
  // A neighbour against the outputs [lo, hi].  log2f is the hardware's
  // logarithm but for subnormal numbers, which it scales first: 5 operations a
  // pair that are left to waves that meet one (B, FP32, with the inverse before
  // it: 2048x2048, r = 7: 1086 -> 1061 us; 450x600, r = 5: 54 -> 50).
  auto neighbour = [&](int lo, int hi, const T (&q)[F]) {
    T tt[G];
    bool small = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      tt[g] = score(g, q);
      if constexpr (BARE) small |= tt[g] < T(1.17549435e-38f);
    }
    if constexpr (BARE) {
      T lg[G];
#pragma unroll
      for (int g = 0; g < G; ++g) lg[g] = __builtin_amdgcn_logf(tt[g]);
      if (__builtin_expect(__any(small), 0)) {
#pragma unroll
        for (int g = 0; g < G; ++g) lg[g] = log2_(tt[g]);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) tt[g] = lg[g];
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (g >= lo && g <= hi) accumulate(g, tt[g], q);
  };

  // input row s of the tile is image row y0 - r + s; row g of the outputs has
  // it in its window while 0 <= s - g <= 2r
  const int rows = 2 * r + G;
  for (int s = part * rows / S; s < (part + 1) * rows / S; ++s) {
    const int64_t gy = y0 - r + s;
    if (gy < 0 || gy >= a.H) continue;
    wave_sync();  // the last row has been read
    for (int col = lane; col < nc; col += TW) {
      const int64_t gx = x0 - r + col;
      if (gx < 0 || gx >= a.W) continue;  // no lane reads this column
      const int64_t i = gy * a.W + gx;
      T v[FQ * E];
#pragma unroll
      for (int k = 0; k < 9; ++k) v[k] = Z[k * a.zp + i];
      if constexpr (DIST == 0) {
#pragma unroll
        for (int k = 0; k < 9; ++k) v[9 + k] = A[k * a.ap + i];
      } else {
        v[F - 1] = log2_(A[i]);
      }
#pragma unroll
      for (int k = F; k < FQ * E; ++k) v[k] = T(0);
#pragma unroll
      for (int k = 0; k < FQ; ++k) {
        VT x;
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = v[k * E + e];
        band[k * BW + col] = x;
      }
    }
    wave_sync();
    const int g_lo = s > 2 * r ? s - 2 * r : 0;
    int g_hi = s < G - 1 ? s : G - 1;
    if (y0 + g_hi >= a.H) g_hi = (int)(a.H - 1 - y0);
    if (inner && g_lo == 0 && g_hi == G - 1) {
#pragma unroll 1
      for (int d = 0; d <= 2 * r; ++d) {
        T q[F];
        read(lane + d, q);
        neighbour(0, G - 1, q);
      }
    } else {
#pragma unroll 1
      for (int d = dlo; d <= dhi; ++d) {
        T q[F];
        read(lane + d, q);
        neighbour(g_lo, g_hi, q);
      }
    }
  }

  auto store = [&](int g, const T (&sum)[9], T total) {
    const int64_t i = (y0 + g) * a.W + px;
    const T inv = T(1) / total;
#pragma unroll
    for (int k = 0; k < 9; ++k) ((T*)a.out)[k * a.op + i] = sum[k] * inv;
    if (a.wsum) ((T*)a.wsum)[i] = total;
  };
  if constexpr (S == 1) {
    if (px >= a.W) return;
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (y0 + g < a.H) store(g, acc[g], ws[g]);
  } else {
    // wave g of the block adds output row g's sums over the parts
    static_assert(S >= G, "a wave per output row");
    T* mine = bands[part];
    wave_sync();
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int k = 0; k < 9; ++k) mine[(g * 10 + k) * TW + lane] = acc[g][k];
      mine[(g * 10 + 9) * TW + lane] = ws[g];
    }
    __syncthreads();
    const int g = part;
    if (g >= G || y0 + g >= a.H || px >= a.W) return;
    T sum[9], total = bands[0][(g * 10 + 9) * TW + lane];
#pragma unroll
    for (int k = 0; k < 9; ++k) sum[k] = bands[0][(g * 10 + k) * TW + lane];
#pragma unroll
    for (int p = 1; p < S; ++p) {
#pragma unroll
      for (int k = 0; k < 9; ++k) sum[k] += bands[p][(g * 10 + k) * TW + lane];
      total += bands[p][(g * 10 + 9) * TW + lane];
    }
    store(g, sum, total);
  }
}

template <class T, int DIST, int G, int S>
void go_nlm(const NlmArgs& a, hipStream_t s) {
  // tile rows beyond a grid's 65535 go to its third dimension
  const unsigned ny = (unsigned)((a.H + G - 1) / G), nz = (ny + 65534) / 65535;
  const dim3 grid((unsigned)((a.W + TW - 1) / TW), (ny + nz - 1) / nz, nz);
  hipLaunchKernelGGL((k_nlm<T, DIST, G, S>), grid, dim3(TW * S), 0, s, a);
}

template <class T, int DIST>
void launch_nlm(const NlmArgs& a, hipStream_t s) {
  constexpr bool KL = DIST == 0;
  if constexpr (std::is_same<T, double>::value) {
    const polsar_host::NlmShape k = polsar_host::nlm_shape_f64(KL, a.H, a.W, a.r);
    if (k.rows == 1) {
      if (k.waves == 1) go_nlm<T, DIST, 1, 1>(a, s);
      else go_nlm<T, DIST, 1, 4>(a, s);
    } else if (k.waves == 8) go_nlm<T, DIST, 2, 8>(a, s);
    else if (k.waves == 4) go_nlm<T, DIST, 2, 4>(a, s);
    else go_nlm<T, DIST, 2, 1>(a, s);
  } else {
    const polsar_host::NlmShape k = polsar_host::nlm_shape(false, KL, a.H, a.W);
    if (k.waves == 8) go_nlm<T, DIST, 2, 8>(a, s);
    else if (k.waves == 4) go_nlm<T, DIST, 2, 4>(a, s);
    else go_nlm<T, DIST, KL ? 3 : 2, 1>(a, s);
  }
}

}  // namespace

extern "C" int polsar_nlm_wishart(int dtype, int distance, int64_t height, int64_t width, int radius,
                                  double n_looks, double h, const void* z, int64_t z_pitch, const void* aux,
                                  int64_t aux_pitch, void* out, int64_t out_pitch, void* wsum, void* stream) {
  if (dtype != POLSAR_F32 && dtype != POLSAR_F64) return POLSAR_E_ARG;
  if (distance != POLSAR_DIST_KL && distance != POLSAR_DIST_BHATTACHARYYA) return POLSAR_E_ARG;
  if (height < 0 || width < 0 || radius < 0 || radius > MAX_R || !(n_looks > 0.0) || !(h > 0.0))
    return POLSAR_E_ARG;
  const bool kl = distance == POLSAR_DIST_KL;
  if (width > (1 << 20) || height > (int64_t)4 * 65535) return POLSAR_E_ARG;
  const int64_t n = height * width;
  const size_t es = dtype == POLSAR_F64 ? 8 : 4;
  const int aux_planes = distance == POLSAR_DIST_KL ? 9 : 1;
  if (n == 0) return POLSAR_OK;
  if (!z || !aux || !out) return POLSAR_E_ARG;
  if (z_pitch < n || out_pitch < n || (aux_planes > 1 && aux_pitch < n)) return POLSAR_E_ARG;
  if ((uintptr_t)z % es || (uintptr_t)aux % es || (uintptr_t)out % es || (wsum && (uintptr_t)wsum % es))
    return POLSAR_E_ALIGN;
  auto lo_hi = [&](const void* p, int planes, int64_t pitch) {
    const uintptr_t lo = (uintptr_t)p;
    return std::make_pair(lo, lo + (uintptr_t)(((planes - 1) * pitch + n) * (int64_t)es));
  };
  auto ov = [](std::pair<uintptr_t, uintptr_t> x, std::pair<uintptr_t, uintptr_t> y) {
    return x.first < y.second && y.first < x.second;
  };
  const auto ro = lo_hi(out, 9, out_pitch);
  if (ov(ro, lo_hi(z, 9, z_pitch)) || ov(ro, lo_hi(aux, aux_planes, aux_pitch))) return POLSAR_E_ALIAS;
  if (wsum) {
    const auto rw = lo_hi(wsum, 1, n);
    if (ov(rw, ro) || ov(rw, lo_hi(z, 9, z_pitch)) || ov(rw, lo_hi(aux, aux_planes, aux_pitch)))
      return POLSAR_E_ALIAS;
  }
  NlmArgs a{z, z_pitch, aux, aux_pitch, out, out_pitch, wsum, height, width, radius, n_looks, h};
  hipStream_t s = (hipStream_t)stream;
  if (dtype == POLSAR_F32) {
    if (kl) launch_nlm<float, 0>(a, s);
    else launch_nlm<float, 1>(a, s);
  } else {
    if (kl) launch_nlm<double, 0>(a, s);
    else launch_nlm<double, 1>(a, s);
  }
  return hipGetLastError() == hipSuccess ? POLSAR_OK : POLSAR_E_HIP;
}
