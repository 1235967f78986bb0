// HIP kernels and C ABI for gfx950: per-pixel 3x3 Hermitian inverse and
// determinant (Alg. 2; Alg. 1 for comparison) and the Wishart term.
//
// Every op is bandwidth-bound streaming over structure-of-arrays planes:
// one lane owns V consecutive pixels (V = 16 or 8 bytes / element size, so
// each plane access is one 128- or 64-bit global load or store), U such
// vectors per tile per lane, and a tile is block*U vectors.  A lane issues
// all of its 9*U (or 18*U) loads before any arithmetic, then all of its
// stores.  Pixels are independent; lanes share only the fixed-order
// reductions of the Wishart sum, the status counters, and the wave's LDS
// queue of FP32 pixels that the quick form leaves over.  This file also holds
// the fused multilook (per-pixel looks), block-diagonal and out-of-core
// streaming entry points.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "../../include/polsar.h"
#include "access.hpp"
#include "common.hpp"
#include "host.hpp"
#include "launch.hpp"

namespace {
using namespace polsar_dev;
using namespace polsar_host;

struct InvDetArgs {
  const void* z;
  int64_t zp;
  void* inv;
  int64_t ip;
  void* det;
  uint8_t* status;
  unsigned long long* counters;
  int64_t n;      // pixels
  int64_t nvec;   // full vectors: n / V
  int64_t tiles;  // ceil(nvec / (block * U)), at least 1
  int64_t tail;   // the block of the last tile
};

// Stores of one pixel-vector's results.
template <class T, int V, bool NT>
__device__ __forceinline__ void store_vec(const InvDetArgs& a, const T (&out)[9][V], const T (&dt)[V],
                                          const int (&st)[V], int64_t v) {
  const int64_t e = v * V;
  if (a.inv) {
    T* inv = (T*)a.inv;
#pragma unroll
    for (int k = 0; k < 9; ++k) store_v<T, V, NT>(inv + k * a.ip + e, out[k]);
  }
  if (a.det) store_v<T, V, NT>((T*)a.det + e, dt);
  if (a.status) store_status<V>(a.status + e, st);
}

// Largest dynamic LDS a launch asks for.
constexpr size_t MAX_DYN_LDS = 64 << 10;

// One pixel-vector of the inverse/determinant with the per-pixel function
// inline (every form but the FP32 compensated one of k_inv_det); the load
// is done by the caller.
template <class T, int OP, int V, bool NT>
__device__ __forceinline__ void inv_det_vec(const InvDetArgs& a, const T (&in)[9][V], int64_t v,
                                            unsigned& c0, unsigned& c1, unsigned& c2) {
  T out[9][V], dt[V];
  int st[V];
#pragma unroll
  for (int l = 0; l < V; ++l) {
    T zz[9], xx[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) zz[k] = in[k][l];
    st[l] = run_pixel<T, OP>(zz, xx, dt[l], a.status || a.counters);
#pragma unroll
    for (int k = 0; k < 9; ++k) out[k][l] = xx[k];
    tally(st[l], c0, c1, c2);
  }
  store_vec<T, V, NT>(a, out, dt, st, v);
}

// Where a kernel takes the pixels after the last full vector: inside the loop
// over tiles the compiler keeps that code's addresses and constants in
// registers throughout, 162 instead of 127 for the FP32 compensated inverse
// (V = 4), whose queue needs the waves.  The other forms stream better with
// few waves resident, and the registers hold their number down: after the
// loop, us on 4096x4096, FP64 compensated 412 (in it, 405), FP32 plain 203
// (199), wide 212 (202), compensated Cholesky 216 (204); three FP64 bands of
// 2000x2001, 344 (315).
template <class T, int OP>
constexpr bool TAIL_AFTER = OP == ADJ_COMP && std::is_same<T, float>::value;

// M: LOADS_NT | STORES_NT.
template <class T, int OP, int V, int U, int M>
__global__ __launch_bounds__(256, OP == ADJ_COMP && sizeof(T) == 4 && U == 1 ? 4 : 1) void k_inv_det(InvDetArgs a) {
  constexpr bool LNT = M & LOADS_NT, NT = M & STORES_NT;
  const T* __restrict__ z = (const T*)a.z;
  const int B = blockDim.x;
  unsigned c0 = 0, c1 = 0, c2 = 0;
  // the n mod V pixels after the last full vector
  auto tail = [&]() {
    const int64_t i = a.nvec * V + threadIdx.x;
    if (i < a.n) {
      T zz[9], xx[9], dt;
#pragma unroll
      for (int k = 0; k < 9; ++k) zz[k] = z[k * a.zp + i];
      const int st = run_pixel<T, OP>(zz, xx, dt, a.status || a.counters);
      tally(st, c0, c1, c2);
      if (a.inv)
#pragma unroll
        for (int k = 0; k < 9; ++k) ((T*)a.inv)[k * a.ip + i] = xx[k];
      if (a.det) ((T*)a.det)[i] = dt;
      if (a.status) a.status[i] = (uint8_t)st;
    }
  };
  for (int64_t tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
    const int64_t v0 = tile * (int64_t)(B * U) + threadIdx.x;
    if constexpr (OP == ADJ_COMP && std::is_same<T, float>::value) {
      // all U vectors through the quick form and one shared queue
      extern __shared__ __align__(16) float polsar_dyn_lds[];
      const int w = threadIdx.x >> 6, nw = B >> 6;
      float* q = polsar_dyn_lds + (size_t)w * 64 * U * V * QUEUE_WORDS;
      uint8_t* qs = (uint8_t*)(polsar_dyn_lds + (size_t)nw * 64 * U * V * QUEUE_WORDS) + w * 64 * U * V;
      bool valid[U];
#pragma unroll
      for (int u = 0; u < U; ++u) valid[u] = v0 + (int64_t)u * B < a.nvec;
      auto load = [&](int u, float (&in)[9][V]) {
#pragma unroll
        for (int k = 0; k < 9; ++k) load_v<float, V, LNT>(z + k * a.zp + (v0 + (int64_t)u * B) * V, in[k]);
      };
      float out[U][9][V], dt[U][V];
      int st[U][V];
      comp_f32_wave<U, V>(load, valid, out, dt, st, q, qs, a.status || a.counters);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!valid[u]) continue;
#pragma unroll
        for (int l = 0; l < V; ++l) tally(st[u][l], c0, c1, c2);
        store_vec<T, V, NT>(a, out[u], dt[u], st[u], v0 + (int64_t)u * B);
      }
    } else {
      T in[U][9][V];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t v = v0 + (int64_t)u * B;
        if (v < a.nvec) {
#pragma unroll
          for (int k = 0; k < 9; ++k) load_v<T, V, LNT>(z + k * a.zp + v * V, in[u][k]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t v = v0 + (int64_t)u * B;
        if (v < a.nvec) inv_det_vec<T, OP, V, NT>(a, in[u], v, c0, c1, c2);
      }
    }
    if (V > 1 && !TAIL_AFTER<T, OP> && tile == a.tiles - 1) tail();
  }
  if (V > 1 && TAIL_AFTER<T, OP> && blockIdx.x == a.tail) tail();
  if (a.counters) flush_counters(a.counters, c0, c1, c2);
}

// ------------------------------------------------------------------ multilook
struct MultilookArgs {
  const void* looks;
  int64_t lp;
  int n_looks;
  double inv_n;  // 1 / n_looks (FP64)
  void* z;  // optional output of the multilook covariance
  int64_t zp;
  InvDetArgs o;  // outputs (o.z unused), n, nvec, tiles
};

// Fused multilook front end + inverse/determinant: per lane V pixels, the N
// looks are streamed (6 planes each) into FP64 accumulators, scaled by 1/N
// (one FP64 multiply per component: exact for N a power of two, else within
// an FP64 rounding of the quotient, far below the storage rounding), Z is
// rounded to the storage type, optionally stored, and inverted exactly as
// k_inv_det inverts a stored Z (the FP32 compensated form through the
// wave's queue).
template <class T, int OP, int V, bool NT>
__global__ __launch_bounds__(256) void k_multilook(MultilookArgs a) {
  const T* __restrict__ S = (const T*)a.looks;
  const int B = blockDim.x;
  unsigned c0 = 0, c1 = 0, c2 = 0;
  const double inv_n = a.inv_n;
  // the n mod V pixels after the last full vector
  auto tail = [&]() {
    const int64_t i = a.o.nvec * V + threadIdx.x;
    if (i < a.o.n) {
      double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
      for (int look = 0; look < a.n_looks; ++look) {
        T s6[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) s6[j] = S[(int64_t)(6 * look + j) * a.lp + i];
        px::look_accumulate(s6, acc);
      }
      T zz[9], xx[9], dt;
#pragma unroll
      for (int k = 0; k < 9; ++k) zz[k] = (T)(acc[k] * inv_n);
      if (a.z)
#pragma unroll
        for (int k = 0; k < 9; ++k) ((T*)a.z)[k * a.zp + i] = zz[k];
      const int st = run_pixel<T, OP>(zz, xx, dt, a.o.status || a.o.counters);
      tally(st, c0, c1, c2);
      if (a.o.inv)
#pragma unroll
        for (int k = 0; k < 9; ++k) ((T*)a.o.inv)[k * a.o.ip + i] = xx[k];
      if (a.o.det) ((T*)a.o.det)[i] = dt;
      if (a.o.status) a.o.status[i] = (uint8_t)st;
    }
  };
  for (int64_t tile = blockIdx.x; tile < a.o.tiles; tile += gridDim.x) {
    const int64_t v = tile * (int64_t)B + threadIdx.x;
    if (v < a.o.nvec) {
      double acc[V][9];
#pragma unroll
      for (int l = 0; l < V; ++l)
#pragma unroll
        for (int k = 0; k < 9; ++k) acc[l][k] = 0.0;
#pragma unroll 2
      for (int look = 0; look < a.n_looks; ++look) {
        T in[6][V];
#pragma unroll
        for (int j = 0; j < 6; ++j) load_v<T, V, NT>(S + (int64_t)(6 * look + j) * a.lp + v * V, in[j]);
#pragma unroll
        for (int l = 0; l < V; ++l) {
          const T s6[6] = {in[0][l], in[1][l], in[2][l], in[3][l], in[4][l], in[5][l]};
          px::look_accumulate(s6, acc[l]);
        }
      }
      T zz[9][V];
#pragma unroll
      for (int l = 0; l < V; ++l)
#pragma unroll
        for (int k = 0; k < 9; ++k) zz[k][l] = (T)(acc[l][k] * inv_n);
      if (a.z) {
#pragma unroll
        for (int k = 0; k < 9; ++k) store_v<T, V, NT>((T*)a.z + k * a.zp + v * V, zz[k]);
      }
      if constexpr (OP == ADJ_COMP && std::is_same<T, float>::value) {
        extern __shared__ __align__(16) float polsar_dyn_lds[];
        const int w = threadIdx.x >> 6, nw = B >> 6;
        float* q = polsar_dyn_lds + (size_t)w * 64 * V * QUEUE_WORDS;
        uint8_t* qs = (uint8_t*)(polsar_dyn_lds + (size_t)nw * 64 * V * QUEUE_WORDS) + w * 64 * V;
        const bool valid[1] = {true};
        auto load = [&](int, float (&in)[9][V]) {
#pragma unroll
          for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int l = 0; l < V; ++l) in[k][l] = zz[k][l];
        };
        float out[1][9][V], dt[1][V];
        int st[1][V];
        comp_f32_wave<1, V>(load, valid, out, dt, st, q, qs, a.o.status || a.o.counters);
#pragma unroll
        for (int l = 0; l < V; ++l) tally(st[0][l], c0, c1, c2);
        store_vec<T, V, NT>(a.o, out[0], dt[0], st[0], v);
      } else {
        inv_det_vec<T, OP, V, NT>(a.o, zz, v, c0, c1, c2);
      }
    }
    if (V > 1 && !TAIL_AFTER<T, OP> && tile == a.o.tiles - 1) tail();
  }
  if (V > 1 && TAIL_AFTER<T, OP> && blockIdx.x == a.o.tail) tail();
  if (a.o.counters) flush_counters(a.o.counters, c0, c1, c2);
}

// ------------------------------------------------------------------ block diagonal
// Pixels whose matrix is block diagonal with K Hermitian 3x3 blocks (several
// frequency bands): each block is inverted on its own, the determinant is the
// product of the block determinants, the status the worst block status.
struct BlockArgs {
  int k;            // blocks per pixel
  void* bdet;       // optional per-block determinants: K planes, pitch bp
  int64_t bp;
  InvDetArgs o;     // z: 9K planes (block b at planes 9b..9b+8), inv likewise
};

template <class T, int OP, int V, bool NT>
__global__ __launch_bounds__(256) void k_blockdiag(BlockArgs a) {
  const T* __restrict__ Z = (const T*)a.o.z;
  const int B = blockDim.x;
  unsigned c0 = 0, c1 = 0, c2 = 0;
  for (int64_t tile = blockIdx.x; tile < a.o.tiles; tile += gridDim.x) {
    const int64_t v = tile * (int64_t)B + threadIdx.x;
    if (v < a.o.nvec) {
      T prod[V];
      int worst[V];
#pragma unroll
      for (int l = 0; l < V; ++l) { prod[l] = T(1); worst[l] = 0; }
      for (int b = 0; b < a.k; ++b) {
        T in[9][V], out[9][V], dt[V];
#pragma unroll
        for (int k = 0; k < 9; ++k) load_v<T, V, NT>(Z + (int64_t)(9 * b + k) * a.o.zp + v * V, in[k]);
#pragma unroll
        for (int l = 0; l < V; ++l) {
          T zz[9], xx[9];
#pragma unroll
          for (int k = 0; k < 9; ++k) zz[k] = in[k][l];
          const int st = run_pixel<T, OP>(zz, xx, dt[l], a.o.status || a.o.counters);
#pragma unroll
          for (int k = 0; k < 9; ++k) out[k][l] = xx[k];
          prod[l] *= dt[l];
          worst[l] = st > worst[l] ? st : worst[l];
        }
        if (a.o.inv)
#pragma unroll
          for (int k = 0; k < 9; ++k) store_v<T, V, NT>((T*)a.o.inv + (int64_t)(9 * b + k) * a.o.ip + v * V, out[k]);
        if (a.bdet) store_v<T, V, NT>((T*)a.bdet + (int64_t)b * a.bp + v * V, dt);
      }
#pragma unroll
      for (int l = 0; l < V; ++l) tally(worst[l], c0, c1, c2);
      if (a.o.det) store_v<T, V, NT>((T*)a.o.det + v * V, prod);
      if (a.o.status) store_status<V>(a.o.status + v * V, worst);
    }
    if (V > 1 && tile == a.o.tiles - 1) {
      const int64_t i = a.o.nvec * V + threadIdx.x;
      if (i < a.o.n) {
        T prod = T(1);
        int worst = 0;
        for (int b = 0; b < a.k; ++b) {
          T zz[9], xx[9], dt;
#pragma unroll
          for (int k = 0; k < 9; ++k) zz[k] = Z[(int64_t)(9 * b + k) * a.o.zp + i];
          const int st = run_pixel<T, OP>(zz, xx, dt, a.o.status || a.o.counters);
          prod *= dt;
          worst = st > worst ? st : worst;
          if (a.o.inv)
#pragma unroll
            for (int k = 0; k < 9; ++k) ((T*)a.o.inv)[(int64_t)(9 * b + k) * a.o.ip + i] = xx[k];
          if (a.bdet) ((T*)a.bdet)[(int64_t)b * a.bp + i] = dt;
        }
        tally(worst, c0, c1, c2);
        if (a.o.det) ((T*)a.o.det)[i] = prod;
        if (a.o.status) a.o.status[i] = (uint8_t)worst;
      }
    }
  }
  if (a.o.counters) flush_counters(a.o.counters, c0, c1, c2);
}

// ------------------------------------------------------------------ Wishart
struct WishartArgs {
  const void* s;
  int64_t sp;
  const void* z;
  int64_t zp;
  double n_looks;
  void* ell;
  double* partial;  // one FP64 partial sum per tile (forward)
  const double* grad_loss;
  void* grad;
  int64_t gp;
  unsigned long long* counters;
  int64_t n, nvec, tiles;
  int fwd, bwd;
};

template <class T, int V, bool NT>
__device__ __forceinline__ double wishart_vec(const WishartArgs& a, const T (&s)[9][V], const T (&z)[9][V],
                                              int64_t v, T gscale, unsigned& c0, unsigned& c1, unsigned& c2) {
  T ell[V], g[9][V];
  double acc = 0.0;
#pragma unroll
  for (int l = 0; l < V; ++l) {
    T ss[9], zz[9], gg[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) { ss[k] = s[k][l]; zz[k] = z[k][l]; }
    bool low = false;
    const int st = px::wishart_pixel<T>(ss, zz, (T)a.n_looks, a.fwd, ell[l], a.bwd, gg, gscale,
                                        a.counters ? &low : nullptr);
    tally(st, c0, c1, c2);
    c1 += low;
    if (a.fwd) acc += (double)ell[l];
    if (a.bwd)
#pragma unroll
      for (int k = 0; k < 9; ++k) g[k][l] = gg[k];
  }
  const int64_t e = v * V;
  if (a.fwd && a.ell) store_v<T, V, NT>((T*)a.ell + e, ell);
  if (a.bwd) {
    T* gp = (T*)a.grad;
#pragma unroll
    for (int k = 0; k < 9; ++k) store_v<T, V, NT>(gp + k * a.gp + e, g[k]);
  }
  return acc;
}

template <class T, int V, int U, int M>
__global__ __launch_bounds__(256) void k_wishart(WishartArgs a) {
  constexpr bool LNT = M & LOADS_NT, NT = M & STORES_NT;
  const T* __restrict__ S = (const T*)a.s;
  const T* __restrict__ Z = (const T*)a.z;
  const int B = blockDim.x;
  const T gscale = a.bwd ? (a.grad_loss ? (T)*a.grad_loss : T(1)) : T(1);
  unsigned c0 = 0, c1 = 0, c2 = 0;
  for (int64_t tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
    const int64_t v0 = tile * (int64_t)(B * U) + threadIdx.x;
    T s[U][9][V], z[U][9][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t v = v0 + (int64_t)u * B;
      if (v < a.nvec) {
#pragma unroll
        for (int k = 0; k < 9; ++k) load_v<T, V, LNT>(S + k * a.sp + v * V, s[u][k]);
#pragma unroll
        for (int k = 0; k < 9; ++k) load_v<T, V, LNT>(Z + k * a.zp + v * V, z[u][k]);
      }
    }
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t v = v0 + (int64_t)u * B;
      if (v < a.nvec) acc += wishart_vec<T, V, NT>(a, s[u], z[u], v, gscale, c0, c1, c2);
    }
    if (V > 1 && tile == a.tiles - 1) {
      const int64_t i = a.nvec * V + threadIdx.x;
      if (i < a.n) {
        T ss[9], zz[9], gg[9], el;
#pragma unroll
        for (int k = 0; k < 9; ++k) { ss[k] = S[k * a.sp + i]; zz[k] = Z[k * a.zp + i]; }
        bool low = false;
        const int st = px::wishart_pixel<T>(ss, zz, (T)a.n_looks, a.fwd, el, a.bwd, gg, gscale,
                                            a.counters ? &low : nullptr);
        tally(st, c0, c1, c2);
        c1 += low;
        if (a.fwd) {
          acc += (double)el;
          if (a.ell) ((T*)a.ell)[i] = el;
        }
        if (a.bwd)
#pragma unroll
          for (int k = 0; k < 9; ++k) ((T*)a.grad)[k * a.gp + i] = gg[k];
      }
    }
    if (a.fwd) {
      const double bs = block_sum(acc);
      if (threadIdx.x == 0) a.partial[tile] = bs;
    }
  }
  if (a.counters) flush_counters(a.counters, c0, c1, c2);
}

// Fixed-order sum of `count` partials into *out (one block of REDUCE_BLOCK
// lanes: the 16,384 partials of a 2048x2048 FP32 call take one round of
// sixteen loads per lane).
__global__ __launch_bounds__(REDUCE_BLOCK) void k_reduce(const double* __restrict__ partial, int64_t count,
                                                double* __restrict__ out) {
  const double s = strided_sum(partial, count);
  if (threadIdx.x == 0) *out = s;
}

// ------------------------------------------------------------------ copy probe
// Output plane k is input plane k mod NI when there are at least as many
// outputs as inputs; with fewer outputs it is the sum of the inputs j with
// j mod NO == k, so that every input plane is read (a plane no output used
// would not be loaded at all).
template <class T, int V, int NI, int NO, bool NT>
__global__ __launch_bounds__(256) void k_copy(const T* __restrict__ src, int64_t sp, T* __restrict__ dst,
                                              int64_t dp, int64_t nvec, int64_t n) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < nvec) {
    T in[NI][V];
#pragma unroll
    for (int k = 0; k < NI; ++k) load_v<T, V, NT>(src + k * sp + v * V, in[k]);
    if constexpr (NI > NO) {
#pragma unroll
      for (int j = NO; j < NI; ++j)
#pragma unroll
        for (int l = 0; l < V; ++l) in[j % NO][l] += in[j][l];
    }
#pragma unroll
    for (int k = 0; k < NO; ++k) store_v<T, V, NT>(dst + k * dp + v * V, in[k % NI]);
  }
  if (blockIdx.x == 0) {
    const int64_t i = nvec * V + threadIdx.x;
    if (i < n)
      for (int k = 0; k < NO; ++k) {
        T x = src[(k % NI) * sp + i];
        for (int j = k + NO; j < NI; j += NO) x += src[j * sp + i];
        dst[k * dp + i] = x;
      }
  }
}

// ------------------------------------------------------------------ host side
LaunchTable g_table;

// Dynamic LDS bytes for a launch: what the kernel needs, raised so that at
// most blocks_per_cu blocks fit in a compute unit's LDS.
int lds_per_cu() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 160 << 10;
  if (!cached[dev]) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess || v <= 0)
      v = 160 << 10;
    cached[dev] = v;
  }
  return cached[dev];
}

size_t launch_lds(const polsar_launch& c, size_t need) {
  if (c.blocks_per_cu <= 0) return need;
  size_t pad = (size_t)lds_per_cu() / (size_t)(c.blocks_per_cu + 1) + 1024;
  pad = std::min<size_t>(pad, MAX_DYN_LDS);
  return std::max(need, pad);
}

int device_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int cu = 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0) cu = 256;
    cached[dev] = cu;
  }
  return cached[dev];
}

// Blocks of a launch over `tiles` tiles: the launch's persistent grid, or
// one block per tile, and at most COUNTER_GRID_PER_CU blocks per CU when the
// call asks for counters.  Pixels are independent and the Wishart partial
// sums are kept per tile, so results do not depend on the grid.
int64_t launch_grid(const polsar_launch& c, int64_t tiles, bool counters) {
  int gpc = c.grid_per_cu;
  if (counters && (gpc == 0 || gpc > COUNTER_GRID_PER_CU)) gpc = COUNTER_GRID_PER_CU;
  int64_t grid = tiles;
  if (gpc > 0) grid = std::min<int64_t>(grid, (int64_t)gpc * device_cus());
  return grid;
}

// Launch helpers: pick the template instance for (V, U, accesses).
template <class T, int OP, int V, int U>
hipError_t go_inv_det(const polsar_launch& c, int64_t grid, InvDetArgs& a, hipStream_t s) {
  const size_t lds =
      launch_lds(c, (OP == ADJ_COMP && std::is_same<T, float>::value) ? comp_queue_bytes(c.block, U * V) : 0);
  const dim3 g((unsigned)grid), b(c.block);
  switch (c.nontemporal ? inv_det_access(a.n, sizeof(T), off_lines(a.z, a.zp, sizeof(T))) : 0) {
    case 0: hipLaunchKernelGGL((k_inv_det<T, OP, V, U, 0>), g, b, lds, s, a); break;
    case STORES_NT: hipLaunchKernelGGL((k_inv_det<T, OP, V, U, STORES_NT>), g, b, lds, s, a); break;
    default: hipLaunchKernelGGL((k_inv_det<T, OP, V, U, LOADS_NT | STORES_NT>), g, b, lds, s, a); break;
  }
  return hipGetLastError();
}

// Vectors per lane per tile actually used: the compensated FP32 kernel
// takes at most two (four run out of registers), and one where the block's
// shared queue for two would pass MAX_DYN_LDS.
template <class T, int OP, int V>
int inv_det_unroll(const polsar_launch& c) {
  if constexpr (OP == ADJ_COMP && std::is_same<T, float>::value) {
    const int u = c.unroll > 2 ? 2 : c.unroll;
    return (u == 2 && comp_queue_bytes(c.block, 2 * V) > MAX_DYN_LDS) ? 1 : u;
  } else {
    return c.unroll;
  }
}

template <class T, int OP, int V>
hipError_t dispatch_inv_det_v(const polsar_launch& c, InvDetArgs& a, hipStream_t s) {
  a.nvec = a.n / V;
  const int unroll = inv_det_unroll<T, OP, V>(c);
  const int64_t per_tile = (int64_t)c.block * unroll;
  a.tiles = std::max<int64_t>(1, (a.nvec + per_tile - 1) / per_tile);
  const int64_t grid = launch_grid(c, a.tiles, a.counters != nullptr);
  a.tail = (a.tiles - 1) % grid;
  if (unroll == 1) return go_inv_det<T, OP, V, 1>(c, grid, a, s);
  if constexpr (OP == ADJ_COMP && std::is_same<T, float>::value) {
    return go_inv_det<T, OP, V, 2>(c, grid, a, s);
  } else {
    if (unroll == 2) return go_inv_det<T, OP, V, 2>(c, grid, a, s);
    return go_inv_det<T, OP, V, 4>(c, grid, a, s);
  }
}

// Access width: 16 bytes per lane per plane (V = 16 / sizeof(T) pixels),
// 8 bytes when the launch asks for it.
template <class T, int OP>
hipError_t dispatch_inv_det(const polsar_launch& c, InvDetArgs& a, hipStream_t s) {
  constexpr int VW = 16 / sizeof(T);
  if (c.vector_bytes == 8) return dispatch_inv_det_v<T, OP, VW / 2>(c, a, s);
  return dispatch_inv_det_v<T, OP, VW>(c, a, s);
}

hipError_t launch_inv_det(int dtype, int op, const polsar_launch& c, InvDetArgs& a, hipStream_t s) {
  if (dtype == POLSAR_F32) {
    switch (op) {
      case ADJ_PLAIN: return dispatch_inv_det<float, ADJ_PLAIN>(c, a, s);
      case ADJ_COMP: return dispatch_inv_det<float, ADJ_COMP>(c, a, s);
      case ADJ_WIDE: return dispatch_inv_det<float, ADJ_WIDE>(c, a, s);
      case CHOL_PLAIN: return dispatch_inv_det<float, CHOL_PLAIN>(c, a, s);
      case CHOL_COMP: return dispatch_inv_det<float, CHOL_COMP>(c, a, s);
      default: return dispatch_inv_det<float, CHOL_WIDE>(c, a, s);
    }
  }
  switch (op) {
    case ADJ_PLAIN: return dispatch_inv_det<double, ADJ_PLAIN>(c, a, s);
    case ADJ_COMP: return dispatch_inv_det<double, ADJ_COMP>(c, a, s);
    default: return dispatch_inv_det<double, CHOL_PLAIN>(c, a, s);
  }
}

// Validates polsar_inv_det arguments; fills `a` on success.
int prepare_inv_det(int dtype, int method, int prec, int64_t n, const void* z, int64_t zp, void* inv,
                    int64_t ip, void* det, uint8_t* status, unsigned long long* counters, InvDetArgs& a) {
  int r0 = check_mode(dtype, method, prec);
  if (r0) return r0;
  if (n < 0) return POLSAR_E_ARG;
  const size_t es = esize(dtype);
  int r = check_planes(z, zp, n, es);
  if (r) return r;
  if (inv && (r = check_planes(inv, ip, n, es))) return r;
  if (det && ((uintptr_t)det % es)) return POLSAR_E_ALIGN;
  if (counters && ((uintptr_t)counters % 8)) return POLSAR_E_ALIGN;
  if (!inv && !det && !status && !counters) return POLSAR_E_ARG;
  if (n > 0) {
    const Range rz = span(z, 9, zp, n, es);
    if (inv) {
      const Range ri = span(inv, 9, ip, n, es);
      if (!(inv == z && ip == zp) && overlap(ri, rz)) return POLSAR_E_ALIAS;
    }
    if (det) {
      const Range rd = span(det, 1, n, n, es);
      if (overlap(rd, rz) || (inv && overlap(rd, span(inv, 9, ip, n, es)))) return POLSAR_E_ALIAS;
    }
    if (status) {
      const Range rs = span(status, 1, n, n, 1);
      if (overlap(rs, rz) || (inv && overlap(rs, span(inv, 9, ip, n, es))) || (det && overlap(rs, span(det, 1, n, n, es))))
        return POLSAR_E_ALIAS;
    }
  }
  a = InvDetArgs{z, zp, inv, ip, det, status, counters, n, 0, 0, 0};
  return POLSAR_OK;
}

// ---- multilook launch
template <class T, int OP, int V>
hipError_t dispatch_multilook_v(const polsar_launch& c, MultilookArgs& a, hipStream_t s) {
  a.o.nvec = a.o.n / V;
  a.o.tiles = std::max<int64_t>(1, (a.o.nvec + c.block - 1) / c.block);
  const int64_t grid = launch_grid(c, a.o.tiles, a.o.counters != nullptr);
  a.o.tail = (a.o.tiles - 1) % grid;
  const size_t lds =
      launch_lds(c, (OP == ADJ_COMP && std::is_same<T, float>::value) ? comp_queue_bytes(c.block, V) : 0);
  if (c.nontemporal)
    hipLaunchKernelGGL((k_multilook<T, OP, V, true>), dim3((unsigned)grid), dim3(c.block), lds, s, a);
  else
    hipLaunchKernelGGL((k_multilook<T, OP, V, false>), dim3((unsigned)grid), dim3(c.block), lds, s, a);
  return hipGetLastError();
}

template <class T, int OP>
hipError_t dispatch_multilook(const polsar_launch& c, MultilookArgs& a, hipStream_t s) {
  constexpr int VW = 16 / sizeof(T);
  if (c.vector_bytes == 8) return dispatch_multilook_v<T, OP, VW / 2>(c, a, s);
  return dispatch_multilook_v<T, OP, VW>(c, a, s);
}

hipError_t launch_multilook(int dtype, int op, const polsar_launch& c, MultilookArgs& a, hipStream_t s) {
  if (dtype == POLSAR_F32) {
    switch (op) {
      case ADJ_PLAIN: return dispatch_multilook<float, ADJ_PLAIN>(c, a, s);
      case ADJ_COMP: return dispatch_multilook<float, ADJ_COMP>(c, a, s);
      case ADJ_WIDE: return dispatch_multilook<float, ADJ_WIDE>(c, a, s);
      case CHOL_PLAIN: return dispatch_multilook<float, CHOL_PLAIN>(c, a, s);
      case CHOL_COMP: return dispatch_multilook<float, CHOL_COMP>(c, a, s);
      default: return dispatch_multilook<float, CHOL_WIDE>(c, a, s);
    }
  }
  switch (op) {
    case ADJ_PLAIN: return dispatch_multilook<double, ADJ_PLAIN>(c, a, s);
    case ADJ_COMP: return dispatch_multilook<double, ADJ_COMP>(c, a, s);
    default: return dispatch_multilook<double, CHOL_PLAIN>(c, a, s);
  }
}

// ---- block-diagonal launch
template <class T, int OP, int V>
hipError_t dispatch_block_v(const polsar_launch& c, BlockArgs& a, hipStream_t s) {
  a.o.nvec = a.o.n / V;
  a.o.tiles = std::max<int64_t>(1, (a.o.nvec + c.block - 1) / c.block);
  const int64_t grid = launch_grid(c, a.o.tiles, a.o.counters != nullptr);
  const size_t lds = launch_lds(c, 0);
  if (c.nontemporal)
    hipLaunchKernelGGL((k_blockdiag<T, OP, V, true>), dim3((unsigned)grid), dim3(c.block), lds, s, a);
  else
    hipLaunchKernelGGL((k_blockdiag<T, OP, V, false>), dim3((unsigned)grid), dim3(c.block), lds, s, a);
  return hipGetLastError();
}

template <class T, int OP>
hipError_t dispatch_block(const polsar_launch& c, BlockArgs& a, hipStream_t s) {
  constexpr int VW = 16 / sizeof(T);
  return dispatch_block_v<T, OP, VW>(c, a, s);
}

hipError_t launch_block(int dtype, int op, const polsar_launch& c, BlockArgs& a, hipStream_t s) {
  if (dtype == POLSAR_F32) {
    switch (op) {
      case ADJ_PLAIN: return dispatch_block<float, ADJ_PLAIN>(c, a, s);
      case ADJ_COMP: return dispatch_block<float, ADJ_COMP>(c, a, s);
      case ADJ_WIDE: return dispatch_block<float, ADJ_WIDE>(c, a, s);
      case CHOL_PLAIN: return dispatch_block<float, CHOL_PLAIN>(c, a, s);
      case CHOL_COMP: return dispatch_block<float, CHOL_COMP>(c, a, s);
      default: return dispatch_block<float, CHOL_WIDE>(c, a, s);
    }
  }
  switch (op) {
    case ADJ_PLAIN: return dispatch_block<double, ADJ_PLAIN>(c, a, s);
    case ADJ_COMP: return dispatch_block<double, ADJ_COMP>(c, a, s);
    default: return dispatch_block<double, CHOL_PLAIN>(c, a, s);
  }
}

// ---- Wishart launch
template <class T, int V, int U>
hipError_t go_wishart(const polsar_launch& c, int64_t grid, WishartArgs& a, hipStream_t s) {
  const size_t lds = launch_lds(c, 0);
  const dim3 g((unsigned)grid), b(c.block);
  const bool off_in = off_lines(a.s, a.sp, sizeof(T)) || off_lines(a.z, a.zp, sizeof(T));
  const bool off_grad = a.bwd && off_lines(a.grad, a.gp, sizeof(T));
  switch (c.nontemporal ? wishart_access(a.n, sizeof(T), a.bwd, off_in, off_grad) : 0) {
    case 0: hipLaunchKernelGGL((k_wishart<T, V, U, 0>), g, b, lds, s, a); break;
    case STORES_NT: hipLaunchKernelGGL((k_wishart<T, V, U, STORES_NT>), g, b, lds, s, a); break;
    default: hipLaunchKernelGGL((k_wishart<T, V, U, LOADS_NT | STORES_NT>), g, b, lds, s, a); break;
  }
  return hipGetLastError();
}

// Pixels per access of a Wishart launch, and its tiles (one partial sum each).
int wishart_vector(const polsar_launch& c, size_t es) {
  const int vw = (int)(16 / es);
  return c.vector_bytes == 8 ? vw / 2 : vw;
}
int64_t wishart_tiles(const polsar_launch& c, int v, int64_t n) {
  const int64_t per_tile = (int64_t)c.block * c.unroll;
  return std::max<int64_t>(1, (n / v + per_tile - 1) / per_tile);
}

template <class T, int V>
hipError_t dispatch_wishart_v(const polsar_launch& c, WishartArgs& a, hipStream_t s) {
  a.nvec = a.n / V;
  a.tiles = wishart_tiles(c, V, a.n);
  const int64_t grid = launch_grid(c, a.tiles, a.counters != nullptr);
  return c.unroll == 1 ? go_wishart<T, V, 1>(c, grid, a, s) : go_wishart<T, V, 2>(c, grid, a, s);
}

template <class T>
hipError_t dispatch_wishart(const polsar_launch& c, WishartArgs& a, hipStream_t s) {
  constexpr int VW = 16 / sizeof(T);
  if (c.vector_bytes == 8) return dispatch_wishart_v<T, VW / 2>(c, a, s);
  return dispatch_wishart_v<T, VW>(c, a, s);
}

// Wishart partial sums (one per tile) of any launch shape: the smallest
// tile is 64 lanes x 1 vector of one element.
int64_t max_wishart_partials(int64_t n) { return std::max<int64_t>(1, (n + 63) / 64); }

}  // namespace

// The launch of a batch plan (in batch.hip); writes: inverses or gradients.
polsar_launch polsar_batch_launch(int dtype, int method, int prec, bool writes) {
  return g_table.batch(dtype, method, prec, writes);
}

// LDS bytes of a launch with this shape (shared with the batch kernel).
size_t polsar_launch_lds_bytes(const polsar_launch& c, size_t need) { return launch_lds(c, need); }

// ============================================================== C ABI
struct polsar_batch;  // defined in batch.hip

extern "C" {

const char* polsar_version(void) { return "polsar-mi355x 0.1 (gfx950)"; }

int64_t polsar_recommended_pitch(int dtype, int64_t n) {
  if ((dtype != POLSAR_F32 && dtype != POLSAR_F64) || n < 0) return -1;
  const int64_t es = (int64_t)esize(dtype);
  const int64_t blk = (64 << 10) / es, half = (32 << 10) / es;
  return (n + blk - 1) / blk * blk + half;
}

const char* polsar_status_string(int status) {
  switch (status) {
    case POLSAR_OK: return "ok";
    case POLSAR_E_ARG: return "invalid argument";
    case POLSAR_E_ALIGN: return "misaligned pointer";
    case POLSAR_E_UNSUPPORTED: return "unsupported combination";
    case POLSAR_E_HIP: return "HIP runtime error";
    case POLSAR_E_WORKSPACE: return "workspace missing or too small";
    case POLSAR_E_ALIAS: return "outputs overlap inputs";
    default: return "unknown status";
  }
}

int polsar_device_compute_units(int* cus) {
  if (!cus) return POLSAR_E_ARG;
  *cus = device_cus();
  return POLSAR_OK;
}

int polsar_wishart_launch_op(int64_t n) { return wishart_op(n); }

int polsar_inv_det_launch_op(int64_t n) { return inv_det_op(n); }

int polsar_get_launch(int op, int dtype, int method, int precision, polsar_launch* out) {
  if (!out || op < 0 || op > 6) return POLSAR_E_ARG;
  *out = g_table.get(op, dtype, method, precision);
  return POLSAR_OK;
}

int polsar_set_launch(int op, int dtype, int method, int precision, const polsar_launch* cfg) {
  if (!cfg || op < 0 || op > 6 || !valid_launch(*cfg, op)) return POLSAR_E_ARG;
  g_table.set(op, dtype, method, precision, *cfg);
  return POLSAR_OK;
}

int polsar_inv_det(int dtype, int method, int precision, int64_t n, const void* z, int64_t z_pitch, void* inv,
                   int64_t inv_pitch, void* det, uint8_t* status, unsigned long long* counters, void* stream) {
  InvDetArgs a;
  int r = prepare_inv_det(dtype, method, precision, n, z, z_pitch, inv, inv_pitch, det, status, counters, a);
  if (r) return r;
  if (n == 0) return POLSAR_OK;
  const polsar_launch c = g_table.inv_det(n, dtype, method, precision, status || counters);
  if (launch_inv_det(dtype, op_code(method, precision), c, a, (hipStream_t)stream) != hipSuccess)
    return POLSAR_E_HIP;
  return POLSAR_OK;
}

int polsar_multilook_inv_det(int dtype, int method, int precision, int64_t n, int n_looks, const void* looks,
                             int64_t looks_pitch, void* z, int64_t z_pitch, void* inv, int64_t inv_pitch,
                             void* det, uint8_t* status, unsigned long long* counters, void* stream) {
  int r = check_mode(dtype, method, precision);
  if (r) return r;
  if (n < 0 || n_looks < 1 || n_looks > 4096) return POLSAR_E_ARG;
  const size_t es = esize(dtype);
  if ((r = check_planes(looks, looks_pitch, n, es))) return r;
  if (z && (r = check_planes(z, z_pitch, n, es))) return r;
  if (inv && (r = check_planes(inv, inv_pitch, n, es))) return r;
  if (det && ((uintptr_t)det % es)) return POLSAR_E_ALIGN;
  if (counters && ((uintptr_t)counters % 8)) return POLSAR_E_ALIGN;
  if (!z && !inv && !det && !status && !counters) return POLSAR_E_ARG;
  if (n > 0) {
    const Range rl = span(looks, 6 * n_looks, looks_pitch, n, es);
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
  MultilookArgs a{looks, looks_pitch, n_looks, 1.0 / n_looks, z, z_pitch,
                  InvDetArgs{nullptr, 0, inv, inv_pitch, det, status, counters, n, 0, 0, 0}};
  const polsar_launch c = g_table.multilook(dtype, method, precision, n_looks, z != nullptr);
  if (launch_multilook(dtype, op_code(method, precision), c, a, (hipStream_t)stream) != hipSuccess)
    return POLSAR_E_HIP;
  return POLSAR_OK;
}

int polsar_blockdiag_inv_det(int dtype, int method, int precision, int64_t n, int n_blocks, const void* z,
                             int64_t z_pitch, void* inv, int64_t inv_pitch, void* det, void* block_det,
                             int64_t block_det_pitch, uint8_t* status, unsigned long long* counters, void* stream) {
  int r = check_mode(dtype, method, precision);
  if (r) return r;
  if (n < 0 || n_blocks < 1 || n_blocks > 1024) return POLSAR_E_ARG;
  const size_t es = esize(dtype);
  if ((r = check_planes(z, z_pitch, n, es))) return r;
  if (inv && (r = check_planes(inv, inv_pitch, n, es))) return r;
  if (block_det && (r = check_planes(block_det, block_det_pitch, n, es))) return r;
  if (det && ((uintptr_t)det % es)) return POLSAR_E_ALIGN;
  if (counters && ((uintptr_t)counters % 8)) return POLSAR_E_ALIGN;
  if (!inv && !det && !block_det && !status && !counters) return POLSAR_E_ARG;
  if (n > 0) {
    const int P = 9 * n_blocks;
    const Range rz = span(z, P, z_pitch, n, es);
    const Range ri = inv ? span(inv, P, inv_pitch, n, es) : Range{0, 0};
    const Range rd = det ? span(det, 1, n, n, es) : Range{0, 0};
    const Range rb = block_det ? span(block_det, n_blocks, block_det_pitch, n, es) : Range{0, 0};
    const Range rs = status ? span(status, 1, n, n, 1) : Range{0, 0};
    const Range all[5] = {rz, ri, rd, rb, rs};
    for (int p = 0; p < 5; ++p)
      for (int q = p + 1; q < 5; ++q) {
        if (p == 0 && q == 1 && inv == z && inv_pitch == z_pitch) continue;  // in place
        if (all[p].hi > all[p].lo && all[q].hi > all[q].lo && overlap(all[p], all[q])) return POLSAR_E_ALIAS;
      }
  }
  if (n == 0) return POLSAR_OK;
  BlockArgs a{n_blocks, block_det, block_det_pitch, InvDetArgs{z, z_pitch, inv, inv_pitch, det, status, counters, n, 0, 0, 0}};
  const polsar_launch c = g_table.get(0, dtype, method, precision);
  if (launch_block(dtype, op_code(method, precision), c, a, (hipStream_t)stream) != hipSuccess) return POLSAR_E_HIP;
  return POLSAR_OK;
}

size_t polsar_wishart_workspace_bytes(int dtype, int64_t n) {
  if (n < 0) return 0;
  (void)dtype;  // the partials are FP64 for either storage type
  return (size_t)max_wishart_partials(n) * sizeof(double);
}

}  // extern "C"

// polsar_wishart_loglik and its allocation-free variant: validation and
// launch with the per-tile partial sums at `ws` (ws_words words of 8 bytes):
// the caller's workspace (its size is checked against the largest tile count
// of any launch), or, when fixed_ws is given, the library's fixed scratch of
// ws_words words (checked against this launch's tile count), whose device
// address fixed_ws returns once every argument has passed validation.
int polsar_wishart_call(int dtype, int pass, int64_t n, const void* sigma, int64_t s_pitch, const void* z,
                        int64_t z_pitch, double n_looks, double* loss, void* ell, const double* grad_loss, void* grad,
                        int64_t g_pitch, double* ws, int64_t ws_words, int (*fixed_ws)(double**),
                        unsigned long long* counters, void* stream) {
  const bool ws_user = fixed_ws == nullptr;
  if (dtype != POLSAR_F32 && dtype != POLSAR_F64) return POLSAR_E_ARG;
  if (pass != POLSAR_FWD && pass != POLSAR_BWD && pass != POLSAR_FWD_BWD) return POLSAR_E_ARG;
  if (n < 0 || !(n_looks > 0.0)) return POLSAR_E_ARG;
  const bool fwd = pass & POLSAR_FWD, bwd = pass & POLSAR_BWD;
  const size_t es = esize(dtype);
  int r = check_planes(sigma, s_pitch, n, es);
  if (r) return r;
  if ((r = check_planes(z, z_pitch, n, es))) return r;
  if (fwd && !loss) return POLSAR_E_ARG;
  if (loss && ((uintptr_t)loss % 8)) return POLSAR_E_ALIGN;
  if (grad_loss && ((uintptr_t)grad_loss % 8)) return POLSAR_E_ALIGN;
  if (ell && ((uintptr_t)ell % es)) return POLSAR_E_ALIGN;
  if (counters && ((uintptr_t)counters % 8)) return POLSAR_E_ALIGN;
  if (bwd && (r = check_planes(grad, g_pitch, n, es))) return r;
  if (fwd && n > 0 && ws_user) {
    if (!ws || ws_words < max_wishart_partials(n)) return POLSAR_E_WORKSPACE;
    if ((uintptr_t)ws % 8) return POLSAR_E_ALIGN;
  }
  if (n > 0) {
    const Range rs = span(sigma, 9, s_pitch, n, es), rz = span(z, 9, z_pitch, n, es);
    if (bwd) {
      const Range rg = span(grad, 9, g_pitch, n, es);
      if (overlap(rg, rs) || overlap(rg, rz)) return POLSAR_E_ALIAS;
    }
    if (fwd && ell) {
      const Range re = span(ell, 1, n, n, es);
      if (overlap(re, rs) || overlap(re, rz) || (bwd && overlap(re, span(grad, 9, g_pitch, n, es))))
        return POLSAR_E_ALIAS;
    }
  }
  const polsar_launch c = g_table.wishart(n, dtype, bwd);
  if (fwd && n > 0 && !ws_user) {
    if (wishart_tiles(c, wishart_vector(c, es), n) > ws_words) return POLSAR_E_WORKSPACE;
    if ((r = fixed_ws(&ws))) return r;
  }
  hipStream_t s = (hipStream_t)stream;
  if (n == 0) {
    if (fwd) {
      // an empty sum is zero: reduce zero partials
      hipLaunchKernelGGL(k_reduce, dim3(1), dim3(REDUCE_BLOCK), 0, s, (const double*)nullptr, (int64_t)0, loss);
      if (hipGetLastError() != hipSuccess) return POLSAR_E_HIP;
    }
    return POLSAR_OK;
  }
  WishartArgs a{sigma, s_pitch, z, z_pitch, n_looks, fwd ? ell : nullptr, fwd ? ws : nullptr, grad_loss,
                bwd ? grad : nullptr, g_pitch, counters, n, 0, 0, fwd ? 1 : 0, bwd ? 1 : 0};
  hipError_t e = dtype == POLSAR_F32 ? dispatch_wishart<float>(c, a, s) : dispatch_wishart<double>(c, a, s);
  if (e != hipSuccess) return POLSAR_E_HIP;
  if (fwd) {
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(REDUCE_BLOCK), 0, s, (const double*)ws, a.tiles, loss);
    if (hipGetLastError() != hipSuccess) return POLSAR_E_HIP;
  }
  return POLSAR_OK;
}

extern "C" {

int polsar_wishart_loglik(int dtype, int pass, int64_t n, const void* sigma, int64_t s_pitch, const void* z,
                          int64_t z_pitch, double n_looks, double* loss, void* ell, const double* grad_loss,
                          void* grad, int64_t g_pitch, void* workspace, size_t ws_bytes,
                          unsigned long long* counters, void* stream) {
  return polsar_wishart_call(dtype, pass, n, sigma, s_pitch, z, z_pitch, n_looks, loss, ell, grad_loss, grad, g_pitch,
                      (double*)workspace, (int64_t)(ws_bytes / sizeof(double)), nullptr, counters, stream);
}

int polsar_autotune_inv_det(int dtype, int method, int precision, int64_t n, const void* z, int64_t z_pitch,
                            void* inv, int64_t inv_pitch, void* det, int reps, polsar_launch* best,
                            float* best_ms, void* stream) {
  InvDetArgs a;
  int r = prepare_inv_det(dtype, method, precision, n, z, z_pitch, inv, inv_pitch, det, nullptr, nullptr, a);
  if (r) return r;
  if (n == 0 || reps <= 0) return POLSAR_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return POLSAR_E_HIP;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return POLSAR_E_HIP;
  }
  const int op = op_code(method, precision);
  polsar_launch win{0, 0, 0, 0, 0, 0};
  float win_ms = 1e30f;
  int rc = POLSAR_OK;
  // mean time per call of `reps` back-to-back calls with launch c, after one
  // untimed call; negative on a HIP error
  auto time_cfg = [&](const polsar_launch& c) -> float {
    InvDetArgs aa = a;
    if (launch_inv_det(dtype, op, c, aa, s) != hipSuccess) return -1.f;
    (void)hipEventRecord(e0, s);
    for (int i = 0; i < reps; ++i) {
      aa = a;
      (void)launch_inv_det(dtype, op, c, aa, s);
    }
    (void)hipEventRecord(e1, s);
    if (hipEventSynchronize(e1) != hipSuccess) return -1.f;
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    return ms / reps;
  };
  // Stage 1, every candidate once: block x unroll x {one tile per block,
  // 8 blocks per CU persistent} x access width x resident-block cap, with
  // streaming accesses.  Stage 2: the six fastest again, in three
  // interleaved passes, ranked by their best pass (single timings of
  // neighbouring candidates differ by a few percent from run to run).
  std::vector<std::pair<float, polsar_launch>> all;
  for (int block : {64, 128, 256})
    for (int unroll : {1, 2})
      for (int gpc : {0, 8})
        for (int vb : {16, 8})
          for (int bpc : {0, 2, 3, 4, 5, 6, 8}) {
            const polsar_launch c{block, unroll, gpc, 1, vb, bpc};
            const float ms = time_cfg(c);
            if (ms < 0.f) { rc = POLSAR_E_HIP; goto done; }
            all.emplace_back(ms, c);
          }
  std::sort(all.begin(), all.end(), [](const auto& x, const auto& y) { return x.first < y.first; });
  all.resize(std::min<size_t>(all.size(), 6));
  for (auto& e : all) e.first = 1e30f;
  for (int pass = 0; pass < 3; ++pass)
    for (auto& e : all) {
      const float ms = time_cfg(e.second);
      if (ms < 0.f) { rc = POLSAR_E_HIP; goto done; }
      e.first = std::min(e.first, ms);
    }
  for (const auto& e : all)
    if (e.first < win_ms) { win_ms = e.first; win = e.second; }
  g_table.set(inv_det_op(n), dtype, method, precision, win);
  if (best) *best = win;
  if (best_ms) *best_ms = win_ms;
done:
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return rc;
}

int polsar_stream_copy(int dtype, int64_t n, const void* src, int64_t src_pitch, int n_in, void* dst,
                       int64_t dst_pitch, int n_out, void* stream) {
  if (dtype != POLSAR_F32 && dtype != POLSAR_F64) return POLSAR_E_ARG;
  if (n < 0) return POLSAR_E_ARG;
  const size_t es = esize(dtype);
  int r = check_planes(src, src_pitch, n, es);
  if (r) return r;
  if ((r = check_planes(dst, dst_pitch, n, es))) return r;
  const bool shape_ok = (n_in == 9 && n_out == 10) || (n_in == 18 && n_out == 9) || (n_in == 18 && n_out == 19) ||
                        (n_in == 24 && n_out == 10) || (n_in == 27 && n_out == 28) || (n_in == 1 && n_out == 1);
  if (!shape_ok) return POLSAR_E_UNSUPPORTED;
  if (!vec_ok(src, src_pitch, es) || !vec_ok(dst, dst_pitch, es)) return POLSAR_E_ALIGN;
  if (n > 0 && overlap(span(src, n_in, src_pitch, n, es), span(dst, n_out, dst_pitch, n, es))) return POLSAR_E_ALIAS;
  if (n == 0) return POLSAR_OK;
  hipStream_t s = (hipStream_t)stream;
  // launch shape: op 4 of the table (block, access width, non-temporal,
  // resident-block cap); one vector per lane, one tile per block
  const polsar_launch c = g_table.get(4, dtype, 0, 0);
  const int VW = (int)(c.vector_bytes / es);
  const int64_t nvec = n / VW;
  const int64_t grid = std::max<int64_t>(1, (nvec + c.block - 1) / c.block);
  const size_t lds = launch_lds(c, 0);
#define POLSAR_COPY(T, V, NI, NO)                                                                              \
  do {                                                                                                        \
    if (c.nontemporal)                                                                                        \
      hipLaunchKernelGGL((k_copy<T, V, NI, NO, true>), dim3((unsigned)grid), dim3(c.block), lds, s,           \
                         (const T*)src, src_pitch, (T*)dst, dst_pitch, nvec, n);                              \
    else                                                                                                      \
      hipLaunchKernelGGL((k_copy<T, V, NI, NO, false>), dim3((unsigned)grid), dim3(c.block), lds, s,          \
                         (const T*)src, src_pitch, (T*)dst, dst_pitch, nvec, n);                              \
  } while (0)
#define POLSAR_COPY_V(T, V)                                                                                    \
  do {                                                                                                        \
    if (n_in == 9) POLSAR_COPY(T, V, 9, 10);                                                                  \
    else if (n_in == 18 && n_out == 9) POLSAR_COPY(T, V, 18, 9);                                              \
    else if (n_in == 18) POLSAR_COPY(T, V, 18, 19);                                                           \
    else if (n_in == 24) POLSAR_COPY(T, V, 24, 10);                                                           \
    else if (n_in == 27) POLSAR_COPY(T, V, 27, 28);                                                           \
    else POLSAR_COPY(T, V, 1, 1);                                                                             \
  } while (0)
  if (dtype == POLSAR_F32) {
    if (VW == 4) POLSAR_COPY_V(float, 4);
    else POLSAR_COPY_V(float, 2);
  } else {
    if (VW == 2) POLSAR_COPY_V(double, 2);
    else POLSAR_COPY_V(double, 1);
  }
#undef POLSAR_COPY_V
#undef POLSAR_COPY
  return hipGetLastError() == hipSuccess ? POLSAR_OK : POLSAR_E_HIP;
}


// ------------------------------------------------------------------ out-of-core streaming
// Host-resident images (larger than device memory, or simply on the host):
// the pixels are cut into chunks; chunk i uses device buffer set i % 2 and
// stream i % 2: one 2-D copy of its 9 input plane segments host -> device,
// the inverse kernel, and 2-D copies of the 9 inverse planes, the det and
// the status segments back.  Work on the two streams overlaps, so the copy
// of one chunk runs while the other is computed.
}  // extern "C"

struct polsar_streamer {
  int dtype, method, precision;
  int64_t chunk, pitch;  // device plane pitch (elements) of each buffer set
  void* dz[2];
  void* dout[2];  // 9 inverse planes + det plane
  uint8_t* dst[2];
  hipStream_t st[2];
};

namespace {
void streamer_release(polsar_streamer* s) {
  if (!s) return;
  for (int b = 0; b < 2; ++b) {
    if (s->st[b]) (void)hipStreamDestroy(s->st[b]);
    if (s->dz[b]) (void)hipFree(s->dz[b]);
    if (s->dout[b]) (void)hipFree(s->dout[b]);
    if (s->dst[b]) (void)hipFree(s->dst[b]);
  }
  delete s;
}
}  // namespace

extern "C" {

int polsar_streamer_create(int dtype, int method, int precision, int64_t chunk_pixels, polsar_streamer** out) {
  if (!out) return POLSAR_E_ARG;
  *out = nullptr;
  int r = check_mode(dtype, method, precision);
  if (r) return r;
  if (chunk_pixels < 1 || chunk_pixels > ((int64_t)1 << 34)) return POLSAR_E_ARG;
  polsar_streamer* s = new polsar_streamer();
  s->dtype = dtype;
  s->method = method;
  s->precision = precision;
  s->chunk = chunk_pixels;
  s->pitch = polsar_recommended_pitch(dtype, chunk_pixels);
  const size_t es = esize(dtype);
  for (int b = 0; b < 2; ++b) {
    if (hipMalloc(&s->dz[b], 9 * s->pitch * es) != hipSuccess || hipMalloc(&s->dout[b], 10 * s->pitch * es) != hipSuccess ||
        hipMalloc((void**)&s->dst[b], (size_t)chunk_pixels) != hipSuccess ||
        hipStreamCreateWithFlags(&s->st[b], hipStreamNonBlocking) != hipSuccess) {
      streamer_release(s);
      return POLSAR_E_HIP;
    }
  }
  *out = s;
  return POLSAR_OK;
}

int polsar_streamer_run(polsar_streamer* s, int64_t n, const void* z, int64_t z_pitch, void* inv, int64_t inv_pitch,
                        void* det, uint8_t* status, unsigned long long* counters) {
  if (!s) return POLSAR_E_ARG;
  if (n < 0) return POLSAR_E_ARG;
  const size_t es = esize(s->dtype);
  int r = check_planes(z, z_pitch, n, es);
  if (r) return r;
  if (inv && (r = check_planes(inv, inv_pitch, n, es))) return r;
  if (det && ((uintptr_t)det % es)) return POLSAR_E_ALIGN;
  if (!inv && !det && !status && !counters) return POLSAR_E_ARG;
  if (counters && ((uintptr_t)counters % 8)) return POLSAR_E_ALIGN;
  if (n > 0) {
    const Range rz = span(z, 9, z_pitch, n, es);
    if (inv && overlap(span(inv, 9, inv_pitch, n, es), rz)) return POLSAR_E_ALIAS;
    if (det && overlap(span(det, 1, n, n, es), rz)) return POLSAR_E_ALIAS;
  }
  const polsar_launch c = g_table.inv_det(s->chunk, s->dtype, s->method, s->precision, status || counters);
  const int op = op_code(s->method, s->precision);
  const size_t P = (size_t)s->pitch * es;
  hipError_t e = hipSuccess;
  for (int64_t off = 0, i = 0; off < n && e == hipSuccess; off += s->chunk, ++i) {
    const int b = (int)(i & 1);
    const int64_t m = std::min<int64_t>(s->chunk, n - off);
    hipStream_t st = s->st[b];
    const size_t w = (size_t)m * es;
    e = hipMemcpy2DAsync(s->dz[b], P, (const char*)z + off * es, (size_t)z_pitch * es, w, 9, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) break;
    InvDetArgs a{s->dz[b], s->pitch, inv ? s->dout[b] : nullptr, s->pitch,
                 det ? (char*)s->dout[b] + 9 * P : nullptr, status ? s->dst[b] : nullptr, counters, m, 0, 0, 0};
    e = launch_inv_det(s->dtype, op, c, a, st);
    if (e != hipSuccess) break;
    if (inv) e = hipMemcpy2DAsync((char*)inv + off * es, (size_t)inv_pitch * es, s->dout[b], P, w, 9, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && det) e = hipMemcpyAsync((char*)det + off * es, (char*)s->dout[b] + 9 * P, w, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && status) e = hipMemcpyAsync(status + off, s->dst[b], (size_t)m, hipMemcpyDeviceToHost, st);
  }
  const hipError_t e0 = hipStreamSynchronize(s->st[0]);
  const hipError_t e1 = hipStreamSynchronize(s->st[1]);
  return (e == hipSuccess && e0 == hipSuccess && e1 == hipSuccess) ? POLSAR_OK : POLSAR_E_HIP;
}

void polsar_streamer_destroy(polsar_streamer* s) { streamer_release(s); }

}  // extern "C"
