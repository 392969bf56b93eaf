// Device pieces of Algorithm 2 (Sec. 4.2): the L2 flow of F_h(k * u) with
// replicate boundary conditions, driven by L-BFGS.
//
// The box field lives inside an array with one more sample on every side. The blur
// and the sweep read the nearest box voxel wherever they would read outside the
// box (BlurEdge kReplicate; the sweep's BOX form), so the margin holds no copies:
// it takes the derivatives that the sweep's stencils leave one sample outside the
// box, which are then added back onto the voxels those samples copy (folded), and
// is zero in the optimiser's vectors, which share the layout. A margin as wide as
// the blur, filled before it and folded after it, took seven more passes per
// evaluation and 13 % longer vectors at 192^3 and sigma_k = 1 (192^3 FP32 energy
// and gradient 287 -> 171 us per call).
#pragma once

#include <hip/hip_runtime.h>

#include "fe_flow.hpp"
#include "fe_kernels.hpp"

namespace fe {

struct PadBox {
  int nx, ny, nz;          // padded array
  int lo[3], hi[3];        // box [lo, hi) in x, y, z
};

// out = folded(g) at every box voxel: the gradient without a blur. Grid
// (ceil(nx ny / 256), nz) over the box.
template <typename T>
__global__ __launch_bounds__(256) void fold_shell(const T* __restrict__ g, T* __restrict__ out, FieldDims d,
                                                  EdgeBox e) {
  const unsigned q = blockIdx.x * 256u + threadIdx.x;
  if (q >= (unsigned)e.nx * (unsigned)e.ny) return;
  const unsigned y = q / (unsigned)e.nx, x = q - y * (unsigned)e.nx;
  out[e.ooff + (size_t)blockIdx.y * e.oplane + (size_t)y * e.orow + x] =
      folded(g, d, e, (int)x, (int)y, e.lo + (int)blockIdx.y);
}

// ---- vector operations of the optimiser (FP64 reductions, fixed order) ----
//
// Every reduction runs on kVecBlocks blocks of kVecThreads threads and leaves
// one FP64 partial per block in a bank of its own. The value of a reduction is
// the combination of its bank in one fixed order (bank_value), which vec_finish
// forms for the host. No block waits for another and no pass needs a device-wide
// fence, which on this GPU costs more than the pass itself when every block
// issues one.

constexpr int kVecBlocks = 256;
constexpr int kVecThreads = 1024;

template <int OP>
__device__ __forceinline__ double vec_combine(double acc, double v) {
  return OP == 2 ? fmax(acc, v) : acc + v;
}

// The value of a bank of kVecBlocks partials: lane l of the block's first wave
// combines partials l, l + 64, l + 128, l + 192 in that order, then a butterfly
// over the wave (each step combines a lane with its partner, and the two orders
// of a commutative operation agree bit for bit, so all lanes finish equal).
// The result is broadcast to the whole block; call from every thread.
template <int OP>
__device__ __forceinline__ double bank_value(const double* __restrict__ bank) {
  static_assert(kVecBlocks == 4 * 64, "bank_value reads four partials per lane");
  __shared__ double s_val;
  if (threadIdx.x < 64) {
    double a = bank[threadIdx.x];
    a = vec_combine<OP>(a, bank[threadIdx.x + 64]);
    a = vec_combine<OP>(a, bank[threadIdx.x + 128]);
    a = vec_combine<OP>(a, bank[threadIdx.x + 192]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a = vec_combine<OP>(a, __shfl_xor(a, off, 64));
    if (threadIdx.x == 0) s_val = a;
  }
  __syncthreads();
  const double v = s_val;
  __syncthreads();   // s_val may be reused by a later call
  return v;
}

// The block's combination of one value per thread into bank[blockIdx.x], in a
// fixed order (each wave's butterfly, then the waves in order).
template <int OP, int NT = kVecThreads>
__device__ __forceinline__ void vec_block_partial(double acc, double* __restrict__ bank) {
  __shared__ double s_w[NT / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc = vec_combine<OP>(acc, __shfl_xor(acc, off, 64));
  if (threadIdx.x % 64 == 0) s_w[threadIdx.x / 64] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = s_w[0];
    for (int k = 1; k < NT / 64; ++k) a = vec_combine<OP>(a, s_w[k]);
    bank[blockIdx.x] = a;
  }
}

// Consecutive vector elements of 16 bytes, moved with one load or store (the vectors
// are whole device allocations, so pack k is aligned). Two FP64 elements rather than
// four: a wave's load then takes whole lines, and the threads' shares of a vector come
// out more even (130^3: 2.1 rounds of 256 x 1024 threads with four, 4.2 with two). At
// 130^3 and 20 history vectors vec_gram then runs 440 MB in 98 us with 1024 threads
// per block; with four elements it took 124 us at its best, 256 threads.
template <typename T>
constexpr int kPack = 16 / (int)sizeof(T);

template <typename T>
struct alignas(16) Pack {
  T v[kPack<T>];
};

// bank <- partials of sum a*b (OP 0), sum |a| (OP 1) or max |a| (OP 2),
// accumulated in FP64 with one accumulator per element of a pack. Grid-stride
// over packs, two packs of each vector in flight per thread; block 0
// takes the tail.
template <typename T, int OP>
__global__ __launch_bounds__(kVecThreads) void vec_reduce(const T* __restrict__ a, const T* __restrict__ b, size_t n,
                                                          double* __restrict__ bank) {
  constexpr int P = kPack<T>;
  const size_t np = n / P, stride = (size_t)gridDim.x * blockDim.x;
  const Pack<T>* pa = reinterpret_cast<const Pack<T>*>(a);
  const Pack<T>* pb = reinterpret_cast<const Pack<T>*>(b);
  double acc[P] = {};
  for (size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < np; i0 += 2 * stride) {
    Pack<T> va[2], vb[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const size_t i = i0 + u * stride;
      va[u] = Pack<T>{};
      vb[u] = Pack<T>{};
      if (i < np) {
        va[u] = pa[i];
        if (OP == 0) vb[u] = pb[i];
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < P; ++k)
        acc[k] = vec_combine<OP>(acc[k], OP == 0 ? double(va[u].v[k]) * double(vb[u].v[k]) : fabs(double(va[u].v[k])));
  }
  if (blockIdx.x == 0 && threadIdx.x < n - P * np) {
    const size_t j = P * np + threadIdx.x;
    acc[0] = vec_combine<OP>(acc[0], OP == 0 ? double(a[j]) * double(b[j]) : fabs(double(a[j])));
  }
  double v = vec_combine<OP>(acc[0], acc[1]);
  if constexpr (P == 4) v = vec_combine<OP>(v, vec_combine<OP>(acc[2], acc[3]));
  vec_block_partial<OP>(v, bank);
}

// ---- the L-BFGS direction through Gram matrices ----
//
// The two-loop recursion only ever combines the history vectors s_i, y_i and
// the gradient g linearly, and its scalars are inner products of those
// vectors. So the host runs the recursion on the inner products (FP64, kept
// up to date as pairs enter and leave the history) and the device makes two
// passes per iteration: vec_gram forms the new pair and every inner product
// the recursion needs, vec_lincomb forms the direction from the coefficients.

constexpr int kDotVecs = 24;    // history vectors per vec_gram pass (all of them up to history 12)
constexpr int kCombVecs = 24;   // vectors per vec_lincomb pass (all 2m + 1 of them up to history 11)

template <typename T>
struct DotList {
  const T* v[kDotVecs];
  int count;
};

template <typename T>
struct CombList {
  const T* v[kCombVecs];
  double c[kCombVecs];
  int count;
};

// The partials of NV values per block, each in a fixed order (the wave's
// butterfly, then the waves in order), into bank k * kVecBlocks + blockIdx.x.
template <int NV, int NT>
__device__ __forceinline__ void vec_block_partials(double (&acc)[NV], int nv, double* __restrict__ banks) {
  __shared__ double s_w[NV][NT / 64];
  // every value takes the butterfly (fixed trip counts keep acc in registers)
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double a = acc[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
    if (threadIdx.x % 64 == 0) s_w[k][threadIdx.x / 64] = a;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < nv; k += NT) {
    double a = s_w[k][0];
    for (int wv = 1; wv < NT / 64; ++wv) a += s_w[k][wv];
    banks[(size_t)k * kVecBlocks + blockIdx.x] = a;
  }
}

// One pass of the Gram update. FORM: first y = g - prev_g and s = t d, stored,
// the banks 0..4 get y.y, y.s, y.g, g.g, g.s (NB = 5; otherwise NB = 0) and the
// bank `gmax` max |g|.
// The first NL list vectors V_k then give g.V_k in bank NB + k. The products
// of y with the history need no pass of their own: y.V = g.V - prev_g.V, and
// the host kept prev_g.V from the previous pass. All NL list entries are read
// (the host points unused ones at g, and only the first `count` reach the
// banks), so the loops have fixed trip counts and every value stays in
// registers. FP64 accumulation, block 0 takes the tail.
// Grid: kVecBlocks blocks of kVecThreads.
template <typename T, bool FORM, int NL>
__global__ __launch_bounds__(kVecThreads) void vec_gram(const T* __restrict__ g, const T* __restrict__ prev_g,
                                                              const T* __restrict__ d, double t, T* __restrict__ y,
                                                              T* __restrict__ s, DotList<T> L, size_t n,
                                                              double* __restrict__ banks, double* __restrict__ gmax) {
  static_assert(NL >= 0 && NL <= kDotVecs && (FORM || NL > 0), "vec_gram list width");
  constexpr int NB = FORM ? 5 : 0;
  constexpr int NV = NB + NL;
  const T tt = T(t);
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  T mx = T(0);
  constexpr int P = kPack<T>;
  const size_t np = n / P, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < np; i += stride) {
    const Pack<T> pg = reinterpret_cast<const Pack<T>*>(g)[i];
    if constexpr (FORM) {
      const Pack<T> pp = reinterpret_cast<const Pack<T>*>(prev_g)[i];
      const Pack<T> pd = reinterpret_cast<const Pack<T>*>(d)[i];
      Pack<T> py, ps;
#pragma unroll
      for (int e = 0; e < P; ++e) {
        py.v[e] = pg.v[e] - pp.v[e];
        ps.v[e] = tt * pd.v[e];
      }
      reinterpret_cast<Pack<T>*>(y)[i] = py;
      reinterpret_cast<Pack<T>*>(s)[i] = ps;
#pragma unroll
      for (int e = 0; e < P; ++e) {
        const double ye = py.v[e], ge = pg.v[e], se = ps.v[e];
        acc[0] += ye * ye;
        acc[1] += ye * se;
        acc[2] += ye * ge;
        acc[3] += ge * ge;
        acc[4] += ge * se;
        mx = fmax(mx, fabs(pg.v[e]));
      }
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const Pack<T> pv = reinterpret_cast<const Pack<T>*>(L.v[k])[i];
#pragma unroll
      for (int e = 0; e < P; ++e) acc[NB + k] += double(pg.v[e]) * double(pv.v[e]);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < n - P * np) {
    const size_t j = P * np + threadIdx.x;
    const double ge = g[j];
    if constexpr (FORM) {
      const T yt = g[j] - prev_g[j], st = tt * d[j];
      y[j] = yt;
      s[j] = st;
      const double ye = yt, se = st;
      acc[0] += ye * ye;
      acc[1] += ye * se;
      acc[2] += ye * ge;
      acc[3] += ge * ge;
      acc[4] += ge * se;
      mx = fmax(mx, fabs(g[j]));
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) acc[NB + k] += ge * double(L.v[k][j]);
  }
  vec_block_partials<NV, kVecThreads>(acc, NB + L.count, banks);
  if constexpr (FORM) vec_block_partial<2, kVecThreads>(double(mx), gmax);
}

// out = sum_k c_k V_k (+ out when acc), accumulated in FP64 and rounded once;
// when dmax is given, its bank gets the partials of max |out|; when x is
// given, x += t out (FP64, rounded once) with the rounded out, which is the
// optimiser's step folded into the pass that forms its direction. All W list
// entries are read (the host pads a short list with zero coefficients on a
// listed vector), so the loop has a fixed trip count. Layout of the work as in
// vec_reduce, but from the end: the last packs of the history are those that the
// Gram pass before it read last, and part of them is still in the memory-side cache
// (130^3 FP64, 21 vectors: 77 us; from the start 88).
template <typename T, int W>
__global__ __launch_bounds__(kVecThreads) void vec_lincomb(CombList<T> L, T* __restrict__ out, int acc, size_t n,
                                                           double* __restrict__ dmax, T* __restrict__ x, double t) {
  static_assert(W >= 1 && W <= kCombVecs, "vec_lincomb width");
  constexpr int P = kPack<T>;
  const size_t np = n / P, stride = (size_t)gridDim.x * blockDim.x;
  double mx = 0.0;
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < np; q += stride) {
    const size_t i = np - 1 - q;
    double a[P] = {};
    if (acc) {
      const Pack<T> po = reinterpret_cast<const Pack<T>*>(out)[i];
#pragma unroll
      for (int e = 0; e < P; ++e) a[e] = double(po.v[e]);
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const Pack<T> pv = reinterpret_cast<const Pack<T>*>(L.v[k])[i];
#pragma unroll
      for (int e = 0; e < P; ++e) a[e] += L.c[k] * double(pv.v[e]);
    }
    Pack<T> r;
#pragma unroll
    for (int e = 0; e < P; ++e) {
      r.v[e] = T(a[e]);
      mx = fmax(mx, fabs(double(r.v[e])));
    }
    reinterpret_cast<Pack<T>*>(out)[i] = r;
    if (x) {
      Pack<T> px = reinterpret_cast<const Pack<T>*>(x)[i];
#pragma unroll
      for (int e = 0; e < P; ++e) px.v[e] = T(double(px.v[e]) + t * double(r.v[e]));
      reinterpret_cast<Pack<T>*>(x)[i] = px;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < n - P * np) {
    const size_t j = P * np + threadIdx.x;
    double a = acc ? double(out[j]) : 0.0;
#pragma unroll
    for (int k = 0; k < W; ++k) a += L.c[k] * double(L.v[k][j]);
    const T r = T(a);
    out[j] = r;
    mx = fmax(mx, fabs(double(r)));
    if (x) x[j] = T(double(x[j]) + t * double(r));
  }
  if (dmax) vec_block_partial<2>(mx, dmax);
}

// Values of consecutive banks for the host: out[k] = bank_value(bank k), a maximum
// for the banks whose bit is set in `maxima` (the first 32), else a sum. Grid: one
// block of 64 per bank.
__global__ __launch_bounds__(64) void vec_finish(const double* __restrict__ banks, double* __restrict__ out,
                                                 unsigned maxima) {
  const unsigned k = blockIdx.x;
  const double* bank = banks + (size_t)k * kVecBlocks;
  const double v = k < 32 && (maxima >> k & 1u) ? bank_value<2>(bank) : bank_value<0>(bank);
  if (threadIdx.x == 0) out[k] = v;
}

// Copy between the box of a padded array and a dense box field [nz][ny][nx]: four
// voxels of a plane per thread, 256 apart, all loaded before the first is stored.
// Grid (ceil(nx ny / 1024), nz) over the box.
template <typename T>
__global__ __launch_bounds__(256) void box_copy(const T* __restrict__ src, T* __restrict__ dst, PadBox b,
                                                int to_padded) {
  constexpr int U = 4;
  const unsigned bx = b.hi[0] - b.lo[0], by = b.hi[1] - b.lo[1], n = bx * by;
  const size_t dz = (size_t)blockIdx.y * n;
  const size_t pz = ((size_t)(blockIdx.y + b.lo[2]) * b.ny + b.lo[1]) * b.nx + b.lo[0];
  const unsigned q0 = blockIdx.x * (256u * U) + threadIdx.x;
  T v[U];
  size_t p[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned q = q0 + 256u * u, y = q / bx;
    p[u] = pz + (size_t)y * b.nx + (q - y * bx);
    if (q < n) v[u] = to_padded ? src[dz + q] : src[p[u]];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned q = q0 + 256u * u;
    if (q < n) dst[to_padded ? p[u] : dz + q] = v[u];
  }
}

}  // namespace fe
