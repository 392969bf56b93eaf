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
// the combination of its bank in one fixed order (bank_value), formed where it
// is needed: by every block of a later vector pass that takes it as a
// coefficient, or by vec_finish for the host. No block waits for another and
// no pass needs a device-wide fence, which on this GPU costs more than the
// pass itself when every block issues one.

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
template <int OP>
__device__ __forceinline__ void vec_block_partial(double acc, double* __restrict__ bank) {
  __shared__ double s_w[kVecThreads / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc = vec_combine<OP>(acc, __shfl_xor(acc, off, 64));
  if (threadIdx.x % 64 == 0) s_w[threadIdx.x / 64] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = s_w[0];
    for (int k = 1; k < kVecThreads / 64; ++k) a = vec_combine<OP>(a, s_w[k]);
    bank[blockIdx.x] = a;
  }
}

// Four consecutive vector elements, moved with 16-byte loads and stores (the
// vectors are whole device allocations, so element 4k is 16-byte aligned).
template <typename T>
struct alignas(16) Pack4 {
  T v[4];
};

// bank <- partials of sum a*b (OP 0), sum |a| (OP 1) or max |a| (OP 2),
// accumulated in FP64 with one accumulator per element of a pack. Grid-stride
// over packs of four, two packs of each vector in flight per thread; block 0
// takes the n % 4 tail.
template <typename T, int OP>
__global__ __launch_bounds__(kVecThreads) void vec_reduce(const T* __restrict__ a, const T* __restrict__ b, size_t n,
                                                          double* __restrict__ bank) {
  const size_t n4 = n / 4, stride = (size_t)gridDim.x * blockDim.x;
  const Pack4<T>* pa = reinterpret_cast<const Pack4<T>*>(a);
  const Pack4<T>* pb = reinterpret_cast<const Pack4<T>*>(b);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n4; i0 += 2 * stride) {
    Pack4<T> va[2], vb[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const size_t i = i0 + u * stride;
      va[u] = Pack4<T>{};
      vb[u] = Pack4<T>{};
      if (i < n4) {
        va[u] = pa[i];
        if (OP == 0) vb[u] = pb[i];
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        acc[k] = vec_combine<OP>(acc[k], OP == 0 ? double(va[u].v[k]) * double(vb[u].v[k]) : fabs(double(va[u].v[k])));
  }
  if (blockIdx.x == 0 && threadIdx.x < n - 4 * n4) {
    const size_t j = 4 * n4 + threadIdx.x;
    acc[0] = vec_combine<OP>(acc[0], OP == 0 ? double(a[j]) * double(b[j]) : fabs(double(a[j])));
  }
  vec_block_partial<OP>(vec_combine<OP>(vec_combine<OP>(acc[0], acc[1]), vec_combine<OP>(acc[2], acc[3])), bank);
}

// ---- the L-BFGS direction through Gram matrices ----
//
// The two-loop recursion only ever combines the history vectors s_i, y_i and
// the gradient g linearly, and its scalars are inner products of those
// vectors. So the host runs the recursion on the inner products (FP64, kept
// up to date as pairs enter and leave the history) and the device makes two
// passes per iteration: vec_gram forms the new pair and every inner product
// the recursion needs, vec_lincomb forms the direction from the coefficients.

// Threads per vec_gram block: a full block for FP32; a quarter for FP64, whose
// accumulators and packs need twice the registers.
template <typename T>
constexpr int gram_threads() { return sizeof(T) == 4 ? kVecThreads : kVecThreads / 4; }
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
// and the banks 0..4 get y.y, y.s, y.g, g.g, g.s (NB = 5; otherwise NB = 0).
// The first NL list vectors V_k then give g.V_k in bank NB + k. The products
// of y with the history need no pass of their own: y.V = g.V - prev_g.V, and
// the host kept prev_g.V from the previous pass. All NL list entries are read
// (the host points unused ones at g, and only the first `count` reach the
// banks), so the loops have fixed trip counts and every value stays in
// registers. FP64 accumulation, packs of four, block 0 takes the n % 4 tail.
// Grid: kVecBlocks blocks of gram_threads<T>().
template <typename T, bool FORM, int NL>
__global__ __launch_bounds__(gram_threads<T>()) void vec_gram(const T* __restrict__ g, const T* __restrict__ prev_g,
                                                              const T* __restrict__ d, double t, T* __restrict__ y,
                                                              T* __restrict__ s, DotList<T> L, size_t n,
                                                              double* __restrict__ banks) {
  static_assert(NL >= 0 && NL <= kDotVecs && (FORM || NL > 0), "vec_gram list width");
  constexpr int NB = FORM ? 5 : 0;
  constexpr int NV = NB + NL;
  const T tt = T(t);
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  const size_t n4 = n / 4, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
    const Pack4<T> pg = reinterpret_cast<const Pack4<T>*>(g)[i];
    if constexpr (FORM) {
      const Pack4<T> pp = reinterpret_cast<const Pack4<T>*>(prev_g)[i];
      const Pack4<T> pd = reinterpret_cast<const Pack4<T>*>(d)[i];
      Pack4<T> py, ps;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        py.v[e] = pg.v[e] - pp.v[e];
        ps.v[e] = tt * pd.v[e];
      }
      reinterpret_cast<Pack4<T>*>(y)[i] = py;
      reinterpret_cast<Pack4<T>*>(s)[i] = ps;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double ye = py.v[e], ge = pg.v[e], se = ps.v[e];
        acc[0] += ye * ye;
        acc[1] += ye * se;
        acc[2] += ye * ge;
        acc[3] += ge * ge;
        acc[4] += ge * se;
      }
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const Pack4<T> pv = reinterpret_cast<const Pack4<T>*>(L.v[k])[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[NB + k] += double(pg.v[e]) * double(pv.v[e]);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < n - 4 * n4) {
    const size_t j = 4 * n4 + threadIdx.x;
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
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) acc[NB + k] += ge * double(L.v[k][j]);
  }
  vec_block_partials<NV, gram_threads<T>()>(acc, NB + L.count, banks);
}

// out = sum_k c_k V_k (+ out when acc), accumulated in FP64 and rounded once;
// when dmax is given, its bank gets the partials of max |out|; when x is
// given, x += t out (FP64, rounded once) with the rounded out, which is the
// optimiser's step folded into the pass that forms its direction. All W list
// entries are read (the host pads a short list with zero coefficients on a
// listed vector), so the loop has a fixed trip count. Layout of the work as in
// vec_reduce.
template <typename T, int W>
__global__ __launch_bounds__(kVecThreads) void vec_lincomb(CombList<T> L, T* __restrict__ out, int acc, size_t n,
                                                           double* __restrict__ dmax, T* __restrict__ x, double t) {
  static_assert(W >= 1 && W <= kCombVecs, "vec_lincomb width");
  const size_t n4 = n / 4, stride = (size_t)gridDim.x * blockDim.x;
  double mx = 0.0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    if (acc) {
      const Pack4<T> po = reinterpret_cast<const Pack4<T>*>(out)[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = double(po.v[e]);
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const Pack4<T> pv = reinterpret_cast<const Pack4<T>*>(L.v[k])[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += L.c[k] * double(pv.v[e]);
    }
    Pack4<T> r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      r.v[e] = T(a[e]);
      mx = fmax(mx, fabs(double(r.v[e])));
    }
    reinterpret_cast<Pack4<T>*>(out)[i] = r;
    if (x) {
      Pack4<T> px = reinterpret_cast<const Pack4<T>*>(x)[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) px.v[e] = T(double(px.v[e]) + t * double(r.v[e]));
      reinterpret_cast<Pack4<T>*>(x)[i] = px;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < n - 4 * n4) {
    const size_t j = 4 * n4 + threadIdx.x;
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

// Values of `count` consecutive sum banks: out[k] = bank_value<0>(bank k).
// Grid: count blocks of 64.
__global__ __launch_bounds__(64) void vec_finish_sums(const double* __restrict__ banks, double* __restrict__ out) {
  const double v = bank_value<0>(banks + (size_t)blockIdx.x * kVecBlocks);
  if (threadIdx.x == 0) out[blockIdx.x] = v;
}

// Values of up to four banks for the host: out[k] = bank_value<op[k]>(bank[k]).
struct BankList {
  const double* bank[4];
  double* out[4];
  int op[4];
  int count;
};

__global__ __launch_bounds__(64) void vec_finish(BankList l) {
  for (int k = 0; k < l.count; ++k) {
    const double v = l.op[k] == 2 ? bank_value<2>(l.bank[k]) : bank_value<0>(l.bank[k]);
    if (threadIdx.x == 0) *l.out[k] = v;
  }
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
