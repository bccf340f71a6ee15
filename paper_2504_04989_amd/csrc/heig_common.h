// Shared by the kernels of the small Hermitian eigensolver: the per-slice
// scratch layout and FP64 complex arithmetic.
#pragma once

#include "common.h"

namespace tsvd {

constexpr int TRI_PMAX = 8;  // workgroups per slice of the blocked tridiagonalisation, at most

static inline size_t heig_per_slice(int m, int k) {
  (void)k;
  const size_t mp = (size_t)(m + 31) / 32 * 32;
  // A (m x m), tau (m), d and e (m each), the partial products exchanged by the
  // workgroups of a slice (2 x TRI_PMAX x mp) and their barrier counters
  size_t b = (size_t)16 * m * m + (size_t)16 * m + (size_t)16 * m;
  b = (b + 255) & ~(size_t)255;
  b += (size_t)2 * TRI_PMAX * mp * 16 + 256;
  return (b + 255) & ~(size_t)255;
}

__device__ __forceinline__ cx<double> cmulc(cx<double> a, cx<double> b) {
  return cx<double>{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// conj(a) * b
__device__ __forceinline__ cx<double> cjmul(cx<double> a, cx<double> b) {
  return cx<double>{a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re};
}

struct HeigView {
  cx<double>* A;  // m x m working matrix (global)
  cx<double>* tau;
  double* d;
  double* e;
  cx<double>* ypg;  // 2 x TRI_PMAX x mp partial products of the slice's workgroups
  unsigned* sync;   // barrier counter and abort flag of the slice's workgroups
  double* fscale;   // partial sums of ||G||_F^2 (PREP_WG of them): the fixed-point scale of the symv sums
};
__device__ __forceinline__ HeigView heig_view(unsigned char* scratch, size_t per_slice, int f, int m) {
  HeigView v;
  unsigned char* base = scratch + (size_t)f * per_slice;
  v.A = reinterpret_cast<cx<double>*>(base);
  v.tau = v.A + (size_t)m * m;
  v.d = reinterpret_cast<double*>(v.tau + m);
  v.e = v.d + m;
  const size_t off = (((size_t)16 * m * m + (size_t)32 * m) + 255) & ~(size_t)255;
  v.ypg = reinterpret_cast<cx<double>*>(base + off);
  const size_t mp = (size_t)(m + 31) / 32 * 32;
  v.sync = reinterpret_cast<unsigned*>(base + off + (size_t)2 * TRI_PMAX * mp * 16);
  v.fscale = reinterpret_cast<double*>(v.sync + 2);
  return v;
}

__device__ __forceinline__ cx<double> cadd(cx<double> a, cx<double> b) { return cx<double>{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cx<double> shfl_xor_cx(cx<double> v, int mask) {
  return cx<double>{__shfl_xor(v.re, mask, 64), __shfl_xor(v.im, mask, 64)};
}
// a += x * y
__device__ __forceinline__ void cfma(cx<double>& a, cx<double> x, cx<double> y) {
  a.re = fma(x.re, y.re, fma(-x.im, y.im, a.re));
  a.im = fma(x.re, y.im, fma(x.im, y.re, a.im));
}
// a += conj(x) * y
__device__ __forceinline__ void cfmac(cx<double>& a, cx<double> x, cx<double> y) {
  a.re = fma(x.re, y.re, fma(x.im, y.im, a.re));
  a.im = fma(x.re, y.im, fma(-x.im, y.re, a.im));
}

// tile t of the lower triangle of tiles with first tile row / column J0 (row-major order)
__device__ __forceinline__ void tri_tile(int t, int J0, int& I, int& J) {
  int a = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((a + 1) * (a + 2) / 2 <= t) ++a;
  while (a * (a + 1) / 2 > t) --a;
  J = t - a * (a + 1) / 2 + J0;
  I = a + J0;
}

// The tridiagonalisation of one slice per workgroup with the triangle in
// registers (m <= TREG_MAX); same outputs in the scratch as the other forms.
constexpr int TREG_MAX = 192;
hipError_t heig_tridiag_reg(const cx<double>* Gpart, int nsum, int64_t part_stride, int m, int batch,
                            unsigned char* scratch, size_t per_slice, int upper_only, hipStream_t s);

}  // namespace tsvd
