// Per-slice shifted Cholesky factorisation of a b x b Hermitian Gram matrix
// and the inverse of its factor, for CholeskyQR orthonormalisation of a
// Krylov block (the per-slice economy QR of Alg. TQR, used on each block of
// the Krylov basis of Alg. 2).
//
// Input: nsum FP64 partial Gram matrices (split-K products W^H W), summed in
// a fixed order (deterministic).  Output: Rinv = R^{-1}, R upper triangular
// with G + s I = R^H R, stored b x b row-major with zeros below the diagonal.
// The shift s = shift_coef * trace(G) is used on the first pass of shifted
// CholeskyQR (Fukaya et al., 2020), which keeps the factorisation defined for
// rank-deficient or ill-conditioned blocks.
//
// One 256-thread workgroup per slice.  b <= 128: one elimination with the entries in
// registers (chol_elim.h).  Wider blocks: chol_inv_kernel, threads arranged 16 x 16
// over (row, column) of the trailing triangle, the lower triangle in packed row
// order in global scratch.
#include "chol_elim.h"
#include "common.h"
#include "kernels.h"

namespace tsvd {

__device__ __forceinline__ int tri(int i, int c) { return i * (i + 1) / 2 + c; }

// mode 0: Gpart holds partial Gram matrices, factor G + shift I = R^H R.
// mode 1: Gpart holds partials of an upper triangular R (its strict lower part
//         is ignored); only the inverse is formed.
__global__ __launch_bounds__(256) void chol_inv_kernel(const cx<double>* __restrict__ Gpart, int nsum,
                                                       int64_t part_stride, cx<double>* __restrict__ Rinv,
                                                       cx<double>* gscratch, int b, double shift_coef, int* info,
                                                       int mode) {
  __shared__ cx<double> colj[1024];
  __shared__ double red[4];
  const int f = blockIdx.x;
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int64_t ntri = (int64_t)b * (b + 1) / 2;
  cx<double>* L = gscratch + (int64_t)f * ntri;
  const cx<double>* G = Gpart + (int64_t)f * b * b;

  if (mode == 1) {
    // L = R^H from the (summed) upper triangle of R
    for (int s = 0; s < nsum; ++s) {
      const cx<double>* Gs = G + s * part_stride;
      for (int i = ty; i < b; i += 16) {
        for (int c = tx; c <= i; c += 16) {
          const cx<double> r = Gs[(int64_t)c * b + i];
          cx<double> v{r.re, -r.im};
          if (s > 0) {
            const cx<double> o = L[tri(i, c)];
            v.re += o.re;
            v.im += o.im;
          }
          L[tri(i, c)] = v;
        }
      }
    }
    __syncthreads();
  } else {
  // Sum the partials into the lower triangle (partial index outermost so the
    // loads of one thread are independent), then the Hermitian average.
    for (int s = 0; s < nsum; ++s) {
      const cx<double>* Gs = G + s * part_stride;
      for (int i = ty; i < b; i += 16) {
#pragma unroll 4
        for (int c = tx; c <= i; c += 16) {
          const cx<double> g = Gs[(int64_t)i * b + c];
          const cx<double> h = Gs[(int64_t)c * b + i];
          cx<double> v{0.5 * (g.re + h.re), 0.5 * (g.im - h.im)};
          if (s > 0) {
            const cx<double> o = L[tri(i, c)];
            v.re += o.re;
            v.im += o.im;
          }
          L[tri(i, c)] = v;
        }
      }
    }
    __syncthreads();
    double tr = 0;
    for (int i = tid; i < b; i += 256) tr += L[tri(i, i)].re;
    tr = block_sum<256>(tr, red);
    const double shift = shift_coef * tr;

    // Right-looking Cholesky, lower: G + shift I = L L^H.
    int bad = 0, rescued = 0;
    for (int j = 0; j < b; ++j) {
      if (shift > 0 && !(L[tri(j, j)].re > shift)) rescued = 1;  // the shift carries this pivot
      const double dj = L[tri(j, j)].re + shift;
      double piv = 1.0;
      if (dj > 0 && isfinite(dj))
        piv = sqrt(dj);
      else
        bad = 1;  // breakdown: keep the factor invertible, report it
      const double inv = 1.0 / piv;
      for (int i = j + 1 + tid; i < b; i += 256) {
        cx<double> v = L[tri(i, j)];
        v.re *= inv;
        v.im *= inv;
        colj[i] = v;
      }
      __syncthreads();
      if (tid == 0) L[tri(j, j)] = cx<double>{piv, 0};
      // L[i][c] -= L[i][j] conj(L[c][j]) for j < c <= i; column j takes its scaled values
      for (int i = j + 1 + ty; i < b; i += 16) {
        const cx<double> a = colj[i];
        if (tx == 0) L[tri(i, j)] = a;
        for (int c = j + 1 + tx; c <= i; c += 16) {
          const cx<double> bb = colj[c];
          cx<double> v = L[tri(i, c)];
          v.re -= a.re * bb.re + a.im * bb.im;
          v.im -= a.im * bb.re - a.re * bb.im;
          L[tri(i, c)] = v;
        }
      }
      __syncthreads();
    }
    if (tid == 0 && bad) atomicAdd(&info[INFO_CHOL_BREAKDOWN], 1);
    if (tid == 0 && rescued) atomicAdd(&info[INFO_CHOL_SHIFTED], 1);
  }

  // In-place inverse of the lower factor, X = L^{-1}: forward elimination of
  // [L | I], one row of X per step; the later right-hand sides are updated
  // with the new row.
  for (int j = 0; j < b; ++j) {
    for (int i = j + 1 + tid; i < b; i += 256) colj[i] = L[tri(i, j)];
    const cx<double> djj = L[tri(j, j)];
    const double den = djj.re * djj.re + djj.im * djj.im;
    const cx<double> inv{djj.re / den, -djj.im / den};
    __syncthreads();
    for (int c = tid; c <= j; c += 256) {
      const cx<double> x = (c == j) ? cx<double>{1.0, 0.0} : L[tri(j, c)];
      L[tri(j, c)] = cx<double>{x.re * inv.re - x.im * inv.im, x.re * inv.im + x.im * inv.re};
    }
    __syncthreads();
    for (int i = j + 1 + ty; i < b; i += 16) {
      const cx<double> lij = colj[i];
      for (int c = tx; c <= j; c += 16) {
        const cx<double> x = L[tri(j, c)];
        cx<double> v = (c == j) ? cx<double>{0.0, 0.0} : L[tri(i, c)];
        v.re -= lij.re * x.re - lij.im * x.im;
        v.im -= lij.re * x.im + lij.im * x.re;
        L[tri(i, c)] = v;
      }
    }
    __syncthreads();
  }
  // R^{-1} = (L^{-1})^H, upper triangular, row-major b x b.
  cx<double>* out = Rinv + (int64_t)f * b * b;
  for (int r = ty; r < b; r += 16) {
    for (int c = tx; c < b; c += 16) {
      cx<double> v{0, 0};
      if (c >= r) {
        const cx<double> x = L[tri(c, r)];
        v = cx<double>{x.re, -x.im};
      }
      out[(int64_t)r * b + c] = v;
    }
  }
}

namespace {

// b <= 128: the elimination of chol_elim.h on the sum of the partials.
template <int NB, int MODE>
__global__ __launch_bounds__(256, 1) void chol_elim_kernel(const cx<double>* __restrict__ Gpart, int nsum,
                                                            int64_t part_stride, cx<double>* __restrict__ Rinv, int b,
                                                            double shift_coef, int* info) {
  constexpr bool TRI = MODE == 1;
  constexpr int TD = 16;
  __shared__ ElimLds<NB> lds;
  const int tid = threadIdx.x;
  const int tx = tid % TD, ty = tid / TD;  // row and column within a block
  const int f = blockIdx.x;
  const cx<double>* G = Gpart + (int64_t)f * b * b;
  cx<double> A[NB][NB];  // A[a][c], a >= c: entry (tx + TD a, ty + TD c) of the lower triangle
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int c = 0; c <= a; ++c) A[a][c] = cx<double>{0.0, 0.0};
  // (all loads of a partial in flight at once: addresses clamped, no branches)
  for (int s = 0; s < nsum; ++s) {
    const cx<double>* Gs = G + s * part_stride;
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int c = 0; c <= a; ++c) {
        const int i = min(tx + TD * a, b - 1), k = min(ty + TD * c, b - 1);
        const cx<double> u = Gs[k * b + i];  // above the diagonal (for the entries that count, i >= k)
        if (MODE == 0) {
          const cx<double> g = Gs[i * b + k];
          A[a][c].re += 0.5 * (g.re + u.re);
          A[a][c].im += 0.5 * (g.im - u.im);
        } else {
          A[a][c].re += u.re;
          A[a][c].im -= u.im;
        }
      }
  }
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int c = 0; c <= a; ++c) {
      const int i = tx + TD * a, k = ty + TD * c;
      cx<double> v = A[a][c];
      if (!TRI && i == k) v.im = 0.0;
      if (i >= b || k > i) v = cx<double>{0.0, 0.0};
      A[a][c] = v;
    }
  cx<double>* out = Rinv + (int64_t)f * b * b;
  chol_eliminate<NB, MODE>(A, b, shift_coef, lds, info, [&](int k, int i, cx<double> v) {
    if (i < b && k < b) out[(int64_t)k * b + i] = v;
  });
}

}  // namespace

bool chol_elim_ok(int64_t b) { return b <= 128; }

static hipError_t chol_inv_elim(const double* Gpart, int nsum, int64_t part_stride, double* Rinv, int b, int batch,
                                double shift_coef, int* info, hipStream_t s, int mode) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(batch), dim3(256), 0, s, (const cx<double>*)Gpart, nsum, part_stride,
                       (cx<double>*)Rinv, b, shift_coef, info);
    return hipGetLastError();
  };
  switch ((b + 15) / 16) {
#define TSVD_CHOL_CASE(n) \
  case n:                 \
    return mode == 1 ? go(chol_elim_kernel<n, 1>) : mode == 2 ? go(chol_elim_kernel<n, 2>) : go(chol_elim_kernel<n, 0>);
    TSVD_CHOL_CASE(1)
    TSVD_CHOL_CASE(2)
    TSVD_CHOL_CASE(3)
    TSVD_CHOL_CASE(4)
    TSVD_CHOL_CASE(5)
    TSVD_CHOL_CASE(6)
    TSVD_CHOL_CASE(7)
    TSVD_CHOL_CASE(8)
#undef TSVD_CHOL_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t chol_inv_ex(const double* Gpart, int nsum, int64_t part_stride, double* Rinv, void* gscratch, int b,
                       int batch, double shift_coef, int* info, hipStream_t s, int mode) {
  if (batch <= 0 || b <= 0) return hipSuccess;
  if (b > 1024) return hipErrorInvalidValue;
  if (chol_elim_ok(b)) return chol_inv_elim(Gpart, nsum, part_stride, Rinv, b, batch, shift_coef, info, s, mode);
  hipLaunchKernelGGL(chol_inv_kernel, dim3(batch), dim3(256), 0, s, (const cx<double>*)Gpart, nsum, part_stride,
                     (cx<double>*)Rinv, (cx<double>*)gscratch, b, shift_coef, info, mode);
  return hipGetLastError();
}

}  // namespace tsvd
