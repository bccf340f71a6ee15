// Cholesky factorisation and inverse of one b x b matrix, b <= 128, by a 256-thread
// workgroup with the entries in registers (the block Grams of CholeskyQR).
#pragma once

#include "common.h"

// b <= 128: factorisation and inverse in one elimination, entries in registers.
// Step j of the right-looking elimination of [G | I] updates every row i > j,
//   A(i, c) -= l_i r_c / d,  l_i = A(i, j),  d = A(j, j),
// with r_c = conj(l_c) for c > j (the rest of G) and r_c = A(j, c) for c < j (the
// rows of L^{-1} so far, in place of the finished columns of G); column j itself
// becomes -l_i / d.  Row j of L^{-1} is A(j, :) / sqrt(d), scaled at the end, so a
// step needs one reciprocal.  mode 1 (inverse of a given triangle): r_c = 0 for
// c > j and d = L(j, j).
// Bound: latency, b steps of one barrier, an LDS round trip, the reciprocal and
// the update (a workgroup per slice; the slices are far fewer than the CUs).  The
// 16 x 16 threads hold the entries (tx + 16 a, ty + 16 c), a >= c, cyclically, so
// the trailing rows stay spread over all of them; one wave per SIMD keeps the
// work that every wave repeats (reciprocal, operand reads) off the others' issue
// slots (32 x 32 threads took 129 us at b = 110).  The blocked form before it (16 x
// 16 tiles, the diagonal tiles in one wave) took 15, 53, 73 and 153 us at b = 10 (9
// slices), 40 (101), 60 (17) and 110 (33); this one 9, 30, 42 and 105 us.
namespace tsvd {

template <int NB>
struct ElimLds {
  cx<double> lv[2][16 * NB], rv[2][16 * NB];  // l and r of the step, by its parity
  cx<double> dv[2];                           // d of the step
  cx<double> sv[16 * NB];                     // the diagonal: of G, then the pivots
  int sbad[4];
};

// In: A[a][c], a >= c, the entry (tx + 16 a, ty + 16 c) of the lower triangle of G
// (of L = R^H, mode 1), zero outside it.  Out: put(k, i, v) for every entry v =
// R^{-1}(k, i) of the padded 16 NB x 16 NB square, zero outside the triangle.
template <int NB, int MODE, typename Put>
__device__ __forceinline__ void chol_eliminate(cx<double> (&A)[NB][NB], int b, double shift_coef, ElimLds<NB>& w,
                                               int* info, Put put) {
  constexpr bool TRI = MODE == 1;
  constexpr int TD = 16;
  auto& lv = w.lv;
  auto& rv = w.rv;
  auto& dv = w.dv;
  auto& sv = w.sv;
  auto& sbad = w.sbad;
  const int tid = threadIdx.x, lane = tid & 63;
  const int tx = tid % TD, ty = tid / TD;  // row and column within a block
#pragma unroll
  for (int a = 0; a < NB; ++a)
    if (tx == ty) sv[tx + TD * a] = A[a][a];
  double shift = 0.0;
  __syncthreads();
  if (!TRI) {
    double tr = 0;
    for (int i = lane; i < b; i += 64) tr += sv[i].re;
    shift = shift_coef * wave_sum(tr);
#pragma unroll
    for (int a = 0; a < NB; ++a)
      if (tx == ty) A[a][a].re += shift;
    __syncthreads();  // sv is read above and takes the pivots below
  }
#pragma unroll
  for (int J = 0; J < NB; ++J) {
    const int jn = min(TD, b - TD * J);
    for (int jj = 0; jj < jn; ++jj) {
      const int j = TD * J + jj, par = j & 1;
      if (ty == jj) {  // column j: l below the diagonal, r on and beyond it
#pragma unroll
        for (int a = J; a < NB; ++a) {
          const int i = tx + TD * a;
          const cx<double> v = A[a][J];
          if (i > j) {
            lv[par][i] = v;
            rv[par][i] = TRI ? cx<double>{0.0, 0.0} : cx<double>{v.re, -v.im};
          } else if (i == j) {
            dv[par] = v;
            rv[par][i] = cx<double>{1.0, 0.0};
          }
        }
      }
      if (tx == jj) {  // row j: r before the diagonal
#pragma unroll
        for (int c = 0; c <= J; ++c)
          if (ty + TD * c < j) rv[par][ty + TD * c] = A[J][c];
      }
      lds_barrier();
      const cx<double> d = dv[par];
      if (tid == 0) sv[j] = d;
      // 1 / d: real positive for a Cholesky pivot, complex for a given triangle
      cx<double> g;
      if (!TRI) {
        // breakdown: 1 keeps the factor invertible (reported at the end)
        const double x = d.re > 0 && isfinite(d.re) ? d.re : 1.0;
        double q = __builtin_amdgcn_rcp(x);
        q = fma(fma(-x, q, 1.0), q, q);
        q = fma(fma(-x, q, 1.0), q, q);
        if (!(x > 1e-290 && x < 1e290)) q = 1.0 / x;
        g = cx<double>{q, 0.0};
      } else {
        const double rden = 1.0 / (d.re * d.re + d.im * d.im);
        g = cx<double>{d.re * rden, -d.im * rden};
      }
      cx<double> r[NB];
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const cx<double> t = rv[par][ty + TD * c];
        r[c] = TRI ? cx<double>{t.re * g.re - t.im * g.im, t.re * g.im + t.im * g.re}
                   : cx<double>{t.re * g.re, t.im * g.re};
      }
#pragma unroll
      for (int a = J; a < NB; ++a) {
        cx<double> l = lv[par][tx + TD * a];
        if (a == J && tx <= jj) l = cx<double>{0.0, 0.0};  // rows up to j are finished
#pragma unroll
        for (int c = 0; c <= a; ++c) {
          cx<double> v = A[a][c];
          if (c == J && ty == jj && (a > J || tx > jj)) v = cx<double>{0.0, 0.0};
          v.re = fma(-l.re, r[c].re, fma(l.im, r[c].im, v.re));
          v.im = fma(-l.re, r[c].im, fma(-l.im, r[c].re, v.im));
          A[a][c] = v;
        }
      }
    }
  }
  __syncthreads();
  // the rows' final scales from the pivots, and the pivots' events
  int bad = 0;
  for (int i = tid; i < b; i += 256) {
    const cx<double> d = sv[i];
    if (TRI) {
      const double rden = 1.0 / (d.re * d.re + d.im * d.im);
      sv[i] = cx<double>{d.re * rden, -d.im * rden};
    } else {
      const bool ok = d.re > 0 && isfinite(d.re);
      if (!ok) bad |= 1;
      if (shift > 0 && !(d.re > 2.0 * shift)) bad |= 2;  // the shift carries this pivot
      sv[i] = cx<double>{ok ? 1.0 / sqrt(d.re) : 1.0, 0.0};
    }
  }
  if (!TRI) {
    const int any1 = __ballot(bad & 1) != 0ull, any2 = __ballot(bad & 2) != 0ull;
    if (lane == 0) sbad[tid >> 6] = any1 | 2 * any2;
  }
  __syncthreads();
  if (!TRI && tid == 0) {
    const int all = sbad[0] | sbad[1] | sbad[2] | sbad[3];
    if (all & 1) atomicAdd(&info[INFO_CHOL_BREAKDOWN], 1);
    if (all & 2) atomicAdd(&info[INFO_CHOL_SHIFTED], 1);
  }
  // R^{-1} = (L^{-1})^H: entry (k, i) from row i of L^{-1}
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const int i = tx + TD * a, k = ty + TD * c;
      cx<double> v{0.0, 0.0};
      if (c <= a && k <= i && i < b) {
        const cx<double> s = sv[i], x = k == i ? cx<double>{1.0, 0.0} : A[a][c <= a ? c : 0];
        v = cx<double>{x.re * s.re - x.im * s.im, -(x.re * s.im + x.im * s.re)};
      }
      put(k, i, v);
    }
}

}  // namespace tsvd
