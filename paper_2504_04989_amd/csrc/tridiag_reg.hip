// Householder tridiagonalisation of the small Hermitian matrices of the
// per-slice SVD (see heig.hip), m <= TREG_MAX, one workgroup per slice, the
// whole triangle on chip.
//
// Bound: the chain of m steps, each a norm, a reflector, a matrix-vector
// product, a dot product and a rank-2 update of a matrix of at most 192 x 192.
// The arithmetic of all steps together is about 0.1 ms of one CU's FP64 rate.
// The streaming form spent 3.5 to 10 us per step on its eight workgroup barriers,
// LDS shuffles and the trailing matrix's round trip through L2.  Here:
//   - the waves hold the 32 x 32 tiles of the lower triangle in registers, 4 x 4
//     entries per lane (diagonal tiles hold both triangles, so no entry is
//     masked).  A wave issues one vector instruction every four cycles and
//     that issue is what a step costs, so sums over lanes go through DPP moves
//     and lane swaps, not LDS;
//   - two barriers per step: after the tile pass (update of step i - 1, column
//     i + 1 as it then stands into LDS, partial sums of y_i = A v_i) and after
//     wave 0 has formed w_i, that column's update, its norm and the next
//     reflector.  The other waves wait for wave 0: the same work in every wave
//     would take issue slots from it;
//   - at most two waves per SIMD, with up to three tiles each: 16 waves have
//     128 registers each and spilled.  The update on the FP64 matrix unit
//     (K = 4, one MFMA per 16 x 16 block and part) measured slower than on the
//     vector unit (m = 100: 0.63 ms against 0.28 ms);
//   - every partial sum of y has its own LDS entry (one per tile row and row) and
//     they are added in a fixed order, so results repeat bit for bit.
// Measured, per launch, streaming form -> here: 30 x 30 over 9 slices 104 ->
// 47 us, 160 x 160 over 101 slices 1.51 -> 0.60 ms, 180 x 180 over 17 slices
// 1.83 -> 0.79 ms (about 3.7 and 4.4 us per step).
#include "common.h"
#include "heig_common.h"

namespace tsvd {
namespace {

// x, y -> (lanes 0-31: the sum over {l, l + 32} of x; lanes 32-63: of y)
__device__ __forceinline__ double swap_add32(double x, double y) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// even rows of 16: the sum over {l, l + 16} of x; odd rows: of y
__device__ __forceinline__ double swap_add16(double x, double y) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// 1 / x to full precision for x within the normal range (two Newton steps on
// the hardware estimate).
__device__ __forceinline__ double rcp_full(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// Reflector of the column (alpha = ar + i ai, x) with ||x||^2 = s2:
// beta = -sign(ar) ||(alpha, x)||, tau = (beta - alpha) / beta (conjugated as
// the callers use it), v = x * scale.  Returns false for the identity.
__device__ __forceinline__ bool reflector(double ar, double ai, double s2, double& beta, cx<double>& tau,
                                          cx<double>& scale) {
  if (s2 == 0.0 && ai == 0.0) {
    beta = ar;
    tau = scale = cx<double>{0, 0};
    return false;
  }
  const double n2 = ar * ar + ai * ai + s2;
  if (n2 > 1e-280 && n2 < 1e280) {
    // sqrt and reciprocals from the hardware estimates by Newton steps
    double r = __builtin_amdgcn_rsq(n2);
    r = r * fma(-0.5 * n2 * r, r, 1.5);
    r = r * fma(-0.5 * n2 * r, r, 1.5);
    double g = n2 * r;
    g = fma(0.5 * r, fma(-g, g, n2), g);
    beta = -copysign(g, ar);
    const double ib = rcp_full(beta);
    const double dr = ar - beta;
    tau = cx<double>{-dr * ib, -ai * ib};
    const double iden = rcp_full(dr * dr + ai * ai);
    scale = cx<double>{dr * iden, -ai * iden};
  } else {
    beta = -copysign(sqrt(n2), ar);
    tau = cx<double>{(beta - ar) / beta, -ai / beta};
    const double dr = ar - beta, den = dr * dr + ai * ai;
    scale = cx<double>{dr / den, -ai / den};
  }
  return true;
}

// Sum of y[0..3] over the eight lanes with the same lane / 8: the lane gets
// the total of element 2 [lane & 4] + [lane & 2].  The partner of the first
// exchange is lane ^ 7 (row_half_mirror), which also differs in bit 2.
__device__ __forceinline__ double sum_cols(const double (&y)[4], int lane) {
  const bool h0 = lane & 4, h1 = lane & 2;
  const double t0 = (h0 ? y[2] : y[0]) + dpp_mov<0x141>(h0 ? y[0] : y[2]);
  const double t1 = (h0 ? y[3] : y[1]) + dpp_mov<0x141>(h0 ? y[1] : y[3]);
  const double u = (h1 ? t1 : t0) + dpp_mov<0x4E>(h1 ? t0 : t1);
  return u + dpp_mov<0xB1>(u);
}
// Sum of y[0..3] over the eight lanes with the same lane % 8: the lane gets
// the total of element 2 [lane & 32] + [lane & 16].
__device__ __forceinline__ double sum_rows(const double (&y)[4]) {
  const double u = swap_add16(swap_add32(y[0], y[2]), swap_add32(y[1], y[3]));
  return u + dpp_mov<0x128>(u);
}

// x, recomputed where it is used: addresses derived from it are not kept in
// registers across the step loop (they were spilled).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// T: tiles per side (m <= 32 T); up to SLOTS tiles in each of the NW waves but
// the first.
template <int T, int NW, int SLOTS>
__global__ __launch_bounds__(64 * NW, 1) void heig_treg_kernel(const cx<double>* __restrict__ Gpart, int nsum,
                                                               int64_t part_stride, int m, unsigned char* scratch,
                                                               size_t per_slice, int upper_only) {
  constexpr int NTL = T * (T + 1) / 2, NTH = 64 * NW, U = (32 * T + 63) / 64, RP = 64 * U;
  static_assert(NTL <= (NW - 1) * SLOTS, "tiles do not fit");
  __shared__ cx<double> vo[RP], wo[RP];  // v and w of the step to be applied (0 outside their rows)
  __shared__ cx<double> v[RP];           // v of the step to be multiplied
  __shared__ cx<double> col[RP];         // the next column before the step's update
  __shared__ cx<double> s_tau;           // of the last reflector
  __shared__ cx<double> part[T][RP];     // partial sums of y: row r's from the tile that pairs its tile row with k
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int la = lane >> 3, lb = lane & 7;
  const int f = blockIdx.x;
  const HeigView hv = heig_view(scratch, per_slice, f, m);
  const cx<double>* G = Gpart + (int64_t)f * m * m;
  // The Hermitian matrix at (r, c) from the partials, zero past m - 1: the
  // average of the two triangles, or the extension of the upper one.
  auto gram4 = [&](const int (&r)[4], const int (&c)[4], cx<double> (&x)[4]) {
    int64_t at[4], ta[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int rr = min(r[e], m - 1), cc = min(c[e], m - 1);
      at[e] = (int64_t)min(rr, cc) * m + max(rr, cc);  // the entry above the diagonal
      ta[e] = (int64_t)max(rr, cc) * m + min(rr, cc);
      x[e] = cx<double>{0, 0};
    }
    for (int s = 0; s < nsum; ++s) {
      const cx<double>* Gs = G + s * part_stride;
      cx<double> g[4], h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] = Gs[at[e]];
      if (!upper_only) {
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = Gs[ta[e]];
#pragma unroll
        for (int e = 0; e < 4; ++e) g[e] = cx<double>{0.5 * (g[e].re + h[e].re), 0.5 * (g[e].im - h[e].im)};
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = cadd(x[e], g[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (r[e] > c[e]) x[e].im = -x[e].im;
      if (r[e] == c[e]) x[e].im = 0.0;
      if (r[e] >= m || c[e] >= m) x[e] = cx<double>{0, 0};
    }
  };
  for (int r = tid; r < RP; r += NTH) {
    vo[r] = wo[r] = v[r] = cx<double>{0, 0};
#pragma unroll
    for (int k = 0; k < T; ++k) part[k][r] = cx<double>{0, 0};
  }
  for (int r = 4 * tid; r < RP; r += 4 * NTH) {
    const int rr[4] = {r, r + 1, r + 2, r + 3}, cc[4] = {0, 0, 0, 0};
    cx<double> x[4];
    gram4(rr, cc, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) col[r + e] = x[e];
  }
  if (tid == 0) s_tau = cx<double>{0, 0};
  // The tile waves and wave 0 run loops of their own (the tiles' registers are
  // not live in wave 0's) that meet at the same two barriers per reflector j.
  if (wv > 0) {
    // this wave's tiles, row-major over the triangle, so that the trailing ones
    // stay spread over the waves
    int tI[SLOTS], tJ[SLOTS];
    bool tok[SLOTS];
    cx<double> a[SLOTS][4][4];  // lane (la, lb): rows 4 la + q, columns lb + 8 p
#pragma unroll
    for (int sl = 0; sl < SLOTS; ++sl) {
      const int t = sl * (NW - 1) + wv - 1;
      tok[sl] = t < NTL;
      tri_tile(tok[sl] ? t : 0, 0, tI[sl], tJ[sl]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = tok[sl] ? 32 * tI[sl] + 4 * la + q : m, c = 32 * tJ[sl] + lb;
        const int rr[4] = {r, r, r, r}, cc[4] = {c, c + 8, c + 16, c + 24};
        gram4(rr, cc, a[sl][q]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // A -= v w^H + w v^H on row q of a lane block x[4], rows from r0, columns
    // from c0 (the column operands vc, wc are read once per tile).
    auto rank2_row = [&](cx<double> (&x)[4], int r, const cx<double> (&vc)[4], const cx<double> (&wc)[4]) {
      const cx<double> vr = vo[r], wr = wo[r];
      const cx<double> nv{-vr.re, -vr.im}, nw{-wr.re, -wr.im};
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        cfmac(x[p], wc[p], nv);
        cfmac(x[p], vc[p], nw);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // row q's part of y = A v: its sum into (yr, yi), the column sums into (zr, zi)
    auto mul_row = [&](const cx<double> (&x)[4], int r, const cx<double> (&vc)[4], double& yr, double& yi,
                       double (&zr)[4], double (&zi)[4]) {
      const cx<double> vr = v[r];
      cx<double> acc{0, 0};
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        cfma(acc, x[p], vc[p]);
        zr[p] = fma(x[p].re, vr.re, fma(x[p].im, vr.im, zr[p]));
        zi[p] = fma(x[p].re, vr.im, fma(-x[p].im, vr.re, zi[p]));
      }
      yr = acc.re;
      yi = acc.im;
      __builtin_amdgcn_sched_barrier(0);
    };
    auto sums = [&](const double (&yr)[4], const double (&yi)[4], const double (&zr)[4], const double (&zi)[4], int r0,
                    int c0, int I, int J) {
      const cx<double> s{sum_cols(yr, lane), sum_cols(yi, lane)};
      if (!(lane & 1)) part[J][r0 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1)] = s;
      if (I != J) {
        const cx<double> z{sum_rows(zr), sum_rows(zi)};
        if (!(lane & 8)) part[I][c0 + 8 * (((lane >> 5) & 1) * 2 + ((lane >> 4) & 1))] = z;
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    __syncthreads();
    for (int j = 0; j < m - 1; ++j) {
      lds_barrier();
      const int J0 = (j + 1) >> 5, pn = ((j + 1) >> 3) & 3;
      const bool mine = lb == ((j + 1) & 7);  // lanes that hold column j + 1 (of their tile column), at p = pn
#pragma unroll
      for (int sl = 0; sl < SLOTS; ++sl) {
        if (!tok[sl] || tJ[sl] < J0) continue;
        const int r0 = 32 * tI[sl] + 4 * fresh(la), c0 = 32 * tJ[sl] + fresh(lb);
        {
          cx<double> vc[4], wc[4];
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            vc[p] = vo[c0 + 8 * p];
            wc[p] = wo[c0 + 8 * p];
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) rank2_row(a[sl][q], r0 + q, vc, wc);
        }
        if (tJ[sl] == J0 && mine) {
#pragma unroll
          for (int p = 0; p < 4; ++p)
            if (p == pn) {
#pragma unroll
              for (int q = 0; q < 4; ++q) col[r0 + q] = a[sl][q][p];
            }
        }
        cx<double> vc[4];
        double yr[4], yi[4], zr[4], zi[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          vc[p] = v[c0 + 8 * p];
          zr[p] = zi[p] = 0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) mul_row(a[sl][q], r0 + q, vc, yr[q], yi[q], zr, zi);
        sums(yr, yi, zr, zi, r0, c0, tI[sl], tJ[sl]);
      }
      lds_barrier();
    }
    return;
  }
  __syncthreads();

  for (int i = -1;; ++i) {
    const int j = i + 1;  // the reflector to be formed
    {
      // y_i; w_i = tau y + alpha v, alpha = -tau (w^H v) / 2 (all zero for i = -1)
      const int Ji = j >> 5;  // first unfinished tile row of step i
      const cx<double> tau = s_tau;
      cx<double> wl[U], vr[U], c1[U], dot{0, 0};
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = lane + 64 * u;
        cx<double> y{0, 0};
#pragma unroll
        for (int k = 0; k < T; ++k)
          {
            const cx<double> t = part[k][r];  // (read whatever k is: a branch per read would serialise them)
            y.re += k >= Ji ? t.re : 0.0;
            y.im += k >= Ji ? t.im : 0.0;
          }
        vr[u] = v[r];
        c1[u] = col[r];
        wl[u] = cmulc(tau, y);
        cfmac(dot, wl[u], vr[u]);  // v is 0 outside the trailing rows
      }
      dot.re = wave_sum(dot.re);
      dot.im = wave_sum(dot.im);
      const cx<double> alpha = cmulc(cx<double>{-0.5 * tau.re, -0.5 * tau.im}, dot);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = lane + 64 * u;
        cfma(wl[u], alpha, vr[u]);
        if (r <= i || r >= m) wl[u] = cx<double>{0, 0};
        vo[r] = vr[u];
        wo[r] = wl[u];
      }
      // column j after update i: c -= v conj(w_j) + w conj(v_j), v_j = 1 (i < 0: both are zero)
      auto row_value = [&](const cx<double>(&x)[U], int r) {
        double re = x[0].re, im = x[0].im;
        if (U > 1) {
          re = r >= 64 ? x[U > 1 ? 1 : 0].re : re;
          im = r >= 64 ? x[U > 1 ? 1 : 0].im : im;
        }
        if (U > 2) {
          re = r >= 128 ? x[U > 2 ? 2 : 0].re : re;
          im = r >= 128 ? x[U > 2 ? 2 : 0].im : im;
        }
        return cx<double>{lane_value(re, r & 63), lane_value(im, r & 63)};
      };
      const cx<double> wj = row_value(wl, j);
      double s2 = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = lane + 64 * u;
        cfmac(c1[u], wj, cx<double>{-vr[u].re, -vr[u].im});
        c1[u].re -= wl[u].re;
        c1[u].im -= wl[u].im;
        if (r > j + 1 && r < m) s2 += c1[u].re * c1[u].re + c1[u].im * c1[u].im;
        if (r == j) hv.d[j] = c1[u].re;
      }
      if (j == m - 1) {
        if (lane == 0) {
          hv.e[j] = 0.0;
          if (m == 1) hv.tau[0] = cx<double>{0, 0};
        }
      } else {
        s2 = wave_sum(s2);
        const cx<double> al = row_value(c1, j + 1);
        double beta;
        cx<double> tau_j, scale;
        reflector(al.re, al.im, s2, beta, tau_j, scale);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int r = lane + 64 * u;
          cx<double> x{0, 0};
          if (r > j && r < m) x = r == j + 1 ? cx<double>{1.0, 0.0} : cmulc(c1[u], scale);
          v[r] = x;
          if (r > j && r < m) hv.A[(int64_t)j * m + r] = x;
        }
        if (lane == 0) {
          hv.e[j] = beta;
          hv.tau[j] = tau_j;
          s_tau = tau_j;
        }
      }
    }
    if (j == m - 1) break;
    lds_barrier();
    lds_barrier();
  }
}

}  // namespace

hipError_t heig_tridiag_reg(const cx<double>* Gpart, int nsum, int64_t part_stride, int m, int batch,
                            unsigned char* scratch, size_t per_slice, int upper_only, hipStream_t s) {
  if (m < 1 || m > TREG_MAX) return hipErrorInvalidValue;
  auto go = [&](auto kernel, int NW) -> hipError_t {
    hipLaunchKernelGGL(kernel, dim3(batch), dim3(64 * NW), 0, s, Gpart, nsum, part_stride, m, scratch, per_slice,
                       upper_only);
    return hipGetLastError();
  };
  // one tile per wave up to six tiles, then at most two waves per SIMD
  switch ((m + 31) / 32) {
    case 1: return go(heig_treg_kernel<1, 2, 1>, 2);
    case 2: return go(heig_treg_kernel<2, 4, 1>, 4);
    case 3: return go(heig_treg_kernel<3, 7, 1>, 7);
    case 4: return go(heig_treg_kernel<4, 8, 2>, 8);
    case 5: return go(heig_treg_kernel<5, 8, 3>, 8);
    default: return go(heig_treg_kernel<6, 8, 3>, 8);
  }
}

}  // namespace tsvd
