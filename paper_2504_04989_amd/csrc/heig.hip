// Top-k eigenpairs of a per-slice m x m Hermitian positive semidefinite
// matrix in FP64: the small decomposition behind the per-slice SVD of
// C_f = Q_f^H A_f in Alg. 2.  With C_f C_f^H = W diag(lambda) W^H, the left
// singular vectors of C_f are W, sigma = sqrt(lambda), and the right singular
// vectors are C_f^H W diag(1/sigma).
//
// Four kernels, all batched over the Fourier slices:
//  1. tridiag   symmetrised sum of the split-K partials, then Householder
//               reduction G = H T H^H, H = H_0 ... H_{m-2},
//               H_j = I - tau_j v_j v_j^H (complex reflectors with real beta,
//               so T is real symmetric).  m <= TREG_MAX: one workgroup per
//               slice with the triangle in registers (tridiag_reg.hip);
//               larger m: one or several workgroups per slice, below.
//  2. bisect    multisection on Sturm counts of T for the k largest
//               eigenvalues, 8, 16 or 64 lanes per eigenvalue.
//  3. invit     one lane per eigenvector: inverse iteration on the pivoted LU
//               of T - lambda I; then the members of a cluster of close
//               eigenvalues are orthogonalised against each other.
//  4. backxf    W = H Z, several workgroups per slice, each owning 8 columns
//               of W in LDS.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "heig_common.h"
#include "kernels.h"


namespace tsvd {

size_t heig_scratch_bytes(int m, int k) { return heig_per_slice(m, k); }

// ---------------------------------------------------------------------------
// 1. Blocked tridiagonalisation for m > TREG_MAX (panels of NB reflectors).
// Within a panel the trailing matrix is only read: step i forms y = A_tr v_i from the matrix as it stood
// at the start of the panel and corrects it with the panel's earlier
// reflectors, y -= V (W^H v) + W (V^H v); the panel's 2 NB rank-one terms
// A -= V W^H + W V^H are applied once at its end.  Only the lower triangle is
// read or written: a 32 x 32 tile below the diagonal feeds both y_R += A v_C
// and y_C += A^H v_R.  Each wave takes whole tiles (the next one is loaded
// while the current one is used), each lane a 4 x 4 block (rows
// 4 (lane / 8) + q, columns lane % 8 + 8 p); row and column sums are
// finished with three lane exchanges each and added into y in LDS.  The
// panel's V and W stay in LDS.  The trailing matrix is read about once per
// step at half size.  The waves' additions into y land in an order that
// depends on timing, so they are made in 64-bit fixed point (integer addition
// is associative): a contribution x is added as rint(x 2^62 / S) with S a power
// of two >= m ||G||_F.  Every partial sum of a row of the trailing matrix times
// v is below S in modulus (|a_rc| <= ||G||_2 <= ||G||_F, |v_c| <= 1), and
// the rounding, below 2^-61 m ||G||_F per contribution, stays under the FP64
// error of the product; the results are bitwise reproducible.
// ---------------------------------------------------------------------------
constexpr int T2_NT = 512;
constexpr int T2_W = T2_NT / 64;

template <int NW = T2_W, bool LEAD_SYNC = true>
__device__ __forceinline__ cx<double> block_sum2(cx<double> v, double* red) {
  v.re = wave_sum(v.re);
  v.im = wave_sum(v.im);
  const int w = threadIdx.x >> 6;
  if (LEAD_SYNC) __syncthreads();  // (skipped when red has not been read since the last barrier)
  if ((threadIdx.x & 63) == 0) {
    red[2 * w] = v.re;
    red[2 * w + 1] = v.im;
  }
  __syncthreads();
  cx<double> r{0, 0};
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    r.re += red[2 * i];
    r.im += red[2 * i + 1];
  }
  return r;
}

// Sum of a 4-vector over the eight lanes that differ only in lane bits X0, X1,
// X2 (three exchanges, halving the vector each time): the result is the total
// of element 2 [lane & X0] + [lane & X1]; the two lanes differing in X2 hold
// the same total.
template <int X0, int X1, int X2>
__device__ __forceinline__ cx<double> reduce4(const cx<double> (&y)[4], int lane) {
  const bool h0 = lane & X0, h1 = lane & X1;
  const cx<double> k0 = h0 ? y[2] : y[0], k1 = h0 ? y[3] : y[1];
  const cx<double> s0 = h0 ? y[0] : y[2], s1 = h0 ? y[1] : y[3];
  const cx<double> t0 = cadd(k0, shfl_xor_cx(s0, X0)), t1 = cadd(k1, shfl_xor_cx(s1, X0));
  const cx<double> kk = h1 ? t1 : t0, ss = h1 ? t0 : t1;
  const cx<double> u = cadd(kk, shfl_xor_cx(ss, X1));
  return cadd(u, shfl_xor_cx(u, X2));
}

// The lane's 4 x 4 block: rows r0 + q, columns c0 + 8 p (eight lanes of a row
// group read one contiguous 128-byte segment per access).  Rows are clamped
// into the matrix; columns past m - 1 (last tile column only) read the next
// row, or for the last row the vectors stored after the matrix, and are masked.
__device__ __forceinline__ void load_block(const cx<double>* A, int m, int r0, int c0, cx<double> (&a)[4][4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const cx<double>* rp = A + (int64_t)min(r0 + q, m - 1) * m + c0;
#pragma unroll
    for (int p = 0; p < 4; ++p) a[q][p] = rp[8 * p];
  }
}

// y_R += A_blk v_C and y_C += A_blk^H v_R for the lane's block; MASK handles
// the tiles on the diagonal, at the first trailing column or past row m - 1.
template <bool MASK>
__device__ __forceinline__ void symv_block(const cx<double> (&a)[4][4], const cx<double>* vcur, int r0, int c0,
                                           int m, int cmin, cx<double> (&yR)[4], cx<double> (&yC)[4]) {
  cx<double> vr[4], vc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    vr[q] = vcur[r0 + q];
    vc[q] = vcur[c0 + 8 * q];
    yR[q] = yC[q] = cx<double>{0, 0};
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      cx<double> x = a[q][p];
      if (MASK) {
        const int r = r0 + q, c = c0 + 8 * p;
        const bool ok = r < m && c >= cmin && r >= c;
        if (!ok) x = cx<double>{0, 0};
        if (r == c) x.im = 0.0;
        cfma(yR[q], x, vc[p]);
        if (r == c) x = cx<double>{0, 0};
        cfmac(yC[p], x, vr[q]);
      } else {
        cfma(yR[q], x, vc[p]);
        cfmac(yC[p], x, vr[q]);
      }
    }
  }
}

// A_blk -= V_R W_C^H + W_R V_C^H over the panel's k < pw terms
__device__ __forceinline__ void rank_block(cx<double> (&a)[4][4], const cx<double>* Vl, const cx<double>* Wl, int MP,
                                           int pw, int r0, int c0) {
  for (int k = 0; k < pw; ++k) {
    cx<double> vr[4], wr[4], vc[4], wc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      vr[q] = Vl[k * MP + r0 + q];
      wr[q] = Wl[k * MP + r0 + q];
      vc[q] = Vl[k * MP + c0 + 8 * q];
      wc[q] = Wl[k * MP + c0 + 8 * q];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const cx<double> nv{-vr[q].re, -vr[q].im}, nw{-wr[q].re, -wr[q].im};
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        // a -= v_r conj(w_c) + w_r conj(v_c)  ==  a += conj(w_c) (-v_r) + conj(v_c) (-w_r)
        cfmac(a[q][p], wc[p], nv);
        cfmac(a[q][p], vc[p], nw);
      }
    }
  }
}

// The slice's matrix, lower triangle only: A = Hermitian part of the sum of
// the nsum partials (or the Hermitian extension of their upper triangle),
// rows p, p + P, ... of it (the workgroup's share).
__device__ __forceinline__ void tri_load_lower(const cx<double>* __restrict__ G, int nsum, int64_t part_stride,
                                               int m, int upper_only, cx<double>* A, int p, int P) {
  for (int i = p; i < m; i += P) {
    for (int c = threadIdx.x; c <= i; c += T2_NT) {
      cx<double> g{0, 0}, h{0, 0};
      for (int s = 0; s < nsum; ++s) {
        const cx<double>* Gs = G + s * part_stride;
        const cx<double> x = Gs[(int64_t)i * m + c], y = Gs[(int64_t)c * m + i];
        g.re += x.re;
        g.im += x.im;
        h.re += y.re;
        h.im += y.im;
      }
      const cx<double> lo = upper_only ? cx<double>{h.re, i == c ? 0.0 : -h.im}
                                       : cx<double>{0.5 * (g.re + h.re), i == c ? 0.0 : 0.5 * (g.im - h.im)};
      A[(int64_t)i * m + c] = lo;
    }
  }
}

// Barrier over the P workgroups of one slice (P > 1; they are co-resident by
// cooperative launch).  ctr[0] counts arrivals, ctr[1] is set once a wait
// runs past its bound: every later wait of the slice then returns at once,
// the kernel finishes with wrong values and the nonfinite counter says so.
__device__ __forceinline__ void group_sync(unsigned* ctr, unsigned& gen, int P, int* info) {
  // every wave waits until its own global stores have reached the L2 (s_waitcnt
  // vmcnt(0)); the one release below then writes the L2 back for the group
  if (P > 1) __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  if (P > 1) {
    ++gen;
    if (threadIdx.x == 0) {
      __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned target = gen * (unsigned)P;
      unsigned spins = 0;
      while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        if (__hip_atomic_load(ctr + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
        __builtin_amdgcn_s_sleep(1);
        if (++spins == (1u << 22)) {  // about a second: only reachable if the group is not co-resident
          __hip_atomic_store(ctr + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicAdd(&info[INFO_NONFINITE], 1);
          break;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // after the relaxed polls
    }
    __syncthreads();
  }
}

// Per slice, PREP_WG workgroups (blockIdx.y): the barrier counters cleared and
// the partial sums of ||G||_F^2 over the rows r = y mod PREP_WG of the summed
// partials (their upper triangle counted twice when only it is valid); the
// tridiagonalisation adds the PREP_WG partials in order and takes the power of
// two S >= m ||G||_F as the fixed-point scale of its symv sums.
constexpr int PREP_WG = 8;
__global__ __launch_bounds__(256) void heig_prep_kernel(const cx<double>* __restrict__ Gpart, int nsum,
                                                        int64_t part_stride, int m, int upper_only,
                                                        unsigned char* scratch, size_t per_slice) {
  __shared__ double red[4];
  const int f = blockIdx.x, y = blockIdx.y;
  const HeigView hv = heig_view(scratch, per_slice, f, m);
  const cx<double>* G = Gpart + (int64_t)f * m * m;
  double acc = 0.0;
  // four rows per pass keep several loads of each thread in flight
  for (int r0 = y; r0 < m; r0 += 4 * PREP_WG) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + u * PREP_WG;
      if (r >= m) continue;
      for (int c = (upper_only ? r : 0) + (int)threadIdx.x; c < m; c += 256) {
        const int64_t t = (int64_t)r * m + c;
        cx<double> g{0, 0};
        for (int s = 0; s < nsum; ++s) {
          const cx<double> x = G[s * part_stride + t];
          g.re += x.re;
          g.im += x.im;
        }
        acc += (upper_only && c != r ? 2.0 : 1.0) * (g.re * g.re + g.im * g.im);
      }
    }
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    hv.fscale[y] = red[0] + red[1] + red[2] + red[3];
    if (y == 0) {
      hv.sync[0] = 0;
      hv.sync[1] = 0;
    }
  }
}

// S = 2^e >= m ||G||_F from the prep kernel's partial sums (fixed order).
__device__ __forceinline__ double tri_fix_scale(const HeigView& hv, int m) {
  double fro2 = 0.0;
  for (int y = 0; y < PREP_WG; ++y) fro2 += hv.fscale[y];
  const double bound = (double)m * sqrt(fro2);
  if (!(bound > 0.0) || !isfinite(bound)) return 1.0;
  int e = 0;
  (void)frexp(bound, &e);  // bound < 2^e
  return ldexp(1.0, e);
}

// Lighter barrier for data exchanged only through device-coherent accesses
// (agent-scope atomic loads and stores, which bypass the XCD's L2): each wave
// waits for its own accesses to complete, then the arrival count is bumped
// and polled without any cache writeback or invalidation.
__device__ __forceinline__ void group_sync_coherent(unsigned* ctr, unsigned& gen, int P, int* info) {
  if (P <= 1) {
    __syncthreads();
    return;
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's coherent stores are complete
  __syncthreads();
  ++gen;
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned target = gen * (unsigned)P;
    unsigned spins = 0;
    while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (__hip_atomic_load(ctr + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
      __builtin_amdgcn_s_sleep(1);
      if (++spins == (1u << 22)) {
        __hip_atomic_store(ctr + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicAdd(&info[INFO_NONFINITE], 1);
        break;
      }
    }
  }
  __syncthreads();
}

template <int NB>
__global__ __launch_bounds__(T2_NT) void heig_tri2_kernel(const cx<double>* __restrict__ Gpart, int nsum,
                                                          int64_t part_stride, int m, int MP, unsigned char* scratch,
                                                          size_t per_slice, int upper_only, int P,
                                                          int* __restrict__ info) {
  extern __shared__ __align__(16) unsigned char smem[];
  cx<double>* vcur = reinterpret_cast<cx<double>*>(smem);  // MP: v of the current step (0 outside its range)
  cx<double>* y = vcur + MP;                                // MP: A_tr v
  cx<double>* col = y + MP;                                 // MP: the updated column of the step
  cx<double>* Vl = col + MP;                                // NB x MP: the panel's reflectors
  cx<double>* Wl = Vl + NB * MP;                            // NB x MP: their update vectors
  cx<double>* xs = Wl + NB * MP;                            // 2 NB: W^H v and V^H v
  __shared__ double red[2 * T2_W];
  __shared__ cx<double> s_tau, s_scale;
  __shared__ int s_skip;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int f = blockIdx.x / P, pg = blockIdx.x - f * P;  // slice, workgroup within the slice
  const bool lead = pg == 0;                             // writes the slice's outputs
  const HeigView hv = heig_view(scratch, per_slice, f, m);
  cx<double>* A = hv.A;
  unsigned* ctr = hv.sync;
  unsigned gen = 0;
  // fixed-point scale factors of the symv sums (powers of two: exact)
  const double fsc = tri_fix_scale(hv, m);
  const double to_fix = ldexp(1.0, 62) / fsc, from_fix = fsc * ldexp(1.0, -62);
  unsigned long long* yq = reinterpret_cast<unsigned long long*>(y);
  tri_load_lower(Gpart + (int64_t)f * m * m, nsum, part_stride, m, upper_only, A, pg, P);
  for (int r = tid; r < (2 * NB + 3) * MP; r += T2_NT) vcur[r] = cx<double>{0, 0};
  const int la = lane >> 3, lb = lane & 7;
  const int T = MP / 32;
  const int w0 = pg * T2_W + wv, wstep = P * T2_W;  // this wave's first tile and tile stride
  group_sync(ctr, gen, P, info);

  // The trailing matrix is only read within a panel, so a step's column and
  // its first symv tiles are requested early: the column one step ahead, the
  // tiles before the column update.  Row indices are clamped into the matrix.
  cx<double> colnext[2];
  for (int j0 = 0; j0 < m - 1; j0 += NB) {
    const int pw = min(NB, m - 1 - j0);
    for (int ii = 0; ii < pw; ++ii) {
      const int i = j0 + ii;
      cx<double> colv[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (ii == 0) colv[u] = A[(int64_t)min(i + tid + u * T2_NT, m - 1) * m + i];
        else colv[u] = colnext[u];
      }
      if (ii + 1 < pw) {
#pragma unroll
        for (int u = 0; u < 2; ++u) colnext[u] = A[(int64_t)min(i + 1 + tid + u * T2_NT, m - 1) * m + i + 1];
      }
      const int sJ0 = (i + 1) >> 5, snT = T - sJ0;
      const int sntile = snT * (snT + 1) / 2;
      auto stile_rc = [&](int t, int& r0, int& c0) {
        int I, J;
        tri_tile(min(t, sntile - 1), sJ0, I, J);
        r0 = 32 * I + 4 * la;
        c0 = 32 * J + lb;
      };
      cx<double> a0[4][4], a1[4][4];
      {
        int r0, c0;
        stile_rc(w0, r0, c0);
        load_block(A, m, r0, c0, a0);
      }
      // (1) column i (rows i..m-1) brought up to date with the panel's earlier terms
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = i + tid + u * T2_NT;
        if (r >= m) continue;
        cx<double> a = colv[u];
        for (int k = 0; k < ii; ++k) {
          const cx<double> vr = Vl[k * MP + r], wr = Wl[k * MP + r];
          const cx<double> vi = Vl[k * MP + i], wi = Wl[k * MP + i];
          // a -= v_r conj(w_i) + w_r conj(v_i)
          a.re -= (vr.re * wi.re + vr.im * wi.im) + (wr.re * vi.re + wr.im * vi.im);
          a.im -= (vr.im * wi.re - vr.re * wi.im) + (wr.im * vi.re - wr.re * vi.im);
        }
        col[r] = a;
      }
      __syncthreads();
      // (2) reflector from alpha = col[i+1], x = col[i+2..m-1]
      double s2 = 0;
      for (int r = i + 2 + tid; r < m; r += T2_NT) s2 += col[r].re * col[r].re + col[r].im * col[r].im;
      s2 = block_sum2(cx<double>{s2, 0.0}, red).re;
      if (tid == 0) {
        const double ar = col[i + 1].re, ai = col[i + 1].im;
        double ei;
        if (s2 == 0.0 && ai == 0.0) {
          s_skip = 1;
          ei = ar;
          s_tau = cx<double>{0, 0};
        } else {
          s_skip = 0;
          const double beta = -copysign(sqrt(ar * ar + ai * ai + s2), ar);
          s_tau = cx<double>{(beta - ar) / beta, -ai / beta};
          const double dr = ar - beta, di = ai;
          const double den = dr * dr + di * di;
          s_scale = cx<double>{dr / den, -di / den};
          ei = beta;
        }
        if (lead) {
          hv.d[i] = col[i].re;
          hv.e[i] = ei;
          hv.tau[i] = s_tau;
        }
      }
      __syncthreads();
      const bool skip = s_skip != 0;
      const cx<double> tau = s_tau, scale = s_scale;
      // v (v[i+1] = 1) into LDS, into the panel and into row i of A; y = 0
      for (int r = i + 1 + tid; r < m; r += T2_NT) {
        cx<double> v;
        if (r == i + 1)
          v = cx<double>{1.0, 0.0};
        else if (skip)
          v = cx<double>{0.0, 0.0};
        else
          v = cmulc(col[r], scale);
        vcur[r] = v;
        Vl[ii * MP + r] = v;
        if (lead) A[(int64_t)i * m + r] = v;
        y[r] = cx<double>{0, 0};
      }
      if (tid == 0) vcur[i] = cx<double>{0, 0};
      __syncthreads();
      // (3a) x1 = W^H v, x2 = V^H v over rows i+1..m-1 (one wave per product)
      for (int dd = wv; dd < 2 * ii; dd += T2_W) {
        const cx<double>* X = (dd < ii ? Wl + dd * MP : Vl + (dd - ii) * MP);
        cx<double> acc{0, 0};
        for (int r = i + 1 + lane; r < m; r += 64) cfmac(acc, X[r], vcur[r]);
        acc.re = wave_sum(acc.re);
        acc.im = wave_sum(acc.im);
        if (lane == 0) xs[dd] = acc;
      }
      // (3b) y = A_tr v over the lower triangle of rows / columns >= i+1
      {
        const int J0 = sJ0, ntile = sntile;
        auto process = [&](const cx<double>(&a)[4][4], int t) {
          int I, J;
          tri_tile(t, J0, I, J);
          const int r0 = 32 * I + 4 * la, c0 = 32 * J + lb;
          cx<double> yR[4], yC[4];
          if (I > J && 32 * J >= i + 1 && 32 * I + 32 <= m)
            symv_block<false>(a, vcur, r0, c0, m, i + 1, yR, yC);
          else
            symv_block<true>(a, vcur, r0, c0, m, i + 1, yR, yC);
          const cx<double> sr = reduce4<4, 2, 1>(yR, lane);
          const cx<double> sc = reduce4<32, 16, 8>(yC, lane);
          auto fix = [&](double x) { return (unsigned long long)(long long)rint(x * to_fix); };
          if (!(lane & 1)) {
            const int q = ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
            atomicAdd(&yq[2 * (r0 + q)], fix(sr.re));
            atomicAdd(&yq[2 * (r0 + q) + 1], fix(sr.im));
          }
          if (!(la & 1)) {
            const int p = ((la >> 2) & 1) * 2 + ((la >> 1) & 1);
            atomicAdd(&yq[2 * (c0 + 8 * p)], fix(sc.re));
            atomicAdd(&yq[2 * (c0 + 8 * p) + 1], fix(sc.im));
          }
        };
        // two tile buffers (the first requested at the start of the step);
        // the next tile is in flight while one is used
        int r0, c0;
        for (int t = w0; t < ntile; t += 2 * wstep) {
          stile_rc(t + wstep, r0, c0);
          load_block(A, m, r0, c0, a1);
          process(a0, t);
          if (t + wstep >= ntile) break;
          stile_rc(t + 2 * wstep, r0, c0);
          load_block(A, m, r0, c0, a0);
          process(a1, t + wstep);
        }
      }
      __syncthreads();
      // the fixed-point sums back to FP64 (each thread converts its own rows)
      for (int r = i + 1 + tid; r < m; r += T2_NT) {
        const long long qr = (long long)yq[2 * r], qi = (long long)yq[2 * r + 1];
        y[r] = cx<double>{(double)qr * from_fix, (double)qi * from_fix};
      }
      __syncthreads();
      if (P > 1) {
        // partial products of the slice's workgroups, summed in workgroup order
        // (double buffered by step parity: a workgroup is at most one exchange ahead)
        double* yb = reinterpret_cast<double*>(hv.ypg + (int64_t)((i & 1) * P) * MP);
        for (int r = i + 1 + tid; r < m; r += T2_NT) {
          double* d = yb + 2 * ((int64_t)pg * MP + r);
          __hip_atomic_store(d, y[r].re, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(d + 1, y[r].im, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        group_sync_coherent(ctr, gen, P, info);
        for (int r = i + 1 + tid; r < m; r += T2_NT) {
          cx<double> acc{0, 0};
          for (int q = 0; q < P; ++q) {
            const double* d = yb + 2 * ((int64_t)q * MP + r);
            acc.re += __hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            acc.im += __hip_atomic_load(d + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          y[r] = acc;
        }
        __syncthreads();
      }
      // (4) y -= V x1 + W x2; w = tau y; w += alpha v with alpha = -tau (w^H v) / 2
      //     (rows i+1..m-1, at most two per thread)
      cx<double> wl[2];
      cx<double> dot{0, 0};
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = i + 1 + tid + u * T2_NT;
        wl[u] = cx<double>{0, 0};
        if (r < m) {
          cx<double> yy = y[r];
          for (int k = 0; k < ii; ++k) {
            const cx<double> nx1{-xs[k].re, -xs[k].im}, nx2{-xs[ii + k].re, -xs[ii + k].im};
            cfma(yy, Vl[k * MP + r], nx1);
            cfma(yy, Wl[k * MP + r], nx2);
          }
          wl[u] = cmulc(tau, yy);
          cfmac(dot, wl[u], vcur[r]);
        }
      }
      dot = block_sum2(dot, red);
      const cx<double> alpha = cmulc(cx<double>{-0.5 * tau.re, -0.5 * tau.im}, dot);
      const bool zero = tau.re == 0.0 && tau.im == 0.0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = i + 1 + tid + u * T2_NT;
        if (r < m) {
          cx<double> w = wl[u];
          cfma(w, alpha, vcur[r]);
          Wl[ii * MP + r] = zero ? cx<double>{0, 0} : w;
        }
      }
      __syncthreads();
    }
    // (5) A -= V W^H + W V^H on the lower triangle of rows / columns >= j0 + pw
    const int rs = j0 + pw;
    if (rs < m) {
      const int J0 = rs >> 5, nT = T - J0;
      const int ntile = nT * (nT + 1) / 2;
      auto tile_rc = [&](int t, int& r0, int& c0) {
        int I, J;
        tri_tile(min(t, ntile - 1), J0, I, J);
        r0 = 32 * I + 4 * la;
        c0 = 32 * J + lb;
      };
      auto process = [&](cx<double>(&a)[4][4], int t) {
        int I, J;
        tri_tile(t, J0, I, J);
        const int r0 = 32 * I + 4 * la, c0 = 32 * J + lb;
        rank_block(a, Vl, Wl, MP, pw, r0, c0);
        if (I > J && 32 * J >= rs && 32 * I + 32 <= m) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            cx<double>* rp = A + (int64_t)(r0 + q) * m + c0;
#pragma unroll
            for (int p = 0; p < 4; ++p) rp[8 * p] = a[q][p];
          }
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
              const int r = r0 + q, c = c0 + 8 * p;
              if (r < m && c >= rs && r >= c) A[(int64_t)r * m + c] = a[q][p];
            }
          }
        }
      };
      cx<double> a0[4][4], a1[4][4];
      int r0, c0;
      tile_rc(w0, r0, c0);
      load_block(A, m, r0, c0, a0);
      for (int t = w0; t < ntile; t += 2 * wstep) {
        tile_rc(t + wstep, r0, c0);
        load_block(A, m, r0, c0, a1);
        process(a0, t);
        if (t + wstep >= ntile) break;
        tile_rc(t + 2 * wstep, r0, c0);
        load_block(A, m, r0, c0, a0);
        process(a1, t + wstep);
      }
    }
    group_sync(ctr, gen, P, info);
  }
  if (tid == 0 && lead) {
    hv.d[m - 1] = A[(int64_t)(m - 1) * m + (m - 1)].re;
    hv.e[m - 1] = 0.0;
  }
}

// Register-resident form for several co-resident workgroups per slice.  The
// 32 x 32 tiles of the lower triangle are dealt out once: tile t (row-major
// over the triangle) belongs to workgroup t mod P, and within it to wave
// (t / P) mod RES_W, slot (t / P) / RES_W (at most RES_SLOTS per wave).  A wave keeps
// its tiles in registers for the whole reduction, in the 4 x 4 lane blocks of
// symv_block, so the trailing matrix is never read from or written to memory:
// every step applies the rank-2 update of the previous reflector in place.
// Per step i, one exchange between the workgroups of the slice:
//   - every workgroup adds its share of y = A_tr v (fixed point, as above) into
//     one slice-wide sum with agent-scope integer atomics, which are exact and
//     order-free, so y is the same in every workgroup and bit for bit the same
//     from run to run;
//   - the owners of column i + 1 publish it as it stands before this step's
//     update; after the exchange every workgroup applies the update to that one
//     column itself, so the next reflector needs no second exchange.
// The reflectors, w and the column update are repeated identically in every
// workgroup (same operands, same operations).  Sums and columns rotate through
// three buffers, so a buffer is cleared or rewritten only after every
// workgroup has passed the exchange that last read it.
// Four waves per workgroup, one per SIMD, so that each may hold up to 512
// registers (the tiles that do not fit the 256 vector registers sit in the
// accumulation registers); four tile slots per wave.
constexpr int RES_NT = 256;
constexpr int RES_W = RES_NT / 64;
constexpr int RES_SLOTS = 4;

// symv_block for the resident tiles with fewer live registers: the column
// operand is read once, the row operand one row of the lane block at a time.
template <bool MASK>
__device__ __forceinline__ void symv_res(const cx<double> (&a)[4][4], const cx<double>* vcur, int r0, int c0, int m,
                                         int cmin, cx<double> (&yR)[4], cx<double> (&yC)[4]) {
  cx<double> vc[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    vc[p] = vcur[c0 + 8 * p];
    yC[p] = cx<double>{0, 0};
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const cx<double> vr = vcur[r0 + q];
    yR[q] = cx<double>{0, 0};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      cx<double> x = a[q][p];
      if (MASK) {
        const int r = r0 + q, c = c0 + 8 * p;
        const bool ok = r < m && c >= cmin && r >= c;
        if (!ok) x = cx<double>{0, 0};
        if (r == c) x.im = 0.0;
        cfma(yR[q], x, vc[p]);
        if (r == c) x = cx<double>{0, 0};
        cfmac(yC[p], x, vr);
      } else {
        cfma(yR[q], x, vc[p]);
        cfmac(yC[p], x, vr);
      }
    }
  }
}

__global__ __launch_bounds__(RES_NT, 1) void heig_trires_kernel(const cx<double>* __restrict__ Gpart, int nsum,
                                                            int64_t part_stride, int m, int MP,
                                                            unsigned char* scratch, size_t per_slice, int upper_only,
                                                            int P, int* __restrict__ info) {
  __shared__ cx<double> col[1024];    // column i (rows >= i), replicated
  __shared__ cx<double> vcur[1024];   // v of the step (0 outside rows i + 1 .. m - 1)
  __shared__ cx<double> wv_[1024];    // w of the step (0 outside)
  __shared__ unsigned long long yq[2 * 1024];  // this workgroup's share of y, fixed point
  __shared__ double red[2 * RES_W];
  __shared__ double red2[2][RES_W];  // per-wave partials of the next step's ||x||^2, by step parity
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int f = blockIdx.x / P, pg = blockIdx.x - f * P;
  const bool lead = pg == 0;
  const HeigView hv = heig_view(scratch, per_slice, f, m);
  cx<double>* Vout = hv.A;  // row i receives v_i (read by the back-transformation)
  unsigned* ctr = hv.sync;
  unsigned gen = 0;
  const double fsc = tri_fix_scale(hv, m);
  const double to_fix = ldexp(1.0, 62) / fsc, from_fix = fsc * ldexp(1.0, -62);
  // exchange buffers: three fixed-point sums (2 u64 per row) and three columns
  unsigned long long* ysum = reinterpret_cast<unsigned long long*>(hv.ypg);
  cx<double>* colx = hv.ypg + 3 * MP;
  const int T = MP / 32, NT = T * (T + 1) / 2;
  const int la = lane >> 3, lb = lane & 7;
  const cx<double>* G = Gpart + (int64_t)f * m * m;
  auto gram = [&](int r, int c) {  // A(r, c), r >= c, from the partials
    cx<double> g{0, 0}, h{0, 0};
    for (int s = 0; s < nsum; ++s) {
      const cx<double>* Gs = G + s * part_stride;
      const cx<double> x = Gs[(int64_t)r * m + c], y = Gs[(int64_t)c * m + r];
      g.re += x.re;
      g.im += x.im;
      h.re += y.re;
      h.im += y.im;
    }
    return upper_only ? cx<double>{h.re, r == c ? 0.0 : -h.im}
                      : cx<double>{0.5 * (g.re + h.re), r == c ? 0.0 : 0.5 * (g.im - h.im)};
  };
  // this wave's tiles
  int tI[RES_SLOTS], tJ[RES_SLOTS];
  bool tok[RES_SLOTS];
  cx<double> a[RES_SLOTS][4][4];
#pragma unroll
  for (int sl = 0; sl < RES_SLOTS; ++sl) {
    const int t = (sl * RES_W + wv) * P + pg;
    tok[sl] = t < NT;
    tri_tile(tok[sl] ? t : 0, 0, tI[sl], tJ[sl]);
    const int r0 = 32 * tI[sl] + 4 * la, c0 = 32 * tJ[sl] + lb;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int r = r0 + q, c = c0 + 8 * p;
        a[sl][q][p] = (tok[sl] && r < m && c <= r) ? gram(r, c) : cx<double>{0, 0};
      }
  }
  for (int r = tid; r < MP; r += RES_NT) {
    col[r] = r < m ? gram(r, 0) : cx<double>{0, 0};
    vcur[r] = wv_[r] = cx<double>{0, 0};
    yq[2 * r] = yq[2 * r + 1] = 0ull;
    if (lead) {
      __hip_atomic_store(&ysum[2 * r], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&ysum[2 * r + 1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  group_sync_coherent(ctr, gen, P, info);

  for (int i = 0; i < m - 1; ++i) {
    const int buf = i % 3;
    unsigned long long* ys = ysum + (int64_t)buf * 2 * MP;
    cx<double>* cxb = colx + (int64_t)buf * MP;
    // (1) reflector from alpha = col[i + 1], x = col[i + 2 .. m - 1] (every workgroup)
    double s2 = 0;
    if (i == 0) {
      for (int r = i + 2 + tid; r < m; r += RES_NT) s2 += col[r].re * col[r].re + col[r].im * col[r].im;
      s2 = block_sum2<RES_W>(cx<double>{s2, 0.0}, red).re;
    } else {
      // formed with the column update of the previous step
#pragma unroll
      for (int w = 0; w < RES_W; ++w) s2 += red2[i & 1][w];
    }
    // every thread forms the same reflector from the same operands
    const double ar = col[i + 1].re, ai = col[i + 1].im;
    const bool skip = s2 == 0.0 && ai == 0.0;
    cx<double> tau{0, 0}, scale{0, 0};
    double ei = ar;
    if (!skip) {
      const double beta = -copysign(sqrt(ar * ar + ai * ai + s2), ar);
      tau = cx<double>{(beta - ar) / beta, -ai / beta};
      const double dr = ar - beta, di = ai;
      const double den = dr * dr + di * di;
      scale = cx<double>{dr / den, -di / den};
      ei = beta;
    }
    if (lead && tid == 0) {
      hv.d[i] = col[i].re;
      hv.e[i] = ei;
      hv.tau[i] = tau;
    }
    for (int r = tid; r < MP; r += RES_NT) {
      cx<double> v{0, 0};
      if (r == i + 1)
        v = cx<double>{1.0, 0.0};
      else if (r > i + 1 && r < m && !skip)
        v = cmulc(col[r], scale);
      vcur[r] = v;
      wv_[r] = cx<double>{0, 0};
      if (lead && r > i && r < m) Vout[(int64_t)i * m + r] = v;
      yq[2 * r] = yq[2 * r + 1] = 0ull;
    }
    __syncthreads();
    // (2) this workgroup's share of y = A_tr v over its resident tiles
    const int J0 = (i + 1) >> 5;
#pragma unroll
    for (int sl = 0; sl < RES_SLOTS; ++sl) {
      if (tok[sl] && tJ[sl] >= J0) {
        const int r0 = 32 * tI[sl] + 4 * la, c0 = 32 * tJ[sl] + lb;
        cx<double> yR[4], yC[4];
        if (tI[sl] > tJ[sl] && 32 * tJ[sl] >= i + 1 && 32 * tI[sl] + 32 <= m)
          symv_res<false>(a[sl], vcur, r0, c0, m, i + 1, yR, yC);
        else
          symv_res<true>(a[sl], vcur, r0, c0, m, i + 1, yR, yC);
        const cx<double> sr = reduce4<4, 2, 1>(yR, lane);
        const cx<double> sc = reduce4<32, 16, 8>(yC, lane);
        auto fix = [&](double x) { return (unsigned long long)(long long)rint(x * to_fix); };
        if (!(lane & 1)) {
          const int q = ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
          atomicAdd(&yq[2 * (r0 + q)], fix(sr.re));
          atomicAdd(&yq[2 * (r0 + q) + 1], fix(sr.im));
        }
        if (!(la & 1)) {
          const int p = ((la >> 2) & 1) * 2 + ((la >> 1) & 1);
          atomicAdd(&yq[2 * (c0 + 8 * p)], fix(sc.re));
          atomicAdd(&yq[2 * (c0 + 8 * p) + 1], fix(sc.im));
        }
      }
    }
    // column i + 1 as it stands before this step's update, from its owners
    const int Jn = (i + 1) >> 5;
#pragma unroll
    for (int sl = 0; sl < RES_SLOTS; ++sl) {
      if (tok[sl] && tJ[sl] == Jn) {
        const int r0 = 32 * tI[sl] + 4 * la, c0 = 32 * tJ[sl] + lb;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          if (c0 + 8 * p != i + 1) continue;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int r = r0 + q;
            if (r >= i + 1 && r < m) {
              double* d = reinterpret_cast<double*>(cxb + r);
              __hip_atomic_store(d, a[sl][q][p].re, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              __hip_atomic_store(d + 1, a[sl][q][p].im, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
          }
        }
      }
    }
    __syncthreads();
    // (3) add the share into the slice-wide sum; clear the sum of step i + 1
    unsigned long long* ysn = ysum + (int64_t)((i + 1) % 3) * 2 * MP;
    for (int r = i + 1 + tid; r < m; r += RES_NT) {
      const unsigned long long qr = yq[2 * r], qi = yq[2 * r + 1];
      if (qr) __hip_atomic_fetch_add(&ys[2 * r], qr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (qi) __hip_atomic_fetch_add(&ys[2 * r + 1], qi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lead)
      for (int r = i + 2 + tid; r < m; r += RES_NT) {
        __hip_atomic_store(&ysn[2 * r], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ysn[2 * r + 1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    group_sync_coherent(ctr, gen, P, info);
    // (4) y, then w = tau y + alpha v with alpha = -tau (w^H v) / 2 (rows i+1..m-1)
    cx<double> wl[2], cn[2];
    cx<double> dot{0, 0};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = i + 1 + tid + u * RES_NT;
      wl[u] = cn[u] = cx<double>{0, 0};
      if (r < m) {
        const long long qr = (long long)__hip_atomic_load(&ys[2 * r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const long long qi = (long long)__hip_atomic_load(&ys[2 * r + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double* d = reinterpret_cast<const double*>(cxb + r);
        cn[u] = cx<double>{__hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                           __hip_atomic_load(d + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
        const cx<double> yy{(double)qr * from_fix, (double)qi * from_fix};
        wl[u] = cmulc(tau, yy);
        cfmac(dot, wl[u], vcur[r]);
      }
    }
    dot = block_sum2<RES_W, false>(dot, red);
    const cx<double> alpha = cmulc(cx<double>{-0.5 * tau.re, -0.5 * tau.im}, dot);
    const bool zero = tau.re == 0.0 && tau.im == 0.0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = i + 1 + tid + u * RES_NT;
      if (r < m) {
        cx<double> w = wl[u];
        cfma(w, alpha, vcur[r]);
        wv_[r] = zero ? cx<double>{0, 0} : w;
      }
    }
    __syncthreads();
    // (5) A -= v w^H + w v^H on the resident tiles (v and w vanish outside the
    // trailing rows, so the finished rows and columns are left as they are)
#pragma unroll
    for (int sl = 0; sl < RES_SLOTS; ++sl) {
      if (tok[sl] && tJ[sl] >= J0) {
        const int r0 = 32 * tI[sl] + 4 * la, c0 = 32 * tJ[sl] + lb;
        cx<double> vc[4], wc[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          vc[p] = vcur[c0 + 8 * p];
          wc[p] = wv_[c0 + 8 * p];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const cx<double> vr = vcur[r0 + q], wr = wv_[r0 + q];
          const cx<double> nv{-vr.re, -vr.im}, nw{-wr.re, -wr.im};
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            cfmac(a[sl][q][p], wc[p], nv);
            cfmac(a[sl][q][p], vc[p], nw);
          }
        }
      }
    }
    // (6) column i + 1 after this step's update, in every workgroup, and the
    // per-wave partial sums of ||col[i + 3 ..]||^2 for the next reflector
    const cx<double> vi = vcur[i + 1], wi = wv_[i + 1];
    double s2n = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = i + 1 + tid + u * RES_NT;
      if (r < m) {
        cx<double> x = cn[u];
        const cx<double> nv{-vcur[r].re, -vcur[r].im}, nw{-wv_[r].re, -wv_[r].im};
        cfmac(x, wi, nv);
        cfmac(x, vi, nw);
        if (r == i + 1) x.im = 0.0;
        col[r] = x;
        if (r >= i + 3) s2n += x.re * x.re + x.im * x.im;
      }
    }
    s2n = wave_sum(s2n);
    if (lane == 0) red2[(i + 1) & 1][wv] = s2n;
    __syncthreads();
  }
  if (tid == 0 && lead) {
    hv.d[m - 1] = col[m - 1].re;
    hv.e[m - 1] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// 2. eigenvalues by multisection (8, 16 or 64 lanes per eigenvalue)
// ---------------------------------------------------------------------------
// Number of eigenvalues of T below x; de holds (d_i, e_{i-1}^2).
__device__ __forceinline__ int sturm_count(const double2* de, int m, double x, double pivmin) {
  int cnt = 0;
  double q = de[0].x - x;
  if (fabs(q) < pivmin) q = -pivmin;
  cnt += q < 0;
#pragma unroll 4
  for (int i = 1; i < m; ++i) {
    // e2 / q with the hardware reciprocal refined by one Newton step (a
    // relative perturbation of e2 at rounding level: the count stays the
    // exact count of a nearby tridiagonal matrix)
    const double2 t = de[i];
    double r = __builtin_amdgcn_rcp(q);
    r = r * fma(-q, r, 2.0);
    q = (t.x - x) - t.y * r;
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0;
  }
  return cnt;
}

__device__ __forceinline__ double wave_min(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// Gershgorin interval of T (widened), pivmin and ||T|| for one wave.
__device__ void tri_bounds(const double* d, const double* e, int m, double* gl, double* gu, double* pivmin,
                           double* tnorm) {
  const int lane = threadIdx.x & 63;
  double lo = 1e300, hi = -1e300, em = 0;
  for (int i = lane; i < m; i += 64) {
    const double r = fabs(e[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0);
    lo = fmin(lo, d[i] - r);
    hi = fmax(hi, d[i] + r);
    em = fmax(em, e[i] * e[i]);
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  em = wave_max(em);
  const double eps = 2.220446049250313e-16;
  const double tn = fmax(fabs(lo), fabs(hi));
  *pivmin = 2.2250738585072014e-308 * fmax(1.0, em);
  *tnorm = tn;
  *gl = lo - 2.0 * eps * tn * m - 2.0 * (*pivmin);
  *gu = hi + 2.0 * eps * tn * m + 2.0 * (*pivmin);
}

// Multisection with L lanes per eigenvalue, 64 / L eigenvalues per wave: each
// round places L points in the interval and keeps the one section that holds
// the eigenvalue.  Bound: the vector issue of m steps per round and wave when
// there are several waves per SIMD, the latency of that chain otherwise.  More
// lanes per eigenvalue mean fewer rounds (9 to 10 for L = 64, 13 for 16, 17 for
// 8) of more waves.  Small eigenvalues are resolved relative to themselves; the
// limit of rounds (an interval 1e-115 of the first) is met by exact zeros only.
template <int L>
__global__ __launch_bounds__(256) void heig_bisect_kernel(int m, int k, unsigned char* scratch, size_t per_slice,
                                                          double* __restrict__ lambda_out, int* info) {
  extern __shared__ __align__(16) unsigned char smem[];
  double2* de = reinterpret_cast<double2*>(smem);
  double* d = reinterpret_cast<double*>(de + m);
  double* e = d + m;
  const int f = blockIdx.x;
  HeigView hv = heig_view(scratch, per_slice, f, m);
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    d[i] = hv.d[i];
    e[i] = hv.e[i];
    const double ep = i > 0 ? hv.e[i - 1] : 0.0;
    de[i] = double2{hv.d[i], ep * ep};
  }
  __syncthreads();
  constexpr int E = 64 / L;  // eigenvalues per wave
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t0 = (blockIdx.y * (blockDim.x >> 6) + wave) * E;
  if (t0 >= k) return;
  const int g = lane / L, l = lane % L;
  const int t = min(t0 + g, k - 1);  // (a group past k repeats the last eigenvalue and does not store it)
  double lo, hi, pivmin, tnorm;
  tri_bounds(d, e, m, &lo, &hi, &pivmin, &tnorm);
  const int idx = m - 1 - t;
  const double eps = 2.220446049250313e-16;
  constexpr int ROUNDS = L >= 64 ? 64 : L >= 16 ? 94 : 121;  // (L + 1)^ROUNDS about 1e115
  bool done = false;
  for (int it = 0; it < ROUNDS; ++it) {
    if (hi - lo <= 2.0 * eps * fmax(fabs(lo), fabs(hi)) + 4.0 * pivmin) done = true;
    if (__ballot(!done) == 0ull) break;
    const double x = lo + (hi - lo) * (double)(l + 1) / (double)(L + 1);
    const int cnt = sturm_count(de, m, x, pivmin);
    unsigned long long above = __ballot(cnt > idx) >> (g * L);  // lanes whose point lies above lambda_idx
    if (L < 64) above &= (1ull << (L & 63)) - 1;
    const int p = above ? __ffsll((long long)above) - 1 : L;  // first such lane of the group
    const double xp = __shfl(x, g * L + (p < L ? p : L - 1), 64);
    const double xm = __shfl(x, g * L + (p > 0 ? p - 1 : 0), 64);
    const double nlo = p > 0 ? xm : lo;
    const double nhi = p < L ? xp : hi;
    if (done) continue;
    if (nlo == lo && nhi == hi) done = true;
    lo = nlo;
    hi = nhi;
  }
  if (l == 0 && t0 + g < k) {
    const double lv = 0.5 * (lo + hi);
    lambda_out[(int64_t)f * k + t] = lv;
    if (!isfinite(lv)) atomicAdd(&info[INFO_NONFINITE], 1);
  }
}

// ---------------------------------------------------------------------------
// 3. eigenvectors of T by inverse iteration (one lane per eigenvector)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double hash_uniform(uint32_t a, uint32_t b) {
  uint32_t h = a * 0x9E3779B1u ^ (b + 0x7F4A7C15u) * 0x85EBCA77u;
  h ^= h >> 15;
  h *= 0x2C1B3C6Du;
  h ^= h >> 12;
  h *= 0x297A2D39u;
  h ^= h >> 15;
  return (double)h * (2.0 / 4294967296.0) - 1.0;
}

// Eigenvalues closer than INVIT_ORTOL ||T|| form a cluster, whose vectors are
// orthogonalised against each other afterwards (heig_cluster_kernel); those
// further apart carry a contamination of at most about eps / 1e-9 = 2e-7 by
// their neighbours.
constexpr double INVIT_ORTOL = 1e-9;
constexpr int INVIT_B = 8;

// One lane's shifted solves with T (in LDS, scaled to ||T|| in [1, 2)): the pivoted
// LU of T - lambda I and its two substitutions, chains of mp dependent steps.
// Rows go in batches of INVIT_B: a batch's operands are read from LDS together,
// so the chain waits for LDS once per batch.  The rows are padded to whole batches
// by uncoupled ones, so that no row takes a branch.  The lanes' arrays are
// interleaved with stride nl (the swap bits with ss).  The entry right of the
// pivot follows from T, the multipliers and the row-swap bits.
struct ShiftedT {
  const double *d, *e;   // mp + 1 each
  double *R, *Mu, *Z;    // mp each: 1 / pivot, multipliers, the iterate
  unsigned char* swaps;  // mp / INVIT_B: swap bits of a batch
  int mp, nl, ss;
  double lv;

  // LU with row interchanges; pivots are kept at or above eps in modulus
  __device__ __forceinline__ void factor() const {
    constexpr int B = INVIT_B;
    const double eps = 2.220446049250313e-16;
    double pc = d[0] - lv, qc = e[0];
    for (int i0 = 0; i0 < mp; i0 += B) {
      double dn[B], eb[B + 1];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        dn[u] = d[i0 + u + 1] - lv;
        eb[u] = e[i0 + u];
      }
      eb[B] = e[i0 + B];
      unsigned bits = 0;
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const double ei = eb[u], an = dn[u], en = eb[u + 1];
        const bool sw = fabs(pc) < fabs(ei);
        double den = sw ? ei : pc;
        den = fabs(den) < eps ? copysign(eps, den) : den;
        double r = __builtin_amdgcn_rcp(den);
        r = fma(fma(-den, r, 1.0), r, r);
        r = fma(fma(-den, r, 1.0), r, r);
        const double mu = (sw ? pc : ei) * r;
        pc = fma(-mu, sw ? an : qc, sw ? qc : an);
        qc = sw ? -mu * en : en;
        R[(i0 + u) * nl] = r;
        Mu[(i0 + u) * nl] = mu;
        bits |= (unsigned)sw << u;
      }
      swaps[(i0 / B) * ss] = (unsigned char)bits;
    }
  }

  // forward elimination of Z * scale, in place
  __device__ __forceinline__ void forward(double scale) const {
    constexpr int B = INVIT_B;
    double zc = Z[0] * scale;
    for (int i0 = 0; i0 < mp; i0 += B) {
      const unsigned bits = swaps[(i0 / B) * ss];
      double zb[B], mb[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        zb[u] = Z[(u < B - 1 ? i0 + u + 1 : min(i0 + B, mp - 1)) * nl] * scale;
        mb[u] = Mu[(i0 + u) * nl];
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const bool sw = (bits >> u) & 1u;
        const double x = sw ? zb[u] : zc, y = sw ? zc : zb[u];
        Z[(i0 + u) * nl] = x;  // (the last row neither swaps nor feeds another)
        zc = fma(-mb[u], x, y);
      }
    }
  }

  // Back substitution into Z, of Z or of rhs(i): the entries right of the pivot
  // are (d_{i+1} - lambda, e_{i+1}) in a swapped row, else e_i, or -mu_{i-1} e_i
  // behind a swapped row.  Returns ||z||^2.
  template <typename Rhs>
  __device__ __forceinline__ double back(Rhs rhs) const {
    constexpr int B = INVIT_B;
    double z1 = 0.0, z2 = 0.0, nrm = 0.0;
    for (int i0 = mp - B; i0 >= 0; i0 -= B) {
      const unsigned bits = swaps[(i0 / B) * ss];
      const unsigned low = i0 > 0 ? swaps[(i0 / B - 1) * ss] >> (B - 1) : 0;  // row i0 - 1 swapped
      double cb[B], mb[B], rb[B], db[B], eb[B + 1];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int i = i0 + u;
        cb[u] = rhs(i);
        mb[u] = Mu[(u > 0 ? i - 1 : max(i - 1, 0)) * nl];
        rb[u] = R[i * nl];
        db[u] = d[i + 1] - lv;
        eb[u] = e[i];
      }
      eb[B] = e[i0 + B];
#pragma unroll
      for (int u = B - 1; u >= 0; --u) {
        const bool sw = (bits >> u) & 1u, swp = (u > 0 ? bits >> (u > 0 ? u - 1 : 0) : low) & 1u;
        const double r1 = sw ? db[u] : (swp ? -mb[u] * eb[u] : eb[u]);
        const double r2 = sw ? eb[u + 1] : 0.0;
        const double v = fma(-r1, z1, fma(-r2, z2, cb[u])) * rb[u];
        Z[(i0 + u) * nl] = v;
        nrm = fma(v, v, nrm);
        z2 = z1;
        z1 = v;
      }
    }
    return nrm;
  }
  __device__ __forceinline__ double back() const {
    return back([&](int i) { return Z[i * nl]; });
  }
};

// Factor that brings ||T|| into [1, 2).
__device__ __forceinline__ double unit_scale(double tnorm) {
  int ex = 0;
  (void)frexp(tnorm, &ex);
  return isfinite(tnorm) && tnorm > 0.0 ? ldexp(1.0, 1 - ex) : 1.0;
}

// One eigenvector per lane, nl of them per one-wave workgroup: the chains of all
// lanes cost what one did when a wave walked one.  Bound: the latency of those
// chains (about 4 m steps).  The reciprocal pivots, multipliers and iterate of
// the lanes are in LDS (24 m nl bytes; fetched from memory instead, the chains
// ran at a third of the speed).
__global__ __launch_bounds__(64) void heig_invit_kernel(int m, int k, int nl, unsigned char* scratch, size_t per_slice,
                                                        const double* __restrict__ lambda, cx<double>* Wout, int* info,
                                                        double vfloor_rel, const int* __restrict__ nvec) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int B = INVIT_B;
  const int mp = (m + B - 1) / B * B;
  double* d = reinterpret_cast<double*>(smem);                // mp + 1
  double* e = d + mp + 1;                                     // mp + 1
  double* R = e + mp + 1;                                     // mp x nl: 1 / pivot
  double* Mu = R + mp * nl;                                   // mp x nl: multipliers
  double* Z = Mu + mp * nl;                                   // mp x nl: the iterate
  unsigned char* swaps = reinterpret_cast<unsigned char*>(Z + mp * nl);  // mp / B x 64: swap bits of a batch
  const int f = blockIdx.x, lane = threadIdx.x;
  HeigView hv = heig_view(scratch, per_slice, f, m);
  for (int i = lane; i <= mp; i += 64) {
    d[i] = i < m ? hv.d[i] : 4.0;
    e[i] = i + 1 < m ? hv.e[i] : 0.0;
  }
  __syncthreads();
  double gl, gu, pivmin, tnorm;
  tri_bounds(d, e, m, &gl, &gu, &pivmin, &tnorm);
  const int t = blockIdx.y * nl + lane;
  const double* lam = lambda + (int64_t)f * k;
  cx<double>* W = Wout + (int64_t)f * m * k + t;
  const bool act = lane < nl && t < k;
  const double up = unit_scale(tnorm);
  __syncthreads();
  for (int i = lane; i < m; i += 64) {
    d[i] *= up;  // (the padding rows keep 4: off any eigenvalue)
    e[i] *= up;
  }
  __syncthreads();
  if (!act) return;  // (one wave, no barrier below)
  // a vector that is not wanted (see heig_topk) is zero
  if ((nvec && t >= nvec[f]) || (vfloor_rel > 0.0 && !(lam[t] > vfloor_rel * lam[0]))) {
    for (int i = 0; i < m; ++i) W[(int64_t)i * k] = cx<double>{0.0, 0.0};
    return;
  }
  if (tnorm == 0.0) {  // the zero matrix: unit vectors
    for (int i = 0; i < m; ++i) W[(int64_t)i * k] = cx<double>{i == t ? 1.0 : 0.0, 0.0};
    return;
  }
  const double eps = 2.220446049250313e-16;
  const ShiftedT s{d, e, R + lane, Mu + lane, Z + lane, swaps + lane, mp, nl, 64, lam[t] * up};
  s.factor();
  // a random right-hand side (zero in the padding rows)
  double nrm = s.back([&](int i) { return i < m ? hash_uniform((uint32_t)t, (uint32_t)i) : 0.0; });
  double scale = nrm > 0.0 ? 1.0 / sqrt(nrm) : 0.0, res = 1.0;
  for (int it = 1; it < 4; ++it) {
    s.forward(scale);
    nrm = s.back();
    // the right-hand side had norm 1 (from the second solve on), so the
    // normalised iterate's residual is 1 / ||z||
    scale = nrm > 0.0 ? 1.0 / sqrt(nrm) : 0.0;
    res = nrm > 0.0 && isfinite(nrm) ? scale : 1.0;
    if (__ballot(!(res <= 16.0 * m * eps)) == 0ull) break;
  }
  if (!(res <= 1e3 * m * eps)) atomicAdd(&info[INFO_EIG_NOCONV], 1);
#pragma unroll 4
  for (int i = 0; i < m; ++i) W[(int64_t)i * k] = cx<double>{s.Z[i * nl] * scale, 0.0};
}

// Orthogonalisation inside the clusters of close eigenvalues, one workgroup per
// slice: classical Gram-Schmidt, twice, in the order of the eigenvalues.  The
// members come out of independent random starts, so they span the cluster's
// invariant subspace, and a combination of members stays within the cluster's
// width (below 1e-9 ||T|| per gap, weighted by the members' contamination eps /
// gap) of an eigenvector.  Where the eigenvalues of a cluster differ by less than
// their rounding, its members lean towards the same few directions; what
// Gram-Schmidt leaves of the later ones is short, and rescaling it raises its
// rounding error.  So each member's residual is measured, and while it is above
// 16 eps ||T|| the member is solved for and orthogonalised again, up to three
// times (190 equal eigenvalues of 192: residual 1e-11 ||T|| without, 2e-14 with).
// A slice without clusters returns at once.
__global__ __launch_bounds__(256) void heig_cluster_kernel(int m, int k, unsigned char* scratch, size_t per_slice,
                                                           const double* __restrict__ lambda, cx<double>* Wout,
                                                           int* info, double vfloor_rel, const int* __restrict__ nvec,
                                                           int lds_cols) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int B = INVIT_B;
  const int mp = (m + B - 1) / B * B;
  double* lam = reinterpret_cast<double*>(smem);  // k
  double* coef = lam + k;                         // k
  double* d = coef + k;                           // mp + 1: T, as in heig_invit_kernel
  double* e = d + mp + 1;                         // mp + 1
  double* R = e + mp + 1;                         // mp
  double* Mu = R + mp;                            // mp
  double* cur = Mu + mp;                          // mp: the vector being orthogonalised
  double* buf = cur + mp;                         // lds_cols x m: the cluster's earlier members
  unsigned char* swaps = reinterpret_cast<unsigned char*>(buf + (size_t)lds_cols * m);  // mp / B
  __shared__ double red[8];
  const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  HeigView hv = heig_view(scratch, per_slice, f, m);
  cx<double>* W = Wout + (int64_t)f * m * k;
  for (int t = tid; t < k; t += 256) lam[t] = lambda[(int64_t)f * k + t];
  double tn = 0;
  for (int i = lane; i < m; i += 64) {
    const double r = (i + 1 < m ? fabs(hv.e[i]) : 0.0) + (i > 0 ? fabs(hv.e[i - 1]) : 0.0);
    tn = fmax(tn, fabs(hv.d[i]) + r);
  }
  tn = wave_max(tn);
  __syncthreads();
  const double ortol = INVIT_ORTOL * tn;
  const double vfloor = vfloor_rel > 0.0 ? vfloor_rel * lam[0] : -1e300;
  bool any = false;
  const int nv = nvec ? nvec[f] : k;
  for (int t = 1 + tid; t < nv; t += 256) any |= lam[t - 1] - lam[t] < ortol;
  if (!__syncthreads_or(any)) return;
  const double eps = 2.220446049250313e-16, up = unit_scale(tn);
  for (int i = tid; i <= mp; i += 256) {
    d[i] = i < m ? hv.d[i] * up : 4.0;
    e[i] = i + 1 < m ? hv.e[i] * up : 0.0;
    if (i < mp) cur[i] = 0.0;
  }
  __syncthreads();
  for (int t0 = 0; t0 + 1 < nv;) {
    int t1 = t0 + 1;
    while (t1 < nv && lam[t1 - 1] - lam[t1] < ortol && (!(vfloor_rel > 0.0) || lam[t1] > vfloor)) ++t1;
    const int n = t1 - t0;
    const bool in_lds = n <= lds_cols;
    auto member = [&](int c, int i) { return in_lds ? buf[(size_t)c * m + i] : W[(int64_t)i * k + t0 + c].re; };
    for (int j = 0; n > 1 && j < n; ++j) {
      const ShiftedT st{d, e, R, Mu, cur, swaps, mp, 1, 1, lam[t0 + j] * up};
      for (int i = tid; i < m; i += 256) cur[i] = W[(int64_t)i * k + t0 + j].re;
      __syncthreads();
      double sc = 0.0;
      int it = 0;
      for (;; ++it) {
        for (int pass = 0; pass < 2 && j > 0; ++pass) {
          for (int c = wv; c < j; c += 4) {
            double s = 0;
            for (int i = lane; i < m; i += 64) s = fma(member(c, i), cur[i], s);
            s = wave_sum(s);
            if (lane == 0) coef[c] = s;
          }
          __syncthreads();
          for (int i = tid; i < m; i += 256) {
            double s = cur[i];
            for (int c = 0; c < j; ++c) s = fma(-coef[c], member(c, i), s);
            cur[i] = s;
          }
          __syncthreads();
        }
        // squared norms of the vector and of (T - lambda) times it
        cx<double> ss{0.0, 0.0};
        for (int i = tid; i < m; i += 256) {
          const double x = cur[i];
          const double y = fma(d[i] - st.lv, x, fma(i > 0 ? e[i - 1] : 0.0, i > 0 ? cur[i - 1] : 0.0,
                                                    e[i] * (i + 1 < m ? cur[i + 1] : 0.0)));
          ss.re = fma(x, x, ss.re);
          ss.im = fma(y, y, ss.im);
        }
        ss = block_sum2<4>(ss, red);
        sc = ss.re > 0 ? 1.0 / sqrt(ss.re) : 0.0;
        const double res = sqrt(ss.im) * sc;
        if (sc > 0.0 && res <= 16.0 * eps) break;
        if (it == 3) {
          if (tid == 0 && !(sc > 0.0 && res <= 1e3 * m * eps)) atomicAdd(&info[INFO_EIG_NOCONV], 1);
          break;
        }
        if (tid == 0) {
          if (it == 0) st.factor();
          st.forward(sc);
          st.back();
        }
        __syncthreads();
      }
      for (int i = tid; i < m; i += 256) {
        const double x = cur[i] * sc;
        if (in_lds) buf[(size_t)j * m + i] = x;
        if (j > 0 || it > 0) W[(int64_t)i * k + t0 + j].re = x;
      }
      __syncthreads();
    }
    t0 = t1;
  }
}

// ---------------------------------------------------------------------------
// 4. back-transformation W = H_0 ... H_{m-2} Z (8 columns per workgroup)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void heig_backxf_kernel(int m, int k, unsigned char* scratch, size_t per_slice,
                                                          cx<double>* __restrict__ Wout) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NC = 8;
  cx<double>* Wl = reinterpret_cast<cx<double>*>(smem);  // m x NC
  cx<double>* vl = Wl + (size_t)m * NC;                   // m
  __shared__ cx<double> sc[NC];
  const int f = blockIdx.x;
  const int c0 = blockIdx.y * NC;
  const int tid = threadIdx.x;
  HeigView hv = heig_view(scratch, per_slice, f, m);
  cx<double>* W = Wout + (int64_t)f * m * k;
  for (int idx = tid; idx < m * NC; idx += 256) {
    const int r = idx / NC, g = idx % NC;
    Wl[idx] = (c0 + g < k) ? W[(int64_t)r * k + c0 + g] : cx<double>{0, 0};
  }
  __syncthreads();
  const int g = tid >> 5, l32 = tid & 31;
  constexpr int PF = 4;  // v elements per thread held in registers (m <= 1024)
  cx<double> nxt[PF];
  auto fetch = [&](int j) {
    const int L = m - j - 1;
    const cx<double>* vg = hv.A + (int64_t)j * m + (j + 1);
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int i = tid + u * 256;
      nxt[u] = i < L ? vg[i] : cx<double>{0, 0};
    }
  };
  if (m >= 2) fetch(m - 2);
  for (int j = m - 2; j >= 0; --j) {
    const cx<double> tau = hv.tau[j];
    const int L = m - j - 1;
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int i = tid + u * 256;
      if (i < L) vl[i] = nxt[u];
    }
    if (j > 0) fetch(j - 1);
    if (tau.re == 0.0 && tau.im == 0.0) continue;
    __syncthreads();
    double sr = 0, si = 0;
    for (int i = l32; i < L; i += 32) {
      const cx<double> t = cjmul(vl[i], Wl[(j + 1 + i) * NC + g]);
      sr += t.re;
      si += t.im;
    }
    for (int o = 16; o > 0; o >>= 1) {
      sr += __shfl_xor(sr, o, 64);
      si += __shfl_xor(si, o, 64);
    }
    if (l32 == 0) sc[g] = cmulc(tau, cx<double>{sr, si});
    __syncthreads();
    for (int idx = tid; idx < L * NC; idx += 256) {
      const int i = idx / NC, gg = idx % NC;
      const cx<double> t = cmulc(vl[i], sc[gg]);
      cx<double>& w = Wl[(j + 1 + i) * NC + gg];
      w.re -= t.re;
      w.im -= t.im;
    }
    __syncthreads();
  }
  for (int idx = tid; idx < m * NC; idx += 256) {
    const int r = idx / NC, gg = idx % NC;
    if (c0 + gg < k) W[(int64_t)r * k + c0 + gg] = Wl[idx];
  }
}

// Back-transformation with the columns in registers: each half-wave owns one
// of the workgroup's 8 columns of W (rows l32 + 32 s), so the product with a
// reflector and the update need only lane exchanges.  The reflectors pass
// through LDS in groups of NB (double-buffered by group; the next group is
// fetched into registers while the current one is applied), one workgroup
// barrier per group: the NB reflectors of a group are applied in order
// with no barrier between them, since no half-wave reads another's column.
// Bound by the chain of one reflector: S LDS reads, S dependent FMAs, the lane
// sum, S more.  Reflectors are stored over all 32 S rows with their zeros, so
// that no read is conditional, the scalar factors lie in LDS, and the sum goes
// through DPP: 78 us for 180 rows (2 slices), 14 for 30 (9 slices), 147 for 150
// (129 slices), where guarded reads, factors from memory and LDS shuffles took
// 191, 31 and 356.
template <int S, int NB>
__global__ __launch_bounds__(256) void heig_backxf2_kernel(int m, int k, unsigned char* scratch, size_t per_slice,
                                                           cx<double>* __restrict__ Wout) {
  constexpr int MP = 32 * S;
  extern __shared__ __align__(16) unsigned char smem[];
  cx<double>* vbuf = reinterpret_cast<cx<double>*>(smem);  // 2 groups x NB x MP
  cx<double>* tau = vbuf + 2 * NB * MP;                    // MP
  const int f = blockIdx.x;
  const int tid = threadIdx.x, g = tid >> 5, l32 = tid & 31;
  const int col = blockIdx.y * 8 + g;
  const bool colok = col < k;
  HeigView hv = heig_view(scratch, per_slice, f, m);
  cx<double>* W = Wout + (int64_t)f * m * k;
  for (int i = tid; i < m - 1; i += 256) tau[i] = hv.tau[i];
  cx<double> w[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int r = l32 + 32 * s;
    w[s] = (colok && r < m) ? W[(int64_t)r * k + col] : cx<double>{0, 0};
  }
  constexpr int PF = (MP + 255) / 256;  // rows per thread and reflector
  // reflectors j0 .. 0 in descending order; group q holds j = j0 - q NB - u, u < NB
  const int j0 = m - 2;
  const int ng = (j0 + NB) / NB;
  cx<double> pre[NB][PF];
  auto fetch = [&](int q) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int j = max(j0 - q * NB - u, 0);
#pragma unroll
      for (int p = 0; p < PF; ++p) pre[u][p] = hv.A[(int64_t)j * m + min(max(tid + p * 256, j + 1), m - 1)];
    }
  };
  auto stage = [&](int q) {
    cx<double>* vb = vbuf + (q & 1) * NB * MP;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int j = j0 - q * NB - u;
#pragma unroll
      for (int p = 0; p < PF; ++p) {
        const int r = tid + p * 256;
        if (r < MP) vb[u * MP + r] = r > j && r < m ? pre[u][p] : cx<double>{0, 0};
      }
    }
  };
  auto apply = [&](int j, const cx<double>* vb) {
    const cx<double> t = tau[j];
    if (t.re == 0.0 && t.im == 0.0) return;
    // the lane's entries of the reflector are read from LDS once, for both
    // the product and the update
    cx<double> vv[S];
#pragma unroll
    for (int s = 0; s < S; ++s) vv[s] = vb[l32 + 32 * s];
    double a0 = 0, a1 = 0, b0 = 0, b1 = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      a0 = fma(vv[s].re, w[s].re, a0);
      b0 = fma(vv[s].re, w[s].im, b0);
      a1 = fma(vv[s].im, w[s].im, a1);
      b1 = fma(vv[s].im, w[s].re, b1);
    }
    const cx<double> sc = cmulc(t, cx<double>{half_sum(a0 + a1), half_sum(b0 - b1)});
#pragma unroll
    for (int s = 0; s < S; ++s) {
      w[s].re = fma(-vv[s].re, sc.re, fma(vv[s].im, sc.im, w[s].re));
      w[s].im = fma(-vv[s].re, sc.im, fma(-vv[s].im, sc.re, w[s].im));
    }
  };
  if (ng > 0) {
    fetch(0);
    stage(0);
    if (ng > 1) fetch(1);
  }
  __syncthreads();
  for (int q = 0; q < ng; ++q) {
    const cx<double>* vb = vbuf + (q & 1) * NB * MP;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int j = j0 - q * NB - u;
      if (j >= 0) apply(j, vb + u * MP);
    }
    if (q + 1 < ng) {
      stage(q + 1);
      if (q + 2 < ng) fetch(q + 2);
    }
    lds_barrier();
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int r = l32 + 32 * s;
    if (colok && r < m) W[(int64_t)r * k + col] = w[s];
  }
}

hipError_t heig_topk(const double* Gpart, int nsum, int64_t part_stride, int m, int k, int batch, double* lambda,
                     double* W, void* scratch, int* info, hipStream_t s, int stages, bool upper_only,
                     double vfloor_rel, const int* nvec) {
  if (batch <= 0) return hipSuccess;
  if (m > 1024 || k > m || k < 1) return hipErrorInvalidValue;
  static bool attr_set = false;
  if (!attr_set) {
    // dynamic LDS limits, leaving room for each kernel's static LDS
    (void)hipFuncSetAttribute((const void*)heig_tri2_kernel<8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              152 * 1024);
    (void)hipFuncSetAttribute((const void*)heig_tri2_kernel<4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024 - 256);
    (void)hipFuncSetAttribute((const void*)heig_tri2_kernel<2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              152 * 1024);
    (void)hipFuncSetAttribute((const void*)heig_backxf_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                              152 * 1024);
    (void)hipGetLastError();
    attr_set = true;
  }
  const size_t per = heig_per_slice(m, k);
  unsigned char* sc = (unsigned char*)scratch;
  const size_t lds_total = 150 * 1024;
  hipError_t e = hipSuccess;
  // 1. tridiagonalisation.  Up to TREG_MAX rows the triangle fits one
  // workgroup's registers: 1.6 to 4.4 us per step, against 3.5 to 10 us for the
  // streaming form at the same sizes and about 8.5 us with several workgroups
  // per slice (an exchange through memory in every step).
  const int MP = (m + 31) / 32 * 32;
  auto sm2 = [&](int nb) { return ((size_t)(2 * nb + 3) * MP + 2 * nb) * sizeof(cx<double>); };
  if ((stages & HEIG_TRIDIAG) && m <= TREG_MAX) {
    if ((e = heig_tridiag_reg((const cx<double>*)Gpart, nsum, part_stride, m, batch, sc, per, upper_only ? 1 : 0, s)) !=
        hipSuccess)
      return e;
  } else if (stages & HEIG_TRIDIAG) {
    // the panel's vectors in LDS: 8 reflectors up to m = 480, 4 up to 928 (all of a
    // CU's 160 KB but the static part), 2 above
    const int nb = sm2(8) <= lds_total ? 8 : sm2(4) <= 160 * 1024 - 256 ? 4 : 2;
    const size_t sm = sm2(nb);
    const void* fn = nb == 8   ? (const void*)heig_tri2_kernel<8>
                     : nb == 4 ? (const void*)heig_tri2_kernel<4>
                               : (const void*)heig_tri2_kernel<2>;
    hipLaunchKernelGGL(heig_prep_kernel, dim3(batch, PREP_WG), dim3(256), 0, s, (const cx<double>*)Gpart, nsum,
                       part_stride, m, upper_only ? 1 : 0, sc, per);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // several co-resident workgroups per slice for large m when the slices
    // leave CUs idle (cooperative launch guarantees co-residency)
    int P = 1;
    if (m >= 256) {
      static int coop = -1, cus = 0;
      if (coop < 0) {
        int dev = 0;
        coop = 0;
        if (hipGetDevice(&dev) == hipSuccess) {
          (void)hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev);
          (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        }
        (void)hipGetLastError();
      }
      if (coop > 0 && cus > 0) P = std::min(TRI_PMAX, cus / batch);
      if (P < 2) P = 1;
    }
    const cx<double>* G = (const cx<double>*)Gpart;
    int nsum_a = nsum, m_a = m, mp_a = MP, up = upper_only ? 1 : 0;
    int64_t ps = part_stride;
    unsigned char* sc_a = sc;
    size_t per_a = per;
    int* info_a = info;
    // the register-resident form when the slice's tiles fit RES_SLOTS per wave
    const int NTt = (MP / 32) * (MP / 32 + 1) / 2;
    bool done = false;
    if (P > 1 && MP <= 2 * RES_NT && NTt <= RES_SLOTS * RES_W * P) {
      void* args[] = {(void*)&G, (void*)&nsum_a, (void*)&ps, (void*)&m_a, (void*)&mp_a, (void*)&sc_a, (void*)&per_a,
                      (void*)&up, (void*)&P, (void*)&info_a};
      if (hipLaunchCooperativeKernel((const void*)heig_trires_kernel, dim3(batch * P), dim3(RES_NT), args, 0, s) ==
          hipSuccess)
        done = true;
      else
        (void)hipGetLastError();  // not co-resident: the streaming form below
    }
    if (!done && P > 1) {
      void* args[] = {(void*)&G, (void*)&nsum_a, (void*)&ps, (void*)&m_a, (void*)&mp_a, (void*)&sc_a, (void*)&per_a,
                      (void*)&up, (void*)&P, (void*)&info_a};
      if (hipLaunchCooperativeKernel(fn, dim3(batch * P), dim3(T2_NT), args, (unsigned)sm, s) != hipSuccess) {
        (void)hipGetLastError();  // not co-resident at this size: one workgroup per slice
        P = 1;
      }
    }
    if (P == 1) {
      auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(batch), dim3(T2_NT), sm, s, G, nsum_a, ps, m_a, mp_a, sc_a, per_a, up, 1, info_a);
      };
      if (nb == 8)
        go(heig_tri2_kernel<8>);
      else if (nb == 4)
        go(heig_tri2_kernel<4>);
      else
        go(heig_tri2_kernel<2>);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // 2. eigenvalues: 4 waves per workgroup.  With at most one wave per SIMD
  // (1024 of them) 64 lanes per eigenvalue take the fewest rounds; past that the
  // waves share issue slots and fewer lanes per eigenvalue cost less.
  if (stages & HEIG_BISECT) {
    const size_t sm = (size_t)4 * m * sizeof(double);
    const int64_t n = (int64_t)batch * k;
    auto go = [&](auto kernel, int per_wave) {
      hipLaunchKernelGGL(kernel, dim3(batch, (k + 4 * per_wave - 1) / (4 * per_wave)), dim3(256), sm, s, m, k, sc, per,
                         lambda, info);
    };
    if (n <= 1024)
      go(heig_bisect_kernel<64>, 1);
    else if (n <= 4096)
      go(heig_bisect_kernel<16>, 4);
    else
      go(heig_bisect_kernel<8>, 8);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // 3. eigenvectors: g workgroups per slice with nl = ceil(k / g) lanes each.
  // The time is a chain of about 4 m steps per round of workgroups whatever nl
  // is, so g is the smallest count with the fewest rounds over the CUs (an LDS
  // of 160 KB holds one workgroup or several); then the clusters.
  if (stages & HEIG_INVIT) {
    const size_t lds_cu = 160 * 1024;
    auto lds_of = [&](int nl) {
      const size_t mp = (size_t)(m + INVIT_B - 1) / INVIT_B * INVIT_B;
      return 16 * (mp + 1) + 24 * mp * nl + mp / INVIT_B * 64;
    };
    int best = 0;
    int64_t best_rounds = 0;
    for (int g = (k + 63) / 64; g <= k; ++g) {
      const size_t lds = lds_of((k + g - 1) / g);
      if (lds > lds_cu) continue;
      const int64_t slots = 256 * (int64_t)std::min<size_t>(lds_cu / lds, 8);
      const int64_t rounds = ((int64_t)batch * g + slots - 1) / slots;
      if (best == 0 || rounds < best_rounds) {
        best = g;
        best_rounds = rounds;
      }
      if (best_rounds == 1) break;
    }
    const int nl = (k + best - 1) / best;
    const size_t sm3 = lds_of(nl);
    if ((e = hipFuncSetAttribute((const void*)heig_invit_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)lds_cu)) != hipSuccess)
      return e;
    hipLaunchKernelGGL(heig_invit_kernel, dim3(batch, (k + nl - 1) / nl), dim3(64), sm3, s, m, k, nl, sc, per, lambda,
                       (cx<double>*)W, info, vfloor_rel, nvec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (k > 1) {
      // up to 60 KB of members in LDS beside T, its factors and the coefficients (at most 58)
      const size_t mp = (size_t)(m + INVIT_B - 1) / INVIT_B * INVIT_B;
      const size_t base = (2 * k + 2 * (mp + 1) + 3 * mp) * sizeof(double) + mp / INVIT_B;
      const int cols = (int)std::min<size_t>(k, 60 * 1024 / (m * sizeof(double)));
      if ((e = hipFuncSetAttribute((const void*)heig_cluster_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   120 * 1024)) != hipSuccess)
        return e;
      hipLaunchKernelGGL(heig_cluster_kernel, dim3(batch), dim3(256), base + (size_t)cols * m * sizeof(double), s, m, k,
                         sc, per, lambda, (cx<double>*)W, info, vfloor_rel, nvec, cols);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  // 4. back-transformation
  const size_t sm4 = ((size_t)m * 8 + m) * sizeof(cx<double>);
  if (stages & HEIG_BACKXF) {
    // two LDS groups of NB reflectors over the padded rows: 4 up to m = 448 (63
    // KB with the factors), 2 above
    const dim3 g5(batch, (k + 7) / 8);
#define TSVD_BACKXF(S, NB)                                                                                     \
  hipLaunchKernelGGL((heig_backxf2_kernel<S, NB>), g5, dim3(256), (2 * NB + 1) * 32 * S * sizeof(cx<double>), s, m, k, \
                     sc, per, (cx<double>*)W)
    if (m <= 32)
      TSVD_BACKXF(1, 4);
    else if (m <= 64)
      TSVD_BACKXF(2, 4);
    else if (m <= 128)
      TSVD_BACKXF(4, 4);
    else if (m <= 192)
      TSVD_BACKXF(6, 4);
    else if (m <= 256)
      TSVD_BACKXF(8, 4);
    else if (m <= 448)
      TSVD_BACKXF(14, 4);
    else if (m <= 640)
      TSVD_BACKXF(20, 2);
#undef TSVD_BACKXF
    else
      hipLaunchKernelGGL(heig_backxf_kernel, dim3(batch, (k + 7) / 8), dim3(256), sm4, s, m, k, sc, per,
                         (cx<double>*)W);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace tsvd
