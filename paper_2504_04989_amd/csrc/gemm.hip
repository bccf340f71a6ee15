// Batched complex GEMM on gfx950 MFMA (16x16x4 f32 / f64).
//
// Complex products use four real MFMA streams per output tile
// (re += ar br - ai bi, im += ar bi + ai br); operands are staged through LDS
// in planar re / im arrays whose layout follows the global layout so that
// both the coalesced global loads and the MFMA fragment reads stay
// bank-conflict-light.  One 256-thread workgroup (4 waves) owns a BM x BN
// output tile; each wave owns a (BM/WM) x (BN/WN) sub-tile of 16x16 MFMA
// tiles.  A K step is 128 bytes of a row (16 values of FP32, 8 of FP64); the
// next one is read into registers while the current one is multiplied out of
// LDS, and LDS is double-buffered, so that a step has one barrier.
//
// What bounds these products is the latency of their operand reads: K is
// short (a rank, a block width, one side of a slice) and a wave has only 8 to
// 64 MFMAs per step to hide it.  With a bounds check around every read, each
// waited for before the next was issued, and one 64 x 64 tile for all shapes,
// the products ran at 20 to 90 TF in FP32 and 8 to 44 in FP64; with all reads
// of a step in flight at clamped addresses and the tile chosen by shape at 50
// to 95 and 17 to 53 (2000 x 30 x 2000 FP32 over 9 slices 438 -> 159 us,
// 256 x 50 x 256 FP64 over 129 slices 154 -> 103 us).
#include "common.h"
#include "kernels.h"

namespace tsvd {

template <typename S, typename T>
__device__ __forceinline__ void ld_cx(const void* base, int64_t idx, T& re, T& im) {
  const cx<S> v = reinterpret_cast<const cx<S>*>(base)[idx];
  re = static_cast<T>(v.re);
  im = static_cast<T>(v.im);
}

// x where keep, else +0 (by bits: an Inf or NaN of a clamped read leaves nothing).
__device__ __forceinline__ float keep_if(float x, bool keep) {
  return __uint_as_float(__float_as_uint(x) & (keep ? 0xffffffffu : 0u));
}
__device__ __forceinline__ double keep_if(double x, bool keep) {
  return __longlong_as_double(__double_as_longlong(x) & (keep ? -1ll : 0ll));
}

template <typename TAs, typename TBs, typename TCs, typename T, bool AC, bool BC, bool BSUM, int BM, int BN, int WM,
          int WN>
__global__ __launch_bounds__(256) void zgemm_kernel(const GemmDesc d) {
  constexpr int NT = 256;
  constexpr int BK = sizeof(T) == 8 ? 8 : 16;  // 128 bytes of a row of either type
  static_assert(WM * WN == 4, "4 waves");
  constexpr int TM = BM / WM / 16;
  constexpr int TN = BN / WN / 16;
  static_assert(TM >= 1 && TN >= 1, "tile");
  constexpr int SA = AC ? (BM + 16) : (BK + 1);  // AC: [k][m], else [m][k]
  constexpr int SB = BC ? (BK + 1) : (BN + 16);  // BC: [n][k], else [k][n]
  constexpr int A_ELEMS = AC ? BK * SA : BM * SA;
  constexpr int B_ELEMS = BC ? BN * SB : BK * SB;
  constexpr int EA = BM * BK / NT;
  constexpr int EB = BK * BN / NT;
  static_assert(EA * NT == BM * BK && EB * NT == BK * BN, "load split");
  typedef typename Mfma<T>::acc_t acc_t;

  __shared__ T sAr[2][A_ELEMS], sAi[2][A_ELEMS], sBr[2][B_ELEMS], sBi[2][B_ELEMS];

  const int tid = threadIdx.x;
  const int f = blockIdx.z % d.batch;
  const int split = blockIdx.z / d.batch;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int M = d.M, N = d.N;
  int kbeg = 0, kend = d.K;
  if (d.nsplit > 1) {
    kbeg = split * d.kchunk;
    kend = min(d.K, kbeg + d.kchunk);
  }
  const cx<TAs>* Ab = reinterpret_cast<const cx<TAs>*>(d.A) + (int64_t)f * d.strideA;
  const cx<TBs>* Bb = reinterpret_cast<const cx<TBs>*>(d.B) + (int64_t)f * d.strideB;
  int64_t lda = d.lda, ldb = d.ldb;

  // Every read is issued without a branch at a clamped address, so that all
  // of a step's reads are in flight together: a clamped row or column feeds
  // only results that are not stored, and what lies past the K range is
  // cleared on its way to LDS.
  T ra_r[EA], ra_i[EA], rb_r[EB], rb_i[EB];
  auto a_m = [&](int i) { return AC ? ((tid + i * NT) % BM) : ((tid + i * NT) / BK); };
  auto a_k = [&](int i) { return AC ? ((tid + i * NT) / BM) : ((tid + i * NT) % BK); };
  auto b_n = [&](int i) { return BC ? ((tid + i * NT) / BK) : ((tid + i * NT) % BN); };
  auto b_k = [&](int i) { return BC ? ((tid + i * NT) % BK) : ((tid + i * NT) / BN); };

  auto gload = [&](int kt) {
#pragma unroll
    for (int i = 0; i < EA; ++i) {
      const int gm = min(m0 + a_m(i), M - 1), gk = min(kt + a_k(i), kend - 1);
      ld_cx<TAs, T>(Ab, AC ? ((int64_t)gk * lda + gm) : ((int64_t)gm * lda + gk), ra_r[i], ra_i[i]);
    }
    int64_t bidx[EB];
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int gn = min(n0 + b_n(i), N - 1), gk = min(kt + b_k(i), kend - 1);
      bidx[i] = BC ? ((int64_t)gn * ldb + gk) : ((int64_t)gk * ldb + gn);
      ld_cx<TBs, T>(Bb, bidx[i], rb_r[i], rb_i[i]);
    }
    if (BSUM) {
      for (int j = 1; j < d.b_nsum; ++j) {
        T r2[EB], i2[EB];
#pragma unroll
        for (int i = 0; i < EB; ++i) ld_cx<TBs, T>(Bb + j * d.b_sum_stride, bidx[i], r2[i], i2[i]);
#pragma unroll
        for (int i = 0; i < EB; ++i) {
          rb_r[i] += r2[i];
          rb_i[i] += i2[i];
        }
      }
    }
  };
  auto sstore = [&](int buf, int kt) {
#pragma unroll
    for (int i = 0; i < EA; ++i) {
      const int m = a_m(i), k = a_k(i);
      const int s = AC ? (k * SA + m) : (m * SA + k);
      const bool in = kt + k < kend;
      sAr[buf][s] = keep_if(ra_r[i], in);
      sAi[buf][s] = keep_if(AC ? -ra_i[i] : ra_i[i], in);
    }
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int n = b_n(i), k = b_k(i);
      const int s = BC ? (n * SB + k) : (k * SB + n);
      const bool in = kt + k < kend;
      sBr[buf][s] = keep_if(rb_r[i], in);
      sBi[buf][s] = keep_if(BC ? -rb_i[i] : rb_i[i], in);
    }
  };

  const int lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave % WM) * (BM / WM), wn0 = (wave / WM) * (BN / WN);
  const int r16 = lane & 15, q4 = lane >> 4;

  acc_t acc_r[TM][TN], acc_i[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      acc_r[a][b] = acc_t{0, 0, 0, 0};
      acc_i[a][b] = acc_t{0, 0, 0, 0};
    }

  for (int seg = 0;; ++seg) {
    if (kbeg < kend) {
      gload(kbeg);
      sstore(0, kbeg);
    }
    int buf = 0;
    for (int kt = kbeg; kt < kend; kt += BK, buf ^= 1) {
      __syncthreads();
      const bool more = kt + BK < kend;
      if (more) gload(kt + BK);
#pragma unroll
      for (int kk = 0; kk < BK; kk += 4) {
        const int kq = kk + q4;
        T ar[TM], ai[TM], nai[TM], br[TN], bi[TN];
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          const int m = wm0 + a * 16 + r16;
          const int s = AC ? (kq * SA + m) : (m * SA + kq);
          ar[a] = sAr[buf][s];
          ai[a] = sAi[buf][s];
          nai[a] = -ai[a];
        }
#pragma unroll
        for (int b = 0; b < TN; ++b) {
          const int n = wn0 + b * 16 + r16;
          const int s = BC ? (n * SB + kq) : (kq * SB + n);
          br[b] = sBr[buf][s];
          bi[b] = sBi[buf][s];
        }
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) acc_r[a][b] = Mfma<T>::run(ar[a], br[b], acc_r[a][b]);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) acc_i[a][b] = Mfma<T>::run(ar[a], bi[b], acc_i[a][b]);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) acc_r[a][b] = Mfma<T>::run(nai[a], bi[b], acc_r[a][b]);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) acc_i[a][b] = Mfma<T>::run(ai[a], br[b], acc_i[a][b]);
      }
      if (more) sstore(buf ^ 1, kt + BK);
    }
    if (seg >= d.nmore) break;
    const GemmDesc::More& e = d.more[seg];
    Ab = reinterpret_cast<const cx<TAs>*>(e.A) + (int64_t)f * e.strideA;
    Bb = reinterpret_cast<const cx<TBs>*>(e.B) + (int64_t)f * e.strideB;
    lda = e.lda;
    ldb = e.ldb;
    kbeg = 0;
    kend = e.K;
    __syncthreads();  // every wave is done with the LDS of the product before
  }

  // epilogue
  cx<TCs>* Cb = reinterpret_cast<cx<TCs>*>(d.C) + (int64_t)f * d.strideC;
  if (d.nsplit > 1) Cb += (int64_t)split * d.c_split_stride;
  const T alpha = static_cast<T>(d.alpha);
  const T beta = static_cast<T>(d.beta);
  const bool acc = d.nsplit <= 1 && d.beta != 0.0;
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    // the old values of a row of tiles are read together, ahead of its stores
    cx<TCs> o[TN][4];
    if (acc) {
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gm = min(m0 + wm0 + a * 16 + Mfma<T>::row(q4, r), M - 1);
          const int gn = min(n0 + wn0 + b * 16 + r16, N - 1);
          o[b][r] = Cb[(int64_t)gm * d.ldc + gn];
        }
    }
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gm = m0 + wm0 + a * 16 + Mfma<T>::row(q4, r);
        const int gn = n0 + wn0 + b * 16 + r16;
        T vr = alpha * acc_r[a][b][r];
        T vi = alpha * acc_i[a][b][r];
        if (acc) {
          vr += beta * static_cast<T>(o[b][r].re);
          vi += beta * static_cast<T>(o[b][r].im);
        }
        if (gm < M && gn < N) {
          cx<TCs> out;
          out.re = static_cast<TCs>(vr);
          out.im = static_cast<TCs>(vi);
          Cb[(int64_t)gm * d.ldc + gn] = out;
        }
      }
  }
}

template <typename TAs, typename TBs, typename TCs, typename T, bool AC, bool BC, bool BSUM, int BM, int BN, int WM,
          int WN>
static hipError_t launch_tile(const GemmDesc& d, hipStream_t s) {
  dim3 grid((d.M + BM - 1) / BM, (d.N + BN - 1) / BN, d.batch * (d.nsplit > 1 ? d.nsplit : 1));
  hipLaunchKernelGGL((zgemm_kernel<TAs, TBs, TCs, T, AC, BC, BSUM, BM, BN, WM, WN>), grid, dim3(256), 0, s, d);
  return hipGetLastError();
}

template <typename TAs, typename TBs, typename TCs, typename T, bool AC, bool BC, bool BSUM>
static hipError_t launch(const GemmDesc& d, hipStream_t s) {
  // 32 x 32 tiles waste the least on ragged edges and keep the most waves per
  // SIMD, which is what hides the reads of these short products: 2000 x 90 x
  // 2000 FP32 over 9 slices 322 us against 464 with 64 x 64 tiles, 256 x 50 x
  // 256 FP64 over 129 slices 103 against 129, 50 x 50 x 256 39 against 51.
  // With 8 or more workgroups for every CU and at most one eighth of the
  // columns padding, the wider tile's fewer operand reads are worth more:
  // 64 x 64 in FP32 (4096 x 4096 x 100, 33 slices: 4636 us against 4971),
  // 64 x 32 in FP64 (256 x 256 x 45, 129 slices: 72 us against 80, and 83
  // with 64 x 64).  128 x 64 and 64 x 16 were no faster anywhere.
  constexpr int WN = sizeof(T) == 8 ? 32 : 64;
  const int64_t mt = (d.M + 63) / 64, nt = (d.N + WN - 1) / WN;
  const int64_t wgs = mt * nt * d.batch * (d.nsplit > 1 ? d.nsplit : 1);
  if (wgs >= 2048 && (nt * WN - d.N) * 8 <= nt * WN)
    return launch_tile<TAs, TBs, TCs, T, AC, BC, BSUM, 64, WN, 2, 2>(d, s);
  return launch_tile<TAs, TBs, TCs, T, AC, BC, BSUM, 32, 32, 2, 2>(d, s);
}

template <typename TAs, typename TBs, typename TCs, typename T>
static hipError_t launch_conj(const GemmDesc& d, hipStream_t s) {
  if (d.a_conj && d.b_conj) return hipErrorInvalidValue;
  if (d.b_nsum > 1) {
    // sums of partial products are the FP64 coefficients of Gram-Schmidt, applied as they are
    if constexpr (sizeof(TBs) == 8 && sizeof(TAs) == sizeof(TCs)) {
      if (!d.a_conj && !d.b_conj) return launch<TAs, TBs, TCs, T, false, false, true>(d, s);
    }
    return hipErrorInvalidValue;
  }
  if (d.b_conj) return launch<TAs, TBs, TCs, T, false, true, false>(d, s);
  return d.a_conj ? launch<TAs, TBs, TCs, T, true, false, false>(d, s)
                  : launch<TAs, TBs, TCs, T, false, false, false>(d, s);
}

hipError_t zgemm(const GemmDesc& d, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0 || d.batch <= 0) return hipSuccess;
  if (d.nsplit > 1 && d.beta != 0.0) return hipErrorInvalidValue;
  if (d.nmore < 0 || d.nmore > 2 || (d.nmore && (d.nsplit > 1 || d.b_nsum > 1))) return hipErrorInvalidValue;
  const DType a = d.ta, b = d.tb, c = d.tc, t = d.compute;
  if (a == DT_F32 && b == DT_F32 && c == DT_F32 && t == DT_F32) return launch_conj<float, float, float, float>(d, s);
  if (a == DT_F64 && b == DT_F64 && c == DT_F64 && t == DT_F64) return launch_conj<double, double, double, double>(d, s);
  if (a == DT_F32 && b == DT_F32 && c == DT_F64 && t == DT_F64) return launch_conj<float, float, double, double>(d, s);
  if (a == DT_F32 && b == DT_F64 && c == DT_F32 && t == DT_F64) return launch_conj<float, double, float, double>(d, s);
  if (a == DT_F32 && b == DT_F64 && c == DT_F32 && t == DT_F32) return launch_conj<float, double, float, float>(d, s);
  if (a == DT_F64 && b == DT_F32 && c == DT_F32 && t == DT_F64) return launch_conj<double, float, float, double>(d, s);
  return hipErrorInvalidValue;
}

}  // namespace tsvd
