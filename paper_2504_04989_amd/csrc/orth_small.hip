// Orthonormalisation of one small block per slice in one workgroup: the whole
// sequence of block Gram-Schmidt against the earlier columns and (shifted)
// CholeskyQR passes with the n x b block W in LDS, in FP64.
//
// For these sizes the sequence is bound by latency: as separate products and
// factorisations it is 15 to 19 launches of 4 to 14 us each, of which the
// arithmetic is a fraction of a microsecond.  Here a pass costs its barriers,
// the b steps of the elimination and a few dozen dependent MFMAs: 64
// x 10 FP64 blocks (five passes, 9 slices) 42 us each against about 170, 150 x 9
// FP32 blocks 37 against about 110.
//
// Products (v_mfma_f64_16x16x4, 16 x 16 tiles): coefficients Q^H W and Grams
// W^H W have the rows cut into one quarter per wave and the four partial tiles
// added in a fixed order; updates W - Q C and W R^{-1} give each wave its own
// tiles of 16 rows, which it alone reads and then writes.  W has 16 NB columns
// and a multiple of 16 rows, zero past b and n; Q is read in place.
#include "chol_elim.h"
#include "common.h"
#include "kernels.h"

namespace tsvd {
namespace {

struct OrthArgs {
  const void* W;  // n x b, row stride ldw, slice stride strideW (complex elements)
  int64_t ldw, strideW;
  const void* Q;  // the ib earlier columns, n x ib
  int64_t ldq, strideQ;
  void* D;        // result, n x b (may be W)
  int64_t ldd, strideD;
  int n, b, ib;
  int nshift, nplain;  // shifted passes before the second projection, unshifted ones after it
  bool third;          // projected once more after the first unshifted pass
  double shift;        // shift coefficient of the shifted passes
  int* info;
};

template <int NB>
struct OrthLds {
  static constexpr int BP = 16 * NB, SW = BP + 1;  // columns and row stride of W, C and R^{-1}
  static size_t bytes(int n, int ib) {
    const size_t rows = (n + 15) / 16 * 16, c = (ib + 15) / 16 * 16;
    return ((rows + (c > BP ? c : BP)) * SW + 2 * 4 * 256) * sizeof(cx<double>);
  }
};

template <typename T>
__device__ __forceinline__ cx<double> ldq(const cx<T>* p) {
  const cx<T> v = *p;
  return cx<double>{(double)v.re, (double)v.im};
}

template <typename T, int NB>
__global__ __launch_bounds__(256, 1) void orth_small_kernel(const OrthArgs a) {
  constexpr int BP = OrthLds<NB>::BP, SW = OrthLds<NB>::SW;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ ElimLds<NB> elim;
  const int f = blockIdx.x;
  const int n = a.n, b = a.b, ib = a.ib;
  const int rows = (n + 15) / 16 * 16, cr = max(BP, (ib + 15) / 16 * 16);
  cx<double>* W = reinterpret_cast<cx<double>*>(smem);
  cx<double>* C = W + rows * SW;   // coefficients, the Gram or R^{-1}
  cx<double>* P = C + cr * SW;     // partial tiles: [2][wave][16 x 16]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, q4 = lane >> 4;
  const cx<T>* Wg = static_cast<const cx<T>*>(a.W) + (int64_t)f * a.strideW;
  const cx<T>* Q = static_cast<const cx<T>*>(a.Q) + (int64_t)f * a.strideQ;

  // W from memory, eight elements of a thread in flight
  for (int e0 = 0; e0 < rows * BP; e0 += 8 * 256) {
    cx<double> v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + u * 256 + tid, r = e / BP, c = e % BP;
      v[u] = ldq(Wg + (int64_t)min(r, n - 1) * a.ldw + min(c, b - 1));
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + u * 256 + tid, r = e / BP, c = e % BP;
      if (r < rows) W[r * SW + c] = r < n && c < b ? v[u] : cx<double>{0.0, 0.0};
    }
  }
  __syncthreads();

  // one step of a complex product: acc += x y, or conj(x) y
  auto mac = [&](f64x4& re, f64x4& im, cx<double> x, cx<double> y, bool conj) {
    const double xi = conj ? -x.im : x.im;
    re = Mfma<double>::run(x.re, y.re, re);
    im = Mfma<double>::run(x.re, y.im, im);
    re = Mfma<double>::run(-xi, y.im, re);
    im = Mfma<double>::run(xi, y.re, im);
  };
  // the sum of the waves' partial tiles (parity par), entry tid
  auto put_part = [&](int par, f64x4 re, f64x4 im) {
    cx<double>* p = P + (par * 4 + wave) * 256;
#pragma unroll
    for (int r = 0; r < 4; ++r) p[Mfma<double>::row(q4, r) * 16 + r16] = cx<double>{re[r], im[r]};
  };
  auto sum_part = [&](int par) {
    const cx<double>* p = P + par * 4 * 256 + tid;
    const cx<double> s0 = p[0], s1 = p[256], s2 = p[512], s3 = p[768];
    return cx<double>{(s0.re + s1.re) + (s2.re + s3.re), (s0.im + s1.im) + (s2.im + s3.im)};
  };
  const int kq = rows / 4;  // rows of a wave's quarter

  // W -= Q (Q^H W)
  auto project = [&]() {
    int par = 0;
    for (int m0 = 0; m0 < ib; m0 += 16) {
      const cx<T>* Qc = Q + min(m0 + r16, ib - 1);
      f64x4 re[NB], im[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t) re[t] = im[t] = f64x4{0.0, 0.0, 0.0, 0.0};
      for (int k0 = wave * kq; k0 < (wave + 1) * kq; k0 += 16) {
        cx<double> x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = ldq(Qc + (int64_t)min(k0 + 4 * u + q4, n - 1) * a.ldq);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (k0 + 4 * u >= (wave + 1) * kq) continue;
#pragma unroll
          for (int t = 0; t < NB; ++t) mac(re[t], im[t], x[u], W[(k0 + 4 * u + q4) * SW + 16 * t + r16], true);
        }
      }
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        put_part(par, re[t], im[t]);
        lds_barrier();
        const int row = m0 + tid / 16;
        const cx<double> s = sum_part(par);
        C[row * SW + 16 * t + tid % 16] = row < ib ? s : cx<double>{0.0, 0.0};
        par ^= 1;
      }
    }
    lds_barrier();
    for (int m0 = 16 * wave; m0 < rows; m0 += 64) {
      const cx<T>* Qr = Q + (int64_t)min(m0 + r16, n - 1) * a.ldq;
      f64x4 re[NB], im[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t) re[t] = im[t] = f64x4{0.0, 0.0, 0.0, 0.0};
      for (int k0 = 0; k0 < ib; k0 += 16) {
        cx<double> x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = ldq(Qr + min(k0 + 4 * u + q4, ib - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int t = 0; t < NB; ++t) mac(re[t], im[t], x[u], C[(k0 + 4 * u + q4) * SW + 16 * t + r16], false);
      }
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + Mfma<double>::row(q4, r);
          if (row < n) {
            cx<double>& w = W[row * SW + 16 * t + r16];
            w.re -= re[t][r];
            w.im -= im[t][r];
          }
        }
    }
    lds_barrier();
  };

  // one CholeskyQR pass: G = W^H W (upper triangle), W <- W R^{-1}
  auto pass = [&](double shift) {
    int par = 0;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = i; j < NB; ++j) {
        f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
        for (int k0 = wave * kq; k0 < (wave + 1) * kq; k0 += 4)
          mac(re, im, W[(k0 + q4) * SW + 16 * i + r16], W[(k0 + q4) * SW + 16 * j + r16], true);
        put_part(par, re, im);
        lds_barrier();
        C[(16 * i + tid / 16) * SW + 16 * j + tid % 16] = sum_part(par);
        par ^= 1;
      }
    lds_barrier();
    const int tx = tid % 16, ty = tid / 16;
    cx<double> A[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int c = 0; c <= i; ++c) {
        const int row = tx + 16 * i, col = ty + 16 * c;
        const cx<double> u = C[col * SW + row];
        A[i][c] = row < b && col <= row ? cx<double>{u.re, row == col ? 0.0 : -u.im} : cx<double>{0.0, 0.0};
      }
    chol_eliminate<NB, 2>(A, b, shift, elim, a.info, [&](int k, int i, cx<double> v) { C[k * SW + i] = v; });
    lds_barrier();
    for (int m0 = 16 * wave; m0 < rows; m0 += 64) {
      f64x4 re[NB], im[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t) re[t] = im[t] = f64x4{0.0, 0.0, 0.0, 0.0};
      for (int k0 = 0; k0 < b; k0 += 4) {
        const cx<double> x = W[(m0 + r16) * SW + k0 + q4];
#pragma unroll
        for (int t = 0; t < NB; ++t) mac(re[t], im[t], x, C[(k0 + q4) * SW + 16 * t + r16], false);
      }
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          W[(m0 + Mfma<double>::row(q4, r)) * SW + 16 * t + r16] = cx<double>{re[t][r], im[t][r]};
    }
    lds_barrier();
  };

  if (ib > 0) project();
  for (int i = 0; i < a.nshift; ++i) pass(a.shift);
  if (ib > 0) project();
  for (int i = 0; i < a.nplain; ++i) {
    if (i > 0 && a.third) project();
    pass(0.0);
  }

  cx<T>* D = static_cast<cx<T>*>(a.D) + (int64_t)f * a.strideD;
  for (int e = tid; e < n * b; e += 256) {
    const int r = e / b, c = e % b;
    const cx<double> v = W[r * SW + c];
    D[(int64_t)r * a.ldd + c] = cx<T>{(T)v.re, (T)v.im};
  }
}

constexpr size_t kOrthLds = 150 * 1024;  // of the 160 KB of a CU, the static part aside

template <typename T, int NB>
hipError_t launch(const OrthArgs& a, int batch, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)orth_small_kernel<T, NB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)kOrthLds);
    (void)hipGetLastError();
    attr = true;
  }
  hipLaunchKernelGGL((orth_small_kernel<T, NB>), dim3(batch), dim3(256), OrthLds<NB>::bytes(a.n, a.ib), s, a);
  return hipGetLastError();
}

}  // namespace

// Wherever W fits in LDS the one workgroup beats the separate launches, by
// more the more slices there are: whole calls of Alg. 2 with 64 x 64 x 1000, b =
// 10 FP64 791 against 1068 us, 256^3, b = 16 FP64 1442 against 1752, 400 x 400 x
// 16, b = 16 FP32 422 against 445.  Past b = 16 the elimination and the one CU's
// FP64 rate weigh more: 100 x 100 x 2, b = 30 FP32 779 against 849, but 180 x
// 180 x 64, b = 32 FP64 1187 against 1165, hence the limit of 160 rows there.
bool orth_small_ok(int64_t n, int64_t b, int64_t ib) {
  if (b > 32 || n > (b <= 16 ? 1024 : 160) || ib > 1024) return false;
  return (b <= 16 ? OrthLds<1>::bytes((int)n, (int)ib) : OrthLds<2>::bytes((int)n, (int)ib)) <= kOrthLds;
}

hipError_t orth_small(DType dt, const void* W, int64_t ldw, int64_t strideW, const void* Q, int64_t ldq,
                      int64_t strideQ, void* D, int64_t ldd, int64_t strideD, int n, int b, int ib, int nshift,
                      int nplain, bool third, double shift, int batch, int* info, hipStream_t s) {
  if (n <= 0 || b <= 0 || batch <= 0) return hipSuccess;
  if (!orth_small_ok(n, b, ib)) return hipErrorInvalidValue;
  const OrthArgs a{W, ldw, strideW, Q, ldq, strideQ, D, ldd, strideD, n, b, ib, nshift, nplain, third, shift, info};
  if (dt == DT_F64) return b <= 16 ? launch<double, 1>(a, batch, s) : launch<double, 2>(a, batch, s);
  return b <= 16 ? launch<float, 1>(a, batch, s) : launch<float, 2>(a, batch, s);
}

}  // namespace tsvd
