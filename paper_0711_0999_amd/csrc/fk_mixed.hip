// FP64 iterative refinement of complex64 inverses (gfx950).
//
// With X ~ A^-1 from the complex64 Gauss-Jordan inversion of A = G0^-1 - W
// Sigma W, one refinement step is Newton's step for the inverse
//     R = I - A X  (FP64),     X <- X + X R  (FP64),
// which squares the relative error.  A X = T X - Sigma_t X with T = G0^-1 the
// bidiagonal-plus-corner matrix, so the residual costs one dense complex GEMM
// with the shared left operand Sigma_t plus an O(N^2) sparse product, and the
// correction one more dense GEMM.
#include "fk_internal.h"
#include "fk_kernels.h"
#include "fk_tile.h"

namespace fk {

// out[m][a][b] = X[m][piv_m[a]][rowcol_m[b]] in FP64 (undo the logical pivoting)
template <typename TI>
__global__ void k_unpermute(const cplx<TI>* __restrict__ x, size_t xstride,
                            int ld, const int* __restrict__ piv,
                            const int* __restrict__ rowcol, int n,
                            c64* __restrict__ out) {
  const int m = blockIdx.z, a = blockIdx.y;
  const int r = piv[(size_t)m * n + a];
  const cplx<TI>* src = x + (size_t)m * xstride + (size_t)r * ld;
  c64* dst = out + (size_t)m * n * n + (size_t)a * n;
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < n;
       b += gridDim.x * blockDim.x) {
    const cplx<TI> v = src[rowcol[(size_t)m * n + b]];
    dst[b] = c64{(double)v.re, (double)v.im};
  }
}

// C[m] = beta Cin[m] + A[m] B[m] for n x n complex128 matrices (leading
// dimension n).  sA = 0 shares A across the batch.  One 64 x 64 tile product
// of the trailing update's form (fk_tile.h) per workgroup.
__global__ __launch_bounds__(256, 2) void k_bgemm(
    c64* __restrict__ C, const c64* __restrict__ Cin, double beta,
    const c64* __restrict__ A, size_t sA, const c64* __restrict__ B, int n,
    int nmat) {
  typedef TileProduct<double, 2> P;
  __shared__ P::Lds lds;
  const int nt = (n + kTile - 1) / kTile;
  const int per_m = nt * nt;
  const int nitems = per_m * nmat;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int chunk = (nitems + 7) >> 3;
  const int it = xcd * chunk + slot;
  if (slot >= chunk || it >= nitems) return;
  const size_t ss = (size_t)n * n;
  const int m = it / per_m, t = it - m * per_m;
  const int tc = t / nt, tr = t - tc * nt;
  P tp;
  tp.begin(lds, A + sA * m, n, tr * kTile, n, B + ss * m, n, tc * kTile, n, n);
  tp.run(lds);
  P::c2* cm = reinterpret_cast<P::c2*>(C + ss * m);
  const P::c2* im = reinterpret_cast<const P::c2*>(Cin + ss * m);
#pragma unroll
  for (int ii = 0; ii < 2; ++ii)
    tp.for_outputs(ii, [&](int, int jj, int v, bool in, unsigned off) {
      if (!in) return;
      P::c2 c = tp.value(ii, jj, v);
      if (beta != 0.0) c += beta * *at_byte(im, off);
      *at_byte(cm, off) = c;
    });
}

// R = I - T X + P in place of P (P = Sigma_t X), T = i I + sub-diagonal tsub
// + corner tcor at (0, n-1); running max |R| into key (nullable).
__global__ void k_residual(c64* __restrict__ P, const c64* __restrict__ X,
                           const c64* __restrict__ tsub,
                           const c64* __restrict__ tcor, int n, int nmat,
                           unsigned long long* __restrict__ key) {
  const size_t ss = (size_t)n * n, total = ss * nmat;
  double mx = 0.0;
  bool bad = false;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x) {
    const int m = (int)(e / ss);
    const size_t f = e - (size_t)m * ss;
    const int i = (int)(f / n), j = (int)(f - (f / n) * n);
    const c64* xm = X + ss * m;
    const c64 xv = xm[f];
    c64 tx{-xv.im, xv.re};  // i * X[i][j]
    const c64 t = (i >= 1) ? tsub[(size_t)m * n + i] : tcor[m];
    const c64 xo = xm[(size_t)((i >= 1) ? i - 1 : n - 1) * n + j];
    tx.re += t.re * xo.re - t.im * xo.im;
    tx.im += t.re * xo.im + t.im * xo.re;
    c64 r = P[e];
    r.re += (i == j ? 1.0 : 0.0) - tx.re;
    r.im -= tx.im;
    P[e] = r;
    const double a = sqrt(r.re * r.re + r.im * r.im);
    if (!(a <= 1.79769313486231570815e308)) bad = true;
    else if (a > mx) mx = a;
  }
  unsigned long long k = bad ? 0x7ff8000000000000ULL
                             : (unsigned long long)__double_as_longlong(mx);
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long o = __shfl_xor(k, off);
    k = o > k ? o : k;
  }
  if (key && (threadIdx.x & 63) == 0) atomicMax(key, k);
}

template <typename TI>
hipError_t launch_unpermute(const cplx<TI>* x, size_t xstride, int ld,
                            const int* piv, const int* rowcol, int n, int nmat,
                            c64* out, hipStream_t st) {
  hipLaunchKernelGGL(k_unpermute<TI>, dim3((n + 255) / 256, n, nmat), dim3(256),
                     0, st, x, xstride, ld, piv, rowcol, n, out);
  return hipGetLastError();
}

hipError_t launch_bgemm(c64* C, const c64* Cin, double beta, const c64* A,
                        size_t sA, const c64* B, int n, int nmat,
                        hipStream_t st) {
  const int nt = (n + kTile - 1) / kTile;
  const long long items = (long long)nt * nt * nmat;
  const int grid = (int)(8 * ((items + 7) / 8));
  hipLaunchKernelGGL(k_bgemm, dim3(grid), dim3(256), 0, st, C, Cin, beta, A,
                     sA, B, n, nmat);
  return hipGetLastError();
}

hipError_t launch_residual(c64* P, const c64* X, const c64* tsub,
                           const c64* tcor, int n, int nmat,
                           unsigned long long* key, hipStream_t st) {
  size_t g = ((size_t)n * n * nmat + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_residual, dim3((int)g), dim3(256), 0, st, P, X, tsub,
                     tcor, n, nmat, key);
  return hipGetLastError();
}

template hipError_t launch_unpermute<float>(const c32*, size_t, int, const int*,
                                            const int*, int, int, c64*,
                                            hipStream_t);
template hipError_t launch_unpermute<double>(const c64*, size_t, int,
                                             const int*, const int*, int, int,
                                             c64*, hipStream_t);

}  // namespace fk
