// Matrix-core building blocks shared by the batched inversion and the
// refinement products (gfx950): the 16x16x4 products and the tile product
// C = A B of complex matrices.
#pragma once

#include "fk_internal.h"

#include <type_traits>

namespace fk {

// 16x16x4 matrix-core products.  Operands: lane l holds A[l%16][l/16] and
// B[l/16][l%16].  The accumulator layout differs between the two precisions
// (measured on gfx950): register v of lane l holds D[row][l%16] with
//   f64: row = (l/16) + 4 v      f32: row = 4 (l/16) + v.
template <typename T> struct Mfma;
template <> struct Mfma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  __device__ static inline v4 run(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static inline int drow(int lk, int v) { return lk + 4 * v; }
};
template <> struct Mfma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  __device__ static inline v4 run(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static inline int drow(int lk, int v) { return 4 * lk + v; }
};

// Element at a byte offset from a uniform base: one 32-bit address register
// and a scalar base per access (a matrix is at most kMaxN^2 elements of 16
// bytes, below 2^32).
template <typename E> __device__ __forceinline__ E* at_byte(E* base, unsigned off) {
  return reinterpret_cast<E*>(reinterpret_cast<char*>(const_cast<typename std::remove_const<E>::type*>(base)) + (size_t)off);
}

// Product of one tile of (32 WR) x 64 by 2 WR waves as WR x 2 blocks of
// 32 x 32.  K runs in chunks of kKC, double-buffered through LDS with the next
// chunk's global loads in flight during the current chunk's products; within a
// chunk the next k-step's operands are read from LDS before the current
// k-step's products.  Each complex product takes three real ones (Gauss):
// P1 = Re a Re b, P2 = Im a Im b and P3 = (Re a + Im a)(Re b + Im b)
// accumulate separately, and value() forms Re = P1 - P2, Im = P3 - P1 - P2: a
// quarter fewer products than the four-product form, with a normwise (not
// componentwise) error bound of the same order.
//
// FP64 matrix instructions and vector instructions share the SIMD's issue: a
// vector instruction beside them costs its 4 to 6 cycles (measured: four FP64
// adds per twelve products 3%, LDS addresses formed in the loop another 11%,
// with two waves per SIMD as with four).  So the loop has hardly any: rows and
// columns are addressed by 32-bit offsets that stay fixed while the scalar
// base advances, tile edges are handled by clamped addresses instead of masks,
// and only a ragged last chunk is masked: 24 vector instructions per 48
// products instead of 72.  Trailing and pre-panel updates of 225 matrices of
// N_c = 1800: 4.51 -> 4.25 ms per launch in FP64, 2.55 -> 2.29 in complex64.
template <typename T, int WR> struct TileProduct {
  typedef typename Mfma<T>::v4 v4;
  static constexpr int TR = 32 * WR, NT = 128 * WR;
  static constexpr int AP = kKC + 1, BP = kTile + 1;
  static constexpr int kLA = TR * kKC / NT;      // chunk loads per thread
  static constexpr int kLB = kKC * kTile / NT;
  static constexpr int AST = NT / kKC, BST = NT / kTile;
  static_assert(NT % kKC == 0 && NT % kTile == 0, "load map");
  typedef T c2 __attribute__((ext_vector_type(2)));   // an element in registers
  struct Lds {
    c2 a[2][TR * AP];
    c2 b[2][kKC * BP];
  };

  v4 p1[2][2], p2[2][2], p3[2][2];
  c2 pa[kLA], pb[kLB];
  unsigned aoff[kLA], boff[kLB];
  const c2* ab;                  // A at (0, k) and B at (k, 0) of the next load
  const c2* bb;
  int K, r0, c0, rows, cols, ldc, ldb;
  int wr, wc, wave, li, lk, ak, ai0, bc, bk0;
  // Tiles with at most 16 valid rows (1) or columns (2) take a strip layout:
  // each wave multiplies one 16 x 16 block along the strip, a quarter of an
  // interior tile's products, instead of a 32 x 32 block that lies mostly
  // outside the matrix (the same for the whole workgroup).
  int edge;

  // A: rows r0 .. of `rows`, K columns from a on (leading dimension lda); B: K
  // rows from b on, columns c0 .. of `cols`.  C has A's leading dimension.
  __device__ __forceinline__ void begin(Lds& lds, const cplx<T>* a, int lda, int r0_,
                                        int rows_, const cplx<T>* b, int ldb_, int c0_,
                                        int cols_, int K_) {
    const int tid = threadIdx.x, lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    wr = wave >> 1;
    wc = wave & 1;
    li = lane & 15;
    lk = lane >> 4;
    // this thread's chunk loads: A rows ai0 + t AST at column ak of the chunk,
    // B rows bk0 + t BST at column bc of the tile
    ak = tid % kKC;
    ai0 = tid / kKC;
    bc = tid % kTile;
    bk0 = tid / kTile;
    K = K_;
    r0 = r0_;
    c0 = c0_;
    rows = rows_;
    cols = cols_;
    ldc = lda;
    ldb = ldb_;
    ab = reinterpret_cast<const c2*>(a);
    bb = reinterpret_cast<const c2*>(b);
    edge = (rows - r0 <= 16) ? 1 : ((cols - c0 <= 16) ? 2 : 0);
    constexpr unsigned E = sizeof(cplx<T>);
#pragma unroll
    for (int t = 0; t < kLA; ++t)
      aoff[t] = ((unsigned)min(r0 + ai0 + AST * t, rows - 1) * lda + ak) * E;
#pragma unroll
    for (int t = 0; t < kLB; ++t)
      boff[t] = ((unsigned)(bk0 + BST * t) * ldb + min(c0 + bc, cols - 1)) * E;
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj)
#pragma unroll
        for (int v = 0; v < 4; ++v) p1[ii][jj][v] = p2[ii][jj][v] = p3[ii][jj][v] = T(0);
    if (K >= kKC) load<false>(0);
    else load<true>(K);
    store(lds, 0);
    if (K < kKC) zero_tail(lds, 0, K);
    __syncthreads();
  }

  // the next chunk of A's columns and B's rows into registers; RAG: only rem
  // of them are left (clamped addresses; zero_tail() follows)
  template <bool RAG> __device__ __forceinline__ void load(int rem) {
    if (!RAG) {
#pragma unroll
      for (int t = 0; t < kLA; ++t) pa[t] = *at_byte(ab, aoff[t]);
#pragma unroll
      for (int t = 0; t < kLB; ++t) pb[t] = *at_byte(bb, boff[t]);
    } else {
      constexpr unsigned E = sizeof(cplx<T>);
#pragma unroll
      for (int t = 0; t < kLA; ++t)
        pa[t] = *at_byte(ab, aoff[t] - (unsigned)max(ak - rem + 1, 0) * E);
#pragma unroll
      for (int t = 0; t < kLB; ++t)
        pb[t] = *at_byte(bb, boff[t] - (unsigned)max(bk0 + BST * t - rem + 1, 0) * ldb * E);
    }
    ab += kKC;
    bb += (size_t)kKC * ldb;
  }
  __device__ __forceinline__ void store(Lds& lds, int buf) {
#pragma unroll
    for (int t = 0; t < kLA; ++t) lds.a[buf][(ai0 + AST * t) * AP + ak] = pa[t];
#pragma unroll
    for (int t = 0; t < kLB; ++t) lds.b[buf][(bk0 + BST * t) * BP + bc] = pb[t];
  }
  // the loaded chunk holds rem columns of A: zeros in the others' places
  __device__ __forceinline__ void zero_tail(Lds& lds, int buf, int rem) {
    if (ak >= rem) {
#pragma unroll
      for (int t = 0; t < kLA; ++t) lds.a[buf][(ai0 + AST * t) * AP + ak] = c2{T(0), T(0)};
    }
  }
  __device__ __forceinline__ void multiply(const Lds& lds, int buf) {
    const c2* as = lds.a[buf] + (32 * wr + li) * AP + lk;
    const c2* bs = lds.b[buf] + lk * BP + 32 * wc + li;
    c2 a[2][2], b[2][2];
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) a[0][ii] = as[16 * ii * AP];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) b[0][jj] = bs[16 * jj];
#pragma unroll
    for (int s = 0; s < kKC / 4; ++s) {
      const int cur = s & 1;
      if (s + 1 < kKC / 4) {
        const int k = 4 * (s + 1);
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) a[cur ^ 1][ii] = as[16 * ii * AP + k];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) b[cur ^ 1][jj] = bs[k * BP + 16 * jj];
      }
      T as_[2], bs_[2];
#pragma unroll
      for (int ii = 0; ii < 2; ++ii) as_[ii] = a[cur][ii].x + a[cur][ii].y;
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) bs_[jj] = b[cur][jj].x + b[cur][jj].y;
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          p1[ii][jj] = Mfma<T>::run(a[cur][ii].x, b[cur][jj].x, p1[ii][jj]);
          p2[ii][jj] = Mfma<T>::run(a[cur][ii].y, b[cur][jj].y, p2[ii][jj]);
          p3[ii][jj] = Mfma<T>::run(as_[ii], bs_[jj], p3[ii][jj]);
        }
    }
  }
  // strip layout: one 16 x 16 block per wave, accumulated in p*[0][0]
  __device__ __forceinline__ int strip_row() const { return edge == 2 ? 16 * wave : 0; }
  __device__ __forceinline__ int strip_col() const { return edge == 1 ? 16 * wave : 0; }
  // waves whose strip block lies inside the tile (the first four of a 128-row
  // tile's eight in a row strip)
  __device__ __forceinline__ bool strip_active() const {
    return edge == 1 ? 16 * wave < kTile : 16 * wave < TR;
  }
  __device__ __forceinline__ void multiply_strip(const Lds& lds, int buf) {
    if (!strip_active()) return;
    const c2* as = lds.a[buf] + (strip_row() + li) * AP + lk;
    const c2* bs = lds.b[buf] + lk * BP + strip_col() + li;
#pragma unroll
    for (int k = 0; k < kKC; k += 4) {
      const c2 a = as[k], b = bs[k * BP];
      p1[0][0] = Mfma<T>::run(a.x, b.x, p1[0][0]);
      p2[0][0] = Mfma<T>::run(a.y, b.y, p2[0][0]);
      p3[0][0] = Mfma<T>::run(a.x + a.y, b.x + b.y, p3[0][0]);
    }
  }

  template <bool STRIP> __device__ __forceinline__ void run_as(Lds& lds) {
    auto mul = [&](int buf) {
      if (STRIP) multiply_strip(lds, buf);
      else multiply(lds, buf);
    };
    const int full = K / kKC, rem = K % kKC, nch = full + (rem ? 1 : 0);
    int buf = 0;
#pragma unroll 1
    for (int kc = 1; kc < nch; ++kc) {
      if (kc < full) load<false>(0);
      else load<true>(rem);
      mul(buf);
      buf ^= 1;
      store(lds, buf);
      if (kc >= full) zero_tail(lds, buf, rem);
      __syncthreads();
    }
    mul(buf);
  }
  // the whole product, from the first chunk that begin() left in LDS
  __device__ __forceinline__ void run(Lds& lds) {
    if (edge) run_as<true>(lds);
    else run_as<false>(lds);
  }

  // row of the matrix that this lane's output (ii, ., v) lies in
  __device__ __forceinline__ int row(int ii, int v) const {
    return r0 + (edge ? strip_row() : 32 * wr) + 16 * ii + Mfma<T>::drow(lk, v);
  }
  // f(ii, jj, v, inside, byte offset in C) for this lane's outputs of block row
  // ii (0 or 1; a strip has only 0)
  template <typename F> __device__ __forceinline__ void for_outputs(int ii, F f) const {
    constexpr unsigned E = sizeof(cplx<T>);
    if (!edge) {
      const int col = c0 + 32 * wc + li;
      const unsigned off = ((unsigned)row(0, 0) * ldc + col) * E;
      const unsigned step = (unsigned)(Mfma<T>::drow(0, 1)) * ldc * E;   // v -> v + 1
      const bool whole = r0 + TR <= rows && c0 + kTile <= cols;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
          f(ii, jj, v, whole || (row(ii, v) < rows && col + 16 * jj < cols),
            off + 16u * ii * ldc * E + v * step + 16u * jj * E);
    } else if (ii == 0 && strip_active()) {
      const int col = c0 + strip_col() + li;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        f(0, 0, v, row(0, v) < rows && col < cols,
          ((unsigned)row(0, v) * ldc + col) * E);
    }
  }
  __device__ __forceinline__ c2 value(int ii, int jj, int v) const {
    const T q1 = p1[ii][jj][v], q2 = p2[ii][jj][v];
    return c2{q1 - q2, (p3[ii][jj][v] - q1) - q2};
  }
};

}  // namespace fk
