// Batched blocked in-place Gauss-Jordan inversion with partial pivoting, for
// gfx950.  This is the hot loop of the lattice step: every (eps, ebar) point
// needs the inverse of the dense complex matrix G0_k^-1 - W Sigma W (the
// "matrix inversion" of the integrand of eq. g_loc, Sec. II).
//
// Outer step S handles the block of kNBO = 128 columns starting at J0 = S*kNBO:
//   panel   (one 512-thread workgroup per matrix) eliminates the block's
//           four 32-column quarters in turn on the n - J0 rows not pivoted in
//           earlier blocks.  For each column the pivot is the largest
//           |re|+|im| among the rows not yet pivoted; groups of kIB columns
//           are eliminated in registers, and the rest of the quarter, the
//           other quarter of the half and then the other half receive the
//           group's (quarter's, half's) transform on the matrix cores.  For
//           few matrices the panel is split into launches per quarter or per
//           group of columns, with its joins between them over all row tiles.
//   gather  copies the pivot rows of the step into a side buffer B (their
//           values before the step outside the block, the block's inverse
//           pivot submatrix inside it); B holds the rows of a group's blocks.
//   fix     the block's columns of the J0 rows pivoted earlier, from that
//           inverse (one small product per row tile).  The block now holds
//           the transformed identity columns M = E[:, P] of all elementary
//           Gauss-Jordan transforms of the step.
//   update  every other column tile: C <- mask_P(C) + M B, a batched complex
//           GEMM on the matrix cores (three real products per complex one),
//           double-buffered K chunks in LDS, two workgroups per CU (four in
//           complex64).  Blocks are applied in groups of kGroup (K up to 512,
//           see block_pos): each block of a group brings the group's earlier
//           blocks' columns up to date and updates the next block's columns;
//           the last one applies all the group's transforms to every other
//           column at once.
// The host runs the update of the next block's columns first; with the
// look-ahead schedule it factors that block on a second stream while the big
// update of the current step runs.
// Rows are never swapped: with r = piv and rinv = rowcol the inverse is
// inv(A)[a][b] = X[r[a]][rinv[b]], which the reduction kernels read directly.
#include "fk_internal.h"
#include "fk_tile.h"

#include <climits>
#include <limits>

namespace fk {

template <typename T>
__device__ inline cplx<T> cmul(const cplx<T>& a, const cplx<T>& b) {
  cplx<T> r;
  r.re = a.re * b.re - a.im * b.im;
  r.im = a.re * b.im + a.im * b.re;
  return r;
}

constexpr int kPW = kPanelThreads / 64;          // waves of the panel kernel
constexpr int kBP = 33;                          // LDS row of a 32-column block
static_assert(kNBO == 2 * kNB && kTile == kNB, "block sizes");

// Pivot key of a candidate z: the bits of |re| + |im| as a signed integer, which
// orders like the value itself; infinities and NaN order above every number.
// The top bit of `taken` puts pivoted and absent rows below all of them.
template <typename T> struct KeyOf;
template <> struct KeyOf<double> { typedef long long type; };
template <> struct KeyOf<float> { typedef int type; };
__device__ __forceinline__ long long pivot_key(const c64& z, unsigned taken) {
  const long long b = __double_as_longlong(fabs(z.re) + fabs(z.im));
  const unsigned hi = ((unsigned)(b >> 32) & 0x7fffffffu) | (taken & 0x80000000u);
  return (long long)(((unsigned long long)hi << 32) | (unsigned)b);
}
__device__ __forceinline__ int pivot_key(const c32& z, unsigned taken) {
  return (int)((__float_as_uint(fabsf(z.re) + fabsf(z.im)) & 0x7fffffffu) |
               (taken & 0x80000000u));
}
__device__ __forceinline__ int key_hi(long long k) { return (int)(k >> 32); }
__device__ __forceinline__ int key_hi(int k) { return k; }
__device__ __forceinline__ int key_lo(long long k) { return (int)((unsigned)k ^ 0x80000000u); }
__device__ __forceinline__ int key_lo(int) { return 0; }

// Maxima over lanes through the ALU's DPP paths (an LDS permute per step would
// cost about 100 cycles of latency in a chain of six).
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_max(int x) {
  return max(x, __builtin_amdgcn_update_dpp(x, x, CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ int max_of_wave(int x) {    // uniform
  x = dpp_max<0x111, 0xf>(x);
  x = dpp_max<0x112, 0xf>(x);
  x = dpp_max<0x114, 0xf>(x);
  x = dpp_max<0x118, 0xf>(x);          // row_shr 8: lane 15 of each row
  x = dpp_max<0x142, 0xa>(x);          // row_bcast 15 into rows 1 and 3
  x = dpp_max<0x143, 0xc>(x);          // row_bcast 31 into rows 2 and 3
  return __builtin_amdgcn_readlane(x, 63);
}

__device__ __forceinline__ unsigned long long ballot(bool b) {
  return __builtin_amdgcn_ballot_w64(b);
}
// Of the lanes in `mask`, which share the upper word of their keys, those with
// the largest key (FP64: one more maximum, over the lower words).
template <typename K>
__device__ __forceinline__ unsigned long long largest_of(unsigned long long mask, K key) {
  if (sizeof(K) == 8 && (mask & (mask - 1)) != 0) {
    const bool in = (mask >> (threadIdx.x & 63)) & 1;
    const int lo = in ? key_lo(key) : INT_MIN;
    const int top = max_of_wave(lo);
    mask = ballot(in && lo == top);
  }
  return mask;
}

// Of the lanes in `mask`, those whose `slot` (below N) is the smallest.
template <int N>
__device__ __forceinline__ unsigned long long first_slot(unsigned long long mask, int slot) {
  const bool in = (mask >> (threadIdx.x & 63)) & 1;
  unsigned long long s = 0;
#pragma unroll 1
  for (int i = 0; i < N && s == 0; ++i) s = ballot(in && slot == i);
  return s;
}

// This thread's index, opaque to the optimizer: what a panel step derives from
// it (lane maps, masks, LDS offsets) is formed where the step begins instead
// of being kept in registers across the whole panel (about 100 of them).
__device__ __forceinline__ int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Where a panel step's matrix entries live: entry e of the block's row list,
// column c of the step's frame.
template <typename T> struct InMemory {          // the matrix, rows by list
  cplx<T>* x;
  const unsigned* off;                           // byte offset of each entry's row
  typedef unsigned Ref;
  __device__ __forceinline__ Ref ref(int e, int c) const {
    return off[e] + (unsigned)c * (unsigned)sizeof(cplx<T>);
  }
  __device__ __forceinline__ cplx<T>* at(Ref r) const { return at_byte(x, r); }
};
template <typename T> struct InLds {             // a quarter held in LDS
  cplx<T>* q;
  typedef int Ref;
  __device__ __forceinline__ Ref ref(int e, int c) const { return e * kBP + c; }
  __device__ __forceinline__ cplx<T>* at(Ref r) const { return q + r; }
};
// The pivot rows' block B of a block update: values and Re + Im (the third
// real product's operand, formed once here instead of by every row tile).
template <typename T, int KW> struct PivotRows {
  cplx<T> v[KW * kBP];
  T s[KW * kBP];
};

// ------------------------------------------------------- panel: block update
// C <- mask(C) + M B on the columns [c0, c0 + cw) (cw <= 32) of one matrix's m
// listed rows, with M the w <= KW already eliminated columns from j0 on, B
// their pivot rows' values there (in LDS, [KW][kBP], zero outside w x cw) and
// the rows whose pivot column pcol lies in [jp, jp + w) masked.  Columns of
// [skip, skip + w) inside the block are left alone (KW < 32: the eliminated
// group inside its own quarter).
// Each wave takes 16 rows x 32 columns at a time and reads M and C straight
// from memory in the matrix cores' operand layouts, the next step's values in
// flight while the current one is multiplied: nothing but B goes through LDS
// and the waves never wait for each other (row tiles staged through LDS with
// two barriers each reached 50-67% of one compute unit's FP64 matrix rate;
// rank-8 passes on the vector ALUs with the row's values shuffled between
// lanes about a quarter).  All loads of a step are waited for after its
// products and before its stores, so that no load ever waits for a store.
// FULL: w = KW and cw = 32 (no lane masks, loads that are always issued).
// Products in the three-product form of the trailing update.
template <typename T, int KW, int NW, bool FULL, typename V>
__device__ __forceinline__ void block_update_as(const V& x, int m,
                             const int* __restrict__ pcol, int j0, int jp, int w,
                             int c0, int cw, int skip,
                             const PivotRows<T, kNB>& B) {
  typedef typename Mfma<T>::v4 v4;
  constexpr int KS = KW < 32 ? KW / 4 : 8;       // k-steps per chunk
  constexpr int NCH = KW / (4 * KS);
  static_assert(NCH * KS * 4 == KW, "chunks");
  const int tid = fresh_tid();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const bool in0 = FULL || li < cw, in1 = FULL || 16 + li < cw;
  const bool st0 = in0 && !(KW < 32 && li >= skip && li < skip + w);
  const bool st1 = in1 && !(KW < 32 && 16 + li >= skip && 16 + li < skip + w);
  struct CTile {                                 // one tile's C and where it is
    cplx<T> c[2][4];
    typename V::Ref at[4];
    int pc[4];
  };
  auto load_c = [&](CTile& ct, int t) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = min(16 * t + Mfma<T>::drow(lk, v), m - 1);
      ct.at[v] = x.ref(e, c0 + li);
      ct.pc[v] = pcol[e];
      if (FULL) {
        ct.c[0][v] = x.at(ct.at[v])[0];
        ct.c[1][v] = x.at(ct.at[v])[16];
      } else {
        ct.c[0][v].re = ct.c[0][v].im = ct.c[1][v].re = ct.c[1][v].im = T(0);
        if (in0) ct.c[0][v] = x.at(ct.at[v])[0];
        if (in1) ct.c[1][v] = x.at(ct.at[v])[16];
      }
    }
  };
  auto load_m = [&](cplx<T> (&mn)[KS], int t, int ch) {
    const int k0 = 4 * KS * ch;
    const cplx<T>* src = x.at(x.ref(min(16 * t + li, m - 1), j0 + k0 + lk));
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (FULL) {
        mn[s] = src[4 * s];
      } else {
        mn[s].re = mn[s].im = T(0);
        if (k0 + 4 * s + lk < w) mn[s] = src[4 * s];
      }
    }
  };
  const int nt = (m + 15) >> 4;
  if (wave >= nt) return;
  // a short product (KW < 32) has the next tile's C in flight too; a long one
  // covers the latency of its own C, which saves the registers
  constexpr bool kNextC = KW < 32;
  cplx<T> a[KS], mn[KS];
  CTile ct, cn;
  load_m(a, wave, 0);
  if (kNextC) load_c(ct, wave);
#pragma unroll 1
  for (int t = wave; t < nt; t += NW) {
    if (!kNextC) load_c(ct, t);
    v4 p1[2], p2[2], p3[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int v = 0; v < 4; ++v) p1[h][v] = p2[h][v] = p3[h][v] = T(0);
#pragma unroll 1
    for (int ch = 0; ch < NCH; ++ch) {
      cplx<T> b[2][2];
      T bsum[2][2];
      const int bo = (4 * ch * KS + lk) * kBP + li;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        b[0][h] = B.v[bo + 16 * h];
        bsum[0][h] = B.s[bo + 16 * h];
      }
      // the next step (past the last one: rows clamped, values unused)
      if (ch + 1 < NCH) load_m(mn, t, ch + 1);
      else load_m(mn, t + NW, 0);
      if (kNextC) load_c(cn, t + NW);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        // the next k-step's B is read during this one's products; the fence
        // keeps the scheduler from reading all of them at once (registers)
        if (s + 1 < KS) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            b[(s + 1) & 1][h] = B.v[bo + 4 * (s + 1) * kBP + 16 * h];
            bsum[(s + 1) & 1][h] = B.s[bo + 4 * (s + 1) * kBP + 16 * h];
          }
        }
        const T as = a[s].re + a[s].im;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const cplx<T> bb = b[s & 1][h];
          p1[h] = Mfma<T>::run(a[s].re, bb.re, p1[h]);
          p2[h] = Mfma<T>::run(a[s].im, bb.im, p2[h]);
          p3[h] = Mfma<T>::run(as, bsum[s & 1][h], p3[h]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);        // vmcnt(0): every load so far
#pragma unroll
      for (int s = 0; s < KS; ++s) a[s] = mn[s];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool keep = !(ct.pc[v] >= jp && ct.pc[v] < jp + w);
        const T q1 = p1[h][v], q2 = p2[h][v];
        ct.c[h][v].re = (q1 - q2) + (keep ? ct.c[h][v].re : T(0));
        ct.c[h][v].im = ((p3[h][v] - q1) - q2) + (keep ? ct.c[h][v].im : T(0));
      }
    if (FULL && 16 * t + 16 <= m) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (KW >= 32 || (h ? st1 : st0)) {
#pragma unroll
          for (int v = 0; v < 4; ++v) x.at(ct.at[v])[16 * h] = ct.c[h][v];
        }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if ((h ? st1 : st0) && 16 * t + Mfma<T>::drow(lk, v) < m)
            x.at(ct.at[v])[16 * h] = ct.c[h][v];
    }
    if (kNextC) ct = cn;
  }
}
template <typename T, int KW, int NW = kPW, typename V>
__device__ __forceinline__ void block_update(const V& x, int m,
                             const int* __restrict__ pcol, int j0, int jp, int w,
                             int c0, int cw, int skip,
                             const PivotRows<T, kNB>& B) {
  if (w == KW && cw == 32)
    block_update_as<T, KW, NW, true>(x, m, pcol, j0, jp, w, c0, cw, skip, B);
  else
    block_update_as<T, KW, NW, false>(x, m, pcol, j0, jp, w, c0, cw, skip, B);
}

// B of block_update: row l, column c = value of list entry pive[l] (the pivot
// row of column l) in column c0 + c, zero outside w x cw and in
// [skip, skip + w) (skip < 0: none).
template <typename T, int KW, typename V>
__device__ __forceinline__ void load_pivot_rows(const V& x, const int* pive, int w, int c0,
                             int cw, int skip, PivotRows<T, kNB>& B) {
  const int tid = fresh_tid();
#pragma unroll
  for (int e0 = 0; e0 < KW * 32; e0 += kPanelThreads) {
    const int e = e0 + tid;
    if (KW * 32 >= kPanelThreads || e < KW * 32) {
      const int l = e >> 5, c = e & 31;
      cplx<T> v = *x.at(x.ref(pive[min(l, w - 1)], c0 + min(c, cw - 1)));
      if (!(l < w && c < cw) || (skip >= 0 && c >= skip && c < skip + w))
        v.re = v.im = T(0);
      B.v[l * kBP + c] = v;
      B.s[l * kBP + c] = v.re + v.im;
    }
  }
}

// -------------------------------------------------- panel: column elimination
// LDS of one group's pivot search: each wave's candidate (key, place and
// the row's values), double-buffered by column parity so that one column's
// reads never meet the next column's writes.
template <typename T, int IB> struct Candidates {
  cplx<T> row[2][kPW][IB];
  int hi[2][kPW];      // upper word of the key
  int entry[2][kPW];   // the candidate's place in the row list
};

// The group's IB columns of the thread's rows, loaded and stored with the
// lanes along the rows (IB lanes per row, whole cache lines per access) and
// transposed through a wave's own part of LDS: one row per lane would touch 64
// lines per access, and a load or store of a group then costs as much as
// eliminating it.
template <typename T, int RPT, int IB>
__device__ __forceinline__ void load_group(const InMemory<T>& x, int m, int c, int iw,
                                           int tid, cplx<T>* stage, cplx<T> (&v)[RPT][IB]) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int RL = 64 / IB, P = IB + 1;        // rows per access, LDS pitch
  cplx<T>* sw = stage + wave * 64 * P;
  const int lr = lane / IB, lc = lane % IB;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int e0 = wave * 64 + i * kPanelThreads;
    if (e0 < m) {                                // the same for the whole wave
      cplx<T> t[IB];
#pragma unroll
      for (int j = 0; j < IB; ++j) {
        t[j].re = t[j].im = T(0);
        const int e = e0 + j * RL + lr;
        if (e < m && lc < iw) t[j] = *x.at(x.ref(e, c + lc));
      }
#pragma unroll
      for (int j = 0; j < IB; ++j) sw[(j * RL + lr) * P + lc] = t[j];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // within the wave
#pragma unroll
      for (int l = 0; l < IB; ++l) v[i][l] = sw[lane * P + l];
      // the next rows' writes follow every lane's reads
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    } else {
#pragma unroll
      for (int l = 0; l < IB; ++l) v[i][l].re = v[i][l].im = T(0);
    }
  }
}
template <typename T, int RPT, int IB>
__device__ __forceinline__ void store_group(const InMemory<T>& x, int m, int c, int iw,
                                            int tid, cplx<T>* stage,
                                            const cplx<T> (&v)[RPT][IB]) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int RL = 64 / IB, P = IB + 1;
  cplx<T>* sw = stage + wave * 64 * P;
  const int lr = lane / IB, lc = lane % IB;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int e0 = wave * 64 + i * kPanelThreads;
    if (e0 < m) {
#pragma unroll
      for (int l = 0; l < IB; ++l) sw[lane * P + l] = v[i][l];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int j = 0; j < IB; ++j) {
        const int e = e0 + j * RL + lr;
        if (e < m && lc < iw) *x.at(x.ref(e, c + lc)) = sw[(j * RL + lr) * P + lc];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
}
template <typename T, int RPT, int IB>
__device__ __forceinline__ void load_group(const InLds<T>& x, int m, int c, int iw,
                                           int tid, cplx<T>*, cplx<T> (&v)[RPT][IB]) {
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int e = tid + i * kPanelThreads;
#pragma unroll
    for (int l = 0; l < IB; ++l) {
      v[i][l].re = v[i][l].im = T(0);
      if (e < m && l < iw) v[i][l] = *x.at(x.ref(e, c + l));
    }
  }
}
template <typename T, int RPT, int IB>
__device__ __forceinline__ void store_group(const InLds<T>& x, int m, int c, int iw,
                                            int tid, cplx<T>*, const cplx<T> (&v)[RPT][IB]) {
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int e = tid + i * kPanelThreads;
#pragma unroll
    for (int l = 0; l < IB; ++l)
      if (e < m && l < iw) *x.at(x.ref(e, c + l)) = v[i][l];
  }
}

// Eliminate IB columns in registers on the m listed rows, with partial
// pivoting; thread tid owns list entries tid + i kPanelThreads, i < RPT, and
// bit i of `taken` is set once that entry is pivoted, or if absent.
// The columns are c .. in the frame of x and ca .. of the matrix.
// The pivot is the largest |re| + |im| of the rows left, compared in full; among
// equal ones the lowest row.  So a row's |re| + |im| is at most the pivot's, and
// a multiplier's modulus at most sqrt(2).  One integer maximum over the keys'
// upper words finds the pivot but for ties, which the lower words (FP64) and then
// the rows' order settle off the common path.  (A maximum over keys cut to 7 to
// 11 mantissa bits, their low bits the row's place, took pivots up to 1 / 128
// below the largest; impurity_1800 9.16 ms as here, loop_150 8.15 -> 8.21 ms.)
// One barrier per column: every wave publishes its best candidate together
// with the candidate's row, so that the row is in LDS when the winner is
// known.  The chain per column bounds it (maximum over the wave's lanes,
// publication, barrier, the reciprocal: about 1000 cycles), so the next
// column's maximum runs beside the rest of the row update, waves without rows
// only take part in the barrier, and RPT is chosen by the rows left.
// The column loop is not unrolled: each step writes a row's columns one slot
// down as it updates them, so that the column to eliminate is always slot 0
// (the row is back in order after IB steps).
template <typename T, int RPT, int IB, typename V>
__device__ __forceinline__ void eliminate_columns(const V& x, const int* rows, int m,
                             int c, int ca, int iw, unsigned& taken,
                             int* __restrict__ piv, int* __restrict__ rowcol, int* pcol,
                             int* pive, int* __restrict__ status, cplx<T>* stage,
                             Candidates<T, IB>& cd) {
  typedef typename KeyOf<T>::type K;
  const int tid = fresh_tid(), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool any = wave * 64 < m;                // this wave holds rows
  cplx<T> v[RPT][IB];
  if (any) load_group<T, RPT, IB>(x, m, c, iw, tid, stage, v);
  else if (lane == 0) cd.hi[0][wave] = cd.hi[1][wave] = INT_MIN;
  // this thread's largest key and the row that holds it (the first of equal ones)
  K best;
  int slot;
  auto thread_best = [&]() {
    best = pivot_key(v[0][0], taken << 31);
    slot = 0;
#pragma unroll
    for (int i = 1; i < RPT; ++i) {
      const K k = pivot_key(v[i][0], taken << (31 - i));
      if (k > best) {
        best = k;
        slot = i;
      }
    }
  };
  thread_best();
  int wmax = any ? max_of_wave(key_hi(best)) : INT_MIN;
#pragma unroll 1
  for (int l = 0; l < iw; ++l) {
    const int par = l & 1;
    if (any) {
      auto publish = [&]() {
        cd.hi[par][wave] = wmax;
        cd.entry[par][wave] = tid + slot * kPanelThreads;
#pragma unroll
        for (int i = 0; i < RPT; ++i)
          if (RPT == 1 || i == slot) {
#pragma unroll
            for (int q = 0; q < IB; ++q) cd.row[par][wave][q] = v[i][q];
          }
      };
      const bool lead = key_hi(best) == wmax;
      unsigned long long top = ballot(lead);
      if (lead) publish();
      if (__builtin_expect((top & (top - 1)) != 0, 0)) {
        // several lanes wrote to the one place: the right one writes again
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        top = largest_of(top, best);
        if (RPT > 1) top = first_slot<RPT>(top, slot);
        if (lane == __builtin_ctzll(top)) publish();
      }
    }
    __syncthreads();
    if (!any) continue;
    // ---- the block's pivot, from the kPW candidates
    int gmax = cd.hi[par][0];
#pragma unroll
    for (int q = 1; q < kPW; ++q) gmax = max(gmax, cd.hi[par][q]);
    const int w8 = lane & (kPW - 1);
    constexpr unsigned long long kWaves = (1ull << kPW) - 1;
    unsigned long long top = ballot(cd.hi[par][w8] == gmax) & kWaves;
    cplx<T> prow[IB];
    int pe;   // its list entry
    auto take = [&]() {
      const int win = __builtin_ctzll(top);
      pe = cd.entry[par][win];
#pragma unroll
      for (int q = 0; q < IB; ++q) prow[q] = cd.row[par][win][q];
    };
    take();
    if (__builtin_expect((top & (top - 1)) != 0, 0)) {
      top = largest_of(top, pivot_key(cd.row[par][w8][0], 0u));
      if (RPT > 1 && (top & (top - 1)) != 0) {
        const int e = (top >> lane) & 1 ? -cd.entry[par][w8] : INT_MIN;
        const int first = max_of_wave(e);
        top = ballot(e == first);
      }
      take();
    }
    const int pi = pe / kPanelThreads;
    // two divisions, not products with 1 / den: that overflows where den is
    // below the smallest normal number while the quotients do not (lattice_150
    // 502 -> 504 us, impurity_1800 9.10 -> 9.16 ms)
    const T den = prow[0].re * prow[0].re + prow[0].im * prow[0].im;
    cplx<T> inv;
    inv.re = prow[0].re / den;
    inv.im = -prow[0].im / den;
    const bool mine = (pe & (kPanelThreads - 1)) == tid;
    if (mine) {
      const int e = min(pe, m - 1), p = rows[e];
      piv[ca + l] = p;
      rowcol[p] = ca + l;
      pcol[e] = ca + l;
      pive[l] = e;
      const T size = fabs(prow[0].re) + fabs(prow[0].im);
      if (__builtin_expect(!(size > T(0) && size < std::numeric_limits<T>::max()), 0))
        atomicCAS(status, 0, size == T(0) ? (1 + ca + l) : -(1 + ca + l));
    }
    // ---- eliminate the column from every other row (Gauss-Jordan): row <-
    // row - t prow with t = row[0] / pivot and -t in this column's place.  The
    // pivot row itself becomes prow / pivot: the same update of a zero row
    // with t = -1 / pivot.
    auto update = [&](int i, const cplx<T>& t, int q) {
      v[i][q - 1].re = fma(t.im, prow[q].im, fma(-t.re, prow[q].re, v[i][q].re));
      v[i][q - 1].im = fma(-t.im, prow[q].re, fma(-t.re, prow[q].im, v[i][q].im));
    };
    // (many rows per thread: no registers to keep every t)
    constexpr bool kOverlap = RPT <= 4;
    cplx<T> t[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      t[i] = cmul(v[i][0], inv);
      if (mine && i == pi) {
        taken |= 1u << i;
        t[i].re = -inv.re;
        t[i].im = -inv.im;
#pragma unroll
        for (int q = 1; q < IB; ++q) v[i][q].re = v[i][q].im = T(0);
      }
      update(i, t[i], 1);
      if (!kOverlap) {
#pragma unroll
        for (int q = 2; q < IB; ++q) update(i, t[i], q);
        v[i][IB - 1].re = -t[i].re;
        v[i][IB - 1].im = -t[i].im;
      }
    }
    thread_best();
    wmax = max_of_wave(key_hi(best));
    if (kOverlap) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
#pragma unroll
        for (int q = 2; q < IB; ++q) update(i, t[i], q);
        v[i][IB - 1].re = -t[i].re;
        v[i][IB - 1].im = -t[i].im;
      }
    }
  }
#pragma unroll 1
  for (int l = iw; l < IB; ++l)   // a short group: back in order
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const cplx<T> f = v[i][0];
#pragma unroll
      for (int q = 1; q < IB; ++q) v[i][q - 1] = v[i][q];
      v[i][IB - 1] = f;
    }
  if (any) store_group<T, RPT, IB>(x, m, c, iw, tid, stage, v);
}

// Outer block S of one matrix.  Rows pivoted in earlier blocks take no part:
// their columns of this block follow from the block's pivot rows afterwards
// (k_fix), so the panel reads and writes only the n - S kNBO remaining rows,
// at most RPT kPanelThreads.  Four 32-column quarters; each eliminates groups
// of IB columns in registers, whose transform then updates the quarter's
// other columns (block_update with KW = IB), and is joined to the other
// quarter of its 64-column half and the halves to each other by updates with
// KW = 32 and 64.  QR > 0: at most QR rows; the quarter is kept in LDS while
// it is factored, so that its groups meet LDS latencies instead of memory's.
// One matrix of N_c = 1800: 1359 -> 695 us per block on average over the
// blocks; 100 matrices of N_c = 150: 370 -> 130 us; 225 of N_c = 1800: 1636 ->
// 1250 us, where the quarters' passes are bound by memory traffic.
// kQuarters: only quarter `only`, on the same rows; the joins are launches of
// k_cross, for which the quarter's pivot rows are copied aside.  kGroups: only
// group `only`; its update of the quarter's other columns is such a launch too.
enum PanelForm { kWhole, kQuarters, kGroups };
template <typename T, int RPT, int IB, int QR, PanelForm FORM>
__global__ __launch_bounds__(kPanelThreads, 1) void k_outer_panel(
    cplx<T>* __restrict__ xbuf, int* __restrict__ pivbuf,
    int* __restrict__ rowcolbuf, const MatDesc* __restrict__ descs, int S,
    int* __restrict__ status, int only, cplx<T>* __restrict__ side) {
  constexpr int kCap = QR > 0 ? QR : RPT * kPanelThreads;
  constexpr bool SPLIT = FORM != kWhole;
  constexpr int kPart = FORM == kGroups ? IB : 32;   // columns of part `only`
  static_assert(kCap <= RPT * kPanelThreads, "panel rows");
  __shared__ PivotRows<T, kNB> B;
  __shared__ Candidates<T, IB> cd;
  // a wave's transpose buffers, or the quarter
  __shared__ cplx<T> stage[QR > 0 ? QR * kBP : kPW * 64 * (IB + 1)];
  __shared__ int rows[kCap];
  __shared__ unsigned roff[kCap];   // byte offset of each entry's row
  __shared__ int pcol[kCap];     // pivot column of each list entry, or -1
  __shared__ int pive[kNBO];     // list entry of each column's pivot row
  __shared__ int cnt[2][kPW];
  const MatDesc d = descs[blockIdx.x];
  const int n = d.n;
  const int J0 = S * kNBO;
  if (J0 >= n || (SPLIT && J0 + kPart * only >= n)) return;
  int* piv = pivbuf + d.ioff;
  int* rowcol = rowcolbuf + d.ioff;
  int* st = status + d.status_idx;

  // list the rows not pivoted before the block (wave ballots, then offsets);
  // m = n - J0 <= kCap: every earlier column pivoted one row
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int m = 0;
  for (int r0 = 0, b = 0; r0 < n; r0 += kPanelThreads, b ^= 1) {
    const int r = r0 + tid;
    const int rc = rowcol[min(r, n - 1)];
    const unsigned long long bal = __ballot(r < n && (rc < 0 || (SPLIT && rc >= J0)));
    if (lane == 0) cnt[b][wave] = (int)__popcll(bal);
    __syncthreads();
    int pos = m + (int)__popcll(bal & ((1ull << lane) - 1ull));
#pragma unroll
    for (int q = 0; q < kPW; ++q) {
      const int k = cnt[b][q];
      pos += q < wave ? k : 0;
      m += k;
    }
    if (((bal >> lane) & 1ull) && pos < kCap) {
      rows[pos] = r;
      roff[pos] = (unsigned)r * (unsigned)d.ld * (unsigned)sizeof(cplx<T>);
      pcol[pos] = rc;
    }
  }
  m = min(m, kCap);
  __syncthreads();
  if (m == 0) return;   // the same for every thread

  unsigned taken = 0;            // see eliminate_columns
  static_assert(RPT <= 32, "bits");
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int e = tid + i * kPanelThreads;
    if (!(e < m && (!SPLIT || pcol[e] < 0))) taken |= 1u << i;
  }

  const int J1 = J0 + kNB;
  const InMemory<T> x{xbuf + d.xoff, roff};
  // update the columns [c0, c0 + cw) with the transform of [j0, j0 + w); the
  // barriers order it after the writes before it and before the reads after
  auto cross32 = [&](int j0, int w, int c0, int cw) {
    load_pivot_rows<T, 32>(x, pive + (j0 - J0), w, c0, cw, -1, B);
    __syncthreads();
    block_update<T, 32>(x, m, pcol, j0, j0, w, c0, cw, 0, B);
    __syncthreads();
  };
  auto cross64 = [&](int j0, int w, int c0) {
#pragma unroll 1
    for (int c = c0; c < min(c0 + kNB, n); c += 32) {
      load_pivot_rows<T, kNB>(x, pive + (j0 - J0), w, c, min(32, n - c), -1, B);
      __syncthreads();
      block_update<T, kNB>(x, m, pcol, j0, j0, w, c, min(32, n - c), 0, B);
      __syncthreads();
    }
  };
  // factor the quarter [c0, c0 + cw), whose columns start at f in the frame
  auto quarter = [&](const auto& view, int f, int c0, int cw) {
#pragma unroll 1
    for (int b0 = 0; b0 < cw; b0 += IB) {
      const int iw = min(IB, cw - b0);
      int* pe = pive + (c0 - J0) + b0;
      eliminate_columns<T, RPT, IB>(view, rows, m, f + b0, c0 + b0, iw, taken, piv,
                                          rowcol, pcol, pe, st, stage, cd);
      __syncthreads();   // pive, pcol and the eliminated columns
      if (cw > IB) {
        load_pivot_rows<T, IB>(view, pe, iw, f, cw, b0, B);
        __syncthreads();
        block_update<T, IB>(view, m, pcol, f + b0, c0 + b0, iw, f, cw, b0, B);
        __syncthreads();
      }
    }
  };
  auto copy_quarter = [&](int c0, int cw, bool out) {
    for (int e = tid; e < 32 * m; e += kPanelThreads) {
      const int r = e >> 5, c = e & 31;
      if (c < cw) {
        if (out) *x.at(x.ref(r, c0 + c)) = stage[r * kBP + c];
        else stage[r * kBP + c] = *x.at(x.ref(r, c0 + c));
      }
    }
    __syncthreads();
  };
  if constexpr (SPLIT) {
    const int c0 = J0 + kPart * only, cw = min(kPart, n - c0);
    if constexpr (FORM == kGroups) {
      eliminate_columns<T, RPT, IB>(x, rows, m, c0, c0, cw, taken, piv, rowcol, pcol,
                                          pive + (c0 - J0), st, stage, cd);
      __syncthreads();
    } else if constexpr (QR > 0) {
      copy_quarter(c0, cw, false);
      quarter(InLds<T>{stage}, 0, c0, cw);
      copy_quarter(c0, cw, true);
    } else {
      quarter(x, c0, c0, cw);
    }
    cplx<T>* out = side + (size_t)blockIdx.x * kNBO * kNBO + (size_t)(c0 - J0) * kNBO;
    for (int e = tid; e < cw * kNBO; e += kPanelThreads) {
      const int l = e / kNBO, c = e % kNBO;
      if (J0 + c < n) out[e] = *x.at(x.ref(pive[c0 - J0 + l], J0 + c));
    }
    return;
  }
#pragma unroll 1
  for (int qi = 0; qi < 6; ++qi) {
    // steps 0, 1, 3, 4: the quarters; 2 and 5: left half to right and back
    if (qi == 2 || qi == 5) {
      const int j0 = qi == 2 ? J0 : J1, c0 = qi == 2 ? J1 : J0;
      if (J1 < n) cross64(j0, min(kNB, n - j0), c0);
      continue;
    }
    const int qq = qi < 2 ? qi : qi - 1;
    const int c0 = J0 + 32 * qq;
    if (c0 >= n) continue;
    const int cw = min(32, n - c0);
    if constexpr (QR > 0) {
      copy_quarter(c0, cw, false);
      quarter(InLds<T>{stage}, 0, c0, cw);
      copy_quarter(c0, cw, true);
    } else {
      quarter(x, c0, c0, cw);
    }
    const int dst = (qq & 1) ? c0 - 32 : c0 + 32;
    if (dst < n) cross32(c0, cw, dst, min(32, n - dst));
  }
}

// Join of a split panel's parts: the columns [co, co + 32 gridDim.z) of block S
// receive the transform of its KW columns from jo on (offsets in the block) on
// all rows not pivoted before the block, 64 rows per workgroup; B was copied
// aside by the parts' launches.  KW < 32: a group inside its own quarter, whose
// columns it leaves alone.
template <typename T, int KW>
__global__ __launch_bounds__(256, 2) void k_cross(
    cplx<T>* __restrict__ xbuf, const int* __restrict__ rowcolbuf,
    const cplx<T>* __restrict__ side, const MatDesc* __restrict__ descs, int S, int jo,
    int co) {
  __shared__ PivotRows<T, kNB> B;
  __shared__ unsigned roff[64];
  __shared__ int pcol[64], count;
  const MatDesc d = descs[blockIdx.y];
  const int n = d.n, J0 = S * kNBO, j0 = J0 + jo;
  const int cz = co + 32 * blockIdx.z, c0 = J0 + cz;
  const int r0 = 64 * blockIdx.x;
  if (j0 >= n || c0 >= n || r0 >= n) return;
  const int w = min(KW, n - j0), cw = min(32, n - c0);
  const int tid = threadIdx.x;
  if (tid < 64) {
    const int r = r0 + tid, rc = rowcolbuf[d.ioff + min(r, n - 1)];
    const unsigned long long bal = __ballot(r < n && (rc < 0 || rc >= J0));
    if ((bal >> tid) & 1ull) {
      const int pos = (int)__popcll(bal & ((1ull << tid) - 1ull));
      roff[pos] = (unsigned)r * (unsigned)d.ld * (unsigned)sizeof(cplx<T>);
      pcol[pos] = rc;
    }
    if (tid == 0) count = (int)__popcll(bal);
  }
  const cplx<T>* src = side + (size_t)blockIdx.y * kNBO * kNBO + (size_t)jo * kNBO + cz;
  for (int e = tid; e < KW * 32; e += 256) {
    const int l = e >> 5, c = e & 31;
    cplx<T> v;
    v.re = v.im = T(0);
    if (l < w && c < cw) v = src[l * kNBO + c];
    B.v[l * kBP + c] = v;
    B.s[l * kBP + c] = v.re + v.im;
  }
  __syncthreads();
  const int m = count;
  if (m == 0) return;
  const InMemory<T> x{xbuf + d.xoff, roff};
  block_update<T, KW, 4>(x, m, pcol, j0, j0, w, c0, cw, KW < 32 ? jo - cz : 0, B);
}

// ------------------------------------------------------------------ gather
template <typename T>
__global__ void k_gather(const cplx<T>* __restrict__ xbuf,
                         cplx<T>* __restrict__ bbuf,
                         const int* __restrict__ pivbuf,
                         const MatDesc* __restrict__ descs, int S) {
  const MatDesc d = descs[blockIdx.y];
  const int l = blockIdx.x;
  const int J0 = S * kNBO;
  if (J0 >= d.n || l >= min(kNBO, d.n - J0)) return;
  const int p = pivbuf[d.ioff + J0 + l];
  const cplx<T>* src = xbuf + d.xoff + (size_t)p * d.ld;
  cplx<T>* dst = bbuf + d.boff + (size_t)(block_brow(d.n, S) + l) * d.ld;
  for (int c = threadIdx.x; c < d.n; c += blockDim.x) dst[c] = src[c];
}

// ----------------------------------------------------------------- fix-up
// Rows pivoted in earlier outer blocks skip the panel.  For such a row r the
// block's Gauss-Jordan steps amount to X[r, P] <- -X0[r, P] Minv, with X0 the
// row's values before the block and Minv = X[R, P] the block's pivot rows R in
// pivot order after the panel (the inverse of X0[R, P]), which the gather has
// copied into B.  Those rows are piv[0, J0) in pivot order; one 512-thread
// workgroup takes 64 of them and all of the block's columns, reading its
// rows' X0 before writing, so the product is formed in place.  Eight waves
// as 2 x 4 blocks of 32 x 32, K in chunks of kKC double-buffered in LDS.
template <typename T>
__global__ __launch_bounds__(512, 1) void k_fix(
    cplx<T>* __restrict__ xbuf, const cplx<T>* __restrict__ bbuf,
    const int* __restrict__ pivbuf, const MatDesc* __restrict__ descs, int S) {
  typedef typename Mfma<T>::v4 v4;
  constexpr int TR = 64, TC = kNBO, NT = 512;
  constexpr int AP = kKC + 1, BP = TC + 1;
  __shared__ cplx<T> As[2][TR * AP];
  __shared__ cplx<T> Bsh[2][kKC * BP];
  constexpr int kLA = TR * kKC / NT;
  constexpr int kLB = kKC * TC / NT;
  static_assert(kLA * NT == TR * kKC && kLB * NT == kKC * TC, "fix tile");

  const MatDesc d = descs[blockIdx.y];
  const int n = d.n, ld = d.ld;
  const int J0 = S * kNBO, i0 = blockIdx.x * TR;
  if (J0 >= n || i0 + TR > J0) return;   // J0 is a multiple of TR
  const int wO = min(kNBO, n - J0);
  const int nch = (wO + kKC - 1) / kKC;
  cplx<T>* xm = xbuf + d.xoff;
  const cplx<T>* bm = bbuf + d.boff + (size_t)block_brow(n, S) * ld;
  const int* piv = pivbuf + d.ioff;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 2, wc = wave & 3;
  const int li = lane & 15, lk = lane >> 4;

  int ra[kLA];
#pragma unroll
  for (int t = 0; t < kLA; ++t) ra[t] = piv[i0 + (tid + t * NT) / kKC];
  cplx<T> pa[kLA], pb[kLB];
  auto load = [&](int kb) {
#pragma unroll
    for (int t = 0; t < kLA; ++t) {
      const int k = (tid + t * NT) % kKC;
      pa[t] = xm[(size_t)ra[t] * ld + J0 + min(kb + k, wO - 1)];
    }
#pragma unroll
    for (int t = 0; t < kLB; ++t) {
      const int e = tid + t * NT;
      const int k = e / TC, c = e % TC;
      pb[t] = bm[(size_t)min(kb + k, wO - 1) * ld + J0 + min(c, wO - 1)];
    }
  };
  auto stash = [&](int kb, int buf) {
#pragma unroll
    for (int t = 0; t < kLA; ++t) {
      const int e = tid + t * NT;
      const int i = e / kKC, k = e % kKC;
      cplx<T> v = pa[t];
      if (!(kb + k < wO)) v.re = v.im = T(0);
      As[buf][i * AP + k] = v;
    }
#pragma unroll
    for (int t = 0; t < kLB; ++t) {
      const int e = tid + t * NT;
      const int k = e / TC, c = e % TC;
      cplx<T> v = pb[t];
      if (!(kb + k < wO && c < wO)) v.re = v.im = T(0);
      Bsh[buf][k * BP + c] = v;
    }
  };
  v4 p1[2][2], p2[2][2], p3[2][2];   // three-product form, as k_update
#pragma unroll
  for (int ii = 0; ii < 2; ++ii)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p1[ii][jj][v] = T(0);
        p2[ii][jj][v] = T(0);
        p3[ii][jj][v] = T(0);
      }
  load(0);
  stash(0, 0);
  __syncthreads();
  for (int kc = 0; kc < nch; ++kc) {
    const int buf = kc & 1;
    const bool more = kc + 1 < nch;
    if (more) load((kc + 1) * kKC);
    const cplx<T>* as = As[buf];
    const cplx<T>* bs = Bsh[buf];
#pragma unroll
    for (int k = 0; k < kKC; k += 4) {
      T ar[2], ai[2], as_[2], br[2], bi[2], bs_[2];
#pragma unroll
      for (int ii = 0; ii < 2; ++ii) {
        const cplx<T> a = as[(32 * wr + 16 * ii + li) * AP + k + lk];
        ar[ii] = a.re;
        ai[ii] = a.im;
        as_[ii] = a.re + a.im;
      }
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const cplx<T> b = bs[(k + lk) * BP + 32 * wc + 16 * jj + li];
        br[jj] = b.re;
        bi[jj] = b.im;
        bs_[jj] = b.re + b.im;
      }
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          p1[ii][jj] = Mfma<T>::run(ar[ii], br[jj], p1[ii][jj]);
          p2[ii][jj] = Mfma<T>::run(ai[ii], bi[jj], p2[ii][jj]);
          p3[ii][jj] = Mfma<T>::run(as_[ii], bs_[jj], p3[ii][jj]);
        }
    }
    if (more) stash((kc + 1) * kKC, buf ^ 1);
    __syncthreads();
  }
  // every global read of the rows is done (last barrier): write in place
#pragma unroll
  for (int ii = 0; ii < 2; ++ii)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = piv[i0 + 32 * wr + 16 * ii + Mfma<T>::drow(lk, v)];
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int col = 32 * wc + 16 * jj + li;
        if (col < wO) {
          cplx<T> c;
          const T q1 = p1[ii][jj][v], q2 = p2[ii][jj][v];
          c.re = q2 - q1;
          c.im = (q1 + q2) - p3[ii][jj][v];
          xm[(size_t)r * ld + J0 + col] = c;
        }
      }
    }
}

// ------------------------------------------------------------------ update
// C <- mask_P(C) + M B for the listed tiles of (32 WR) x 64: 2 WR waves as
// WR x 2 blocks of 32 x 32 (WR = 2: 64 x 64 tiles, two workgroups per CU;
// WR = 4: 128 x 64 tiles sharing each B chunk, one workgroup per CU).
// Edge tiles load clamped rows and columns and do not store what lies outside.
template <typename T, int WR>
__global__ __launch_bounds__(128 * WR, 4 / WR) void k_update(
    cplx<T>* __restrict__ xbuf, const cplx<T>* __restrict__ bbuf,
    const int* __restrict__ rowcolbuf, const MatDesc* __restrict__ descs,
    const TileItem* __restrict__ items, int nitems) {
  typedef TileProduct<T, WR> P;
  __shared__ typename P::Lds lds;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int per = gridDim.x >> 3;
  const int chunk = (nitems + 7) >> 3;
  const int lo = xcd * chunk, hi = min(nitems, lo + chunk);

  for (int it = lo + slot; it < hi; it += per) {
    const TileItem ti = items[it];
    const MatDesc d = descs[ti.mat];
    const int n = d.n, ld = d.ld;
    // M = columns [J0, J0 + wO), B = side-buffer rows [b0, b0 + wO)
    const int J0 = ti.jb * kNBO, wO = ti.kw;
    const int r0 = ti.tr * P::TR, c0 = ti.tc * kTile;
    cplx<T>* xm = xbuf + d.xoff;
    const int* rowcol = rowcolbuf + d.ioff;
    P tp;
    tp.begin(lds, xm + J0, ld, r0, n, bbuf + d.boff + (size_t)ti.b0 * ld, ld, c0, n, wO);
    tp.run(lds);
    typename P::c2* xc = reinterpret_cast<typename P::c2*>(xm);
    // C and the pivot columns of the rows this lane writes: all at once in FP64;
    // by halves in complex64, whose 120 registers (instead of 146) let four
    // workgroups share a CU (85.5 -> 83.1 ms for 225 matrices of N_c = 1800;
    // FP64 by halves: 155.9 -> 157.2)
    constexpr int kRows = sizeof(T) == 8 ? 2 : 1;
#pragma unroll
    for (int i0 = 0; i0 < 2; i0 += kRows) {
      int rcv[kRows][4];
      typename P::c2 cv[kRows][2][4];
#pragma unroll
      for (int q = 0; q < kRows; ++q) {
#pragma unroll
        for (int v = 0; v < 4; ++v) rcv[q][v] = rowcol[min(tp.row(i0 + q, v), n - 1)];
        tp.for_outputs(i0 + q, [&](int, int jj, int v, bool in, unsigned off) {
          if (in) cv[q][jj][v] = *at_byte(xc, off);
        });
      }
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        tp.for_outputs(i0 + q, [&](int ii, int jj, int v, bool in, unsigned off) {
          const bool keep = !(rcv[q][v] >= J0 && rcv[q][v] < J0 + wO);
          typename P::c2 c = tp.value(ii, jj, v);
          c.x += keep ? cv[q][jj][v].x : T(0);
          c.y += keep ? cv[q][jj][v].y : T(0);
          if (in) *at_byte(xc, off) = c;
        });
    }
    if (per < hi - lo) __syncthreads();   // LDS free for the next item
  }
}

// --------------------------------------------------------------- launchers
template <typename T>
hipError_t gje_panel(cplx<T>* x, int* piv, int* rowcol, const MatDesc* d,
                     int nmat, int nmax, int S, int* status, cplx<T>* side,
                     hipStream_t st, int* launches) {
  const int left = nmax - S * kNBO;    // rows left of the largest matrix
  if (nmat <= 0 || left <= 0) return hipSuccess;
  if (nmax > kMaxN) return hipErrorInvalidValue;
  // by the rows left: quarters of at most 192 (complex64 448) rows stay in
  // LDS; then one, two or four rows per thread; beyond 2048 rows four columns
  // per register block keep the rows in registers
  auto one = [&](auto kernel, int only) {
    hipLaunchKernelGGL(kernel, dim3(nmat), dim3(kPanelThreads), 0, st, x, piv, rowcol, d, S,
                       status, only, side);
    ++*launches;
  };
  constexpr int kC64 = sizeof(T) == 4 ? 448 : 0;
  constexpr int kMany = kMaxN / kPanelThreads;
  // few matrices leave most CUs idle while one CU each joins the panel's
  // parts: the joins then run as launches over all row tiles
  if (!side || nmat > kSplitMats || left <= kSplitRows) {
    if (left <= 192) one(k_outer_panel<T, 1, kIB, 192, kWhole>, 0);
    else if (left <= kC64) one(k_outer_panel<T, 1, kIB, kC64, kWhole>, 0);
    else if (left <= kPanelThreads) one(k_outer_panel<T, 1, kIB, 0, kWhole>, 0);
    else if (left <= 2 * kPanelThreads) one(k_outer_panel<T, 2, kIB, 0, kWhole>, 0);
    else if (left <= 4 * kPanelThreads) one(k_outer_panel<T, 4, kIB, 0, kWhole>, 0);
    else if (left <= 6 * kPanelThreads) one(k_outer_panel<T, 6, 4, 0, kWhole>, 0);
    else one(k_outer_panel<T, kMany, 4, 0, kWhole>, 0);
    return hipGetLastError();
  }
  auto cross = [&](auto kernel, int jo, int co, int nz) {
    if (jo >= left || co >= left) return;
    hipLaunchKernelGGL(kernel, dim3((nmax + 63) / 64, nmat, nz), dim3(256), 0, st, x, rowcol,
                       side, d, S, jo, co);
    ++*launches;
  };
  // With more than 512 rows the groups' updates of a quarter too are launches
  // over all row tiles: one CU would move the quarter through memory once per
  // group.  One matrix of N_c = 1800 10.6 -> 9.1 ms per impurity update, 25 of
  // N_c = 4100 224 -> 215 ms.  Beyond 1024 rows level at 64 matrices and faster
  // with fewer; from 513 to 1024 rows the launches cost more than they save
  // above kGroupMats (N_c = 1000: 16 matrices 5.36 -> 5.07 ms, 32 7.46 -> 7.35,
  // 48 9.65 both, 64 11.7 -> 11.9); up to 512 rows no difference.
  auto groups = [&](auto kernel, auto join, int ib, int o) {
    for (int g = o; g < std::min(o + 32, left); g += ib) {
      one(kernel, g / ib);
      cross(join, g, o, 1);
    }
  };
  auto quarter = [&](int o) {
    const int q = o / 32;
    if (left <= kC64) one(k_outer_panel<T, 1, kIB, kC64, kQuarters>, q);
    else if (left <= kPanelThreads) one(k_outer_panel<T, 1, kIB, 0, kQuarters>, q);
    else if (left <= 2 * kPanelThreads && nmat > kGroupMats)
      one(k_outer_panel<T, 2, kIB, 0, kQuarters>, q);
    else if (left <= 2 * kPanelThreads)
      groups(k_outer_panel<T, 2, kIB, 0, kGroups>, k_cross<T, kIB>, kIB, o);
    else if (left <= 4 * kPanelThreads)
      groups(k_outer_panel<T, 4, kIB, 0, kGroups>, k_cross<T, kIB>, kIB, o);
    else if (left <= 6 * kPanelThreads)
      groups(k_outer_panel<T, 6, 4, 0, kGroups>, k_cross<T, 4>, 4, o);
    else groups(k_outer_panel<T, kMany, 4, 0, kGroups>, k_cross<T, 4>, 4, o);
  };
  for (int h = 0; h < 2; ++h) {
    const int o = kNB * h;
    if (o >= left) break;
    quarter(o);
    cross(k_cross<T, 32>, o, o + 32, 1);
    if (o + 32 < left) quarter(o + 32);
    cross(k_cross<T, 32>, o + 32, o, 1);
    cross(k_cross<T, kNB>, o, kNB - o, 2);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t gje_gather(const cplx<T>* x, cplx<T>* bbuf, const int* piv,
                      const MatDesc* d, int nmat, int S, hipStream_t st) {
  if (nmat <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather<T>, dim3(kNBO, nmat), dim3(256), 0, st, x, bbuf,
                     piv, d, S);
  return hipGetLastError();
}

template <typename T>
hipError_t gje_fix(cplx<T>* x, const cplx<T>* bbuf, const int* piv,
                   const MatDesc* d, int nmat, int S, hipStream_t st) {
  if (nmat <= 0 || S <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fix<T>, dim3(S * kNBO / 64, nmat), dim3(512), 0, st, x,
                     bbuf, piv, d, S);
  return hipGetLastError();
}

template <typename T>
hipError_t gje_update(cplx<T>* x, const cplx<T>* bbuf, const int* rowcol,
                      const MatDesc* d, const TileItem* items, int nitems,
                      int variant, hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  // one workgroup per item (a persistent grid of two workgroups per CU
  // measured 4% slower: the dispatcher already overlaps the tiles' prologues)
  const int grid = 8 * ((nitems + 7) / 8);
  if (variant == 1)
    hipLaunchKernelGGL((k_update<T, 4>), dim3(grid), dim3(512), 0, st, x, bbuf,
                       rowcol, d, items, nitems);
  else
    hipLaunchKernelGGL((k_update<T, 2>), dim3(grid), dim3(256), 0, st, x, bbuf,
                       rowcol, d, items, nitems);
  return hipGetLastError();
}

#define FK_INST(T)                                                            \
  template hipError_t gje_panel<T>(cplx<T>*, int*, int*, const MatDesc*, int, \
                                   int, int, int*, cplx<T>*, hipStream_t,     \
                                   int*);                                     \
  template hipError_t gje_gather<T>(const cplx<T>*, cplx<T>*, const int*,     \
                                    const MatDesc*, int, int, hipStream_t);   \
  template hipError_t gje_fix<T>(cplx<T>*, const cplx<T>*, const int*,       \
                                 const MatDesc*, int, int, hipStream_t);      \
  template hipError_t gje_update<T>(cplx<T>*, const cplx<T>*, const int*,     \
                                    const MatDesc*, const TileItem*, int, int, \
                                    hipStream_t);
FK_INST(double)
FK_INST(float)

}  // namespace fk
