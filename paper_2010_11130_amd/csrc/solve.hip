// air_solve / air_solve_adjoint: FGMRES(m) with right preconditioning by one
// lAIR V-cycle (Section 3 coarse-grid correction; Section 4: no
// pre-relaxation, post-relaxation on F points then all points, here F,F,C
// Jacobi sweeps) on the scaled facet system, and the transposed cycle for
// the adjoint.  Also reconstruction and slab coupling.
//
// Sparse kernels: G lanes per CSR row (G chosen from the mean row length),
// partial sums combined with cross-lane shuffles; rows are contiguous, so a
// group reads its row's values and column indices with unit stride.  A
// relaxation sweep on the point set X (F or C) writes a second buffer
// (Jacobi: every update reads the previous iterate) and copies the other
// rows.  The FGMRES orthogonalisation is classical Gram-Schmidt applied
// twice, with multi-vector dot products reduced in a fixed order.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "prof.h"
#include "system.h"

namespace ah {

enum { SP_MV = 0, SP_RES = 1, SP_SWEEP = 2, SP_ADDMV = 3, SP_SWEEP_P = 4, SP_SWEEP_LIST = 5, SP_SWEEP_ORD = 6,
       SP_RESTRICT = 7, SP_SO_P = 8, SP_SO_E = 9, SP_SO_C = 10, SP_SO = 11 };

// MODE SP_MV:      y = A x
// MODE SP_RES:     y = b - A x
// MODE SP_SWEEP:   y_i = x_i + omega (b_i - (A x)_i) / d_i  for cf_i == X (all rows if cf null), else x_i
// MODE SP_ADDMV:   y = b + A x
// MODE SP_SWEEP_P: the sweep applied to the interpolated iterate x = P e,
//                  read on the fly as x_j = e[pc[j]] (0 where pc[j] < 0);
//                  rows outside X get x_i = e[pc[i]]
// MODE SP_SWEEP_LIST: the sweep on the rows listed in pc[0..n) only; other
//                  rows of y are not written
// MODE SP_SWEEP_ORD: SP_SWEEP_LIST on a copy of the listed rows stored in
//                  list order: item ii's entries at rp[ii] .. rp[ii + 1]
// y2 (sweeps, optional): the updated rows are also written there.
// A values may be null (all ones).
template <class TA, class TX, class TY, int G, int MODE>
__global__ __launch_bounds__(256) void k_csr(int64_t n, const int64_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                             const TA* __restrict__ av, const TX* __restrict__ x,
                                             const TY* __restrict__ b, const TY* __restrict__ d,
                                             const int8_t* __restrict__ cf, int X, TY omega, TY* __restrict__ y,
                                             const int32_t* __restrict__ pc, TY* __restrict__ y2) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ii = gid / G;
  const int g = (int)(gid % G);
  if (ii >= n) return;
  constexpr bool LS = MODE == SP_SWEEP_LIST || MODE == SP_SWEEP_ORD;
  const int64_t i = LS ? (int64_t)pc[ii] : ii;
  constexpr bool SW = MODE == SP_SWEEP || MODE == SP_SWEEP_P || LS;
  const bool active = LS || !SW || !cf || cf[i] == X;
  // the listed sweeps load the row's own x, b and d before the gather
  TY xpre = 0, bpre = 0, dpre = 0;
  if (LS) {
    xpre = (TY)x[i];
    bpre = b[i];
    dpre = d[i];
  }
  TY acc = 0;
  if (active) {
    const int64_t kr = MODE == SP_SWEEP_ORD ? ii : i;
    const int64_t k1 = rp[kr + 1];
    int64_t kb = rp[kr] + g;
    if (MODE != SP_SWEEP_P && av) {
      // four independent column / value / x loads in flight per lane
      TY acc1 = 0, acc2 = 0, acc3 = 0;
      for (; kb + 3 * G < k1; kb += 4 * G) {
        const int32_t c0 = ci[kb], c1 = ci[kb + G], c2 = ci[kb + 2 * G], c3 = ci[kb + 3 * G];
        const TY a0 = (TY)av[kb], a1 = (TY)av[kb + G], a2 = (TY)av[kb + 2 * G], a3 = (TY)av[kb + 3 * G];
        acc += a0 * (TY)x[c0];
        acc1 += a1 * (TY)x[c1];
        acc2 += a2 * (TY)x[c2];
        acc3 += a3 * (TY)x[c3];
      }
      if (kb < k1) {
        // the last one to three entries of the lane in one step: the loads
        // are clamped to the row's last entry (no branch between them) and
        // the entries past the row weigh zero
        const int64_t l = k1 - 1;
        const int64_t q1 = kb + G < l ? kb + G : l, q2 = kb + 2 * G < l ? kb + 2 * G : l;
        const int32_t c0 = ci[kb], c1 = ci[q1], c2 = ci[q2];
        TY a0 = (TY)av[kb], a1 = (TY)av[q1], a2 = (TY)av[q2];
        a1 = kb + G < k1 ? a1 : (TY)0;
        a2 = kb + 2 * G < k1 ? a2 : (TY)0;
        acc += a0 * (TY)x[c0];
        acc1 += a1 * (TY)x[c1];
        acc2 += a2 * (TY)x[c2];
        kb = k1;
      }
      acc += (acc1 + acc2) + acc3;
    }
    for (int64_t k = kb; k < k1; k += G) {
      TY a = av ? (TY)av[k] : (TY)1;
      if (MODE == SP_SWEEP_P) {
        const int32_t c = pc[ci[k]];
        acc += c >= 0 ? a * (TY)x[c] : (TY)0;
      } else {
        acc += a * (TY)x[ci[k]];
      }
    }
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, G);
  if (g != 0) return;
  if (MODE == SP_MV) y[i] = acc;
  else if (MODE == SP_RES) y[i] = b[i] - acc;
  else if (MODE == SP_ADDMV) y[i] = b[i] + acc;
  else {
    TY xi;
    if (MODE == SP_SWEEP_P) {
      const int32_t c = pc[i];
      xi = c >= 0 ? (TY)x[c] : (TY)0;
    } else {
      xi = LS ? xpre : (TY)x[i];
    }
    if (active) {
      const TY di = LS ? dpre : d[i];
      const TY bi = LS ? bpre : b[i];
      if (fabs((double)di) >= 1e-30) xi += omega * (bi - acc) / di;
      if (y2) y2[i] = xi;
    }
    y[i] = xi;
  }
}

// Level-0 operator by off-diagonal facet blocks (scaled system: identity
// diagonal blocks).  Scalar row i = R B + m holds, for each of the nb
// off-diagonal blocks of block row R, B contiguous values whose columns are
// B ocol[s] + 0..B-1; one column index serves B values and all B rows of the
// block row, so the row stream is the values alone.  Modes SP_MV, SP_RES and
// SP_SWEEP_LIST as in k_csr, with d_i = 1; SP_SWEEP_ORD: SP_SWEEP_LIST with
// item ii's values at soff[ii] of a copy of the listed rows in list order.
// SP_SO and SP_SO_P, SP_SO_E, SP_SO_C (block AIR, even B): the sweeps of
// k_fbb's SP_SWEEP_ORD and of its modes of the same names, by rows: row ii is
// row ii % B of block item ii / B of the copy (list, optr and ocol per item).
// For even B a lane takes two values and two entries of x per load (a row, a
// block and a facet's unknowns all start on an even offset), so the lanes of
// a row read whole lines and half the load instructions are issued: 64^2
// slab, p = 2 (84 MB of values, in the Infinity Cache), all rows: 20.0 us with
// a value per load, 18.7 with two.  At B = 3 a lane takes a whole block.
template <class TA, class TX, class TY, int B, int G, int MODE>
__global__ __launch_bounds__(256) void k_fb(int64_t n, const int64_t* __restrict__ optr,
                                            const int32_t* __restrict__ ocol, const TA* __restrict__ ov,
                                            const TX* __restrict__ x, const TY* __restrict__ b, TY omega,
                                            TY* __restrict__ y, const int32_t* __restrict__ list,
                                            TY* __restrict__ y2, const int64_t* __restrict__ soff,
                                            const TX* __restrict__ xc, const int32_t* __restrict__ own) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ii = gid / G;
  const int g = (int)(gid % G);
  if (ii >= n) return;
  constexpr bool SO = MODE == SP_SO || MODE == SP_SO_P || MODE == SP_SO_E || MODE == SP_SO_C;
  static_assert(!SO || B % 2 == 0, "block items by rows: even B");
  const int64_t kk = SO ? ii / B : 0;
  const int64_t i = SO ? (int64_t)list[kk] * B + (ii - kk * B)
                       : MODE == SP_SWEEP_LIST || MODE == SP_SWEEP_ORD ? (int64_t)list[ii] : ii;
  // the row's own x and b, loaded by every lane ahead of the gather
  TY xi;
  if (MODE == SP_SO_P) {
    const int64_t po = own[kk];
    const TY t = (TY)xc[(po >= 0 ? po : 0) * B + (ii - kk * B)];
    xi = po >= 0 ? t : (TY)0;
  } else {
    xi = (TY)(MODE == SP_SO_E ? x[ii] : MODE == SP_SO_C ? xc[ii] : x[i]);
  }
  const TY bi = MODE == SP_MV ? (TY)0 : b[i];
  const int64_t R = SO ? kk : i / B;
  const int m = SO ? (int)(ii - kk * B) : (int)(i - R * B);
  const int64_t o0 = optr[R];
  const int len = (int)(optr[R + 1] - o0) * B;
  const TA* __restrict__ v = MODE == SP_SWEEP_ORD ? ov + soff[ii] : ov + o0 * (B * B) + (int64_t)m * len;
  const int32_t* __restrict__ cb = ocol + o0;
  TY acc = 0, acc1 = 0, acc2 = 0, acc3 = 0;
  int e = g;
  if constexpr (B % 2 == 0) {
    constexpr int H = B / 2;
    typedef TA TA2 __attribute__((ext_vector_type(2)));
    // x may be the caller's vector, aligned to its values only
    typedef TX TX2 __attribute__((ext_vector_type(2), aligned(sizeof(TX))));
    const TA2* __restrict__ v2 = reinterpret_cast<const TA2*>(v);
    const TX2* __restrict__ x2 = reinterpret_cast<const TX2*>(x);
    const TX2* __restrict__ xc2 = reinterpret_cast<const TX2*>(xc);
    // pair q of the row: entries 2 (q % H) and the next of column block cb[q / H]
    const auto pair = [&](int q) -> TX2 {
      const int64_t J = cb[q / H];
      const int c = q % H;
      if constexpr (MODE == SP_SO_P) {
        const TX2 t = xc2[(J >= 0 ? J : 0) * H + c];   // loaded in every case: no branch before the wait
        return J >= 0 ? t : TX2{0, 0};
      } else if constexpr (MODE == SP_SO_E || MODE == SP_SO_C) {
        const TX2* __restrict__ xs = J >= 0 ? x2 + J * H : xc2 + (~J) * H;
        return xs[c];
      } else {
        return x2[J * H + c];
      }
    };
    const int np = len / 2;
    for (; e + 3 * G < np; e += 4 * G) {
      const TA2 a0 = v2[e], a1 = v2[e + G], a2 = v2[e + 2 * G], a3 = v2[e + 3 * G];
      const TX2 x0 = pair(e), x1 = pair(e + G), y0 = pair(e + 2 * G), y1 = pair(e + 3 * G);
      acc += (TY)a0.x * (TY)x0.x + (TY)a0.y * (TY)x0.y;
      acc1 += (TY)a1.x * (TY)x1.x + (TY)a1.y * (TY)x1.y;
      acc2 += (TY)a2.x * (TY)y0.x + (TY)a2.y * (TY)y0.y;
      acc3 += (TY)a3.x * (TY)y1.x + (TY)a3.y * (TY)y1.y;
    }
    for (; e < np; e += G) {
      const TA2 a0 = v2[e];
      const TX2 x0 = pair(e);
      acc += (TY)a0.x * (TY)x0.x + (TY)a0.y * (TY)x0.y;
    }
  } else {
    const int nb = len / B;
    for (; e + G < nb; e += 2 * G) {
      const int64_t J0 = cb[e], J1 = cb[e + G];
      const TA* __restrict__ v0 = v + e * B;
      const TA* __restrict__ v1 = v0 + G * B;
      TA a0[B], a1[B];
      TX x0[B], x1[B];
#pragma unroll
      for (int c = 0; c < B; ++c) {
        a0[c] = v0[c];
        a1[c] = v1[c];
      }
#pragma unroll
      for (int c = 0; c < B; ++c) {
        x0[c] = x[J0 * B + c];
        x1[c] = x[J1 * B + c];
      }
#pragma unroll
      for (int c = 0; c < B; ++c) acc += (TY)a0[c] * (TY)x0[c];
#pragma unroll
      for (int c = 0; c < B; ++c) acc1 += (TY)a1[c] * (TY)x1[c];
    }
    if (e < nb) {
      const int64_t J = cb[e];
#pragma unroll
      for (int c = 0; c < B; ++c) acc += (TY)v[e * B + c] * (TY)x[J * B + c];
    }
  }
  acc += (acc1 + acc2) + acc3;
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, G);
  if (g != 0) return;
  acc += xi;
  if (MODE == SP_MV) {
    y[i] = acc;
  } else if (MODE == SP_RES) {
    y[i] = bi - acc;
  } else {
    const TY xn = xi + omega * (bi - acc);
    y[MODE == SP_SO_P || MODE == SP_SO_E ? ii : i] = xn;
    if (y2) y2[i] = xn;
  }
}

// A coarse level read by full blocks (every block of block row R, the
// diagonal one included; row m of R at (m nb + s) B + c from the block row's
// value base: voff[R] into the CSR values av where voff[R] >= 0, else ~voff[R]
// into the side array ax): the Jacobi sweep of SP_SWEEP_LIST on the listed
// rows with the diagonal d, as k_csr.  LP lanes per row, a lane per block
// (s = g, g + LP, ...): a lane reads the block's column index, the row's B
// contiguous values of the block and the B contiguous values of x (wide
// loads: a third of the load instructions of a lane per value).  ORD: item
// k's row is described by rec[k] (its values at rec[k].voff of a copy in
// sweep order in av, its blocks from bcol[rec[k].o0]), one load that does
// not wait for the list.  The row's own x, b and d are loaded before the
// gather and a lane takes two blocks per step, so that the loads of a wave
// wait on three latencies rather than one per block; the sum runs in block
// order, as one block at a time would.
template <class TA, class TX, class TY, int B, int LP, bool ORD>
__global__ __launch_bounds__(256) void k_fbr(int64_t n, const int32_t* __restrict__ list,
                                             const int64_t* __restrict__ bptr, const int32_t* __restrict__ bcol,
                                             const int64_t* __restrict__ voff, const AhRowRec* __restrict__ rec,
                                             const TA* __restrict__ av, const TA* __restrict__ ax,
                                             const TX* __restrict__ x, const TY* __restrict__ b,
                                             const TY* __restrict__ d, TY omega, TY* __restrict__ y,
                                             TY* __restrict__ y2) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ii = gid / LP;
  const int g = (int)(gid % LP);
  if (ii >= n) return;
  const int64_t i = list[ii];
  int64_t o0;
  int nb;
  const TA* __restrict__ v;
  if (ORD) {
    const AhRowRec r = rec[ii];
    o0 = r.o0;
    nb = r.nb;
    v = av + r.voff;
  } else {
    const int64_t R = i / B;
    const int m = (int)(i - R * B);
    o0 = bptr[R];
    nb = (int)(bptr[R + 1] - o0);
    const int64_t vo = voff[R];
    v = (vo >= 0 ? av + vo : ax + ~vo) + (int64_t)m * nb * B;
  }
  // every lane loads them (one address per row): no branch for the
  // compiler to wait behind
  TY xi = (TY)x[i];
  const TY bi = b[i], di = d[i];
  const int32_t* __restrict__ cb = bcol + o0;
  TY acc = 0;
  int sl = g;
  for (; sl + LP < nb; sl += 2 * LP) {
    const int64_t J0 = cb[sl], J1 = cb[sl + LP];
    const TA* __restrict__ v0 = v + sl * B;
    const TA* __restrict__ v1 = v0 + LP * B;
    TA a0[B], a1[B];
    TX x0[B], x1[B];
#pragma unroll
    for (int c = 0; c < B; ++c) {
      a0[c] = v0[c];
      a1[c] = v1[c];
    }
#pragma unroll
    for (int c = 0; c < B; ++c) {
      x0[c] = x[J0 * B + c];
      x1[c] = x[J1 * B + c];
    }
#pragma unroll
    for (int c = 0; c < B; ++c) acc += (TY)a0[c] * (TY)x0[c];
#pragma unroll
    for (int c = 0; c < B; ++c) acc += (TY)a1[c] * (TY)x1[c];
  }
  if (sl < nb) {
    const int64_t J = cb[sl];
    const TA* __restrict__ vr = v + sl * B;
#pragma unroll
    for (int c = 0; c < B; ++c) acc += (TY)vr[c] * (TY)x[J * B + c];
  }
#pragma unroll
  for (int o = LP / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, LP);
  if (g != 0) return;
  if (fabs((double)di) >= 1e-30) xi += omega * (bi - acc) / di;
  if (y2) y2[i] = xi;
  y[i] = xi;
}

// The same operator by facet block rows: LPB lanes per block row R, a lane
// per off-diagonal block s of the row (s = g, g + LPB, ...).  A lane reads
// the block's column index once, its B values of x once, and the B x B
// values of the block (row m, column c at (m nb + s) B + c), accumulating
// one sum per row of the block row; the B sums are reduced across the
// lanes and lane m mod LPB writes row R B + m.  Each x value is gathered once for
// the B rows that use it (k_fb gathers it once per row).  Items are block
// rows: all of them (SP_MV, SP_RES), or the blocks of a row list made of
// whole blocks in increasing order (SP_SWEEP_LIST: block k is list[k B] / B),
// or (SP_SWEEP_ORD) the block rows list[k] of a copy of the operator stored
// in that order (item k's blocks at optr[k] .. optr[k + 1]); both sweep.
// SP_RESTRICT: the restriction R = [Z I] of block AIR by coarse blocks k,
// Z's blocks at optr[k] .. optr[k + 1], the identity on the fine block
// list[k B] / B: y[k B + m] = x[R B + m] + (Z x)_m.
// SP_SO_P, SP_SO_E, SP_SO_C: SP_SWEEP_ORD where the iterate is P e_c, or
// P e_c on the C blocks and the F blocks' values on the F blocks, with
// e_c = xc and block one-point P (a copy of coarse blocks), read without
// forming P e_c; the F blocks' values are kept compact, F item k's block at
// k B.  SP_SO_P takes column blocks J >= 0 as coarse blocks of xc (J < 0:
// zero) and the own block from xc at own[k]; SP_SO_E and SP_SO_C take
// J >= 0 as compact F block J of x and J < 0 as coarse block ~J of xc, the
// own block from x at k B (SP_SO_E) or, for the C blocks in coarse order,
// from coarse block k of xc (SP_SO_C).  SP_SO_P and SP_SO_E write y compact
// (y2 at the rows' own places), SP_SO_C writes y at the rows' places.  The
// sums are the ones SP_SWEEP_ORD forms on the interpolated vector.
template <class TA, class TX, class TY, int B, int LPB, int MODE>
__global__ __launch_bounds__(256) void k_fbb(int64_t nbr, const int64_t* __restrict__ optr,
                                             const int32_t* __restrict__ ocol, const TA* __restrict__ ov,
                                             const TX* __restrict__ x, const TY* __restrict__ b, TY omega,
                                             TY* __restrict__ y, const int32_t* __restrict__ list,
                                             TY* __restrict__ y2, const TX* __restrict__ xc,
                                             const int32_t* __restrict__ own) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t kk = gid / LPB;
  const int g = (int)(gid % LPB);
  if (kk >= nbr) return;
  constexpr bool SO = MODE == SP_SO_P || MODE == SP_SO_E || MODE == SP_SO_C;
  const int64_t R = MODE == SP_SWEEP_LIST || MODE == SP_RESTRICT ? (int64_t)list[kk * B] / B
                    : MODE == SP_SWEEP_ORD || SO ? (int64_t)list[kk] : kk;
  const int64_t ko = MODE == SP_SWEEP_ORD || MODE == SP_RESTRICT || SO ? kk : R;
  const int64_t o0 = optr[ko];
  const int nb = (int)(optr[ko + 1] - o0);
  const TA* __restrict__ v = ov + o0 * (B * B);
  // the own block's values: from xc (clamped to coarse block 0 and zeroed
  // where P gives none) or from x
  constexpr bool oc = MODE == SP_SO_P || MODE == SP_SO_C;
  const int64_t po = MODE == SP_SO_P ? (int64_t)own[kk] : MODE == SP_SO_C ? kk : 0;
  const TX* __restrict__ xo = oc ? xc + (int64_t)(po >= 0 ? po : 0) * B : x + (MODE == SP_SO_E ? kk : R) * B;
  const bool oz = oc && po < 0;
  // with a lane per row of the block row, its own x and b are loaded before
  // the gather (their latency overlaps it)
  // (fewer lanes than rows, small blocks: every lane loads all B of them)
  constexpr bool PRE = LPB >= B;
  constexpr bool PALL = !PRE && B <= 4;
  constexpr bool NB = MODE != SP_MV && MODE != SP_RESTRICT;
  TY xpre = 0, bpre = 0;
  TY xall[PALL ? B : 1], ball[PALL ? B : 1];
  if (PRE) {
    const int gp = g < B ? g : B - 1;
    const TY t = (TY)xo[gp];   // loaded in every case: no branch before the wait
    xpre = oz ? (TY)0 : t;
    if (NB) bpre = b[R * B + gp];
  }
  if (PALL) {
#pragma unroll
    for (int m = 0; m < B; ++m) {
      const TY t = (TY)xo[m];
      xall[m] = oz ? (TY)0 : t;
      ball[m] = NB ? b[R * B + m] : (TY)0;
    }
  }
  TY acc[B];
#pragma unroll
  for (int m = 0; m < B; ++m) acc[m] = 0;
  for (int sl = g; sl < nb; sl += LPB) {
    const int64_t J = ocol[o0 + sl];
    TY xv[B];
    if (MODE == SP_SO_P) {
      const TX* __restrict__ xs = xc + (J >= 0 ? J : 0) * B;
#pragma unroll
      for (int c = 0; c < B; ++c) {
        const TY t = (TY)xs[c];   // loaded in every case: no branch before the wait
        xv[c] = J >= 0 ? t : (TY)0;
      }
    } else if (MODE == SP_SO_E || MODE == SP_SO_C) {
      const TX* __restrict__ xs = J >= 0 ? x + J * B : xc + (~J) * B;
#pragma unroll
      for (int c = 0; c < B; ++c) xv[c] = (TY)xs[c];
    } else {
#pragma unroll
      for (int c = 0; c < B; ++c) xv[c] = (TY)x[J * B + c];
    }
#pragma unroll
    for (int m = 0; m < B; ++m) {
      const TA* __restrict__ vr = v + ((int64_t)m * nb + sl) * B;
#pragma unroll
      for (int c = 0; c < B; ++c) acc[m] += (TY)vr[c] * xv[c];
    }
  }
#pragma unroll
  for (int m = 0; m < B; ++m)
#pragma unroll
    for (int o = LPB / 2; o > 0; o >>= 1) acc[m] += __shfl_xor(acc[m], o, LPB);
#pragma unroll
  for (int m = 0; m < B; ++m) {
    if (m % LPB != g) continue;      // lane m mod LPB writes row m
    const int64_t i = R * B + m;
    const TY xi = PRE ? xpre : PALL ? xall[PALL ? m : 0] : oz ? (TY)0 : (TY)xo[m];
    const TY bi = PRE ? bpre : PALL ? ball[PALL ? m : 0] : NB ? b[i] : (TY)0;
    const TY a = acc[m] + xi;
    if (MODE == SP_RESTRICT) {
      y[kk * B + m] = a;
    } else if (MODE == SP_MV) {
      y[i] = a;
    } else if (MODE == SP_RES) {
      y[i] = bi - a;
    } else {
      const TY xn = xi + omega * (bi - a);
      y[MODE == SP_SO_P || MODE == SP_SO_E ? kk * B + m : i] = xn;
      if (y2) y2[i] = xn;
    }
  }
}

// One level of the ordered forward sweep on level 0 (flow order of Lemma
// 3.1): x_i <- b_i - sum of a_ij x_j over the off-diagonal blocks (the
// diagonal blocks are the identity), written to xn.  Blocks of earlier
// levels are read from xn (already swept), blocks of the row's own level
// from xo (values before the level: Jacobi inside a level), later levels
// from xn (still equal to xo).  cols holds ~J for a block J on the row's
// level.  rec: one record per item {item, first value slot of its block row,
// blocks in the row, 0}; BLK: items are blocks and row k is
// rec[k / B].x B + k mod B, otherwise items are rows.
template <class TA, class T, int B, int G, bool BLK>
__global__ __launch_bounds__(256) void k_gs_fb(int64_t n, const int4* __restrict__ rec,
                                               const int32_t* __restrict__ cols, const TA* __restrict__ ov,
                                               const T* __restrict__ b, const T* __restrict__ xo, T* xn) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ii = gid / G;
  const int g = (int)(gid % G);
  if (ii >= n) return;
  const int4 r = rec[BLK ? ii / B : ii];
  const int64_t i = BLK ? (int64_t)r.x * B + ii % B : (int64_t)r.x;
  const int m = (int)(i % B);
  const int64_t o0 = r.y;
  const int len = r.z * B;
  const TA* __restrict__ v = ov + o0 * (B * B) + (int64_t)m * len;
  const int32_t* __restrict__ cb = cols + o0;
  T acc = 0, acc1 = 0;
  int e = g;
  for (; e + G < len; e += 2 * G) {
    const int e1 = e + G;
    const int32_t j0 = cb[e / B], j1 = cb[e1 / B];
    const T* s0 = j0 < 0 ? xo : xn;
    const T* s1 = j1 < 0 ? xo : xn;
    acc += (T)v[e] * s0[(int64_t)(j0 < 0 ? ~j0 : j0) * B + e % B];
    acc1 += (T)v[e1] * s1[(int64_t)(j1 < 0 ? ~j1 : j1) * B + e1 % B];
  }
  if (e < len) {
    const int32_t j0 = cb[e / B];
    acc += (T)v[e] * (j0 < 0 ? xo : xn)[(int64_t)(j0 < 0 ? ~j0 : j0) * B + e % B];
  }
  acc += acc1;
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, G);
  if (g == 0) xn[i] = b[i] - acc;
}

// One level k of the transposed (backward) ordered sweep of the adjoint
// cycle, on the rows of A^T (scalar CSR with its diagonal):
// yn_i = yo_i + (g_i - (A^T y~)_i) / d_i, y~ from yo on the row's own level
// (lev of the column's block == k) and from yn elsewhere.
template <class T, int G, bool BLK>
__global__ __launch_bounds__(256) void k_gs_csr(int64_t n, const int32_t* __restrict__ items, int B,
                                                const int64_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                                const T* __restrict__ v, const T* __restrict__ d,
                                                const T* __restrict__ g, const int32_t* __restrict__ lev, int k,
                                                const T* __restrict__ yo, T* yn) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ii = gid / G;
  const int lane = (int)(gid % G);
  if (ii >= n) return;
  const int64_t i = BLK ? (int64_t)items[ii / B] * B + ii % B : (int64_t)items[ii];
  T acc = 0;
  for (int64_t q = rp[i] + lane; q < rp[i + 1]; q += G) {
    const int32_t j = ci[q];
    acc += v[q] * (lev[j / B] == k ? yo : yn)[j];
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, G);
  if (lane == 0) yn[i] = yo[i] + (g[i] - acc) / d[i];
}

// One level of the coarse end: what the cycle reads, and the lanes per row of
// its sweeps and of the restriction into the next level.
struct EndLevel {
  const int64_t *rp, *Rp;
  const int32_t *ci, *pcol, *Rc;
  const double *v, *d, *Rv;
  const int32_t* list[2];   // its F and its C points
  int n, nc, gA, gR;
};
constexpr int END_LEVELS = 32;
struct EndLevels {
  EndLevel lv[END_LEVELS];
};

// Run f(G) with G the compile-time lane count for the runtime value g.
template <class F>
__device__ inline void end_with_lanes(int g, F&& f) {
  switch (g) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    default: f(std::integral_constant<int, 16>{}); break;
  }
}

// f(i, s) for the rows i = row(0) .. row(n - 1) of a CSR matrix, s the row times
// the NC vectors x (interleaved), in every lane of the row's G lanes; the next
// row's extent is loaded ahead.
template <int END_T, int G, int NC, class Row, class F>
__device__ inline void end_rows(int n, Row&& row, const int64_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                const double* __restrict__ av, const double* x, F&& f) {
  const int g = threadIdx.x % G;
  int ii = threadIdx.x / G;
  int i = ii < n ? row(ii) : 0;
  int k = ii < n ? (int)rp[i] : 0, k1 = ii < n ? (int)rp[i + 1] : 0;
  while (ii < n) {
    const int in = ii + END_T / G, j = in < n ? row(in) : 0;
    const int kn = in < n ? (int)rp[j] : 0, kn1 = in < n ? (int)rp[j + 1] : 0;
    double s[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) s[q] = 0.0;
#pragma unroll 4
    for (k += g; k < k1; k += G) {
      const double v = av[k];
      const double* xc = x + ci[k] * NC;
#pragma unroll
      for (int q = 0; q < NC; ++q) s[q] += v * xc[q];
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1)
#pragma unroll
      for (int q = 0; q < NC; ++q) s[q] += __shfl_xor(s[q], o, G);
    f(i, g, s);
    ii = in;
    i = j;
    k = kn;
    k1 = kn1;
  }
}

// The matrix of the cycle from level 0 of E down: a workgroup applies the
// cycle (restrictions, coarsest inverse, one-point interpolation and Jacobi
// sweeps over the F or C points) to NC columns of the identity, with the vectors
// in LDS and the levels' matrices from L2, and writes its columns of B (and rows
// of B^T).  Runs once per hierarchy; it replaces the same walk in every cycle.
// Bound by the latency of the row loads in the one workgroup that a CU's LDS
// holds, so 16 waves, rows by lists and the next extent ahead: 1956 rows on five
// levels 322 us with 8 waves over all rows, 228 now.  Where the vectors leave room
// for two workgroups, 8 waves each (540 rows: 34 us; 47 with 16).
template <int NC, int END_T>
__global__ __launch_bounds__(END_T) void k_end_cols(EndLevels E, int nlev, const double* __restrict__ cinv, int nsw,
                                                    double omega, double* __restrict__ B, double* __restrict__ Bt) {
  extern __shared__ double sm[];
  const int t = threadIdx.x;
  const int last = nlev - 1;
  const int N = E.lv[0].n;
  const int j0 = blockIdx.x * NC;
  int tot = 0;
  for (int l = 0; l < nlev; ++l) tot += E.lv[l].n;
  double* const bs = sm;                 // right-hand sides, level after level
  double* const ys = sm + tot * NC;      // the level's result
  double* const xs = ys + N * NC;        // the other sweep buffer
  for (int k = t; k < N * NC; k += END_T) bs[k] = k / NC == j0 + k % NC ? 1.0 : 0.0;
  __syncthreads();
  int at = 0;
  for (int l = 0; l < last; ++l) {
    const EndLevel& L = E.lv[l];
    const int nc = E.lv[l + 1].n;
    const double* b = bs + at * NC;
    double* cb = bs + (at + L.n) * NC;
    end_with_lanes(L.gR, [&](auto GC) {
      constexpr int G = decltype(GC)::value;
      end_rows<END_T, G, NC>(nc, [](int i) { return i; }, L.Rp, L.Rc, L.Rv, b, [&](int i, int g, const double* s) {
        if (g == 0)
#pragma unroll
          for (int q = 0; q < NC; ++q) cb[i * NC + q] = s[q];
      });
    });
    __syncthreads();
    at += L.n;
  }
  {
    const int nL = E.lv[last].n;
    const double* b = bs + at * NC;
    for (int i = t / 8; i < nL; i += END_T / 8) {
      double s[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) s[q] = 0.0;
      for (int j = t % 8; j < nL; j += 8) {
        const double c = cinv[(int64_t)i * nL + j];
#pragma unroll
        for (int q = 0; q < NC; ++q) s[q] += c * b[j * NC + q];
      }
#pragma unroll
      for (int o = 4; o > 0; o >>= 1)
#pragma unroll
        for (int q = 0; q < NC; ++q) s[q] += __shfl_xor(s[q], o, 8);
      if (t % 8 == 0)
#pragma unroll
        for (int q = 0; q < NC; ++q) ys[i * NC + q] = s[q];
    }
    __syncthreads();
  }
  // up: x = P e_c, then the sweeps x -> y (-> x -> y); a sweep's other points
  // are in both buffers already where the sweep before was over the same list
  for (int l = last - 1; l >= 0; --l) {
    const EndLevel& L = E.lv[l];
    at -= L.n;
    const double* b = bs + at * NC;
    double* cur = xs;
    double* dst = ys;
    for (int i = t; i < L.n; i += END_T) {
      const int c = L.pcol[i];
#pragma unroll
      for (int q = 0; q < NC; ++q) cur[i * NC + q] = c >= 0 ? ys[c * NC + q] : 0.0;
    }
    __syncthreads();
    for (int w = 0; w < nsw; ++w) {
      const int X = (nsw == 1 || w < 2) ? 0 : 1;
      const int32_t* mine = L.list[X];
      const int nX = X ? L.nc : L.n - L.nc, nO = L.n - nX;
      if (w != 1)
        for (int ii = t; ii < nO; ii += END_T) {
          const int i = L.list[!X][ii];
#pragma unroll
          for (int q = 0; q < NC; ++q) dst[i * NC + q] = cur[i * NC + q];
        }
      end_with_lanes(L.gA, [&](auto GC) {
        constexpr int G = decltype(GC)::value;
        end_rows<END_T, G, NC>(nX, [&](int ii) { return mine[ii]; }, L.rp, L.ci, L.v, cur,
                        [&](int i, int g, const double* s) {
                          if (g != 0) return;
                          const double d = L.d[i];
#pragma unroll
                          for (int q = 0; q < NC; ++q) {
                            double x = cur[i * NC + q];
                            if (fabs(d) >= 1e-30) x += omega * (b[i * NC + q] - s[q]) / d;
                            dst[i * NC + q] = x;
                          }
                        });
      });
      __syncthreads();
      double* const o = cur;
      cur = dst;
      dst = o;
    }
  }
  for (int k = t; k < N * NC; k += END_T) {
    const int i = k / NC, q = k % NC;
    if (j0 + q < N) {
      B[(int64_t)i * N + j0 + q] = ys[k];
      if (Bt) Bt[(int64_t)(j0 + q) * N + i] = ys[k];
    }
  }
}

// z = B r, a wave per row, FP64 matrix and sums: the coarse end of the cycle
// (or of the transposed one) in one launch.  Latency bound (1209 rows, the
// fifth level of the 64^2 slab at p = 2: 6 us); the walk over those levels
// that it replaces took 35 us per cycle, 20 of them in one workgroup.
template <class T>
__global__ __launch_bounds__(256) void k_end_mv(int n, const double* __restrict__ B, const T* __restrict__ r,
                                                T* __restrict__ z) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= n) return;
  const double* __restrict__ b = B + (int64_t)row * n;
  double acc = 0.0;
#pragma unroll 16
  for (int j = lane; j < n; j += 64) acc += b[j] * (double)r[j];
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) z[row] = (T)acc;
}

// x = y = P e_c (one-point interpolation, both sweep buffers)
template <class T>
__global__ void k_interp2(int64_t n, const int32_t* __restrict__ pcol, const T* __restrict__ ec,
                          T* __restrict__ x, T* __restrict__ y) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int32_t c = pcol[i];
  T v = c >= 0 ? ec[c] : (T)0;
  x[i] = v;
  y[i] = v;
}

// First Jacobi sweep of the transposed cycle from y = 0 on the points of
// set X (cf == X): y_X = omega g_X / d_X, zero elsewhere, into both buffers.
template <class T>
__global__ void k_sweep_from_zero(int64_t n, const int8_t* __restrict__ cf, int X, const T* __restrict__ g,
                                  const T* __restrict__ d, T omega, T* __restrict__ x, T* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const T v = cf[i] == X && fabs((double)d[i]) >= 1e-30 ? omega * g[i] / d[i] : (T)0;
  x[i] = v;
  y[i] = v;
}

// b = P^T r on the coarse points (four lanes per row; P has a one per fine point
// at most), and where x is given the coarse level's first sweep on it
// (k_sweep_from_zero), which saves that launch.
template <class T>
__global__ __launch_bounds__(256) void k_restrict_pt(int64_t n, const int64_t* __restrict__ ptr,
                                                     const int32_t* __restrict__ col, const T* __restrict__ r,
                                                     T* __restrict__ b, const int8_t* __restrict__ cf, int X,
                                                     const T* __restrict__ d, T omega, T* __restrict__ x,
                                                     T* __restrict__ y) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = gid / 4;
  if (i >= n) return;
  T acc = 0;
  const int64_t k1 = ptr[i + 1];
  for (int64_t k = ptr[i] + (gid & 3); k < k1; k += 4) acc += r[col[k]];
  acc += __shfl_xor(acc, 2, 4);
  acc += __shfl_xor(acc, 1, 4);
  if (gid & 3) return;
  b[i] = acc;
  if (!x) return;
  const T v = cf[i] == X && fabs((double)d[i]) >= 1e-30 ? omega * acc / d[i] : (T)0;
  x[i] = v;
  y[i] = v;
}

static inline int64_t nF0(const AhLevel& L) { return L.n - L.nc; }

template <class TA, class TB>
__global__ void k_cast(int64_t n, const TA* __restrict__ a, TB* __restrict__ b) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (TB)a[i];
}

// partial[v][blk] = sum over the block's rows of V_v . w (v < k), and
// partial[k][blk] = w . w.  Vectors are rows of V with stride ldv.
constexpr int DOT_T = 256;
constexpr int DOT_V = 4;

__global__ __launch_bounds__(DOT_T) void k_multidot(int64_t n, int k, const double* __restrict__ V, int64_t ldv,
                                                    const double* __restrict__ w, double* __restrict__ partial,
                                                    int nblk) {
  __shared__ double red[DOT_V][DOT_T / 64];
  const int v0 = blockIdx.y * DOT_V;
  double acc[DOT_V] = {0, 0, 0, 0};
  for (int64_t i = (int64_t)blockIdx.x * DOT_T + threadIdx.x; i < n; i += (int64_t)nblk * DOT_T) {
    double wi = w[i];
#pragma unroll
    for (int q = 0; q < DOT_V; ++q) {
      int v = v0 + q;
      if (v < k) acc[q] += V[(int64_t)v * ldv + i] * wi;
      else if (v == k) acc[q] += wi * wi;
    }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < DOT_V; ++q) {
    double a = acc[q];
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if (lane == 0) red[q][wv] = a;
  }
  __syncthreads();
  if (threadIdx.x < DOT_V) {
    int v = v0 + threadIdx.x;
    if (v <= k) {
      double s = 0.0;
      for (int q = 0; q < DOT_T / 64; ++q) s += red[threadIdx.x][q];
      partial[(int64_t)v * nblk + blockIdx.x] = s;
    }
  }
}

__global__ __launch_bounds__(256) void k_reduce_partial(int nblk, const double* __restrict__ partial,
                                                        double* __restrict__ out, int accumulate) {
  __shared__ double red[256];
  const int v = blockIdx.x;
  double s = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 256) s += partial[(int64_t)v * nblk + b];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[v] = accumulate ? out[v] + red[0] : red[0];
}

// ---- CGS2 below 2^21 unknowns, five launches per iteration: dots, update,
// dots, update with the norm, and k_cgs_finish, which normalises w into the
// next basis vector and hands the scalars to the host.  The basis (2.7 MB per
// vector on the 64^2 slab at p = 2) stays in the Infinity Cache, so the passes
// are bound by how many loads are in flight, not by HBM: each thread of the dot
// pass has two rows of eight vectors and w under way, each of the update pass
// two rows of eight vectors.  At 16 vectors there: dots 15.0 us with one row of
// four vectors in flight and 335 partials per dot, 12.0 now; update 19 to
// 21 us, 13.0 now.
constexpr int CGS_T = 512;      // threads per block of the dot pass
constexpr int CGS_B = 128;      // most row blocks of the dot pass: partials per dot
constexpr int CGS_V = 8;        // vectors per block of the dot pass
constexpr int CGS_UB = 512;     // most blocks of the update pass: partials of the norm
constexpr int CGS_ONE_R = 2;    // most rows per thread of the one-workgroup step
constexpr int CGS_ONE_K = 15;   // and most vectors

// The eight sums of a wave together (each exchange halves what a lane carries):
// lanes 8 q .. 8 q + 7 return the wave's sum of acc[q].
__device__ inline double cgs_wave_sums(double (&acc)[CGS_V]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int h = CGS_V / 2; h >= 1; h >>= 1) {
    const bool up = lane & (8 * h);
#pragma unroll
    for (int q = 0; q < h; ++q) {
      const double keep = up ? acc[q + h] : acc[q], send = up ? acc[q] : acc[q + h];
      acc[q] = keep + __shfl_xor(send, 8 * h, 64);
    }
  }
  for (int o = 4; o > 0; o >>= 1) acc[0] += __shfl_xor(acc[0], o, 64);
  return acc[0];
}

// partial[v][blk] = V_v . w over the block's rows (v < k), w . w at v = k.
__global__ __launch_bounds__(CGS_T) void k_cgs_dot(int64_t n, int k, const double* __restrict__ V, int64_t ldv,
                                                  const double* __restrict__ w, double* __restrict__ partial) {
  __shared__ double red[CGS_T / 64][CGS_V];
  const int v0 = blockIdx.y * CGS_V;
  const double* p[CGS_V];
#pragma unroll
  for (int q = 0; q < CGS_V; ++q) p[q] = v0 + q < k ? V + (int64_t)(v0 + q) * ldv : w;
  double acc[CGS_V];
#pragma unroll
  for (int q = 0; q < CGS_V; ++q) acc[q] = 0.0;
  const int64_t st = (int64_t)gridDim.x * CGS_T;
  for (int64_t i = (int64_t)blockIdx.x * CGS_T + threadIdx.x; i < n; i += 2 * st) {
    const int64_t i2 = i + st < n ? i + st : i;
    const double w0 = w[i], w1 = i + st < n ? w[i2] : 0.0;
    double a0[CGS_V], a1[CGS_V];
#pragma unroll
    for (int q = 0; q < CGS_V; ++q) {
      a0[q] = p[q][i];
      a1[q] = p[q][i2];
    }
#pragma unroll
    for (int q = 0; q < CGS_V; ++q) acc[q] += a0[q] * w0 + a1[q] * w1;
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double sum = cgs_wave_sums(acc);
  if ((lane & 7) == 0) red[wv][lane >> 3] = sum;
  __syncthreads();
  const int t = threadIdx.x;
  if (t < CGS_V && v0 + t <= k) {
    double x = 0.0;
#pragma unroll
    for (int q = 0; q < CGS_T / 64; ++q) x += red[q][t];
    partial[(int64_t)(v0 + t) * gridDim.x + blockIdx.x] = x;
  }
}

// h = the dots' sums over their nb <= CGS_B partials (every block, fixed
// order), w -= sum_{v<k} V_v h_v; block 0 stores h[0..k] in hout.  pout (or
// null): partials of the updated w . w per block.  Dynamic LDS: k + 1 doubles.
__global__ __launch_bounds__(256) void k_cgs_update(int64_t n, int k, const double* __restrict__ V, int64_t ldv,
                                                    const double* __restrict__ partial, int nb,
                                                    double* __restrict__ w, double* __restrict__ hout,
                                                    double* __restrict__ pout) {
  extern __shared__ double hs[];
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int v0 = wv * 4; v0 <= k; v0 += 16) {   // a wave sums four dots at a time
    double x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double* pv = partial + (int64_t)min(v0 + q, k) * nb;
      x[q] = 0.0;
#pragma unroll
      for (int u = 0; u < CGS_B; u += 64) x[q] += lane + u < nb ? pv[lane + u] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      for (int o = 32; o > 0; o >>= 1) x[q] += __shfl_xor(x[q], o, 64);
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (v0 + q <= k) hs[v0 + q] = x[q];
  }
  __syncthreads();
  if (blockIdx.x == 0)
    for (int v = threadIdx.x; v <= k; v += 256) hout[v] = hs[v];
  double nrm = 0.0;
  const int64_t st = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += 2 * st) {
    const bool two = i + st < n;
    const int64_t i2 = two ? i + st : i;
    const double w0 = w[i], w1 = w[i2];
    double s0 = 0.0, s1 = 0.0;
    int v = 0;
    for (; v + 8 <= k; v += 8) {
      double a0[8], a1[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double* pv = V + (int64_t)(v + q) * ldv;
        a0[q] = pv[i];
        a1[q] = pv[i2];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        s0 += a0[q] * hs[v + q];
        s1 += a1[q] * hs[v + q];
      }
    }
    if (v < k) {   // the last one to seven in one step: clamped loads of weight zero
      double a0[7], a1[7];
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        const double* pv = V + (int64_t)min(v + q, k - 1) * ldv;
        a0[q] = pv[i];
        a1[q] = pv[i2];
      }
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        const double hq = v + q < k ? hs[v + q] : 0.0;
        s0 += a0[q] * hq;
        s1 += a1[q] * hq;
      }
    }
    const double x0 = w0 - s0, x1 = w1 - s1;
    w[i] = x0;
    nrm += x0 * x0;
    if (two) {
      w[i2] = x1;
      nrm += x1 * x1;
    }
  }
  if (!pout) return;
  for (int o = 32; o > 0; o >>= 1) nrm += __shfl_xor(nrm, o, 64);
  if (lane == 0) red[wv] = nrm;
  __syncthreads();
  if (threadIdx.x == 0) pout[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// A whole step of CGS2 in one workgroup: h1 = V^T w, w -= V h1, h2 = V^T w,
// w -= V h2, out = w / |w|, and the scalars as k_cgs_finish leaves them.  R rows
// per thread, w in registers throughout.  Four passes over V by one CU against five
// dependent launches of about 4 us each.  1,536 unknowns, us per iteration with one
// launch and with five: 32 and 34 to 38 at 4 to 10 vectors, 42 and 37 to 41 at 10 to
// 20, 52 and 38 to 46 at 20 to 28, so up to two batches of eight (w . w is one of
// them); 5,184 unknowns at eight rows per thread: 96 and 66.  Dynamic LDS:
// 17 (k + 1) doubles.
template <int R>
__global__ __launch_bounds__(1024) void k_cgs_one(int64_t n, int k, const double* __restrict__ V, int64_t ldv,
                                                  const double* __restrict__ w, double* __restrict__ out,
                                                  double* __restrict__ hn, double* __restrict__ h1,
                                                  double* __restrict__ h2, int off, double* host,
                                                  unsigned long long* flag, unsigned long long seq) {
  extern __shared__ double hs[];
  constexpr int NW = 16;
  double* red = hs + k + 1;   // [NW][k + 1]
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  unsigned i[R];
  double x[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool in = r * 1024 + t < n;
    i[r] = in ? r * 1024 + t : (unsigned)n - 1;
    x[r] = in ? w[i[r]] : 0.0;
  }
  for (int pass = 0; pass < 2; ++pass) {
    for (int v = 0; v <= k; v += CGS_V) {
      double a[CGS_V][R], acc[CGS_V];
#pragma unroll
      for (int q = 0; q < CGS_V; ++q)
        if (v + q < k) {
          const double* pv = V + (int64_t)(v + q) * ldv;
#pragma unroll
          for (int r = 0; r < R; ++r) a[q][r] = pv[i[r]];
        }
#pragma unroll
      for (int q = 0; q < CGS_V; ++q) {
        acc[q] = 0.0;
        if (v + q <= k)
#pragma unroll
          for (int r = 0; r < R; ++r) acc[q] += (v + q < k ? a[q][r] : x[r]) * x[r];
      }
      const double sum = cgs_wave_sums(acc);
      if ((lane & 7) == 0 && v + (lane >> 3) <= k) red[wv * (k + 1) + v + (lane >> 3)] = sum;
    }
    __syncthreads();
    for (int v = t; v <= k; v += 1024) {
      double h = 0.0;
#pragma unroll
      for (int q = 0; q < NW; ++q) h += red[q * (k + 1) + v];
      hs[v] = h;
      (pass ? h2 : h1)[v] = h;
      if (host) host[pass * off + v] = h;
    }
    __syncthreads();
    double s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = 0.0;
    for (int v = 0; v < k; v += CGS_V) {
      double a[CGS_V][R];
#pragma unroll
      for (int q = 0; q < CGS_V; ++q)
        if (v + q < k) {
          const double* pv = V + (int64_t)(v + q) * ldv;
#pragma unroll
          for (int r = 0; r < R; ++r) a[q][r] = pv[i[r]];
        }
#pragma unroll
      for (int q = 0; q < CGS_V; ++q)
        if (v + q < k)
#pragma unroll
          for (int r = 0; r < R; ++r) s[r] += a[q][r] * hs[v + q];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = r * 1024 + t < n ? x[r] - s[r] : 0.0;
  }
  double nn = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) nn += x[r] * x[r];
  for (int o = 32; o > 0; o >>= 1) nn += __shfl_xor(nn, o, 64);
  if (lane == 0) red[wv] = nn;
  __syncthreads();
  nn = 0.0;
#pragma unroll
  for (int q = 0; q < NW; ++q) nn += red[q];
  const double s = 1.0 / sqrt(nn);
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r * 1024 + t < n) out[i[r]] = x[r] * s;
  if (t <= k || t == 0) __threadfence_system();   // the waves that wrote to the host
  if (t == 0) {
    *hn = nn;
    if (host) host[2 * off] = nn;
  }
  __syncthreads();
  if (host && t == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// out = w / |w| with |w|^2 the sum of the np <= CGS_UB partials (out null: the
// sum alone), and the scalars for the host: |w|^2 to hn, and where the host
// can see device stores (host not null) h1[0..k], h2[0..k] and |w|^2 into its
// buffer at 0, off and 2 off, then seq into flag, which the host polls.
__global__ __launch_bounds__(256) void k_cgs_finish(int64_t n, const double* __restrict__ w,
                                                    const double* __restrict__ part, int np, double* __restrict__ out,
                                                    double* __restrict__ hn, int k, int off,
                                                    const double* __restrict__ h1, const double* __restrict__ h2,
                                                    double* host, unsigned long long* flag, unsigned long long seq) {
  __shared__ double red[4];
  const int t = threadIdx.x;
  double x = 0.0;
#pragma unroll
  for (int u = 0; u < CGS_UB; u += 256) x += t + u < np ? part[t + u] : 0.0;
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  if ((t & 63) == 0) red[t >> 6] = x;
  __syncthreads();
  const double nn = (red[0] + red[1]) + (red[2] + red[3]);
  if (blockIdx.x == 0) {
    if (host) {
      for (int v = t; v <= k; v += 256) {
        host[v] = h1[v];
        host[off + v] = h2[v];
      }
      if (t == 0) host[2 * off] = nn;
      __threadfence_system();
      __syncthreads();
      if (t == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (t == 0) *hn = nn;
  }
  if (!out) return;
  const double s = 1.0 / sqrt(nn);
  for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < n; i += (int64_t)gridDim.x * 256) out[i] = w[i] * s;
}

// Delayed CGS2 (the second projection of each basis vector is done one
// step late, together with the first projection of the next one), dot pass.
// With the j finished basis vectors Q_l = V[l] (l < j), the candidate
// u = V[j] and the new vector w (or none): block partials of Q_l.u at row l,
// Q_l.w at row j + l, then u.u, u.w, w.w at rows 2j, 2j+1, 2j+2.  Blocks
// along y take DD_V basis vectors each; the blocks of y = 0 also form the
// three scalars.
constexpr int DD_V = 8;

__global__ __launch_bounds__(256) void k_dcgs_dot(int64_t n, int j, const double* __restrict__ V,
                                                  const double* __restrict__ w, double* __restrict__ partial,
                                                  int nblk) {
  __shared__ double red[2 * DD_V + 3][4];
  const int l0 = blockIdx.y * DD_V;
  const int nl = min(DD_V, j - l0);
  const double* __restrict__ u = V + (int64_t)j * n;
  const bool first = blockIdx.y == 0;
  double aa[DD_V], cc[DD_V];
#pragma unroll
  for (int q = 0; q < DD_V; ++q) aa[q] = cc[q] = 0.0;
  double su = 0.0, sw = 0.0, ww = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)nblk * 256) {
    const double ui = u[i];
    const double wi = w ? w[i] : 0.0;
#pragma unroll
    for (int q = 0; q < DD_V; ++q)
      if (q < nl) {
        const double qv = V[(int64_t)(l0 + q) * n + i];
        aa[q] += qv * ui;
        cc[q] += qv * wi;
      }
    if (first) {
      su += ui * ui;
      sw += ui * wi;
      ww += wi * wi;
    }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  auto wave_sum = [&](double a) {
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    return a;
  };
#pragma unroll
  for (int q = 0; q < DD_V; ++q) {
    const double a = wave_sum(aa[q]);
    const double c = wave_sum(cc[q]);
    if (lane == 0) { red[q][wv] = a; red[DD_V + q][wv] = c; }
  }
  {
    const double a = wave_sum(su), b = wave_sum(sw), c = wave_sum(ww);
    if (lane == 0) { red[2 * DD_V][wv] = a; red[2 * DD_V + 1][wv] = b; red[2 * DD_V + 2][wv] = c; }
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < 2 * DD_V + 3) {
    const double s = red[t][0] + red[t][1] + red[t][2] + red[t][3];
    int row = -1;
    if (t < DD_V) { if (t < nl) row = l0 + t; }
    else if (t < 2 * DD_V) { if (t - DD_V < nl) row = j + l0 + (t - DD_V); }
    else if (first) row = 2 * j + (t - 2 * DD_V);
    if (row >= 0) partial[(int64_t)row * nblk + blockIdx.x] = s;
  }
}

// cnt device values into pinned host memory, then seq into the flag that the
// host polls; one wave.
__global__ __launch_bounds__(64) void k_hand_over(int cnt, const double* __restrict__ v, double* host,
                                                  unsigned long long* flag, unsigned long long seq) {
  for (int t = threadIdx.x; t < cnt; t += 64) host[t] = v[t];
  __threadfence_system();
  if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Delayed CGS2, update pass: with coef = [a (j), c (j), d, 1/r], the
// finished vector q = (u - Q a) / r is written over u = V[j] and the next
// candidate (w - Q c - q d) / r into V[j+1] (one read of Q for both).  The
// coefficients come with the launch (arg) where they fit, else from coef.
// Dynamic LDS: 2j + 2 doubles.
constexpr int DCGS_ARG = 256;
struct DcgsCoef {
  double c[DCGS_ARG];
};
__global__ __launch_bounds__(256) void k_dcgs_update(int64_t n, int j, double* __restrict__ V,
                                                     const double* __restrict__ w,
                                                     const double* __restrict__ coef, DcgsCoef arg) {
  extern __shared__ double cf[];
  for (int t = threadIdx.x; t < 2 * j + 2; t += blockDim.x) cf[t] = coef ? coef[t] : arg.c[t];
  __syncthreads();
  const double d = cf[2 * j], rinv = cf[2 * j + 1];
  double* __restrict__ u = V + (int64_t)j * n;
  double* __restrict__ un = V + (int64_t)(j + 1) * n;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double sa = 0.0, sc = 0.0;
    for (int l = 0; l < j; ++l) {
      const double qv = V[(int64_t)l * n + i];
      sa += qv * cf[l];
      sc += qv * cf[j + l];
    }
    const double q = (u[i] - sa) * rinv;
    u[i] = q;
    un[i] = (w[i] - sc - q * d) * rinv;
  }
}

// x += sum_v Z_v c_v, the coefficients with the launch.
constexpr int COMB_MAX = 128;
struct CombCoef {
  double c[COMB_MAX];
};
template <class TV>
__global__ __launch_bounds__(256) void k_combine(int64_t n, int k, const TV* __restrict__ Z, int64_t ldz, CombCoef cf,
                                                 double* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
#pragma unroll 8
  for (int v = 0; v < k; ++v) s += (double)Z[(int64_t)v * ldz + i] * cf.c[v];
  x[i] += s;
}

// Block scaling of a right-hand side by D_b^-1 (trans = 0) or D_b^-T.
__global__ void k_blockscale(int64_t nfree, int b, const double* __restrict__ dinv, const double* __restrict__ x,
                             double* __restrict__ y, int trans) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nfree * b) return;
  int64_t R = i / b;
  int m = (int)(i % b);
  double s = 0.0;
  for (int k = 0; k < b; ++k)
    s += (trans ? dinv[R * b * b + k * b + m] : dinv[R * b * b + m * b + k]) * x[R * b + k];
  y[i] = s;
}

static inline dim3 g1(int64_t n, int t = 256) { return dim3((unsigned)cdiv(std::max<int64_t>(n, 1), t)); }

static int pick_g(int64_t nnz, int64_t n) {
  double avg = n ? (double)nnz / (double)n : 0.0;
  if (avg < 24) return 4;
  if (avg < 48) return 8;
  if (avg < 80) return 16;
  return 32;
}

template <class TA, class TX, class TY, int MODE>
static ah_status csr_g(int G, int64_t n, const int64_t* rp, const int32_t* ci, const TA* av, const TX* x, const TY* b,
                       const TY* d, const int8_t* cf, int X, TY omega, TY* y, hipStream_t st,
                       const char* tag = nullptr, double bytes = 0.0, const int32_t* pc = nullptr,
                       TY* y2 = nullptr) {
  if (n == 0) return AH_OK;
  ProfScope ps;
  prof_begin(ps, tag, st, bytes);
  dim3 grid((unsigned)cdiv(n * G, 256));
  switch (G) {
    case 2: hipLaunchKernelGGL((k_csr<TA, TX, TY, 2, MODE>), grid, dim3(256), 0, st, n, rp, ci, av, x, b, d, cf, X, omega, y, pc, y2); break;
    case 4: hipLaunchKernelGGL((k_csr<TA, TX, TY, 4, MODE>), grid, dim3(256), 0, st, n, rp, ci, av, x, b, d, cf, X, omega, y, pc, y2); break;
    case 8: hipLaunchKernelGGL((k_csr<TA, TX, TY, 8, MODE>), grid, dim3(256), 0, st, n, rp, ci, av, x, b, d, cf, X, omega, y, pc, y2); break;
    case 16: hipLaunchKernelGGL((k_csr<TA, TX, TY, 16, MODE>), grid, dim3(256), 0, st, n, rp, ci, av, x, b, d, cf, X, omega, y, pc, y2); break;
    default: hipLaunchKernelGGL((k_csr<TA, TX, TY, 32, MODE>), grid, dim3(256), 0, st, n, rp, ci, av, x, b, d, cf, X, omega, y, pc, y2); break;
  }
  prof_end(ps);
  AH_LAUNCHED();
  return AH_OK;
}

// Lanes per row of k_fb: about eight values per lane (the row is one chain of
// dependent loads per lane, so short rows per lane and more rows per wave keep
// more loads in flight).  B = 3 takes a block per lane and step, so two lanes
// serve a row of six blocks (scalar AIR, 48^3 cube at p = 1: 65.8 ms with two,
// 66.9 with four, 68.4 with eight lanes).
static int fb_lanes(int64_t nvals, int64_t n, int B) {
  const double avg = n ? (double)nvals / (double)n : 0.0;
  if (avg < 12 || (B % 2 && avg < 8 * B)) return 2;
  if (avg < 48) return 4;
  if (avg < 96) return 8;
  return 16;
}

template <class TA, class TX, class TY, int MODE, int B>
static void fb_launch(int G, dim3 grid, hipStream_t st, int64_t n, const int64_t* optr, const int32_t* ocol,
                      const TA* ov, const TX* x, const TY* b, TY omega, TY* y, const int32_t* list, TY* y2,
                      const int64_t* soff, const TX* xc, const int32_t* own) {
#define FB(GG) hipLaunchKernelGGL((k_fb<TA, TX, TY, B, GG, MODE>), grid, dim3(256), 0, st, n, optr, ocol, ov, x, b, \
                                  omega, y, list, y2, soff, xc, own)
  switch (G) {
    case 2: FB(2); break;
    case 4: FB(4); break;
    case 8: FB(8); break;
    default: FB(16); break;
  }
#undef FB
}

// Level-0 rows in the facet-block layout (k_fb): n rows (the listed ones for
// SP_SWEEP_LIST), block size B, G in {2, 4, 8, 16}.
template <class TA, class TX, class TY, int MODE>
static ah_status fb_g(int B, int G, int64_t n, const int64_t* optr, const int32_t* ocol, const TA* ov, const TX* x,
                      const TY* b, TY omega, TY* y, hipStream_t st, const char* tag = nullptr, double bytes = 0.0,
                      const int32_t* list = nullptr, TY* y2 = nullptr, const int64_t* soff = nullptr,
                      const TX* xc = nullptr, const int32_t* own = nullptr) {
  if (n == 0) return AH_OK;
  if (G != 2 && G != 4 && G != 8) G = 16;
  ProfScope ps;
  prof_begin(ps, tag, st, bytes);
  const dim3 grid((unsigned)cdiv(n * G, 256));
  bool done = false;
  const auto go = [&](auto BC) {
    fb_launch<TA, TX, TY, MODE, decltype(BC)::value>(G, grid, st, n, optr, ocol, ov, x, b, omega, y, list, y2, soff,
                                                     xc, own);
    done = true;
  };
  if (B == 2) go(std::integral_constant<int, 2>{});
  if (B == 4) go(std::integral_constant<int, 4>{});
  if (B == 6) go(std::integral_constant<int, 6>{});
  if (B == 10) go(std::integral_constant<int, 10>{});
  if constexpr (MODE != SP_SO && MODE != SP_SO_P && MODE != SP_SO_E && MODE != SP_SO_C)
    if (B == 3) go(std::integral_constant<int, 3>{});
  if (!done) { set_error("unsupported facet block size %d", B); return AH_EUNSUPPORTED; }
  prof_end(ps);
  AH_LAUNCHED();
  return AH_OK;
}

// Sweep of the listed rows of a level read by full blocks (k_fbr); av the
// level's CSR values, ax its side array, in the cycle's precision.  Lanes
// per row: 4 in FP64, 2 in FP32 (C3 level 1, about six blocks per row:
// F sweep 656 / 436 us against 859 / 716 us with 8 lanes; AH_L1LP = 2, 4
// or 8 at setup overrides).
template <class T>
static ah_status fbr_g(const AhLevel& L, const T* av, const T* ax, int64_t n, const int32_t* list, const T* x,
                       const T* b, const T* d, T omega, T* y, hipStream_t st, const char* tag, double bytes,
                       T* y2 = nullptr, const AhRowRec* rec = nullptr) {
  if (n == 0) return AH_OK;
  const int LP = L.blp ? L.blp : sizeof(T) == 8 ? 4 : 2;
  ProfScope ps;
  prof_begin(ps, tag, st, bytes);
  const dim3 grid((unsigned)cdiv(n * LP, 256));
#define FBR(BB, LL)                                                                                         \
  do {                                                                                                      \
    if (rec)                                                                                                \
      hipLaunchKernelGGL((k_fbr<T, T, T, BB, LL, true>), grid, dim3(256), 0, st, n, list, L.bptr, L.bcol,   \
                         (const int64_t*)nullptr, rec, av, ax, x, b, d, omega, y, y2);                      \
    else                                                                                                    \
      hipLaunchKernelGGL((k_fbr<T, T, T, BB, LL, false>), grid, dim3(256), 0, st, n, list, L.bptr, L.bcol,  \
                         L.bvoff, (const AhRowRec*)nullptr, av, ax, x, b, d, omega, y, y2);                 \
  } while (0)
#define FBR_L(BB) switch (LP) { case 2: FBR(BB, 2); break; case 4: FBR(BB, 4); break; default: FBR(BB, 8); break; }
  switch (L.bb) {
    case 2: FBR_L(2); break;
    case 3: FBR_L(3); break;
    case 6: FBR_L(6); break;
    default: prof_end(ps); set_error("unsupported block size %d", L.bb); return AH_EUNSUPPORTED;
  }
#undef FBR_L
#undef FBR
  prof_end(ps);
  AH_LAUNCHED();
  return AH_OK;
}

// Whether the level-0 kernels run by facet block rows (k_fbb): for odd B.  For
// even B the rows' paired loads are faster on every size measured (p = 2: 64^2
// slab SpMV 38.9 -> 18.7 us; mapped 36^3, forward and adjoint, 292 -> 253 ms;
// block AIR on a 32^3 cube 64 -> 50 ms); at B = 3 a row's values cannot be
// paired, and one gather of x for the whole block wins (96^3 SpMV 1.36 -> 1.0 ms).
static bool by_blocks(const ah_hier* h, int B) { return h->fbb && B % 2; }

// Lanes per block row of k_fbb from the mean number of off-diagonal blocks per
// block row (six in 2-D + time: eight lanes).
static int fbb_lanes(int64_t nvals, int64_t n, int B) {
  const double nb = n ? (double)nvals / ((double)n * B) : 0.0;
  if (nb <= 2.0) return 2;
  if (nb <= 4.0) return 4;
  return 8;
}

template <class TA, class TX, class TY, int MODE, int B>
static void fbb_launch(int L, int64_t nbr, hipStream_t st, const int64_t* optr, const int32_t* ocol, const TA* ov,
                       const TX* x, const TY* b, TY omega, TY* y, const int32_t* list, TY* y2, const TX* xc,
                       const int32_t* own) {
#define FBB(LP) hipLaunchKernelGGL((k_fbb<TA, TX, TY, B, LP, MODE>), dim3((unsigned)cdiv(nbr * LP, 256)), dim3(256), 0, \
                                   st, nbr, optr, ocol, ov, x, b, omega, y, list, y2, xc, own)
  switch (L) {
    case 2: FBB(2); break;
    case 4: FBB(4); break;
    default: FBB(8); break;
  }
#undef FBB
}

// k_fbb over n rows (the listed ones for SP_SWEEP_LIST, whole blocks in
// increasing order), block size B, L lanes per block row.
template <class TA, class TX, class TY, int MODE>
static ah_status fbb_g(int B, int L, int64_t n, const int64_t* optr, const int32_t* ocol, const TA* ov, const TX* x,
                       const TY* b, TY omega, TY* y, hipStream_t st, const char* tag = nullptr, double bytes = 0.0,
                       const int32_t* list = nullptr, TY* y2 = nullptr, const TX* xc = nullptr,
                       const int32_t* own = nullptr) {
  if (n == 0) return AH_OK;
  if (n % B) { set_error("block-row sweep over %lld rows, not whole blocks of %d", (long long)n, B); return AH_EINVAL; }
  const int64_t nbr = n / B;
  ProfScope ps;
  prof_begin(ps, tag, st, bytes);
  bool done = false;
  const auto go = [&](auto BC) {
    fbb_launch<TA, TX, TY, MODE, decltype(BC)::value>(L, nbr, st, optr, ocol, ov, x, b, omega, y, list, y2, xc, own);
    done = true;
  };
  if (B == 3) go(std::integral_constant<int, 3>{});
  if constexpr (MODE == SP_RESTRICT) {   // the other modes run by rows for even B
    if (B == 2) go(std::integral_constant<int, 2>{});
    if (B == 4) go(std::integral_constant<int, 4>{});
    if (B == 6) go(std::integral_constant<int, 6>{});
    if (B == 10) go(std::integral_constant<int, 10>{});
  }
  if (!done) { set_error("unsupported facet block size %d", B); return AH_EUNSUPPORTED; }
  prof_end(ps);
  AH_LAUNCHED();
  return AH_OK;
}

// Level-0 kernel over n rows of the facet-block layout: by block rows
// (k_fbb) where the rows are whole blocks (all rows, or block AIR point
// lists), else by rows (k_fb).
template <class T, int MODE>
static ah_status fb_any(const ah_hier* h, const AhLevel& L, bool blocks, int64_t n, const T* ov, const T* x,
                        const T* b, T om, T* y, hipStream_t st, const char* tag = nullptr, double bytes = 0.0,
                        const int32_t* list = nullptr, T* y2 = nullptr) {
  if (blocks && by_blocks(h, L.ob)) {
    const int lp = h->lpb ? h->lpb : fbb_lanes(L.nov, L.n, L.ob);
    return fbb_g<T, T, T, MODE>(L.ob, lp, n, L.optr, L.ocol, ov, x, b, om, y, st, tag, bytes, list, y2);
  }
  const int Gb = h->g0 ? h->g0 : fb_lanes(L.nov, L.n, L.ob);
  return fb_g<T, T, T, MODE>(L.ob, Gb, n, L.optr, L.ocol, ov, x, b, om, y, st, tag, bytes, list, y2);
}

// Algorithmic bytes of a Jacobi sweep on the point set X of level L: the X
// rows of A once, x once, b and d on X, the X updates written.
template <class T>
static double sweep_bytes(const AhLevel& L, int X) {
  const double w = sizeof(T);
  const int64_t nX = X == 0 ? L.nF : L.n - L.nF;
  const int64_t nnzX = X == 0 ? L.nnzF : L.nnz - L.nnzF;
  return (double)nnzX * (w + 4.0) + (double)(nX + 1) * 8.0 + (double)L.n * w + (double)nX * 3.0 * w;
}

// The same for a level-0 sweep in the off-diagonal facet-block layout: the
// X rows' values, every block column index and block-row offset, the list,
// x once, b on X, the X updates written (twice with a second output).
// With xc (the sweeps reading P e_c from e_c): the iterate read once is e_c
// (first F sweep) or x on F and e_c on C, and the first F sweep reads the
// F blocks' coarse blocks under P.
template <class T>
static double fb_sweep_bytes(const AhLevel& L, int X, bool y2, int xc = 0) {
  const double w = sizeof(T);
  const int64_t nX = X == 0 ? L.nF : L.n - L.nF;
  const int64_t nvX = X == 0 ? L.novF : L.nov - L.novF;
  const double xonce = xc == 1 ? (double)L.nc * w : (double)L.n * w;
  const double own = xc == 1 ? (double)(nX / L.ob) * 4.0 : 0.0;
  return (double)nvX * w + (double)(L.nov / (L.ob * L.ob)) * 4.0 + (double)(L.n / L.ob + 1) * 8.0 +
         (double)nX * 4.0 + xonce + own + (double)nX * (y2 ? 3.0 : 2.0) * w;
}

// The same for a sweep of a coarse level read by full blocks: the X rows'
// values, every block column index, the block-row offsets and value bases
// (or, from the copy in sweep order, the X rows' 16-byte records), the list,
// x once, b and d on X, the X updates written (twice with a second output).
template <class T>
static double fbr_sweep_bytes(const AhLevel& L, int X, bool y2) {
  const double w = sizeof(T);
  const int64_t nX = X == 0 ? L.nF : L.n - L.nF;
  const int64_t nvX = X == 0 ? L.nbvF : L.nbv - L.nbvF;
  const double rows = L.bsrec ? (double)nX * 16.0 : (double)(L.n / L.bb) * 16.0 + 8.0;
  return (double)nvX * w + (double)(L.nbv / (L.bb * L.bb)) * 4.0 + rows + (double)nX * 4.0 + (double)L.n * w +
         (double)nX * (y2 ? 4.0 : 3.0) * w;
}

// Algorithmic bytes of the block restriction: Z's values, one column index
// per block, the coarse-block offsets, the fine list, x on the neighbourhood
// blocks and the own blocks once (at most all of x), the coarse vector
// written.
template <class T>
static double rz_bytes(const AhLevel& L) {
  const double w = sizeof(T);
  const int64_t nblk = L.nrz / ((int64_t)L.ob * L.ob);
  return (double)L.nrz * w + (double)nblk * 4.0 + (double)(L.nc / L.ob + 1) * 8.0 + (double)L.nc * 4.0 +
         (double)L.n * w + (double)L.nc * w;
}

// LDS of k_end_cols for the levels from l0 down, per column.
static int64_t end_lds(const ah_hier* h, int l0) {
  int64_t tot = 0;
  for (size_t l = l0; l < h->lev.size(); ++l) tot += h->lev[l].n;
  return (tot + 2 * h->lev[l0].n) * (int64_t)sizeof(double);
}

constexpr int64_t END_LDS_MAX = 160 * 1024;

// The coarse end starts at the first level of at most end_max rows whose
// levels' vectors fit in LDS (an ordered relaxation keeps level 0 out), at the
// latest on the coarsest level.  A dense cycle costs its n^2 values once per
// application, a walk over the levels about 3 us per launch, four or five
// launches each (64^2 slab at p = 2, 17 cycles: 4.47 ms per solve with the end
// at 512 rows, 4.33 at 1535, 4.26 at 2048 (34 MB); 25^3 cube at p = 1 14.6, 14.0
// and 13.6 ms).  Level 0 is taken only up to half as many rows: its matrix has
// to pay for itself within one solve of a few cycles.
void coarse_end_pick(ah_hier* h, int64_t end_max) {
  const int nl = (int)h->lev.size();
  int l = nl > 1 && h->prm.relax >= 2 ? 1 : 0;
  while (l < nl - 1 && (h->lev[l].n > (l == 0 ? end_max / 2 : end_max) || end_lds(h, l) > END_LDS_MAX)) ++l;
  h->end0 = l;
}

__global__ void k_dense_transpose(int n, const double* __restrict__ A, double* __restrict__ At) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < (int64_t)n * n) At[(k % n) * n + k / n] = A[k];
}

// Lanes per row for n rows of mean length avg in a workgroup of nt threads.
static int end_lanes(int64_t n, int64_t nnz, int nt) {
  const int64_t avg = n ? nnz / n : 1;
  int g = 1;
  while (g < 16 && 4 * g < avg) g *= 2;
  while (g < 16 && 2 * g * n <= nt && g < avg) g *= 2;
  return g;
}

ah_status coarse_end_build(ah_hier* h, hipStream_t st) {
  const int nl = (int)h->lev.size(), l0 = h->end0;
  const int64_t n = h->lev[l0].n;
  if (n == 0) return AH_OK;
  double *B = nullptr, *Bt = nullptr;
  if (h->prm.adjoint) AH_TRY(h->arena.get(&Bt, n * n));
  if (l0 == nl - 1) {
    h->end_mat = h->cinv;
    if (Bt) {
      hipLaunchKernelGGL(k_dense_transpose, g1(n * n), dim3(256), 0, st, (int)n, h->cinv, Bt);
      AH_LAUNCHED();
    }
  } else {
    AH_TRY(h->arena.get(&B, n * n));
    const int64_t lds = end_lds(h, l0);
    const int cols = 2 * lds <= END_LDS_MAX ? 2 : 1;
    const int nt = 2 * cols * lds <= END_LDS_MAX ? 512 : 1024;
    EndLevels E{};
    for (int l = l0; l < nl; ++l) {
      const AhLevel& L = h->lev[l];
      EndLevel& e = E.lv[l - l0];
      e.rp = L.rowptr; e.ci = L.col; e.v = L.val; e.d = L.diag; e.pcol = L.pcol;
      e.list[0] = L.flist; e.list[1] = L.clist;
      e.Rp = L.Rptr; e.Rc = L.Rcol; e.Rv = L.Rval;
      e.n = (int)L.n;
      e.nc = (int)L.nc;
      e.gA = end_lanes(L.n, L.nnz, nt);
      e.gR = l + 1 < nl ? end_lanes(L.nc, L.nnzR, nt) : 1;
    }
    const int nsw = h->prm.relax == 1 ? 1 : 3;
    const auto k = cols == 2 ? (nt == 512 ? k_end_cols<2, 512> : k_end_cols<2, 1024>)
                             : (nt == 512 ? k_end_cols<1, 512> : k_end_cols<1, 1024>);
    static std::once_flag once;
    std::call_once(once, [] {
      for (const void* f : {(const void*)k_end_cols<1, 512>, (const void*)k_end_cols<2, 512>,
                            (const void*)k_end_cols<1, 1024>, (const void*)k_end_cols<2, 1024>})
        (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, END_LDS_MAX);
    });
    hipLaunchKernelGGL(k, dim3((unsigned)cdiv(n, cols)), dim3(nt), (unsigned)(cols * lds), st, E, nl - l0, h->cinv,
                       nsw, h->prm.omega, B, Bt);
    AH_LAUNCHED();
    h->end_mat = B;
  }
  h->end_mat_t = Bt;
  return AH_OK;
}

template <class T>
struct Ops;
template <>
struct Ops<double> {
  static const double* A(const AhLevel& L) { return L.val; }
  static const double* AT(const AhLevel& L) { return L.ATval; }
  static const double* R(const AhLevel& L) { return L.Rval; }
  static const double* RT(const AhLevel& L) { return L.RTval; }
  static const double* d(const AhLevel& L) { return L.diag; }
  static const double* O(const AhLevel& L) { return L.oval; }
  static const double* OT(const AhLevel& L) { return L.otval; }
  static const double* BX(const AhLevel& L) { return L.baux; }
  static const double* SO(const AhLevel& L) { return L.soval; }
  static const double* CO(const AhLevel& L) { return L.coval; }
  static const double* RZ(const AhLevel& L) { return L.rzval; }
  static double* b(AhLevel& L) { return L.b; }
  static double* x(AhLevel& L) { return L.x; }
  static double* y(AhLevel& L) { return L.y; }
  static double* e(AhLevel& L) { return L.e; }
};
template <>
struct Ops<float> {
  static const float* A(const AhLevel& L) { return L.val32; }
  static const float* AT(const AhLevel& L) { return L.ATval32; }
  static const float* R(const AhLevel& L) { return L.Rval32; }
  static const float* RT(const AhLevel& L) { return L.RTval32; }
  static const float* d(const AhLevel& L) { return L.diag32; }
  static const float* O(const AhLevel& L) { return L.oval32; }
  static const float* OT(const AhLevel& L) { return L.otval32; }
  static const float* BX(const AhLevel& L) { return L.baux32; }
  static const float* SO(const AhLevel& L) { return L.soval32; }
  static const float* CO(const AhLevel& L) { return L.coval32; }
  static const float* RZ(const AhLevel& L) { return L.rzval32; }
  static float* b(AhLevel& L) { return L.b32; }
  static float* x(AhLevel& L) { return L.x32; }
  static float* y(AhLevel& L) { return L.y32; }
  static float* e(AhLevel& L) { return L.e32; }
};

// Ordered sweeps on level 0 (relax 2: all points; relax 3: F points, then
// all points), one launch per level of the flow order, from xo into xn
// (xn must hold the same values as xo on entry).
template <class TA, class T, int B, int G>
static void gs_fb_level(bool blk, int64_t nrows, const int4* rec, const ah_hier* h, const TA* ov, const T* b,
                        const T* xo, T* xn, hipStream_t st) {
  const dim3 grid((unsigned)cdiv(nrows * G, 256));
  if (blk)
    hipLaunchKernelGGL((k_gs_fb<TA, T, B, G, true>), grid, dim3(256), 0, st, nrows, rec, h->ord_cols, ov, b, xo, xn);
  else
    hipLaunchKernelGGL((k_gs_fb<TA, T, B, G, false>), grid, dim3(256), 0, st, nrows, rec, h->ord_cols, ov, b, xo, xn);
}

template <class T, int B>
static ah_status gs_fb_sweep_b(const ah_hier* h, bool fonly, const T* ov, const T* b, const T* xo, T* xn,
                               hipStream_t st) {
  const AhLevel& L = h->lev[0];
  const int G = fb_lanes(L.nov, L.n, L.ob) <= 4 ? 4 : 8;
  const std::vector<int64_t>& lp = fonly ? h->ord_lptrF : h->ord_lptr;
  const int64_t scale = fonly ? 1 : B;
  const int4* rec = fonly ? h->ord_finfo : h->ord_info;
  for (size_t k = 0; k + 1 < lp.size(); ++k) {
    const int64_t nr = (lp[k + 1] - lp[k]) * scale;
    if (nr == 0) continue;
    if (G == 4)
      gs_fb_level<T, T, B, 4>(!fonly, nr, rec + lp[k], h, ov, b, xo, xn, st);
    else
      gs_fb_level<T, T, B, 8>(!fonly, nr, rec + lp[k], h, ov, b, xo, xn, st);
  }
  AH_LAUNCHED();
  return AH_OK;
}

// Algorithmic bytes of one ordered sweep: the swept rows of A once (values,
// one column index per block, block offsets), x once, b read and the rows
// written, the item lists.
template <class T>
static double gs_sweep_bytes(const AhLevel& L, bool fonly) {
  const double w = sizeof(T);
  const int64_t nX = fonly ? L.nF : L.n;
  const int64_t nvX = fonly ? L.novF : L.nov;
  return (double)nvX * w + (double)(L.nov / (L.ob * L.ob)) * 4.0 + (double)(L.n / L.ob + 1) * 8.0 +
         (double)L.n * w + (double)nX * 2.0 * w + (double)(fonly ? nX : L.n / L.ob) * 4.0;
}

template <class T>
static ah_status gs_fb_sweep(const ah_hier* h, bool fonly, const T* ov, const T* b, const T* xo, T* xn,
                             hipStream_t st) {
  const AhLevel& L = h->lev[0];
  ProfScope ps;
  prof_begin(ps, fonly ? (sizeof(T) == 8 ? "gs0_f" : "gs0_f_f32") : (sizeof(T) == 8 ? "gs0" : "gs0_f32"), st,
             gs_sweep_bytes<T>(L, fonly));
  ah_status rc = AH_OK;
  switch (L.ob) {
    case 2: rc = gs_fb_sweep_b<T, 2>(h, fonly, ov, b, xo, xn, st); break;
    case 3: rc = gs_fb_sweep_b<T, 3>(h, fonly, ov, b, xo, xn, st); break;
    case 4: rc = gs_fb_sweep_b<T, 4>(h, fonly, ov, b, xo, xn, st); break;
    case 6: rc = gs_fb_sweep_b<T, 6>(h, fonly, ov, b, xo, xn, st); break;
    case 10: rc = gs_fb_sweep_b<T, 10>(h, fonly, ov, b, xo, xn, st); break;
    default: set_error("unsupported facet block size %d", L.ob); rc = AH_EUNSUPPORTED;
  }
  prof_end(ps);
  return rc;
}

// Transposed ordered sweep on the rows of A_0^T, levels in reverse order,
// from yo into yn (equal on entry).
template <class T>
static ah_status gs_csr_sweep_t(const ah_hier* h, bool fonly, const T* atv, const T* d, const T* g, const T* yo,
                                T* yn, hipStream_t st) {
  const AhLevel& L = h->lev[0];
  const std::vector<int64_t>& lp = fonly ? h->ord_lptrF : h->ord_lptr;
  const int B = L.ob;
  const int64_t scale = fonly ? 1 : B;
  const int32_t* items = fonly ? h->ord_frows : h->ord;
  if (lp.size() < 2) return AH_OK;
  for (size_t k = lp.size() - 1; k-- > 0;) {
    const int64_t nr = (lp[k + 1] - lp[k]) * scale;
    if (nr == 0) continue;
    const dim3 grid((unsigned)cdiv(nr * 8, 256));
    if (fonly)
      hipLaunchKernelGGL((k_gs_csr<T, 8, false>), grid, dim3(256), 0, st, nr, items + lp[k], B, L.ATptr, L.ATcol,
                         atv, d, g, h->ord_level, (int)k, yo, yn);
    else
      hipLaunchKernelGGL((k_gs_csr<T, 8, true>), grid, dim3(256), 0, st, nr, items + lp[k], B, L.ATptr, L.ATcol,
                         atv, d, g, h->ord_level, (int)k, yo, yn);
  }
  AH_LAUNCHED();
  return AH_OK;
}

// The forward cycle b -> out, in two parts.  The way down restricts b to the
// coarse end and applies it; the way up interpolates and sweeps level after
// level.  A level's correction is its e buffer, level 0's is out, which must
// differ from b and from level 0's sweep buffers x and y (the second F sweep
// writes its rows into out while other rows still read y).
template <class T>
static ah_status end_apply(ah_hier* h, const T* b, T* out, hipStream_t st) {
  const AhLevel& L = h->lev[h->end0];
  if (L.n == 0) return AH_OK;
  hipLaunchKernelGGL(k_end_mv<T>, dim3((unsigned)cdiv(L.n, 4)), dim3(256), 0, st, (int)L.n, h->end_mat, b, out);
  AH_LAUNCHED();
  return AH_OK;
}

// b_{l+1} = R_l b
template <class T>
static ah_status restrict_level(ah_hier* h, int l, const T* b, hipStream_t st) {
  AhLevel& L = h->lev[l];
  AhLevel& C = h->lev[l + 1];
  const int GR = pick_g(L.nnzR, L.nc);
  if (l == 0 && L.rzptr && Ops<T>::RZ(L)) {
    // block AIR: R = [Z I] by coarse blocks
    const int lp = fbb_lanes(L.nrz, L.nc, L.ob);
    AH_TRY((fbb_g<T, T, T, SP_RESTRICT>(L.ob, lp, L.nc, L.rzptr, L.rzcol, Ops<T>::RZ(L), b, (const T*)nullptr, (T)0,
                                        Ops<T>::b(C), st, sizeof(T) == 8 ? "restrict0" : "restrict0_f32",
                                        rz_bytes<T>(L), L.clist)));
  } else {
    AH_TRY((csr_g<T, T, T, SP_MV>(GR, L.nc, L.Rptr, L.Rcol, Ops<T>::R(L), b, (const T*)nullptr, (const T*)nullptr,
                                  (const int8_t*)nullptr, 0, (T)0, Ops<T>::b(C), st)));
  }
  return AH_OK;
}

// out = P e_c, then the level's sweeps
template <class T>
static ah_status relax_level(ah_hier* h, int l, const T* b, const T* ec, T* out, hipStream_t st) {
  AhLevel& L = h->lev[l];
  const int nsw = h->prm.relax == 1 ? 1 : 3;
  const int G = (l == 0 && h->g0) ? h->g0 : (l > 0 && h->gc) ? h->gc : pick_g(L.nnz, L.n);
  const T om = (T)h->prm.omega;
  const int64_t nF = L.n - L.nc;
  if (l > 0 && L.n < h->list_min) {
    // small coarse levels (launch-latency bound): the first F sweep reads
    // P e_c through pcol and writes every row of y (C rows: P e_c); the
    // second F sweep writes every row of x and its F rows into out; the C
    // sweep visits the C points from their list and writes them into out
    if (nsw == 1) {
      AH_TRY((csr_g<T, T, T, SP_SWEEP_P>(G, L.n, L.rowptr, L.col, Ops<T>::A(L), ec, b, Ops<T>::d(L), L.cf, 0, om,
                                         out, st, nullptr, 0.0, L.pcol)));
      return AH_OK;
    }
    T* x = Ops<T>::x(L);
    T* y = Ops<T>::y(L);
    AH_TRY((csr_g<T, T, T, SP_SWEEP_P>(G, L.n, L.rowptr, L.col, Ops<T>::A(L), ec, b, Ops<T>::d(L), L.cf, 0, om, y,
                                       st, nullptr, 0.0, L.pcol)));
    AH_TRY((csr_g<T, T, T, SP_SWEEP>(G, L.n, L.rowptr, L.col, Ops<T>::A(L), y, b, Ops<T>::d(L), L.cf, 0, om, x, st,
                                     nullptr, 0.0, nullptr, out)));
    AH_TRY((csr_g<T, T, T, SP_SWEEP_LIST>(G, L.nc, L.rowptr, L.col, Ops<T>::A(L), x, b, Ops<T>::d(L), L.cf, 1, om,
                                          out, st, nullptr, 0.0, L.clist)));
    return AH_OK;
  }
  // level 0 and large coarse levels (bandwidth bound): x = y = P e_c, then
  // the F sweeps visit the F points only (from the F list) and the C sweep
  // the C points only, so the C entries of x and y keep the interpolated
  // values through the F sweeps: F1 x -> y, F2 y -> x (its rows also written
  // into out), C x -> out.  With one F sweep, y is out.
  if (l == 0 && h->prm.relax >= 2) {
    // ordered sweeps in the flow order: y = out = P e_c; (relax 3: F sweep
    // y -> out, y = out;) sweep over all points y -> out
    T* y = Ops<T>::y(L);
    hipLaunchKernelGGL((k_interp2<T>), g1(L.n), dim3(256), 0, st, L.n, L.pcol, ec, y, out);
    AH_LAUNCHED();
    const T* ov = Ops<T>::O(L);
    if (h->prm.relax == 3) {
      AH_TRY(gs_fb_sweep<T>(h, true, ov, b, y, out, st));
      AH_HIP(hipMemcpyAsync(y, out, L.n * sizeof(T), hipMemcpyDeviceToDevice, st));
    }
    return gs_fb_sweep<T>(h, false, ov, b, y, out, st);
  }
  T* x = Ops<T>::x(L);
  T* y = nsw == 1 ? out : Ops<T>::y(L);
  // block AIR on level 0 with the encoded copy: the sweeps read P e_c from
  // e_c, so P e_c is never formed
  const bool pfree = l == 0 && nsw == 3 && L.sperm && L.soce && Ops<T>::SO(L);
  if (!pfree) {
    hipLaunchKernelGGL((k_interp2<T>), g1(L.n), dim3(256), 0, st, L.n, L.pcol, ec, x, y);
    AH_LAUNCHED();
  }
  // level-0 timing tags, and level 1's where it is read by full blocks
  const bool t1 = l == 1 && L.bb;
  const char* tf = l == 0 ? (sizeof(T) == 8 ? "relax0_f" : "relax0_f_f32")
                   : t1 ? (sizeof(T) == 8 ? "relax1_f" : "relax1_f_f32") : nullptr;
  const char* tc = l == 0 ? (sizeof(T) == 8 ? "relax0_c" : "relax0_c_f32")
                   : t1 ? (sizeof(T) == 8 ? "relax1_c" : "relax1_c_f32") : nullptr;
  if (l == 0 && L.sperm && Ops<T>::SO(L)) {
    // block AIR with the sweep-ordered copy: the F blocks, then the C
    // blocks, each set one contiguous range of block rows
    const T* so = Ops<T>::SO(L);
    const int64_t nbF = nF / L.ob;
    const double bf1 = fb_sweep_bytes<T>(L, 0, false, 1), bf2 = fb_sweep_bytes<T>(L, 0, true, 2);
    const double bc2 = fb_sweep_bytes<T>(L, 1, false, 2);
    if (by_blocks(h, L.ob)) {
      const int lp = h->lpb ? h->lpb : fbb_lanes(L.nov, L.n, L.ob);
      if (pfree) {
        // F1: P e_c -> y; F2: y on F, e_c on C -> x and out; C: x on F, e_c on C -> out
        AH_TRY((fbb_g<T, T, T, SP_SO_P>(L.ob, lp, nF, L.soptr, L.socp, so, ec, b, om, y, st, tf, bf1, L.sperm,
                                        nullptr, ec, L.soown)));
        AH_TRY((fbb_g<T, T, T, SP_SO_E>(L.ob, lp, nF, L.soptr, L.soce, so, y, b, om, x, st, tf, bf2, L.sperm, out, ec,
                                        nullptr)));
        AH_TRY((fbb_g<T, T, T, SP_SO_C>(L.ob, lp, L.nc, L.soptr + nbF, L.soce, so, x, b, om, out, st, tc, bc2,
                                        L.sperm + nbF, nullptr, ec)));
        return AH_OK;
      }
      AH_TRY((fbb_g<T, T, T, SP_SWEEP_ORD>(L.ob, lp, nF, L.soptr, L.socol, so, x, b, om, y, st, tf,
                                           fb_sweep_bytes<T>(L, 0, false), L.sperm)));
      if (nsw == 1) return AH_OK;
      AH_TRY((fbb_g<T, T, T, SP_SWEEP_ORD>(L.ob, lp, nF, L.soptr, L.socol, so, y, b, om, x, st, tf,
                                           fb_sweep_bytes<T>(L, 0, true), L.sperm, out)));
      AH_TRY((fbb_g<T, T, T, SP_SWEEP_ORD>(L.ob, lp, L.nc, L.soptr + nbF, L.socol, so, x, b, om, out, st, tc,
                                           fb_sweep_bytes<T>(L, 1, false), L.sperm + nbF)));
      return AH_OK;
    }
    const int Gb = h->g0 ? h->g0 : fb_lanes(L.nov, L.n, L.ob);
    if (pfree) {
      AH_TRY((fb_g<T, T, T, SP_SO_P>(L.ob, Gb, nF, L.soptr, L.socp, so, ec, b, om, y, st, tf, bf1, L.sperm, nullptr,
                                     nullptr, ec, L.soown)));
      AH_TRY((fb_g<T, T, T, SP_SO_E>(L.ob, Gb, nF, L.soptr, L.soce, so, y, b, om, x, st, tf, bf2, L.sperm, out,
                                     nullptr, ec)));
      AH_TRY((fb_g<T, T, T, SP_SO_C>(L.ob, Gb, L.nc, L.soptr + nbF, L.soce, so, x, b, om, out, st, tc, bc2,
                                     L.sperm + nbF, nullptr, nullptr, ec)));
      return AH_OK;
    }
    AH_TRY((fb_g<T, T, T, SP_SO>(L.ob, Gb, nF, L.soptr, L.socol, so, x, b, om, y, st, tf,
                                 fb_sweep_bytes<T>(L, 0, false), L.sperm)));
    if (nsw == 1) return AH_OK;
    AH_TRY((fb_g<T, T, T, SP_SO>(L.ob, Gb, nF, L.soptr, L.socol, so, y, b, om, x, st, tf,
                                 fb_sweep_bytes<T>(L, 0, true), L.sperm, out)));
    AH_TRY((fb_g<T, T, T, SP_SO>(L.ob, Gb, L.nc, L.soptr + nbF, L.socol, so, x, b, om, out, st, tc,
                                 fb_sweep_bytes<T>(L, 1, false), L.sperm + nbF)));
    return AH_OK;
  }
  if (l == 0 && !L.fblk && L.rsoff && Ops<T>::SO(L)) {
    // scalar AIR: the rows' values in sweep order (the F rows, then the C rows)
    const T* so = Ops<T>::SO(L);
    const int Gb = h->g0 ? h->g0 : fb_lanes(L.nov, L.n, L.ob);
    AH_TRY((fb_g<T, T, T, SP_SWEEP_ORD>(L.ob, Gb, nF, L.optr, L.ocol, so, x, b, om, y, st, tf,
                                        fb_sweep_bytes<T>(L, 0, false), L.flist, nullptr, L.rsoff)));
    if (nsw == 1) return AH_OK;
    AH_TRY((fb_g<T, T, T, SP_SWEEP_ORD>(L.ob, Gb, nF, L.optr, L.ocol, so, y, b, om, x, st, tf,
                                        fb_sweep_bytes<T>(L, 0, true), L.flist, out, L.rsoff)));
    AH_TRY((fb_g<T, T, T, SP_SWEEP_ORD>(L.ob, Gb, L.nc, L.optr, L.ocol, so, x, b, om, out, st, tc,
                                        fb_sweep_bytes<T>(L, 1, false), L.clist, nullptr, L.rsoff + nF)));
    return AH_OK;
  }
  if (l == 0 && L.ob && Ops<T>::O(L)) {
    const T* ov = Ops<T>::O(L);
    AH_TRY((fb_any<T, SP_SWEEP_LIST>(h, L, L.fblk, nF, ov, x, b, om, y, st, tf, fb_sweep_bytes<T>(L, 0, false),
                                     L.flist)));
    if (nsw == 1) return AH_OK;
    AH_TRY((fb_any<T, SP_SWEEP_LIST>(h, L, L.fblk, nF, ov, y, b, om, x, st, tf, fb_sweep_bytes<T>(L, 0, true),
                                     L.flist, out)));
    AH_TRY((fb_any<T, SP_SWEEP_LIST>(h, L, L.fblk, L.nc, ov, x, b, om, out, st, tc, fb_sweep_bytes<T>(L, 1, false),
                                     L.clist)));
    return AH_OK;
  }
  if (l > 0 && L.bb && Ops<T>::A(L) && Ops<T>::BX(L)) {
    // level 1 under block AIR: the sweeps read it by full blocks
    const T* av = Ops<T>::A(L);
    const T* ax = Ops<T>::BX(L);
    const T* d = Ops<T>::d(L);
    if (Ops<T>::SO(L) && L.bsrec) {
      // from the copy in sweep order: the F rows, then the C rows
      const T* so = Ops<T>::SO(L);
      AH_TRY(fbr_g<T>(L, so, so, nF, L.flist, x, b, d, om, y, st, tf, fbr_sweep_bytes<T>(L, 0, false), nullptr,
                      L.bsrec));
      if (nsw == 1) return AH_OK;
      AH_TRY(fbr_g<T>(L, so, so, nF, L.flist, y, b, d, om, x, st, tf, fbr_sweep_bytes<T>(L, 0, true), out,
                      L.bsrec));
      AH_TRY(fbr_g<T>(L, so, so, L.nc, L.clist, x, b, d, om, out, st, tc, fbr_sweep_bytes<T>(L, 1, false), nullptr,
                      L.bsrec + nF));
      return AH_OK;
    }
    AH_TRY(fbr_g<T>(L, av, ax, nF, L.flist, x, b, d, om, y, st, tf, fbr_sweep_bytes<T>(L, 0, false)));
    if (nsw == 1) return AH_OK;
    AH_TRY(fbr_g<T>(L, av, ax, nF, L.flist, y, b, d, om, x, st, tf, fbr_sweep_bytes<T>(L, 0, true), out));
    AH_TRY(fbr_g<T>(L, av, ax, L.nc, L.clist, x, b, d, om, out, st, tc, fbr_sweep_bytes<T>(L, 1, false)));
    return AH_OK;
  }
  if (l > 0 && L.coptr && Ops<T>::CO(L)) {
    // the rows' entries in sweep order: the F rows, then the C rows
    const T* co = Ops<T>::CO(L);
    const T* d = Ops<T>::d(L);
    AH_TRY((csr_g<T, T, T, SP_SWEEP_ORD>(G, nF, L.coptr, L.cocol, co, x, b, d, L.cf, 0, om, y, st, tf,
                                         sweep_bytes<T>(L, 0), L.flist)));
    if (nsw == 1) return AH_OK;
    AH_TRY((csr_g<T, T, T, SP_SWEEP_ORD>(G, nF, L.coptr, L.cocol, co, y, b, d, L.cf, 0, om, x, st, tf,
                                         sweep_bytes<T>(L, 0), L.flist, out)));
    AH_TRY((csr_g<T, T, T, SP_SWEEP_ORD>(G, L.nc, L.coptr + nF, L.cocol, co, x, b, d, L.cf, 1, om, out, st, tc,
                                         sweep_bytes<T>(L, 1), L.clist)));
    return AH_OK;
  }
  AH_TRY((csr_g<T, T, T, SP_SWEEP_LIST>(G, nF, L.rowptr, L.col, Ops<T>::A(L), x, b, Ops<T>::d(L), L.cf, 0, om, y,
                                        st, tf, sweep_bytes<T>(L, 0), L.flist)));
  if (nsw == 1) return AH_OK;
  AH_TRY((csr_g<T, T, T, SP_SWEEP_LIST>(G, nF, L.rowptr, L.col, Ops<T>::A(L), y, b, Ops<T>::d(L), L.cf, 0, om, x,
                                        st, tf, sweep_bytes<T>(L, 0), L.flist, out)));
  AH_TRY((csr_g<T, T, T, SP_SWEEP_LIST>(G, L.nc, L.rowptr, L.col, Ops<T>::A(L), x, b, Ops<T>::d(L), L.cf, 1, om,
                                        out, st, tc, sweep_bytes<T>(L, 1), L.clist)));
  return AH_OK;
}

template <class T>
static ah_status vcycle_down(ah_hier* h, const T* b, hipStream_t st) {
  for (int l = 0; l < h->end0; ++l) AH_TRY(restrict_level<T>(h, l, l ? Ops<T>::b(h->lev[l]) : b, st));
  AhLevel& E = h->lev[h->end0];
  return h->end0 ? end_apply<T>(h, Ops<T>::b(E), Ops<T>::e(E), st) : AH_OK;
}

template <class T>
static ah_status vcycle_up(ah_hier* h, const T* b, T* out, hipStream_t st) {
  if (h->end0 == 0) return end_apply<T>(h, b, out, st);
  for (int l = h->end0 - 1; l >= 0; --l)
    AH_TRY(relax_level<T>(h, l, l ? Ops<T>::b(h->lev[l]) : b, Ops<T>::e(h->lev[l + 1]),
                          l ? Ops<T>::e(h->lev[l]) : out, st));
  return AH_OK;
}

// One F sweep of the transposed cycle on level l, from -> to.
template <class T>
static ah_status vcycle_t_fsweep(ah_hier* h, AhLevel& L, int l, const T* from, const T* g, T* to, hipStream_t st) {
  const T om = (T)h->prm.omega;
  if (l == 0 && Ops<T>::OT(L))   // A_0^T by facet blocks
    return fb_any<T, SP_SWEEP_LIST>(h, L, L.fblk, nF0(L), Ops<T>::OT(L), from, g, om, to, st, nullptr, 0.0, L.flist);
  return csr_g<T, T, T, SP_SWEEP_LIST>(pick_g(L.nnz, L.n), nF0(L), L.ATptr, L.ATcol, Ops<T>::AT(L), from, g,
                                       Ops<T>::d(L), L.cf, 0, om, to, st, nullptr, 0.0, L.flist);
}

// The transposed cycle's sweeps up to the first one over the F points on level 0
// (false: an ordered relaxation, or level 0 in the coarse end).  Few launches, as
// they are wasted after the last step of a solve.
static bool vcycle_t_starts(const ah_hier* h) { return h->end0 > 0 && h->prm.relax < 2; }

template <class T>
static ah_status vcycle_t_start(ah_hier* h, const T* g, hipStream_t st) {
  AhLevel& L = h->lev[0];
  const T om = (T)h->prm.omega;
  T* cur = Ops<T>::x(L);
  T* alt = Ops<T>::y(L);
  // the first sweep (C points, or the F points with one sweep) starts from
  // zero, y_X = omega g_X / d_X, written to both buffers; the F sweeps then
  // alternate over the F list
  const int X = h->prm.relax == 1 ? 0 : 1;
  hipLaunchKernelGGL((k_sweep_from_zero<T>), g1(L.n), dim3(256), 0, st, L.n, L.cf, X, g, Ops<T>::d(L), om, cur, alt);
  AH_LAUNCHED();
  return h->prm.relax == 1 ? AH_OK : vcycle_t_fsweep<T>(h, L, 0, cur, g, alt, st);
}

// Transposed cycle on level l: g -> out (out may alias g above the coarse end,
// not the level's x or y).  On level 0 the start (vcycle_t_start) is done, on the
// levels below the first sweep came with the restriction.  The recursion writes
// its result over the coarse level's input (or into x on the first level of the
// coarse end).
template <class T>
static ah_status vcycle_t(ah_hier* h, int l, const T* g, T* out, hipStream_t st) {
  AhLevel& L = h->lev[l];
  if (l == h->end0) {
    if (L.n == 0) return AH_OK;
    hipLaunchKernelGGL(k_end_mv<T>, dim3((unsigned)cdiv(L.n, 4)), dim3(256), 0, st, (int)L.n, h->end_mat_t, g, out);
    AH_LAUNCHED();
    return AH_OK;
  }
  AhLevel& C = h->lev[l + 1];
  const int G = pick_g(L.nnz, L.n);
  const T om = (T)h->prm.omega;
  T* cur = Ops<T>::x(L);
  T* alt = Ops<T>::y(L);
  const bool fbt = l == 0 && h->prm.relax < 2 && Ops<T>::OT(L);
  if (l == 0 && h->prm.relax >= 2) {
    AH_HIP(hipMemsetAsync(cur, 0, L.n * sizeof(T), st));
    // transposed ordered sweeps: all points, then (relax 3) F points
    AH_HIP(hipMemsetAsync(alt, 0, L.n * sizeof(T), st));
    AH_TRY(gs_csr_sweep_t<T>(h, false, Ops<T>::AT(L), Ops<T>::d(L), g, cur, alt, st));
    std::swap(cur, alt);
    if (h->prm.relax == 3) {
      AH_HIP(hipMemcpyAsync(alt, cur, L.n * sizeof(T), hipMemcpyDeviceToDevice, st));
      AH_TRY(gs_csr_sweep_t<T>(h, true, Ops<T>::AT(L), Ops<T>::d(L), g, cur, alt, st));
      std::swap(cur, alt);
    }
  } else if (h->prm.relax != 1) {
    if (l > 0) AH_TRY(vcycle_t_fsweep<T>(h, L, l, cur, g, alt, st));
    AH_TRY(vcycle_t_fsweep<T>(h, L, l, alt, g, cur, st));
  }
  // residual g - A^T y, restricted by P^T
  if (fbt)
    AH_TRY((fb_any<T, SP_RES>(h, L, true, L.n, Ops<T>::OT(L), cur, g, (T)0, alt, st)));
  else
    AH_TRY((csr_g<T, T, T, SP_RES>(G, L.n, L.ATptr, L.ATcol, Ops<T>::AT(L), cur, g, (const T*)nullptr,
                                   (const int8_t*)nullptr, 0, (T)0, alt, st)));
  const bool sweeps = l + 1 < h->end0;
  if (L.nc > 0) {
    hipLaunchKernelGGL(k_restrict_pt<T>, g1(4 * L.nc), dim3(256), 0, st, L.nc, L.PTptr, L.PTcol, alt, Ops<T>::b(C), C.cf,
                       h->prm.relax == 1 ? 0 : 1, Ops<T>::d(C), om, sweeps ? Ops<T>::x(C) : nullptr,
                       sweeps ? Ops<T>::y(C) : nullptr);
    AH_LAUNCHED();
  }
  T* ec = sweeps ? Ops<T>::b(C) : Ops<T>::x(C);
  AH_TRY(vcycle_t<T>(h, l + 1, Ops<T>::b(C), ec, st));
  // out = y + R^T e_c
  const int GR = pick_g(L.nnzR, L.n);
  AH_TRY((csr_g<T, T, T, SP_ADDMV>(GR, L.n, L.RTptr, L.RTcol, Ops<T>::RT(L), ec, cur, (const T*)nullptr,
                                   (const int8_t*)nullptr, 0, (T)0, out, st)));
  return AH_OK;
}

// Preconditioner application on level 0 for the requested precision:
// r (FP64, level-0 scaled space) -> z (FP64) or z32 (FP32).  A caller may
// enqueue the first part (the forward cycle's way down, the transposed one's
// start) ahead of the rest.
static ah_status precond_down(ah_hier* h, const double* r, int precision, int transpose, hipStream_t st) {
  AhLevel& L = h->lev[0];
  if (precision) {
    hipLaunchKernelGGL((k_cast<double, float>), g1(L.n), dim3(256), 0, st, L.n, r, L.b32);
    AH_LAUNCHED();
  }
  if (transpose) {
    if (!vcycle_t_starts(h)) return AH_OK;
    return precision ? vcycle_t_start<float>(h, L.b32, st) : vcycle_t_start<double>(h, r, st);
  }
  return precision ? vcycle_down<float>(h, L.b32, st) : vcycle_down<double>(h, r, st);
}
static ah_status precond_up(ah_hier* h, const double* r, double* z, float* z32, int precision, int transpose,
                            hipStream_t st) {
  const float* r32 = h->lev[0].b32;
  if (transpose) return precision ? vcycle_t<float>(h, 0, r32, z32, st) : vcycle_t<double>(h, 0, r, z, st);
  return precision ? vcycle_up<float>(h, r32, z32, st) : vcycle_up<double>(h, r, z, st);
}
static ah_status precond(ah_hier* h, const double* r, double* z, float* z32, int precision, int transpose,
                         hipStream_t st) {
  AH_TRY(precond_down(h, r, precision, transpose, st));
  return precond_up(h, r, z, z32, precision, transpose, st);
}

// ------------------------------------------------------------ FGMRES
// Workspace of one FGMRES solve: basis V [(m+1)][n], preconditioned vectors
// Z [m][n] (FP64 cycle) or Z32 (FP32 cycle), w, r, the scaled right-hand
// side, the reduction partials [(2m+4)][1024], the device scalars [4 (m+3)]
// and a host staging array of 4 (m+3) doubles for the Hessenberg column.
// air_solve takes it from buffers the hierarchy keeps; air_solve_noalloc
// carves it out of the library's static scratch array.
struct KWork {
  double* V = nullptr;
  double* Z = nullptr;
  float* Z32 = nullptr;
  double* w = nullptr;
  double* r = nullptr;
  double* bhat = nullptr;
  double* partial = nullptr;
  double* hdev = nullptr;
  double* host = nullptr;
  bool polled = false;         // host is pinned: kernels store the scalars and a flag there
};

static ah_status ensure_workspace(ah_hier* h, int m, int precision, hipStream_t st, KWork* W) {
  const int64_t n = h->lev[0].n;
  if (!(h->m_alloc >= m && (precision == 0 ? h->Z != nullptr : h->Z32 != nullptr))) {
    Arena& ar = h->arena;
    ar.stream = st;   // the workspace is allocated on the solving stream
    if (h->m_alloc < m) {
      AH_TRY(ar.get(&h->V, (int64_t)(m + 1) * n));
      AH_TRY(ar.get(&h->w, n));
      AH_TRY(ar.get(&h->r, n));
      AH_TRY(ar.get(&h->bhat, n));
      AH_TRY(ar.get(&h->partial, (int64_t)(2 * m + 4) * 1024));
      AH_TRY(ar.get(&h->hdev, 4 * (m + 3)));
      h->Z = nullptr;
      h->Z32 = nullptr;
      h->m_alloc = m;
    }
    // Z and Z32 hold the full capacity m_alloc (>= m): a later call with a
    // restart up to m_alloc reuses them without a new check
    if (precision == 0 && !h->Z) AH_TRY(ar.get(&h->Z, (int64_t)h->m_alloc * n));
    if (precision == 1 && !h->Z32) AH_TRY(ar.get(&h->Z32, (int64_t)h->m_alloc * n));
  }
  W->V = h->V;
  W->Z = precision == 0 ? h->Z : nullptr;
  W->Z32 = precision == 1 ? h->Z32 : nullptr;
  W->w = h->w;
  W->r = h->r;
  W->bhat = h->bhat;
  W->partial = h->partial;
  W->hdev = h->hdev;
  W->host = pinned_scratch(4 * (m + 3) + 1);
  if (!W->host) { set_error("pinned host allocation failed"); return AH_ENOMEM; }
  W->polled = h->poll;
  return AH_OK;
}

// ---------------------------------------------------------- BiCGSTAB
// Device scalars: [0] rho = r_hat.r, [1] r.r, [2] r_hat.v, [3] v.v,
// [4] s.t, [5] t.t, [6] s.s, [7] r.r after the step, [8] rho_old,
// [9] alpha, [10] omega.
enum { BC_RHO = 0, BC_RV = 2, BC_ST = 4, BC_TT = 5, BC_SS = 6, BC_RR = 7, BC_RHOOLD = 8, BC_ALPHA = 9,
       BC_OMEGA = 10, BC_N = 11 };

// p = r + beta (p - omega v), beta = (rho / rho_old) (alpha / omega)
__global__ void k_bicg_p(int64_t n, const double* __restrict__ r, const double* __restrict__ v,
                         double* __restrict__ p, const double* __restrict__ sc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double beta = (sc[BC_RHO] / sc[BC_RHOOLD]) * (sc[BC_ALPHA] / sc[BC_OMEGA]);
  p[i] = r[i] + beta * (p[i] - sc[BC_OMEGA] * v[i]);
}

// alpha = rho / (r_hat.v), s = r - alpha v, block partial sums of s.s
__global__ __launch_bounds__(256) void k_bicg_s(int64_t n, const double* __restrict__ r,
                                                const double* __restrict__ v, double* __restrict__ s,
                                                double* __restrict__ sc, double* __restrict__ partial, int nblk) {
  __shared__ double red[4];
  const double alpha = sc[BC_RHO] / sc[BC_RV];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)nblk * 256) {
    const double si = r[i] - alpha * v[i];
    s[i] = si;
    acc += si * si;
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    if (blockIdx.x == 0) sc[BC_ALPHA] = alpha;
  }
}

// x += alpha p_hat (the step ended on s)
__global__ void k_bicg_xhalf(int64_t n, const double* __restrict__ ph, double* __restrict__ x,
                             const double* __restrict__ sc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] += sc[BC_ALPHA] * ph[i];
}

// omega = (t.s) / (t.t), x += alpha p_hat + omega s_hat, r = s - omega t,
// block partial sums of r.r; rho_old = rho
__global__ __launch_bounds__(256) void k_bicg_xr(int64_t n, const double* __restrict__ ph,
                                                 const double* __restrict__ sh, const double* __restrict__ s,
                                                 const double* __restrict__ t, double* __restrict__ x,
                                                 double* __restrict__ r, double* __restrict__ sc,
                                                 double* __restrict__ partial, int nblk) {
  __shared__ double red[4];
  const double tt = sc[BC_TT];
  const double omega = tt > 0.0 ? sc[BC_ST] / tt : 0.0;
  const double alpha = sc[BC_ALPHA];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)nblk * 256) {
    x[i] += alpha * ph[i] + omega * sh[i];
    const double ri = s[i] - omega * t[i];
    r[i] = ri;
    acc += ri * ri;
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    if (blockIdx.x == 0) {
      sc[BC_OMEGA] = omega;
      sc[BC_RHOOLD] = sc[BC_RHO];
    }
  }
}

// Blocks of the multi-vector dot kernels (at most 1024, about four rows per
// thread).
static int dot_blocks(int64_t n) { return (int)std::min<int64_t>(1024, std::max<int64_t>(1, cdiv(n, DOT_T * 4))); }

// out[0..k] = V[0..k-1].w and w.w (k vectors plus the norm), on the device.
static ah_status multidot(int64_t n, int k, const double* V, const double* w, double* partial, double* out,
                          hipStream_t st) {
  int nblk = (int)std::min<int64_t>(1024, std::max<int64_t>(1, cdiv(n, DOT_T * 4)));
  dim3 grid(nblk, (unsigned)cdiv(k + 1, DOT_V));
  hipLaunchKernelGGL(k_multidot, grid, dim3(DOT_T), 0, st, n, k, V, n, w, partial, nblk);
  AH_LAUNCHED();
  hipLaunchKernelGGL(k_reduce_partial, dim3(k + 1), dim3(256), 0, st, nblk, partial, out, 0);
  AH_LAUNCHED();
  return AH_OK;
}

// Level-0 operator of a Krylov solve: scalar CSR, and for a scaled system's
// forward operator also the off-diagonal facet-block layout (ob > 0), which
// is then the one applied.
struct Op {
  const int64_t* rp;
  const int32_t* ci;
  const double* v;
  int ob = 0;
  const int64_t* optr = nullptr;
  const int32_t* ocol = nullptr;
  const double* ov = nullptr;
  int64_t nov = 0;
  int lpb = 0;                 // > 0: the facet-block layout by block rows (k_fbb), that many lanes each
};

static int op_lanes(const ah_hier* h, const Op& A, int64_t n) {
  if (h->g0) return h->g0;
  return A.ob ? fb_lanes(A.nov, n, A.ob) : pick_g(h->lev[0].nnz, n);
}

// Algorithmic bytes of y = A x (x of width wx): the operator once, x once,
// y written.
static double op_mv_bytes(const ah_hier* h, const Op& A, int64_t n, double wx) {
  if (A.ob) return (double)A.nov * 8.0 + (double)(A.nov / (A.ob * A.ob)) * 4.0 + (double)(n / A.ob + 1) * 8.0 +
                   (double)n * wx + (double)n * 8.0;
  return (double)h->lev[0].nnz * 12.0 + (double)(n + 1) * 8.0 + (double)n * wx + (double)n * 8.0;
}

// y = A x (SP_MV) or y = b - A x (SP_RES).
template <class TX, int MODE>
static ah_status op_apply(const Op& A, int G, int64_t n, const TX* x, const double* b, double* y, hipStream_t st,
                          const char* tag = nullptr, double bytes = 0.0) {
  if (A.ob && A.lpb)
    return fbb_g<double, TX, double, MODE>(A.ob, A.lpb, n, A.optr, A.ocol, A.ov, x, b, 0.0, y, st, tag, bytes);
  if (A.ob)
    return fb_g<double, TX, double, MODE>(A.ob, G, n, A.optr, A.ocol, A.ov, x, b, 0.0, y, st, tag, bytes);
  return csr_g<double, TX, double, MODE>(G, n, A.rp, A.ci, A.v, x, b, (const double*)nullptr,
                                         (const int8_t*)nullptr, 0, 0.0, y, st, tag, bytes);
}

// x += sum_v Z_v y_v, v < k.
static ah_status combine_add(int k, const double* y, int64_t n, const KWork& W, int precision, double* x,
                             hipStream_t st) {
  for (int v0 = 0; v0 < k; v0 += COMB_MAX) {
    CombCoef cf;
    const int kc = std::min(COMB_MAX, k - v0);
    std::copy(y + v0, y + v0 + kc, cf.c);
    if (precision == 0)
      hipLaunchKernelGGL(k_combine<double>, g1(n), dim3(256), 0, st, n, kc, W.Z + (int64_t)v0 * n, n, cf, x);
    else
      hipLaunchKernelGGL(k_combine<float>, g1(n), dim3(256), 0, st, n, kc, W.Z32 + (int64_t)v0 * n, n, cf, x);
    AH_LAUNCHED();
  }
  return AH_OK;
}

// b = 0: x = 0.  Waits for the stream as every other end of a solve does: the
// host has seen the norm, but the kernel that stored it may still be writing
// the first basis vector, in a workspace that another solve may use next.
static ah_status zero_solution(int64_t n, double* x, hipStream_t st, ah_solve_info* info) {
  AH_HIP(hipMemsetAsync(x, 0, n * sizeof(double), st));
  AH_HIP(hipStreamSynchronize(st));
  if (info) { info->iters = 0; info->converged = 1; info->relres = 0; info->true_relres = 0; }
  return AH_OK;
}

static ah_status fgmres_dcgs2(ah_hier* h, const KWork& W, Op A, const double* bvec, double* x,
                              const ah_solve_params& prm, int transpose, hipStream_t st, ah_solve_info* info);

static ah_status fgmres_cgs2(ah_hier* h, const KWork& W, Op A, const double* bvec, double* x,
                             const ah_solve_params& prm, int transpose, hipStream_t st, ah_solve_info* info);

static ah_status fgmres(ah_hier* h, const KWork& W, Op A, const double* bvec, double* x, const ah_solve_params& prm,
                        int transpose, hipStream_t st, ah_solve_info* info) {
  const ah_status rc = (h->lev[0].n >= h->dcgs_min ? fgmres_dcgs2 : fgmres_cgs2)(h, W, A, bvec, x, prm, transpose, st,
                                                                                 info);
  // launches of a solve that stopped early may still store into its buffers
  if (rc < 0) (void)hipStreamSynchronize(st);
  return rc;
}

static ah_status fgmres_cgs2(ah_hier* h, const KWork& W, Op A, const double* bvec, double* x,
                             const ah_solve_params& prm, int transpose, hipStream_t st, ah_solve_info* info) {
  const int64_t n = h->lev[0].n;
  const int m = std::max(1, prm.restart);
  const int G0 = op_lanes(h, A, n);
  double* hd = W.hdev;
  double* hh = W.host;
  auto t0 = std::chrono::steady_clock::now();
  double* h1 = hd;               // [k+1]: dots, then ||w0||^2 at [k]
  double* h2 = hd + (m + 2);     // [k+1]
  double* hn = hd + 2 * (m + 2); // [1]
  double* pn = W.partial + (int64_t)(m + 2) * CGS_B;   // norm partials, clear of the (k+1) nb dot partials
  const int nb = (int)std::min<int64_t>(CGS_B, std::max<int64_t>(1, cdiv(n, CGS_T)));
  const int nu = (int)std::min<int64_t>(CGS_UB, std::max<int64_t>(1, cdiv(n, 512)));
  // The scalars of a step reach the host through its pinned buffer: the last
  // kernel stores them and then the step's number into a flag, which the host
  // polls.  Without one (polled false) they are copied.
  unsigned long long* flag = reinterpret_cast<unsigned long long*>(hh + 4 * (m + 3));
  unsigned long long seq = 0;
  if (W.polled) __atomic_store_n(flag, 0ull, __ATOMIC_RELEASE);
  auto dots = [&](int k, const double* w) {
    hipLaunchKernelGGL(k_cgs_dot, dim3(nb, (unsigned)cdiv(k + 1, CGS_V)), dim3(CGS_T), 0, st, n, k, W.V, n, w,
                       W.partial);
  };
  auto update = [&](int k, double* hout, double* pout) {
    hipLaunchKernelGGL(k_cgs_update, dim3(nu), dim3(256), (unsigned)((k + 1) * sizeof(double)), st, n, k, W.V, n,
                       W.partial, nb, W.w, hout, pout);
  };
  auto one = [&](int k, double* out) {
    ++seq;
    hipLaunchKernelGGL(n <= 1024 ? k_cgs_one<1> : k_cgs_one<2>, dim3(1), dim3(1024), (unsigned)(17 * (k + 1) * sizeof(double)), st, n, k, W.V, n, W.w, out,
                       hn, h1, h2, m + 2, W.polled ? hh : nullptr, flag, seq);
  };
  auto finish = [&](const double* w, const double* part, int np, double* out, int k) -> ah_status {
    ++seq;
    hipLaunchKernelGGL(k_cgs_finish, dim3(out ? nu : 1), dim3(256), 0, st, n, w, part, np, out, hn, k, m + 2, h1, h2,
                       W.polled ? hh : nullptr, flag, seq);
    AH_LAUNCHED();
    return AH_OK;
  };
  auto wait = [&]() -> ah_status {
    if (!W.polled) {
      AH_HIP(hipMemcpyAsync(hh, hd, (2 * (m + 2) + 1) * sizeof(double), hipMemcpyDeviceToHost, st));
      AH_HIP(hipStreamSynchronize(st));
      return AH_OK;
    }
    return poll_flag(flag, seq, st);
  };
  // ||b||; with x = 0 b is also the first residual
  const bool zero = !prm.x0_given;
  dots(0, bvec);
  AH_TRY(finish(bvec, W.partial, nb, zero ? W.V : nullptr, -1));
  AH_TRY(wait());
  const double bnorm = std::sqrt(hh[2 * (m + 2)]);
  std::vector<double> H((size_t)(m + 1) * m, 0.0), cs(m), sn(m), g(m + 1), y(m);
  int its = 0;
  bool converged = false;
  double relres = 1.0, true_rel = 1.0;
  ah_status status = AH_OK;
  if (!(bnorm > 0.0)) return zero_solution(n, x, st, info);
  if (!std::isfinite(bnorm)) { set_error("air_solve: non-finite right-hand side"); return AH_EBREAKDOWN; }
  for (bool first = true;; first = false) {
    double beta = bnorm;
    if (!first || !zero) {
      // r = b - A x
      AH_TRY((op_apply<double, SP_RES>(A, G0, n, x, bvec, W.r, st)));
      dots(0, W.r);
      AH_TRY(finish(W.r, W.partial, nb, W.V, -1));
      AH_TRY(wait());
      beta = std::sqrt(hh[2 * (m + 2)]);
    }
    true_rel = beta / bnorm;
    relres = true_rel;
    if (!std::isfinite(beta)) { set_error("air_solve: breakdown (NaN residual)"); status = AH_EBREAKDOWN; break; }
    if (beta <= prm.tol * bnorm) { converged = true; break; }
    if (its >= prm.maxit) break;
    std::fill(g.begin(), g.end(), 0.0);
    g[0] = beta;
    int kdone = 0;
    bool down = false;   // the cycle's way down for V[j] is enqueued already
    for (int j = 0; j < m; ++j) {
      double* vj = W.V + (int64_t)j * n;
      double* zj = W.Z ? W.Z + (int64_t)j * n : nullptr;
      float* zj32 = W.Z32 ? W.Z32 + (int64_t)j * n : nullptr;
      if (down)
        AH_TRY(precond_up(h, vj, zj, zj32, prm.precision, transpose, st));
      else
        AH_TRY(precond(h, vj, zj, zj32, prm.precision, transpose, st));
      const double by = op_mv_bytes(h, A, n, prm.precision ? 4.0 : 8.0);
      if (prm.precision == 0)
        AH_TRY((op_apply<double, SP_MV>(A, G0, n, zj, (const double*)nullptr, W.w, st,
                                        transpose ? nullptr : "spmv0", by)));
      else
        AH_TRY((op_apply<float, SP_MV>(A, G0, n, zj32, (const double*)nullptr, W.w, st,
                                       transpose ? nullptr : "spmv0", by)));
      ++its;
      const int k = j + 1;
      double* vk = W.V + (int64_t)k * n;
      if (n <= 1024 * CGS_ONE_R && k <= CGS_ONE_K) {
        one(k, vk);
        AH_LAUNCHED();
      } else {
        dots(k, W.w);
        update(k, h1, nullptr);
        dots(k, W.w);
        update(k, h2, pn);
        AH_TRY(finish(W.w, pn, nu, vk, k));
      }
      // the next cycle's way down runs while the host takes this step's
      // scalars (wasted after the last step of a solve: a few launches)
      down = W.polled && k < m && its < prm.maxit;
      if (down) AH_TRY(precond_down(h, vk, prm.precision, transpose, st));
      AH_TRY(wait());
      const double w0 = std::sqrt(hh[k]);
      const double hnorm = std::sqrt(hh[2 * (m + 2)]);
      if (!std::isfinite(hnorm) || !std::isfinite(w0)) {
        set_error("air_solve: breakdown (NaN in Arnoldi)");
        status = AH_EBREAKDOWN;
        kdone = j;
        break;
      }
      for (int i = 0; i < k; ++i) H[(size_t)i * m + j] = hh[i] + hh[(m + 2) + i];
      H[(size_t)k * m + j] = hnorm;
      for (int i = 0; i < j; ++i) {
        double a = H[(size_t)i * m + j], b = H[(size_t)(i + 1) * m + j];
        H[(size_t)i * m + j] = cs[i] * a + sn[i] * b;
        H[(size_t)(i + 1) * m + j] = -sn[i] * a + cs[i] * b;
      }
      const double a = H[(size_t)j * m + j], bb = H[(size_t)k * m + j];
      const double den = std::hypot(a, bb);
      if (den == 0.0) { cs[j] = 1.0; sn[j] = 0.0; } else { cs[j] = a / den; sn[j] = bb / den; }
      H[(size_t)j * m + j] = cs[j] * a + sn[j] * bb;
      H[(size_t)k * m + j] = 0.0;
      g[k] = -sn[j] * g[j];
      g[j] = cs[j] * g[j];
      kdone = k;
      relres = std::fabs(g[k]) / bnorm;
      const bool happy = hnorm <= 1e-14 * w0;
      if (std::fabs(g[k]) <= prm.tol * bnorm || happy || its >= prm.maxit) break;
    }
    if (status != AH_OK && kdone == 0) break;
    for (int i = kdone - 1; i >= 0; --i) {
      double s = g[i];
      for (int c = i + 1; c < kdone; ++c) s -= H[(size_t)i * m + c] * y[c];
      y[i] = s / H[(size_t)i * m + i];
    }
    AH_TRY(combine_add(kdone, y.data(), n, W, prm.precision, x, st));
    if (status != AH_OK) break;
  }
  AH_HIP(hipStreamSynchronize(st));
  if (info) {
    info->iters = its;
    info->converged = converged ? 1 : 0;
    info->relres = relres;
    info->true_relres = true_rel;
    info->t_solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  if (status != AH_OK) return status;
  return converged ? AH_OK : AH_ENOCONV;
}

// FGMRES with delayed CGS2 orthogonalisation: the basis is read twice per
// iteration instead of four times.  The candidate u_j (w_{j-1} projected
// once, not normalised) is preconditioned and multiplied right away,
// z~_j = M u_j, w_j = A z~_j; one dot pass then gives Q^T u_j, |u_j|^2,
// Q^T w_j and u_j.w_j.  The second projection of u_j finishes it,
// u_j = Q a + r_jj q_j with r_jj = sqrt(|u_j|^2 - |a|^2), and completes
// Hessenberg column j-1 (+a, subdiagonal r_jj).  Since A is linear,
// A z_j = (w_j - A Z a) / r_jj for z_j = (z~_j - Z a) / r_jj, which gives
// column j from the dots and the finished columns, and the next candidate
// u_{j+1} = (w_j - Q c - q_j d) / r_jj, formed in one update pass together
// with q_j.  The solution uses z~ directly: Z~ = Z R with R upper triangular
// (column j = [a; r_jj]), so x += Z~ (R^-1 y).  Convergence of column j-1
// is known one step late, after z~_j and w_j are formed: one extra cycle
// per restart cycle, which is why the plain CGS2 loop is kept for small
// systems.
static ah_status fgmres_dcgs2(ah_hier* h, const KWork& W, Op A, const double* bvec, double* x,
                              const ah_solve_params& prm, int transpose, hipStream_t st, ah_solve_info* info) {
  const int64_t n = h->lev[0].n;
  const int m = std::max(1, prm.restart);
  const int G0 = op_lanes(h, A, n);
  double* hd = W.hdev;
  double* hh = W.host;
  double* coef_d = hd + (2 * m + 3);
  double* coef_h = hh + (2 * m + 3);
  const int nblk = dot_blocks(n);
  auto t0 = std::chrono::steady_clock::now();
  // The sums of a step reach the host through its pinned buffer and a polled
  // flag, the coefficients go back as launch arguments: between the two passes
  // the device waits for one look of the host (3,967,488 unknowns, 34 iterations:
  // 37.6 ms with a copy and a synchronisation each way, 37.1 so).
  unsigned long long* flag = reinterpret_cast<unsigned long long*>(hh + 4 * (m + 3));
  unsigned long long seq = 0;
  if (W.polled) __atomic_store_n(flag, 0ull, __ATOMIC_RELEASE);
  auto fetch = [&](int cnt) -> ah_status {
    if (!W.polled) {
      AH_HIP(hipMemcpyAsync(hh, hd, cnt * sizeof(double), hipMemcpyDeviceToHost, st));
      AH_HIP(hipStreamSynchronize(st));
      return AH_OK;
    }
    hipLaunchKernelGGL(k_hand_over, dim3(1), dim3(64), 0, st, cnt, hd, hh, flag, ++seq);
    AH_LAUNCHED();
    return poll_flag(flag, seq, st);
  };
  AH_TRY(multidot(n, 0, W.V, bvec, W.partial, hd, st));
  AH_TRY(fetch(1));
  const double bnorm = std::sqrt(hh[0]);
  if (!(bnorm > 0.0)) return zero_solution(n, x, st, info);
  if (!std::isfinite(bnorm)) { set_error("air_solve: non-finite right-hand side"); return AH_EBREAKDOWN; }
  // Hr: Hessenberg columns as formed (rows 0..m); Hg: the same after the
  // Givens rotations; Rt: the triangular factor of Z~ = Z R
  std::vector<double> Hr((size_t)(m + 1) * m), Hg((size_t)(m + 1) * m), Rt((size_t)m * m), cs(m), sn(m),
      g(m + 1), y(m), t(m);
  int its = 0;
  bool converged = false;
  double relres = 1.0, true_rel = 1.0;
  ah_status status = AH_OK;
  for (bool first = true;; first = false) {
    // u_0 = r = b - A x, the first candidate (r_00 = ||r||); b where x = 0
    double beta = bnorm;
    if (first && !prm.x0_given) {
      AH_HIP(hipMemcpyAsync(W.V, bvec, n * sizeof(double), hipMemcpyDeviceToDevice, st));
    } else {
      AH_TRY((op_apply<double, SP_RES>(A, G0, n, x, bvec, W.V, st)));
      AH_TRY(multidot(n, 0, W.V, W.V, W.partial, hd, st));
      AH_TRY(fetch(1));
      beta = std::sqrt(hh[0]);
    }
    true_rel = beta / bnorm;
    relres = true_rel;
    if (!std::isfinite(beta)) { set_error("air_solve: breakdown (NaN residual)"); status = AH_EBREAKDOWN; break; }
    if (beta <= prm.tol * bnorm) { converged = true; break; }
    if (its >= prm.maxit) break;
    std::fill(Hr.begin(), Hr.end(), 0.0);
    std::fill(g.begin(), g.end(), 0.0);
    g[0] = beta;
    int kdone = 0;
    double wnorm_prev = 0.0;   // ||A z_{j-1}||, for the breakdown test
    for (int j = 0; j <= m; ++j) {
      double* uj = W.V + (int64_t)j * n;
      const bool more = j < m && its + (j >= 1 ? 1 : 0) < prm.maxit;
      if (more) {
        double* zj = W.Z ? W.Z + (int64_t)j * n : nullptr;
        float* zj32 = W.Z32 ? W.Z32 + (int64_t)j * n : nullptr;
        AH_TRY(precond(h, uj, prm.precision == 0 ? zj : nullptr, prm.precision == 1 ? zj32 : nullptr,
                       prm.precision, transpose, st));
        const double by = op_mv_bytes(h, A, n, prm.precision ? 4.0 : 8.0);
        if (prm.precision == 0)
          AH_TRY((op_apply<double, SP_MV>(A, G0, n, zj, (const double*)nullptr, W.w, st,
                                          transpose ? nullptr : "spmv0", by)));
        else
          AH_TRY((op_apply<float, SP_MV>(A, G0, n, zj32, (const double*)nullptr, W.w, st,
                                         transpose ? nullptr : "spmv0", by)));
      }
      {
        ProfScope ps;
        prof_begin(ps, transpose ? nullptr : "arnoldi_dot", st, (double)(j + 2) * n * 8.0);
        hipLaunchKernelGGL(k_dcgs_dot, dim3(nblk, (unsigned)std::max<int64_t>(1, cdiv(j, DD_V))), dim3(256), 0, st,
                           n, j, W.V, more ? W.w : nullptr, W.partial, nblk);
        prof_end(ps);
        AH_LAUNCHED();
      }
      hipLaunchKernelGGL(k_reduce_partial, dim3(2 * j + 3), dim3(256), 0, st, nblk, W.partial, hd, 0);
      AH_LAUNCHED();
      AH_TRY(fetch(2 * j + 3));
      const double* a = hh;
      const double* c = hh + j;
      const double alpha = hh[2 * j], gamma = hh[2 * j + 1], omega = hh[2 * j + 2];
      double aa = 0.0, ac = 0.0;
      for (int i = 0; i < j; ++i) { aa += a[i] * a[i]; ac += a[i] * c[i]; }
      if (!std::isfinite(alpha) || !std::isfinite(gamma) || !std::isfinite(omega) || !std::isfinite(aa)) {
        set_error("air_solve: breakdown (NaN in Arnoldi)");
        status = AH_EBREAKDOWN;
        break;
      }
      const double rjj = alpha > aa ? std::sqrt(alpha - aa) : 0.0;
      if (j >= 1) {
        // column j-1 is complete: A z_{j-1} = Q (h + a) + r_jj q_j
        const int k = j - 1;
        for (int i = 0; i < j; ++i) Hr[(size_t)i * m + k] += a[i];
        Hr[(size_t)j * m + k] = rjj;
        for (int i = 0; i <= j; ++i) Hg[(size_t)i * m + k] = Hr[(size_t)i * m + k];
        for (int i = 0; i < k; ++i) {
          const double p = Hg[(size_t)i * m + k], q = Hg[(size_t)(i + 1) * m + k];
          Hg[(size_t)i * m + k] = cs[i] * p + sn[i] * q;
          Hg[(size_t)(i + 1) * m + k] = -sn[i] * p + cs[i] * q;
        }
        const double p = Hg[(size_t)k * m + k], q = Hg[(size_t)j * m + k];
        const double den = std::hypot(p, q);
        if (den == 0.0) { cs[k] = 1.0; sn[k] = 0.0; } else { cs[k] = p / den; sn[k] = q / den; }
        Hg[(size_t)k * m + k] = cs[k] * p + sn[k] * q;
        Hg[(size_t)j * m + k] = 0.0;
        g[j] = -sn[k] * g[k];
        g[k] = cs[k] * g[k];
        ++its;
        kdone = j;
        relres = std::fabs(g[j]) / bnorm;
        const bool happy = rjj <= 1e-14 * wnorm_prev;
        if (std::fabs(g[j]) <= prm.tol * bnorm || happy || its >= prm.maxit) break;
      }
      if (!more || !(rjj > 0.0)) break;
      // R column j, then Hessenberg column j as formed (rows 0..j)
      for (int i = 0; i < j; ++i) Rt[(size_t)i * m + j] = a[i];
      Rt[(size_t)j * m + j] = rjj;
      const double d = (gamma - ac) / rjj;
      for (int i = 0; i <= j; ++i) {
        double s = i < j ? c[i] : d;
        for (int l = std::max(0, i - 1); l < j; ++l) s -= Hr[(size_t)i * m + l] * a[l];
        Hr[(size_t)i * m + j] = s / rjj;
      }
      wnorm_prev = std::sqrt(omega) / rjj;
      DcgsCoef arg;
      const bool fits = 2 * j + 2 <= DCGS_ARG;
      double* to = fits ? arg.c : coef_h;
      for (int i = 0; i < j; ++i) { to[i] = a[i]; to[j + i] = c[i]; }
      to[2 * j] = d;
      to[2 * j + 1] = 1.0 / rjj;
      if (!fits) AH_HIP(hipMemcpyAsync(coef_d, coef_h, (2 * j + 2) * sizeof(double), hipMemcpyHostToDevice, st));
      {
        ProfScope ps;
        prof_begin(ps, transpose ? nullptr : "arnoldi_update", st, (double)(j + 4) * n * 8.0);
        hipLaunchKernelGGL(k_dcgs_update, dim3(nblk), dim3(256), (unsigned)((2 * j + 2) * sizeof(double)), st, n, j,
                           W.V, W.w, fits ? nullptr : coef_d, arg);
        prof_end(ps);
        AH_LAUNCHED();
      }
    }
    if (status != AH_OK && kdone == 0) break;
    // y from the rotated Hessenberg, then t = R^-1 y, x += Z~ t
    for (int i = kdone - 1; i >= 0; --i) {
      double s = g[i];
      for (int cc = i + 1; cc < kdone; ++cc) s -= Hg[(size_t)i * m + cc] * y[cc];
      y[i] = s / Hg[(size_t)i * m + i];
    }
    for (int i = kdone - 1; i >= 0; --i) {
      double s = y[i];
      for (int cc = i + 1; cc < kdone; ++cc) s -= Rt[(size_t)i * m + cc] * t[cc];
      t[i] = s / Rt[(size_t)i * m + i];
    }
    AH_TRY(combine_add(kdone, t.data(), n, W, prm.precision, x, st));
    if (status != AH_OK) break;
  }
  AH_HIP(hipStreamSynchronize(st));
  if (info) {
    info->iters = its;
    info->converged = converged ? 1 : 0;
    info->relres = relres;
    info->true_relres = true_rel;
    info->t_solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  if (status != AH_OK) return status;
  return converged ? AH_OK : AH_ENOCONV;
}

// Right-preconditioned BiCGSTAB (the paper's Krylov method, Section 4) on
// A x = b: per step p_hat = M p, v = A p_hat, s = r - alpha v, then
// s_hat = M s, t = A s_hat, x += alpha p_hat + omega s_hat, r = s - omega t.
// The scalars stay on the device; the host reads ||s|| and ||r|| once per
// half step.  Convergence is confirmed by the true residual; a vanishing
// or non-finite rho, r_hat.v or omega restarts from the current iterate.
static ah_status bicgstab(ah_hier* h, Op A, const double* bvec, double* x, const ah_solve_params& prm,
                          int transpose, hipStream_t st, ah_solve_info* info) {
  const int64_t n = h->lev[0].n;
  // workspace: 8 vectors, then 3072 reduction partials (two dots of at most
  // 1024 blocks each), then the BC_N device scalars
  if (!h->bcg) {
    h->arena.stream = st;
    AH_TRY(h->arena.get(&h->bcg, 8 * n + 3072 + 16));
  }
  if (prm.precision == 1 && !h->bcg32) {
    h->arena.stream = st;
    AH_TRY(h->arena.get(&h->bcg32, n));
  }
  double* r = h->bcg;
  double* rh = r + n;
  double* p = rh + n;
  double* v = p + n;
  double* sv = v + n;
  double* tv = sv + n;
  double* ph = tv + n;
  double* sh = ph + n;
  double* part = h->bcg + 8 * n;
  double* sc = part + 3072;
  const int G0 = op_lanes(h, A, n);
  const int nblk = (int)std::min<int64_t>(1024, std::max<int64_t>(1, cdiv(n, 256 * 4)));
  double* hh = pinned_scratch(16);
  if (!hh) { set_error("pinned host allocation failed"); return AH_ENOMEM; }
  auto read_sc = [&](int count) -> ah_status {
    AH_HIP(hipMemcpyAsync(hh, sc, count * sizeof(double), hipMemcpyDeviceToHost, st));
    AH_HIP(hipStreamSynchronize(st));
    return AH_OK;
  };
  auto apply_m = [&](const double* in, double* out) -> ah_status {
    if (prm.precision == 0) return precond(h, in, out, nullptr, 0, transpose, st);
    AH_TRY(precond(h, in, nullptr, h->bcg32, 1, transpose, st));
    hipLaunchKernelGGL((k_cast<float, double>), g1(n), dim3(256), 0, st, n, h->bcg32, out);
    AH_LAUNCHED();
    return AH_OK;
  };
  auto spmv = [&](const double* in, double* out) -> ah_status {
    return op_apply<double, SP_MV>(A, G0, n, in, (const double*)nullptr, out, st, transpose ? nullptr : "spmv0",
                                   op_mv_bytes(h, A, n, 8.0));
  };
  auto t0 = std::chrono::steady_clock::now();
  AH_TRY(multidot(n, 0, rh, bvec, part, sc, st));
  AH_TRY(read_sc(1));
  const double bnorm = std::sqrt(hh[0]);
  int its = 0;
  bool converged = false;
  double relres = 1.0, true_rel = 1.0;
  ah_status status = AH_OK;
  if (!(bnorm > 0.0)) return zero_solution(n, x, st, info);
  if (!std::isfinite(bnorm)) { set_error("air_solve: non-finite right-hand side"); return AH_EBREAKDOWN; }
  const double ones[3] = {1.0, 1.0, 1.0};
  while (true) {
    // (re)start: r = b - A x, r_hat = r, p = v = 0, rho_old = alpha = omega = 1
    AH_TRY((op_apply<double, SP_RES>(A, G0, n, x, bvec, r, st)));
    AH_TRY(multidot(n, 0, rh, r, part, sc + BC_RR, st));
    AH_TRY(read_sc(BC_N));
    true_rel = std::sqrt(hh[BC_RR]) / bnorm;
    relres = true_rel;
    if (!std::isfinite(true_rel)) { set_error("air_solve: breakdown (NaN residual)"); status = AH_EBREAKDOWN; break; }
    if (true_rel <= prm.tol) { converged = true; break; }
    if (its >= prm.maxit) break;
    AH_HIP(hipMemcpyAsync(rh, r, n * sizeof(double), hipMemcpyDeviceToDevice, st));
    AH_HIP(hipMemsetAsync(p, 0, 2 * n * sizeof(double), st));   // p and v
    std::memcpy(hh + 8, ones, sizeof(ones));
    AH_HIP(hipMemcpyAsync(sc + BC_RHOOLD, hh + 8, 3 * sizeof(double), hipMemcpyHostToDevice, st));
    bool restart = false;
    while (its < prm.maxit) {
      AH_TRY(multidot(n, 1, rh, r, part, sc + BC_RHO, st));      // rho, r.r
      hipLaunchKernelGGL(k_bicg_p, g1(n), dim3(256), 0, st, n, r, v, p, sc);
      AH_LAUNCHED();
      AH_TRY(apply_m(p, ph));
      AH_TRY(spmv(ph, v));
      ++its;
      AH_TRY(multidot(n, 1, rh, v, part, sc + BC_RV, st));      // r_hat.v, v.v
      hipLaunchKernelGGL(k_bicg_s, dim3(nblk), dim3(256), 0, st, n, r, v, sv, sc, part, nblk);
      AH_LAUNCHED();
      hipLaunchKernelGGL(k_reduce_partial, dim3(1), dim3(256), 0, st, nblk, part, sc + BC_SS, 0);
      AH_LAUNCHED();
      AH_TRY(read_sc(BC_N));
      const double snorm = std::sqrt(hh[BC_SS]);
      if (!std::isfinite(snorm) || hh[BC_RHO] == 0.0 || hh[BC_RV] == 0.0) { restart = true; break; }
      if (snorm <= prm.tol * bnorm) {
        hipLaunchKernelGGL(k_bicg_xhalf, g1(n), dim3(256), 0, st, n, ph, x, sc);
        AH_LAUNCHED();
        relres = snorm / bnorm;
        break;
      }
      AH_TRY(apply_m(sv, sh));
      AH_TRY(spmv(sh, tv));
      AH_TRY(multidot(n, 1, sv, tv, part, sc + BC_ST, st));     // s.t, t.t
      hipLaunchKernelGGL(k_bicg_xr, dim3(nblk), dim3(256), 0, st, n, ph, sh, sv, tv, x, r, sc, part, nblk);
      AH_LAUNCHED();
      hipLaunchKernelGGL(k_reduce_partial, dim3(1), dim3(256), 0, st, nblk, part, sc + BC_RR, 0);
      AH_LAUNCHED();
      AH_TRY(read_sc(BC_N));
      const double rnorm = std::sqrt(hh[BC_RR]);
      relres = rnorm / bnorm;
      if (!std::isfinite(rnorm)) { restart = true; break; }
      if (rnorm <= prm.tol * bnorm || hh[BC_OMEGA] == 0.0) break;
    }
    (void)restart;   // either way the outer loop recomputes the true residual
  }
  AH_HIP(hipStreamSynchronize(st));
  if (info) {
    info->iters = its;
    info->converged = converged ? 1 : 0;
    info->relres = relres;
    info->true_relres = true_rel;
    info->t_solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  if (status != AH_OK) return status;
  return converged ? AH_OK : AH_ENOCONV;
}

// ------------------------------------------------ allocation-free solve
// The FGMRES workspace of air_solve_noalloc lives in this file-scope device
// array (one copy per GPU, held until the process ends).  In host code the
// name is only a stand-in for the symbol: the device address of each GPU's
// copy comes from hipGetSymbolAddress, looked up once per device with that
// device current, and only that address is passed to kernels.
constexpr size_t kScratchBytes = (size_t)AH_NOALLOC_SCRATCH_BYTES;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

static std::mutex g_scratch_mu;
static std::vector<char*> g_scratch_addr;   // indexed by device id

static ah_status scratch_address(char** out) {
  int dev = 0;
  AH_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if ((int)g_scratch_addr.size() <= dev) g_scratch_addr.resize(dev + 1, nullptr);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      set_error("air_solve_noalloc: hipGetSymbolAddress of the scratch array failed (%s)", hipGetErrorString(e));
      return AH_EHIP;
    }
    g_scratch_addr[dev] = static_cast<char*>(p);
  }
  *out = g_scratch_addr[dev];
  return AH_OK;
}

// Lays the FGMRES workspace for n unknowns and restart m out from base in
// 256-byte aligned pieces (base == nullptr: sizes only); returns the bytes.
static size_t carve_workspace(char* base, int64_t n, int m, int precision, KWork* W) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> char* {
    char* p = base ? base + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return p;
  };
  const size_t nd = (size_t)n * sizeof(double);
  W->V = reinterpret_cast<double*>(take((size_t)(m + 1) * nd));
  if (precision == 0)
    W->Z = reinterpret_cast<double*>(take((size_t)m * nd));
  else
    W->Z32 = reinterpret_cast<float*>(take((size_t)m * (size_t)n * sizeof(float)));
  W->w = reinterpret_cast<double*>(take(nd));
  W->r = reinterpret_cast<double*>(take(nd));
  W->bhat = reinterpret_cast<double*>(take(nd));
  W->partial = reinterpret_cast<double*>(take((size_t)(2 * m + 4) * 1024 * sizeof(double)));
  W->hdev = reinterpret_cast<double*>(take((size_t)4 * (m + 3) * sizeof(double)));
  return off;
}

}  // namespace ah

using namespace ah;

extern "C" void ah_solve_defaults(ah_solve_params* p) {
  if (!p) return;
  p->tol = 1e-8;
  p->restart = 100;
  p->maxit = 1000;
  p->precision = 0;
  p->x0_given = 0;
  p->method = 0;
}

static ah_status check_solve(const ah_hier* h, const ah_solve_params* prm, int transpose) {
  if (!h || !prm) { set_error("air_solve: null argument"); return AH_EINVAL; }
  if (prm->precision == 1 && !h->prm.fp32_cycle) {
    set_error("air_solve: FP32 cycle requested but the hierarchy was built without fp32_cycle");
    return AH_EINVAL;
  }
  if (prm->precision < 0 || prm->precision > 1 || prm->restart < 1 || prm->maxit < 0 || !(prm->tol > 0.0) ||
      prm->method < 0 || prm->method > 1) {
    set_error("air_solve: invalid parameters");
    return AH_EINVAL;
  }
  if (transpose && !h->prm.adjoint) {
    set_error("air_solve_adjoint: hierarchy built without adjoint = 1");
    return AH_EINVAL;
  }
  return AH_OK;
}

// Forward solve with a given workspace (W.bhat holds the scaled
// right-hand side when rhs is given).
static ah_status solve_forward(ah_hier* h, const KWork& W, const double* rhs, double* x, const ah_solve_params& prm,
                               hipStream_t st, ah_solve_info* info) {
  const ah_system* s = h->sys;
  const int64_t n = s->n;
  const double* b = s->d_Hhat;
  if (rhs) {
    hipLaunchKernelGGL(k_blockscale, g1(n), dim3(256), 0, st, s->nfree, s->b, s->d_Dinv, rhs, W.bhat, 0);
    AH_LAUNCHED();
    b = W.bhat;
  }
  if (!prm.x0_given) AH_HIP(hipMemsetAsync(x, 0, n * sizeof(double), st));
  Op A{s->d_rowptr, s->d_col, s->d_val};
  const AhLevel& L0 = h->lev[0];
  if (L0.ob) {
    A.ob = L0.ob;
    A.optr = L0.optr;
    A.ocol = L0.ocol;
    A.ov = L0.oval;
    A.nov = L0.nov;
    A.lpb = by_blocks(h, L0.ob) ? (h->lpb ? h->lpb : fbb_lanes(L0.nov, n, L0.ob)) : 0;
  }
  if (prm.method == 1) return bicgstab(h, A, b, x, prm, 0, st, info);
  return fgmres(h, W, A, b, x, prm, 0, st, info);
}

extern "C" ah_status air_solve(const ah_hier* hc, const double* rhs, double* x, const ah_solve_params* prm,
                               void* stream, ah_solve_info* info) {
  AH_TRY(check_solve(hc, prm, 0));
  if (hc->sys->n == 0) {   // nothing to solve
    if (info) { std::memset(info, 0, sizeof(*info)); info->converged = 1; }
    return AH_OK;
  }
  if (!x) { set_error("air_solve: null x"); return AH_EINVAL; }
  ah_hier* h = const_cast<ah_hier*>(hc);
  hipStream_t st = as_stream(stream);
  KWork W;
  AH_TRY(ensure_workspace(h, std::max(1, prm->restart), prm->precision, st, &W));
  return solve_forward(h, W, rhs, x, *prm, st, info);
}

extern "C" ah_status air_solve_noalloc(const ah_hier* hc, const double* rhs, double* x,
                                       const ah_solve_params* prm, void* stream, ah_solve_info* info) {
  AH_TRY(check_solve(hc, prm, 0));
  if (prm->method != 0) {
    set_error("air_solve_noalloc: only FGMRES (method 0) runs without allocation");
    return AH_EUNSUPPORTED;
  }
  if (prm->restart > AH_NOALLOC_MAX_RESTART) {
    set_error("air_solve_noalloc: restart %d exceeds %d", prm->restart, AH_NOALLOC_MAX_RESTART);
    return AH_EUNSUPPORTED;
  }
  if (hc->sys->n == 0) {
    if (info) { std::memset(info, 0, sizeof(*info)); info->converged = 1; }
    return AH_OK;
  }
  if (!x) { set_error("air_solve_noalloc: null x"); return AH_EINVAL; }
  ah_hier* h = const_cast<ah_hier*>(hc);
  hipStream_t st = as_stream(stream);
  const int m = std::max(1, prm->restart);
  const int64_t n = h->sys->n;
  KWork W;
  const size_t need = carve_workspace(nullptr, n, m, prm->precision, &W);
  if (need > kScratchBytes) {
    set_error("air_solve_noalloc: workspace of %zu bytes (n = %lld, restart = %d) exceeds the %zu-byte scratch array",
              need, (long long)n, m, kScratchBytes);
    return AH_EUNSUPPORTED;
  }
  char* base = nullptr;
  AH_TRY(scratch_address(&base));
  carve_workspace(base, n, m, prm->precision, &W);
  // the thread's pinned staging where it exists (a setup on this thread leaves
  // it), else a pageable array and copies
  static thread_local double stage[4 * (AH_NOALLOC_MAX_RESTART + 3)];
  W.host = pinned_existing(4 * (m + 3) + 1);
  W.polled = W.host && h->poll;
  if (!W.host) W.host = stage;
  return solve_forward(h, W, rhs, x, *prm, st, info);
}

extern "C" ah_status air_solve_adjoint(const ah_hier* hc, const double* g, double* lam, const ah_solve_params* prm,
                                       void* stream, ah_solve_info* info) {
  AH_TRY(check_solve(hc, prm, 1));
  if (hc->sys->n == 0) {
    if (info) { std::memset(info, 0, sizeof(*info)); info->converged = 1; }
    return AH_OK;
  }
  if (!g || !lam) { set_error("air_solve_adjoint: null argument"); return AH_EINVAL; }
  ah_hier* h = const_cast<ah_hier*>(hc);
  hipStream_t st = as_stream(stream);
  const ah_system* s = h->sys;
  const int64_t n = s->n;
  KWork W;
  AH_TRY(ensure_workspace(h, std::max(1, prm->restart), prm->precision, st, &W));
  double* mu = W.bhat;   // S_hat^T mu = g, then lam = D_b^-T mu
  AhLevel& L0 = h->lev[0];
  if (!L0.ATptr && !L0.otval) {
    set_error("air_solve_adjoint: transposed level-0 operator missing");
    return AH_EINVAL;
  }
  AH_HIP(hipMemsetAsync(mu, 0, n * sizeof(double), st));   // zero initial guess
  Op AT{L0.ATptr, L0.ATcol, L0.ATval};
  if (L0.otval) {
    AT.ob = L0.ob;
    AT.optr = L0.optr;
    AT.ocol = L0.ocol;
    AT.ov = L0.otval;
    AT.nov = L0.nov;
    AT.lpb = by_blocks(h, L0.ob) ? (h->lpb ? h->lpb : fbb_lanes(L0.nov, n, L0.ob)) : 0;
  }
  ah_status rc = prm->method == 1 ? bicgstab(h, AT, g, mu, *prm, 1, st, info)
                                   : fgmres(h, W, AT, g, mu, *prm, 1, st, info);
  if (rc < 0) return rc;
  hipLaunchKernelGGL(k_blockscale, g1(n), dim3(256), 0, st, s->nfree, s->b, s->d_Dinv, mu, lam, 1);
  AH_LAUNCHED();
  AH_HIP(hipStreamSynchronize(st));
  return rc;
}

extern "C" ah_status ah_vcycle_apply(const ah_hier* hc, const double* r, double* z, int precision, int transpose,
                                     void* stream) {
  if (!hc || !r || !z) { set_error("ah_vcycle_apply: null argument"); return AH_EINVAL; }
  ah_hier* h = const_cast<ah_hier*>(hc);
  if (precision == 1 && !h->prm.fp32_cycle) { set_error("ah_vcycle_apply: no FP32 operators"); return AH_EINVAL; }
  if (transpose && !h->prm.adjoint) { set_error("ah_vcycle_apply: no transposes"); return AH_EINVAL; }
  hipStream_t st = as_stream(stream);
  const int64_t n = h->lev[0].n;
  if (precision == 0) return precond(h, r, z, nullptr, 0, transpose, st);
  float* z32 = nullptr;
  Arena tmp;
  tmp.stream = st;
  AH_TRY(tmp.get(&z32, n));
  AH_TRY(precond(h, r, nullptr, z32, 1, transpose, st));
  hipLaunchKernelGGL((k_cast<float, double>), g1(n), dim3(256), 0, st, n, z32, z);
  AH_LAUNCHED();
  AH_HIP(hipStreamSynchronize(st));
  tmp.release();
  return AH_OK;
}
