// hdg_assemble: element blocks of the space-time HDG bilinear form
// (Section 2.3), static condensation (Section 2.5), deterministic scatter
// into the free-facet block pattern, Dirichlet elimination, and the left
// facet-block-diagonal scaling of Section 4 fused into the conversion to the
// scalar CSR matrix used by AIR.  Also reconstruction, slab coupling and
// the adjoint gradient kernel.
//
// A wave assembles one element or, where its matrices are small, four.  The
// element basis is the nodal Lagrange basis on the reference simplex of the
// cell; facet unknowns use the nodal Lagrange basis on the sorted-vertex facet
// simplex.  Rows = test functions, columns = trial functions:
//   A(u,v) = int_K (-u a_hat.grad_hat v + nu grad u.grad v)
//            + sum_F int_F [(a+ + tau) u v - nu (grad u.n) v - nu u (grad v.n)]
//   B(l,v) = sum_F int_F [(a- - tau) l v + nu l (grad v.n)]
//   C(u,m) = sum_F int_F [-(a+ + tau) u m + nu (grad u.n) m]
//   D(l,m) = sum_F int_F [-(a- - tau) l m] + [F Neumann] int_F a+ l m
//   F(v) = int_K f v,  G(m) = [F Neumann] int_F g m
// with a_n = n_t + a.n, a+ = (a_n+|a_n|)/2, a- = (a_n-|a_n|)/2,
// tau = nu alpha / h_K, h_K = |det J|^(1/D); grad = spatial gradient.
#include <cmath>

#include "prof.h"
#include "system.h"

namespace ah {

template <int D, int P>
struct Sz {
  static constexpr int NU = D == 2 ? (P + 1) * (P + 2) / 2 : (P + 1) * (P + 2) * (P + 3) / 6;
  static constexpr int B = D == 2 ? (P + 1) : (P + 1) * (P + 2) / 2;
  static constexpr int NFc = D + 1;
  static constexpr int NL = NFc * B;
  static constexpr int N1 = P + 2;
  static constexpr int NQ = D == 2 ? N1 * N1 : N1 * N1 * N1;
  static constexpr int NQF = D == 2 ? N1 : N1 * N1;
  static constexpr int BS = B * (B + 1) / 2;   // packed symmetric facet matrices
  static constexpr int DS = D * (D + 1) / 2;
  // lanes per element: 16 where a lane can hold the whole of A_K, else a wave
  static constexpr int G = NU <= 6 ? 16 : 64;
  static constexpr int EPB = 64 / G;           // elements per (one-wave) workgroup
};

struct ElemArgs {
  int64_t ne;
  const double* vert;
  const int32_t* cell;
  const int32_t* elem_facet;
  const uint8_t* facet_loc;
  const int8_t* kind;
  const int32_t* bf_index;
  const int32_t* free_rank;
  const int32_t* elem_slot;
  const double* a_vert;
  const double* a_qe;      // velocity at the element quadrature points [ne][nq][D-1], or null
  const double* a_qf;      // velocity at the facet quadrature points [nf][nqf][D-1], or null
  const double* f_q;
  const double* g_q;
  const double* vol_w;
  const double* vol_lam;
  const double* vol_phi;
  const double* vol_dphi;
  const double* fac_w;
  const double* fac_mu;
  const double* fac_psi;
  const double* fac_proj;
  const double* fac_pp;    // [nqf][b(b+1)/2] products of facet basis functions
  const double* fac_mass;  // [b(b+1)/2] facet mass matrix over |F|
  const double* ten_adv;   // [(D+1) D][nu nu] reference advection tensor
  const double* ten_dif;   // [D(D+1)/2][nu nu] reference diffusion tensor
  const double* ten_dn;    // [D+1][D][nu nu] facet normal-derivative tensors
  double nu, alpha;
  double* bval;            // off-diagonal blocks of S
  double* Dg;              // [ne][D+1][b][b] the elements' parts of its diagonal blocks
  double* Hk;              // [ne][nl] the elements' parts of H
  int add_off;             // off-diagonal blocks may get two parts (a cell given twice): add to zeros
  double* lamD;
  double* Ainv;
  double* Bm;
  double* Cm;
  double* Fv;
  int* err;
  // gradient mode
  const double* lam_fwd;   // [n_free] forward solution (Dirichlet traces from lamD)
  const double* lam_adj;   // [n_free] adjoint solution (zero on Dirichlet facets)
  double* dJdf_q;          // [ne][nq]
  double* dnu_elem;        // [ne]
  int8_t node[64];         // element node at lattice indices (i_1, ..): sum i_k (p+1)^(k-1)
  int8_t fnode[10][3];     // barycentric indices of the facet nodes
};

// The element's matrices in LDS.  With a nodal element basis the trace of
// basis function i on facet F is the facet function of node i, or zero where
// node i is not on F, so every facet term comes from three facet matrices
//   MA = int (a+ + tau) psi psi,  MB = int (a- - tau) psi psi,
//   Z  = nu int (d phi_i/dn) psi  (from ten_dn, no quadrature)
// by scattering: A gets MA - Z - Z^T, B_F = MB + Z, C_F = Z^T - MA and
// D_F = -MB (+ int a+ psi psi on Neumann facets).  Only the upwind weights
// a+ and a- need points: two packed b x b sums per facet.
template <int D, int P>
struct ElemSmem {
  using S = Sz<D, P>;
  double X[(D + 1) * D];
  double av[(D + 1) * (D - 1)];
  double Jinv[D * D];
  double absdet, tau;
  double nrm[(D + 1) * D];
  double area[D + 1];
  double eta[(D + 1) * D];
  double vcoef[(D + 1) * D + S::DS];   // beta_kr, then G_rs (r <= s)
  int fid[D + 1], kindf[D + 1], bidx[D + 1];
  int8_t loc[(D + 1) * D];
  int8_t fnode[(D + 1) * S::B];        // element node of facet node m
  int8_t pos[(D + 1) * S::NU];         // facet node of element node i, or -1
  double MA[(D + 1) * S::BS], MB[(D + 1) * S::BS], DD[(D + 1) * S::BS];
  double F[S::NU], y[S::NU], LD[S::NL];
  union {
    double A[S::NU * S::NU];
    struct {
      double wf[S::NQ];                // W_q f_q at the element points
      double cap[(D + 1) * S::NQF], cam[(D + 1) * S::NQF];   // W a+, W a- at the facet points
      double Fp[S::G];
    } q;
  };
  union {
    double ZC[S::NL * S::NU];          // Z by (facet, facet node; element node), then C
    double beta[S::NQ * D];            // J^-1 (1, a(x_q)) (velocity at the points)
  };
};

// Packed index of a symmetric entry.
__device__ inline int sym(int m, int n) { return m >= n ? m * (m + 1) / 2 + n : n * (n + 1) / 2 + m; }

// Element geometry: inverse Jacobian, penalty, facet normals and areas, and
// which element nodes lie on which facet.  g: lane of the element's S::G.
template <int D, int P>
__device__ void elem_geometry(const ElemArgs& a, ElemSmem<D, P>& sm, int64_t e, int g, double nu_eff, double alpha,
                              bool live) {
  using S = Sz<D, P>;
  constexpr int G = S::G;
  for (int t = g; t < (D + 1) * D; t += G) {
    sm.X[t] = a.vert[(int64_t)a.cell[e * (D + 1) + t / D] * D + t % D];
    sm.loc[t] = a.facet_loc[e * (D + 1) * D + t];
  }
  for (int t = g; t < (D + 1) * (D - 1); t += G)
    sm.av[t] = a.a_vert ? a.a_vert[(int64_t)a.cell[e * (D + 1) + t / (D - 1)] * (D - 1) + t % (D - 1)] : 0.0;
  if (g < D + 1) {
    const int f = a.elem_facet[e * (D + 1) + g];
    sm.fid[g] = f;
    sm.kindf[g] = a.kind[f];
    sm.bidx[g] = a.bf_index[f];
  }
  for (int t = g; t < (D + 1) * S::NU; t += G) sm.pos[t] = -1;
  for (int k = g; k < S::NL; k += G) sm.LD[k] = 0.0;
  __syncthreads();
  for (int t = g; t < (D + 1) * S::B; t += G) {
    const int f = t / S::B, m = t % S::B;
    int at = 0;
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const int v = sm.loc[f * D + s];   // local vertex; its lattice index is coordinate v (v > 0)
      int w = a.fnode[m][s];
      for (int c = 1; c < v; ++c) w *= P + 1;
      at += v > 0 ? w : 0;
    }
    const int i = a.node[at];
    sm.fnode[t] = (int8_t)i;
    sm.pos[f * S::NU + i] = (int8_t)m;
  }
  if (g == 0) {
    double J[D * D];   // J[r][c] = X[c+1][r] - X[0][r]
    for (int r = 0; r < D; ++r)
      for (int c = 0; c < D; ++c) J[r * D + c] = sm.X[(c + 1) * D + r] - sm.X[r];
    double det;
    double Ji[D * D];
    if (D == 2) {
      det = J[0] * J[3] - J[1] * J[2];
      Ji[0] = J[3] / det; Ji[1] = -J[1] / det; Ji[2] = -J[2] / det; Ji[3] = J[0] / det;
    } else {
      double c00 = J[4] * J[8] - J[5] * J[7], c01 = J[5] * J[6] - J[3] * J[8], c02 = J[3] * J[7] - J[4] * J[6];
      det = J[0] * c00 + J[1] * c01 + J[2] * c02;
      Ji[0] = c00 / det; Ji[1] = (J[2] * J[7] - J[1] * J[8]) / det; Ji[2] = (J[1] * J[5] - J[2] * J[4]) / det;
      Ji[3] = c01 / det; Ji[4] = (J[0] * J[8] - J[2] * J[6]) / det; Ji[5] = (J[2] * J[3] - J[0] * J[5]) / det;
      Ji[6] = c02 / det; Ji[7] = (J[1] * J[6] - J[0] * J[7]) / det; Ji[8] = (J[0] * J[4] - J[1] * J[3]) / det;
    }
    for (int k = 0; k < D * D; ++k) sm.Jinv[k] = Ji[k];
    const double ad = fabs(det);
    sm.absdet = ad;
    sm.tau = nu_eff * alpha / (D == 2 ? sqrt(ad) : cbrt(ad));
    if (live && (!(ad > 0.0) || !isfinite(ad))) atomicOr(a.err, 2);
  }
  __syncthreads();
  if (g < D + 1) {
    const double fact = D == 2 ? 2.0 : 6.0;
    double gr[D], gn = 0.0;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      double v = 0.0;
      if (g == 0)
        for (int r = 0; r < D; ++r) v -= sm.Jinv[r * D + c];
      else
        v = sm.Jinv[(g - 1) * D + c];
      gr[c] = v;
      gn += v * v;
    }
    gn = sqrt(gn);
#pragma unroll
    for (int c = 0; c < D; ++c) { gr[c] = -gr[c] / gn; sm.nrm[g * D + c] = gr[c]; }
    sm.area[g] = D * (sm.absdet / fact) * gn;
#pragma unroll
    for (int r = 0; r < D; ++r) {
      double v = 0.0;
#pragma unroll
      for (int c = 1; c < D; ++c) v += sm.Jinv[r * D + c] * gr[c];
      sm.eta[g * D + r] = v;
    }
  }
  __syncthreads();
}

// A, MA, MB, DD, Z, F and the Dirichlet traces.  advect = false and nu_eff = 1
// gives the nu-derivative of the blocks.
template <int D, int P>
__device__ void elem_integrate(const ElemArgs& a, ElemSmem<D, P>& sm, int64_t e, int g, double nu_eff, bool advect,
                               bool data) {
  using S = Sz<D, P>;
  constexpr int NU = S::NU, B = S::B, BS = S::BS, NQ = S::NQ, NQF = S::NQF, G = S::G, DS = S::DS;
  // volume coefficients: with a_k = (1, a at vertex k), beta_kr = (J^-1 a_k)_r
  // and G_rs = sum over the spatial c of Jinv[r][c] Jinv[s][c],
  //   A_ij = |det J| (nu sum_{r<=s} G_rs M^rs_ij - sum_kr beta_kr T^kr_ij)
  for (int t = g; t < (D + 1) * D + DS; t += G) {
    double v = 0.0;
    if (t < (D + 1) * D) {
      const int k = t / D, r = t % D;
      if (advect) {
        v = sm.Jinv[r * D];
        for (int c = 1; c < D; ++c) v += sm.Jinv[r * D + c] * sm.av[k * (D - 1) + c - 1];
      }
    } else {
      int u = t - (D + 1) * D, r = 0;
      while (u >= D - r) { u -= D - r; ++r; }
      for (int c = 1; c < D; ++c) v += sm.Jinv[r * D + c] * sm.Jinv[(r + u) * D + c];
    }
    sm.vcoef[t] = v;
  }
  const bool has_f = data && a.f_q;
  if (has_f)
    for (int q = g; q < NQ; q += G) sm.q.wf[q] = a.vol_w[q] * sm.absdet * a.f_q[e * NQ + q];
  // upwind weights at the facet points
  if (advect)
    for (int t = g; t < (D + 1) * NQF; t += G) {
      const int f = t / NQF, q = t % NQF;
      double an = sm.nrm[f * D];
#pragma unroll
      for (int c = 1; c < D; ++c) {
        double v = 0.0;
        if (a.a_qf)
          v = a.a_qf[((int64_t)sm.fid[f] * NQF + q) * (D - 1) + c - 1];
        else
          for (int s = 0; s < D; ++s) v += a.fac_mu[q * D + s] * sm.av[sm.loc[f * D + s] * (D - 1) + c - 1];
        an += v * sm.nrm[f * D + c];
      }
      const double W = a.fac_w[q] * sm.area[f];
      sm.q.cap[t] = W * (0.5 * (an + fabs(an)));
      sm.q.cam[t] = W * (0.5 * (an - fabs(an)));
    }
  if (data && a.g_q)
    for (int t = g; t < (D + 1) * B; t += G) {
      const int f = t / B, m = t % B;
      if (sm.kindf[f] != 1) continue;
      const double* gq = a.g_q + (int64_t)sm.bidx[f] * NQF;
      double acc = 0.0;
      for (int q = 0; q < NQF; ++q) acc += a.fac_proj[m * NQF + q] * gq[q];
      sm.LD[t] = acc;
    }
  __syncthreads();
  for (int t = g; t < (D + 1) * BS; t += G) {
    const int f = t / BS, mn = t % BS;
    double ap = 0.0, am = 0.0;
    if (advect) {
#pragma unroll 5
      for (int q = 0; q < NQF; ++q) {
        const double pp = a.fac_pp[q * BS + mn];
        ap += sm.q.cap[f * NQF + q] * pp;
        am += sm.q.cam[f * NQF + q] * pp;
      }
    }
    const double w = sm.tau * sm.area[f] * a.fac_mass[mn];
    sm.MA[t] = ap + w;
    sm.MB[t] = am - w;
    sm.DD[t] = w - am + ((sm.kindf[f] == 2) ? ap : 0.0);
  }
  // F_i = sum_q W_q f_q phi_i(x_q), the points dealt to G / NU lanes per i
  constexpr int PARTS = G / NU;
  if (has_f && g < PARTS * NU) {
    const int i = g % NU;
    double acc = 0.0;
    for (int q = g / NU; q < NQ; q += PARTS) acc += sm.q.wf[q] * a.vol_phi[q * NU + i];
    sm.q.Fp[g] = acc;
  }
  __syncthreads();
  for (int i = g; i < NU; i += G) {
    double acc = 0.0;
    if (has_f)
#pragma unroll
      for (int k = 0; k < PARTS; ++k) acc += sm.q.Fp[k * NU + i];
    sm.F[i] = acc;
  }
  __syncthreads();
  // velocity given at the quadrature points: the advective part of A_ij is
  // sum_q w_q phi_j(x_q) beta_q . grad phi_i(x_q), beta_q = J^-1 (1, a(x_q))
  const bool aq = advect && a.a_qe;
  if (aq) {
    for (int k = g; k < NQ * D; k += G) {
      const int q = k / D, r = k % D;
      double v = sm.Jinv[r * D];
      for (int c = 1; c < D; ++c) v += sm.Jinv[r * D + c] * a.a_qe[((int64_t)e * NQ + q) * (D - 1) + c - 1];
      sm.beta[k] = v;
    }
    __syncthreads();
    for (int idx = g; idx < NU * NU; idx += G) {
      const int i = idx / NU, j = idx % NU;
      double adv = 0.0;
      for (int q = 0; q < NQ; ++q) {
        double gr = 0.0;
#pragma unroll
        for (int r = 0; r < D; ++r) gr += sm.beta[q * D + r] * a.vol_dphi[(q * NU + i) * D + r];
        adv += a.vol_w[q] * a.vol_phi[q * NU + j] * gr;
      }
      sm.A[idx] = adv;
    }
    __syncthreads();
  }
  for (int t = g; t < S::NL * NU; t += G) {
    const int fm = t / NU, i = t % NU, f = fm / B;
    const int j = sm.fnode[fm];
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < D; ++r) v += sm.eta[f * D + r] * a.ten_dn[((f * D + r) * NU + j) * NU + i];
    sm.ZC[t] = nu_eff * sm.area[f] * v;
  }
  __syncthreads();
  for (int idx = g; idx < NU * NU; idx += G) {
    const int i = idx / NU, j = idx % NU;
    double adv = 0.0, dif = 0.0;
    if (aq) {
      adv = sm.A[idx];
    } else {
#pragma unroll
      for (int kr = 0; kr < (D + 1) * D; ++kr) adv += sm.vcoef[kr] * a.ten_adv[kr * NU * NU + idx];
    }
#pragma unroll
    for (int rs = 0; rs < DS; ++rs) dif += sm.vcoef[(D + 1) * D + rs] * a.ten_dif[rs * NU * NU + idx];
    double v = sm.absdet * (nu_eff * dif - adv);
#pragma unroll
    for (int f = 0; f <= D; ++f) {
      const int mi = sm.pos[f * NU + i], mj = sm.pos[f * NU + j];
      if (mj >= 0) v -= sm.ZC[(f * B + mj) * NU + i];
      if (mi >= 0) v -= sm.ZC[(f * B + mi) * NU + j];
      if (mi >= 0 && mj >= 0) v += sm.MA[f * BS + sym(mi, mj)];
    }
    sm.A[idx] = v;
  }
  __syncthreads();
}

// Entry r of column (facet lf, node m) of B_K.
template <int D, int P>
__device__ inline double elem_b(const ElemSmem<D, P>& sm, int r, int lf, int m) {
  using S = Sz<D, P>;
  const int q = sm.pos[lf * S::NU + r];
  const double z = sm.ZC[(lf * S::B + m) * S::NU + r];
  return q >= 0 ? z + sm.MB[lf * S::BS + sym(q, m)] : z;
}

// Z -> C_K in place: C = Z^T - MA at the facet's nodes.
template <int D, int P>
__device__ inline void elem_z_to_c(ElemSmem<D, P>& sm, int g) {
  using S = Sz<D, P>;
  for (int t = g; t < S::NL * S::NU; t += S::G) {
    const int fm = t / S::NU, lf = fm / S::B;
    const int q = sm.pos[lf * S::NU + t % S::NU];
    if (q >= 0) sm.ZC[t] -= sm.MA[lf * S::BS + sym(q, fm % S::B)];
  }
}

// Value of a double in lane src (uniform) for the whole wave.
__device__ inline double wave_bcast(double v, int src) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
  return __hiloint2double(hi, lo);
}

__device__ inline int wave_bcast(int v, int src) { return __builtin_amdgcn_readlane(v, src); }

// Element blocks, X = A^-1 [B | I] by Gauss-Jordan with partial pivoting in
// registers, and the condensed block S_K = D_K - C_K A_K^-1 B_K with its
// right-hand side.  Each off-diagonal block of S belongs to one element and is
// stored plainly; the diagonal blocks and H have up to two parts, kept per
// element and summed per facet afterwards, so nothing is zeroed or added
// atomically.
//
// Bound by the FP64 vector and LDS pipes, not by HBM (2-D + time, p = 2: 24,576
// elements take 199 us; p = 1, 5.3M elements 10.4 ms; before, with a monomial
// basis, every facet term by quadrature and one element per wave: 616 us and
// 48.5 ms).  Small elements (nu <= 6): 16 lanes each, a lane holding all of A
// and one column, four elements to a wave; larger ones: a wave each, a lane a
// column of [A | B | F | I], the pivot column broadcast by readlane.
template <int D, int P>
__global__ __launch_bounds__(64) void k_element(ElemArgs a) {
  using S = Sz<D, P>;
  constexpr int NU = S::NU, NL = S::NL, B = S::B, G = S::G;
  __shared__ ElemSmem<D, P> sm_[S::EPB];
  const int g = threadIdx.x % G;
  ElemSmem<D, P>& sm = sm_[G == 64 ? 0 : threadIdx.x / G];
  const int64_t e0 = (int64_t)blockIdx.x * S::EPB + (G == 64 ? 0 : threadIdx.x / G);
  const bool live = e0 < a.ne;
  const int64_t e = live ? e0 : a.ne - 1;
  elem_geometry<D, P>(a, sm, e, g, a.nu, a.alpha, live);
  elem_integrate<D, P>(a, sm, e, g, a.nu, true, true);
  bool singular = false;
  // this lane's column of A^-1 [B | I]: xs; its column of B_K (or -1), and of
  // the identity (or -1)
  double xs[NU];
  int cc = -1, ci = -1;
  if constexpr (G == 16) {
    static_assert(G != 16 || NL + NU <= 16, "a lane per column");
    cc = g < NL ? g : -1;
    ci = g >= NL && g < NL + NU ? g - NL : -1;
    double M[NU][NU];
#pragma unroll
    for (int r = 0; r < NU; ++r) {
      xs[r] = cc >= 0 ? elem_b<D, P>(sm, r, cc / B, cc % B) : r == ci ? 1.0 : 0.0;
#pragma unroll
      for (int c = 0; c < NU; ++c) M[r][c] = sm.A[r * NU + c];
    }
    if (a.Bm && live && cc >= 0)
#pragma unroll
      for (int r = 0; r < NU; ++r) a.Bm[(e * NU + r) * NL + cc] = xs[r];
#pragma unroll
    for (int k = 0; k < NU; ++k) {
#pragma unroll
      for (int r = k + 1; r < NU; ++r) {
        const bool sw = fabs(M[r][k]) > fabs(M[k][k]);
#pragma unroll
        for (int c = k; c < NU; ++c) {
          const double u = M[k][c], v = M[r][c];
          M[k][c] = sw ? v : u;
          M[r][c] = sw ? u : v;
        }
        const double u = xs[k], v = xs[r];
        xs[k] = sw ? v : u;
        xs[r] = sw ? u : v;
      }
      if (!(fabs(M[k][k]) > 0.0) || !isfinite(M[k][k])) singular = true;
      const double inv = 1.0 / M[k][k];
#pragma unroll
      for (int c = k + 1; c < NU; ++c) M[k][c] *= inv;
      xs[k] *= inv;
#pragma unroll
      for (int r = 0; r < NU; ++r) {
        if (r == k) continue;
#pragma unroll
        for (int c = k + 1; c < NU; ++c) M[r][c] -= M[r][k] * M[k][c];
        xs[r] -= M[r][k] * xs[k];
      }
    }
    __syncthreads();
    // A^-1 F from the identity columns, through A's place
    if (ci >= 0)
#pragma unroll
      for (int r = 0; r < NU; ++r) {
        sm.A[r * NU + ci] = xs[r];
        if (a.Ainv && live) a.Ainv[(e * NU + r) * NU + ci] = xs[r];
      }
    __syncthreads();
    if (g < NU) {
      double v = 0.0;
#pragma unroll
      for (int c = 0; c < NU; ++c) v += sm.A[g * NU + c] * sm.F[c];
      sm.y[g] = v;
    }
  } else {
    // columns of [A | B F I], lane l holds columns l + 64 u
    constexpr int NC = NU + NL + 1 + NU;
    constexpr int CPL = (NC + 63) / 64;
    static_assert(NU + NL + 1 <= 64, "the columns of A, B and F in the first slot");
    double col[CPL][NU];
#pragma unroll
    for (int u = 0; u < CPL; ++u) {
      const int c = g + 64 * u;
#pragma unroll
      for (int r = 0; r < NU; ++r) {
        double v = 0.0;
        if (c < NU) v = sm.A[r * NU + c];
        else if (c < NU + NL) v = elem_b<D, P>(sm, r, (c - NU) / B, (c - NU) % B);
        else if (c == NU + NL) v = sm.F[r];
        else if (c < NC) v = (r == c - NU - NL - 1) ? 1.0 : 0.0;
        col[u][r] = v;
      }
    }
    cc = g >= NU && g < NU + NL ? g - NU : -1;
    if (a.Bm && cc >= 0)
#pragma unroll
      for (int r = 0; r < NU; ++r) a.Bm[(e * NU + r) * NL + cc] = col[0][r];
#pragma unroll
    for (int k = 0; k < NU; ++k) {
      // pivot search in column k (lane k, slot 0): first largest |a_rk|, r >= k
      double best = fabs(col[0][k]);
      int p = k;
#pragma unroll
      for (int r = k + 1; r < NU; ++r) {
        const double v = fabs(col[0][r]);
        if (v > best) { best = v; p = r; }
      }
      p = wave_bcast(p, k);
      if (p != k) {
#pragma unroll
        for (int r = k + 1; r < NU; ++r)
          if (p == r)   // uniform
#pragma unroll
            for (int u = 0; u < CPL; ++u) {
              const double v = col[u][k];
              col[u][k] = col[u][r];
              col[u][r] = v;
            }
      }
      // the pivot column, now in lane k
      double f[NU];
#pragma unroll
      for (int r = 0; r < NU; ++r) f[r] = wave_bcast(col[0][r], k);
      if (!(fabs(f[k]) > 0.0) || !isfinite(f[k])) singular = true;
      const double inv = 1.0 / f[k];
#pragma unroll
      for (int u = 0; u < CPL; ++u) {
        const double xk = col[u][k] * inv;
#pragma unroll
        for (int r = 0; r < NU; ++r) col[u][r] = r == k ? xk : col[u][r] - f[r] * xk;
      }
    }
    // kept element inverse: the identity columns now hold A^-1
    if (a.Ainv) {
#pragma unroll
      for (int u = 0; u < CPL; ++u) {
        const int c = g + 64 * u - NU - NL - 1;
        if (c < 0 || c >= NU) continue;
#pragma unroll
        for (int r = 0; r < NU; ++r) a.Ainv[(e * NU + r) * NU + c] = col[u][r];
      }
    }
    if (g == NU + NL)
#pragma unroll
      for (int r = 0; r < NU; ++r) sm.y[r] = col[0][r];
#pragma unroll
    for (int r = 0; r < NU; ++r) xs[r] = col[0][r];
  }
  if (singular && live && g == 0) atomicOr(a.err, 1);
  __syncthreads();
  // keep C and F; y = A^-1 (F - B[:, Dir] lambda_D)
  elem_z_to_c<D, P>(sm, g);
  bool dir = false;
#pragma unroll
  for (int lf = 0; lf <= D; ++lf) dir |= sm.kindf[lf] == 1;
  if (__any(dir)) {
    for (int lf = 0; lf <= D; ++lf)
      for (int m = 0; m < B; ++m) {
        if (dir && sm.kindf[lf] == 1 && cc == lf * B + m)
#pragma unroll
          for (int r = 0; r < NU; ++r) sm.y[r] -= xs[r] * sm.LD[cc];
        __syncthreads();
      }
  }
  __syncthreads();
  if (a.Cm && live) {
    for (int k = g; k < NL * NU; k += G) a.Cm[e * NL * NU + k] = sm.ZC[k];
    for (int k = g; k < NU; k += G) a.Fv[e * NU + k] = sm.F[k];
  }
  // S_K = D_K - C_K X column by column
  if (cc >= 0 && live) {
    const int cb = cc / B, cm = cc % B;
    const int32_t* slot = a.elem_slot + e * (D + 1) * (D + 1);
#pragma unroll
    for (int rb = 0; rb <= D; ++rb) {
      const int sl = slot[rb * (D + 1) + cb];
      const bool on = rb == cb;
      double* out = on ? a.Dg + (e * (D + 1) + rb) * B * B + cm : a.bval + (int64_t)sl * B * B + cm;
      if (!on && sl < 0) continue;
#pragma unroll 2
      for (int rm = 0; rm < B; ++rm) {
        double v = on ? sm.DD[rb * S::BS + sym(rm, cm)] : 0.0;
        const double* C = sm.ZC + (rb * B + rm) * NU;
#pragma unroll
        for (int k = 0; k < NU; ++k) v -= C[k] * xs[k];
        if (!on && a.add_off) unsafeAtomicAdd(out + rm * B, v);
        else out[rm * B] = v;
      }
    }
  }
  // H_K = -C_K y - D_K[:, Dir] lambda_D
  for (int r = g; r < NL; r += G) {
    const int lf = r / B, rm = r % B;
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < NU; ++k) v -= sm.ZC[r * NU + k] * sm.y[k];
    if (sm.kindf[lf] == 1) {
      for (int n = 0; n < B; ++n) v -= sm.DD[lf * S::BS + sym(rm, n)] * sm.LD[lf * B + n];
      if (live) a.lamD[(int64_t)sm.fid[lf] * B + rm] = sm.LD[r];
    }
    if (live) a.Hk[e * NL + r] = v;
  }
}

// Inverse of each free facet's diagonal block (Gauss-Jordan, partial
// pivoting).  All register arrays are indexed with compile-time indices
// (unrolled loops, predicated row swaps) so they stay in registers.
//
// The diagonal block and H of a facet are the sums of its at most two elements'
// parts (slots e (D+1) + lf, in element order).
template <int B>
__global__ __launch_bounds__(64) void k_diag_inv(int64_t nfree, const int32_t* __restrict__ fslot,
                                                 const double* __restrict__ Dg, double* __restrict__ dinv, int* err) {
  int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nfree) return;
  const int64_t s0 = fslot[2 * r], s1 = fslot[2 * r + 1];
  double M[B][B], I[B][B];
#pragma unroll
  for (int i = 0; i < B; ++i)
#pragma unroll
    for (int j = 0; j < B; ++j) {
      M[i][j] = Dg[s0 * B * B + i * B + j];
      I[i][j] = i == j ? 1.0 : 0.0;
    }
  if (s1 >= 0) {
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
      for (int j = 0; j < B; ++j) M[i][j] += Dg[s1 * B * B + i * B + j];
  }
  double scale = 0.0;
#pragma unroll
  for (int i = 0; i < B; ++i)
#pragma unroll
    for (int j = 0; j < B; ++j) scale = fmax(scale, fabs(M[i][j]));
  bool bad = !(scale > 0.0) || !isfinite(scale);
#pragma unroll
  for (int c = 0; c < B; ++c) {
    int p = c;
    double best = fabs(M[c][c]);
#pragma unroll
    for (int q = c + 1; q < B; ++q)
      if (fabs(M[q][c]) > best) { best = fabs(M[q][c]); p = q; }
    if (!(best > 1e-14 * scale)) bad = true;
#pragma unroll
    for (int q = c + 1; q < B; ++q) {
      if (q == p) {
#pragma unroll
        for (int j = 0; j < B; ++j) {
          double x = M[c][j]; M[c][j] = M[q][j]; M[q][j] = x;
          x = I[c][j]; I[c][j] = I[q][j]; I[q][j] = x;
        }
      }
    }
    double d = M[c][c];
    if (d == 0.0) d = 1.0;
    const double inv = 1.0 / d;
#pragma unroll
    for (int j = 0; j < B; ++j) { M[c][j] *= inv; I[c][j] *= inv; }
#pragma unroll
    for (int q = 0; q < B; ++q) {
      if (q == c) continue;
      const double f = M[q][c];
#pragma unroll
      for (int j = 0; j < B; ++j) { M[q][j] -= f * M[c][j]; I[q][j] -= f * I[c][j]; }
    }
  }
  if (bad) atomicOr(err, 4);
#pragma unroll
  for (int i = 0; i < B; ++i)
#pragma unroll
    for (int j = 0; j < B; ++j) dinv[r * B * B + i * B + j] = I[i][j];
}

// H0 of every free facet unknown: the sum of its elements' parts.
__global__ void k_h_sum(int64_t n, int B, const int32_t* __restrict__ fslot, const double* __restrict__ Hk,
                        double* __restrict__ H) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t R = i / B;
  const int m = (int)(i - R * B);
  const int64_t s0 = fslot[2 * R], s1 = fslot[2 * R + 1];
  H[i] = s1 >= 0 ? Hk[s0 * B + m] + Hk[s1 * B + m] : Hk[s0 * B + m];
}

// Unscaled systems keep the diagonal blocks of S in its block pattern.
__global__ void k_diag_store(int64_t nfree, int B, const int64_t* __restrict__ bptr,
                             const int32_t* __restrict__ bcol, const int32_t* __restrict__ fslot,
                             const double* __restrict__ Dg, double* __restrict__ bval) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nfree) return;
  int64_t s = bptr[r];
  while (bcol[s] != r) ++s;
  const int64_t s0 = fslot[2 * r], s1 = fslot[2 * r + 1];
  for (int k = 0; k < B * B; ++k) bval[s * B * B + k] = Dg[s0 * B * B + k] + (s1 >= 0 ? Dg[s1 * B * B + k] : 0.0);
}

// Scalar CSR of the level-0 operator on the structural pattern of the free
// facets (entries that happen to be zero are kept).  Scaled system: row
// R*B+m of D_b^-1 S, whose diagonal block is the identity, so the row holds
// its diagonal entry 1 and the B entries of every off-diagonal block, in
// column order; unscaled: the B entries of every block of S, the diagonal
// block included.  Row offsets follow from the block pattern (scaled:
// B R + B^2 odb_ptr[R] for the block row, 1 + B (nb - 1) per row).
template <int B>
__global__ void k_scaled_rowptr(int64_t nfree, const int64_t* __restrict__ bptr,
                                const int64_t* __restrict__ optr, int unscaled, int64_t* __restrict__ rowptr) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n = nfree * B;
  if (i > n) return;
  const int64_t R = i / B;
  const int m = (int)(i - R * B);
  if (unscaled) {
    const int64_t nb = R < nfree ? bptr[R + 1] - bptr[R] : 0;
    rowptr[i] = (int64_t)B * B * bptr[R] + (int64_t)m * B * nb;
  } else {
    const int64_t nob = R < nfree ? optr[R + 1] - optr[R] : 0;
    rowptr[i] = (int64_t)B * R + (int64_t)B * B * optr[R] + (int64_t)m * (1 + B * nob);
  }
}

// A thread per (block row, column of it): a free facet couples to at most the
// 2 D + 1 facets of its two cells, so thread t of a workgroup takes column
// t % NC of the workgroup's block row t / NC, reads that column of S's block
// once and writes its B scaled entries into the B scalar rows, and into the
// off-diagonal facet-block copy (oval, scaled systems); the rows' D_b^-1 are
// staged in LDS.  Bound by HBM: 8 bytes in and 20 out per entry (p = 1, 96^3
// mesh: 764M entries in 4.35 ms; a wave per block row, two thirds of its lanes
// idle at three columns a block, took 8.94 ms = 2.4 TB/s; p = 2 slab: 123 us,
// now 80).
template <int D, int B>
struct CsrSz {
  static constexpr int NB = 2 * D + 1;        // blocks of a block row, the diagonal one included
  static constexpr int NC = NB * B;
  static constexpr int ROWS = 256 / NC;       // block rows per workgroup
};

template <int D, int B>
__global__ __launch_bounds__(256) void k_csr_scaled(int64_t nfree, const int64_t* __restrict__ bptr,
                                                    const int32_t* __restrict__ bcol, const double* __restrict__ bval,
                                                    const double* __restrict__ dinv, int32_t* __restrict__ col,
                                                    double* __restrict__ val, int unscaled,
                                                    const int64_t* __restrict__ optr, double* __restrict__ oval) {
  using S = CsrSz<D, B>;
  __shared__ double sd[S::ROWS * B * B];
  const int64_t R0 = (int64_t)blockIdx.x * S::ROWS;
  if (!unscaled) {
    const int nd = (int)min((int64_t)S::ROWS, nfree - R0) * B * B;
    for (int k = threadIdx.x; k < nd; k += 256) sd[k] = dinv[R0 * B * B + k];
  }
  __syncthreads();
  const int rr = threadIdx.x / S::NC, c = threadIdx.x % S::NC;
  const int64_t R = R0 + rr;
  if (rr >= S::ROWS || R >= nfree) return;
  const int64_t s0 = bptr[R];
  const int nb = (int)(bptr[R + 1] - s0);
  if (c >= nb * B) return;
  const int64_t o0 = unscaled ? 0 : optr[R];
  const int nob = nb - 1;
  // first entry of the block row and the length of each of its rows
  const int64_t base = unscaled ? (int64_t)B * B * s0 : (int64_t)B * R + (int64_t)B * B * o0;
  const int rlen = unscaled ? B * nb : 1 + B * nob;
  const int j = c / B, n = c % B;
  const int64_t s = s0 + j;
  const int32_t C = bcol[s];
  if (!unscaled && C == R) {
    // the identity block: one diagonal entry per row
    col[base + (int64_t)n * rlen + j * B] = (int32_t)(R * B + n);
    val[base + (int64_t)n * rlen + j * B] = 1.0;
    return;
  }
  double bc[B];
#pragma unroll
  for (int k = 0; k < B; ++k) bc[k] = bval[s * B * B + k * B + n];
  // one diagonal entry precedes the blocks after the diagonal block
  const int pos = unscaled || C < R ? c : c - B + 1;
  const int64_t ob = o0 * B * B + (C < R ? j : j - 1) * B + n;
#pragma unroll
  for (int m = 0; m < B; ++m) {
    const int64_t rs = base + (int64_t)m * rlen + pos;
    col[rs] = (int32_t)(C * B + n);
    if (unscaled) {
      val[rs] = bc[m];
    } else {
      double v = 0.0;
#pragma unroll
      for (int k = 0; k < B; ++k) v += sd[(rr * B + m) * B + k] * bc[k];
      val[rs] = v;
      oval[ob + (int64_t)m * nob * B] = v;
    }
  }
}

template <int B>
__global__ void k_ident_blocks(int64_t nfree, double* __restrict__ dinv) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nfree * B * B) return;
  const int k = (int)(i % (B * B));
  dinv[i] = (k / B == k % B) ? 1.0 : 0.0;
}

template <int B>
__global__ void k_hhat(int64_t nfree, const double* __restrict__ dinv, const double* __restrict__ H,
                       double* __restrict__ hhat) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nfree * B) return;
  int64_t R = i / B;
  int m = (int)(i % B);
  double v = 0.0;
  for (int k = 0; k < B; ++k) v += dinv[R * B * B + m * B + k] * H[R * B + k];
  hhat[i] = v;
}

// Neumann term of the right-hand side (Section 2.3, the data term on the
// initial plane and on Neumann facets): H = H0 + G with
// G_f[m] = |F| sum_q w_q g_q psi_m(x_q) on every free boundary facet of
// Neumann kind.  |F| from the Gram determinant of the facet's edges; the
// facet rule weights sum to one.  One thread per (boundary facet, node);
// each free facet occurs once, so the updates do not collide.
template <int B>
__global__ void k_neumann(int64_t nbf, int D, int nqf, const int32_t* __restrict__ bfacets,
                          const int8_t* __restrict__ kind, const int32_t* __restrict__ free_rank,
                          const int32_t* __restrict__ facet_vert, const double* __restrict__ vert,
                          const double* __restrict__ fac_w, const double* __restrict__ fac_psi,
                          const double* __restrict__ g_q, double* __restrict__ H) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nbf * B) return;
  const int64_t bf = idx / B;
  const int m = (int)(idx % B);
  const int32_t f = bfacets[bf];
  if (kind[f] != 2) return;
  const int32_t fr = free_rank[f];
  if (fr < 0) return;
  double X[3][3];
  for (int s = 0; s < D; ++s)
    for (int c = 0; c < D; ++c) X[s][c] = vert[(int64_t)facet_vert[(int64_t)f * D + s] * D + c];
  double area;
  if (D == 2) {
    double e0 = X[1][0] - X[0][0], e1 = X[1][1] - X[0][1];
    area = sqrt(e0 * e0 + e1 * e1);
  } else {
    double u[3], v[3];
    for (int c = 0; c < 3; ++c) { u[c] = X[1][c] - X[0][c]; v[c] = X[2][c] - X[0][c]; }
    double g00 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    double g11 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
    double g01 = u[0] * v[0] + u[1] * v[1] + u[2] * v[2];
    area = 0.5 * sqrt(fmax(g00 * g11 - g01 * g01, 0.0));
  }
  double acc = 0.0;
#pragma unroll 5
  for (int q = 0; q < nqf; ++q) acc += fac_w[q] * g_q[bf * nqf + q] * fac_psi[q * B + m];
  H[(int64_t)fr * B + m] += area * acc;
}

// Physical quadrature points (element rule and boundary-facet rule).
__global__ void k_quad_points_elem(int64_t ne, int D, int nq, const double* __restrict__ vert,
                                   const int32_t* __restrict__ cell, const double* __restrict__ lam,
                                   double* __restrict__ xq) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= ne * nq) return;
  int64_t e = idx / nq;
  int q = (int)(idx % nq);
  for (int c = 0; c < D; ++c) {
    double v = 0.0;
    for (int k = 0; k <= D; ++k) v += lam[q * (D + 1) + k] * vert[(int64_t)cell[e * (D + 1) + k] * D + c];
    xq[idx * D + c] = v;
  }
}

__global__ void k_quad_points_bfacet(int64_t nbf, int D, int nqf, const double* __restrict__ vert,
                                     const int32_t* __restrict__ bfacets, const int32_t* __restrict__ fvert,
                                     const double* __restrict__ mu, double* __restrict__ xq) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nbf * nqf) return;
  int64_t k = idx / nqf;
  int q = (int)(idx % nqf);
  int64_t f = bfacets[k];
  for (int c = 0; c < D; ++c) {
    double v = 0.0;
    for (int s = 0; s < D; ++s) v += mu[q * D + s] * vert[(int64_t)fvert[f * D + s] * D + c];
    xq[idx * D + c] = v;
  }
}

// Adjoint gradient per element: with U = A^-1 (F - B Lambda) and
// w = -A^-T C^T lam, the derivative of J through F_K at the volume
// quadrature points, W_q w . phi(x_q), and the nu-derivative
// -w.(A1 U + B1 Lambda) - lam.(C1 U + D1 Lambda) with X1 = dX/dnu.
template <int D, int P>
__global__ __launch_bounds__(64) void k_grad(ElemArgs a) {
  using S = Sz<D, P>;
  constexpr int NU = S::NU, NL = S::NL, B = S::B, NQ = S::NQ, G = S::G;
  struct Vec { double L[NL], La[NL], R[NU], T[NU], U[NU], W[NU]; };
  __shared__ ElemSmem<D, P> sm_[S::EPB];
  __shared__ Vec sv_[S::EPB];
  const int g = threadIdx.x % G;
  ElemSmem<D, P>& sm = sm_[G == 64 ? 0 : threadIdx.x / G];
  Vec& sv = sv_[G == 64 ? 0 : threadIdx.x / G];
  const int64_t e0 = (int64_t)blockIdx.x * S::EPB + (G == 64 ? 0 : threadIdx.x / G);
  const bool live = e0 < a.ne;
  const int64_t e = live ? e0 : a.ne - 1;
  elem_geometry<D, P>(a, sm, e, g, 1.0, a.alpha, live);
  elem_integrate<D, P>(a, sm, e, g, 1.0, false, false);
  const double* Ai = a.Ainv + e * NU * NU;
  const double* Bo = a.Bm + e * NU * NL;
  const double* Co = a.Cm + e * NL * NU;
  const double* Fo = a.Fv + e * NU;
  for (int r = g; r < NL; r += G) {
    int lf = r / B, m = r % B, f = sm.fid[lf];
    int fr = a.free_rank[f];
    sv.L[r] = fr >= 0 ? a.lam_fwd[(int64_t)fr * B + m] : a.lamD[(int64_t)f * B + m];
    sv.La[r] = fr >= 0 ? a.lam_adj[(int64_t)fr * B + m] : 0.0;
  }
  __syncthreads();
  for (int i = g; i < NU; i += G) {
    double r = Fo[i];
    for (int c = 0; c < NL; ++c) r -= Bo[i * NL + c] * sv.L[c];
    sv.R[i] = r;
    double tt = 0.0;
    for (int c = 0; c < NL; ++c) tt += Co[c * NU + i] * sv.La[c];
    sv.T[i] = tt;
  }
  __syncthreads();
  for (int i = g; i < NU; i += G) {
    double u = 0.0, w = 0.0;
    for (int k = 0; k < NU; ++k) {
      u += Ai[i * NU + k] * sv.R[k];
      w -= Ai[k * NU + i] * sv.T[k];
    }
    sv.U[i] = u;
    sv.W[i] = w;
  }
  __syncthreads();
  if (a.dJdf_q && live)
    for (int q = g; q < NQ; q += G) {
      double v = 0.0;
      for (int i = 0; i < NU; ++i) v += sv.W[i] * a.vol_phi[q * NU + i];
      a.dJdf_q[e * NQ + q] = a.vol_w[q] * sm.absdet * v;
    }
  double acc = 0.0;
  for (int i = g; i < NU; i += G) {
    double v = 0.0;
    for (int j = 0; j < NU; ++j) v += sm.A[i * NU + j] * sv.U[j];
    for (int c = 0; c < NL; ++c) v += elem_b<D, P>(sm, i, c / B, c % B) * sv.L[c];
    acc -= sv.W[i] * v;
  }
  __syncthreads();
  elem_z_to_c<D, P>(sm, g);
  __syncthreads();
  for (int r = g; r < NL; r += G) {
    double v = 0.0;
    for (int j = 0; j < NU; ++j) v += sm.ZC[r * NU + j] * sv.U[j];
    int lf = r / B, m = r % B;
    for (int n = 0; n < B; ++n) v += sm.DD[lf * S::BS + sym(m, n)] * sv.L[lf * B + n];
    acc -= sv.La[r] * v;
  }
  for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, G);
  if (g == 0 && live) a.dnu_elem[e] = acc;
}

// ------------------------------------------------------------ dispatch
template <int D, int P>
static ah_status launch_element(const ElemArgs& a, hipStream_t st) {
  if (a.ne == 0) return AH_OK;
  using S = Sz<D, P>;
  // algorithmic bytes per element: cell, vertices, vertex velocity, facet
  // maps, source values in; condensed block, right-hand side and the kept
  // element blocks out
  const double per = (D + 1) * (4.0 + D * 8.0 + (D - 1) * 8.0 + 4.0 + D) + S::NQ * 8.0 +
                     (S::NL * S::NL + S::NL) * 8.0 +
                     (a.Ainv ? (S::NU * S::NU + 2.0 * S::NU * S::NL + S::NU) * 8.0 : 0.0);
  ProfScope ps;
  prof_begin(ps, "element", st, per * (double)a.ne);
  hipLaunchKernelGGL((k_element<D, P>), dim3((unsigned)cdiv(a.ne, S::EPB)), dim3(64), 0, st, a);
  prof_end(ps);
  AH_LAUNCHED();
  return AH_OK;
}

static ah_status element_dispatch(int D, int p, const ElemArgs& a, hipStream_t st) {
  if (D == 2 && p == 1) return launch_element<2, 1>(a, st);
  if (D == 2 && p == 2) return launch_element<2, 2>(a, st);
  if (D == 2 && p == 3) return launch_element<2, 3>(a, st);
  if (D == 3 && p == 1) return launch_element<3, 1>(a, st);
  if (D == 3 && p == 2) return launch_element<3, 2>(a, st);
  if (D == 3 && p == 3) return launch_element<3, 3>(a, st);
  set_error("unsupported dim_st/p");
  return AH_EUNSUPPORTED;
}

// parts: the arena of Dg, given back before the matrix is allocated.
template <int D, int B>
static ah_status scale_to_csr(ah_system* s, const ah_mesh* m, const double* Dg, Arena& parts, hipStream_t st,
                              int* d_err) {
  const int64_t nfree = s->nfree;
  const int64_t n = nfree * B;
  Arena& ar = s->arena;
  if (s->unscaled) {
    hipLaunchKernelGGL(k_diag_store, dim3(cdiv(std::max<int64_t>(nfree, 1), 256)), dim3(256), 0, st, nfree, B,
                       m->d_bsr_ptr, m->d_bsr_col, m->d_facet_slot, Dg, s->d_bval);
    hipLaunchKernelGGL(k_ident_blocks<B>, dim3(cdiv(std::max<int64_t>(nfree * B * B, 1), 256)), dim3(256), 0, st,
                       nfree, s->d_Dinv);
  } else
    hipLaunchKernelGGL(k_diag_inv<B>, dim3(cdiv(std::max<int64_t>(nfree, 1), 64)), dim3(64), 0, st, nfree,
                       m->d_facet_slot, Dg, s->d_Dinv, d_err);
  AH_LAUNCHED();
  parts.release();
  const int64_t nob = (int64_t)m->odb_col.size();
  s->nnz = s->unscaled ? (int64_t)B * B * s->nnzb : n + (int64_t)B * B * nob;
  if (s->nnz >= ((int64_t)1 << 31)) {
    set_error("level-0 matrix has %lld entries (limit 2^31)", (long long)s->nnz);
    return AH_EUNSUPPORTED;
  }
  AH_TRY(ar.get(&s->d_rowptr, n + 1));
  AH_TRY(ar.get(&s->d_col, s->nnz));
  AH_TRY(ar.get(&s->d_val, s->nnz));
  if (!s->unscaled) AH_TRY(ar.get(&s->d_odv, nob * B * B));
  hipLaunchKernelGGL(k_scaled_rowptr<B>, dim3((unsigned)cdiv(n + 1, 256)), dim3(256), 0, st, nfree, m->d_bsr_ptr,
                     (const int64_t*)m->d_odb_ptr, (int)s->unscaled, s->d_rowptr);
  AH_LAUNCHED();
  const dim3 gw((unsigned)cdiv(std::max<int64_t>(nfree, 1), CsrSz<D, B>::ROWS));
  hipLaunchKernelGGL((k_csr_scaled<D, B>), gw, dim3(256), 0, st, nfree, m->d_bsr_ptr, m->d_bsr_col, s->d_bval,
                     s->d_Dinv, s->d_col, s->d_val, (int)s->unscaled, (const int64_t*)m->d_odb_ptr, s->d_odv);
  AH_LAUNCHED();
  return AH_OK;
}

// H = H0 + Neumann term of g_q (NULL: none), then H_hat = D_b^-1 H.
template <int B>
static ah_status rhs_from_neumann(ah_system* s, const double* g_q, hipStream_t st) {
  const ah_mesh* m = s->mesh;
  const int64_t n = s->nfree * B;
  if (n == 0) return AH_OK;
  AH_HIP(hipMemcpyAsync(s->d_H, s->d_H0, n * sizeof(double), hipMemcpyDeviceToDevice, st));
  const int64_t nbf = (int64_t)m->bfacets.size();
  if (g_q && nbf > 0) {
    hipLaunchKernelGGL(k_neumann<B>, dim3((unsigned)cdiv(nbf * B, 128)), dim3(128), 0, st, nbf, m->D, s->nqf,
                       m->d_bfacets, m->d_kind, m->d_free_rank, m->d_facet_vert, m->d_vert, s->tab->d_fac_w,
                       s->tab->d_fac_psi, g_q, s->d_H);
    AH_LAUNCHED();
  }
  hipLaunchKernelGGL(k_hhat<B>, dim3((unsigned)cdiv(n, 128)), dim3(128), 0, st, s->nfree, s->d_Dinv, s->d_H,
                     s->d_Hhat);
  AH_LAUNCHED();
  return AH_OK;
}

static ah_status rhs_dispatch(int b, ah_system* s, const double* g_q, hipStream_t st) {
  switch (b) {
    case 2: return rhs_from_neumann<2>(s, g_q, st);
    case 3: return rhs_from_neumann<3>(s, g_q, st);
    case 4: return rhs_from_neumann<4>(s, g_q, st);
    case 6: return rhs_from_neumann<6>(s, g_q, st);
    case 10: return rhs_from_neumann<10>(s, g_q, st);
  }
  set_error("unsupported facet block size %d", b);
  return AH_EUNSUPPORTED;
}

static ah_status scale_dispatch(int b, ah_system* s, const ah_mesh* m, const double* Dg, Arena& parts,
                                hipStream_t st, int* d_err) {
  const int D = m->D;
  if (D == 2 && b == 2) return scale_to_csr<2, 2>(s, m, Dg, parts, st, d_err);
  if (D == 2 && b == 3) return scale_to_csr<2, 3>(s, m, Dg, parts, st, d_err);
  if (D == 2 && b == 4) return scale_to_csr<2, 4>(s, m, Dg, parts, st, d_err);
  if (D == 3 && b == 3) return scale_to_csr<3, 3>(s, m, Dg, parts, st, d_err);
  if (D == 3 && b == 6) return scale_to_csr<3, 6>(s, m, Dg, parts, st, d_err);
  if (D == 3 && b == 10) return scale_to_csr<3, 10>(s, m, Dg, parts, st, d_err);
  set_error("unsupported facet block size %d", b);
  return AH_EUNSUPPORTED;
}

static void fill_common(ElemArgs& a, const ah_mesh* m, const RefTables& t) {
  a.ne = m->ne;
  a.vert = m->d_vert;
  a.cell = m->d_cell;
  a.elem_facet = m->d_elem_facet;
  a.facet_loc = m->d_facet_loc;
  a.kind = m->d_kind;
  a.bf_index = m->d_bf_index;
  a.free_rank = m->d_free_rank;
  a.elem_slot = m->d_elem_slot;
  a.vol_w = t.d_vol_w;
  a.vol_lam = t.d_vol_lam;
  a.vol_phi = t.d_vol_phi;
  a.vol_dphi = t.d_vol_dphi;
  a.fac_w = t.d_fac_w;
  a.fac_mu = t.d_fac_mu;
  a.fac_psi = t.d_fac_psi;
  a.fac_proj = t.d_fac_proj;
  a.fac_pp = t.d_fac_pp;
  a.fac_mass = t.d_fac_mass;
  a.ten_adv = t.d_ten_adv;
  a.ten_dif = t.d_ten_dif;
  a.ten_dn = t.d_ten_dn;
  for (int i = 0; i < t.nu; ++i) {
    int at = 0;
    for (int c = t.D - 1; c >= 0; --c) at = at * (t.p + 1) + t.node[i * t.D + c];
    a.node[at] = (int8_t)i;
  }
  for (int m = 0; m < t.b; ++m)
    for (int c = 0; c < t.D; ++c) a.fnode[m][c] = (int8_t)t.fnode[m * t.D + c];
}

template <int D, int P>
static ah_status launch_grad(const ElemArgs& a, hipStream_t st) {
  if (a.ne == 0) return AH_OK;
  hipLaunchKernelGGL((k_grad<D, P>), dim3((unsigned)cdiv(a.ne, Sz<D, P>::EPB)), dim3(64), 0, st, a);
  AH_LAUNCHED();
  return AH_OK;
}

ah_status grad_dispatch(const ah_system* s, const double* a_vert, const double* lam_fwd, const double* lam_adj,
                        double* dJdf_q, double* dnu_elem, hipStream_t st) {
  ElemArgs a{};
  fill_common(a, s->mesh, *s->tab);
  a.a_vert = a_vert;
  a.nu = 1.0;
  a.alpha = s->alpha;
  a.lamD = s->d_lamD;
  a.Ainv = s->d_Ainv;
  a.Bm = s->d_Bm;
  a.Cm = s->d_Cm;
  a.Fv = s->d_Fv;
  a.lam_fwd = lam_fwd;
  a.lam_adj = lam_adj;
  a.dJdf_q = dJdf_q;
  a.dnu_elem = dnu_elem;
  int* err = nullptr;
  Arena tmp;
  tmp.stream = st;
  AH_TRY(tmp.get(&err, 1));
  a.err = err;
  ah_status rc;
  const int D = s->D, p = s->p;
  if (D == 2 && p == 1) rc = launch_grad<2, 1>(a, st);
  else if (D == 2 && p == 2) rc = launch_grad<2, 2>(a, st);
  else if (D == 2 && p == 3) rc = launch_grad<2, 3>(a, st);
  else if (D == 3 && p == 1) rc = launch_grad<3, 1>(a, st);
  else if (D == 3 && p == 2) rc = launch_grad<3, 2>(a, st);
  else if (D == 3 && p == 3) rc = launch_grad<3, 3>(a, st);
  else { set_error("unsupported dim_st/p"); rc = AH_EUNSUPPORTED; }
  tmp.release();
  return rc;
}

}  // namespace ah

using namespace ah;

extern "C" ah_status ah_quad_points(const ah_mesh* mc, int p, double* xq_elem, double* xq_bfacet, void* stream) {
  if (!mc) { set_error("null mesh"); return AH_EINVAL; }
  ah_mesh* m = const_cast<ah_mesh*>(mc);
  hipStream_t st = as_stream(stream);
  Arena tmp;
  tmp.stream = st;
  std::shared_ptr<const RefTables> tab;
  AH_TRY(ref_tables(m->D, p, tmp, tab));
  const RefTables& t = *tab;
  double* d_vert = nullptr;
  int32_t *d_cell = nullptr, *d_bf = nullptr, *d_fv = nullptr;
  AH_TRY(tmp.get(&d_vert, m->vert.size()));
  AH_TRY(tmp.get(&d_cell, m->cell.size()));
  AH_TRY(tmp.get(&d_bf, m->bfacets.size()));
  AH_TRY(tmp.get(&d_fv, m->facet_vert.size()));
  AH_HIP(hipMemcpyAsync(d_vert, m->vert.data(), m->vert.size() * 8, hipMemcpyHostToDevice, st));
  AH_HIP(hipMemcpyAsync(d_cell, m->cell.data(), m->cell.size() * 4, hipMemcpyHostToDevice, st));
  AH_HIP(hipMemcpyAsync(d_bf, m->bfacets.data(), m->bfacets.size() * 4, hipMemcpyHostToDevice, st));
  AH_HIP(hipMemcpyAsync(d_fv, m->facet_vert.data(), m->facet_vert.size() * 4, hipMemcpyHostToDevice, st));
  if (xq_elem && m->ne) {
    hipLaunchKernelGGL(k_quad_points_elem, dim3(cdiv(m->ne * t.nq, 256)), dim3(256), 0, st, m->ne, m->D, t.nq, d_vert,
                       d_cell, t.d_vol_lam, xq_elem);
    AH_LAUNCHED();
  }
  if (xq_bfacet && m->nbf) {
    hipLaunchKernelGGL(k_quad_points_bfacet, dim3(cdiv(m->nbf * t.nqf, 256)), dim3(256), 0, st, m->nbf, m->D, t.nqf,
                       d_vert, d_bf, d_fv, t.d_fac_mu, xq_bfacet);
    AH_LAUNCHED();
  }
  AH_HIP(hipStreamSynchronize(st));
  tmp.release();
  return AH_OK;
}

static ah_status assemble_impl(const ah_mesh* mc, const ah_hdg_params* prm, double nu, const double* a_vert,
                               const double* a_qe, const double* a_qf, const double* f_q, const double* g_q,
                               void* stream, ah_system** out) {
  if (!(nu >= 0.0) || !std::isfinite(nu)) { set_error("hdg_assemble: nu must be finite and >= 0"); return AH_EINVAL; }
  if (!mc->bc_set) { set_error("hdg_assemble: boundary kinds not set"); return AH_EINVAL; }
  *out = nullptr;
  ah_mesh* m = const_cast<ah_mesh*>(mc);
  hipStream_t st = as_stream(stream);
  AH_TRY(mesh_upload(m, st));
  ah_system* s = new ah_system();
  s->arena.stream = st;
  s->mesh = m;
  s->D = m->D;
  s->p = prm->p;
  s->visc = nu;
  s->alpha = prm->alpha > 0.0 ? prm->alpha : 10.0 * prm->p * prm->p;
  s->keep = prm->keep_element_data != 0;
  s->unscaled = prm->no_block_scale != 0;
  auto fail = [&](ah_status code) { delete s; return code; };
  ah_status rc = ref_tables(m->D, prm->p, s->arena, s->tab);
  if (rc) return fail(rc);
  const RefTables& t = *s->tab;
  s->nu = t.nu; s->b = t.b; s->nl = (m->D + 1) * t.b; s->nq = t.nq; s->nqf = t.nqf;
  s->nfree = m->nfree;
  s->n = m->nfree * t.b;
  s->nnzb = (int64_t)m->bsr_col.size();
  Arena& ar = s->arena;
  if ((rc = ar.get(&s->d_bval, s->nnzb * t.b * t.b))) return fail(rc);
  if ((rc = ar.get(&s->d_H, s->n))) return fail(rc);
  if ((rc = ar.get(&s->d_H0, s->n))) return fail(rc);
  if ((rc = ar.get(&s->d_Hhat, s->n))) return fail(rc);
  if ((rc = ar.get(&s->d_Dinv, s->nfree * t.b * t.b))) return fail(rc);
  if ((rc = ar.get(&s->d_lamD, m->nf * t.b))) return fail(rc);
  if (s->keep) {
    if ((rc = ar.get(&s->d_Ainv, m->ne * t.nu * t.nu))) return fail(rc);
    if ((rc = ar.get(&s->d_Bm, m->ne * t.nu * s->nl))) return fail(rc);
    if ((rc = ar.get(&s->d_Cm, m->ne * s->nl * t.nu))) return fail(rc);
    if ((rc = ar.get(&s->d_Fv, m->ne * t.nu))) return fail(rc);
  }
  int* d_err = nullptr;
  if ((rc = ar.get(&d_err, 1))) return fail(rc);
  // the elements' parts of the diagonal blocks and of H, summed per facet and
  // then given back, before the matrix (which takes more) is allocated
  Arena tmp;
  tmp.stream = st;
  auto fail_tmp = [&](ah_status code) { tmp.release(); return fail(code); };
  double *Dg = nullptr, *Hk = nullptr;
  if ((rc = tmp.get(&Dg, m->ne * (m->D + 1) * t.b * t.b))) return fail_tmp(rc);
  if ((rc = tmp.get(&Hk, m->ne * s->nl))) return fail_tmp(rc);
  if (hipMemsetAsync(d_err, 0, sizeof(int), st) != hipSuccess ||
      (m->shared_pairs &&
       hipMemsetAsync(s->d_bval, 0, s->nnzb * t.b * t.b * sizeof(double), st) != hipSuccess) ||
      hipMemsetAsync(s->d_lamD, 0, m->nf * t.b * sizeof(double), st) != hipSuccess) {
    set_error("hdg_assemble: memset failed");
    return fail_tmp(AH_EHIP);
  }
  ElemArgs a{};
  fill_common(a, m, t);
  a.a_vert = a_vert;
  a.a_qe = a_qe;
  a.a_qf = a_qf;
  a.f_q = f_q;
  a.g_q = g_q;
  a.nu = nu;
  a.alpha = s->alpha;
  a.bval = s->d_bval;
  a.Dg = Dg;
  a.Hk = Hk;
  a.add_off = m->shared_pairs;
  a.lamD = s->d_lamD;
  a.Ainv = s->d_Ainv;
  a.Bm = s->d_Bm;
  a.Cm = s->d_Cm;
  a.Fv = s->d_Fv;
  a.err = d_err;
  if ((rc = element_dispatch(m->D, prm->p, a, st))) return fail_tmp(rc);
  if (s->n > 0)
    hipLaunchKernelGGL(k_h_sum, dim3((unsigned)cdiv(s->n, 256)), dim3(256), 0, st, s->n, t.b, m->d_facet_slot, Hk,
                       s->d_H0);
  if ((rc = scale_dispatch(t.b, s, m, Dg, tmp, st, d_err))) return fail_tmp(rc);
  if ((rc = rhs_dispatch(t.b, s, g_q, st))) return fail(rc);
  int herr = 0;
  if ((rc = read_bytes(d_err, &herr, sizeof(int), st))) return fail(rc);
  if (herr) {
    set_error("hdg_assemble: singular %s", (herr & 4) ? "facet diagonal block (characteristic facet at nu = 0?)"
                                                      : (herr & 2) ? "element (degenerate cell)" : "element block A_K");
    return fail(AH_ESINGULAR);
  }
  *out = s;
  return AH_OK;
}

extern "C" ah_status ah_quad_points_facets(const ah_mesh* mc, int p, double* xq_facet, void* stream) {
  if (!mc || !xq_facet) { set_error("ah_quad_points_facets: null argument"); return AH_EINVAL; }
  ah_mesh* m = const_cast<ah_mesh*>(mc);
  if (m->nf == 0) return AH_OK;
  hipStream_t st = as_stream(stream);
  Arena tmp;
  tmp.stream = st;
  std::shared_ptr<const RefTables> tab;
  AH_TRY(ref_tables(m->D, p, tmp, tab));
  const RefTables& t = *tab;
  std::vector<int32_t> ids((size_t)m->nf);
  for (int64_t f = 0; f < m->nf; ++f) ids[(size_t)f] = (int32_t)f;
  double* d_vert = nullptr;
  int32_t *d_ids = nullptr, *d_fv = nullptr;
  AH_TRY(tmp.get(&d_vert, m->vert.size()));
  AH_TRY(tmp.get(&d_ids, ids.size()));
  AH_TRY(tmp.get(&d_fv, m->facet_vert.size()));
  AH_HIP(hipMemcpyAsync(d_vert, m->vert.data(), m->vert.size() * 8, hipMemcpyHostToDevice, st));
  AH_HIP(hipMemcpyAsync(d_ids, ids.data(), ids.size() * 4, hipMemcpyHostToDevice, st));
  AH_HIP(hipMemcpyAsync(d_fv, m->facet_vert.data(), m->facet_vert.size() * 4, hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(k_quad_points_bfacet, dim3(cdiv(m->nf * t.nqf, 256)), dim3(256), 0, st, m->nf, m->D, t.nqf,
                     d_vert, d_ids, d_fv, t.d_fac_mu, xq_facet);
  AH_LAUNCHED();
  AH_HIP(hipStreamSynchronize(st));
  tmp.release();
  return AH_OK;
}

extern "C" ah_status hdg_assemble(const ah_mesh* mc, const ah_hdg_params* prm, double nu, const double* a_vert,
                                  const double* f_q, const double* g_q, void* stream, ah_system** out) {
  if (!mc || !prm || !out || !a_vert) { set_error("hdg_assemble: null argument"); return AH_EINVAL; }
  return assemble_impl(mc, prm, nu, a_vert, nullptr, nullptr, f_q, g_q, stream, out);
}

extern "C" ah_status hdg_assemble_q(const ah_mesh* mc, const ah_hdg_params* prm, double nu, const double* a_qe,
                                    const double* a_qf, const double* f_q, const double* g_q, void* stream,
                                    ah_system** out) {
  if (!mc || !prm || !out || !a_qe || !a_qf) { set_error("hdg_assemble_q: null argument"); return AH_EINVAL; }
  return assemble_impl(mc, prm, nu, nullptr, a_qe, a_qf, f_q, g_q, stream, out);
}

extern "C" ah_status hdg_update_neumann(ah_system* s, const double* g_q, void* stream) {
  if (!s) { set_error("hdg_update_neumann: null system"); return AH_EINVAL; }
  return rhs_dispatch(s->b, s, g_q, as_stream(stream));
}

extern "C" void ah_system_destroy(ah_system* s) { delete s; }

extern "C" ah_status ah_system_sizes(const ah_system* s, int64_t* n, int* b, int64_t* nnz) {
  if (!s) { set_error("null system"); return AH_EINVAL; }
  if (n) *n = s->n;
  if (b) *b = s->b;
  if (nnz) *nnz = s->nnz;
  return AH_OK;
}

extern "C" ah_status ah_system_export(const ah_system* s, int64_t* row_ptr, int32_t* col, double* val,
                                      double* h_hat, double* dinv, double* lam_dir, void* stream) {
  if (!s) { set_error("null system"); return AH_EINVAL; }
  hipStream_t st = as_stream(stream);
  if (row_ptr) AH_HIP(hipMemcpyAsync(row_ptr, s->d_rowptr, (s->n + 1) * 8, hipMemcpyDeviceToDevice, st));
  if (col) AH_HIP(hipMemcpyAsync(col, s->d_col, s->nnz * 4, hipMemcpyDeviceToDevice, st));
  if (val) AH_HIP(hipMemcpyAsync(val, s->d_val, s->nnz * 8, hipMemcpyDeviceToDevice, st));
  if (h_hat) AH_HIP(hipMemcpyAsync(h_hat, s->d_Hhat, s->n * 8, hipMemcpyDeviceToDevice, st));
  if (dinv) AH_HIP(hipMemcpyAsync(dinv, s->d_Dinv, s->nfree * s->b * s->b * 8, hipMemcpyDeviceToDevice, st));
  if (lam_dir) AH_HIP(hipMemcpyAsync(lam_dir, s->d_lamD, s->mesh->nf * s->b * 8, hipMemcpyDeviceToDevice, st));
  return AH_OK;
}
