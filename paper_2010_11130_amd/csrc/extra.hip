// Reconstruction of the element unknowns (Section 2.5), slab coupling
// (Section 2.4), adjoint gradients with respect to the source and nu, and
// Gaussian source fields.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "system.h"

namespace ah {

struct ElemTables;

// Full facet trace of element e's facets: free DOFs from lam (free numbering),
// Dirichlet facets from lamD (or zero when dir_zero).
__device__ inline double trace_at(const int32_t* free_rank, const double* lam, const double* lamD, int f, int m,
                                  int b, bool dir_zero) {
  int fr = free_rank[f];
  if (fr >= 0) return lam[(int64_t)fr * b + m];
  return dir_zero ? 0.0 : lamD[(int64_t)f * b + m];
}

// U_K = A_K^-1 (F_K - B_K Lambda_K): values at the element lattice (nodal basis).
__global__ void k_reconstruct(int64_t ne, int D, int nu, int b, const int32_t* __restrict__ elem_facet,
                              const int32_t* __restrict__ free_rank, const double* __restrict__ lam,
                              const double* __restrict__ lamD, const double* __restrict__ Ainv,
                              const double* __restrict__ Bm, const double* __restrict__ Fv,
                              double* __restrict__ U) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne) return;
  const int nl = (D + 1) * b;
  double L[40], r[20];
  for (int lf = 0; lf <= D; ++lf) {
    int f = elem_facet[e * (D + 1) + lf];
    for (int m = 0; m < b; ++m) L[lf * b + m] = trace_at(free_rank, lam, lamD, f, m, b, false);
  }
  for (int i = 0; i < nu; ++i) {
    double s = Fv[e * nu + i];
    for (int c = 0; c < nl; ++c) s -= Bm[(e * nu + i) * nl + c] * L[c];
    r[i] = s;
  }
  for (int i = 0; i < nu; ++i) {
    double s = 0.0;
    for (int k = 0; k < nu; ++k) s += Ainv[(e * nu + i) * nu + k] * r[k];
    U[e * nu + i] = s;
  }
}

// Inflow data of the next slab: g at the facet points = previous trace.
struct FacetLattice {
  int8_t beta[10][3];
};

__global__ void k_inflow(int64_t npair, int D, int p, int b, int nqf, const int32_t* __restrict__ pair,
                         const uint8_t* __restrict__ perm, const double* __restrict__ fac_mu,
                         const int32_t* __restrict__ src_free_rank, const double* __restrict__ lam_prev,
                         const double* __restrict__ lamD_prev, FacetLattice lat, double* __restrict__ g) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= npair * nqf) return;
  int64_t k = idx / nqf;
  int q = (int)(idx % nqf);
  int bi = pair[2 * k], f = pair[2 * k + 1];
  double mu[3] = {0, 0, 0};
  for (int s = 0; s < D; ++s) mu[perm[k * D + s]] = fac_mu[q * D + s];
  double v = 0.0;
  for (int m = 0; m < b; ++m) {
    double psi = 1.0;
    for (int s = 0; s < D; ++s)
      for (int j = 0; j < lat.beta[m][s]; ++j) psi *= (p * mu[s] - j) / (j + 1.0);
    v += psi * trace_at(src_free_rank, lam_prev, lamD_prev, f, m, b, false);
  }
  g[(int64_t)bi * nqf + q] = v;
}

template <class T>
__global__ void k_sum_partial(int64_t n, const T* __restrict__ x, double* __restrict__ partial) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) s += (double)x[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void k_sum_final(int nb, const double* __restrict__ partial, double* __restrict__ out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < nb; ++k) s += partial[k];
    *out = s;
  }
}

// 2^(j/32) rounded to double, and what the rounding left out.
__constant__ const double EXP_HI[32] = {
    0x1.0000000000000p+0, 0x1.059b0d3158574p+0, 0x1.0b5586cf9890fp+0, 0x1.11301d0125b51p+0,
    0x1.172b83c7d517bp+0, 0x1.1d4873168b9aap+0, 0x1.2387a6e756238p+0, 0x1.29e9df51fdee1p+0,
    0x1.306fe0a31b715p+0, 0x1.371a7373aa9cbp+0, 0x1.3dea64c123422p+0, 0x1.44e086061892dp+0,
    0x1.4bfdad5362a27p+0, 0x1.5342b569d4f82p+0, 0x1.5ab07dd485429p+0, 0x1.6247eb03a5585p+0,
    0x1.6a09e667f3bcdp+0, 0x1.71f75e8ec5f74p+0, 0x1.7a11473eb0187p+0, 0x1.82589994cce13p+0,
    0x1.8ace5422aa0dbp+0, 0x1.93737b0cdc5e5p+0, 0x1.9c49182a3f090p+0, 0x1.a5503b23e255dp+0,
    0x1.ae89f995ad3adp+0, 0x1.b7f76f2fb5e47p+0, 0x1.c199bdd85529cp+0, 0x1.cb720dcef9069p+0,
    0x1.d5818dcfba487p+0, 0x1.dfc97337b9b5fp+0, 0x1.ea4afa2a490dap+0, 0x1.f50765b6e4540p+0};
__constant__ const float EXP_LO[32] = {
    0.0f, 5.109225029e-17f, 8.551889706e-17f, -7.899853967e-17f, -3.046782080e-17f, 1.041027846e-16f,
    8.912812676e-17f, 3.829204837e-17f, 3.982015231e-17f, -7.712630693e-17f, 4.658027592e-17f, 2.667932131e-18f,
    2.538250279e-17f, -2.858731210e-17f, 7.700948380e-17f, -6.770511659e-17f, -9.667293313e-17f, -3.023758135e-17f,
    -3.483994557e-17f, -1.016455328e-16f, 7.949834810e-17f, -1.013691647e-17f, 2.470719257e-17f, -1.012567991e-16f,
    8.199010021e-17f, -1.851380418e-17f, 2.960140695e-17f, 1.822745843e-17f, 3.283107224e-17f, -6.122763413e-17f,
    -1.061994606e-16f, 8.960767791e-17f};

// exp(x) for x <= 0 (NaN stays NaN), by the table-driven method of P. T. P.
// Tang (ACM TOMS 15, 1989): x = (32 e + j) ln2/32 + r with |r| <= ln2/64,
// exp(x) = 2^e 2^(j/32) (1 + p(r)), p the Taylor series to r^6 (next term
// below 4e-18), the table with its rounding error, in LDS (its 32 doubles
// fill the 64 banks once).  14 FP64 operations instead of the general
// function's about 25.
__device__ inline double exp_neg(double x, const double* hi, const float* lo) {
  x = x < -746.0 ? -746.0 : x;   // 0 either way
  const double magic = 6755399441055744.0;   // 1.5 * 2^52: rounds to an integer in the low bits
  const double t = fma(x, 0x1.71547652b82fep+5, magic);
  const double k = t - magic;
  const int n = __double2loint(t);
  double r = fma(k, -0x1.62e42fefa39efp-6, x);   // exact: both are multiples of 2^-58
  r = fma(k, -0x1.abc9e3b39803fp-61, r);
  double q = fma(r, 1.0 / 720.0, 1.0 / 120.0);
  q = fma(r, q, 1.0 / 24.0);
  q = fma(r, q, 1.0 / 6.0);
  q = fma(r, q, 0.5);
  const double p = fma(r * r, q, r);
  const double h = hi[n & 31];
  return ldexp(h + fma(h, p, (double)lo[n & 31]), n >> 5);
}

__device__ inline void exp_table(double* hi, float* lo) {
  if (threadIdx.x < 32) {
    hi[threadIdx.x] = EXP_HI[threadIdx.x];
    lo[threadIdx.x] = EXP_LO[threadIdx.x];
  }
  __syncthreads();
}

// -|x - X_k|^2 / (2 w^2)
template <int D>
__device__ inline double gauss_arg(const double* x, const double* __restrict__ c, double inv2w2) {
  double r2 = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) { const double d = x[a] - c[a]; r2 += d * d; }
  return -r2 * inv2w2;
}

// f(X) = sum_k c_k exp(-|X - X_k|^2 / (2 w^2)): S waves share 64 P points, each
// with every S-th centre, whose coordinates are wave-uniform (scalar) loads.
// Bound by the FP64 vector units: about 24 operations per (point, centre)
// pair against 8 (D + 1) bytes per point.  5.3M points x 256 centres: 1997 us
// with the general exponential and a point per thread, 1208 us now.
template <int D, int P, int S>
__global__ __launch_bounds__(256) void k_gauss(int64_t npts, const double* __restrict__ X, int K,
                                               const double* __restrict__ C, double inv2w2,
                                               const double* __restrict__ c, double* __restrict__ f) {
  __shared__ double hi[32];
  __shared__ float lo[32];
  __shared__ double red[S > 1 ? S * 64 * P : 1];
  exp_table(hi, lo);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = ((int64_t)blockIdx.x * (4 / S) + wv / S) * (64 * P) + lane;
  double x[P][D], s[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int64_t i = i0 + 64 * p;
    s[p] = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) x[p][a] = i < npts ? X[i * D + a] : 0.0;
  }
  for (int k = wv % S; k < K; k += S) {
    const double ck = c[k];
#pragma unroll
    for (int p = 0; p < P; ++p) s[p] = fma(ck, exp_neg(gauss_arg<D>(x[p], C + (int64_t)k * D, inv2w2), hi, lo), s[p]);
  }
  if (S > 1) {
#pragma unroll
    for (int p = 0; p < P; ++p) red[(wv * P + p) * 64 + lane] = s[p];
    __syncthreads();
    for (int t = threadIdx.x; t < 64 * P; t += 256) {
      const int64_t i = (int64_t)blockIdx.x * (64 * P) + t;
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < S; ++w) v += red[w * 64 * P + t];
      if (i < npts) f[i] = v;
    }
    return;
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (i0 + 64 * p < npts) f[i0 + 64 * p] = s[p];
}

// partial[blk][k] = sum over the block's 256 P points of y(X) phi_k(X), for
// the block's kc centres from blockIdx.y kc on (kc <= 64, a multiple of 8).
// A thread keeps its P points in registers and walks the centres eight at a
// time; the eight sums of a wave are reduced together, each exchange step
// halving the number of values a lane still carries (10 exchanges for eight
// sums, not 48).  Bound like k_gauss.  One centre per block row instead read
// X and y once per centre: 5567 us at 5.3M points x 256 centres (44 GB of
// cache reads, 7.9 TB/s), 1352 us now and 26 for the sums over blocks.
template <int D, int P>
__global__ __launch_bounds__(256) void k_gauss_t(int64_t npts, const double* __restrict__ X, int K,
                                                 const double* __restrict__ C, double inv2w2,
                                                 const double* __restrict__ y, double* __restrict__ partial, int kc) {
  __shared__ double hi[32];
  __shared__ float lo[32];
  __shared__ double red[4][64];
  exp_table(hi, lo);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * (256 * P) + threadIdx.x;
  double x[P][D], yv[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int64_t i = i0 + 256 * p;
    yv[p] = i < npts ? y[i] : 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) x[p][a] = i < npts ? X[i * D + a] : 0.0;
  }
  const int k0 = blockIdx.y * kc, k1 = min(K, k0 + kc);
  for (int kb = k0; kb < k1; kb += 8) {
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double* ck = C + (int64_t)min(kb + q, K - 1) * D;
      double s = 0.0;
#pragma unroll
      for (int p = 0; p < P; ++p) s = fma(yv[p], exp_neg(gauss_arg<D>(x[p], ck, inv2w2), hi, lo), s);
      v[q] = s;
    }
#pragma unroll
    for (int h = 4; h >= 1; h >>= 1) {
      const bool up = lane & (8 * h);
#pragma unroll
      for (int q = 0; q < h; ++q) {
        const double keep = up ? v[q + h] : v[q], send = up ? v[q] : v[q + h];
        v[q] = keep + __shfl_xor(send, 8 * h, 64);
      }
    }
    for (int o = 4; o > 0; o >>= 1) v[0] += __shfl_xor(v[0], o, 64);
    if ((lane & 7) == 0) red[wv][kb - k0 + (lane >> 3)] = v[0];
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < k1 - k0) partial[(int64_t)blockIdx.x * K + k0 + t] = red[0][t] + red[1][t] + red[2][t] + red[3][t];
}

// out[k] = sum over blocks of partial[blk][k] (add: on top of what is there),
// eight k per workgroup.
__global__ __launch_bounds__(256) void k_cols_sum(int K, int nblk, const double* __restrict__ partial,
                                                  double* __restrict__ out, int add) {
  __shared__ double red[256];
  const int k = blockIdx.x * 8 + (threadIdx.x & 7);
  double s = 0.0;
  if (k < K)
    for (int b = threadIdx.x >> 3; b < nblk; b += 32) s += partial[(int64_t)b * K + k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o >= 8; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x < 8 && k < K) out[k] = add ? out[k] + red[threadIdx.x] : red[threadIdx.x];
}

// A few points per SIMD make the kernels latency bound: from 2^19 points on
// a wave carries several points per lane (four forward, eight transposed, the
// centres' scalar loads and the reductions shared between them), below that
// four waves share the centres of 64 points.
constexpr int64_t GAUSS_MANY = (int64_t)1 << 19;

template <int D>
static void gauss_launch(int64_t npts, const double* X, int K, const double* C, double inv2w2, const double* c,
                         double* f, hipStream_t st) {
  if (npts >= GAUSS_MANY)
    hipLaunchKernelGGL((k_gauss<D, 4, 1>), dim3((unsigned)cdiv(npts, 1024)), dim3(256), 0, st, npts, X, K, C, inv2w2,
                       c, f);
  else
    hipLaunchKernelGGL((k_gauss<D, 1, 4>), dim3((unsigned)cdiv(npts, 64)), dim3(256), 0, st, npts, X, K, C, inv2w2,
                       c, f);
}

template <int D>
static ah_status gauss_t_launch(int64_t npts, const double* X, int K, const double* C, double inv2w2,
                                const double* y, double* dc, Arena& tmp, hipStream_t st) {
  const bool many = npts >= GAUSS_MANY;
  const int per = many ? 2048 : 256;   // points per block
  const int kc = many ? 64 : 8;
  // the points in pieces whose partial sums take at most 32 MB (or 256 per
  // centre): one piece up to 8.4M points with 1024 centres or fewer
  const int64_t most = std::max<int64_t>(256, std::min<int64_t>(4096, ((int64_t)1 << 22) / K));
  double* part = nullptr;
  AH_TRY(tmp.get(&part, (int64_t)K * std::min(most, std::max<int64_t>(1, cdiv(npts, per)))));
  int64_t i0 = 0;
  do {
    const int64_t m = std::min(npts - i0, most * per);
    const int nblk = (int)std::max<int64_t>(1, cdiv(m, per));
    const dim3 grid(nblk, (unsigned)cdiv(K, kc));
    if (many)
      hipLaunchKernelGGL((k_gauss_t<D, 8>), grid, dim3(256), 0, st, m, X + i0 * D, K, C, inv2w2, y + i0, part, kc);
    else
      hipLaunchKernelGGL((k_gauss_t<D, 1>), grid, dim3(256), 0, st, m, X + i0 * D, K, C, inv2w2, y + i0, part, kc);
    hipLaunchKernelGGL(k_cols_sum, dim3((unsigned)cdiv(K, 8)), dim3(256), 0, st, K, nblk, part, dc, (int)(i0 > 0));
    i0 += m;
  } while (i0 < npts);
  AH_LAUNCHED();
  return AH_OK;
}

ah_status grad_dispatch(const ah_system* s, const double* a_vert, const double* lam_fwd, const double* lam_adj,
                        double* dJdf_q, double* dnu_elem, hipStream_t st);

}  // namespace ah

using namespace ah;

extern "C" ah_status hdg_reconstruct(const ah_system* s, const double* lam, double* U, void* stream) {
  if (!s || !lam || !U) { set_error("hdg_reconstruct: null argument"); return AH_EINVAL; }
  if (!s->keep) { set_error("hdg_reconstruct: system assembled without keep_element_data"); return AH_EINVAL; }
  hipStream_t st = as_stream(stream);
  const ah_mesh* m = s->mesh;
  if (m->ne == 0) return AH_OK;
  hipLaunchKernelGGL(k_reconstruct, dim3((unsigned)cdiv(m->ne, 128)), dim3(128), 0, st, m->ne, s->D, s->nu, s->b,
                     m->d_elem_facet, m->d_free_rank, lam, s->d_lamD, s->d_Ainv, s->d_Bm, s->d_Fv, U);
  AH_LAUNCHED();
  return AH_OK;
}

extern "C" ah_status hdg_inflow_from_trace(const ah_system* prev, const double* lam_prev, ah_mesh* m,
                                           double* g_q_next, void* stream) {
  if (!prev || !lam_prev || !m || !g_q_next) { set_error("hdg_inflow_from_trace: null argument"); return AH_EINVAL; }
  if (prev->D != m->D) { set_error("hdg_inflow_from_trace: dimensions differ"); return AH_EINVAL; }
  hipStream_t st = as_stream(stream);
  AH_TRY(mesh_pair_time_planes(m, prev->mesh, st));
  if (m->npair == 0) return AH_OK;
  FacetLattice lat{};
  std::vector<int> idx;
  lattice(prev->D - 1, prev->p, idx);
  for (int k = 0; k < prev->b; ++k) {
    int s0 = prev->p;
    for (int a = 0; a < prev->D - 1; ++a) { lat.beta[k][a + 1] = (int8_t)idx[k * (prev->D - 1) + a]; s0 -= idx[k * (prev->D - 1) + a]; }
    lat.beta[k][0] = (int8_t)s0;
  }
  hipLaunchKernelGGL(k_inflow, dim3((unsigned)cdiv(m->npair * prev->nqf, 256)), dim3(256), 0, st, m->npair, prev->D,
                     prev->p, prev->b, prev->nqf, m->d_pair, m->d_pair_perm, prev->tab->d_fac_mu,
                     prev->mesh->d_free_rank, lam_prev, prev->d_lamD, lat, g_q_next);
  AH_LAUNCHED();
  return AH_OK;
}

extern "C" ah_status hdg_assemble_grad(const ah_system* s, const double* a_vert, const double* lam_fwd,
                                       const double* lam_adj, double* dJdf_q, double* dJdnu, void* stream) {
  if (!s || !lam_fwd || !lam_adj) { set_error("hdg_assemble_grad: null argument"); return AH_EINVAL; }
  if (!s->keep) { set_error("hdg_assemble_grad: system assembled without keep_element_data"); return AH_EINVAL; }
  hipStream_t st = as_stream(stream);
  const int64_t ne = s->mesh->ne;
  Arena tmp;
  tmp.stream = st;
  double* dnu_e = nullptr;
  AH_TRY(tmp.get(&dnu_e, std::max<int64_t>(ne, 1)));
  AH_TRY(grad_dispatch(s, a_vert, lam_fwd, lam_adj, dJdf_q, dnu_e, st));
  if (dJdnu) {
    const int nb = 256;
    double* part = nullptr;
    double* outd = nullptr;
    AH_TRY(tmp.get(&part, nb));
    AH_TRY(tmp.get(&outd, 1));
    hipLaunchKernelGGL(k_sum_partial<double>, dim3(nb), dim3(256), 0, st, ne, dnu_e, part);
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(64), 0, st, nb, part, outd);
    AH_LAUNCHED();
    AH_HIP(hipMemcpyAsync(dJdnu, outd, sizeof(double), hipMemcpyDeviceToHost, st));
  }
  AH_HIP(hipStreamSynchronize(st));
  tmp.release();
  return AH_OK;
}

extern "C" ah_status ah_source_gauss(int D, int64_t npts, const double* X, int K, const double* centers, double width,
                                     const double* c, double* f, void* stream) {
  if (!X || !centers || !c || !f || D < 1 || D > 3 || K < 0 || !(width > 0)) {
    set_error("ah_source_gauss: invalid arguments");
    return AH_EINVAL;
  }
  if (npts == 0) return AH_OK;
  hipStream_t st = as_stream(stream);
  const double s = 1.0 / (2.0 * width * width);
  if (D == 1) gauss_launch<1>(npts, X, K, centers, s, c, f, st);
  else if (D == 2) gauss_launch<2>(npts, X, K, centers, s, c, f, st);
  else gauss_launch<3>(npts, X, K, centers, s, c, f, st);
  AH_LAUNCHED();
  return AH_OK;
}

extern "C" ah_status ah_source_gauss_T(int D, int64_t npts, const double* X, int K, const double* centers,
                                       double width, const double* y, double* dc, void* stream) {
  if (!X || !centers || !y || !dc || D < 1 || D > 3 || K <= 0 || !(width > 0)) {
    set_error("ah_source_gauss_T: invalid arguments");
    return AH_EINVAL;
  }
  hipStream_t st = as_stream(stream);
  Arena tmp;
  tmp.stream = st;
  const double s = 1.0 / (2.0 * width * width);
  ah_status rc = D == 1 ? gauss_t_launch<1>(npts, X, K, centers, s, y, dc, tmp, st)
               : D == 2 ? gauss_t_launch<2>(npts, X, K, centers, s, y, dc, tmp, st)
                        : gauss_t_launch<3>(npts, X, K, centers, s, y, dc, tmp, st);
  if (rc < 0) { tmp.release(); return rc; }
  AH_HIP(hipStreamSynchronize(st));
  tmp.release();
  return AH_OK;
}
