// Library objects built on the device: the assembled facet system and the
// AIR hierarchy, plus device utilities shared by the kernels.
#pragma once

#include <initializer_list>

#include "common.h"

struct ah_system {
  ah_mesh* mesh = nullptr;
  int D = 0, p = 0, nu = 0, b = 0, nl = 0, nq = 0, nqf = 0;
  double visc = 0.0, alpha = 0.0;
  bool keep = false;
  bool unscaled = false;      // no facet-block scaling (S_hat = S, D_b^-1 = I)
  ah::Arena arena;
  std::shared_ptr<const ah::RefTables> tab;
  int64_t n = 0;        // free DOFs
  int64_t nfree = 0;    // free facets
  int64_t nnzb = 0;     // blocks of the free-facet pattern
  double* d_bval = nullptr;   // [nnzb][b][b] unscaled S
  double* d_H = nullptr;      // [n] unscaled H after Dirichlet elimination
  double* d_H0 = nullptr;     // [n] the same without the Neumann term
  double* d_Hhat = nullptr;   // [n]
  double* d_Dinv = nullptr;   // [nfree][b][b]
  double* d_lamD = nullptr;   // [nf][b]
  int64_t nnz = 0;            // scaled scalar CSR (level 0)
  int64_t* d_rowptr = nullptr;
  int32_t* d_col = nullptr;
  double* d_val = nullptr;
  // the same operator by off-diagonal facet blocks (scaled systems only; the
  // diagonal blocks of S_hat are the identity): block row R with nb blocks
  // holds [b][nb][b] values from (mesh odb_ptr[R]) b^2 on, so scalar row
  // R b + m is contiguous and its entry (s, c) has column b odb_col[.] + c
  double* d_odv = nullptr;    // [nnzb - nfree][b][b]
  // element data kept for reconstruction and the adjoint
  double* d_Ainv = nullptr;   // [ne][nu][nu]
  double* d_Bm = nullptr;     // [ne][nu][nl]
  double* d_Cm = nullptr;     // [ne][nl][nu]
  double* d_Fv = nullptr;     // [ne][nu]
  ~ah_system() { arena.release(); }
};

namespace ah {

// Choose the first level of the dense coarse end (at most end_max rows) and
// form the matrices that apply the cycle from there down (once per hierarchy).
void coarse_end_pick(ah_hier* h, int64_t end_max);
ah_status coarse_end_build(ah_hier* h, hipStream_t st);
// Flow order of the level-0 facet blocks for the ordered relaxations
// (Lemma 3.1): block levels, blocks and F rows grouped by level.
ah_status flow_order_build(ah_hier* h, hipStream_t st);

// Exclusive prefix sum of n int64 values into out[0..n] (out[n] = total).
ah_status scan_i64(const int64_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp);
// Same for int32 counts producing int64 offsets.
// (vmax, where given: the largest value on the device, at least 0)
ah_status scan_i32_to_i64(const int32_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp, int* vmax = nullptr);
// Read a few small device values (multiples of 4 bytes, at most 64 each) in
// stream order: one launch stores them into pinned host memory and sets a flag
// that the host polls, instead of a copy per value and a synchronization.
struct ReadItem {
  const void* dev;
  void* host;
  size_t bytes;
};
ah_status read_values(std::initializer_list<ReadItem> items, hipStream_t st);
// scan_i32_to_i64 (zero, where given: n values cleared on the way) and then
// read_values, one launch where one workgroup does the scan.
ah_status scan_i32_read(const int32_t* in, int64_t* out, int64_t n, hipStream_t st, Arena& tmp, int* vmax,
                        int32_t* zero, std::initializer_list<ReadItem> items);
ah_status read_i64(const int64_t* d, int64_t* h, hipStream_t st);
ah_status read_bytes(const void* d, void* h, size_t bytes, hipStream_t st);
// Wait until the pinned flag holds seq; AH_EHIP if the stream ends without it.
ah_status poll_flag(const unsigned long long* flag, unsigned long long seq, hipStream_t st);

constexpr int WAVE = 64;

}  // namespace ah

// Where one row of a coarse level read by full blocks sits in the sweep-ordered
// copy: the row's values from voff, its nb block columns from bcol[o0]; one
// 16-byte load per row.
struct alignas(16) AhRowRec {
  int64_t voff;
  int32_t o0;
  int32_t nb;
};

// One level of the AIR hierarchy (scalar CSR, int64 row offsets).
struct AhLevel {
  int64_t n = 0, nnz = 0;
  int64_t* rowptr = nullptr;
  int32_t* col = nullptr;
  double* val = nullptr;
  float* val32 = nullptr;
  double* diag = nullptr;
  float* diag32 = nullptr;
  // coarsening (all but the coarsest level)
  int64_t nc = 0;
  int64_t nF = 0, nnzF = 0;    // F rows and their stored entries
  int8_t* cf = nullptr;        // 1 = C, 0 = F
  int32_t* pcol = nullptr;     // one-point interpolation: coarse column or -1
  int32_t* clist = nullptr;    // fine index of each C point (coarse order)
  int32_t* flist = nullptr;    // fine index of each F point (increasing)
  // level 0 of a scaled system: the operator by off-diagonal facet blocks
  // (identity diagonal blocks), ob = block size, 0 where not available
  int ob = 0;
  bool fblk = false;           // F and C points are whole facet blocks (block AIR): block-row sweeps
  int64_t nov = 0;             // stored values (off-diagonal blocks * ob^2)
  int64_t novF = 0;            // of which in F rows
  const int64_t* optr = nullptr;
  const int32_t* ocol = nullptr;
  const double* oval = nullptr;
  float* oval32 = nullptr;
  // block AIR: a copy of that operator with its block rows in sweep order
  // (the F blocks, then the C blocks, each increasing): item k is block row
  // sperm[k], its blocks at soptr[k] .. soptr[k + 1] of socol / soval
  const int32_t* sperm = nullptr;
  const int64_t* soptr = nullptr;
  // scalar AIR: the values of the listed rows in sweep order instead (the F
  // rows, then the C rows), item k's row at rsoff[k] of soval / soval32
  const int64_t* rsoff = nullptr;
  const int32_t* socol = nullptr;
  const double* soval = nullptr;
  float* soval32 = nullptr;
  // block AIR, for sweeps that read the interpolated correction P e_c from
  // e_c itself (one-point P copies coarse blocks): per block o of the copy,
  // socp[o] the coarse block that P copies into column block socol[o] (-1:
  // none, zero) and soce[o] = the F item of an F column block (its values
  // kept compact), ~(its coarse block) for a C one; soown[k] the coarse
  // block P copies into item k's
  // own block row (-1: none; a C item k >= nbF is coarse block k - nbF, since
  // the C list is in coarse order)
  const int32_t* socp = nullptr;
  const int32_t* soce = nullptr;
  const int32_t* soown = nullptr;
  // the transposed operator in the same layout (adjoint cycle): block (I, J)
  // holds the transpose of block (J, I); null where the CSR A^T is used
  double* otval = nullptr;
  float* otval32 = nullptr;
  // a coarse level made of ob x ob blocks (level 1 under block AIR) read by
  // full blocks: block row R has bptr[R + 1] - bptr[R] blocks with column
  // blocks bcol[bptr[R] ..], row m's values at (m nb + s) bb + c from base
  // bvoff[R] of the CSR values (val / val32) where bvoff[R] >= 0, else from
  // ~bvoff[R] of baux / baux32 (zero-filled blocks); bb = 0 where not built
  int bb = 0;
  int blp = 0;                 // lanes per row of its sweeps (0: by precision)
  int64_t nbv = 0;             // stored values
  int64_t nbvF = 0;            // of which in F rows
  int64_t nbaux = 0;           // of which in the side array
  const int64_t* bptr = nullptr;
  const int32_t* bcol = nullptr;
  const int64_t* bvoff = nullptr;
  const double* baux = nullptr;
  float* baux32 = nullptr;
  // and its rows' values once more in sweep order (the F rows, then the C
  // rows, each in list order): item k's row at bsrec[k].voff of soval /
  // soval32, its block columns at bcol[bsrec[k].o0 ..], bsrec[k].nb of them
  const AhRowRec* bsrec = nullptr;
  // a coarse level swept from its point lists (no full-block view): its
  // rows' entries once more in sweep order (the F rows, then the C rows,
  // each in list order): item k's entries at coptr[k] .. coptr[k + 1] of
  // cocol / coval / coval32
  const int64_t* coptr = nullptr;
  const int32_t* cocol = nullptr;
  const double* coval = nullptr;
  float* coval32 = nullptr;
  // block AIR on level 0: R = [Z I] by coarse blocks, Z's b x b blocks (the
  // neighbourhood F blocks) with row m of coarse block k at
  // (rzptr[k] b + m nb) b, column blocks rzcol; null where not built
  const int64_t* rzptr = nullptr;
  const int32_t* rzcol = nullptr;
  const double* rzval = nullptr;
  float* rzval32 = nullptr;
  int64_t nrz = 0;             // stored values of Z
  int64_t nnzR = 0;
  int64_t* Rptr = nullptr;
  int32_t* Rcol = nullptr;
  double* Rval = nullptr;
  float* Rval32 = nullptr;
  // transposes for the adjoint cycle
  int64_t* ATptr = nullptr;
  int32_t* ATcol = nullptr;
  double* ATval = nullptr;
  float* ATval32 = nullptr;
  int64_t* RTptr = nullptr;    // R^T: rows = fine points
  int32_t* RTcol = nullptr;
  double* RTval = nullptr;
  float* RTval32 = nullptr;
  int64_t* PTptr = nullptr;    // P^T: rows = coarse points, entries = fine points (weight 1)
  int64_t nnzP = 0;
  int32_t* PTcol = nullptr;
  // cycle work vectors; e receives the level's correction from the finer
  // level's recursion, so it never aliases the sweep buffers x and y
  double* b = nullptr;
  double* x = nullptr;
  double* y = nullptr;
  double* e = nullptr;
  float* b32 = nullptr;
  float* x32 = nullptr;
  float* y32 = nullptr;
  float* e32 = nullptr;
};

struct ah_hier {
  const ah_system* sys = nullptr;
  // the coarse end: from level end0 down the cycle is one dense matrix, row i
  // of it at end_mat + i n (end_mat_t: of its transpose, adjoint hierarchies);
  // on the coarsest level that is the inverse
  int end0 = 0;
  const double* end_mat = nullptr;
  const double* end_mat_t = nullptr;
  int g0 = 0;                  // lanes per row of the level-0 kernels (0: from the mean row length)
  int fbb = 1;                 // level-0 kernels by facet block rows where the rows are whole blocks
  bool poll = true;            // FGMRES scalars by a polled flag (else by copies)
  int lpb = 0;                 // lanes per block row of those (0: from the mean blocks per row)
  // FGMRES uses delayed CGS2 from this many unknowns on: two passes over the
  // basis per iteration instead of four, but a host round trip between them.
  // ms per solve with CGS2 and with the delayed form (same iterations): slabs at
  // p = 2, 0.34M 2.49 and 2.58, 0.77M 5.00 and 5.08, 1.4M 9.66 and 9.49; cubes at
  // p = 1, scalar AIR, 0.29M 4.80 and 4.67, 0.63M 9.11 and 8.71, 2.0M 26.2 and
  // 23.4; block AIR, 0.97M 9.84 and 9.29, 2.0M 19.4 and 17.4, 3.1M 32.4 and 27.8.
  // So the line stands above the place where the two meet (0.3M to 1M).
  int64_t dcgs_min = (int64_t)1 << 21;
  int gc = 0;                  // lanes per row of the coarse-level kernels (0: from the mean row length)
  int64_t list_min = (int64_t)1 << 16;   // coarse levels from this many rows on sweep their F and C lists
  ah::Arena arena;
  ah_air_params prm{};
  std::vector<AhLevel> lev;
  double* cinv = nullptr;      // dense inverse of the coarsest matrix [nL][nL]
  int64_t nfallback = 0;
  // flow order of the level-0 facet blocks (ordered relaxations): level k
  // holds the blocks ord[ord_lptr[k] .. ord_lptr[k+1]) and the F rows
  // ord_frows[ord_lptrF[k] .. ord_lptrF[k+1])
  int32_t* ord = nullptr;
  int32_t* ord_level = nullptr;  // [blocks] level of each block
  int32_t* ord_frows = nullptr;
  int32_t* ord_cols = nullptr;   // level-0 block columns, ~J where J is on the row's level
  // per position of ord / ord_frows: {block or row, first value slot of the
  // block row, its number of blocks, 0}, so a sweep reads one record per row
  // before its values
  int4* ord_info = nullptr;
  int4* ord_finfo = nullptr;
  std::vector<int64_t> ord_lptr, ord_lptrF;
  int ord_breaks = 0;            // rounds that broke a cycle
  // FGMRES workspace (allocated on first solve)
  int m_alloc = 0;
  double* V = nullptr;         // [(m+1)][n]
  double* Z = nullptr;         // [m][n] (FP64 cycle)
  float* Z32 = nullptr;        // [m][n] (FP32 cycle)
  double* w = nullptr;
  double* r = nullptr;
  double* bhat = nullptr;
  double* bcg = nullptr;       // BiCGSTAB vectors [8][n] (allocated on first use)
  float* bcg32 = nullptr;      // FP32 cycle output [n]
  double* partial = nullptr;   // reduction partials
  double* hdev = nullptr;      // [4 (m+3)] device scalars
  ~ah_hier();
};
