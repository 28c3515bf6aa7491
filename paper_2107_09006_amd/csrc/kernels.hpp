// Device-side data of a handle and the host launchers of every kernel.
#pragma once

#include "internal.hpp"

namespace lsq2l {

struct DevMatrix {            // A and its transpose (device copies owned by the handle)
  int32_t m = 0, n = 0;
  int64_t nnz = 0;
  int32_t* rowptr = nullptr;  // m + 1
  int32_t* colind = nullptr;  // nnz
  double* vals = nullptr;     // nnz
  int32_t* trowptr = nullptr; // n + 1
  int32_t* trow = nullptr;    // nnz
  double* tvals = nullptr;    // nnz
  int32_t* tperm = nullptr;   // nnz: A^T entry k is vals[tperm[k]]
  int spmv_group = 0;         // A x: 0 row blocks through LDS, else lanes per row
  int spmvt_group = 0;        // A^T y, the same
  int32_t* blk = nullptr;     // LDS row blocks of A (spmv_blocks(nnz) + 1)
  int32_t* tblk = nullptr;    // the same for A^T
};

struct DevPlan {              // subdomain layout (device copies of HostPlan)
  SubDesc* subs = nullptr;
  int32_t* omega = nullptr;
  int32_t* xi = nullptr;
  int32_t* part = nullptr;
  int32_t* locown = nullptr;
  int32_t* tileF = nullptr;
  int64_t* tileOff = nullptr;
  int32_t* own_ptr = nullptr;
  int32_t* own_pos = nullptr;
  SubDesc* subs_ord = nullptr;     // subs by decreasing stored factor tiles: launches with
                                   // one workgroup per subdomain start the largest first
  int max_np = 0;             // largest padded local size
  int min_nG = 0, max_nG = 0;  // least and largest interface size
  // layout of the solve factor only: where each position lives in the local
  // vectors (loc index, -1 on padding; null: loc_off + position), and
  // scratch local vectors for the subdomains solved in global memory
  int32_t* sperm = nullptr;
  double* yscratch = nullptr;
  const SubDesc* heavy() const { return subs_ord ? subs_ord : subs; }
};

constexpr int SOLVE_DPACK = 640;      // entries of a packed diagonal inverse
constexpr int SOLVE_FAR_INTS = 14;    // entries of SolveStream::far0 per subdomain
// What the local solves read (k_solve.hip): the streams of both sweeps and
// the packed diagonal inverses, in the type of the factors, with their tables
struct SolveStream {
  int cap = 0;                            // largest padded subdomain that they solve (0: none are there)
  void *fwd = nullptr, *bwd = nullptr;    // as many entries as the factor's envelope, and a tile
  void* dpack = nullptr;                  // SOLVE_DPACK entries per diagonal tile
  uint16_t* nfar[2] = {nullptr, nullptr}; // slabs of every step (tile_base + step)
  int32_t* pos[2] = {nullptr, nullptr};   // per tile and group of eight: its slab, -1: none
  int32_t* desc[2] = {nullptr, nullptr};  // per slab: its group of eight
  int32_t* far0 = nullptr;                // per subdomain and sweep: first slab of each helper, count
  int32_t* scol = nullptr;                // per position: global column (-1: padding)
  double* sscale = nullptr;               // and its scaling
};

struct DevCoarse {            // coarse space and coarse operator
  PairDesc* pairs = nullptr;
  int32_t* pair_rows = nullptr;   // (pos in Xi_i, pos in Xi_j) per shared row
  SegDesc* segs = nullptr;
  int32_t* eF = nullptr;          // envelope of E (tile rows, global coarse numbering)
  int64_t* eOff = nullptr;
  int32_t* e_seg_of_tile = nullptr;
  int32_t* erows = nullptr;       // per tile column K: tile rows I > K with F(I) <= K
  int64_t* eptr = nullptr;
  int32_t* einv_bin_ptr = nullptr;   // per workgroup of the inverse: its column blocks
  int32_t* einv_bin_cols = nullptr;
  int4* e_items = nullptr;        // (pair, row block, column block) work items of E
  double* e_part = nullptr;       // row partials of the symmetric coarse solve
  double* e_u = nullptr;          // column partials of the symmetric coarse solve, per chunk
  int4* e_chunks = nullptr;       // (tile column, first row tile, row tiles) per chunk
  int32_t* e_chunk_ptr = nullptr; // chunks of each tile column
  int e_nchunks = 0;
};

// row tiles per chunk of the symmetric coarse solve (one row per thread of
// a 256-thread workgroup)
constexpr int ESYM_ROWTILES = 8;

// --- device transpose of A (hand-written radix sort) ------------------------
size_t transpose_temp_bytes(int64_t nnz, int32_t n);   // 24 bytes per entry (16 with one pass), and the histogram
size_t transpose_temp_least(int64_t nnz, int32_t n);   // 8 bytes per entry (0 with one pass), and the histogram
void launch_permute_rows(hipStream_t st, int32_t m, const int32_t* perm, const int32_t* rowptr,
                         const int32_t* colind, const double* vals, const int32_t* prowptr,
                         int32_t* pcolind, double* pvals);
// trowptr (n + 1), trow and tperm (nnz) written; tvals written if not null
// (vals must then be given); temp holds transpose_temp_bytes(nnz, n) bytes, or
// fewer, down to transpose_temp_least(nnz, n)
hipError_t launch_transpose(hipStream_t st, int32_t m, int32_t n, int64_t nnz, const int32_t* rowptr,
                            const int32_t* colind, const double* vals, int32_t* trowptr,
                            int32_t* trow, double* tvals, int32_t* tperm, void* temp,
                            size_t temp_bytes);
// one instance of the input of a (batched) setup, with its first row,
// column and entry in the concatenation
struct InstDesc {
  const int64_t* rowptr;
  const int32_t* colind;
  const double* vals;
  int64_t m, n, nnz, r0, c0, e0;
};
enum { CSR_FIRST = 0, CSR_LAST, CSR_MONO, CSR_RANGE, CSR_ORDER, CSR_KINDS };
// the concatenated, checked CSR of all S instances (see k_concat_rows):
// rp (M + 1), ci and vals (NNZ), bad (CSR_KINDS smallest failing rows)
void launch_concat(hipStream_t st, int S, const InstDesc* d, int64_t M, int64_t NNZ, int32_t* rp,
                   int32_t* ci, double* vals, unsigned long long* bad);
// flag (one int32, device) = 1 if a column index lies outside [0, n)
void launch_check_cols(hipStream_t st, int64_t nnz, const int32_t* colind, int32_t n, int32_t* flag);

// --- sparse kernels -------------------------------------------------------
// group 0: row blocks staged through LDS (needs the block table blk of the
// matrix, else one lane per row), their loads streaming if the matrix is
// larger than the last-level cache; SPMV_ROWS_CACHED / SPMV_ROWS_STREAM: row
// blocks with cached / streaming loads; 1 .. 64: lanes per row
enum { SPMV_ROWS_CACHED = -1, SPMV_ROWS_STREAM = -2 };
void launch_spmv(hipStream_t st, int32_t nrows, const int32_t* rowptr, const int32_t* colind,
                 const double* vals, const double* x, double* y, int group, int64_t nnz,
                 const int32_t* blk,
                 const int32_t* place = nullptr);
void launch_gather(hipStream_t st, int64_t n, const int32_t* perm, const double* in, double* out);
// the LDS row blocks of a CSR matrix: spmv_blocks(nnz) blocks, described by
// a table of spmv_table_len(nnz) int32 (first row and its start, per block)
int64_t spmv_blocks(int64_t nnz);
int64_t spmv_table_len(int64_t nnz);
void launch_row_blocks(hipStream_t st, int32_t nrows, const int32_t* rowptr, int64_t nnz, int32_t* blk);
void launch_grad_vals(hipStream_t st, int32_t m, const int32_t* rowptr, const int32_t* colind,
                      const double* r, const double* lam, const double* Alam, const double* x,
                      double* out);

// --- vector / reduction kernels --------------------------------------------
constexpr int RED_BLOCKS = 256;   // most partial sums per segment
constexpr int RED_TOTAL = 8192;   // workgroups of a reduction beyond which the chunks grow
constexpr int MDOT_BLOCKS = 64;   // most chunks per segment of the Gram-Schmidt products
// counters of the workgroups of a segment: one per COUNT_GROUP of them and
// one for the groups, COUNT_STRIDE int32 apart (128 bytes)
constexpr int COUNT_GROUP = 16, COUNT_STRIDE = 32;
constexpr int COUNT_LEN = (1 + RED_BLOCKS / COUNT_GROUP) * COUNT_STRIDE;
// A workgroup's part of a concatenated vector: len elements from lo, chunk k of
// the n chunks of instance seg; slot: its counters, where n > 1
struct Chunk {
  int64_t lo;
  int32_t len, seg, k, n, slot, unused;
};
struct Chunks {
  const Chunk* c = nullptr;   // device table
  int32_t n = 0;
};
// The instances' parts of a concatenated vector (device offsets) and their cuts:
// into chunks of a reduction, into pieces of 1,024 elements, and into chunks of
// the Gram-Schmidt products.  Every instance has at least one of each.
struct Segments {
  const int64_t* ptr;
  int S;
  Chunks red, fine, mdot;
};
enum ScalarOp { OP_R0 = 0, OP_RHO_INIT = 1, OP_ALPHA = 2, OP_RNORM = 3, OP_BETA = 4, OP_SUM = 5,
                LSQR_INIT_BETA = 8, LSQR_INIT_ALPHA = 9, LSQR_BETA = 10, LSQR_ALPHA = 11 };
struct Scalars {
  double *rho, *alpha, *beta, *rn2, *r0n2, *pq;
  int32_t* done;      // 0 active, 1 converged, 2 breakdown
  int32_t* its;       // iterations of each instance (x updated while active)
  int32_t* h_done;    // pinned host copy of done, written by every OP_RNORM
};
// LSQR: per-instance scalars, LSQR_NSC per instance
enum LsqrSc { LS_ALPHA = 0, LS_BETA, LS_RHOBAR, LS_PHIBAR, LS_ANORM2, LS_T1, LS_T2, LS_TEST,
              LS_RNORM0, LS_NSC };
constexpr int LSQR_NSC = LS_NSC;
// What a reduction does with its sums (per segment): op, and its operands.
// partial holds 2 RED_BLOCKS doubles per segment; count COUNT_LEN int32 per
// slot (segment of more than one chunk), zero between launches.
struct Reduction {
  int op;
  int two;            // the pass forms two sums
  double tol;         // OP_RNORM: squared tolerance; LSQR_ALPHA: tolerance
  double* partial;
  int32_t* count;
  double* out;        // OP_SUM
  double* lsqr;       // LSQR scalars
  Scalars sc;
};
// the vectors of a pass (see k_reduce)
enum { RED_DOT = 0, RED_DOT2, RED_COPY, RED_START, RED_SUB, RED_AXPY, RED_LSQR };
struct RedVec {
  const double *a = nullptr, *b = nullptr, *c = nullptr;
  double *o = nullptr, *o2 = nullptr, *keep = nullptr;
  int first = 0;
};
// the chunks of the segments seg (host offsets): size elements, at most most per segment
std::vector<Chunk> make_chunks(const std::vector<int64_t>& seg, int64_t size, int64_t most);
int64_t reduction_chunk(int64_t total);   // size of a reduction's over a vector of that length
void launch_reduce(hipStream_t st, int kind, const Segments& G, const RedVec& V, const Reduction& R);
void launch_xpby(hipStream_t st, const Segments& G, const double* beta, const double* z, double* p);
void launch_sub(hipStream_t st, int64_t n, const double* a, const double* b, double* out);
void launch_add(hipStream_t st, int64_t n, const double* a, const double* b, double* out);
void launch_fill(hipStream_t st, int64_t n, double v, double* out);
void launch_copy(hipStream_t st, int64_t n, const double* a, double* out);
void launch_fill_i32(hipStream_t st, int64_t n, int32_t v, int32_t* out);
// a fixed pseudo-random vector in [-1, 1) (start of the power method)
void launch_hash_fill(hipStream_t st, int64_t n, double* out);

// --- LSQR (left-preconditioned, M^{-1} inner product) ------------------------
// u *= 1 / beta (m-space)
void launch_lsqr_unorm(hipStream_t st, int64_t m, int S, const int64_t* seg_row, const double* sc,
                       const int32_t* done, double* u);
// q = q - beta zh (n-space)
void launch_lsqr_q(hipStream_t st, int64_t n, int S, const int64_t* seg_col, const double* sc,
                   const int32_t* done, const double* zh, double* q, int first);
// zh = q / alpha; v = s / alpha; x += t1 w; w = v + t2 w (first: w = v, x untouched)
void launch_lsqr_update(hipStream_t st, int64_t n, int S, const int64_t* seg_col, const double* sc,
                        const int32_t* done, const double* q, const double* s, double* zh,
                        double* v, double* w, double* x, int first);

// --- GMRES -------------------------------------------------------------------
// h[s * ld + i] = V_i . w over segment s (i < k); sum (may be null) += h
// partial: RED_BLOCKS * ld doubles per segment; count: COUNT_STRIDE int32 per
// segment and MDOT vectors, zero between launches
constexpr int MDOT = 8;           // vectors of one workgroup
void launch_multidot(hipStream_t st, const Segments& G, int64_t n, int k, const double* V,
                     const double* w, double* partial, int32_t* count, int ld, double* h,
                     double* sum);
// w -= sum_{i<k} V_i h[s * ld + i]
void launch_multi_axpy(hipStream_t st, int S, const int64_t* seg_ptr, int64_t n, int k,
                       const double* V, const double* h, int ld, double* w);
// out = sum_{i<k} V_i y[s * ld + i]
void launch_multi_gemv(hipStream_t st, int S, const int64_t* seg_ptr, int64_t n, int k,
                       const double* V, const double* y, int ld, double* out);
// out_k = a_k / sqrt(nrm2[segment]) (0 where the norm is zero or the instance is done)
void launch_normalize_seg(hipStream_t st, int64_t n, int S, const int64_t* seg_ptr,
                          const double* nrm2, const int32_t* done, const double* a, double* out);

// --- device planner ----------------------------------------------------------
// in-place exclusive scan of v[0 .. n); work: scan_work_len(n) int32
int64_t scan_work_len(int64_t n);
void launch_exclusive_scan(hipStream_t st, int64_t n, int32_t* v, int32_t* work);
// see k_plan.hip; with out null the counting pass
void launch_iota(hipStream_t st, int64_t n, int32_t* out);
void launch_locown(hipStream_t st, int32_t n, const int32_t* pcols, const int32_t* part, const int32_t* pptr,
                   int32_t* locown);
void launch_row_runs(hipStream_t st, int32_t m, const int32_t* rowptr, const int2* owner, int32_t* ptr,
                     int32_t* out);
void launch_seg_first(hipStream_t st, int32_t nseg, int64_t len, const int32_t* ptr, const int32_t* key,
                      int32_t* first);
void launch_seg_pack(hipStream_t st, int32_t nseg, int64_t len, const int32_t* ptr, const int32_t* key,
                     const int32_t* at, int32_t* out, int32_t* optr);
void launch_plan_stat(hipStream_t st, const DevMatrix& M, int32_t jump, unsigned long long* stat);
void launch_plan_size(hipStream_t st, int32_t m, const int32_t* rowptr, const int32_t* qptr,
                      unsigned long long* size);
void launch_col_parts(hipStream_t st, int32_t n, const int32_t* trowptr, const int32_t* trow,
                      const int32_t* qptr, const int32_t* qpart, const int32_t* part, int32_t* ptr,
                      int32_t* out);
void launch_plan_omega(hipStream_t st, int32_t nsub, const SubDesc* subs, const int32_t* pptr,
                       const int32_t* pcols, const int32_t* goff, const int32_t* gamma, int32_t* omega,
                       int32_t* F);
void launch_plan_envelope(hipStream_t st, const int32_t* qptr, const int32_t* qpart, const DevMatrix& M,
                          const int2* owner, const SubDesc* subs, const int32_t* goff,
                          const int32_t* gamma, int32_t* F);
void launch_tile_offsets(hipStream_t st, int32_t nsub, const SubDesc* subs, const int32_t* F, int64_t* off,
                         int64_t* stored);
void launch_own_maps(hipStream_t st, int32_t n, const int32_t* part, const int32_t* locown,
                     const SubDesc* subs, const int32_t* goff, const int32_t* optr, const int32_t* opart,
                     const int32_t* operm, int32_t* own_ptr, int32_t* own_pos);
void launch_pair_count(hipStream_t st, int64_t nx, const int32_t* xi, const int32_t* qperm,
                       const int32_t* qptr, int32_t* cnt);
void launch_pair_fill(hipStream_t st, int64_t nx, const int32_t* qperm, const int32_t* qpart,
                      const int32_t* xoff, const int32_t* at, int4* rec);
void launch_row_keys(hipStream_t st, int32_t m, int32_t n, const int32_t* rowptr, const int32_t* colind,
                     int32_t* key);
void launch_perm_len(hipStream_t st, int32_t m, const int32_t* perm, const int32_t* rowptr, int32_t* len);

// --- subdomain kernels -------------------------------------------------------
// with inv (not null), also the envelope F8 of the global-order layouts gsub:
// per eight rows the first position they reach (launch_solve_env_init first)
// scale non-null: assemble S C_ii S and S Ct_GG S directly (S = scale, from
// launch_col_scale), identity on the padding diagonal
// owner: per entry of A the part and local position of its column
// (launch_entry_owner), or null: looked up; fac need not be cleared
void launch_entry_owner(hipStream_t st, const DevPlan& P, const DevMatrix& M, int2* owner);
void launch_assemble(hipStream_t st, int nsub, const DevPlan& P, const DevMatrix& M, const int2* owner,
                     double* fac, double* ctg, const int32_t* inv, const SubDesc* gsub, int32_t* F8,
                     const double* scale);
void launch_equilibrate(hipStream_t st, int nsub, const DevPlan& P, double* fac, double* ctg,
                        double* scale);
// tiles, rows: stored tiles and tile rows of the layout; interior_only: factor
// the interior tile columns only (L_I and L_GI)
void launch_chol_local(hipStream_t st, int nsub, const DevPlan& P, int64_t tiles, int64_t rows, double* fac,
                       double* dinv, int32_t* status, bool interior_only = false);
// the same in FP32 (FP32 MFMA, FP32 accumulation)
void launch_chol_local_f32(hipStream_t st, int nsub, const DevPlan& P, int64_t tiles, int64_t rows,
                           float* fac, float* dinv, int32_t* status);
// solve factor in the global-column order of each subdomain: inv (indexed
// like loc) maps an [I, Gamma] position to its global-order position;
// gsub describes the global-order layout (np, ntiles, tile_base); F8 (four per
// tile row), initialized here to the diagonal, gets its envelope from the
// assembly
void launch_solve_inv(hipStream_t st, int nsub, const DevPlan& P, int32_t* inv);
void launch_solve_env_init(hipStream_t st, int nsub, const SubDesc* gsub, int32_t* F8);
// Ps.sperm (filled with -1 first) from the chosen layouts (ssub.spare set:
// global order)
void launch_solve_perm(hipStream_t st, int nsub, const DevPlan& P, const SubDesc* ssub,
                       const int32_t* inv, int32_t* sperm);
// the solve layout's matrix (double) from the assembled, equilibrated C_ii
void launch_gather_solve(hipStream_t st, int nsub, const DevPlan& P, const DevPlan& Ps,
                         const double* fac, double* out);
void launch_to_float(hipStream_t st, int64_t n, const double* src, float* dst);
// the layout of the chosen solve factor on the device: tile counts of the
// global-order layouts (tiles[i]) from the envelope F8, then the envelope
// tables of the layouts ssub (spare set: global order)
void launch_layout_count(hipStream_t st, int nsub, const SubDesc* gsub, const int32_t* F8, int32_t* tiles);
void launch_layout_fill(hipStream_t st, int nsub, const DevPlan& P, const SubDesc* ssub,
                        const SubDesc* gsub, const int32_t* F8, int32_t* tileF, int64_t* tileOff);
// streams of the layout P (tiles: its stored tiles; F8 and gsub as above, for
// subdomains with spare set): tables, gather maps, entries
void launch_stream_layout(hipStream_t st, int nsub, const DevPlan& P, const int32_t* F8,
                          const SubDesc* gsub, int64_t tiles, const SolveStream& S);
void launch_solve_cols(hipStream_t st, int nsub, const DevPlan& P, const DevPlan& Lay,
                       const double* scale, const SolveStream& S);
template <typename T>
void launch_stream_pack(hipStream_t st, int nsub, const DevPlan& P, const T* fac, const T* dinv,
                        const SolveStream& S);
// loc = S C_ii^{-1} S R_i r for every subdomain (S the equilibration)
template <typename T>
void launch_local_solve(hipStream_t st, int nsub, const DevPlan& P, const SolveStream& S, const T* fac,
                        const T* dinv, const double* r, double* loc);
int local_solve_cap(bool f32);    // largest subdomain that the streams solve (FP32 or FP64 factors)
// allows the streaming local solve its dynamic LDS (once per process)
hipError_t local_solve_configure();
// restricted: each column takes its owner's interior value only (R_i^T D_i, eq. RAS)
void launch_scatter_local(hipStream_t st, int32_t n, const DevPlan& P, const double* loc,
                          const double* X, const double* dcoarse, double* z, bool restricted = false);
void launch_scatter_local(hipStream_t st, int32_t n, const DevPlan& P, const double* loc,
                          const float* X, const double* dcoarse, double* z, bool restricted = false);
// ||C(Omega_Ii, :)||_F^2 of every subdomain from the assembled (unscaled) C_ii
void launch_frob_interior(hipStream_t st, int nsub, const DevPlan& P, const double* fac,
                          double* out);
// C_ii += s I on the real (non-padding) positions
void launch_add_diag(hipStream_t st, int nsub, const DevPlan& P, double s, double* fac);

// --- local factors from thin QR factorizations (k_qr.hip) --------------------
// QR_SEL: L_I and L_GI of the layout P from the rows Xi_i (out = fac, dinv);
// QR_SOLVE: the whole factor of C_ii in the layout Lay (the solve layout, inv
// the [I, Gamma] -> global-order position map of its permuted subdomains);
// QR_GAMMA: R_G of A(Xi_i, Omega_Gamma_i) into the dense interface matrices
// (out = ctg, zeroed by the caller).  The factor arrays must be zero on
// entry; strip holds 32 * total_loc doubles, zero on entry and on return;
// qscr holds 2 total_loc + nsub int32 (row-stream tables).
// status: first failing subdomain + 1 (zero or non-finite diagonal, or a
// layout beyond the kernel's tables).
enum { QR_SEL = 0, QR_SOLVE = 1, QR_GAMMA = 2 };
constexpr int QR_STRIP_ROWS = 32;
void launch_qr_local(hipStream_t st, int mode, int nsub, const DevPlan& P, const DevPlan& Lay,
                     const DevMatrix& M, const int32_t* inv, const double* scale, double* out,
                     double* dinv, double* strip, int32_t* qscr, int64_t total_loc, int32_t* status);
// scale = 1 / ||A(:, c)|| per position of the layout P (0 on padding)
void launch_col_scale(hipStream_t st, int nsub, const DevPlan& P, const DevMatrix& M, double* scale);

// --- coarse space ------------------------------------------------------------
void launch_gamma_T(hipStream_t st, int nsub, const DevPlan& P, const double* fac, double* Tg);
// ld x ld work matrices per subdomain of the selection (work holds
// SEL_WORK_MATS * total_g doubles; Y, the selected vectors, is the first)
constexpr int SEL_WORK_MATS = 5;
// qr_range: ctg holds the interface factors R_G of the QR route (k_qr.hip)
// instead of Ct_GG, and the range basis comes from a pivoted QR of them
void launch_select(hipStream_t st, int nsub, const DevPlan& P, const double* ctg, const double* Tg,
                   double* work, double tau, int nev_max, int32_t* p_out, double* sig_out,
                   int qr_range = 0);
void launch_coarse_X(hipStream_t st, int nsub, const DevPlan& P, const double* fac,
                     const double* dinv, const double* scale, const double* work,
                     const double* sig, double* X);
void launch_coarse_W(hipStream_t st, int nsub, const DevPlan& P, const DevMatrix& M,
                     const double* X, double* W);
void launch_coarse_E(hipStream_t st, int nitems, const DevPlan& P, const DevCoarse& Cc,
                     const double* W, double* efac);
// diagonal blocks of E += s X_i^T X_i (the rows sqrt(s) e_j of a shifted C)
void launch_coarse_E_shift(hipStream_t st, int nitems, const DevPlan& P, const DevCoarse& Cc,
                           const double* X, double s, double* efac);
// one step of the tile Cholesky of E for a list of independent diagonal
// blocks (jobs of EJOB_INTS ints, see k_echol_step); echol_job_blocks gives
// the workgroups one job takes
constexpr int EJOB_INTS = 6;
int echol_job_blocks(int nr, int npr);
void launch_echol_step(hipStream_t st, const DevCoarse& Cc, const int32_t* jobs, int njobs,
                       int nblocks, double* efac, double* edinv, int32_t* status);
void launch_tile_transpose(hipStream_t st, int64_t ntiles, const double* in, double* out);
void launch_einv(hipStream_t st, int nbins, const DevCoarse& Cc, const double* efac,
                 const double* edinv, const double* efacT, const double* edinvT, double* einv);
void launch_coarse_restrict(hipStream_t st, int nsub, const DevPlan& P, int max_p, const double* X,
                            const double* r, double* c);
void launch_coarse_restrict(hipStream_t st, int nsub, const DevPlan& P, int max_p, const float* X,
                            const double* r, double* c);
void launch_set_values(hipStream_t st, int64_t n, const int64_t* idx, double v, double* out);
void launch_einv_gemv(hipStream_t st, int64_t n0, int S, const DevCoarse& Cc, const double* einv,
                      const double* c, double* d);

}  // namespace lsq2l
