// kernels.hpp -- launch interface between the C-ABI layer (mpdd.cpp) and the
// HIP kernels.  Internal to libmpdd.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mpdd {

class ScratchCache;       // scratch.hpp

// Arguments of one plain dd update, passed by value to the kernels.
struct GemmParams {
  int64_t m, n, k;
  double alpha_hi, alpha_lo, beta_hi, beta_lo;
  const double *a_hi, *a_lo;
  int64_t lda;
  const double *b_hi, *b_lo;
  int64_t ldb;
  double *c_hi, *c_lo;
  int64_t ldc;
  // where beta C is read, if not in c (null): the update goes from one matrix
  // into another
  const double *ci_hi, *ci_lo;
  int64_t ldci;
  double *w_hi, *w_lo;  // k-split partial sums, [z][j*m + i]
  int64_t kchunk;       // k-range per k-split slice (multiple of the tile depth)
  int tiles_m, tiles_n;
  int tri;              // 0 full matrix, 1 upper triangle, 2 lower triangle
  int beta_zero;        // C is not read
};

// One request of a served group: its update (kchunk = k, no split) and the
// op flags (bit 0: op(A) transposed, bit 1: op(B) transposed).
struct ServeReq {
  GemmParams p;
  int flags;
  int pad_;
};

// One work item of a group: a C tile of a request.
struct ServeItem {
  int req;
  int bi, bj;
};

struct TileInfo {
  int bm, bn, bk, threads;
};

int tile_count();
const TileInfo* tile_info(int id);

hipError_t launch_gemm(int tile, const GemmParams& p, bool ta, bool tb, bool accurate,
                       int splitk, hipStream_t st);
// Entries of C that a guarded modular product left to the plain one:
// entry[j*lde + i] = 1 (else 0; stored for the whole tiles of the product),
// block[bj*ldf + bi] = 0 where no entry of the 64 x 64 block (bi, bj) is, else 1,
// or 2 (the real dd and the qd form, not the long and the complex one) where all
// are, those past C's edges included.
struct CrtFailed {
  const uint8_t *block, *entry;
  int64_t ldf, lde;
};
// How they are computed: tiles and k-ranges by the estimated time of all of C (if
// much has failed, that is what is to be done), and the scratch of the ranges' sums
// (flag_bytes for a flag a tile, then the sums; 0 if not split).  Split only
// where that is estimated to save a fifth, since it takes a launch more, 4 us, in
// every call: 1031 x 64 x 4001, but not 1024^3 or 8192 x 64 x 8192.  parts: ranges
// summed one after the other, where the plain product's k-split is finer.
struct FailedPlan {
  int tile = 0, splits = 1, parts = 1, tiles_m = 0, tiles_n = 0, blocks = 0;
  int64_t kchunk = 0;
  size_t flag_bytes = 0, bytes = 0;
};
FailedPlan failed_plan(int tri, int64_t m, int64_t n, int64_t k);
hipError_t launch_gemm_failed(const GemmParams& p, bool ta, bool tb, const CrtFailed& failed,
                              const FailedPlan& plan, void* scratch, hipStream_t st);
hipError_t launch_splitk_reduce(const GemmParams& p, int splitk, hipStream_t st);
// Persistent grouped kernel over the `which`-th item list: counts[c] items per
// tile shape, lists stored back to back starting at base + *items_offset
// (read on the device).
hipError_t launch_grouped_list(int tile, const char* base, const ServeReq* reqs,
                               const int* counts, const int* items_offset, int which, int grid,
                               hipStream_t st);
hipError_t launch_scale(const GemmParams& p, hipStream_t st);

// Complex dd epilogue of Cgemm (complex.hip): C <- alpha P + beta C when
// use_p, else C <- beta C; beta_zero: C is not read.  alpha / beta are
// {re.hi, re.lo, im.hi, im.lo}.
struct CEpilogue {
  int64_t m, n;
  double alpha[4], beta[4];
  const double *p_rh, *p_rl, *p_ih, *p_il;
  int64_t ldp;
  double *c_rh, *c_rl, *c_ih, *c_il;
  int64_t ldc;
  int use_p, beta_zero;
  // three_m: p_r = R1, p_i = R2, q = R3; P = (R1 - R2) + i (R3 - R1 - R2)
  const double *q_h, *q_l;
  int three_m;
};
hipError_t launch_cgemm_epilogue(const CEpilogue& p, hipStream_t st);
// out = x + s y elementwise over a rows x cols matrix (x, y: hi / lo planes
// with leading dimension ld; out compact, ld = rows), in dd (s = +-1).
hipError_t launch_dd_axpy_planes(const double* x_hi, const double* x_lo, const double* y_hi,
                                 const double* y_lo, int64_t ld, double s, int64_t rows,
                                 int64_t cols, double* o_hi, double* o_lo, hipStream_t st);

// Quad-double Rgemm (qd.hip): four planes per matrix, alpha / beta as
// {x0, x1, x2, x3}.  scale_only: C <- beta C (alpha = 0 or k = 0);
// beta_zero: C is not read.
struct QgemmParams {
  int64_t m, n, k;
  double alpha[4], beta[4];
  const double* a[4];
  int64_t lda;
  const double* b[4];
  int64_t ldb;
  double* c[4];
  int64_t ldc;
  int beta_zero, scale_only;
};
hipError_t launch_qgemm(const QgemmParams& p, bool ta, bool tb, hipStream_t st);
// The entries that a guarded modular product left.
hipError_t launch_qgemm_failed(const QgemmParams& p, bool ta, bool tb, const CrtFailed& failed,
                               hipStream_t st);

// Cholesky block column (potrf.hip): factor the rows x jb block column (jb <=
// 64, jb <= rows) read from s (ld lds) in the lower view (upper = 1: stored
// transposed) into a (ld lda): the diagonal block's triangle and the rows
// below it.  *info is the factorisation's failure word: if it is already
// non-zero the kernel does nothing; if a pivot of this block fails it becomes
// offset + the 1-based order of that pivot within the block.
hipError_t launch_potrf_panel(const double* s_hi, const double* s_lo, int64_t lds, double* a_hi,
                              double* a_lo, int64_t lda, int64_t rows, int jb, int upper,
                              long long* info, long long offset, hipStream_t st);
// {hi, lo} pairs <-> hi / lo planes (n elements).
hipError_t launch_split_pairs(const double* pairs, double* hi, double* lo, int64_t n,
                              hipStream_t st);
hipError_t launch_join_pairs(const double* hi, const double* lo, double* pairs, int64_t n,
                             hipStream_t st);

}  // namespace mpdd

namespace mpdd {

// Split-form (Ozaki) Rgemm (ozaki.hip), or with tri = 1 / 2 the upper / lower
// triangle of an Rsyrk (m == n, B == A, tb == !ta).  Returns 0 or an
// MPDD_ERR_* code.
int ozaki_gemm(const void* opts, int tri, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
               double alpha_hi, double alpha_lo, const double* a_hi, const double* a_lo,
               int64_t lda, const double* b_hi, const double* b_lo, int64_t ldb,
               double beta_hi, double beta_lo, double* c_hi, double* c_lo, int64_t ldc,
               hipStream_t st, ScratchCache& pool);

// Modular product in place of the plain one, the entries whose error is not
// bounded by the plain product's computed plainly (ozaki.hip).
// Returns 0, MPDD_ERR_SCRATCH or MPDD_ERR_UNSUPPORTED (nothing enqueued: the
// plain product is the caller's) or MPDD_ERR_HIP.
int ozaki_guarded_gemm(int tri, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                       double alpha_hi, double alpha_lo, const double* a_hi, const double* a_lo,
                       int64_t lda, const double* b_hi, const double* b_lo, int64_t ldb,
                       double beta_hi, double beta_lo, double* c_hi, double* c_lo, int64_t ldc,
                       hipStream_t st, ScratchCache& pool);
// Estimated time (us) of the guarded modular product: of all launches by the
// entries read (residues) and written, and the products' rounds.  The kernels have
// become faster since it was fitted: estimated and measured 74 and 60 at 600^3, 140
// and 105 at 1024^3, 596 and 461 at 2048^3, 3585 and 2632 at 4096^3, so that near the
// line the plain kernels are taken.  And of the complex product (126 and 136 at
// 512^3, 399 and 318 at 1024^3) and of the form for a long and a short operand (123 and
// 99 at 1031 x 64 x 4001, 704 and 706 at 8192 x 64 x 8192; 1e30: not applicable).
double guarded_us(int tri, int64_t m, int64_t n, int64_t k);
double guarded_complex_us(int64_t m, int64_t n, int64_t k);
double guarded_long_us(int64_t m, int64_t n, int64_t k);
int ozaki_guarded_long_gemm(bool ta, bool tb, int64_t m, int64_t n, int64_t k, double alpha_hi,
                            double alpha_lo, const double* a_hi, const double* a_lo, int64_t lda,
                            const double* b_hi, const double* b_lo, int64_t ldb, double beta_hi,
                            double beta_lo, double* c_hi, double* c_lo, int64_t ldc,
                            hipStream_t st, ScratchCache& pool);

// Split-form qd Rgemm (ozaki.hip; INT8 slices): alpha, beta four parts each,
// a, b, c four planes each; alpha != 0 and k > 0.  Returns 0 or MPDD_ERR_*.
int ozaki_qgemm(const void* opts, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                const double* alpha, const double* const* a, int64_t lda,
                const double* const* b, int64_t ldb, const double* beta, int beta_zero,
                double* const* c, int64_t ldc, hipStream_t st, ScratchCache& pool);

// Split-form building blocks (ozaki.hip).
int ozaki_split_entry(int algo, bool trans, int64_t rows, int64_t k, const double* hi,
                      const double* lo, int64_t ld, int nslices, int wfirst, int w, int* exps,
                      void* slices, int64_t ldq, int64_t rows_p, hipStream_t st, ScratchCache& pool);
int ozaki_digit_widths(int algo, int64_t k, int nslices, int* wfirst, int* w);

}  // namespace mpdd
