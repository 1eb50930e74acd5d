// potrf.hip -- panel kernel of the blocked dd Cholesky (Rpotrf).
//
// Rpotrf (MPLAPACK: LAPACK's DPOTRF on multiple-precision values) factors a
// symmetric positive definite A as L L^T (uplo 'L') or U^T U (uplo 'U').
// The blocked algorithm (mpdd.cpp) runs the O(n^3) work on the dd product kernels
// and calls this kernel once per block column of jb <= 64 columns: it reads
// the updated block column from its copy (s, ld lds) and writes its
// factor to A (ld lda).  It works in the "lower view" L(i, l) of the block
// column (L(i, l) = A(i, l) for 'L', A(l, i) for 'U'): rows 0 .. jb-1 are the
// diagonal block, the rows below are solved against its factor.
//
// Diagonal block.  Square-root-free elimination, column by column: column c
// of the reduced block is X(i) = L(i,c) sqrt(d), d the pivot (d <= 0 or NaN:
// info = offset + c+1 and stop; d stays in place), and the trailing entries
// take L(i,l) -= X(i) (X(l) / d).  The square roots wait for the end, where
// every column takes its own at once: L(i,c) = X(i) / sqrt(d_c).  Each of the
// workgroup's 512 threads keeps its entries of the triangle (packed by columns,
// at most 5) in registers; a step reads X(i) and X(l) from LDS, and the owners
// of the next column write theirs to the other buffer: one barrier a column.
// The wave with the next pivot forms its reciprocal.  The finished
// columns' entries drop out of the loop in steps of 512 (its body is compiled
// for each number of entries left), and the entries of a thread are
// independent chains, which is what a column's time is made of.
//
// Rows below.  A row p takes p(l) -= p(c) U(l,c) for l > c, column after
// column, with U(l,c) = L(l,c) / L(c,c) in LDS, and L(i,c) = p(c) / L(c,c) at
// the end: one or two rows per wave, lane = column, p(c) broadcast through scalar
// registers.  (All of it on values scaled by powers of two: panel_scale.)  Substitution needs no inverse of the block (half of the work of
// its elimination before) and no product launch.
//
// Every workgroup factors the diagonal block for itself (they would wait for
// one that did) and then solves its rows, 8 or 16 at a time; workgroup 0 writes
// the block's factor.  All arithmetic is the accurate dd add / multiply of
// dd.hpp and the division / square root of dd_ext.hpp.
//
// Bound: the chain of the diagonal block (64 dependent columns of a reciprocal,
// a multiply, a dd multiply-subtract and a barrier, about 0.8 us each), hidden
// by nothing: 73 us a block column of 64 at n = 2048 (60 for the last ones), of which
// 15 are the rows.
// Before (the elimination of [S | I] in LDS by one workgroup, then a product by
// the inverse): 76 + 19 us.  With the single-rounding-error "lean" multiply-add
// the factor's error tripled and the time did not fall, so the accurate
// operations stay.
#include "dd_ext.hpp"
#include "kernels.hpp"

#pragma clang fp contract(off)

namespace mpdd {

namespace {

constexpr int PANEL_MAX = 64;       // largest block order
constexpr int PANEL_THREADS = 512;
constexpr int PANEL_ROWS = 16;      // most rows below solved at a time (two per wave)
constexpr int PANEL_PACK = PANEL_MAX * (PANEL_MAX + 1) / 2;
constexpr int PANEL_SLOTS = (PANEL_PACK + PANEL_THREADS - 1) / PANEL_THREADS;

__device__ __forceinline__ int64_t lv(int upper, int64_t i, int64_t l, int64_t lda) {
  return upper ? (l + i * lda) : (i + l * lda);
}

// 1 / d for a normalised dd d > 0: the reciprocal of the leading part to full
// binary64 (v_rcp_f64 and two Newton steps), then one dd correction by the
// remainder r = 1 - d y: y (1 + r) leaves r^2, at most 2^-106.  Scaled by the
// exponent, so that the ends of the range behave as the middle.
__device__ __forceinline__ ddv dd_recip(ddv d) {
  const int e = __builtin_amdgcn_frexp_exp(d.hi);
  const double h = ldexp(d.hi, -e), l = ldexp(d.lo, -e);
  double y = __builtin_amdgcn_rcp(h);
  y = __builtin_fma(y, __builtin_fma(-h, y, 1.0), y);
  y = __builtin_fma(y, __builtin_fma(-h, y, 1.0), y);
  const double r = __builtin_fma(-l, y, __builtin_fma(-h, y, 1.0));
  const ddv q = fast_two_sum(y, y * r);
  return {ldexp(q.hi, -e), ldexp(q.lo, -e)};
}

// dd_mul without its last, exact renormalisation: the low part may reach a few
// ulps of the high one, which the steps that take it (another product, an
// addition) allow.
__device__ __forceinline__ ddv dd_mul_raw(ddv x, ddv y) {
  const ddv c = two_prod(x.hi, y.hi);
  const double t0 = x.lo * y.lo;
  const double t1 = __builtin_fma(x.hi, y.lo, t0);
  return {c.hi, c.lo + __builtin_fma(x.lo, y.hi, t1)};
}

__device__ __forceinline__ double lane_bcast(double x, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

struct PanelSmem {
  double2 x[2][PANEL_MAX];                   // the current and the next column
  double2 rd[2];                             // 1 / their pivots
  double2 inv[PANEL_MAX];                    // 1 / L(c,c)
  double2 l[PANEL_MAX][PANEL_MAX + 1];       // [column][row]: the block, then X, then U
  double2 rows[PANEL_MAX][PANEL_ROWS + 1];   // [column][row]: the rows being solved
  int sc[PANEL_MAX];                         // scale exponents (see panel_scale)
};

// The exponent s of row (and column) i of the diagonal block: the elimination
// runs on L(i,l) 2^(s_i + s_l), whose diagonal lies in [1/4, 2).  Without it
// the low part of a reciprocal 1 / d falls below the binary64 range from d =
// 2^968 on (an order 150 matrix scaled by 2^994: 2.5e5 instead of 0.31 units
// 2^-104 of the factor's norm); a square root and a division, which need no
// scaling, are twice as long in the chain.
__device__ __forceinline__ int panel_scale(double d) {
  return d > 0.0 && d < __builtin_inf() ? -(__builtin_amdgcn_frexp_exp(d) >> 1) : 0;
}

__device__ __forceinline__ double2 scaled(double2 v, int e) {
  return make_double2(ldexp(v.x, e), ldexp(v.y, e));
}

// Columns c0 .. c1-1, with the entries J .. PANEL_SLOTS-1 of every thread;
// returns 0, or 1 + the column of the first failing pivot.
template <int J>
__device__ __forceinline__ int panel_columns(PanelSmem& sm, int wave, int c0, int c1, int jb,
                                             const int (&si)[PANEL_SLOTS],
                                             const int (&sl)[PANEL_SLOTS],
                                             ddv (&z)[PANEL_SLOTS]) {
  for (int c = c0; c < c1; ++c) {
    const int b = c & 1;
    __syncthreads();                         // column c is there
    const double2 d = sm.x[b][c];
    if (!(d.x > 0.0)) return c + 1;          // (the same for every thread)
    if (c + 1 == jb) break;
    double2 xi[PANEL_SLOTS], xl[PANEL_SLOTS];
#pragma unroll
    for (int j = J; j < PANEL_SLOTS; ++j) {
      xi[j] = sm.x[b][si[j]];
      xl[j] = sm.x[b][sl[j]];
    }
    const ddv rd{sm.rd[b].x, sm.rd[b].y};
    // (entries of finished columns are updated as well: nobody reads them)
#pragma unroll
    for (int j = J; j < PANEL_SLOTS; ++j) {
      const ddv t = dd_mul_raw(ddv{xi[j].x, xi[j].y}, dd_mul_raw(ddv{xl[j].x, xl[j].y}, rd));
      z[j] = dd_add(z[j], dd_neg(t));
    }
#pragma unroll
    for (int j = J; j < PANEL_SLOTS; ++j)
      if (sl[j] == c + 1) {
        const double2 v = make_double2(z[j].hi, z[j].lo);
        sm.x[b ^ 1][si[j]] = v;
        sm.l[c + 1][si[j]] = v;
      }
    // 1 / d of the next column, by the wave that holds its pivot (the first
    // entry of column c + 1; every lane computes, the pivot's one is kept)
    const int q = (c + 1) * jb - c * (c + 1) / 2, jp = q / PANEL_THREADS;
    if ((q % PANEL_THREADS) / 64 == wave) {
      ddv zp = z[PANEL_SLOTS - 1];
#pragma unroll
      for (int j = J; j + 1 < PANEL_SLOTS; ++j)
        if (jp == j) zp = z[j];
      const ddv r = dd_recip(zp);
      if ((int)(threadIdx.x & 63) == q % 64) sm.rd[b ^ 1] = make_double2(r.hi, r.lo);
    }
  }
  return 0;
}

// TWO: rows below 16 at a time, two per wave; else 8, one per wave.
template <bool TWO>
__global__ void __launch_bounds__(PANEL_THREADS)
dd_potrf_panel(const double* __restrict__ s_hi, const double* __restrict__ s_lo, int64_t lds,
               double* __restrict__ a_hi, double* __restrict__ a_lo, int64_t lda, int64_t rows,
               int jb, int upper, long long* info, long long offset) {
  __shared__ PanelSmem sm;
  // the critical path of the factorisation, beside the workgroups of the bulk
  // update: issue first
  __builtin_amdgcn_s_setprio(3);
  // An earlier block of this factorisation failed: leave this one alone.  A
  // failure of this very block, which workgroup 0 may be recording already
  // (offset + its pivot's order), does not count: every wave of every workgroup
  // takes the same way whatever it reads, and finds that pivot itself.
  const long long before = __hip_atomic_load(info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (before != 0 && before <= offset) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int t = tid; t < PANEL_MAX * PANEL_MAX; t += PANEL_THREADS) {
    const int p = t & (PANEL_MAX - 1), q = t / PANEL_MAX;     // lanes along memory
    const int i = upper ? q : p, l = upper ? p : q;
    if (i >= jb || l > i) continue;
    const int64_t o = lv(upper, i, l, lds);
    const double2 v = make_double2(s_hi[o], s_lo[o]);
    sm.l[l][i] = v;
    if (i == l) sm.sc[i] = panel_scale(v.x);
  }
  __syncthreads();

  // this thread's entries, packed by columns: entry q of column l starts at
  // l jb - l (l - 1) / 2.  (A missing one: the last of the triangle again, not
  // published.)
  int si[PANEL_SLOTS], sl[PANEL_SLOTS];
  ddv z[PANEL_SLOTS];
  const int pack = jb * (jb + 1) / 2;
#pragma unroll
  for (int j = 0; j < PANEL_SLOTS; ++j) {
    // counted from the end the columns are 1, 2, 3, ... long
    const int q = pack - 1 - (tid + PANEL_THREADS * j);
    int r = q < 0 ? 0 : (int)((__builtin_sqrtf(8.0f * (float)q + 1.0f) - 1.0f) * 0.5f);
    if ((r + 1) * (r + 2) / 2 <= q) ++r;
    if (r * (r + 1) / 2 > q) --r;
    const bool on = q >= 0;
    sl[j] = on ? jb - 1 - r : -1;
    si[j] = on ? jb - 1 - (q - r * (r + 1) / 2) : 0;
    const double2 v = on ? scaled(sm.l[sl[j]][si[j]], sm.sc[si[j]] + sm.sc[sl[j]])
                         : make_double2(0.0, 0.0);
    z[j] = ddv{v.x, v.y};
    if (sl[j] == 0) {
      sm.x[0][si[j]] = v;
      sm.l[0][si[j]] = v;
      if (si[j] == 0) {
        const ddv r = dd_recip(z[j]);
        sm.rd[0] = make_double2(r.hi, r.lo);
      }
    }
    if (!on) sl[j] = 0;                      // (column 0 is published already)
  }

  // the column from which the first J entries of every thread are finished
  auto from = [&](int J) {
    const int q = pack - PANEL_THREADS * J;  // entries left
    int r = 0;
    while (r * (r + 1) / 2 < q) ++r;         // columns that hold them
    return q <= 0 ? jb : jb - r;
  };
  int fail = 0, c = 0;
#define PHASE(J)                                                                      \
  if (!fail) {                                                                        \
    const int to = (J) + 1 < PANEL_SLOTS ? max(c, from((J) + 1)) : jb;                 \
    fail = panel_columns<J>(sm, wave, c, to, jb, si, sl, z);                                \
    c = to;                                                                           \
  }
  PHASE(0)
  PHASE(1)
  PHASE(2)
  PHASE(3)
  PHASE(4)
#undef PHASE
  static_assert(PANEL_SLOTS == 5, "one phase per entry");
  const int done = fail ? fail - 1 : jb;     // finished columns
  __syncthreads();
  ddv piv{0.0, 0.0};
  if (tid < done) {
    const double2 d = sm.l[tid][tid];
    piv = dd_sqrt(ddv{d.x, d.y});
    const ddv q = dd_div(ddv{1.0, 0.0}, piv);
    sm.inv[tid] = make_double2(q.hi, q.lo);
  }
  __syncthreads();
  // the (partial, on failure) factor, and U in its place
  if (tid < done) sm.l[tid][tid] = make_double2(piv.hi, piv.lo);
  __syncthreads();
  for (int t = tid; t < PANEL_MAX * PANEL_MAX; t += PANEL_THREADS) {
    const int p = t & (PANEL_MAX - 1), q = t / PANEL_MAX;
    const int i = upper ? q : p, l = upper ? p : q;
    if (i >= jb || l > i) continue;
    ddv v{sm.l[l][i].x, sm.l[l][i].y};
    const ddv r{sm.inv[l].x, sm.inv[l].y};
    if (i > l && l < done) {
      v = dd_mul(v, r);
      const ddv u = dd_mul(v, r);
      sm.l[l][i] = make_double2(u.hi, u.lo);
    }
    if (blockIdx.x == 0) {
      // back from the scaled values: the factor, and the failing column's X
      // (columns after it are as they were read)
      const int e = l < done ? sm.sc[i] : l == done ? sm.sc[i] + sm.sc[l] : 0;
      const double2 w = scaled(make_double2(v.hi, v.lo), -e);
      const int64_t o = lv(upper, i, l, lda);
      a_hi[o] = w.x;
      a_lo[o] = w.y;
    }
  }
  if (fail) {
    if (blockIdx.x == 0 && tid == 0)
      __hip_atomic_store(info, offset + fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }

  constexpr int R = TWO ? PANEL_ROWS : PANEL_ROWS / 2;
  const int64_t below = rows - jb;
  for (int64_t r0 = (int64_t)blockIdx.x * R; r0 < below; r0 += (int64_t)gridDim.x * R) {
    __syncthreads();                         // U is there; the rows before are stored
    for (int t = tid; t < PANEL_MAX * R; t += PANEL_THREADS) {
      const int l = upper ? t & (PANEL_MAX - 1) : t / R;
      const int i = upper ? t / PANEL_MAX : t & (R - 1);
      double2 v = make_double2(0.0, 0.0);
      if (l < jb && r0 + i < below) {
        const int64_t o = lv(upper, jb + r0 + i, l, lds);
        v = scaled(make_double2(s_hi[o], s_lo[o]), sm.sc[l]);
      }
      sm.rows[l][i] = v;
    }
    __syncthreads();
    // rows wave and (TWO) wave + 8, lane = column
    const double2 v0 = sm.rows[lane][wave], v1 = sm.rows[lane][wave + (TWO ? 8 : 0)];
    ddv p0{v0.x, v0.y}, p1{v1.x, v1.y};
    double2 u = sm.l[0][lane];
    for (int k = 0; k + 1 < jb; ++k) {
      const double2 next = sm.l[k + 1][lane];
      const ddv b0{lane_bcast(p0.hi, k), lane_bcast(p0.lo, k)};
      const ddv b1{lane_bcast(p1.hi, k), lane_bcast(p1.lo, k)};
      const ddv uu = lane > k ? ddv{u.x, u.y} : ddv{0.0, 0.0};
      p0 = dd_add(p0, dd_neg(dd_mul_raw(b0, uu)));
      if (TWO) p1 = dd_add(p1, dd_neg(dd_mul_raw(b1, uu)));
      u = next;
    }
    const ddv r{sm.inv[lane].x, sm.inv[lane].y};
    p0 = dd_mul(p0, r);
    p1 = dd_mul(p1, r);
    sm.rows[lane][wave] = make_double2(p0.hi, p0.lo);
    if (TWO) sm.rows[lane][wave + 8] = make_double2(p1.hi, p1.lo);
    __syncthreads();
    for (int t = tid; t < PANEL_MAX * R; t += PANEL_THREADS) {
      const int l = upper ? t & (PANEL_MAX - 1) : t / R;
      const int i = upper ? t / PANEL_MAX : t & (R - 1);
      if (l >= jb || r0 + i >= below) continue;
      const int64_t o = lv(upper, jb + r0 + i, l, lda);
      a_hi[o] = sm.rows[l][i].x;
      a_lo[o] = sm.rows[l][i].y;
    }
  }
}

}  // namespace

hipError_t launch_potrf_panel(const double* s_hi, const double* s_lo, int64_t lds, double* a_hi,
                              double* a_lo, int64_t lda, int64_t rows, int jb, int upper,
                              long long* info, long long offset, hipStream_t st) {
  if (jb < 1 || jb > PANEL_MAX || rows < jb) return hipErrorInvalidValue;
  // (one workgroup per CU: 87 KB of LDS; 8 rows at a time while that keeps
  // them to one pass each)
  const bool two = rows - jb > 256 * PANEL_ROWS / 2;
  const int64_t r = two ? PANEL_ROWS : PANEL_ROWS / 2, tiles = (rows - jb + r - 1) / r;
  const unsigned grid = (unsigned)(tiles < 1 ? 1 : tiles > 256 ? 256 : tiles);
  hipLaunchKernelGGL(two ? dd_potrf_panel<true> : dd_potrf_panel<false>, dim3(grid), dim3(PANEL_THREADS), 0, st, s_hi, s_lo, lds, a_hi,
                     a_lo, lda, rows, jb, upper, info, offset);
  return hipGetLastError();
}

}  // namespace mpdd
