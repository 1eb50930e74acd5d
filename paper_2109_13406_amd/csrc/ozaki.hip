// ozaki.hip -- split-form dd Rgemm on the matrix cores of gfx950.
//
// The manual contains no split method; this is the error-free splitting of a
// matrix product (Ozaki, Ogita, Oishi, Rump 2012) in the integer-unit form of
// Ootomo, Ozaki and Yokota (2024), applied to dd operands:
//
//  scale    sigma_r = frexp exponent of max_l |x_rl.hi| for every row of op(A)
//           and every column of op(B) ("row operand"), so |x| < 2^sigma.
//  slice    y = x * 2^-sigma (exact); digit t: z = y * 2^w_t, q_t = rint(z.hi),
//           y = TwoSum(z.hi - q_t, z.lo).  INT8 form: w_1 = 6 and w_t = 8 while
//           nslices*k < 2^17 (a later digit that rounds to 128, or reaches it
//           by a carry, loses 256 and the digit before it gains one, so every
//           later digit is in [-128, 127]), else w_t = 7 (|q| <= 64); FP64
//           form: w_1 = w - 1, w_t = w with w chosen so that every sum of
//           nslices*k digit products stays an integer < 2^53.  Digits are
//           stored k-contiguous per row, in tiles padded with zeros.
//  products for every anti-diagonal d = t + u (2 <= d <= s + 1):
//           X_d = sum_t Q_t Q'_{d-t}^T, exact: int8 x int8 -> int32 on the
//           INT8 MFMA (|X_d| <= s*k*2^(2w-2) < 2^31), or FP64 MFMA on integers.
//  combine  P = sum_d X_d 2^-(2 w_1 + w (d-2)), added in dd (DWPlusFP) from the
//           smallest weight up; P * 2^(sigma_i + tau_j); C = alpha*P + beta*C.
// Binary64 arithmetic appears only in scaling, slicing and combining.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "../../include/mpdd.h"
#include "dd.hpp"
#include "crt.hpp"
#include "kernels.hpp"
#include "qd.hpp"
#include "scratch.hpp"

#pragma clang fp contract(off)

namespace mpdd {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

static __constant__ const CrtMods kCrtMods = crt_make_mods();
static __constant__ const CrtSums kCrtSums = crt_make_sums();
static __constant__ const CrtDigits kCrtDigits = crt_make_digits();
static __constant__ const CrtCombineTable<CrtCombineConsts, CRT_MAX_LIMBS, CRT_LIMB_BITS>
    kCrtCombine = crt_make_combine<CrtCombineConsts, CRT_MAX_LIMBS, CRT_LIMB_BITS>();
static __constant__ const CrtCombineTable<CrtCombineConsts26, CRT_MAX_LIMBS26, CRT_LIMB26>
    kCrtCombine26 = crt_make_combine<CrtCombineConsts26, CRT_MAX_LIMBS26, CRT_LIMB26>();

// Tile geometry of the FP64 product kernel; slice buffers are padded to the
// product kernel's tile.
constexpr int OZ_BM = 128;      // rows of op(A) per workgroup tile (FP64 form)
constexpr int OZ_BN = 128;      // columns of op(B) per workgroup tile (FP64 form)
constexpr int OZ_KPAD = 64;     // k padding of the slice rows

// ---- scale -------------------------------------------------------------------------

// Row operand element (r, l) lives at x[r*sr + l*sl].  Rows contiguous across
// lanes (sr == 1): a workgroup takes 64 rows x one chunk of OZ_SCALE_CHUNK
// columns; lane r%64 of wave w reads columns w, w+4, ... of the chunk (each
// wave load is 64 consecutive doubles), the 4 waves' maxima meet in LDS, and
// the chunk maximum goes to part[chunk][row].  oz_scale_finish reduces the
// chunks and takes the frexp exponent.
constexpr int OZ_SCALE_CHUNK = 512;

__global__ void __launch_bounds__(256)
oz_scale_part_cols(const double* __restrict__ x, int64_t sr, int64_t sl, int64_t rows, int64_t k, double* __restrict__ part) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r = (int64_t)blockIdx.x * 64 + lane;
  const int64_t l0 = (int64_t)blockIdx.y * OZ_SCALE_CHUNK;
  const int64_t l1 = (l0 + OZ_SCALE_CHUNK < k) ? l0 + OZ_SCALE_CHUNK : k;
  double mx = 0.0;
  if (r < rows)
    for (int64_t l = l0 + wave; l < l1; l += 4) mx = fmax(mx, fabs(x[r * sr + l * sl]));
  red[wave][lane] = mx;
  __syncthreads();
  if (wave == 0 && r < rows) {
    mx = fmax(fmax(red[0][lane], red[1][lane]), fmax(red[2][lane], red[3][lane]));
    part[(int64_t)blockIdx.y * rows + r] = mx;
  }
}

__global__ void __launch_bounds__(256)
oz_scale_finish(const double* __restrict__ part, int64_t rows, int nchunks,
                int* __restrict__ exps) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  double mx = 0.0;
  for (int c = 0; c < nchunks; ++c) mx = fmax(mx, part[(int64_t)c * rows + r]);
  int e = 0;
  if (mx != 0.0) frexp(mx, &e);
  exps[r] = e;
}

// Rows contiguous along l (sl == 1): one wave per row, lanes walk l.
__global__ void __launch_bounds__(256)
oz_scale_rows_wave(const double* __restrict__ x, int64_t sr, int64_t sl, int64_t rows, int64_t k, int* __restrict__ exps) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (r >= rows) return;
  double mx = 0.0;
  for (int64_t l = lane; l < k; l += 64) mx = fmax(mx, fabs(x[r * sr + l * sl]));
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  if (lane == 0) {
    int e = 0;
    if (mx != 0.0) frexp(mx, &e);
    exps[r] = e;
  }
}

// Partial row maxima (and sums of squares and of magnitudes) of both row operands
// of a modular product in one launch: a workgroup takes 64 rows of one operand and
// one of nch <= 16 chunks of l, and writes pmax[chunk][row], psum and pabs;
// the residue kernel reduces a row's chunks itself, so that no finishing
// launch stands between them.  (At 2048^2 the two operands took 83 us in
// three launches of 128, 512 and 8 workgroups.)  Rows contiguous across
// lanes: lane = row, the four waves take every fourth l, and meet in LDS;
// else 16 lanes walk the l of a row and meet by lane exchanges.
constexpr int CRT_SCALE_CHUNKS = 16;

__global__ void __launch_bounds__(256)
oz_crt_scale(CrtOperand opa, CrtOperand opb, int blocks_a, int64_t k, int64_t chunk) {
  __shared__ double red[3][4][64];
  const bool first = (int)blockIdx.x < blocks_a;
  const CrtOperand& op = first ? opa : opb;
  const int64_t r0 = (int64_t)(first ? blockIdx.x : blockIdx.x - blocks_a) * 64;
  const int64_t l0 = (int64_t)blockIdx.y * chunk;
  const int64_t l1 = (l0 + chunk < k) ? l0 + chunk : k;
  const double* __restrict__ x = op.hi;
  const double* __restrict__ x2 = op.hi2;
  const int64_t sr = op.sr, sl = op.sl, rows = op.rows;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (op.bad && blockIdx.y == 0 && tid < 64) op.bad[r0 + tid] = 0;
  if (r0 >= rows) return;                      // padding rows only
  double* __restrict__ pmax = op.pmax + (int64_t)blockIdx.y * rows;
  double* __restrict__ psum = op.psum + (int64_t)blockIdx.y * rows;
  double* __restrict__ pabs = op.pabs + (int64_t)blockIdx.y * rows;
  if (sr == 1) {
    const int64_t r = (r0 + lane < rows) ? r0 + lane : rows - 1;
    double mx = 0.0, sm = 0.0, ab = 0.0;
    int64_t l = l0 + wave;
    for (; l + 28 < l1; l += 32) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = fabs(x[r + (l + 4 * u) * sl]);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        mx = fmax(mx, v[u]);
        sm = fma(v[u], v[u], sm);
        ab += v[u];
      }
    }
    for (; l < l1; l += 4) {
      const double v = fabs(x[r + l * sl]);
      mx = fmax(mx, v);
      sm = fma(v, v, sm);
      ab += v;
    }
    if (x2)
      for (l = l0 + wave; l < l1; l += 4) {
        const double v = fabs(x2[r + l * sl]);
        mx = fmax(mx, v);
        sm = fma(v, v, sm);
        ab += v;
      }
    red[0][wave][lane] = mx;
    red[1][wave][lane] = sm;
    red[2][wave][lane] = ab;
    __syncthreads();
    if (wave == 0 && r0 + lane < rows) {
      pmax[r0 + lane] = fmax(fmax(red[0][0][lane], red[0][1][lane]),
                             fmax(red[0][2][lane], red[0][3][lane]));
      psum[r0 + lane] = (red[1][0][lane] + red[1][1][lane]) + (red[1][2][lane] + red[1][3][lane]);
      pabs[r0 + lane] = (red[2][0][lane] + red[2][1][lane]) + (red[2][2][lane] + red[2][3][lane]);
    }
    return;
  }
  const int sub = tid & 15;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int64_t rr = r0 + it * 16 + (tid >> 4);
    const int64_t r = rr < rows ? rr : rows - 1;
    const double* __restrict__ xr = x + r * sr;
    double mx = 0.0, sm = 0.0, ab = 0.0;
    int64_t l = l0 + sub;
    for (; l + 48 < l1; l += 64) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = fabs(xr[l + 16 * u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        mx = fmax(mx, v[u]);
        sm = fma(v[u], v[u], sm);
        ab += v[u];
      }
    }
    for (; l < l1; l += 16) {
      const double v = fabs(xr[l]);
      mx = fmax(mx, v);
      sm = fma(v, v, sm);
      ab += v;
    }
    if (x2)
      for (l = l0 + sub; l < l1; l += 16) {
        const double v = fabs(x2[r * sr + l]);
        mx = fmax(mx, v);
        sm = fma(v, v, sm);
        ab += v;
      }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      mx = fmax(mx, __shfl_xor(mx, off));
      sm += __shfl_xor(sm, off);
      ab += __shfl_xor(ab, off);
    }
    if (sub == 0 && rr < rows) {
      pmax[rr] = mx;
      psum[rr] = sm;
      pabs[rr] = ab;
    }
  }
}

// ---- slice -------------------------------------------------------------------------

// One 64 x 64 block of the row operand per workgroup of 512 threads.
// Elements of both planes are read with lanes along whichever index is
// contiguous in memory and staged in LDS; then each thread turns 4
// consecutive l of two rows (8-bit digits kept in registers: one 4-byte
// store per digit, 16 threads store a row's 64 digits of a slice together)
// or 8 consecutive l of one row (the other forms: 8 int8 or 8 doubles per
// digit) into digits and writes them k-contiguously.  Rows >= rows and
// l >= k (padding) get zero digits.
//
// 8-bit int8 digits: a later digit of 128 does not fit, so it is carried into
// the digit before it (it loses 2^w = 256, that digit gains one; the value
// does not change).  A carry can turn a 127 into 128, so it runs on through
// digits of 127: a digit of 128 carries out, and so does each 127 directly
// before it in a run that ends in 128; any other digit ends the run.  With at
// most 16 digits the raw digits of an element stay in registers and every
// carry is known once its last digit is: digit t is then stored as
// raw_t + carry_in_t wrapped to 8 bits (a carried 128 + c becomes c - 128, a
// carried 127 + 1 becomes -128, the others do not wrap).  Longer digit
// strings take two passes: the first finds the carries, the second recomputes
// the digits and stores them carried.
//
// The remainder after a digit, (z.hi - q) + z.lo, is formed with FastTwoSum:
// z.hi - q is exact and a whole multiple of ulp(z.hi) (q is an integer, and
// |z.hi - q| <= 1/2 keeps it within z.hi's binade or below), so it is zero or
// at least ulp(z.hi) in magnitude, while |z.lo| <= ulp(z.hi)/2 for a
// normalised pair -- FastTwoSum's condition holds and it returns the same
// pair as TwoSum in half the operations.
constexpr int OZ_SLICE_REG_DIGITS = 16;

template <typename T>
__global__ void __launch_bounds__(512, 2)
oz_slice(const double* __restrict__ xh, const double* __restrict__ xl, int64_t sr, int64_t sl,
         int64_t rows, int64_t k, const int* __restrict__ exps, int nslices, int wfirst, int w,
         T* __restrict__ q, int64_t ldq, int64_t plane) {
  // staging for the hi and the lo plane (66.5 KB: two workgroups fit a CU),
  // so that both planes' loads are in flight together
  __shared__ double t[2][64][65];
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.y * 64;
  const int64_t l0 = (int64_t)blockIdx.x * 64;
  const bool lanes_on_r = (sr == 1);
  const int rr = tid >> 3;
  const int lb = (tid & 7) * 8;
  const int64_t r = r0 + rr;
  const int e = (r < rows) ? exps[r] : 0;
  {
    double v[2][8];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const double* __restrict__ src = half ? xl : xh;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int a = tid & 63, b = (tid >> 6) + 8 * c;
        const int ri = lanes_on_r ? a : b;
        const int li = lanes_on_r ? b : a;
        const int64_t rg = r0 + ri, lg = l0 + li;
        v[half][c] = (rg < rows && lg < k) ? src[rg * sr + lg * sl] : 0.0;
      }
    }
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int a = tid & 63, b = (tid >> 6) + 8 * c;
        t[half][lanes_on_r ? a : b][lanes_on_r ? b : a] = v[half][c];
      }
  }
  __syncthreads();
  // scaled element i of this thread's 8 (the staging is not written again)
  auto scaled = [&](int i) {
    return ddv{ldexp(t[0][rr][lb + i], -e), ldexp(t[1][rr][lb + i], -e)};
  };
  T* out = q + r * ldq + l0 + lb;
  const bool carry = sizeof(T) == 1 && w > 7;

  if constexpr (sizeof(T) == 1) {
    if (carry && nslices <= OZ_SLICE_REG_DIGITS) {
      // here a thread takes 4 consecutive l of two rows, rq and rq + 32, so
      // that the 16 threads of a row store its 64 digits of a slice in one
      // contiguous piece; fw[t]: carried digit t of the 4 elements, one byte
      // each (one 4-byte store per digit)
      const int rq = tid >> 4, lq = (tid & 15) * 4;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int row = rq + 32 * g;
        const int eg = (r0 + row < rows) ? exps[r0 + row] : 0;
        uint32_t fw[OZ_SLICE_REG_DIGITS];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ddv z{ldexp(t[0][row][lq + i], -eg), ldexp(t[1][row][lq + i], -eg)};
          int raw[OZ_SLICE_REG_DIGITS];
          uint32_t run = 0, cm = 0;              // bit t of cm: carry out of digit t
#pragma unroll
          for (int d = 0; d < OZ_SLICE_REG_DIGITS; ++d) {
            raw[d] = 0;
            if (d < nslices) {
              const int shift = (d == 0) ? wfirst : w;
              const double zh = ldexp(z.hi, shift), zl = ldexp(z.lo, shift);
              const double qd = rint(zh);
              z = fast_two_sum(zh - qd, zl);
              raw[d] = (int)qd;
              if (d > 0) {
                const uint32_t bit = 1u << d;
                if (raw[d] >= 128) {
                  cm |= run | bit;
                  run = 0;
                } else if (raw[d] == 127) {
                  run |= bit;
                } else {
                  run = 0;
                }
              }
            }
          }
#pragma unroll
          for (int d = 0; d < OZ_SLICE_REG_DIGITS; ++d) {
            const uint32_t byte = (uint32_t)(raw[d] + (int)((cm >> (d + 1)) & 1u)) & 0xFFu;
            if (i == 0)
              fw[d] = byte;
            else
              fw[d] |= byte << (8 * i);
          }
        }
        T* o = q + (r0 + row) * ldq + l0 + lq;
#pragma unroll
        for (int d = 0; d < OZ_SLICE_REG_DIGITS; ++d)
          if (d < nslices) *(uint32_t*)(o + (int64_t)d * plane) = fw[d];
      }
      return;
    }
  }

  ddv y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) y[i] = scaled(i);
  // (longer 8-bit digit strings) first pass: the carries; bit d of cm[i] is
  // the carry out of digit d of element i
  uint64_t cm[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) cm[i] = 0;
  if (carry) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      ddv z = y[i];
      uint64_t run = 0, c = 0;
      for (int d = 0; d < nslices; ++d) {
        const int shift = (d == 0) ? wfirst : w;
        const double zh = ldexp(z.hi, shift), zl = ldexp(z.lo, shift);
        const double qd = rint(zh);
        z = fast_two_sum(zh - qd, zl);
        if (d == 0) continue;
        const uint64_t bit = (uint64_t)1 << d;
        if (qd >= 128.0) {
          c |= run | bit;
          run = 0;
        } else if (qd == 127.0) {
          run |= bit;
        } else {
          run = 0;
        }
      }
      cm[i] = c;
    }
  }
  for (int d = 0; d < nslices; ++d) {
    const int shift = (d == 0) ? wfirst : w;
    T dig[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const double zh = ldexp(y[i].hi, shift), zl = ldexp(y[i].lo, shift);
      const double qd = rint(zh);
      // carry in from digit d + 1, carry out of digit d
      const int cin = (int)((cm[i] >> (d + 1)) & 1), cout = (int)((cm[i] >> d) & 1);
      dig[i] = (sizeof(T) == 1) ? (T)((int)qd + cin - (cout << w)) : (T)qd;
      y[i] = fast_two_sum(zh - qd, zl);
    }
    T* o = out + (int64_t)d * plane;
    if constexpr (sizeof(T) == 1) {
      uint2 pack;
      pack.x = (uint32_t)(uint8_t)dig[0] | ((uint32_t)(uint8_t)dig[1] << 8) |
               ((uint32_t)(uint8_t)dig[2] << 16) | ((uint32_t)(uint8_t)dig[3] << 24);
      pack.y = (uint32_t)(uint8_t)dig[4] | ((uint32_t)(uint8_t)dig[5] << 8) |
               ((uint32_t)(uint8_t)dig[6] << 16) | ((uint32_t)(uint8_t)dig[7] << 24);
      *(uint2*)o = pack;
    } else {
#pragma unroll
      for (int i = 0; i < 8; i += 2) *(double2*)(o + i) = double2{dig[i], dig[i + 1]};
    }
  }
}

// Largest y with y (y + 1) / 2 <= t.
__device__ __forceinline__ int oz_tri_root(int t) {
  int y = (int)((__builtin_sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while ((y + 1) * (y + 2) / 2 <= t) ++y;
  while (y * (y + 1) / 2 > t) --y;
  return y;
}

// Tiles of one anti-diagonal group: the whole tiles_m x tiles_n grid, or for
// a triangle (tri 1: upper, tile row <= tile column; 2: lower; square
// tiles, tiles_m == tiles_n) only the tiles_m (tiles_m + 1) / 2 tiles that
// meet it.
__host__ __device__ __forceinline__ int oz_group_tiles(int tri, int tiles_m, int tiles_n) {
  return tri ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
}

// Workgroup b -> (anti-diagonal d, C tile (bi, bj)).  Groups of
// oz_group_tiles workgroups share one d, largest d (longest sum) first.
// Inside a group, each of the 8 XCDs (workgroups are dealt to them
// round-robin) receives a contiguous run of the tile sequence, and that
// sequence walks the C grid in 8 x 8 super-tiles (bi fastest inside one):
// the workgroups an XCD runs at the same time then cover a compact block of
// C and read a few row panels of op(A) and column panels of op(B), which its
// L2 holds, instead of every row panel of op(A) against one column panel.
// A triangle with tiles_m a multiple of 8 is walked in the same 8 x 8
// blocks: first the blocks off the diagonal (64 tiles each, blocks column by
// column), then the diagonal blocks (their 36 tiles each), so that every
// XCD's run holds an equal number of tiles; other triangles column by column.
// runs false: b is already in the order of the groups and their sequences.
__device__ __forceinline__ void oz_tile_of(int b, int tri, int tiles_m, int tiles_n, int nslices,
                                           int& d, int& bi, int& bj, bool runs = true) {
  const int tiles = oz_group_tiles(tri, tiles_m, tiles_n);
  d = nslices + 1 - b / tiles;
  int r = b % tiles;
  if (runs && (tiles & 7) == 0) r = (r & 7) * (tiles >> 3) + (r >> 3);
  if (tri) {
    int x, y;                                  // tile (x, y) with x <= y
    if ((tiles_m & 7) == 0) {
      const int s8 = tiles_m >> 3, off = 64 * (s8 * (s8 - 1) / 2);
      if (r < off) {
        const int by = oz_tri_root(r >> 6) + 1, bx = (r >> 6) - by * (by - 1) / 2;
        x = bx * 8 + (r & 7);
        y = by * 8 + ((r >> 3) & 7);
      } else {
        const int db = (r - off) / 36, w = (r - off) % 36;
        const int yy = oz_tri_root(w);
        x = db * 8 + (w - yy * (yy + 1) / 2);
        y = db * 8 + yy;
      }
    } else {
      y = oz_tri_root(r);
      x = r - y * (y + 1) / 2;
    }
    bi = (tri == 1) ? x : y;
    bj = (tri == 1) ? y : x;
    return;
  }
  if ((tiles_m & 7) == 0 && (tiles_n & 7) == 0) {
    const int st = r >> 6, w = r & 63, stm = tiles_m >> 3;
    bi = (st % stm) * 8 + (w & 7);
    bj = (st / stm) * 8 + (w >> 3);
  } else {
    bi = r % tiles_m;
    bj = r / tiles_m;
  }
}

// ---- products: INT8 ---------------------------------------------------------------------

// The balanced residue of the integer y (|y| < 2^45) modulo m, its low byte in
// the result's low byte: q = rint(y / m) and y - q m, the rounding and the
// conversion by additions of 1.5 x 2^52 (which round to an integer and leave
// its low bits in the low word): full-rate operations, where v_rndne_f64 and
// v_cvt_i32_f64 are not.
__device__ __forceinline__ uint32_t crt_reduce(double y, double m, double minv) {
  constexpr double MAGIC = 0x1.8p52;
  const double q = fma(y, minv, MAGIC) - MAGIC;
  return (uint32_t)__builtin_bit_cast(uint64_t, fma(-q, m, y) + MAGIC);
}

// The low bytes of four words.
__device__ __forceinline__ uint32_t crt_pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return __builtin_amdgcn_perm(b, a, 0x0c0c0400u) | __builtin_amdgcn_perm(d, c, 0x04000c0cu);
}

// Four consecutive entries (rows i..i+3 of one column) of a residue product,
// |X| < 2^31, reduced modulo m: X (1/m) is within 2^-29 of X/m, so the nearest
// integer q is found and X - q m (exact) is the balanced residue (for m = 256
// possibly +128, whose byte is that of -128: the same class).  X becomes a
// double by its bits.  The word of the four int8 residues, and its store.
__device__ __forceinline__ uint32_t crt_word4(int v0, int v1, int v2, int v3, double m,
                                              double minv) {
  auto red = [&](int v) {
    // 2^52 + 2^31 + v, by bits
    const double x = __builtin_bit_cast(double, ((uint64_t)0x43300000u << 32) |
                                                    ((uint32_t)v ^ 0x80000000u)) -
                     (0x1p52 + 0x1p31);
    return crt_reduce(x, m, minv);
  };
  return crt_pack4(red(v0), red(v1), red(v2), red(v3));
}

__device__ __forceinline__ void crt_store4(int8_t* p, int v0, int v1, int v2, int v3, double m,
                                           double minv) {
  *(uint32_t*)p = crt_word4(v0, v1, v2, v3, m, minv);
}

// Transposes four words across the four rows of 16 lanes: word h of row r
// becomes word r of row h.
__device__ __forceinline__ v4i crt_swap4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
  const auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
  const auto lo = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return v4i{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
}

// X_d tile (WM x WN) for anti-diagonal d: sum over t of Q_t(rows) Q'_{d-t}(cols)^T
// with k-contiguous int8 rows.  GM x GN waves; each wave owns (WM/GM) x (WN/GN)
// outputs = (WM/GM/16) x (WN/GN/16) v_mfma_i32_16x16x64_i8
// tiles (int32 accumulators, held in AGPRs when they do not fit beside the
// fragments), so each 16-byte LDS fragment feeds several MFMAs.  A stage holds
// a W x 64-byte block of each operand in LDS (double buffered; 16-byte chunks
// XOR-permuted per row, i8_lds, so stores and fragment reads avoid bank
// conflicts).
// For an MFMA, lane l supplies row l % 16, bytes 16*(l/16) .. +15 of the
// k-step, for both operands, so every k pairs up.  Accumulation is exact in
// int32.  Variants (selected by mpdd_opts.tile_id for the INT8 form):
//   0: 256 x 256, 2 x 2 waves (128 x 128 each, 1 workgroup per CU)
//   1: 256 x 128, 2 x 2 waves (128 x 64 each, 2 workgroups per CU)
//   2: 128 x 128, 2 x 2 waves (64 x 64 each, 3 workgroups per CU)
//   3: 256 x 256, 2 x 4 waves (128 x 64 each, 512 threads: 2 waves per SIMD)
//   4: 256 x 256, 4 x 4 waves (64 x 64 each, 1024 threads: 4 waves per SIMD)
//   5, 6: the tiling of 3 in oz_gemm_i8_dma below (6 is the default)
//   7: 256 x 256, 2 x 2 waves in oz_gemm_i8_dma (1 wave per SIMD)
//   8: as 6 with v_mfma_i32_32x32x32_i8 (4 x 2 tiles of 32 x 32 per wave)
constexpr int I8_BK = 64;
constexpr int I8_PITCH = 64;   // bytes per staged row (one k-step), no padding

// LDS position of 16-byte chunk c of staged row r: chunks are permuted by an
// XOR with ((r >> 1) ^ (r >> 2)) & 3, so that both the staging stores (each 8
// or 16 lanes write 2 or 4 whole rows) and the fragment reads (lanes l read
// chunk l / 16 of rows r0 + l % 16, r0 a multiple of 16) touch distinct banks
// whether the LDS serves 8 lanes per 128 bytes or 16 lanes per 256 bytes.
__device__ __forceinline__ int i8_lds(int r, int c) {
  return r * I8_PITCH + ((c ^ ((r >> 1) ^ (r >> 2))) & 3) * 16;
}
constexpr int I8_PAD = 256;     // slice rows are padded to this for every variant

template <int WM, int WN, int GM, int GN>
__global__ void __launch_bounds__(64 * GM * GN, (WM * WN / (GM * GN) > 128 * 64) ? 1 : (GM * GN > 8 ? 4 : 2))
oz_gemm_i8(const int8_t* __restrict__ qa, const int8_t* __restrict__ qb, int32_t* __restrict__ x,
           int64_t kp, int64_t plane_a, int64_t plane_b, int64_t mp, int64_t np, int nslices,
           int tiles_m, int tiles_n, int tri) {
  constexpr int NT = 64 * GM * GN;             // threads: a GM x GN grid of waves
  constexpr int WR = WM / GM, WC = WN / GN;    // outputs per wave
  constexpr int FA = WR / 16, FB = WC / 16;    // 16-row fragments per wave
  constexpr int SR = NT / 4;                   // rows staged per pass (4 threads per row)
  constexpr int EA = WM / SR, EB = WN / SR;    // 16-byte staging loads per thread
  static_assert(WM % SR == 0 && WN % SR == 0, "staging must cover the tile");
  __shared__ __attribute__((aligned(16))) int8_t As[2][WM * I8_PITCH];
  __shared__ __attribute__((aligned(16))) int8_t Bs[2][WN * I8_PITCH];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % GM, wn = wave / GM;

  int d, bi, bj;
  oz_tile_of(blockIdx.x, tri, tiles_m, tiles_n, nslices, d, bi, bj);
  const int64_t i0 = (int64_t)bi * WM, j0 = (int64_t)bj * WN;

  v4i acc[FA][FB];
#pragma unroll
  for (int a = 0; a < FA; ++a)
#pragma unroll
    for (int c = 0; c < FB; ++c) acc[a][c] = v4i{0, 0, 0, 0};

  // staging: thread loads 16 bytes (chunk tid%4) of rows tid/4 + 64*e.  Global
  // loads run two k-steps ahead of the MFMAs (two register sets, used
  // alternately), so a load has two steps of matrix work to arrive before
  // its data is written to LDS.
  const int srow = tid >> 2, schunk = tid & 3, scol = schunk * 16;
  const int64_t ksteps = kp / I8_BK;
  const int64_t total = (int64_t)(d - 1) * ksteps;
  v4i ra0[EA], rb0[EB], ra1[EA], rb1[EB];

  auto gload = [&](int64_t s, v4i (&ra)[EA], v4i (&rb)[EB]) {
    const int t = 1 + (int)(s / ksteps);          // slice of op(A); op(B) slice d - t
    const int64_t l0 = (s % ksteps) * I8_BK;
    const int8_t* pa = qa + (int64_t)(t - 1) * plane_a + (i0 + srow) * kp + l0 + scol;
    const int8_t* pb = qb + (int64_t)(d - t - 1) * plane_b + (j0 + srow) * kp + l0 + scol;
#pragma unroll
    for (int e = 0; e < EA; ++e) ra[e] = *(const v4i*)(pa + SR * e * kp);
#pragma unroll
    for (int e = 0; e < EB; ++e) rb[e] = *(const v4i*)(pb + SR * e * kp);
  };
  auto sstore = [&](int buf, const v4i (&ra)[EA], const v4i (&rb)[EB]) {
#pragma unroll
    for (int e = 0; e < EA; ++e) *(v4i*)&As[buf][i8_lds(srow + SR * e, schunk)] = ra[e];
#pragma unroll
    for (int e = 0; e < EB; ++e) *(v4i*)&Bs[buf][i8_lds(srow + SR * e, schunk)] = rb[e];
  };
  const int fr = lane & 15, fc = lane >> 4;
  auto compute = [&](int cur) {
    v4i af[FA], bf[FB];
#pragma unroll
    for (int a = 0; a < FA; ++a)
      af[a] = *(const v4i*)&As[cur][i8_lds(wm * WR + a * 16 + fr, fc)];
#pragma unroll
    for (int c = 0; c < FB; ++c)
      bf[c] = *(const v4i*)&Bs[cur][i8_lds(wn * WC + c * 16 + fr, fc)];
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
      for (int c = 0; c < FB; ++c)
        acc[a][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[c], acc[a][c], 0, 0, 0);
  };

  // step s computes LDS buffer s & 1; even steps load into set 0 and store
  // set 1, odd steps the other way round.  kp is a multiple of 2 * I8_BK, so
  // the step count is even and both halves of every iteration run.
  gload(0, ra0, rb0);
  gload(1, ra1, rb1);
  sstore(0, ra0, rb0);
  __syncthreads();
  // (the loads and stores are unconditional, so that the wait counts are the
  // same on every iteration; past the end they re-read the last step, whose
  // data is stored but never used)
  for (int64_t s = 0; s < total; s += 2) {
    gload(s + 2 < total ? s + 2 : total - 1, ra0, rb0);
    // keep the loads ahead of the MFMAs (not for the 256 x 256 tile, whose
    // accumulators leave no room for the longer-lived staging registers)
    if constexpr (WR * WC <= 128 * 64) __builtin_amdgcn_sched_barrier(0);
    compute(0);
    sstore(1, ra1, rb1);
    __syncthreads();
    gload(s + 3 < total ? s + 3 : total - 1, ra1, rb1);
    if constexpr (WR * WC <= 128 * 64) __builtin_amdgcn_sched_barrier(0);
    compute(1);
    sstore(0, ra0, rb0);
    __syncthreads();
  }

  // C layout of a 16x16 INT8 MFMA tile: lane l holds rows 4*(l/16) + 0..3 of column l%16.
  int32_t* xd = x + (int64_t)(d - 2) * mp * np;
#pragma unroll
  for (int a = 0; a < FA; ++a)
#pragma unroll
    for (int c = 0; c < FB; ++c) {
      const int64_t i = i0 + wm * WR + a * 16 + (lane >> 4) * 4;
      const int64_t j = j0 + wn * WC + c * 16 + (lane & 15);
      *(v4i*)&xd[j * mp + i] = acc[a][c];
    }
}

// Direct-to-LDS form of the same product (variant 5): the digits travel from
// global memory straight into LDS (global_load_lds_dwordx4: lane l of a wave
// writes 16 bytes at M0 + 16 l), so no registers stage them and no ds_write
// stores them.  NS stages form a ring; the loads of a stage are issued NS - 1
// steps before its matrix work, and one barrier per step both publishes the
// stage about to be used and frees the one about to be refilled.  A DMA
// instruction fills 16 staged rows (1 KB, the i8_lds layout); each lane picks
// the global chunk that the layout places at its slot, so the XOR permutation
// is applied on the global side.
// Wait until at most VM of this wave's global loads (here: LDS DMA) and LGKM
// of its LDS reads are outstanding, then meet the workgroup barrier.  One asm
// statement with a memory clobber, so that no LDS access moves across it.
template <int VM, int LGKM>
__device__ __forceinline__ void i8_sync() {
  static_assert(VM >= 0 && VM <= 63 && LGKM >= 0 && LGKM <= 15, "s_waitcnt fields");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)\n\ts_barrier" ::"n"(VM), "n"(LGKM) : "memory");
}

template <int WM, int WN, int GM, int GN, int NS, bool PF, bool M32, bool CRT = false>
__global__ void __launch_bounds__(64 * GM * GN, (WM * WN <= 128 * 128) ? 2 : 1)
oz_gemm_i8_dma(const int8_t* __restrict__ qa, const int8_t* __restrict__ qb,
               int32_t* __restrict__ x, int64_t kp, int64_t plane_a, int64_t plane_b, int64_t mp,
               int64_t np, int nslices, int tiles_m, int tiles_n, int tri,
               int crt_count, int crt_total, int crt_group, CrtGuard guard) {
  constexpr int NW = GM * GN;                  // waves
  constexpr int WR = WM / GM, WC = WN / GN;    // outputs per wave
  constexpr int MT = M32 ? 32 : 16;            // MFMA tile edge
  constexpr int KS = M32 ? 2 : 1;              // MFMA k-slabs per 64-byte step
  constexpr int FA = WR / MT, FB = WC / MT;    // fragments per wave and slab
  constexpr int RA = WM / NW, RB = WN / NW;    // rows of each operand one wave stages
  constexpr int LA = RA / 16, LB = RB / 16;    // DMA instructions per operand and step
  constexpr int STAGE = (WM + WN) * I8_PITCH;  // bytes per stage
  static_assert(RA % 16 == 0 && RB % 16 == 0, "a DMA instruction stages 16 rows");
  __shared__ __attribute__((aligned(1024))) int8_t smem[NS * STAGE];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % GM, wn = wave / GM;

  int d, bi, bj;
  if constexpr (CRT) {
    // Products with fewer tiles than the chip holds workgroups run several
    // groups of planes at once.  Each XCD then takes a run of the whole sequence
    // (group by group) instead of a few tiles of every group: at 2048^2 half a plane's
    // 64 tiles, 12 panels in its L2 a step, instead of 8 tiles of 4 planes, 36.
    // (1024^3, 32 planes: 58.5 -> 49.3 us, and 46.0 with the stores of crt_epilogue.)
    constexpr int SLOTS = WM == 256 ? 256 : 512;
    int b = blockIdx.x;
    const bool runs = oz_group_tiles(tri, tiles_m, tiles_n) >= SLOTS;
    if (!runs) {
      const int base = b / SLOTS * SLOTS, len = min(SLOTS, (int)gridDim.x - base);
      const int x = (b - base) & 7, q = (b - base) >> 3;
      b = base + x * (len >> 3) + min(x, len & 7) + q;
    }
    oz_tile_of(b, tri, tiles_m, tiles_n, nslices, d, bi, bj, runs);
  } else {
    oz_tile_of(blockIdx.x, tri, tiles_m, tiles_n, nslices, d, bi, bj);
  }
  if constexpr (CRT) {
    if (guard.mag && blockIdx.x == 0)            // (oz_crt_combine_c marks failed blocks)
      for (int64_t i = tid; i < (mp / 64) * (np / 64); i += 64 * NW) guard.block[i] = 0;
    if (guard.check) {
      // every entry of the tile failed: nothing of it will be read
      constexpr int NI = WM / 64, NB = NI * (WN / 64);
      const bool some =
          lane < NB && guard.block[((int64_t)bj * (WN / 64) + lane / NI) * guard.ldf +
                                   (int64_t)bi * NI + lane % NI] != 2;
      if (__ballot(some) == 0) return;
    }
  }
  // a guarded product: the thresholds of the tile's rows and columns (four a lane,
  // looked at when the first steps are on their way)
  float4 trow{}, tcol{};
  if constexpr (CRT) {
    if (guard.rows) {
      if (lane < WM / 4) trow = *(const float4*)(guard.ta + (int64_t)bi * WM + 4 * lane);
      if (lane < WN / 4) tcol = *(const float4*)(guard.tb + (int64_t)bj * WN + 4 * lane);
    }
  }
  // modular form: group d - 2 of crt_group consecutive residue planes; the
  // workgroup multiplies plane ct0 + g of both operands for each g in turn
  // (one k-sweep each, slice it - 1 of both operands below), storing each
  // product when its sweep ends
  int ct0 = 0;
  if constexpr (CRT) {
    ct0 = (d - 2) * crt_group;
    const int here = min(crt_group, crt_total - ct0);
    qa += (int64_t)ct0 * plane_a;
    qb += (int64_t)ct0 * plane_b;
    d = here + 1;
  }
  const int64_t i0 = (int64_t)bi * WM, j0 = (int64_t)bj * WN;

  typedef int v16i __attribute__((ext_vector_type(16)));
  typedef typename std::conditional<M32, v16i, v4i>::type accv;
  accv acc[FA][FB];
#pragma unroll
  for (int a = 0; a < FA; ++a)
#pragma unroll
    for (int c = 0; c < FB; ++c) acc[a][c] = accv{};

  // lane l of a DMA instruction fills staged row r0 + l/4 (r0 a multiple of
  // 16), physical chunk l%4, which holds logical chunk (l%4) ^ g(row); g
  // depends only on the row's low four bits, i.e. on l/4
  const int lr = lane >> 2;
  const int lc = ((lane & 3) ^ (lr >> 1) ^ (lr >> 2)) & 3;
  const int64_t ksteps = kp / I8_BK;
  const int64_t total = (int64_t)(d - 1) * ksteps;
  const int8_t* ga = qa + (i0 + wave * RA + lr) * kp + lc * 16;
  const int8_t* gb = qb + (j0 + wave * RB + lr) * kp + lc * 16;

  // Steps are issued in order, step x into stage x % NS; (it, il0) is the
  // slice and k offset of the next one.  Steps past the end re-load the last
  // step (into a stage no later step reads), so that every step issues the
  // same loads and the wait counts are constants.
  int it = 1, ibuf = 0;
  int64_t il0 = 0, inext = 0;
  auto issue = [&]() {
    const int8_t* pa = ga + (int64_t)(it - 1) * plane_a + il0;
    // op(B) slice d - t (the modular form: the same plane as op(A))
    const int8_t* pb = gb + (int64_t)(CRT ? it - 1 : d - it - 1) * plane_b + il0;
    int8_t* st = smem + ibuf * STAGE;
#pragma unroll
    for (int e = 0; e < LA; ++e)
      __builtin_amdgcn_global_load_lds(
          (const void*)(pa + (int64_t)16 * e * kp),
          (__attribute__((address_space(3))) void*)(st + (wave * RA + 16 * e) * I8_PITCH), 16, 0,
          0);
#pragma unroll
    for (int e = 0; e < LB; ++e)
      __builtin_amdgcn_global_load_lds(
          (const void*)(pb + (int64_t)16 * e * kp),
          (__attribute__((address_space(3))) void*)(st + WM * I8_PITCH +
                                                    (wave * RB + 16 * e) * I8_PITCH),
          16, 0, 0);
    if (++inext < total) {
      il0 += I8_BK;
      if (il0 == kp) {
        il0 = 0;
        ++it;
      }
    }
    ibuf = (ibuf + 1 == NS) ? 0 : ibuf + 1;
  };
  // fragment row and 16-byte chunk of this lane: 16 x 16 x 64 MFMAs take
  // row l % 16, chunk l / 16; 32 x 32 x 32 ones take row l % 32, chunk
  // 2 h + l / 32 of k-slab h
  const int fr = lane & (MT - 1), fc = lane / MT;
  auto fetch = [&](int buf, v4i (&af)[KS * FA], v4i (&bf)[KS * FB]) {
    const int8_t* As = smem + buf * STAGE;
    const int8_t* Bs = As + WM * I8_PITCH;
#pragma unroll
    for (int h = 0; h < KS; ++h) {
#pragma unroll
      for (int a = 0; a < FA; ++a)
        af[h * FA + a] = *(const v4i*)&As[i8_lds(wm * WR + a * MT + fr, KS * h + fc)];
#pragma unroll
      for (int c = 0; c < FB; ++c)
        bf[h * FB + c] = *(const v4i*)&Bs[i8_lds(wn * WC + c * MT + fr, KS * h + fc)];
    }
  };
  auto mfma = [&](const v4i (&af)[KS * FA], const v4i (&bf)[KS * FB]) {
#pragma unroll
    for (int h = 0; h < KS; ++h)
#pragma unroll
      for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int c = 0; c < FB; ++c) {
          if constexpr (M32)
            acc[a][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[h * FA + a], bf[h * FB + c],
                                                              acc[a][c], 0, 0, 0);
          else
            acc[a][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[c], acc[a][c], 0, 0, 0);
        }
  };
  // The fragments read one step earlier have long arrived: waiting for them
  // (lgkmcnt(0), before the next prefetch is issued) costs nothing and tells
  // the compiler that the MFMAs need not wait for the prefetch.
  auto frags_landed = [&]() {
    __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0); vmcnt, expcnt not waited on
    __builtin_amdgcn_sched_barrier(0);
  };
  // modular form: store the finished product of plane ct as int8 residues
  // modulo modulus ct % crt_count (a complex or qd product runs three products
  // per modulus, planes t, count + t, 2 count + t) and clear the accumulators
  // C layout: 16 x 16 tile, lane l holds rows 4 (l / 16) + 0..3 of column
  // l % 16; 32 x 32 tile, lane l holds rows 8 g + 4 (l / 32) + 0..3 of column
  // l % 32 in registers 4 g .. 4 g + 3
  auto crt_epilogue = [&](int ct) {
    if constexpr (!M32) {
      if (guard.mag && ct >= guard.plane) {
        int32_t* xm = guard.mag + (int64_t)(ct - guard.plane) * mp * np;
#pragma unroll
        for (int a = 0; a < FA; ++a)
#pragma unroll
          for (int c = 0; c < FB; ++c) {
            const int64_t j = j0 + wn * WC + c * MT + (lane & (MT - 1));
            *(v4i*)(xm + j * mp + i0 + wm * WR + a * MT + (lane >> 4) * 4) = acc[a][c];
            acc[a][c] = accv{};
          }
        return;
      }
      if (ct == guard.plane) {
        // the magnitude product: an entry passes if it is at least its row's
        // threshold plus its column's (a NaN, from a row or column that may
        // not take this path, fails).  One byte per entry goes out, and one
        // per 64 x 64 block: no, some or all of its entries failed.
        static_assert(!CRT || M32 || (WC == 64 && WR % 64 == 0), "one byte per 64 x 64 block");
        float tj[FB];
#pragma unroll
        for (int c = 0; c < FB; ++c) {
          const int64_t j = j0 + wn * WC + c * MT + (lane & (MT - 1));
          tj[c] = guard.bb[j] ? __builtin_nanf("") : guard.tb[j];
        }
#pragma unroll
        for (int h = 0; h < WR / 64; ++h) {
          uint32_t some = 0u, every = 0x01010101u;
#pragma unroll
          for (int a = 4 * h; a < 4 * h + 4; ++a) {
            const int64_t i = i0 + wm * WR + a * MT + (lane >> 4) * 4;
            const float4 ti = *(const float4*)(guard.ta + i);
            const int4 bi4 = *(const int4*)(guard.ba + i);
#pragma unroll
            for (int c = 0; c < FB; ++c) {
              const int64_t j = j0 + wn * WC + c * MT + (lane & (MT - 1));
              const uint32_t f0 = (bi4.x != 0) | !((float)acc[a][c][0] >= ti.x + tj[c]);
              const uint32_t f1 = (bi4.y != 0) | !((float)acc[a][c][1] >= ti.y + tj[c]);
              const uint32_t f2 = (bi4.z != 0) | !((float)acc[a][c][2] >= ti.z + tj[c]);
              const uint32_t f3 = (bi4.w != 0) | !((float)acc[a][c][3] >= ti.w + tj[c]);
              const uint32_t f = f0 | (f1 << 8) | (f2 << 16) | (f3 << 24);
              *(uint32_t*)(guard.entry + j * mp + i) = f;
              some |= f;
              every &= f;
              acc[a][c] = accv{};
            }
          }
          const bool any = __ballot(some != 0) != 0, all = __ballot(every != 0x01010101u) == 0;
          if (lane == 0)
            guard.block[((j0 + wn * WC) >> 6) * guard.ldf + ((i0 + wm * WR) >> 6) + h] =
                (uint8_t)(all ? 2 : any ? 1 : 0);
        }
        return;
      }
    }
    int8_t* xq = (int8_t*)x + (int64_t)ct * mp * np;
    const int mt = ct % crt_count;
    const double mm = kCrtMods.t[mt].m, mi = kCrtMods.t[mt].minv;
    if constexpr (M32) {
#pragma unroll
      for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int c = 0; c < FB; ++c) {
          const int64_t j = j0 + wn * WC + c * MT + (lane & (MT - 1));
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int64_t i = i0 + wm * WR + a * MT + 8 * g + 4 * (lane >> 5);
            crt_store4(xq + j * mp + i, acc[a][c][4 * g], acc[a][c][4 * g + 1],
                       acc[a][c][4 * g + 2], acc[a][c][4 * g + 3], mm, mi);
          }
          acc[a][c] = accv{};
          __builtin_amdgcn_sched_barrier(0);   // one tile's temporaries at a time
        }
    } else {
      // four tiles (64 rows) at a time: the lanes of a column exchange their
      // words, so that each stores 16 rows and a column's 64 go out in one piece
      // (4 rows a lane, 16 bytes a column and store, an epilogue took 12 us)
#pragma unroll
      for (int c = 0; c < FB; ++c) {
        int8_t* xc = xq + (j0 + wn * WC + c * MT + (lane & (MT - 1))) * mp + i0 + wm * WR +
                     16 * (lane >> 4);
#pragma unroll
        for (int a = 0; a + 3 < FA; a += 4) {
          uint32_t w[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            w[u] = crt_word4(acc[a + u][c][0], acc[a + u][c][1], acc[a + u][c][2],
                             acc[a + u][c][3], mm, mi);
            acc[a + u][c] = accv{};
            __builtin_amdgcn_sched_barrier(0); // one tile's temporaries at a time
          }
          *(v4i*)(xc + 16 * a) = crt_swap4(w[0], w[1], w[2], w[3]);
        }
      }
    }
  };
  int64_t next_end = ksteps;                   // step count at which the current product ends
  int done = 0;                                // products of the group stored so far

  constexpr int PER = LA + LB;                 // DMA instructions per step and wave
  // LDS reads that may stay in flight at a barrier: the prefetch (FA + FB
  // reads), capped by the 4-bit counter (waiting for its oldest read as well
  // is harmless)
  constexpr int PFQ = (KS * (FA + FB) < 15) ? KS * (FA + FB) : 15;

#pragma unroll
  for (int q = 0; q < NS - 1; ++q) issue();
  if constexpr (CRT) {
    if (guard.rows) {
      // No row or no column may take this path (nor have its residues been
      // written): every entry has failed.
      auto some = [&](const float4& t, int64_t first, int64_t used, int edge) {
        const int64_t i = first + 4 * lane;
        return __ballot(lane < edge / 4 &&
                        ((t.x == t.x && i < used) || (t.y == t.y && i + 1 < used) ||
                         (t.z == t.z && i + 2 < used) || (t.w == t.w && i + 3 < used))) != 0;
      };
      if (!some(trow, i0, guard.rows, WM) || !some(tcol, j0, guard.cols, WN)) {
        __builtin_amdgcn_s_waitcnt(0x0F70);      // (the steps' loads into the LDS: vmcnt(0))
        if (!guard.mag && guard.plane >= ct0 && guard.plane < ct0 + d - 1) {
          constexpr int ONES = 0x01010101;
          for (int e = tid; e < WM * WN / 16; e += 64 * NW)
            *(v4i*)(guard.entry + (j0 + e / (WM / 16)) * mp + i0 + e % (WM / 16) * 16) =
                v4i{ONES, ONES, ONES, ONES};
          for (int e = tid; e < (WM / 64) * (WN / 64); e += 64 * NW)
            guard.block[((j0 >> 6) + e / (WM / 64)) * guard.ldf + (i0 >> 6) + e % (WM / 64)] = 2;
        }
        return;
      }
    }
  }
  if constexpr (!PF) {
    // step s: issued 0 .. s + NS - 2, so step s has landed once the loads of
    // NS - 2 later steps remain; no LDS read is in flight at the barrier (the
    // reads of step s - 1 fed its MFMAs), so stage (s - 1) % NS may be refilled
    for (int64_t s = 0; s < total; ++s) {
      i8_sync<(NS - 2) * PER, 0>();
      issue();                                 // step s + NS - 1
      v4i af[KS * FA], bf[KS * FB];
      fetch((int)(s % NS), af, bf);
      mfma(af, bf);
      if constexpr (CRT) {
        if (s + 1 == next_end) {
          crt_epilogue(ct0 + done++);
          next_end += ksteps;
        }
      }
    }
  } else {
    // fragments of step s + 1 are read from LDS while the MFMAs of step s run
    // (two register sets).  At step s, issued 0 .. s + NS - 2: step s + 1 has
    // landed once the loads of NS - 3 later steps remain; the LDS reads of the
    // prefetch of step s (FA + FB, the youngest) may still be in flight, those
    // of step s - 1 are done, so stage (s - 1) % NS may be refilled.
    static_assert(NS >= 4, "prefetch needs four stages");
    v4i af0[KS * FA], bf0[KS * FB], af1[KS * FA], bf1[KS * FB];
    i8_sync<(NS - 2) * PER, 0>();
    fetch(0, af0, bf0);
    // total is even (kp is a multiple of 2 * I8_BK)
    for (int64_t s = 0; s < total; s += 2) {
      i8_sync<(NS - 3) * PER, PFQ>();
      issue();                                 // step s + NS - 1
      frags_landed();
      fetch((int)((s + 1) % NS), af1, bf1);
      mfma(af0, bf0);
      // after the last pair this prefetches a stage no step uses: harmless
      i8_sync<(NS - 3) * PER, PFQ>();
      issue();                                 // step s + NS
      frags_landed();
      fetch((int)((s + 2) % NS), af0, bf0);
      mfma(af1, bf1);
      if constexpr (CRT) {
        // a sweep ends after an even step count (ksteps is even)
        if (s + 2 == next_end) {
          crt_epilogue(ct0 + done++);
          next_end += ksteps;
        }
      }
    }
  }
  // the loads past the end must land before the workgroup's LDS is released
  __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0), lgkmcnt not waited on
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (CRT) return;
  int32_t* xd = x + (int64_t)(d - 2) * mp * np;
#pragma unroll
  for (int a = 0; a < FA; ++a)
#pragma unroll
    for (int c = 0; c < FB; ++c) {
      const int64_t j = j0 + wn * WC + c * MT + (lane & (MT - 1));
      if constexpr (M32) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int64_t i = i0 + wm * WR + a * MT + 8 * g + 4 * (lane >> 5);
          *(v4i*)&xd[j * mp + i] = v4i{acc[a][c][4 * g], acc[a][c][4 * g + 1],
                                       acc[a][c][4 * g + 2], acc[a][c][4 * g + 3]};
        }
      } else {
        const int64_t i = i0 + wm * WR + a * MT + (lane >> 4) * 4;
        *(v4i*)&xd[j * mp + i] = acc[a][c];
      }
    }
}

// ---- products: FP64 ---------------------------------------------------------------------

// Same tiling with v_mfma_f64_16x16x4_f64: a k-step stages 16 doubles per row;
// lane l supplies row l % 16 at k-offset l / 16 of each 4-deep MFMA.  Digit
// products and all their partial sums are integers below 2^53, so the FP64
// accumulation is exact in any order.
constexpr int F64_BK = 16;
constexpr int F64_PITCH = 17;

__global__ void __launch_bounds__(256)
oz_gemm_f64(const double* __restrict__ qa, const double* __restrict__ qb, double* __restrict__ x,
            int64_t kp, int64_t plane_a, int64_t plane_b, int64_t mp, int64_t np, int nslices,
            int tiles_m, int tiles_n, int tri) {
  __shared__ double As[2][OZ_BM * F64_PITCH];
  __shared__ double Bs[2][OZ_BN * F64_PITCH];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;

  int d, bi, bj;
  oz_tile_of(blockIdx.x, tri, tiles_m, tiles_n, nslices, d, bi, bj);
  const int64_t i0 = (int64_t)bi * OZ_BM, j0 = (int64_t)bj * OZ_BN;

  v4d acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = v4d{0.0, 0.0, 0.0, 0.0};

  // staging: 128 rows x 16 doubles per operand = 2048 doubles; 8 per thread:
  // thread handles row (tid / 2) and 8 consecutive k at (tid % 2) * 8.
  const int srow = tid >> 1, scol = (tid & 1) * 8;
  const int64_t ksteps = kp / F64_BK;
  const int64_t total = (int64_t)(d - 1) * ksteps;
  double ra[8], rb[8];

  auto gload = [&](int64_t s) {
    const int t = 1 + (int)(s / ksteps);
    const int64_t l0 = (s % ksteps) * F64_BK;
    const double* pa = qa + (int64_t)(t - 1) * plane_a + (i0 + srow) * kp + l0 + scol;
    const double* pb = qb + (int64_t)(d - t - 1) * plane_b + (j0 + srow) * kp + l0 + scol;
#pragma unroll
    for (int e = 0; e < 8; ++e) { ra[e] = pa[e]; rb[e] = pb[e]; }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      As[buf][srow * F64_PITCH + scol + e] = ra[e];
      Bs[buf][srow * F64_PITCH + scol + e] = rb[e];
    }
  };

  gload(0);
  sstore(0);
  __syncthreads();
  const int fr = lane & 15, fk = lane >> 4;
  for (int64_t s = 0; s < total; ++s) {
    const int cur = (int)(s & 1);
    if (s + 1 < total) gload(s + 1);
#pragma unroll
    for (int kk = 0; kk < F64_BK; kk += 4) {
      double af[4], bf[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) af[a] = As[cur][(wm * 64 + a * 16 + fr) * F64_PITCH + kk + fk];
#pragma unroll
      for (int c = 0; c < 4; ++c) bf[c] = Bs[cur][(wn * 64 + c * 16 + fr) * F64_PITCH + kk + fk];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[a], bf[c], acc[a][c], 0, 0, 0);
    }
    if (s + 1 < total) sstore(cur ^ 1);
    __syncthreads();
  }

  // C layout of the FP64 16x16 MFMA tile: lane l, register e holds row
  // 4*e + l/16 of column l%16 (unlike the INT8 form's 4*(l/16) + e).
  double* xd = x + (int64_t)(d - 2) * mp * np;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int64_t i = i0 + wm * 64 + a * 16 + (lane >> 4);
      const int64_t j = j0 + wn * 64 + c * 16 + (lane & 15);
#pragma unroll
      for (int e = 0; e < 4; ++e) xd[j * mp + i + 4 * e] = acc[a][c][e];
    }
}

// ---- combine -------------------------------------------------------------------------

// Four consecutive rows i0 .. i0+3 of one column j per thread (for a
// triangle, only its entries are read and written): each
// anti-diagonal sum is one 16-byte (int32) or 32-byte (fp64) load per thread
// (plane rows are padded to a multiple of 256, so the four are in range and
// aligned); the C entries (when read) are loaded first and a batch of NB
// anti-diagonals (8 int32, 4 fp64) is loaded before any is added, so that
// many loads are in flight at once.  Per entry the steps are the same as one
// entry at a time: smallest weight first (d = nslices+1 down to 2),
// DWPlusFP, then the scale and alpha / beta.
template <typename XT>
__global__ void __launch_bounds__(256)
oz_combine(const XT* __restrict__ x, int64_t mp, int64_t np, int nslices, int wfirst, int w,
           const int* __restrict__ ea, const int* __restrict__ eb, int64_t m, int64_t n,
           double alpha_hi, double alpha_lo, double beta_hi, double beta_lo, int beta_zero,
           double* __restrict__ c_hi, double* __restrict__ c_lo, int64_t ldc, int tri) {
  typedef XT xv4 __attribute__((ext_vector_type(4)));
  constexpr int NB = sizeof(XT) == 4 ? 8 : 4;
  const int64_t mq = (m + 3) / 4;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= mq * n) return;
  const int64_t i0 = (gid % mq) * 4, j = gid / mq;
  // rows of column j that are updated: all, or the triangle's (tri 1:
  // upper, i <= j; 2: lower, i >= j); a thread with none of them returns
  // before reading anything (its tile may not have been computed)
  const int64_t ilo = (tri == 2) ? j : 0, ihi = (tri == 1) ? j : m - 1;
  if (i0 > ihi || i0 + 3 < ilo) return;
  auto updated = [&](int64_t i) { return i < m && i >= ilo && i <= ihi; };
  const XT* xp = x + j * mp + i0;
  const int64_t plane = mp * np;
  double ch[4] = {0.0, 0.0, 0.0, 0.0}, cl[4] = {0.0, 0.0, 0.0, 0.0};
  if (!beta_zero) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (updated(i0 + r)) {
        ch[r] = c_hi[i0 + r + j * ldc];
        cl[r] = c_lo[i0 + r + j * ldc];
      }
  }
  ddv p[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) p[r] = ddv{0.0, 0.0};
  for (int d0 = nslices + 1; d0 >= 2; d0 -= NB) {
    xv4 v[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u)
      v[u] = d0 - u >= 2 ? *(const xv4*)(xp + (int64_t)(d0 - u - 2) * plane) : xv4{0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      if (d0 - u < 2) continue;
      const int sh = -(2 * wfirst + w * (d0 - u - 2));
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = dd_add_d(p[r], ldexp((double)v[u][r], sh));
    }
  }
  const ddv alpha{alpha_hi, alpha_lo}, beta{beta_hi, beta_lo};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t i = i0 + r;
    if (!updated(i)) continue;
    const int e = ea[i] + eb[j];
    ddv pr{ldexp(p[r].hi, e), ldexp(p[r].lo, e)};
    ddv res = dd_mul(alpha, pr);
    const int64_t ci = i + j * ldc;
    if (!beta_zero) res = dd_add(res, dd_mul(beta, ddv{ch[r], cl[r]}));
    c_hi[ci] = res.hi;
    c_lo[ci] = res.lo;
  }
}

// ---- split form for quad-double operands -------------------------------------------

// Slices of a row operand of quad-doubles (x0 + x1 + x2 + x3, four planes),
// INT8 digits only.  Staging as in oz_slice (one 33 KB buffer, each part in
// turn); each thread then turns 8 consecutive l of one row into digits.
// Digit t: z = y 2^w_t (exact), q_t = rint(z0), z0 - q_t (exact), then two
// TwoSum sweeps renormalise the four parts: every TwoSum is error-free, so
// the remainder stays exact, and after the bottom-up sweep z0 is the
// rounded value of the remainder with the rest below about ulp(z0), which
// keeps the next digit within the balanced range of oz_slice.  8-bit digits
// are carried as there, in two passes (the carries first; digit strings up
// to 64 long); 7-bit digits need no carries.
constexpr int OZ_QD_MAX_SLICES = 48;

__global__ void __launch_bounds__(512)
oz_slice_qd(const double* __restrict__ x0, const double* __restrict__ x1,
            const double* __restrict__ x2, const double* __restrict__ x3, int64_t sr, int64_t sl,
            int64_t rows, int64_t k, const int* __restrict__ exps, int nslices, int wfirst, int w,
            int8_t* __restrict__ q, int64_t ldq, int64_t plane) {
  __shared__ double t[64][65];
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.y * 64;
  const int64_t l0 = (int64_t)blockIdx.x * 64;
  const bool lanes_on_r = (sr == 1);
  const int rr = tid >> 3;
  const int lb = (tid & 7) * 8;
  const int64_t r = r0 + rr;
  const int e = (r < rows) ? exps[r] : 0;
  qacc y[8];
#pragma unroll
  for (int part = 0; part < 4; ++part) {
    const double* __restrict__ src = part == 0 ? x0 : part == 1 ? x1 : part == 2 ? x2 : x3;
    double v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int a = tid & 63, b = (tid >> 6) + 8 * c;
      const int ri = lanes_on_r ? a : b;
      const int li = lanes_on_r ? b : a;
      const int64_t rg = r0 + ri, lg = l0 + li;
      v[c] = (rg < rows && lg < k) ? src[rg * sr + lg * sl] : 0.0;
    }
    if (part) __syncthreads();                 // the previous part has been read
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int a = tid & 63, b = (tid >> 6) + 8 * c;
      t[lanes_on_r ? a : b][lanes_on_r ? b : a] = v[c];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const double xv = ldexp(t[rr][lb + i], -e);
      if (part == 0) y[i].s0 = xv;
      else if (part == 1) y[i].s1 = xv;
      else if (part == 2) y[i].s2 = xv;
      else y[i].s3 = xv;
    }
  }
  // one digit of z (in place: z becomes the remainder)
  auto digit = [](qacc& z, int shift) -> int {
    z.s0 = ldexp(z.s0, shift);
    z.s1 = ldexp(z.s1, shift);
    z.s2 = ldexp(z.s2, shift);
    z.s3 = ldexp(z.s3, shift);
    const double qd = rint(z.s0);
    z.s0 = z.s0 - qd;
    qd_renorm(z);
    return (int)qd;
  };
  // bit d of cm[i]: the carry out of digit d of element i (8-bit digits)
  uint64_t cm[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) cm[i] = 0;
  if (w > 7) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      qacc z = y[i];
      uint64_t run = 0, c = 0;
      for (int d = 0; d < nslices; ++d) {
        const int qv = digit(z, d == 0 ? wfirst : w);
        if (d == 0) continue;
        const uint64_t bit = (uint64_t)1 << d;
        if (qv >= 128) {
          c |= run | bit;
          run = 0;
        } else if (qv == 127) {
          run |= bit;
        } else {
          run = 0;
        }
      }
      cm[i] = c;
    }
  }
  int8_t* out = q + r * ldq + l0 + lb;
  for (int d = 0; d < nslices; ++d) {
    const int shift = (d == 0) ? wfirst : w;
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int qv = digit(y[i], shift);
      const int cin = (int)((cm[i] >> (d + 1)) & 1), cout = (int)((cm[i] >> d) & 1);
      const uint32_t byte = (uint32_t)(qv + cin - (cout << w)) & 0xFFu;
      if (i < 4)
        lo |= byte << (8 * i);
      else
        hi |= byte << (8 * (i - 4));
    }
    *(uint2*)(out + (int64_t)d * plane) = uint2{lo, hi};
  }
}

// qd combine: one output (i, j) per thread.  The anti-diagonal sums are
// added in qd from the smallest weight up (each X_d 2^-e_d is an exact
// binary64: TwoSum into the leading part, the errors passed down the
// levels, renormalised), then the exact power-of-two scale, then
// C = alpha P + beta C as qd products by levels (beta = 0: C not read).
__global__ void __launch_bounds__(256)
oz_combine_qd(const int32_t* __restrict__ x, int64_t mp, int64_t np, int nslices, int wfirst,
              int w, const int* __restrict__ ea, const int* __restrict__ eb, int64_t m, int64_t n,
              double4 alpha, double4 beta, int beta_zero, double* __restrict__ c0,
              double* __restrict__ c1, double* __restrict__ c2, double* __restrict__ c3,
              int64_t ldc) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= m * n) return;
  const int64_t i = gid % m, j = gid / m;
  const int64_t plane = mp * np;
  const int32_t* xp = x + j * mp + i;
  qacc p{0.0, 0.0, 0.0, 0.0};
  for (int d = nslices + 1; d >= 2; --d) {
    const double v = ldexp((double)xp[(int64_t)(d - 2) * plane], -(2 * wfirst + w * (d - 2)));
    double e;
    ts(p.s0, v, p.s0, e);
    ts(p.s1, e, p.s1, e);
    ts(p.s2, e, p.s2, e);
    p.s3 = p.s3 + e;
    qd_renorm(p);
  }
  const double4 pf = qd_final(p);
  const int sc = ea[i] + eb[j];
  const double4 ps{ldexp(pf.x, sc), ldexp(pf.y, sc), ldexp(pf.z, sc), ldexp(pf.w, sc)};
  const int64_t ci = i + j * ldc;
  qacc r{0.0, 0.0, 0.0, 0.0};
  qd_madd(r, alpha, ps);
  if (!beta_zero) {
    qd_renorm(r);
    qd_madd(r, beta, double4{c0[ci], c1[ci], c2[ci], c3[ci]});
  }
  const double4 o = qd_final(r);
  c0[ci] = o.x;
  c1[ci] = o.y;
  c2[ci] = o.z;
  c3[ci] = o.w;
}

// ---- modular split form ------------------------------------------------------------

// Residues of a row operand.  Element x of row r becomes the integer
// x' = t1 + t2 on the grid of P bits below 2^sigma_r: z = x 2^(P - sigma_r)
// (exact, zh + zl), t1 = rint(zh), t2 = rint((zh - t1) + zl), |x'| <= 2^P.
// Plane t (0-based) receives x' modulo modulus t, balanced (odd m: in
// [-(m-1)/2, (m-1)/2]; m = 256: the low byte), as int8 at
// q + t*plane + r*ldq + l; padding rows and columns get 0.
//
// x' is handled in 26-bit chunks: t1 = u 2^52 + v (u = rint(t1 2^-52); v is
// an integer with |v| <= 2^51, so the fma that forms it is exact),
// w = v + t2 (exact: |w| < 2^53 while P <= 104), u = u1 2^26 + u0 and
// w = w1 2^26 + w0 (|u0|, |w0| <= 2^25).  Then x' = u1 2^78 + u0 2^52 +
// w1 2^26 + w0, and y = u1 c78 + u0 c52 + w1 c26 + w0 (c_j = 2^j mod m) is
// congruent to x' and below 2^37 in magnitude, exact in binary64.  For odd m,
// y/m lies at least 1/(2m) from a half-integer while y * (1/m) is within
// 2^-23 of it, so q = rint(y * (1/m)) is the nearest integer and y - q m
// (one exact fma) the balanced residue.  m = 256 is plane 0: the low byte of
// w0 (w0 = x' modulo 2^26).
//
// A workgroup takes a block of 32 rows x 128 l: both planes are loaded with
// lanes along the contiguous index and staged in LDS (74 KB: two workgroups
// per CU); each thread then converts 8 consecutive l of one row and stores
// one 8-byte word per modulus, so the 16 threads of a row write its 128
// residues of a plane as one 128-byte line.  Columns l >= ldq (ldq is a
// multiple of 64) are neither stored nor, beyond k, read.  The 16 threads of
// a row first reduce the row's partial maxima (oz_crt_scale) to its exponent;
// the workgroups of the first columns write the exponents out.
//
// Both operands of a product go in one launch (row blocks [0, blocks_a) are
// A's): at 1024^2 one operand alone is 256 workgroups, half of what the chip
// holds.
//
// Complex operands: sign = -1 negates every entry (a conjugated imaginary
// part; the grid integer of -x is -x'); with add_q non-null the kernel also
// writes sum_q = add_q + these residues, reduced to the balanced range
// (the residues of the sum of the two grid integers, e.g. Ar' + Ai').
//
// GUARD (see the default route in mpdd.cpp): plane `count` receives the
// magnitude digits floor(|x| 2^(7 - sigma_r)) in 0 .. 127; thr[r] the row's
// share of the threshold, coef * Q with Q = (sum_l x_rl^2)^(1/2) 2^-sigma_r:
// -inf for a zero or padding row (it is exact), NaN for a row that must not
// take the modular route: a row of few terms, whose plain products round less,
// non-finite entries, or an exponent near the ends of the range.  bad[r] is set
// where a pair is not normalised.  A row of few terms has both Q^2 <
// CRT_GUARD_MIN_TERMS and S = sum_l |x_rl| 2^-sigma_r < CRT_GUARD_MIN_SUM: one
// with a large S beside a small Q^2 has S^2 / Q^2 > 8 terms' worth (as eight equal
// ones), one of them dominant, as in Gram and Schur matrices and Cholesky
// factors, and its entries pass or fail by their own bounds like any others.  (By
// Q^2 alone every row of a Gram matrix was refused, 1024^3 490 us instead of 100.
// Root mean square error of its product with a uniform one, and of its square, in
// units of 2^-104 |A||B|: 0.010 and 0.026, plain product 0.14 and 0.21.)
// KIND: 0 no guard, 1 guard, 2 guard of a complex product (the real or the
// imaginary parts of an operand; Q over both, and the digits go to two planes).
__device__ __forceinline__ float crt_threshold(double mx, double sum, double mags, int ex,
                                               float coef) {
  if (mx == 0.0 && sum == 0.0) return -__builtin_inff();
  const double q2 = ldexp(sum, -2 * ex);
  const bool few = !(q2 >= CRT_GUARD_MIN_TERMS) && !(ldexp(mags, -ex) >= CRT_GUARD_MIN_SUM);
  if (few || !(q2 <= 0x1p40) || ex > CRT_GUARD_MAX_EXP ||
      ex < -CRT_GUARD_MAX_EXP)
    return __builtin_nanf("");
  return (float)__builtin_sqrt(q2) * coef;
}

template <int KIND>
__global__ void __launch_bounds__(512, 2)
oz_crt_residues(CrtOperand opa, CrtOperand opb, int blocks_a, int64_t k, int nch, int count,
                int p, int64_t ldq, float coef) {
  constexpr bool GUARD = KIND != 0;
  // element l of a staged row sits at column l + l/8 (one padding double
  // every 8), so the 16 threads of a row, reading 8 consecutive elements each,
  // hit distinct banks; the odd row pitch staggers the rows
  constexpr int PITCH = 145;
  __shared__ double t[2][32][PITCH];
  auto col = [](int l) { return l + (l >> 3); };
  const bool first = (int)blockIdx.y < blocks_a;
  const CrtOperand& op = first ? opa : opb;
  const double* __restrict__ xh = op.hi;
  const double* __restrict__ xl = op.lo;
  const int64_t sr = op.sr, sl = op.sl, rows = op.rows, plane = op.rows_p * ldq;
  const double sign = op.sign;
  const int8_t* add_q = op.add_q;
  int8_t* sum_q = op.sum_q;
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)(first ? blockIdx.y : blockIdx.y - blocks_a) * 32;
  const int64_t l0 = (int64_t)blockIdx.x * 128;
  const bool lanes_on_r = (sr == 1);
  const int row = tid >> 4;
  // this row's exponent (and magnitude sum), from its chunks' partial values
  double mx = 0.0, sum = 0.0, mags = 0.0;
  if (r0 + row < rows && (tid & 15) < nch) {
    const int64_t at = (int64_t)(tid & 15) * rows + r0 + row;
    mx = op.pmax[at];
    if (GUARD) {
      sum = op.psum[at];
      mags = op.pabs[at];
    }
  }
  {
    // entry e of the block: lanes on r, 32 consecutive rows per half-wave;
    // else 64 consecutive l of one row per wave
    double v[2][8];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const double* __restrict__ src = half ? xl : xh;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int e = tid + 512 * c;             // 0 .. 4095 over the 32 x 128 block
        const int ri = lanes_on_r ? (e & 31) : (e >> 7);
        const int li = lanes_on_r ? (e >> 5) : (e & 127);
        const int64_t rg = r0 + ri, lg = l0 + li;
        v[half][c] = (rg < rows && lg < k) ? src[rg * sr + lg * sl] : 0.0;
      }
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      mx = fmax(mx, __shfl_xor(mx, off));
      if (GUARD) {
        sum += __shfl_xor(sum, off);
        mags += __shfl_xor(mags, off);
      }
    }
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int e = tid + 512 * c;
        const int ri = lanes_on_r ? (e & 31) : (e >> 7);
        const int li = lanes_on_r ? (e >> 5) : (e & 127);
        t[half][ri][col(li)] = v[half][c];
      }
  }
  int ex = 0;
  if (mx != 0.0) frexp(mx, &ex);
  float thr = 0.0f;
  if (GUARD) thr = crt_threshold(mx, sum, mags, ex, coef);
  if (l0 == 0 && (tid & 15) == 0) {
    if (r0 + row < rows) op.exps[r0 + row] = ex;
    if (GUARD) op.thr[r0 + row] = thr;
  }
  if constexpr (GUARD) {
    // (no row of these may take the modular route: nobody reads what they hold)
    if (!__syncthreads_or(r0 + row < rows && thr == thr)) return;
  } else {
    __syncthreads();
  }
  const int lq = (tid & 15) * 8;
  if (l0 + lq >= ldq) return;
  const int sh = p - ex;
  double u1[8], u0[8], w1[8], w0[8];
  uint32_t mag[2] = {0u, 0u};
  bool denorm = false;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int c = col(lq) + i;                 // lq is a multiple of 8
    const double xhv = t[0][row][c], xlv = t[1][row][c];
    const double zh = ldexp(sign * xhv, sh), zl = ldexp(sign * xlv, sh);
    if (GUARD) {
      denorm |= !(fabs(xlv) * 0x1p52 <= fabs(xhv));
      const int g = (int)ldexp(fabs(xhv), 7 - ex);
      mag[i >> 2] |= ((uint32_t)g & 0x7Fu) << (8 * (i & 3));
    }
    const double t1 = rint(zh);
    const double t2 = rint((zh - t1) + zl);
    const double u = rint(t1 * 0x1p-52);
    const double w = fma(-u, 0x1p52, t1) + t2;
    u1[i] = rint(u * 0x1p-26);
    u0[i] = fma(-u1[i], 0x1p26, u);
    w1[i] = rint(w * 0x1p-26);
    w0[i] = fma(-w1[i], 0x1p26, w);
  }
  const int64_t off = op.stepwise
                          ? (((l0 + lq) >> 6) * op.rows_p + r0 + row) * 64 + ((l0 + lq) & 63)
                          : (r0 + row) * ldq + l0 + lq;
  int8_t* o = op.q + off;
  if (GUARD) {
    if (denorm) op.bad[r0 + row] = 1;
    if constexpr (KIND == 2) {
      *(uint2*)(op.mag + off) = uint2{mag[0], mag[1]};
      *(uint2*)(op.mag2 + off) = uint2{mag[0], mag[1]};
    } else {
      *(uint2*)(o + (int64_t)count * plane) = uint2{mag[0], mag[1]};
    }
  }
  // residues of the sum: byte-wise add, then one correction into the
  // balanced range (|a + b| <= m - 1 for odd m; modulo 256 the byte add wraps)
  auto add_store = [&](int m, const uint32_t (&word)[2]) {
    const uint2 a = *(const uint2*)(add_q + (int64_t)m * plane + off);
    const int mm = (int)kCrtMods.t[m].m, h = (mm - 1) / 2;
    uint32_t out[2] = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t aw = (i < 4) ? a.x : a.y;
      int v = (int)(int8_t)(aw >> (8 * (i & 3))) + (int)(int8_t)(word[i >> 2] >> (8 * (i & 3)));
      if (m > 0) v = (v > h) ? v - mm : (v < -h) ? v + mm : v;
      out[i >> 2] |= ((uint32_t)v & 0xFFu) << (8 * (i & 3));
    }
    *(uint2*)(sum_q + (int64_t)m * plane + off) = uint2{out[0], out[1]};
  };
  {
    uint32_t word[2] = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i) word[i >> 2] |= ((uint32_t)(int)w0[i] & 0xFFu) << (8 * (i & 3));
    *(uint2*)o = uint2{word[0], word[1]};
    if (KIND != 1 && add_q) add_store(0, word);
  }
#pragma unroll
  for (int m = 1; m < CRT_MAX_MODULI; ++m) {
    if (m >= count) break;
    const CrtMod& cm = kCrtMods.t[m];
    uint32_t res[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const double y = fma(u1[i], cm.c78, fma(u0[i], cm.c52, fma(w1[i], cm.c26, w0[i])));
      res[i] = crt_reduce(y, cm.m, cm.minv);
    }
    const uint32_t word[2] = {crt_pack4(res[0], res[1], res[2], res[3]),
                              crt_pack4(res[4], res[5], res[6], res[7])};
    *(uint2*)(o + (int64_t)m * plane) = uint2{word[0], word[1]};
    if (KIND != 1 && add_q) add_store(m, word);
  }
}

// The exact integer X = S - q M from its limb sums S_l (S = sum_l S_l 2^(39 l)
// congruent to X modulo M, |S_l| < 2^51, |X| <= M/4), rounded to a dd: q =
// rint(sum_l S_l g_l), X_l = S_l - q M_l (exact), carries into balanced limbs,
// then DWPlusFP from the lowest limb up.
template <int L>
__device__ __forceinline__ ddv crt_limbs_to_dd(const double (&s)[L], const CrtCombineConsts& cst) {
  double est = 0.0;
#pragma unroll
  for (int l = L - 1; l >= 0; --l) est = fma(s[l], cst.g[l], est);
  const double qm = rint(est);
  double xl[L];
#pragma unroll
  for (int l = 0; l < L; ++l) xl[l] = fma(-qm, cst.ml[l], s[l]);
#pragma unroll
  for (int l = 0; l + 1 < L; ++l) {
    const double c = rint(xl[l] * 0x1p-39);
    xl[l] = fma(-c, 0x1p39, xl[l]);
    xl[l + 1] += c;
  }
  ddv acc{xl[0], 0.0};
#pragma unroll
  for (int l = 1; l < L; ++l) acc = dd_add_d(acc, ldexp(xl[l], CRT_LIMB_BITS * l));
  return acc;
}

// Reconstruction: entry (i, j) from the balanced residues r_t of its
// `count` per-modulus products (int8 planes, entry at plane t, [j*mp + i]).
// S = sum_t r_t W_t is congruent to the product X modulo M, and
// |S| <= 32 * 128 * M.  In base 256, S_d = sum_t r_t W_t,d (balanced digits of the
// weights, |S_d| < 2^19) is a product of a 32 x 32 matrix of weights and the
// residues: one v_mfma_i32_32x32x32_i8 for 32 entries, exact.  Four digits make
// a limb of 32 bits (|.| < 2^44, exact in binary64); q = rint(S / M) (estimated
// as sum_l S_l g_l, error far below the 1/4 margin: |X| <= M/4) is removed limb
// by limb (|q M_l| < 2^45: exact), which leaves the exact integer X = S - q M in
// limbs; carries bring every limb but the top one into [-2^31, 2^31] (each step
// exact), and the limbs are added into a dd from the lowest up (DWPlusFP:
// relative error about 2^-104 overall).  Finally X 2^(sigma_i + tau_j - 2P)
// and C = alpha X' + beta C, as in oz_combine.
//
// Lanes l and l + 32 share a group of four consecutive rows: each loads the group's
// 4-byte words of 16 planes and transposes them into the products' operands; lane
// half h receives digits 16 h .. 16 h + 15 of all four entries, forms their limbs
// and exchanges half of them, so that it finishes rows 2 h and 2 h + 1.  A
// triangle (tri 1 upper, 2 lower) updates only its entries.
//
// Bound: vector instructions (the sums in 39-bit limbs by binary64 fmas, 250 of
// the 420 operations an entry, are 60 here) and the residues' and C's bytes:
// 1024^2, 31 planes 23.8 -> 19.0 us (64 MB, 14.6 us as a copy); 2048^2, 26
// planes 91.7 -> 69.8 us.
//
// SPLIT (a product of oz_crt_long): plane t of split s at s * count + t; the splits'
// products are added (|S_d| < 2^23 for up to 16), and the guard's comparison is
// made here, on the sums of the magnitude products.
template <bool SPLIT>
__global__ void __launch_bounds__(256)
oz_crt_combine(const int8_t* __restrict__ x, int64_t mp, int64_t np, int count, int p,
               const int* __restrict__ ea, const int* __restrict__ eb,
               int64_t m, int64_t n, double alpha_hi, double alpha_lo, double beta_hi,
               double beta_lo, int beta_zero, double* __restrict__ c_hi,
               double* __restrict__ c_lo, int64_t ldc, int tri,
               CrtFailed failed, CrtSplitSum sum) {
  typedef int v16i __attribute__((ext_vector_type(16)));
  const CrtSum& cst = kCrtSums.c[count - 1];
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int64_t mq = (m + 3) / 4, groups = mq * n;
  const int64_t first = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32;
  if (first >= groups) return;                   // (a whole wave)
  const bool there = first + (lane & 31) < groups;
  const int64_t gid = there ? first + (lane & 31) : groups - 1;
  const int64_t i0 = (gid % mq) * 4, j = gid / mq;
  const int64_t ilo = (tri == 2) ? j : 0, ihi = (tri == 1) ? j : m - 1;
  if (__ballot(there && !(i0 > ihi || i0 + 3 < ilo)) == 0) return;
  // a guarded product: entries that failed are dd_gemm_failed's
  const int64_t plane = mp * np;
  uint32_t skip = 0u;
  if constexpr (SPLIT) {
    // (mp is a multiple of 64: the four rows are there)
    v4i g{};
    for (int q = 0; q < sum.splits; ++q) g += *(const v4i*)(sum.mag + q * plane + j * mp + i0);
    const float4 ti = *(const float4*)(sum.ta + i0);
    const int4 bi4 = *(const int4*)(sum.ba + i0);
    const float tj = sum.bb[j] ? __builtin_nanf("") : sum.tb[j];
    const uint32_t f0 = (bi4.x != 0) | !((float)g[0] >= ti.x + tj);
    const uint32_t f1 = (bi4.y != 0) | !((float)g[1] >= ti.y + tj);
    const uint32_t f2 = (bi4.z != 0) | !((float)g[2] >= ti.z + tj);
    const uint32_t f3 = (bi4.w != 0) | !((float)g[3] >= ti.w + tj);
    skip = f0 | (f1 << 8) | (f2 << 16) | (f3 << 24);
    if (h == 0 && there) {
      *(uint32_t*)(sum.entry + j * mp + i0) = skip;
      if (skip) sum.block[(j >> 6) * (mp >> 6) + (i0 >> 6)] = 1;
    }
  } else if (failed.entry) {
    skip = *(const uint32_t*)(failed.entry + j * mp + i0);
  }
  // this lane's two rows
  bool mine[2];
  double ch[2] = {0.0, 0.0}, cl[2] = {0.0, 0.0};
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int64_t i = i0 + 2 * h + r;
    mine[r] = there && i < m && i >= ilo && i <= ihi && !((skip >> (8 * (2 * h + r))) & 1u);
    if (!beta_zero && mine[r]) {
      ch[r] = c_hi[i + j * ldc];
      cl[r] = c_lo[i + j * ldc];
    }
  }
  if (__ballot(mine[0] || mine[1]) == 0) return;
  const v4i wt = *(const v4i*)&cst.w[lane & 31][16 * h];
  v16i sd[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) sd[e] = v16i{};
  const int8_t* xp = x + j * mp + i0;
  const int splits = SPLIT ? sum.splits : 1;
  for (int q = 0; q < splits; ++q) {
    uint32_t v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      // (planes past the moduli have weight 0)
      const int t = min(16 * h + u, count - 1);
      v[u] = *(const uint32_t*)(xp + (int64_t)t * plane);
    }
    xp += (int64_t)count * plane;
    v4i op[4];                                   // [entry]: its 16 residues
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t *w = v + 4 * c;
      // bytes 0 0' 1 1' and 2 2' 3 3' of two words
      const uint32_t l01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
      const uint32_t h01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
      const uint32_t l23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
      const uint32_t h23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
      op[0][c] = (int)__builtin_amdgcn_perm(l23, l01, 0x05040100u);
      op[1][c] = (int)__builtin_amdgcn_perm(l23, l01, 0x07060302u);
      op[2][c] = (int)__builtin_amdgcn_perm(h23, h01, 0x05040100u);
      op[3][c] = (int)__builtin_amdgcn_perm(h23, h01, 0x07060302u);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      sd[e] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wt, op[e], sd[e], 0, 0, 0);
  }
  const ddv alpha{alpha_hi, alpha_lo}, beta{beta_hi, beta_lo};
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    // limbs of entries r and r + 2 (this half's four each); after the exchange
    // s[0 .. 3] are the low and s[4 .. 7] the high limbs of entry r + 2 h
    double s[8];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      double v[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const v16i& y = sd[r + 2 * e];
        const int lo = y[4 * l + 1] * 256 + y[4 * l], hi = y[4 * l + 3] * 256 + y[4 * l + 2];
        v[e] = fma((double)hi, 65536.0, (double)lo);
      }
      const uint64_t b0 = __builtin_bit_cast(uint64_t, v[0]);
      const uint64_t b1 = __builtin_bit_cast(uint64_t, v[1]);
      const auto xl = __builtin_amdgcn_permlane32_swap((uint32_t)b0, (uint32_t)b1, false, false);
      const auto xh = __builtin_amdgcn_permlane32_swap((uint32_t)(b0 >> 32), (uint32_t)(b1 >> 32),
                                                       false, false);
      s[l] = __builtin_bit_cast(double, (uint64_t)xl[0] | ((uint64_t)xh[0] << 32));
      s[l + 4] = __builtin_bit_cast(double, (uint64_t)xl[1] | ((uint64_t)xh[1] << 32));
    }
    if (!mine[r]) continue;
    double est = 0.0;
#pragma unroll
    for (int l = 7; l >= 0; --l) est = fma(s[l], cst.g[l], est);
    const double qm = rint(est);
#pragma unroll
    for (int l = 0; l < 8; ++l) s[l] = fma(-qm, cst.ml[l], s[l]);
#pragma unroll
    for (int l = 0; l < 7; ++l) {
      const double c = rint(s[l] * 0x1p-32);
      s[l] = fma(-c, 0x1p32, s[l]);
      s[l + 1] += c;
    }
    ddv acc{s[0], 0.0};
    double unit = 1.0;
#pragma unroll
    for (int l = 1; l < 8; ++l) {
      unit *= 0x1p32;
      acc = dd_add_d(acc, s[l] * unit);
    }
    const int64_t i = i0 + 2 * h + r;
    const int e = ea[i] + eb[j] - 2 * p;
    ddv pr{ldexp(acc.hi, e), ldexp(acc.lo, e)};
    ddv res = dd_mul(alpha, pr);
    const int64_t ci = i + j * ldc;
    if (!beta_zero) res = dd_add(res, dd_mul(beta, ddv{ch[r], cl[r]}));
    c_hi[ci] = res.hi;
    c_lo[ci] = res.lo;
  }
}

// Guarded product with a short operand Y (64 of its rows at a time: block
// vectors, panels) and a long one X.  The pipeline above would write X's
// residues and read them back, 64 bytes an entry where the entry has 16, which takes
// as long as the plain product by 64 columns; here a workgroup converts its 32
// rows of X step by step (64 terms) into LDS and multiplies them at once.  X's
// entries are read here once, and once (the high words) by oz_crt_scale.
//
// Two kinds of waves, one barrier a step, LDS double buffered: 4 convert step s + 1
// while 8 multiply step s, each of these 4 planes, whose 32 x 64 products stay in
// 128 registers.  (All waves doing both, the conversion of a step waited for the
// products' operands from L2 and the next entries from memory, and the registers
// spilled: 670 to 880 us at 8192 x 64 x 8192, this way 580.)
//
// Conversion, on the matrix cores: the grid integer x' = sum_c v_c 2^(30 c)
// (c = 0 .. 3; |v_c| < 2^31, |v_3| < 2^23) gives 15 balanced bytes, each v_c
// its four by (v + 0x808080) ^ 0x808080; times the digits' weights modulo
// every modulus (kCrtDigits), |y| <= 2^18, by one v_mfma_i32_32x32x16_i8
// per 32 entries, whose lane (modulus, l / 32) ends up with 4 consecutive l of
// four rows.  Reduction in binary32: q = rint(y (1/m)), within 2^-14 of y/m, which is
// at least 1/510 from a half-integer for odd m, by a fused multiply-add of
// 1.5 2^23, and the low byte of y - q m by a 24-bit multiply-add: 3 operations
// where the binary64 residues of oz_crt_residues take 6.  The last plane takes
// the guard's magnitude digits (as there), which travel as byte 3 of v_3.
//
// LDS: plane t at t * 2048; 16 bytes (l) of row r, chunk c at slot
// (64 (r / 16) + 16 c + (r % 16)) ^ (t % 16), so that neither the stores (32 planes
// at once) nor the fragment reads meet in a bank.  Y's planes are stored
// [l / 64][row][64]: a step of a plane is 4 KB in one piece (row by row, 8 KB
// apart, they met in one L2 channel: 1230 us).  SWAP: X is op(B) (its rows are
// columns of C).  The k range is split over workgroups where row blocks are few;
// the reconstruction adds the splits.
//
// Bound: the converting waves' vector instructions, one wave a SIMD, 6 clocks each
// (~1300 a step), 4.5 us a step; the memory time of X is 1.9 us of it.  8192 x 64 x
// 8192: 613 us in a trace, with scale, Y's residues and reconstruction 670 to 706
// (plain kernel 1400, pipeline 1390).
constexpr int LONG_PRODUCTS = 8, LONG_CONVERT = 4;   // waves of each kind

template <bool SWAP>
__global__ void __launch_bounds__(64 * (LONG_PRODUCTS + LONG_CONVERT), 3)
oz_crt_long(CrtOperand op, CrtLong q) {
  typedef int v16i __attribute__((ext_vector_type(16)));
  constexpr int PLANE = 2048;
  __shared__ __attribute__((aligned(16))) int8_t smem[2][CRT_MAX_MODULI * PLANE];
  __shared__ int rowexp[32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the column blocks of a row block land 8 apart (on one XCD, one after the
  // other), so that X's step comes from its L2 the second time
  const int per = q.rbs * q.cbs;
  const int split = (int)blockIdx.x / per;
  int b = (int)blockIdx.x % per;
  const int full = q.rbs / 8 * 8;
  int rb, cb;
  if (b < full * q.cbs) {
    const int g = b / (8 * q.cbs), rem = b % (8 * q.cbs);
    cb = rem / 8;
    rb = 8 * g + rem % 8;
  } else {
    b -= full * q.cbs;
    cb = b / (q.rbs - full);
    rb = full + b % (q.rbs - full);
  }
  const int64_t r0 = (int64_t)rb * 32, c0 = (int64_t)cb * 64;
  if (blockIdx.x == 0)
    for (int i = tid; i < q.blocks; i += 64 * (LONG_PRODUCTS + LONG_CONVERT)) q.block[i] = 0;
  bool taken = false;            // a row (tid < 512), a column that may take this path
  if (tid >= 512 && tid < 576) {
    const int64_t y = c0 + tid - 512;
    const float t = q.ythr[y];
    taken = y < q.yused && t == t;
  }
  if (tid < 512) {
    // the rows' exponents and thresholds from their chunks' partial values
    const int row = tid >> 4;
    double mx = 0.0, sum = 0.0, mags = 0.0;
    if (r0 + row < op.rows && (tid & 15) < q.nch) {
      const int64_t at = (int64_t)(tid & 15) * op.rows + r0 + row;
      mx = op.pmax[at];
      sum = op.psum[at];
      mags = op.pabs[at];
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      mx = fmax(mx, __shfl_xor(mx, off));
      sum += __shfl_xor(sum, off);
      mags += __shfl_xor(mags, off);
    }
    int ex = 0;
    if (mx != 0.0) frexp(mx, &ex);
    const float thr = crt_threshold(mx, sum, mags, ex, q.coef);
    taken = r0 + row < op.rows && thr == thr;
    if ((tid & 15) == 0) {
      rowexp[row] = ex;
      if (cb == 0 && split == 0) {
        if (r0 + row < op.rows) op.exps[r0 + row] = ex;
        op.thr[r0 + row] = thr;
      }
    }
  }
  // (every entry fails by its threshold: what this block would store is not read)
  if (!__syncthreads_or(tid < 512 && taken) || !__syncthreads_or(tid >= 512 && taken)) return;

  const int s0 = split * q.steps_per;
  const int s1 = min(q.steps, s0 + q.steps_per);
  if (wave >= LONG_PRODUCTS) {
    // this lane's entries of a step: row `row`, l = 32 lh + 4 i + lane % 4.  Rows
    // and l past the end re-read the last ones: Y's residues there are zero, and
    // rows past the end are not stored.
    const int mt = wave & 1, lh = (wave - LONG_PRODUCTS) >> 1;
    const int row = 16 * mt + 8 * (lane >> 5) + ((lane & 31) >> 2);
    const int ex = rowexp[row];
    const double scale = ldexp(1.0, q.p - ex), mscale = ldexp(1.0, 7 - q.p);
    const bool rowin = r0 + row < op.rows;
    const int l0 = 32 * lh + (lane & 3), klast = (int)q.k - 1;
    const char* __restrict__ xrow = (const char*)(op.hi + min(r0 + row, op.rows - 1) * op.sr);
    const int64_t lo_at = (const char*)op.lo - (const char*)op.hi, sl8 = op.sl * 8;
    double vh[8], vl[8];
    auto load = [&](int s, int i) {
      const char* at = xrow + (uint32_t)min(s * 64 + l0 + 4 * i, klast) * sl8;
      vh[i] = *(const double*)at;
      vl[i] = *(const double*)(at + lo_at);
    };
    // the lane's modulus (column of the conversion) and its digits' weights
    const int t = lane & 31, h = lane >> 5;
    const long wt = *(const long*)&kCrtDigits.w[t][8 * h];
    const bool last = t == CRT_MAX_MODULI - 1;
    const float minv = last ? 1.0f / 256.0f : (float)kCrtMods.t[t].minv;
    const int negm = last ? -256 : -(int)kCrtMods.t[t].m;
    // where 16 bytes of row h of the wave's 16 go (row + 2 g + 8 half: an XOR)
    const int put = t * PLANE + (64 * mt + 32 * lh + (h ^ (t & 15))) * 16;
    bool denorm = false;
    // the step in vh, vl into out; each entry is replaced by the one a step on
    auto convert = [&](int8_t* out, int next) {
      constexpr double MAGIC = 0x1.8p52;       // x + MAGIC: rint(x), its low word the integer
      auto low = [](double v) { return (int)(uint32_t)__builtin_bit_cast(uint64_t, v); };
      auto bytes = [](int v) { return (v + 0x808080) ^ 0x808080; };
      // entry i's digits: [half], digits 0 .. 7 in lanes 0 .. 31 and 8 .. 15 in the
      // others, of rows 0 .. 7 of the wave's 16 and of rows 8 .. 15
      auto digits = [&](int i, long (&dig)[2]) {
        denorm |= !(fabs(vl[i]) * 0x1p52 <= fabs(vh[i]));
        double z = vh[i] * scale, w = vl[i] * scale;
        load(next, i);
        const int g = low(fma(fabs(z), mscale, -0.5) + MAGIC);
        const double q3 = fma(z, 0x1p-90, MAGIC);
        z = fma(-(q3 - MAGIC), 0x1p90, z);
        const double q2 = fma(z, 0x1p-60, MAGIC);
        z = fma(-(q2 - MAGIC), 0x1p60, z);
        const double q1 = fma(z, 0x1p-30, MAGIC);
        z = fma(-(q1 - MAGIC), 0x1p30, z);
        const double qw = fma(w, 0x1p-30, MAGIC);
        w = fma(-(qw - MAGIC), 0x1p30, w);
        const int d0 = bytes(low((z + w) + MAGIC)), d1 = bytes(low(q1) + low(qw));
        const int d2 = bytes(low(q2));
        const int d3 = (bytes(low(q3)) & 0xFFFFFF) | (g << 24);
        const auto e0 = __builtin_amdgcn_permlane32_swap(d0, d2, false, false);
        const auto e1 = __builtin_amdgcn_permlane32_swap(d1, d3, false, false);
#pragma unroll
        for (int half = 0; half < 2; ++half)
          dig[half] = (long)((uint64_t)(uint32_t)e0[half] | ((uint64_t)(uint32_t)e1[half] << 32));
      };
      // the products run one ahead of the reductions (half an entry each)
      long dig[2];
      v16i y[2];
      digits(0, dig);
      y[0] = __builtin_amdgcn_mfma_i32_32x32x16_i8(dig[0], wt, v16i{}, 0, 0, 0);
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        int words[4][2][4];                    // [e][half][g]: row 8 half + 2 g + h
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            if (half == 0) {
              y[1] = __builtin_amdgcn_mfma_i32_32x32x16_i8(dig[1], wt, v16i{}, 0, 0, 0);
            } else if (4 * ch + e < 7) {
              digits(4 * ch + e + 1, dig);
              y[0] = __builtin_amdgcn_mfma_i32_32x32x16_i8(dig[0], wt, v16i{}, 0, 0, 0);
            }
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
              uint32_t r[4];
#pragma unroll
              for (int n = 0; n < 4; ++n) {
                const int yv = y[half][4 * g4 + n];
                const float qf = fmaf((float)yv, minv, 0x1.8p23f);
                // (the low 24 bits of qf's pattern are 2^22 + q, and 2^22 m is
                // 0 modulo 256)
                r[n] = (uint32_t)(__mul24((int)__builtin_bit_cast(uint32_t, qf), negm) + yv);
              }
              words[e][half][g4] = (int)crt_pack4(r[0], r[1], r[2], r[3]);
              // (formed here, not where they are stored)
              asm volatile("" : "+v"(words[e][half][g4]));
            }
          }
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4)
            *(v4i*)(out + (put ^ (128 * half + 32 * g4)) + 256 * ch) =
                v4i{words[0][half][g4], words[1][half][g4], words[2][half][g4],
                    words[3][half][g4]};
      }
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) load(s0, i);
    convert(smem[s0 & 1], s0 + 1);
    __syncthreads();
    for (int s = s0; s < s1; ++s) {
      if (s + 1 < s1) convert(smem[(s + 1) & 1], s + 2);
      __syncthreads();
    }
    if (denorm && rowin) op.bad[r0 + row] = 1;
    return;
  }

  v4i acc[4][2][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[u][a][c] = v4i{};
  // Y's planes of this wave (the last is its magnitude digits, plane `count`;
  // planes past the moduli are computed on it too and not stored), two
  // fragments (32 rows of Y) at a time, the next two on their way
  const int ylane = (int)(c0 + (lane & 15)) * 64 + (lane >> 4) * 16;
  v4i yf[2][2];
  auto fetch = [&](int s, int part) {
    const int8_t* ys = q.yq + (int64_t)min(4 * wave + part / 2, q.count) * q.yplane +
                       (int64_t)s * (q.yrows * 64) + 2048 * (part & 1);
#pragma unroll
    for (int c = 0; c < 2; ++c) yf[part & 1][c] = *(const v4i*)(ys + ylane + 1024 * c);
  };
  fetch(s0, 0);
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    const int8_t* buf = smem[s & 1];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int tp = 4 * wave + u;
      v4i xf[2];
#pragma unroll
      for (int a = 0; a < 2; ++a)
        xf[a] = *(const v4i*)(buf + tp * PLANE + ((64 * a + lane) ^ (tp & 15)) * 16);
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        if (2 * u + part < 7)
          fetch(s, 2 * u + part + 1);
        else if (s + 1 < s1)
          fetch(s + 1, 0);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            v4i& d = acc[u][a][2 * part + c];
            d = SWAP ? __builtin_amdgcn_mfma_i32_16x16x64_i8(yf[part][c], xf[a], d, 0, 0, 0)
                     : __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[a], yf[part][c], d, 0, 0, 0);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
  }
  const int64_t plane = q.mp * q.np;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int tp = 4 * wave + u;
    if (tp >= q.count && tp != CRT_MAX_MODULI - 1) continue;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const v4i v = acc[u][a][c];
        // entry (i, j) of C: four consecutive i
        const int64_t xr = r0 + 16 * a, yr = c0 + 16 * c;
        const int64_t i = (SWAP ? yr : xr) + 4 * (lane >> 4), j = (SWAP ? xr : yr) + (lane & 15);
        if (tp == CRT_MAX_MODULI - 1)
          *(v4i*)(q.mag + (int64_t)split * plane + j * q.mp + i) = v;
        else
          crt_store4(q.x + ((int64_t)split * q.count + tp) * plane + j * q.mp + i, v[0], v[1],
                     v[2], v[3], kCrtMods.t[tp].m, kCrtMods.t[tp].minv);
        __builtin_amdgcn_sched_barrier(0);
      }
  }
}

// Complex reconstruction: plane t, count + t and 2 count + t hold the
// residues of T1 = Ar' Br', T2 = Ai' Bi' and T3 = (Ar' + Ai')(Br' + Bi')
// modulo modulus t; Re X = T1 - T2 and Im X = T3 - T1 - T2 modulo it
// (|.| <= 384 before the reduction, which rint(y (1/m)) m makes balanced
// exactly), each part rebuilt as in oz_crt_combine and scaled by
// 2^(sigma_i + tau_j - 2P) into the dd planes of P (leading dimension ldp);
// the complex alpha / beta update is the caller's.  Four rows per thread.
template <int L>
__global__ void __launch_bounds__(256)
oz_crt_combine_c(const int8_t* __restrict__ x, int64_t mp, int64_t np, int count, int p,
                 const int* __restrict__ ea,
                 const int* __restrict__ eb, int64_t m, int64_t n, double* __restrict__ prh,
                 double* __restrict__ prl, double* __restrict__ pih, double* __restrict__ pil,
                 int64_t ldp, CrtGuard guard) {
  constexpr int NB = 4;
  const CrtCombineConsts& cst = kCrtCombine.c[count - 1];
  const int64_t mq = (m + 3) / 4;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= mq * n) return;
  const int64_t i0 = (gid % mq) * 4, j = gid / mq;
  const int64_t plane = mp * np;
  const int8_t* xp = x + j * mp + i0;
  if (guard.mag) {
    // |Ar||Br| + |Ai||Bi| and |Ar||Bi| + |Ai||Br| bound the plain errors of the two
    // parts; an entry takes both parts plainly if either fails (as in the
    // real guard; mp is a multiple of 64: the four rows are there)
    const int32_t* g = guard.mag + j * mp + i0;
    const v4i re = *(const v4i*)g + *(const v4i*)(g + plane);
    const v4i im = *(const v4i*)(g + 2 * plane) + *(const v4i*)(g + 3 * plane);
    const float tj = guard.bb[j] ? __builtin_nanf("") : guard.tb[j];
    uint32_t failed = 0u;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float t = guard.ba[i0 + r] ? __builtin_nanf("") : guard.ta[i0 + r] + tj;
      failed |= (uint32_t)(!((float)re[r] >= t) | !((float)im[r] >= t)) << (8 * r);
    }
    *(uint32_t*)(guard.entry + j * mp + i0) = failed;
    if (failed) guard.block[(j >> 6) * guard.ldf + (i0 >> 6)] = 1;
    if (failed == 0x01010101u) return;
  }
  double sr[4][L], si[4][L];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int l = 0; l < L; ++l) sr[r][l] = si[r][l] = 0.0;
#pragma unroll
  for (int t0 = 0; t0 < CRT_MAX_MODULI; t0 += NB) {
    if (t0 >= count) break;
    uint32_t v1[NB], v2[NB], v3[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const bool on = t0 + u < count;
      const int8_t* q = xp + (int64_t)(t0 + u) * plane;
      v1[u] = on ? *(const uint32_t*)q : 0u;
      v2[u] = on ? *(const uint32_t*)(q + (int64_t)count * plane) : 0u;
      v3[u] = on ? *(const uint32_t*)(q + (int64_t)2 * count * plane) : 0u;
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int tt = t0 + u;
      if (tt >= count) break;
      const double mm = kCrtMods.t[tt].m, mi = kCrtMods.t[tt].minv;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a1 = (int)(int8_t)(v1[u] >> (8 * r));
        const int a2 = (int)(int8_t)(v2[u] >> (8 * r));
        const int a3 = (int)(int8_t)(v3[u] >> (8 * r));
        const double yr = (double)(a1 - a2), yi = (double)(a3 - a1 - a2);
        const double re = fma(-rint(yr * mi), mm, yr), im = fma(-rint(yi * mi), mm, yi);
#pragma unroll
        for (int l = 0; l < L; ++l) {
          sr[r][l] = fma(re, cst.w[tt][l], sr[r][l]);
          si[r][l] = fma(im, cst.w[tt][l], si[r][l]);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t i = i0 + r;
    if (i >= m) continue;
    const int e = ea[i] + eb[j] - 2 * p;
    const ddv xr = crt_limbs_to_dd<L>(sr[r], cst), xi = crt_limbs_to_dd<L>(si[r], cst);
    const int64_t pi = i + j * ldp;
    prh[pi] = ldexp(xr.hi, e);
    prl[pi] = ldexp(xr.lo, e);
    pih[pi] = ldexp(xi.hi, e);
    pil[pi] = ldexp(xi.lo, e);
  }
}

// qd row operand: residues of X1, X0 and X1 + X0, where X' = X1 2^104 + X0
// is the entry's integer on the grid of 208 bits below 2^sigma_r: each part
// x_p gives t_p = rint(x_p 2^(208 - sigma_r)) (exact scaling), cut into 26-bit
// chunks from the top (j = 7 .. 1: c = rint(t 2^(-26 j)), t -= c 2^(26 j),
// exact; the rest is chunk 0); C_j = sum_p c_pj (|C_j| < 2^28), X0 = sum_{j<4}
// C_j 2^(26 j), X1 = sum_{j>=4} C_j 2^(26 (j-4)).  Per modulus
// y1 = C4 + C5 c26 + C6 c52 + C7 c78 and y0 likewise (< 2^38, exact), each
// reduced as in oz_crt_residues, and the balanced sum of the two residues.
// Planes: X1 residues at q1, X0 at q0, the sums at qs (each count planes of
// rows_p x ldq).  Two of the four parts are staged in LDS at a time
// (37 KB, so the registers, not the LDS, bound the workgroups per CU); a
// thread converts 4 consecutive l of one row (block: 32 rows x
// 64 l) and stores one 4-byte word per modulus and set.  GUARD: magnitude
// digits at plane 3 count, thresholds and marks, as in oz_crt_residues.
template <bool GUARD>
__global__ void __launch_bounds__(512, 2)
oz_crt_residues_qd(CrtQdOperand opa, CrtQdOperand opb, int blocks_a, int64_t k, int nch,
                   int count, int64_t ldq, float coef) {
  constexpr int PITCH = 73;                    // 64 columns + one pad per 8
  __shared__ double t[2][32][PITCH];
  auto col = [](int l) { return l + (l >> 3); };
  const bool first = (int)blockIdx.y < blocks_a;
  const CrtQdOperand& op = first ? opa : opb;
  const double* __restrict__ x0 = op.x[0];
  const double* __restrict__ x1 = op.x[1];
  const double* __restrict__ x2 = op.x[2];
  const double* __restrict__ x3 = op.x[3];
  const int64_t sr = op.s.sr, sl = op.s.sl, rows = op.s.rows, plane = op.s.rows_p * ldq;
  int8_t* __restrict__ q1 = op.s.q;
  int8_t* __restrict__ q0 = q1 + (int64_t)count * plane;
  int8_t* __restrict__ qs = q0 + (int64_t)count * plane;
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)(first ? blockIdx.y : blockIdx.y - blocks_a) * 32;
  const int64_t l0 = (int64_t)blockIdx.x * 64;
  const bool lanes_on_r = (sr == 1);
  const int row = tid >> 4, lq = (tid & 15) * 4;
  // the row's exponent from its chunks' partial maxima, as in oz_crt_residues
  double mx = 0.0, sum = 0.0, mags = 0.0;
  if (r0 + row < rows && (tid & 15) < nch) {
    const int64_t at = (int64_t)(tid & 15) * rows + r0 + row;
    mx = op.s.pmax[at];
    if (GUARD) {
      sum = op.s.psum[at];
      mags = op.s.pabs[at];
    }
  }
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
    mx = fmax(mx, __shfl_xor(mx, off));
    if (GUARD) {
      sum += __shfl_xor(sum, off);
      mags += __shfl_xor(mags, off);
    }
  }
  int ex = 0;
  if (mx != 0.0) frexp(mx, &ex);
  if (l0 == 0 && (tid & 15) == 0) {
    if (r0 + row < rows) op.s.exps[r0 + row] = ex;
    if (GUARD) op.s.thr[r0 + row] = crt_threshold(mx, sum, mags, ex, coef);
  }
  const int sh = CRT_QD_GRID_BITS - ex;
  uint32_t mag = 0u;
  bool denorm = false;
  double last[4] = {0.0, 0.0, 0.0, 0.0};
  double C[8][4];
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) C[j][i] = 0.0;
#pragma unroll
  for (int pair = 0; pair < 2; ++pair) {
    if (pair) __syncthreads();                 // the first pair has been read
    double v[2][4];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const double* __restrict__ src = pair ? (half ? x3 : x2) : (half ? x1 : x0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int e = tid + 512 * c;           // 0 .. 2047 over the 32 x 64 block
        const int ri = lanes_on_r ? (e & 31) : (e >> 6);
        const int li = lanes_on_r ? (e >> 5) : (e & 63);
        const int64_t rg = r0 + ri, lg = l0 + li;
        v[half][c] = (rg < rows && lg < k) ? src[rg * sr + lg * sl] : 0.0;
      }
    }
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int e = tid + 512 * c;
        const int ri = lanes_on_r ? (e & 31) : (e >> 6);
        const int li = lanes_on_r ? (e >> 5) : (e & 63);
        t[half][ri][col(li)] = v[half][c];
      }
    __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double xv = t[half][row][col(lq) + i];
        if (GUARD) {
          // normalised: each part at most half an ulp of the one before
          if (pair == 0 && half == 0)
            mag |= ((uint32_t)(int)ldexp(fabs(xv), 7 - ex) & 0x7Fu) << (8 * i);
          else
            denorm |= !(fabs(xv) * 0x1p52 <= last[i]);
          last[i] = fabs(xv);
        }
        double tv = rint(ldexp(xv, sh));
#pragma unroll
        for (int j = 7; j >= 1; --j) {
          const double c = rint(ldexp(tv, -26 * j));
          tv = fma(-c, ldexp(1.0, 26 * j), tv);
          C[j][i] += c;
        }
        C[0][i] += tv;
      }
  }
  if (l0 + lq >= ldq) return;
  const int64_t off = (r0 + row) * ldq + l0 + lq;
  if (GUARD) {
    if (denorm) op.s.bad[r0 + row] = 1;
    *(uint32_t*)(qs + (int64_t)count * plane + off) = mag;
  }
#pragma unroll
  for (int m = 0; m < CRT_MAX_MODULI; ++m) {
    if (m >= count) break;
    const CrtMod& cm = kCrtMods.t[m];
    const double mm = cm.m, mi = cm.minv;
    const int mint = (int)mm, h = (mint - 1) / 2;
    uint32_t w1 = 0u, w0 = 0u, ws = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double y1 = fma(C[7][i], cm.c78, fma(C[6][i], cm.c52, fma(C[5][i], cm.c26, C[4][i])));
      const double y0 = fma(C[3][i], cm.c78, fma(C[2][i], cm.c52, fma(C[1][i], cm.c26, C[0][i])));
      const int a = (int)(int8_t)crt_reduce(y1, mm, mi), b = (int)(int8_t)crt_reduce(y0, mm, mi);
      int sum = a + b;
      if (m > 0) sum = (sum > h) ? sum - mint : (sum < -h) ? sum + mint : sum;
      w1 |= ((uint32_t)a & 0xFFu) << (8 * i);
      w0 |= ((uint32_t)b & 0xFFu) << (8 * i);
      ws |= ((uint32_t)sum & 0xFFu) << (8 * i);
    }
    *(uint32_t*)(q1 + (int64_t)m * plane + off) = w1;
    *(uint32_t*)(q0 + (int64_t)m * plane + off) = w0;
    *(uint32_t*)(qs + (int64_t)m * plane + off) = ws;
  }
}

// qd reconstruction, one entry per thread: the residues of A = X1 Y1 (planes
// 0 .. count-1), B = X0 Y0 (count ..) and C = (X1 + X0)(Y1 + Y0) (2 count ..)
// give each of the three exactly in 26-bit limbs, as in crt_limbs_to_dd
// (|S_l| < 2^39; q M_l < 2^39), with carries into balanced limbs; then the
// product A 2^208 + (C - A - B) 2^104 + B limb by limb (offsets 8 and 4
// limbs), carried again, and the limbs, scaled by 2^(26 l + sigma_i + tau_j
// - 416), added into a qd from the lowest up, two limbs at a time (TwoSum
// cascade and renormalisation per pair); then C = alpha P + beta C in qd as
// oz_combine_qd.
__global__ void __launch_bounds__(256)
oz_crt_combine_qdm(const int8_t* __restrict__ x, int64_t mp, int64_t np, int count,
                   const int* __restrict__ ea, const int* __restrict__ eb, int64_t m, int64_t n, double4 alpha, double4 beta,
                   int beta_zero, double* __restrict__ c0, double* __restrict__ c1,
                   double* __restrict__ c2, double* __restrict__ c3, int64_t ldc,
                   CrtFailed failed) {
  constexpr int L = CRT_MAX_LIMBS26;
  const CrtCombineConsts26& cst = kCrtCombine26.c[count - 1];
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= m * n) return;
  const int64_t i = gid % m, j = gid / m;
  // (failed entries of a guarded product are qd_gemm_failed's)
  if (failed.entry && failed.entry[j * mp + i]) return;
  const int64_t plane = mp * np;
  const int8_t* xp = x + j * mp + i;
  double sa[L], sb[L], sc[L];
#pragma unroll
  for (int l = 0; l < L; ++l) sa[l] = sb[l] = sc[l] = 0.0;
#pragma unroll
  for (int t = 0; t < CRT_MAX_MODULI; ++t) {
    if (t >= count) break;
    const double ra = (double)xp[(int64_t)t * plane];
    const double rb = (double)xp[(int64_t)(count + t) * plane];
    const double rc = (double)xp[(int64_t)(2 * count + t) * plane];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      sa[l] = fma(ra, cst.w[t][l], sa[l]);
      sb[l] = fma(rb, cst.w[t][l], sb[l]);
      sc[l] = fma(rc, cst.w[t][l], sc[l]);
    }
  }
  // each sum minus its multiple of M, exact limbs
  auto finish = [&](double (&s)[L]) {
    double est = 0.0;
#pragma unroll
    for (int l = L - 1; l >= 0; --l) est = fma(s[l], cst.g[l], est);
    const double qm = rint(est);
#pragma unroll
    for (int l = 0; l < L; ++l) s[l] = fma(-qm, cst.ml[l], s[l]);
  };
  finish(sa);
  finish(sb);
  finish(sc);
  // P = A 2^208 + (C - A - B) 2^104 + B in limbs of 26 bits
  constexpr int T = L + 8;
  double tl[T];
#pragma unroll
  for (int l = 0; l < T; ++l) tl[l] = 0.0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    tl[l] += sb[l];
    tl[l + 4] += sc[l] - sa[l] - sb[l];
    tl[l + 8] += sa[l];
  }
#pragma unroll
  for (int l = 0; l + 1 < T; ++l) {
    const double c = rint(tl[l] * 0x1p-26);
    tl[l] = fma(-c, 0x1p26, tl[l]);
    tl[l + 1] += c;
  }
  // two balanced limbs make one exact binary64 (|l0 + l1 2^26| < 2^52), so
  // the qd takes T / 2 additions
  const int e = ea[i] + eb[j] - 2 * CRT_QD_GRID_BITS;
  qacc p{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int l = 0; l < T; l += 2) {
    const double pair = fma(tl[l + 1], 0x1p26, tl[l]);
    const double v = ldexp(pair, 26 * l + e);
    double er;
    ts(p.s0, v, p.s0, er);
    ts(p.s1, er, p.s1, er);
    ts(p.s2, er, p.s2, er);
    p.s3 = p.s3 + er;
    qd_renorm(p);
  }
  const double4 ps = qd_final(p);
  const int64_t ci = i + j * ldc;
  qacc r{0.0, 0.0, 0.0, 0.0};
  qd_madd(r, alpha, ps);
  if (!beta_zero) {
    qd_renorm(r);
    qd_madd(r, beta, double4{c0[ci], c1[ci], c2[ci], c3[ci]});
  }
  const double4 o = qd_final(r);
  c0[ci] = o.x;
  c1[ci] = o.y;
  c2[ci] = o.z;
  c3[ci] = o.w;
}

// ---- host orchestration -------------------------------------------------------------

static int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

// Digit widths of a kind for k terms and nslices slices.
static bool digit_widths(int algo, int64_t k, int nslices, int& wfirst, int& w) {
  if (algo == MPDD_OZAKI_I8) {
    // |X_d| <= nslices * k * 2^(2w-2) must stay below 2^31: 8-bit later
    // digits (|q| <= 128) while nslices * k < 2^17, 7-bit ones (|q| <= 64)
    // while nslices * k < 2^19
    const int64_t terms = (int64_t)nslices * k;
    wfirst = 6;
    w = (terms < ((int64_t)1 << 17)) ? 8 : 7;
    return terms < ((int64_t)1 << 19);
  }
  int64_t terms = std::max<int64_t>(1, (int64_t)nslices * k);
  int lg = 0;
  while (((int64_t)1 << lg) < terms) ++lg;
  w = (55 - lg) / 2;
  wfirst = w - 1;
  return wfirst >= 1;
}

// Scale exponents + slices of one row operand (rows x k) into padded buffers.
// `part` is scratch for the chunked maxima (rows * ceil(k / OZ_SCALE_CHUNK)
// doubles, only used when the rows are contiguous across lanes).
// Scale exponents of one row operand (rows x k) from its leading plane.
static void scale_operand(const double* hi, int64_t sr, int64_t sl, int64_t rows, int64_t k,
                          int* exps, double* part, hipStream_t st) {
  if (sl == 1 || k == 0) {
    hipLaunchKernelGGL(oz_scale_rows_wave, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st,
                       hi, sr, sl, rows, k, exps);
  } else {
    const int nchunks = (int)((k + OZ_SCALE_CHUNK - 1) / OZ_SCALE_CHUNK);
    hipLaunchKernelGGL(oz_scale_part_cols, dim3((unsigned)((rows + 63) / 64), nchunks), dim3(256),
                       0, st, hi, sr, sl, rows, k, part);
    hipLaunchKernelGGL(oz_scale_finish, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st,
                       part, rows, nchunks, exps);
  }
}

template <typename T>
static hipError_t split_operand(const double* hi, const double* lo, int64_t sr, int64_t sl,
                                int64_t rows, int64_t k, int* exps, T* q, int64_t ldq,
                                int64_t rows_p, int nslices, int wfirst, int w, double* part,
                                hipStream_t st) {
  scale_operand(hi, sr, sl, rows, k, exps, part, st);
  dim3 grid((unsigned)(ldq / 64), (unsigned)(rows_p / 64));
  hipLaunchKernelGGL(oz_slice<T>, grid, dim3(512), 0, st, hi, lo, sr, sl, rows, k, exps, nslices,
                     wfirst, w, q, ldq, rows_p * ldq);
  return hipGetLastError();
}

static size_t part_bytes(int64_t rows, int64_t k) {
  const int64_t nchunks = (k + OZ_SCALE_CHUNK - 1) / OZ_SCALE_CHUNK;
  return (size_t)((rows * std::max<int64_t>(nchunks, 1) * 8 + 255) / 256 * 256);
}

// Workgroup tile (rows, columns) of an INT8 product variant.
static int i8_tile_rows(int var) { return var == 2 ? 128 : 256; }
static int i8_tile_cols(int var) { return (var == 0 || var >= 3) ? 256 : 128; }

// One launch of the INT8 slice products of every anti-diagonal (variant var).
static void launch_i8_products(int var, unsigned nblocks, const int8_t* qa, const int8_t* qb,
                               int32_t* x, int64_t kp, int64_t mp, int64_t np, int s, int tiles_m,
                               int tiles_n, int tri, hipStream_t st) {
  if (var >= 5) {
    auto kern = (var == 5)   ? oz_gemm_i8_dma<256, 256, 2, 4, 4, false, false>
                : (var == 6) ? oz_gemm_i8_dma<256, 256, 2, 4, 4, true, false>
                : (var == 7) ? oz_gemm_i8_dma<256, 256, 2, 2, 4, true, false>
                             : oz_gemm_i8_dma<256, 256, 2, 4, 4, true, true>;
    hipLaunchKernelGGL(kern, dim3(nblocks), dim3(var == 7 ? 256 : 512), 0, st, qa, qb, x, kp,
                       mp * kp, np * kp, mp, np, s, tiles_m, tiles_n, tri, 1, 0, 1,
                       CrtGuard{});
    return;
  }
  auto kern = (var == 0)   ? oz_gemm_i8<256, 256, 2, 2>
              : (var == 1) ? oz_gemm_i8<256, 128, 2, 2>
              : (var == 2) ? oz_gemm_i8<128, 128, 2, 2>
              : (var == 3) ? oz_gemm_i8<256, 256, 2, 4>
                           : oz_gemm_i8<256, 256, 4, 4>;
  const unsigned nthreads = (var == 4) ? 1024 : (var >= 3) ? 512 : 256;
  hipLaunchKernelGGL(kern, dim3(nblocks), dim3(nthreads), 0, st, qa, qb, x, kp, mp * kp, np * kp,
                     mp, np, s, tiles_m, tiles_n, tri);
}

// The residue products of the modular form: one group of workgroups per
// modulus, entries reduced to int8 residues (variants 5, 6 and 8; 6 is the
// default).
static bool crt_variant(int var) { return var == 5 || var == 6 || var == 8; }
constexpr int CRT_VAR_128 = 9;   // 128 x 128 tiles (chosen by crt_tiling only)

// The workgroup tile and planes per workgroup of nprod residue products of an
// m x n result (k padded to kp).  A workgroup takes `group` consecutive planes
// of its tile in turn, which pays the pipeline fill once per group; a launch
// runs in rounds of the workgroups that the chip holds: 256 of 256 x 256 (one
// per CU) or 512 of 128 x 128 (two per CU, each k-step of the pair 0.6 of the
// large tile's time for half its work: the small tile reads twice the LDS
// bytes per product).  The pair with the least rounds x steps is taken: the
// small tile where the large one would leave CUs idle or pad most (512^3), the
// large one from about 1024^3 on.
struct CrtTiling {
  int var, edge, group;
  double cost;
};

static CrtTiling crt_tiling(int var, int tri, int64_t m, int64_t n, int64_t kp, int nprod) {
  const int64_t ksteps = kp / I8_BK;
  constexpr int64_t FILL = 8;                 // k-steps' worth of fill, drain and stores
  CrtTiling best{var >= 0 ? var : 6, 256, 1, 0.0};
  for (int edge = 256; edge >= 128; edge /= 2) {
    if (edge == 128 && var >= 0) break;       // the caller's tiling
    const int tm = (int)((m + edge - 1) / edge), tn = (int)((n + edge - 1) / edge);
    const int64_t tiles = oz_group_tiles(tri, tm, tn);
    const int64_t slots = edge == 256 ? 256 : 512;
    for (int g = 1; g <= 16; ++g) {
      if (g > nprod) break;
      const int64_t wgs = tiles * ((nprod + g - 1) / g);
      const double c = (double)((wgs + slots - 1) / slots) * (double)(g * ksteps + FILL) *
                       (edge == 256 ? 1.0 : 0.6);
      if (best.cost == 0.0 || c < best.cost)
        best = CrtTiling{edge == 256 ? (var >= 0 ? var : 6) : CRT_VAR_128, edge, g, c};
    }
  }
  return best;
}

// nprod products of residue planes (plane t of both operands into plane t
// of x), plane t modulo modulus t % count; with a guard, one more product of
// the magnitude planes, which stores flags.
static void launch_crt_products(const CrtTiling& tl, const int8_t* qa, const int8_t* qb,
                                int8_t* x, int64_t kp, int64_t mp, int64_t np, int nprod,
                                int count, int tri, const CrtGuard& guard,
                                hipStream_t st) {
  auto kern = (tl.var == 5)             ? oz_gemm_i8_dma<256, 256, 2, 4, 4, false, false, true>
              : (tl.var == 6)           ? oz_gemm_i8_dma<256, 256, 2, 4, 4, true, false, true>
              : (tl.var == CRT_VAR_128) ? oz_gemm_i8_dma<128, 128, 2, 2, 4, true, false, true>
                                        : oz_gemm_i8_dma<256, 256, 2, 4, 4, true, true, true>;
  const int tiles_m = (int)(mp / tl.edge), tiles_n = (int)(np / tl.edge);
  const int ngroups = (nprod + tl.group - 1) / tl.group;
  const unsigned nblocks = (unsigned)(oz_group_tiles(tri, tiles_m, tiles_n) * ngroups);
  hipLaunchKernelGGL(kern, dim3(nblocks), dim3(tl.var == CRT_VAR_128 ? 256 : 512), 0, st, qa, qb,
                     (int32_t*)x, kp, mp * kp, np * kp, mp, np, ngroups, tiles_m, tiles_n, tri,
                     count, nprod, tl.group, guard);
}

// Chunks of l of the partial row maxima, and the bytes of one operand's
// partials (maxima, then both sums).
static int64_t crt_chunks(int64_t k) {
  return std::min<int64_t>(CRT_SCALE_CHUNKS, std::max<int64_t>(1, (k + 63) / 64));
}

static size_t crt_part_bytes(int64_t rows) {
  return (size_t)round_up(3 * CRT_SCALE_CHUNKS * rows * (int64_t)sizeof(double), 256);
}

static void crt_set_parts(CrtOperand& op, void* part) {
  op.pmax = (double*)part;
  op.psum = op.pmax + CRT_SCALE_CHUNKS * op.rows;
  op.pabs = op.psum + CRT_SCALE_CHUNKS * op.rows;
}

// Partial row maxima of one operand or (b non-null) of both.
static void launch_crt_scale(const CrtOperand& a, const CrtOperand* b, int64_t k,
                             hipStream_t st) {
  const int ba = (int)(a.rows_p / 64), bb = b ? (int)(b->rows_p / 64) : 0;
  const int64_t nch = crt_chunks(k), chunk = (k + nch - 1) / nch;
  hipLaunchKernelGGL(oz_crt_scale, dim3((unsigned)(ba + bb), (unsigned)nch), dim3(256), 0, st, a,
                     b ? *b : a, ba, k, chunk);
}

// Residues of one operand or of both (their partial maxima first); guarded
// when the operands carry thresholds.
static void launch_crt_residues(const CrtOperand& a, const CrtOperand* b, int64_t k, int count,
                                int p, int64_t ldq, float coef,
                                hipStream_t st) {
  const int ba = (int)(a.rows_p / 32), bb = b ? (int)(b->rows_p / 32) : 0;
  const dim3 grid((unsigned)((ldq + 127) / 128), (unsigned)(ba + bb));
  auto kern = !a.thr ? oz_crt_residues<0> : a.mag ? oz_crt_residues<2> : oz_crt_residues<1>;
  hipLaunchKernelGGL(kern, grid, dim3(512), 0, st, a, b ? *b : a, ba, k, (int)crt_chunks(k),
                     count, p, ldq, coef);
}

// The guard's scratch: thresholds and marks of both operands' rows, a byte per
// entry and per 64 x 64 block.
static size_t crt_guard_bytes(int64_t mp, int64_t np) {
  return (size_t)round_up((mp + np) * 8 + mp * np + (mp / 64) * (np / 64), 256);
}

static CrtGuard crt_guard_at(void* at, int64_t mp, int64_t np, CrtOperand& a, CrtOperand& b) {
  a.thr = (float*)at;
  b.thr = a.thr + mp;
  a.bad = (int*)(b.thr + np);
  b.bad = a.bad + mp;
  CrtGuard g{};
  g.ta = a.thr;
  g.tb = b.thr;
  g.ba = a.bad;
  g.bb = b.bad;
  g.entry = (uint8_t*)(b.bad + np);
  g.block = g.entry + mp * np;
  g.ldf = mp / 64;
  g.plane = -1;
  return g;
}

static void launch_crt_combine(const int8_t* x, int64_t mp, int64_t np, int count,
                               int p, const int* ea, const int* eb,
                               int64_t m, int64_t n, double alpha_hi, double alpha_lo,
                               double beta_hi, double beta_lo, int beta_zero, double* c_hi,
                               double* c_lo, int64_t ldc, int tri, const CrtGuard& guard,
                               hipStream_t st, const CrtSplitSum* sum = nullptr) {
  auto kern = sum ? oz_crt_combine<true> : oz_crt_combine<false>;
  const unsigned cb = (unsigned)(((m + 3) / 4 * n + 127) / 128);
  hipLaunchKernelGGL(kern, dim3(cb), dim3(256), 0, st, x, mp, np, count, p, ea, eb, m, n,
                     alpha_hi, alpha_lo, beta_hi, beta_lo, beta_zero, c_hi, c_lo, ldc, tri,
                     guard.entry ? CrtFailed{guard.block, guard.entry, guard.ldf, mp}
                                 : CrtFailed{},
                     sum ? *sum : CrtSplitSum{});
}

// Modular split form (MPDD_OZAKI_CRT): residues of op(A) and op(B) (a
// triangle: op(A)'s serve both), one INT8 product per modulus, reconstruction.
// alpha = 0 and k = 0 are the caller's.
//
// guarded: the product stands in for the plain one (mpdd.cpp's default route,
// whose comment derives the guard): the grid is CRT_GUARD_BITS wide or more,
// and the entries of C for which its error is not bounded by the plain
// product's are left to the plain kernel, which runs last.  A call
// whose scratch would exceed CRT_GUARD_SCRATCH, or cannot be had, returns
// MPDD_ERR_SCRATCH with nothing enqueued.
constexpr size_t CRT_GUARD_SCRATCH = (size_t)8 << 30;

static int ozaki_crt_gemm(const mpdd_opts* opts, bool guarded, int tri, bool ta, bool tb,
                          int64_t m, int64_t n, int64_t k, double alpha_hi, double alpha_lo,
                          const double* a_hi, const double* a_lo, int64_t lda,
                          const double* b_hi, const double* b_lo, int64_t ldb, double beta_hi,
                          double beta_lo, double* c_hi, double* c_lo, int64_t ldc,
                          hipStream_t st, ScratchCache& pool) {
  if (k > CRT_MAX_K) return MPDD_ERR_UNSUPPORTED;
  int p = 0;
  const int count = guarded ? crt_guard_count(k, &p)
                            : opts->nslices ? opts->nslices : crt_default_count(k);
  if (count < 1 || count > CRT_MAX_MODULI) return MPDD_ERR_UNSUPPORTED;
  if (!guarded) p = crt_exponent(k, count);
  if (p == 0) return MPDD_ERR_UNSUPPORTED;
  const int var = opts && opts->tile_id >= 0 ? opts->tile_id : -1;
  if (var >= 0 && !crt_variant(var)) return MPDD_ERR_UNSUPPORTED;
  const bool beta_zero = beta_hi == 0.0 && beta_lo == 0.0;
  const int64_t kp = round_up(k, 2 * I8_BK);
  const int planes = count + (guarded ? 1 : 0);
  const CrtTiling tl = crt_tiling(var, tri, m, n, kp, planes);
  const int64_t mp = round_up(m, tl.edge), np = round_up(n, tl.edge);
  const size_t qa_bytes = round_up((size_t)planes * mp * kp, 256);
  const size_t qb_bytes = tri ? 0 : round_up((size_t)planes * np * kp, 256);
  const size_t x_bytes = (size_t)count * mp * np;   // int8 residues of the products
  const size_t e_bytes = round_up((m + n) * sizeof(int), 256);
  const size_t pa_bytes = crt_part_bytes(m), pb_bytes = tri ? 0 : crt_part_bytes(n);
  const size_t g_bytes = guarded ? crt_guard_bytes(mp, np) : 0;
  const FailedPlan plan = guarded ? failed_plan(tri, m, n, k) : FailedPlan();
  const size_t total = qa_bytes + qb_bytes + x_bytes + e_bytes + pa_bytes + pb_bytes + g_bytes +
                       plan.bytes;
  if (guarded && total > CRT_GUARD_SCRATCH) return MPDD_ERR_SCRATCH;
  void* ws = nullptr;
  if (pool.get(&ws, total, st, guarded) != hipSuccess)
    return guarded ? MPDD_ERR_SCRATCH : MPDD_ERR_ALLOC;    // (the plain product needs none)
  char* at = (char*)ws;
  auto take = [&](size_t bytes) {
    char* q = at;
    at += bytes;
    return q;
  };
  CrtOperand A{}, B{};
  A.hi = a_hi; A.lo = a_lo;
  A.sr = ta ? lda : 1; A.sl = ta ? 1 : lda;
  A.rows = m; A.rows_p = mp; A.sign = 1.0;
  A.q = (int8_t*)take(qa_bytes);
  B.hi = b_hi; B.lo = b_lo;
  B.sr = tb ? 1 : ldb; B.sl = tb ? ldb : 1;
  B.rows = n; B.rows_p = np; B.sign = 1.0;
  B.q = tri ? A.q : (int8_t*)take(qb_bytes);
  int8_t* x = (int8_t*)take(x_bytes);
  A.exps = (int*)take(e_bytes);
  B.exps = tri ? A.exps : A.exps + m;
  crt_set_parts(A, take(pa_bytes));
  if (!tri) crt_set_parts(B, take(pb_bytes));
  CrtGuard guard{};
  guard.plane = -1;
  float coef = 0.0f;
  if (guarded) {
    guard = crt_guard_at(take(g_bytes), mp, np, A, B);
    guard.plane = count;
    guard.rows = m;
    guard.cols = n;
    if (tri) {                    // op(B)'s columns are op(A)'s rows
      guard.tb = guard.ta;
      guard.bb = guard.ba;
    }
    // 2^(14 + 104 - p - 1), and 2 % for the roundings of the threshold itself
    coef = (float)(1.02 * std::ldexp(1.0, 117 - p));
  }
  launch_crt_scale(A, tri ? nullptr : &B, k, st);
  launch_crt_residues(A, tri ? nullptr : &B, k, count, p, kp, coef, st);
  launch_crt_products(tl, A.q, B.q, x, kp, mp, np, planes, count, tri, guard, st);
  launch_crt_combine(x, mp, np, count, p, A.exps, B.exps, m, n, alpha_hi, alpha_lo,
                     beta_hi, beta_lo, (int)beta_zero, c_hi, c_lo, ldc, tri, guard, st);
  hipError_t e = hipGetLastError();
  if (guarded && e == hipSuccess) {
    GemmParams g{};
    g.m = m; g.n = n; g.k = k;
    g.alpha_hi = alpha_hi; g.alpha_lo = alpha_lo;
    g.beta_hi = beta_hi; g.beta_lo = beta_lo;
    g.a_hi = a_hi; g.a_lo = a_lo; g.lda = lda;
    g.b_hi = b_hi; g.b_lo = b_lo; g.ldb = ldb;
    g.c_hi = c_hi; g.c_lo = c_lo; g.ldc = ldc;
    g.tri = tri;
    g.beta_zero = beta_zero;
    e = launch_gemm_failed(g, ta, tb, CrtFailed{guard.block, guard.entry, guard.ldf, mp}, plan,
                           take(plan.bytes), st);
  }
  const hipError_t ef = pool.put(ws, st);
  if (e != hipSuccess || ef != hipSuccess) return MPDD_ERR_HIP;
  return 0;
}

int ozaki_guarded_gemm(int tri, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                       double alpha_hi, double alpha_lo, const double* a_hi, const double* a_lo,
                       int64_t lda, const double* b_hi, const double* b_lo, int64_t ldb,
                       double beta_hi, double beta_lo, double* c_hi, double* c_lo, int64_t ldc,
                       hipStream_t st, ScratchCache& pool) {
  return ozaki_crt_gemm(nullptr, true, tri, ta, tb, m, n, k, alpha_hi, alpha_lo, a_hi, a_lo, lda,
                        b_hi, b_lo, ldb, beta_hi, beta_lo, c_hi, c_lo, ldc, st, pool);
}

// The k-split of a product of oz_crt_long: rounds of 256 workgroups (one per CU)
// of `steps / splits` steps, and about 5 steps' worth of start and stores; *cost
// in steps.
static int crt_long_splits(int64_t blocks, int64_t steps, int64_t* cost) {
  int best = 1;
  *cost = 0;
  for (int s = 1; s <= 16 && (s == 1 || 4 * s <= steps); ++s) {
    const int64_t c = (blocks * s + 255) / 256 * ((steps + s - 1) / s + 5);
    if (*cost == 0 || c < *cost) {
      best = s;
      *cost = c;
    }
  }
  return best;
}

double guarded_us(int tri, int64_t m, int64_t n, int64_t k) {
  const double in = 1e-6 * (double)(tri ? m : m + n) * (double)k;
  const double out = (tri ? 0.5e-6 : 1e-6) * (double)m * (double)n;
  const CrtTiling tl = crt_tiling(-1, tri, m, n, round_up(k, 2 * I8_BK), CRT_MAX_MODULI);
  return 33.0 + 15.5 * in + 22.0 * out + 1.29 * tl.cost;
}

double guarded_complex_us(int64_t m, int64_t n, int64_t k) {
  const double in = 1e-6 * (double)(m + n) * (double)k, out = 1e-6 * (double)m * (double)n;
  const CrtTiling tl = crt_tiling(-1, 0, m, n, round_up(k, 2 * I8_BK), 3 * CRT_MAX_MODULI + 1);
  return 45.0 + 57.0 * in + 76.0 * out + 1.29 * tl.cost;
}

double guarded_long_us(int64_t m, int64_t n, int64_t k) {
  int p = 0;
  const int count = crt_guard_count(k, &p);
  if (count < 1 || count >= CRT_MAX_MODULI) return 1e30;
  const int64_t lo = std::min(m, n), hi = std::max(m, n);
  int64_t cost = 0;
  crt_long_splits((hi + 63) / 64 * 2 * ((lo + 63) / 64), (k + 63) / 64, &cost);
  return 60.0 + 4.0 * (double)cost + 8.0 / 4.8e6 * (double)hi * (double)k;
}

// The guarded product of a long and a short operand (oz_crt_long); the
// arguments and results of ozaki_guarded_gemm.
int ozaki_guarded_long_gemm(bool ta, bool tb, int64_t m, int64_t n, int64_t k, double alpha_hi,
                            double alpha_lo, const double* a_hi, const double* a_lo, int64_t lda,
                            const double* b_hi, const double* b_lo, int64_t ldb, double beta_hi,
                            double beta_lo, double* c_hi, double* c_lo, int64_t ldc,
                            hipStream_t st, ScratchCache& pool) {
  int p = 0;
  const int count = k <= CRT_MAX_K ? crt_guard_count(k, &p) : 0;
  // 31 moduli: the last of the 32 planes is the magnitude digits'
  if (count < 1 || count >= CRT_MAX_MODULI) return MPDD_ERR_UNSUPPORTED;
  p = std::min(p, CRT_LONG_MAX_BITS);
  const bool swap = n > m, beta_zero = beta_hi == 0.0 && beta_lo == 0.0;
  const int64_t kp = round_up(k, 2 * I8_BK);
  const int64_t mp = round_up(m, 64), np = round_up(n, 64);
  const int64_t xr = swap ? n : m, yr = swap ? m : n, xp = swap ? np : mp, yp = swap ? mp : np;
  CrtLong q{};
  q.k = k; q.yplane = yp * kp; q.yrows = yp;
  q.nch = (int)crt_chunks(k);
  q.p = p; q.count = count;
  q.coef = (float)(1.02 * std::ldexp(1.0, 117 - p));
  q.mp = mp; q.np = np;
  q.steps = (int)((k + 63) / 64);
  q.rbs = (int)(xp / 32); q.cbs = (int)(yp / 64);
  int64_t cost = 0;
  const int splits = crt_long_splits((int64_t)q.rbs * q.cbs, q.steps, &cost);
  q.steps_per = (q.steps + splits - 1) / splits;
  const int parts = (q.steps + q.steps_per - 1) / q.steps_per;   // (no split without steps)
  const size_t y_bytes = round_up((size_t)(count + 1) * yp * kp, 256);
  const size_t x_bytes = round_up((size_t)parts * count * mp * np, 256);
  const size_t mag_bytes = round_up((size_t)parts * mp * np * 4, 256);
  const size_t e_bytes = round_up((m + n) * sizeof(int), 256);
  const size_t px_bytes = crt_part_bytes(xr), py_bytes = crt_part_bytes(yr);
  const size_t g_bytes = crt_guard_bytes(mp, np);
  const FailedPlan plan = failed_plan(0, m, n, k);
  const size_t total = y_bytes + x_bytes + mag_bytes + e_bytes + px_bytes + py_bytes + g_bytes +
                       plan.bytes;
  if (total > CRT_GUARD_SCRATCH) return MPDD_ERR_SCRATCH;
  void* ws = nullptr;
  if (pool.get(&ws, total, st, true) != hipSuccess) return MPDD_ERR_SCRATCH;
  char* at = (char*)ws;
  auto take = [&](size_t bytes) {
    char* r = at;
    at += bytes;
    return r;
  };
  CrtOperand A{}, B{};
  A.hi = a_hi; A.lo = a_lo;
  A.sr = ta ? lda : 1; A.sl = ta ? 1 : lda;
  A.rows = m; A.rows_p = mp; A.sign = 1.0;
  B.hi = b_hi; B.lo = b_lo;
  B.sr = tb ? 1 : ldb; B.sl = tb ? ldb : 1;
  B.rows = n; B.rows_p = np; B.sign = 1.0;
  CrtOperand& X = swap ? B : A;
  CrtOperand& Y = swap ? A : B;
  Y.q = (int8_t*)take(y_bytes);
  Y.stepwise = 1;
  q.yq = Y.q;
  q.x = (int8_t*)take(x_bytes);
  q.mag = (int32_t*)take(mag_bytes);
  A.exps = (int*)take(e_bytes);
  B.exps = A.exps + m;
  crt_set_parts(X, take(px_bytes));
  crt_set_parts(Y, take(py_bytes));
  const CrtGuard guard = crt_guard_at(take(g_bytes), mp, np, A, B);
  q.ythr = Y.thr;
  q.yused = Y.rows;
  q.block = guard.block;
  q.blocks = (int)((mp / 64) * (np / 64));
  launch_crt_scale(X, &Y, k, st);
  launch_crt_residues(Y, nullptr, k, count, p, kp, q.coef, st);
  hipLaunchKernelGGL(swap ? oz_crt_long<true> : oz_crt_long<false>,
                     dim3((unsigned)(q.rbs * q.cbs * parts)), dim3(64 * (LONG_PRODUCTS + LONG_CONVERT)),
                     0, st, X, q);
  const CrtSplitSum sum{q.mag, parts, guard.ta, guard.tb, guard.ba, guard.bb, guard.block,
                        guard.entry};
  launch_crt_combine(q.x, mp, np, count, p, A.exps, B.exps, m, n, alpha_hi, alpha_lo, beta_hi,
                     beta_lo, (int)beta_zero, c_hi, c_lo, ldc, 0, guard, st, &sum);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    GemmParams g{};
    g.m = m; g.n = n; g.k = k;
    g.alpha_hi = alpha_hi; g.alpha_lo = alpha_lo;
    g.beta_hi = beta_hi; g.beta_lo = beta_lo;
    g.a_hi = a_hi; g.a_lo = a_lo; g.lda = lda;
    g.b_hi = b_hi; g.b_lo = b_lo; g.ldb = ldb;
    g.c_hi = c_hi; g.c_lo = c_lo; g.ldc = ldc;
    g.beta_zero = beta_zero;
    e = launch_gemm_failed(g, ta, tb, CrtFailed{guard.block, guard.entry, guard.ldf, mp}, plan,
                           take(plan.bytes), st);
  }
  const hipError_t ef = pool.put(ws, st);
  if (e != hipSuccess || ef != hipSuccess) return MPDD_ERR_HIP;
  return 0;
}

int ozaki_crt_cgemm(const void* opts_v, bool guarded, int opa, int opb, int64_t m, int64_t n, int64_t k,
                    const double* const* a, int64_t lda, const double* const* b, int64_t ldb,
                    double* prh, double* prl, double* pih, double* pil, hipStream_t st,
                    ScratchCache& pool) {
  const mpdd_opts* opts = (const mpdd_opts*)opts_v;
  // (guarded: two magnitude products are added in 32 bits, 2 k 127^2 < 2^31)
  if (k > CRT_MAX_K || (guarded && k > CRT_MAX_K / 2)) return MPDD_ERR_UNSUPPORTED;
  int p = 0;
  const int count = guarded ? crt_guard_count(k, &p, 3)
                            : opts->nslices ? opts->nslices : crt_default_count(k, 3);
  if (count < 1 || count > CRT_MAX_MODULI) return MPDD_ERR_UNSUPPORTED;
  if (!guarded) p = crt_exponent(k, count, 3);
  if (p == 0) return MPDD_ERR_UNSUPPORTED;
  const int var = opts && opts->tile_id >= 0 ? opts->tile_id : -1;
  if (var >= 0 && !crt_variant(var)) return MPDD_ERR_UNSUPPORTED;
  const int limbs = crt_limbs(count);
  const int64_t kp = round_up(k, 2 * I8_BK);
  const int planes = 3 * count + (guarded ? 4 : 0);
  const CrtTiling tl = crt_tiling(var, 0, m, n, kp, planes);
  const int64_t mp = round_up(m, tl.edge), np = round_up(n, tl.edge);
  // three residue sets per operand (re, im, re + im) and three products
  // (and guarded: magnitude digits of the parts, in the order of the four
  // products Gr Gr, Gi Gi, Gr Gi, Gi Gr)
  const size_t qa_bytes = (size_t)planes * mp * kp, qb_bytes = (size_t)planes * np * kp;
  const size_t x_bytes = (size_t)3 * count * mp * np;
  const size_t e_bytes = round_up((m + n) * sizeof(int), 256);
  const size_t g_bytes = guarded ? (size_t)16 * mp * np + crt_guard_bytes(mp, np) : 0;
  const FailedPlan plan = guarded ? failed_plan(0, m, n, k) : FailedPlan();
  const size_t total = round_up(qa_bytes, 256) + round_up(qb_bytes, 256) + round_up(x_bytes, 256) +
                       e_bytes + crt_part_bytes(m) + crt_part_bytes(n) + g_bytes + plan.bytes;
  if (guarded && total > CRT_GUARD_SCRATCH) return MPDD_ERR_SCRATCH;
  void* ws = nullptr;
  if (pool.get(&ws, total, st, guarded) != hipSuccess)
    return guarded ? MPDD_ERR_SCRATCH : MPDD_ERR_ALLOC;
  int8_t* qa = (int8_t*)ws;
  int8_t* qb = qa + round_up(qa_bytes, 256);
  int8_t* x = qb + round_up(qb_bytes, 256);
  int* ea = (int*)(x + round_up(x_bytes, 256));
  int* eb = ea + m;
  char* part = (char*)ea + e_bytes;
  const int64_t sa = (int64_t)count * mp * kp, sb = (int64_t)count * np * kp;
  // one exponent per row over both parts; the imaginary residues negated for
  // a conjugated operand, and the residues of re + im formed beside them
  CrtOperand A{}, B{};
  A.hi = a[0]; A.lo = a[1]; A.hi2 = a[2];
  A.sr = opa ? lda : 1; A.sl = opa ? 1 : lda;
  A.rows = m; A.rows_p = mp; A.sign = 1.0;
  A.exps = ea; A.q = qa;
  crt_set_parts(A, part);
  B.hi = b[0]; B.lo = b[1]; B.hi2 = b[2];
  B.sr = opb ? 1 : ldb; B.sl = opb ? ldb : 1;
  B.rows = n; B.rows_p = np; B.sign = 1.0;
  B.exps = eb; B.q = qb;
  crt_set_parts(B, part + crt_part_bytes(m));
  CrtGuard guard{};
  guard.plane = -1;
  float coef = 0.0f;
  const int64_t ga = mp * kp, gb = np * kp;      // bytes of a residue plane
  if (guarded) {
    int32_t* mag = (int32_t*)(part + crt_part_bytes(m) + crt_part_bytes(n));
    guard = crt_guard_at(mag + 4 * mp * np, mp, np, A, B);
    guard.mag = mag;
    guard.plane = 3 * count;
    guard.rows = m;
    guard.cols = n;
    coef = (float)(1.02 * std::ldexp(1.0, 117 - p));
    A.mag = qa + 3 * sa; A.mag2 = A.mag + 2 * ga;
    B.mag = qb + 3 * sb; B.mag2 = B.mag + 3 * gb;
  }
  launch_crt_scale(A, &B, k, st);
  launch_crt_residues(A, &B, k, count, p, kp, coef, st);
  A.hi = a[2]; A.lo = a[3]; A.q = qa + sa;
  A.sign = opa == 2 ? -1.0 : 1.0;
  A.add_q = qa; A.sum_q = qa + 2 * sa;
  B.hi = b[2]; B.lo = b[3]; B.q = qb + sb;
  B.sign = opb == 2 ? -1.0 : 1.0;
  B.add_q = qb; B.sum_q = qb + 2 * sb;
  if (guarded) {
    A.mag = qa + 3 * sa + ga; A.mag2 = A.mag + 2 * ga;
    B.mag = qb + 3 * sb + gb; B.mag2 = B.mag + gb;
  }
  launch_crt_residues(A, &B, k, count, p, kp, coef, st);
  launch_crt_products(tl, qa, qb, x, kp, mp, np, planes, count, 0, guard, st);
  auto kern = (limbs <= 1)   ? oz_crt_combine_c<1>
              : (limbs == 2) ? oz_crt_combine_c<2>
              : (limbs == 3) ? oz_crt_combine_c<3>
              : (limbs == 4) ? oz_crt_combine_c<4>
              : (limbs == 5) ? oz_crt_combine_c<5>
              : (limbs == 6) ? oz_crt_combine_c<6>
                             : oz_crt_combine_c<7>;
  const unsigned cbk = (unsigned)(((m + 3) / 4 * n + 255) / 256);
  hipLaunchKernelGGL(kern, dim3(cbk), dim3(256), 0, st, x, mp, np, count, p, ea, eb, m, n,
                     prh, prl, pih, pil, m, guard);
  hipError_t e = hipGetLastError();
  if (guarded && e == hipSuccess) {
    // the failed entries: the four plain products
    const double sga = A.sign, sgb = B.sign;
    const double *const ah[4] = {a[0], a[2], a[0], a[2]}, *const al[4] = {a[1], a[3], a[1], a[3]};
    const double *const bh[4] = {b[0], b[2], b[2], b[0]}, *const bl[4] = {b[1], b[3], b[3], b[1]};
    const double al4[4] = {1.0, -sga * sgb, sgb, sga};
    for (int q = 0; q < 4 && e == hipSuccess; ++q) {
      GemmParams g{};
      g.m = m; g.n = n; g.k = k;
      g.alpha_hi = al4[q];
      g.beta_hi = (q & 1) ? 1.0 : 0.0;
      g.beta_zero = (q & 1) ? 0 : 1;
      g.a_hi = ah[q]; g.a_lo = al[q]; g.lda = lda;
      g.b_hi = bh[q]; g.b_lo = bl[q]; g.ldb = ldb;
      g.c_hi = q < 2 ? prh : pih; g.c_lo = q < 2 ? prl : pil; g.ldc = m;
      e = launch_gemm_failed(g, opa != 0, opb != 0,
                             CrtFailed{guard.block, guard.entry, guard.ldf, mp}, plan,
                             (char*)ws + (total - plan.bytes), st);
    }
  }
  const hipError_t ef = pool.put(ws, st);
  if (e != hipSuccess || ef != hipSuccess) return MPDD_ERR_HIP;
  return 0;
}

int ozaki_crt_qgemm(const void* opts_v, bool guarded, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                    const double* alpha, const double* const* a, int64_t lda,
                    const double* const* b, int64_t ldb, const double* beta, int beta_zero,
                    double* const* c, int64_t ldc, hipStream_t st, ScratchCache& pool) {
  const mpdd_opts* opts = (const mpdd_opts*)opts_v;
  const int count = opts && opts->nslices ? opts->nslices : crt_qd_default_count(k);
  if (k > CRT_MAX_K || !crt_qd_count_ok(k, count)) return MPDD_ERR_UNSUPPORTED;
  const int var = opts && opts->tile_id >= 0 ? opts->tile_id : -1;
  if (var >= 0 && !crt_variant(var)) return MPDD_ERR_UNSUPPORTED;
  const int64_t kp = round_up(k, 2 * I8_BK);
  const CrtTiling tl = crt_tiling(var, 0, m, n, kp, 3 * count);
  const int64_t mp = round_up(m, tl.edge), np = round_up(n, tl.edge);
  const int planes = 3 * count + (guarded ? 1 : 0);
  const size_t qa_bytes = (size_t)planes * mp * kp, qb_bytes = (size_t)planes * np * kp;
  const size_t x_bytes = (size_t)3 * count * mp * np;
  const size_t e_bytes = round_up((m + n) * sizeof(int), 256);
  const size_t g_bytes = guarded ? crt_guard_bytes(mp, np) : 0;
  const size_t total = round_up(qa_bytes, 256) + round_up(qb_bytes, 256) + x_bytes + e_bytes +
                       crt_part_bytes(m) + crt_part_bytes(n) + g_bytes;
  if (guarded && total > CRT_GUARD_SCRATCH) return MPDD_ERR_SCRATCH;
  void* ws = nullptr;
  if (pool.get(&ws, total, st, guarded) != hipSuccess)
    return guarded ? MPDD_ERR_SCRATCH : MPDD_ERR_ALLOC;
  int8_t* qa = (int8_t*)ws;
  int8_t* qb = qa + round_up(qa_bytes, 256);
  int8_t* x = qb + round_up(qb_bytes, 256);
  int* ea = (int*)(x + x_bytes);
  int* eb = ea + m;
  char* part = (char*)ea + e_bytes;
  // residue sets: X1 (planes 0 ..), X0 (count ..), X1 + X0 (2 count ..)
  CrtQdOperand A{}, B{};
  for (int t = 0; t < 4; ++t) {
    A.x[t] = a[t];
    B.x[t] = b[t];
  }
  A.s.hi = a[0];
  A.s.sr = ta ? lda : 1; A.s.sl = ta ? 1 : lda;
  A.s.rows = m; A.s.rows_p = mp;
  A.s.exps = ea; A.s.q = qa;
  crt_set_parts(A.s, part);
  B.s.hi = b[0];
  B.s.sr = tb ? 1 : ldb; B.s.sl = tb ? ldb : 1;
  B.s.rows = n; B.s.rows_p = np;
  B.s.exps = eb; B.s.q = qb;
  crt_set_parts(B.s, part + crt_part_bytes(m));
  CrtGuard guard{};
  guard.plane = -1;
  // the default route's guard (mpdd.cpp) for a grid of P = 208 bits and the qd
  // unit 2^-209; each of an entry's parts is rounded to the grid, so the
  // rounding is at most 2^-P:
  //   2^-P 2^(sigma_i + tau_j) (Q_i + Q_j) <= 2 x 2^-209 (|A||B|)_ij
  float coef = 0.0f;
  if (guarded) {
    guard = crt_guard_at(part + crt_part_bytes(m) + crt_part_bytes(n), mp, np, A.s, B.s);
    coef = 1.02f * 0x1p14f;
  }
  launch_crt_scale(A.s, &B.s, k, st);
  hipLaunchKernelGGL(guarded ? oz_crt_residues_qd<true> : oz_crt_residues_qd<false>,
                     dim3((unsigned)(kp / 64), (unsigned)((mp + np) / 32)), dim3(512), 0, st, A,
                     B, (int)(mp / 32), k, (int)crt_chunks(k), count, kp, coef);
  if (guarded) {
    // the magnitude product first: the 90 residue products then skip the
    // tiles of which nothing will be used
    CrtTiling one = tl;
    one.group = 1;
    guard.plane = 0;
    launch_crt_products(one, qa + (size_t)3 * count * mp * kp, qb + (size_t)3 * count * np * kp, x,
                        kp, mp, np, 1, 1, 0, guard, st);
    guard.plane = -1;
    guard.check = 1;
  }
  launch_crt_products(tl, qa, qb, x, kp, mp, np, 3 * count, count, 0, guard, st);
  const CrtFailed failed =
      guarded ? CrtFailed{guard.block, guard.entry, guard.ldf, mp} : CrtFailed{};
  hipLaunchKernelGGL(oz_crt_combine_qdm, dim3((unsigned)((m * n + 255) / 256)), dim3(256), 0, st,
                     x, mp, np, count, ea, eb, m, n,
                     double4{alpha[0], alpha[1], alpha[2], alpha[3]},
                     double4{beta[0], beta[1], beta[2], beta[3]}, beta_zero, c[0], c[1], c[2],
                     c[3], ldc, failed);
  hipError_t e = hipGetLastError();
  if (guarded && e == hipSuccess) {
    QgemmParams q{};
    q.m = m; q.n = n; q.k = k;
    for (int t = 0; t < 4; ++t) {
      q.alpha[t] = alpha[t];
      q.beta[t] = beta[t];
      q.a[t] = a[t];
      q.b[t] = b[t];
      q.c[t] = c[t];
    }
    q.lda = lda; q.ldb = ldb; q.ldc = ldc;
    q.beta_zero = beta_zero;
    e = launch_qgemm_failed(q, ta, tb, failed, st);
  }
  const hipError_t ef = pool.put(ws, st);
  if (e != hipSuccess || ef != hipSuccess) return MPDD_ERR_HIP;
  return 0;
}

int ozaki_gemm(const void* opts_v, int tri, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
               double alpha_hi, double alpha_lo, const double* a_hi, const double* a_lo,
               int64_t lda, const double* b_hi, const double* b_lo, int64_t ldb, double beta_hi,
               double beta_lo, double* c_hi, double* c_lo, int64_t ldc, hipStream_t st,
               ScratchCache& pool) {
  const mpdd_opts* opts = (const mpdd_opts*)opts_v;
  const int algo = opts->algo;
  const bool beta_zero = beta_hi == 0.0 && beta_lo == 0.0;
  if ((alpha_hi == 0.0 && alpha_lo == 0.0) || k == 0) {
    GemmParams p{};
    p.m = m; p.n = n; p.k = k;
    p.beta_hi = beta_hi; p.beta_lo = beta_lo;
    p.c_hi = c_hi; p.c_lo = c_lo; p.ldc = ldc;
    p.beta_zero = beta_zero;
    p.tri = tri;
    return launch_scale(p, st) == hipSuccess ? 0 : MPDD_ERR_HIP;
  }
  if (algo == MPDD_OZAKI_CRT)
    return ozaki_crt_gemm(opts, false, tri, ta, tb, m, n, k, alpha_hi, alpha_lo, a_hi, a_lo, lda, b_hi,
                          b_lo, ldb, beta_hi, beta_lo, c_hi, c_lo, ldc, st, pool);
  int s = opts->nslices;
  if (s == 0) s = (algo == MPDD_OZAKI_I8) ? 16 : 7;
  if (s < 1 || s > 40) return MPDD_ERR_UNSUPPORTED;
  int wfirst, w;
  if (!digit_widths(algo, k, s, wfirst, w)) return MPDD_ERR_UNSUPPORTED;

  const bool i8 = (algo == MPDD_OZAKI_I8);
  // INT8 slice rows are padded to an even number of product k-steps
  const int64_t kp = round_up(k, i8 ? 2 * I8_BK : OZ_KPAD);
  // INT8 product variant (tile_id) and its workgroup tile
  // (default 6: 256 x 256 with 8 waves -- the largest tile, so the least data
  // moved per product, two waves per SIMD -- with the digits loaded straight
  // into a four-stage LDS ring and each step's fragments read during the
  // previous step's MFMAs; fastest measured at n = 4096 and 8192)
  const int var = (i8 && opts->tile_id >= 0) ? opts->tile_id : 6;
  if (i8 && var > 8) return MPDD_ERR_UNSUPPORTED;
  // a triangle is walked in square tiles (variant 1's are 256 x 128)
  if (tri && i8 && var == 1) return MPDD_ERR_UNSUPPORTED;
  const int64_t tbm = i8 ? i8_tile_rows(var) : OZ_BM;
  const int64_t tbn = i8 ? i8_tile_cols(var) : OZ_BN;
  const int64_t mp = round_up(m, i8 ? I8_PAD : OZ_BM), np = round_up(n, i8 ? I8_PAD : OZ_BN);
  const size_t esz = i8 ? 1 : 8;
  const size_t xsz = i8 ? 4 : 8;
  // a triangle (Rsyrk: op(B) = op(A)^T, m == n) uses op(A)'s slices and
  // exponents for op(B) as well: the columns of op(B) are the rows of op(A)
  const size_t qa_bytes = (size_t)s * mp * kp * esz;
  const size_t qb_bytes = tri ? 0 : (size_t)s * np * kp * esz;
  const size_t x_bytes = (size_t)s * mp * np * xsz;
  const size_t e_bytes = round_up((m + n) * sizeof(int), 256);
  const size_t p_bytes = std::max(part_bytes(m, k), part_bytes(n, k));
  const size_t total =
      round_up(qa_bytes, 256) + round_up(qb_bytes, 256) + x_bytes + e_bytes + p_bytes;
  void* ws = nullptr;
  if (pool.get(&ws, total, st) != hipSuccess) return MPDD_ERR_ALLOC;
  char* base = (char*)ws;
  void* qa = base;
  void* qb = tri ? qa : base + round_up(qa_bytes, 256);
  void* x = base + round_up(qa_bytes, 256) + round_up(qb_bytes, 256);
  int* ea = (int*)((char*)x + x_bytes);
  int* eb = tri ? ea : ea + m;
  double* part = (double*)((char*)ea + e_bytes);

  // row operand of A: op(A)(i, l); of B: op(B)(l, j) as element (j, l)
  const int64_t a_sr = ta ? lda : 1, a_sl = ta ? 1 : lda;
  const int64_t b_sr = tb ? 1 : ldb, b_sl = tb ? ldb : 1;
  hipError_t e;
  if (i8) {
    e = split_operand<int8_t>(a_hi, a_lo, a_sr, a_sl, m, k, ea, (int8_t*)qa, kp, mp, s, wfirst, w,
                              part, st);
    if (e == hipSuccess && !tri)
      e = split_operand<int8_t>(b_hi, b_lo, b_sr, b_sl, n, k, eb, (int8_t*)qb, kp, np, s, wfirst,
                                w, part, st);
  } else {
    e = split_operand<double>(a_hi, a_lo, a_sr, a_sl, m, k, ea, (double*)qa, kp, mp, s, wfirst, w,
                              part, st);
    if (e == hipSuccess && !tri)
      e = split_operand<double>(b_hi, b_lo, b_sr, b_sl, n, k, eb, (double*)qb, kp, np, s, wfirst,
                                w, part, st);
  }
  const int tiles_m = (int)(mp / tbm), tiles_n = (int)(np / tbn);
  const unsigned nblocks = (unsigned)(oz_group_tiles(tri, tiles_m, tiles_n) * s);
  if (e == hipSuccess) {
    if (i8)
      launch_i8_products(var, nblocks, (const int8_t*)qa, (const int8_t*)qb, (int32_t*)x, kp, mp,
                         np, s, tiles_m, tiles_n, tri, st);
    else
      hipLaunchKernelGGL(oz_gemm_f64, dim3(nblocks), dim3(256), 0, st, (const double*)qa,
                         (const double*)qb, (double*)x, kp, mp * kp, np * kp, mp, np, s, tiles_m,
                         tiles_n, tri);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    const unsigned cb = (unsigned)(((m + 3) / 4 * n + 255) / 256);
    if (i8)
      hipLaunchKernelGGL(oz_combine<int32_t>, dim3(cb), dim3(256), 0, st, (const int32_t*)x, mp,
                         np, s, wfirst, w, ea, eb, m, n, alpha_hi, alpha_lo, beta_hi, beta_lo,
                         (int)beta_zero, c_hi, c_lo, ldc, tri);
    else
      hipLaunchKernelGGL(oz_combine<double>, dim3(cb), dim3(256), 0, st, (const double*)x, mp, np,
                         s, wfirst, w, ea, eb, m, n, alpha_hi, alpha_lo, beta_hi, beta_lo,
                         (int)beta_zero, c_hi, c_lo, ldc, tri);
    e = hipGetLastError();
  }
  hipError_t ef = pool.put(ws, st);
  if (e != hipSuccess) return MPDD_ERR_HIP;
  return ef == hipSuccess ? 0 : MPDD_ERR_HIP;
}

// Split-form qd Rgemm (INT8 slices): scale and slice op(A) and op(B) from
// their quad-double planes, the same exact slice products per anti-diagonal
// as the dd form, combined in qd.  alpha = 0 and k = 0 are the caller's.
int ozaki_qgemm(const void* opts_v, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                const double* alpha, const double* const* a, int64_t lda,
                const double* const* b, int64_t ldb, const double* beta, int beta_zero,
                double* const* c, int64_t ldc, hipStream_t st, ScratchCache& pool) {
  const mpdd_opts* opts = (const mpdd_opts*)opts_v;
  if (opts->algo != MPDD_OZAKI_I8) return MPDD_ERR_UNSUPPORTED;
  int s = opts->nslices;
  if (s == 0) s = 32;
  if (s < 1 || s > OZ_QD_MAX_SLICES) return MPDD_ERR_UNSUPPORTED;
  int wfirst, w;
  if (!digit_widths(MPDD_OZAKI_I8, k, s, wfirst, w)) return MPDD_ERR_UNSUPPORTED;
  const int var = opts->tile_id >= 0 ? opts->tile_id : 6;
  if (var > 8) return MPDD_ERR_UNSUPPORTED;
  const int64_t kp = round_up(k, 2 * I8_BK);
  const int64_t mp = round_up(m, I8_PAD), np = round_up(n, I8_PAD);
  const size_t qa_bytes = (size_t)s * mp * kp, qb_bytes = (size_t)s * np * kp;
  const size_t x_bytes = (size_t)s * mp * np * sizeof(int32_t);
  const size_t e_bytes = round_up((m + n) * sizeof(int), 256);
  const size_t p_bytes = std::max(part_bytes(m, k), part_bytes(n, k));
  void* ws = nullptr;
  if (pool.get(&ws, round_up(qa_bytes, 256) + round_up(qb_bytes, 256) + x_bytes +
                                      e_bytes + p_bytes, st) != hipSuccess)
    return MPDD_ERR_ALLOC;
  int8_t* qa = (int8_t*)ws;
  int8_t* qb = qa + round_up(qa_bytes, 256);
  int32_t* x = (int32_t*)(qb + round_up(qb_bytes, 256));
  int* ea = (int*)((char*)x + x_bytes);
  int* eb = ea + m;
  double* part = (double*)((char*)ea + e_bytes);
  // row operand of A: op(A)(i, l); of B: op(B)(l, j) as element (j, l)
  const int64_t a_sr = ta ? lda : 1, a_sl = ta ? 1 : lda;
  const int64_t b_sr = tb ? 1 : ldb, b_sl = tb ? ldb : 1;
  scale_operand(a[0], a_sr, a_sl, m, k, ea, part, st);
  hipLaunchKernelGGL(oz_slice_qd, dim3((unsigned)(kp / 64), (unsigned)(mp / 64)), dim3(512), 0,
                     st, a[0], a[1], a[2], a[3], a_sr, a_sl, m, k, ea, s, wfirst, w, qa, kp,
                     mp * kp);
  scale_operand(b[0], b_sr, b_sl, n, k, eb, part, st);
  hipLaunchKernelGGL(oz_slice_qd, dim3((unsigned)(kp / 64), (unsigned)(np / 64)), dim3(512), 0,
                     st, b[0], b[1], b[2], b[3], b_sr, b_sl, n, k, eb, s, wfirst, w, qb, kp,
                     np * kp);
  const int tiles_m = (int)(mp / i8_tile_rows(var)), tiles_n = (int)(np / i8_tile_cols(var));
  launch_i8_products(var, (unsigned)(tiles_m * tiles_n * s), qa, qb, x, kp, mp, np, s, tiles_m,
                     tiles_n, 0, st);
  hipLaunchKernelGGL(oz_combine_qd, dim3((unsigned)((m * n + 255) / 256)), dim3(256), 0, st, x,
                     mp, np, s, wfirst, w, ea, eb, m, n,
                     double4{alpha[0], alpha[1], alpha[2], alpha[3]},
                     double4{beta[0], beta[1], beta[2], beta[3]}, beta_zero, c[0], c[1], c[2],
                     c[3], ldc);
  const hipError_t e = hipGetLastError();
  const hipError_t ef = pool.put(ws, st);
  if (e != hipSuccess || ef != hipSuccess) return MPDD_ERR_HIP;
  return 0;
}

// Exposed building block: scale exponents and digit slices of op(X).
int ozaki_split_entry(int algo, bool trans, int64_t rows, int64_t k, const double* hi,
                      const double* lo, int64_t ld, int nslices, int wfirst, int w, int* exps,
                      void* slices, int64_t ldq, int64_t rows_p, hipStream_t st,
                      ScratchCache& pool) {
  const int64_t sr = trans ? ld : 1, sl = trans ? 1 : ld;
  void* part = nullptr;
  const size_t pb = algo == MPDD_OZAKI_CRT ? crt_part_bytes(rows) : part_bytes(rows, k);
  if (pool.get(&part, pb, st) != hipSuccess) return MPDD_ERR_ALLOC;
  hipError_t e;
  if (algo == MPDD_OZAKI_CRT) {
    // residues: nslices moduli, the grid of crt_exponent (checked by the caller)
    CrtOperand op{};
    op.hi = hi; op.lo = lo;
    op.sr = sr; op.sl = sl; op.rows = rows; op.rows_p = rows_p; op.sign = 1.0;
    op.exps = exps; op.q = (int8_t*)slices;
    crt_set_parts(op, part);
    launch_crt_scale(op, nullptr, k, st);
    launch_crt_residues(op, nullptr, k, nslices, crt_exponent(k, nslices), ldq, 0.0f, st);
    e = hipGetLastError();
  } else if (algo == MPDD_OZAKI_I8)
    e = split_operand<int8_t>(hi, lo, sr, sl, rows, k, exps, (int8_t*)slices, ldq, rows_p,
                              nslices, wfirst, w, (double*)part, st);
  else
    e = split_operand<double>(hi, lo, sr, sl, rows, k, exps, (double*)slices, ldq, rows_p, nslices,
                              wfirst, w, (double*)part, st);
  hipError_t ef = pool.put(part, st);
  if (e != hipSuccess) return MPDD_ERR_HIP;
  return ef == hipSuccess ? 0 : MPDD_ERR_HIP;
}

int ozaki_digit_widths(int algo, int64_t k, int nslices, int* wfirst, int* w) {
  int a, b;
  if (!digit_widths(algo, k, nslices, a, b)) return MPDD_ERR_UNSUPPORTED;
  *wfirst = a;
  *w = b;
  return 0;
}

}  // namespace mpdd
