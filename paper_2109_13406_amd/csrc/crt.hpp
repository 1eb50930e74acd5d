// crt.hpp -- constants of the modular (Chinese-remainder) split form: the
// moduli, the integer grid width P, and the per-modulus constants of its
// residue, product and reconstruction kernels, all formed at compile time.
// Internal to libmpdd.
//
// The form (after the integer modular emulation of a floating-point matrix
// product by Ozaki, Uchino and Imamura, "Ozaki scheme II", 2025, applied to
// dd operands): each row of op(A) and column of op(B) is rounded to integers
// on a grid of P bits below its largest |hi| (x' = rint(zh) + rint((zh -
// rint(zh)) + zl), z = x 2^(P - sigma)); the integers are reduced modulo
// `count` pairwise coprime moduli <= 256 to balanced residues that fit int8;
// one exact INT8 product per modulus; the exact integer product is rebuilt
// from the residues of its entries by Chinese remaindering and rounded to dd.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mpdd {

class ScratchCache;       // scratch.hpp

constexpr int CRT_MAX_MODULI = 32;   // moduli a call may use
constexpr int CRT_MAX_BITS = 104;    // widest grid: the chunks of x' stay below 2^53
constexpr int CRT_LIMB_BITS = 39;    // reconstruction limbs: 32 * 2^7 * 2^39 < 2^52
constexpr int CRT_MAX_LIMBS = 7;     // 7 * 39 >= 257 bits > bits of 256^32
constexpr int64_t CRT_MAX_K = ((int64_t)1 << 17) - 1;   // k 128^2 < 2^31

// Constants of one modulus: m, 1/m, and 2^26, 2^52, 2^78 modulo m (x' = u1
// 2^78 + u0 2^52 + w1 2^26 + w0 in 26-bit chunks); one cache line.
struct CrtMod {
  double m, minv, c26, c52, c78, pad[3];
};
struct CrtMods {
  CrtMod t[CRT_MAX_MODULI];
};

// Reconstruction constants in 26-bit limbs (the qd form, whose three
// sub-products are recombined limb-wise at offsets of 104 = 4 x 26 bits).
constexpr int CRT_LIMB26 = 26;
constexpr int CRT_MAX_LIMBS26 = 10;     // 10 * 26 >= 257
struct CrtCombineConsts26 {
  double w[CRT_MAX_MODULI][CRT_MAX_LIMBS26];
  double ml[CRT_MAX_LIMBS26], g[CRT_MAX_LIMBS26];
};

// The qd form: grid of 208 bits, split at 2^104; its three sub-products
// (each below 2^212 k in magnitude) are recovered when M >= 2^(215 +
// ceil(log2 k)).
constexpr int CRT_QD_GRID_BITS = 208;

// One row operand of a modular product, as its scale and residue kernels take
// it: element (r, l) of the planes at [r*sr + l*sl], r < rows, l < k.
struct CrtOperand {
  const double *hi, *lo;
  const double* hi2;            // a second plane that counts for the row maxima, or null
  int64_t sr, sl, rows, rows_p; // rows_p: rows of a residue plane (padding included)
  double *pmax, *psum, *pabs;   // partial row maxima, sums of squares and of magnitudes
                                // [chunk][rows] (the sums are a guard's)
  int* exps;                    // row exponents
  int8_t* q;                    // residue planes
  double sign;
  const int8_t* add_q;          // complex operands: residues to add, or null
  int8_t* sum_q;                // and where the sums go
  float* thr;                   // guarded products: rows_p thresholds, and
  int* bad;                     // rows_p marks of rows with unnormalised pairs (null: no guard)
  int8_t *mag, *mag2;           // a guarded complex product: where the magnitude digits go, twice
  int stepwise;                 // residue planes as [l / 64][rows_p][64] (oz_crt_long's operand)
};

// A row operand of quad-doubles: its four planes (s: the scale kernel's view
// of the leading one, and the layout).
struct CrtQdOperand {
  const double* x[4];
  CrtOperand s;
};

// The guard of a modular product that stands in for the plain one: residue
// plane `plane` holds magnitude digits instead (-1: no guard), ta / tb and
// ba / bb the operands' thresholds and marks; block and entry as in CrtFailed.
struct CrtGuard {
  const float *ta, *tb;
  const int *ba, *bb;
  uint8_t *block, *entry;
  int64_t ldf;
  int plane;
  int32_t* mag;                 // a complex product: planes from `plane` on are four magnitude
                                // products, stored here as they are [4][np][mp]
  int check;                    // block is there already: skip tiles that failed whole
  int64_t rows, cols;           // of C: skip tiles all of whose rows or columns are refused
                                // (0: don't look)
};
constexpr double CRT_GUARD_MIN_TERMS = 2.0;   // smallest sum (x / 2^sigma)^2 of a row, or
constexpr double CRT_GUARD_MIN_SUM = 4.0;     // smallest sum |x| / 2^sigma
constexpr int CRT_GUARD_MAX_EXP = 400;        // largest |sigma|
constexpr int CRT_GUARD_BITS = 109;           // narrowest grid of the guarded product

// Reconstruction constants: the CRT weights W_t = (M/m_t) ((M/m_t)^-1 mod
// m_t) in base-2^39 limbs; the limbs of M; and g_l = 2^(39 l) / M (rounded),
// which estimate the multiple of M to remove.
struct CrtCombineConsts {
  double w[CRT_MAX_MODULI][CRT_MAX_LIMBS];
  double ml[CRT_MAX_LIMBS], g[CRT_MAX_LIMBS];
};

// The moduli: from 256 down, every integer coprime to all the moduli
// already taken.
struct CrtModuliList {
  int m[CRT_MAX_MODULI];
};
constexpr CrtModuliList crt_make_moduli() {
  CrtModuliList out{};
  int got = 0;
  for (int m = 256; got < CRT_MAX_MODULI && m >= 2; --m) {
    bool ok = true;
    for (int i = 0; i < got && ok; ++i) {
      int a = m, b = out.m[i];
      while (b) {
        const int t = a % b;
        a = b;
        b = t;
      }
      ok = (a == 1);
    }
    if (ok) out.m[got++] = m;
  }
  return out;
}
inline constexpr CrtModuliList CRT_MODULI = crt_make_moduli();

constexpr double crt_pow2(int e) {
  double v = 1.0;
  for (int i = 0; i < e; ++i) v *= 2.0;
  return v;
}

// Unsigned multiword integer, 32-bit words, least significant first (enough
// for the product of 32 moduli <= 256 and a weight below it).
struct CrtBig {
  uint32_t w[10] = {};
  constexpr void mul(uint32_t s) {
    uint64_t carry = 0;
    for (uint32_t& x : w) {
      const uint64_t v = (uint64_t)x * s + carry;
      x = (uint32_t)v;
      carry = v >> 32;
    }
  }
  constexpr uint32_t divmod(uint32_t s) {        // *this /= s; returns the remainder
    uint64_t rem = 0;
    for (int i = 9; i >= 0; --i) {
      const uint64_t v = (rem << 32) | w[i];
      w[i] = (uint32_t)(v / s);
      rem = v % s;
    }
    return (uint32_t)rem;
  }
  constexpr int bits() const {
    for (int i = 9; i >= 0; --i)
      if (w[i]) return 32 * i + 32 - __builtin_clz(w[i]);
    return 0;
  }
  constexpr uint64_t field(int pos, int nbits) const {   // bits [pos, pos + nbits), nbits <= 40
    uint64_t v = 0;
    for (int i = pos >> 5, got = -(pos & 31); got < nbits && i < 10; ++i, got += 32)
      v |= got < 0 ? (uint64_t)w[i] >> -got : (uint64_t)w[i] << got;
    return v & (((uint64_t)1 << nbits) - 1);
  }
  constexpr double approx() const {
    double v = 0.0;
    for (int i = 9; i >= 0; --i) v = v * 4294967296.0 + (double)w[i];
    return v;
  }
};

constexpr CrtBig crt_modulus_product(int count) {
  CrtBig M;
  M.w[0] = 1;
  for (int t = 0; t < count; ++t) M.mul((uint32_t)CRT_MODULI.m[t]);
  return M;
}

struct CrtBits {
  int b[CRT_MAX_MODULI + 1];
};
constexpr CrtBits crt_make_bits() {
  CrtBits out{};
  for (int c = 1; c <= CRT_MAX_MODULI; ++c) out.b[c] = crt_modulus_product(c).bits();
  return out;
}
inline constexpr CrtBits CRT_BITS = crt_make_bits();

// Bit length of M for 1 .. CRT_MAX_MODULI moduli (0 for a count outside that
// range).
inline int crt_modulus_bits(int count) {
  return count < 1 || count > CRT_MAX_MODULI ? 0 : CRT_BITS.b[count];
}

// 39-bit limbs of the reconstruction for `count` moduli.
inline int crt_limbs(int count) {
  return (crt_modulus_bits(count) + CRT_LIMB_BITS - 1) / CRT_LIMB_BITS;
}

// P: the largest P <= CRT_MAX_BITS with 4 k 2^(2P) <= M (so that every
// entry of the integer product, at most k 2^(2P) in magnitude, lies in
// [-M/4, M/4] and is recovered exactly); 0 when count is out of range or
// no P >= 1 fits.
// A complex product (margin 3) needs 8 k 2^(2P) <= M: its parts are sums of
// two products, at most 2 k 2^(2P) in magnitude.
// (Capped at `cap`; the chunks of x' and the sums of its residues stay exact
// up to P = 114: where t2 exceeds 2^51 in magnitude, t1 is a multiple of 2^52
// and v is 0, and |y| < 2^45.)
inline int crt_exponent(int64_t k, int count, int margin = 2, int cap = CRT_MAX_BITS) {
  if (count < 1 || count > CRT_MAX_MODULI) return 0;
  int lk = 0;
  while (((int64_t)1 << lk) < k) ++lk;            // ceil(log2 k), k >= 1
  const int fl = crt_modulus_bits(count) - 1;
  int p = (fl - margin - lk);
  p = p >= 0 ? p / 2 : -1;
  if (p > cap) p = cap;
  return p >= 1 ? p : 0;
}

// Moduli count used when the caller passes 0: the fewest whose grid reaches
// CRT_MAX_BITS for this k (CRT_MAX_MODULI if none does).
inline int crt_default_count(int64_t k, int margin = 2) {
  for (int c = 1; c <= CRT_MAX_MODULI; ++c)
    if (crt_exponent(k, c, margin) == CRT_MAX_BITS) return c;
  return CRT_MAX_MODULI;
}

// The moduli count of a guarded product: the fewest whose grid reaches
// CRT_GUARD_BITS (0: none); *p the grid width they give.
inline int crt_guard_count(int64_t k, int* p, int margin = 2) {
  for (int c = 1; c <= CRT_MAX_MODULI; ++c) {
    *p = crt_exponent(k, c, margin, 114);
    if (*p >= CRT_GUARD_BITS) return c;
  }
  return 0;
}

// The constant tables, which the device code keeps in its constant memory
// (indexed by the moduli count less one).  As kernel arguments, 1.3 to 2.5 KB
// by value, they made a launch cost the host 3.9 us instead of 2.4.
constexpr CrtMods crt_make_mods() {
  CrtMods out{};
  for (int t = 0; t < CRT_MAX_MODULI; ++t) {
    const int m = CRT_MODULI.m[t];
    int r = 1 % m, c[3] = {0, 0, 0};
    for (int e = 1; e <= 78; ++e) {
      r = (2 * r) % m;
      if (e % 26 == 0) c[e / 26 - 1] = r;
    }
    out.t[t] = CrtMod{(double)m, 1.0 / m, (double)c[0], (double)c[1], (double)c[2], {}};
  }
  return out;
}

// Weights of an integer's base-256 digits modulo the moduli (the conversion of
// oz_crt_long): the integer is sum_c v_c 2^(30 c), c = 0 .. 3, and v_c the sum of
// its bytes (balanced) 256^b; byte 3 of v_3 is free and holds the magnitude
// digit, which the last column alone takes.  w[t][4 c + b] = 2^(30 c + 8 b) mod
// m_t, balanced.
struct CrtDigits {
  signed char w[CRT_MAX_MODULI][16];
};
constexpr CrtDigits crt_make_digits() {
  CrtDigits out{};
  for (int t = 0; t + 1 < CRT_MAX_MODULI; ++t) {
    const int m = CRT_MODULI.m[t];
    for (int i = 0; i < 15; ++i) {
      int r = 1 % m;
      for (int e = 0; e < 30 * (i / 4) + 8 * (i % 4); ++e) r = (2 * r) % m;
      out.w[t][i] = (signed char)(2 * r >= m ? r - m : r);   // m = 256: 128 as -128
    }
  }
  out.w[CRT_MAX_MODULI - 1][15] = 1;
  return out;
}

// A guarded product whose one operand (X, at most 64 columns of the other, Y,
// at a time) is converted where it is multiplied: oz_crt_long.
struct CrtLong {
  const int8_t* yq;             // Y's residue planes, its magnitude digits plane `count`
  int64_t k, yplane, yrows;     // bytes and rows of a plane of Y, [l / 64][yrows][64]
  int nch, p, count;
  float coef;
  int8_t* x;                    // residues of the products [split][count][np][mp]
  int32_t* mag;                 // magnitude products [split][np][mp]
  int64_t mp, np;
  int steps, steps_per;         // 64-term steps: all, and of a split
  int rbs, cbs;                 // blocks of 32 rows of X and of 64 of Y
  uint8_t* block;               // the guard's block bytes (cleared here) and their number
  int blocks;
  const float* ythr;            // Y's thresholds, of yused rows
  int64_t yused;
};
constexpr int CRT_LONG_MAX_BITS = 112;          // widest grid: v_3 fits three bytes

// What the reconstruction of such a product needs more: the splits to add up
// and the guard's inputs (mag null: not such a product).
struct CrtSplitSum {
  const int32_t* mag;
  int splits;
  const float *ta, *tb;
  const int *ba, *bb;
  uint8_t *block, *entry;
};

// The weight of modulus t among `count`: (M/m_t) ((M/m_t)^-1 mod m_t).
constexpr CrtBig crt_weight(const CrtBig& M, int t) {
  const int m = CRT_MODULI.m[t];
  CrtBig W = M;
  W.divmod((uint32_t)m);                       // exact: m divides M
  CrtBig tmp = W;
  const int64_t r = tmp.divmod((uint32_t)m);   // M/m_t mod m_t (coprime to m_t)
  // inverse of r modulo m (extended Euclid)
  int64_t a = r, b = m, x0 = 1, x1 = 0;
  while (b) {
    const int64_t q = a / b, ta = a - q * b, tx = x0 - q * x1;
    a = b;
    b = ta;
    x0 = x1;
    x1 = tx;
  }
  W.mul((uint32_t)(((x0 % m) + m) % m));
  return W;
}

// The constants of every count, limbs of BITS bits.
template <typename Consts, int LIMBS, int BITS>
struct CrtCombineTable {
  Consts c[CRT_MAX_MODULI];
};
template <typename Consts, int LIMBS, int BITS>
constexpr CrtCombineTable<Consts, LIMBS, BITS> crt_make_combine() {
  CrtCombineTable<Consts, LIMBS, BITS> out{};
  for (int count = 1; count <= CRT_MAX_MODULI; ++count) {
    Consts& cc = out.c[count - 1];
    const CrtBig M = crt_modulus_product(count);
    for (int t = 0; t < count; ++t) {
      const CrtBig W = crt_weight(M, t);
      for (int l = 0; l < LIMBS; ++l) cc.w[t][l] = (double)W.field(BITS * l, BITS);
    }
    const double minv = 1.0 / M.approx();
    for (int l = 0; l < LIMBS; ++l) {
      cc.ml[l] = (double)M.field(BITS * l, BITS);
      cc.g[l] = minv * crt_pow2(BITS * l);
    }
  }
  return out;
}

// The reconstruction on the matrix cores (oz_crt_combine): the weights of a
// count's moduli in balanced base-256 digits (32 of them), row by row as a
// v_mfma_i32_32x32x32_i8 whose lane half h is to end up with digits 16 h + r, r =
// 0 .. 15, in register r; and M and g_l = 2^(32 l) / M in 32-bit limbs.
struct CrtSum {
  signed char w[32][CRT_MAX_MODULI];
  double ml[8], g[8];
};
struct CrtSums {
  CrtSum c[CRT_MAX_MODULI];
};
constexpr CrtSums crt_make_sums() {
  CrtSums out{};
  for (int count = 1; count <= CRT_MAX_MODULI; ++count) {
    CrtSum& cs = out.c[count - 1];
    const CrtBig M = crt_modulus_product(count);
    for (int t = 0; t < count; ++t) {
      const CrtBig W = crt_weight(M, t);
      int carry = 0;
      for (int d = 0; d < 32; ++d) {
        int v = (int)W.field(8 * d, 8) + carry;
        carry = v >= 128 ? 1 : 0;
        v -= 256 * carry;
        cs.w[8 * ((d % 16) / 4) + 4 * (d / 16) + d % 4][t] = (signed char)v;
      }
    }
    const double minv = 1.0 / M.approx();
    for (int l = 0; l < 8; ++l) {
      cs.ml[l] = (double)M.field(32 * l, 32);
      cs.g[l] = minv * crt_pow2(32 * l);
    }
  }
  return out;
}

inline bool crt_qd_count_ok(int64_t k, int count) {
  if (count < 1 || count > CRT_MAX_MODULI) return false;
  int lk = 0;
  while (((int64_t)1 << lk) < k) ++lk;
  return crt_modulus_bits(count) - 1 >= 215 + lk;
}

inline int crt_qd_default_count(int64_t k) {
  for (int c = 1; c <= CRT_MAX_MODULI; ++c)
    if (crt_qd_count_ok(k, c)) return c;
  return 0;
}

// Complex modular product (ozaki.hip): P = op(A) op(B) of complex dd
// operands (planes re.hi, re.lo, im.hi, im.lo; op 0 'N', 1 'T', 2 'C') into
// the dd planes (prh, prl) + i (pih, pil), leading dimension m, with three
// residue products per modulus (Re = T1 - T2, Im = T3 - T1 - T2).  k >= 1.
// guarded (opts null): in place of the four plain products; also returns
// MPDD_ERR_SCRATCH (nothing enqueued).
int ozaki_crt_cgemm(const void* opts, bool guarded, int opa, int opb, int64_t m, int64_t n, int64_t k,
                    const double* const* a, int64_t lda, const double* const* b, int64_t ldb,
                    double* prh, double* prl, double* pih, double* pil, hipStream_t st,
                    ScratchCache& pool);

// qd modular product (ozaki.hip): C = alpha op(A) op(B) + beta C on qd
// planes (x0..x3), three residue products per modulus (Karatsuba on the
// 2^104 split).  k >= 1, alpha != 0.  guarded (opts null): in place of the
// plain qd product; also returns MPDD_ERR_SCRATCH (nothing enqueued).
int ozaki_crt_qgemm(const void* opts, bool guarded, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                    const double* alpha, const double* const* a, int64_t lda,
                    const double* const* b, int64_t ldb, const double* beta, int beta_zero,
                    double* const* c, int64_t ldc, hipStream_t st, ScratchCache& pool);

}  // namespace mpdd
