// Prime-field arithmetic for BN254 on the CDNA4 integer pipes.
//
// Elements are 8 x 32-bit little-endian limbs in Montgomery form (R = 2^256),
// always fully reduced to [0, m).  Multiplication is word-serial Montgomery
// (coarsely integrated operand scanning) built on 32x32+64 -> 64 multiply-adds,
// which the compiler lowers to v_mad_u64_u32.  The same code serves F_p (curve
// coordinates) and F_r (scalars), selected by a traits class.  Everything is
// __host__ __device__ so the arithmetic can also be exercised on the CPU.
#pragma once
#include <cstdint>
#include "constants.hpp"
#include "divsteps.hpp"

#ifndef __HIPCC__
#define __host__
#define __device__
#define __forceinline__ inline
#endif

#define HD __host__ __device__
#define DEV __host__ __device__ __forceinline__
// large routines are kept out of line so every kernel does not carry its own copy
#if defined(VC_WIDE) || defined(VC_INLINE_HELPERS)
// (the 8-lane kernels hold a few registers per element: their helpers are inlined, so that
// operands passed by reference stay in registers instead of going through scratch memory;
// a one-lane file may ask for the same)
#define NOINL __host__ __device__ __forceinline__
#else
#define NOINL __host__ __device__ __attribute__((noinline))
#endif

struct FpP {
  static constexpr const uint32_t *M = bn::P_MOD;
  static constexpr uint32_t INV = bn::P_INV;
  static constexpr const uint32_t *M29 = bn::P_MOD29;
  static constexpr uint32_t INV29 = bn::P_INV29;
  static constexpr const uint32_t *ONE = bn::P_ONE;
  static constexpr const uint32_t *R2 = bn::P_R2;
  static constexpr const uint32_t *MINUS2 = bn::P_MINUS_2;
};
struct FpR {
  static constexpr const uint32_t *M = bn::R_MOD;
  static constexpr uint32_t INV = bn::R_INV;
  static constexpr const uint32_t *M29 = bn::R_MOD29;
  static constexpr uint32_t INV29 = bn::R_INV29;
  static constexpr const uint32_t *ONE = bn::R_ONE;
  static constexpr const uint32_t *R2 = bn::R_R2;
  static constexpr const uint32_t *MINUS2 = bn::R_MINUS_2;
};

#ifdef VC_WIDE
#include "field_wide.hpp"
#else
struct fe {
  uint32_t l[8];
};

// Host builds may count field multiplications (to state per-operation work exactly).
#if !defined(__HIP_DEVICE_COMPILE__) && defined(VC_COUNT_MULS)
inline uint64_t &fmul_counter() {
  static thread_local uint64_t c = 0;
  return c;
}
#define COUNT_FMUL() (fmul_counter()++)
#else
#define COUNT_FMUL()
#endif

DEV fe fe_zero() {
  fe o;
#pragma unroll
  for (int i = 0; i < 8; i++) o.l[i] = 0;
  return o;
}

DEV fe fe_const(const uint32_t *c) {
  fe o;
#pragma unroll
  for (int i = 0; i < 8; i++) o.l[i] = c[i];
  return o;
}

template <class F> DEV fe f_one() { return fe_const(F::ONE); }

DEV bool fe_is_zero(const fe &a) {
  uint32_t t = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) t |= a.l[i];
  return t == 0;
}

DEV bool fe_eq(const fe &a, const fe &b) {
  uint32_t t = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) t |= a.l[i] ^ b.l[i];
  return t == 0;
}

// a - m if a >= m (a < 2m, a < 2^256)
template <class F> DEV void f_reduce_once(fe &a) {
  uint32_t d[8];
  uint64_t bw = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    uint64_t t = (uint64_t)a.l[i] - F::M[i] - bw;
    d[i] = (uint32_t)t;
    bw = t >> 63;
  }
#pragma unroll
  for (int i = 0; i < 8; i++) a.l[i] = bw ? a.l[i] : d[i];
}

template <class F> DEV fe f_add(const fe &a, const fe &b) {
  fe s;
  uint64_t c = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    c += (uint64_t)a.l[i] + b.l[i];
    s.l[i] = (uint32_t)c;
    c >>= 32;
  }
  f_reduce_once<F>(s);  // m < 2^254, so the sum never carries out of 256 bits
  return s;
}

template <class F> DEV fe f_sub(const fe &a, const fe &b) {
  fe d;
  uint64_t bw = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    uint64_t t = (uint64_t)a.l[i] - b.l[i] - bw;
    d.l[i] = (uint32_t)t;
    bw = t >> 63;
  }
  // add m back when the difference went negative
  uint64_t c = 0;
  uint32_t mask = bw ? 0xffffffffu : 0u;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    c += (uint64_t)d.l[i] + (F::M[i] & mask);
    d.l[i] = (uint32_t)c;
    c >>= 32;
  }
  return d;
}

template <class F> DEV fe f_neg(const fe &a) { return f_sub<F>(fe_zero(), a); }
template <class F> DEV fe f_dbl(const fe &a) { return f_add<F>(a, a); }

// a / 2 mod m
template <class F> DEV fe f_half(const fe &a) {
  uint32_t mask = (a.l[0] & 1) ? 0xffffffffu : 0u;
  uint32_t t[9];
  uint64_t c = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    c += (uint64_t)a.l[i] + (F::M[i] & mask);
    t[i] = (uint32_t)c;
    c >>= 32;
  }
  t[8] = (uint32_t)c;
  fe o;
#pragma unroll
  for (int i = 0; i < 8; i++) o.l[i] = (t[i] >> 1) | (t[i + 1] << 31);
  return o;
}

// ---- products by way of 9 limbs of 29 bits.  With 32-bit limbs every partial product takes
// two more instructions for its carries (583 vector instructions a product, 0.99 us alone on a
// SIMD, 96 G products/s on the device); 29-bit limbs sum up in 64-bit columns without any.
namespace r29 {
static constexpr uint32_t MASK = 0x1fffffffu;

// limb j of a 2^shift: bits [29 j - shift, 29 j - shift + 29) of a
template <int SHIFT> DEV void split(const fe &a, uint32_t *x) {
#pragma unroll
  for (int j = 0; j < 9; j++) {
    const int b = 29 * j - SHIFT;
    if (b < 0) {
      x[j] = (a.l[0] << -b) & MASK;
    } else {
      const int w = b >> 5, s = b & 31;
      uint32_t v = a.l[w] >> s;
      if (s > 3 && w + 1 < 8) v |= a.l[w + 1] << (32 - s);
      x[j] = v & MASK;
    }
  }
}

// t = c (18 columns below 2^62.5) 2^{-261} mod m, below 2 m for a value below m 2^{261}; limbs
// 0 .. 7 below 2^29
template <class F> DEV void mont(uint64_t *c, uint32_t *t) {
#pragma unroll
  for (int k = 0; k < 9; k++) {
    const uint32_t q = ((uint32_t)c[k] * F::INV29) & MASK;
#pragma unroll
    for (int j = 0; j < 9; j++) c[k + j] += (uint64_t)q * F::M29[j];
    c[k + 1] += c[k] >> 29;
  }
#pragma unroll
  for (int j = 0; j < 8; j++) {
    t[j] = (uint32_t)c[9 + j] & MASK;
    c[10 + j] += c[9 + j] >> 29;
  }
  t[8] = (uint32_t)c[17];
}

// the same, canonical and packed for a value below 2 m 2^{261}
template <class F> DEV fe reduce(uint64_t *c) {
  uint32_t t[9];
  mont<F>(c, t);
  fe o;
#pragma unroll
  for (int w = 0; w < 8; w++) {
    const int b = 32 * w, j = b / 29, s = b % 29;
    uint32_t v = t[j] >> s;
    if (j + 1 < 9) v |= t[j + 1] << (29 - s);
    if (s > 26 && j + 2 < 9) v |= t[j + 2] << (58 - s);
    o.l[w] = v;
  }
  f_reduce_once<F>(o);
  return o;
}

DEV void zero_cols(uint64_t *c) {
#pragma unroll
  for (int k = 0; k < 18; k++) c[k] = 0;
}
// o = x y 2^{-261}, o = x^2 2^{-261} (o may be x)
template <class F> DEV void mul(const uint32_t *x, const uint32_t *y, uint32_t *o) {
  uint64_t c[18];
  zero_cols(c);
#pragma unroll
  for (int i = 0; i < 9; i++)
#pragma unroll
    for (int j = 0; j < 9; j++) c[i + j] += (uint64_t)x[i] * y[j];
  mont<F>(c, o);
}
template <class F> DEV void sqr(const uint32_t *x, uint32_t *o) {
  uint64_t c[18];
  zero_cols(c);
#pragma unroll
  for (int i = 0; i < 9; i++) {
    c[2 * i] += (uint64_t)x[i] * x[i];
    const uint32_t d = 2 * x[i];
#pragma unroll
    for (int j = i + 1; j < 9; j++) c[i + j] += (uint64_t)d * x[j];
  }
  mont<F>(c, o);
}
}  // namespace r29

// Montgomery product a b R^{-1} mod m (R = 2^256): (32 a) b 2^{-261}, below 2 m before the last
// subtraction when one operand is below m
template <class F> DEV fe f_mul(const fe &a, const fe &b) {
  COUNT_FMUL();
  uint32_t x[9], y[9];
  r29::split<5>(a, x);
  r29::split<0>(b, y);
  uint64_t c[18];
#pragma unroll
  for (int k = 0; k < 18; k++) c[k] = 0;
#pragma unroll
  for (int i = 0; i < 9; i++)
#pragma unroll
    for (int j = 0; j < 9; j++) c[i + j] += (uint64_t)x[i] * y[j];
  return r29::reduce<F>(c);
}

// the square, 2 (4a)^2 2^{-261}: 45 partial products instead of 81, each once with its
// multiplicity (2 on the diagonal, 4 off it) on one limb
template <class F> DEV fe f_sqr(const fe &a) {
  COUNT_FMUL();
  uint32_t y[9];
  r29::split<2>(a, y);
  uint64_t c[18];
#pragma unroll
  for (int k = 0; k < 18; k++) c[k] = 0;
#pragma unroll
  for (int i = 0; i < 9; i++) {
    c[2 * i] += (uint64_t)(2 * y[i]) * y[i];
    const uint32_t d = 4 * y[i];
#pragma unroll
    for (int j = i + 1; j < 9; j++) c[i + j] += (uint64_t)d * y[j];
  }
  return r29::reduce<F>(c);
}

// small constant multiple by repeated doubling/adding
template <class F> DEV fe f_mul_small(const fe &a, int k) {
  fe acc = fe_zero(), base = a;
  while (k) {
    if (k & 1) acc = f_add<F>(acc, base);
    base = f_dbl<F>(base);
    k >>= 1;
  }
  return acc;
}

template <class F> DEV fe f_to_mont(const fe &a) { return f_mul<F>(a, fe_const(F::R2)); }
template <class F> DEV fe f_from_mont(const fe &a) {
  fe one = fe_zero();
  one.l[0] = 1;
  return f_mul<F>(a, one);
}

// a^e for a fixed 256-bit exponent (little-endian limbs)
template <class F> NOINL fe f_pow(const fe &a, const uint32_t *e) {
  fe acc = f_one<F>();
  for (int i = 255; i >= 0; i--) {
    acc = f_sqr<F>(acc);
    if ((e[i >> 5] >> (i & 31)) & 1) acc = f_mul<F>(acc, a);
  }
  return acc;
}

// the same by sliding windows of up to 4 bits, on loose limbs from start to end (factor 2^{261}: 32 a
// is below 2^5 m, its square's reduction below 8 m, all later values below 2.4 m): 253 squarings and 59
// products of the 8 odd powers for a square root's exponent, a third of the time of f_pow.  e is
// not zero and the same in every lane.
template <class F> DEV fe f_pow_fixed(const fe &a, const uint32_t *e) {
  uint32_t T[8][9], acc[9];
  r29::split<5>(a, T[0]);
  r29::sqr<F>(T[0], acc);
#pragma unroll
  for (int k = 1; k < 8; k++) r29::mul<F>(T[k - 1], acc, T[k]);
  auto bit = [e](int i) { return e[i >> 5] >> (i & 31) & 1; };
  bool first = true;
#pragma unroll 1
  for (int i = 255; i >= 0;) {
    if (!bit(i)) {
      if (!first) r29::sqr<F>(acc, acc);
      i--;
      continue;
    }
    int lo = i >= 3 ? i - 3 : 0;
    while (!bit(lo)) lo++;
    uint32_t d = 0, y[9];
    for (int k = i; k >= lo; k--) d = 2 * d + bit(k);
#pragma unroll
    for (int j = 0; j < 9; j++) y[j] = T[0][j];
#pragma unroll
    for (int k = 1; k < 8; k++)
#pragma unroll
      for (int j = 0; j < 9; j++) y[j] = d >> 1 == (uint32_t)k ? T[k][j] : y[j];
    if (first) {
#pragma unroll
      for (int j = 0; j < 9; j++) acc[j] = y[j];
      first = false;
    } else {
#pragma unroll 1
      for (int k = i; k >= lo; k--) r29::sqr<F>(acc, acc);
      r29::mul<F>(acc, y, acc);
    }
    i = lo - 1;
  }
  // back to the factor 2^{256}: times 2^{256} (bit 24 of limb 8)
  uint64_t c[18];
  r29::zero_cols(c);
#pragma unroll
  for (int j = 0; j < 9; j++) c[8 + j] = (uint64_t)acc[j] << 24;
  return r29::reduce<F>(c);
}

template <class F> NOINL fe f_inv(const fe &a) { return f_pow<F>(a, F::MINUS2); }

// canonical integer compare: a > b
DEV bool fe_gt_canon(const fe &a, const uint32_t *b) {
  bool gt = false, decided = false;
#pragma unroll
  for (int i = 7; i >= 0; i--) {
    if (!decided && a.l[i] != b[i]) {
      gt = a.l[i] > b[i];
      decided = true;
    }
  }
  return gt;
}

DEV bool fe_lt_mod(const fe &a, const uint32_t *m) {
  uint64_t bw = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    uint64_t t = (uint64_t)a.l[i] - m[i] - bw;
    bw = t >> 63;
  }
  return bw != 0;
}

DEV uint32_t fe_word(const fe &a, int i) { return a.l[i]; }
DEV fe fe_from_words(const uint32_t *w) { return fe_const(w); }

// Montgomery-form inverse: (aR)^{-1} R^3 R^{-1} = a^{-1} R (R3 = R^3 mod m); 0 maps to 0
template <class F> NOINL fe f_inv_fast(const fe &A, const uint32_t *R3) {
  if (fe_is_zero(A)) return fe_zero();
  fe r;
  divsteps::inverse<F>(A.l, r.l);
  return f_mul<F>(r, fe_const(R3));
}

#ifdef __HIPCC__
// the same for an input that is equal in every lane of a fully active wavefront
template <class F> __device__ __forceinline__ fe f_inv_uniform(const fe &A, const uint32_t *R3) {
  fe a, r;
#pragma unroll
  for (int i = 0; i < 8; i++) a.l[i] = __builtin_amdgcn_readfirstlane(A.l[i]);
  if (fe_is_zero(a)) return fe_zero();
  divsteps::inverse_uniform<F>(a.l, r.l);
  return f_mul<F>(r, fe_const(R3));
}
#endif
#endif  // VC_WIDE

#define fp_add f_add<FpP>
#define fp_sub f_sub<FpP>
#define fp_neg f_neg<FpP>
#define fp_dbl f_dbl<FpP>
#define fp_mul f_mul<FpP>
#define fp_sqr f_sqr<FpP>
#define fp_half f_half<FpP>
#define fp_inv f_inv<FpP>
#define fr_add f_add<FpR>
#define fr_sub f_sub<FpR>
#define fr_mul f_mul<FpR>
#define fr_inv f_inv<FpR>

#define fp_inv_fast(a) f_inv_fast<FpP>(a, bn::P_R3)
#define fr_inv_fast(a) f_inv_fast<FpR>(a, bn::R_R3)
