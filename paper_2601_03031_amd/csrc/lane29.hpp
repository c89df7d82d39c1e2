// Base-field arithmetic and group law for one lane per element where throughput decides: the
// packed layout (field.hpp) packs, reduces and unpacks around every product, a third of its
// instructions, and the Jacobian formulas test for exceptional cases at every addition.
//
// Numbers are 9 signed limbs of 29 bits with the factor 2^261 (a packed element times 32).  A
// product leaves its limbs centred, in [-2^28, 2^28); sums and differences are limb by limb.  With the
// limbs of the factors of product n within A_n 2^28 and B_n 2^28 (one "unit": 2^28), a sum of products
// with one reduction keeps its 64-bit columns below 2^63 if the A_n B_n add up to at most 12:
// 9 sum A_n B_n + 18 (the reduction's) < 128 = 2^63 / 2^56.  Its value is below 0.5 p + sum |a_n b_n| /
// 169 p, so that no sum of a formula needs a reduction by p.  The formulas of every kernel are run on
// bounds of limbs and values (lane_models.hpp, tests/test_host_lane.py): from the identity on, with affine
// points below 32 p or sums of such added, coordinates stay below 0.81 p on G1 and 0.54 p on G2; the columns
// reach 0.84 of 2^63 at most, limbs 0.63 of 2^31.
#pragma once
#include "curve.hpp"

namespace lane {

struct fl {
  int32_t l[9];
};
static constexpr int32_t HALF = 1 << 28, MASK = (1 << 29) - 1;

#ifdef __HIP_DEVICE_COMPILE__
#define LANE_ORDER() __builtin_amdgcn_sched_barrier(0)
#else
#define LANE_ORDER()
#endif

HD __forceinline__ fl add(const fl &a, const fl &b) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = a.l[j] + b.l[j];
  return o;
}
HD __forceinline__ fl sub(const fl &a, const fl &b) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = a.l[j] - b.l[j];
  return o;
}
HD __forceinline__ fl neg(const fl &a) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = -a.l[j];
  return o;
}
// -a for m = 1, a for 0
HD __forceinline__ fl neg_if(const fl &a, uint32_t m) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = (a.l[j] ^ -(int32_t)m) + (int32_t)m;
  return o;
}
// k a (k units more a limb), k a with the carries taken once (one unit again, for |k| up to 16 and
// limbs within two units)
HD __forceinline__ fl times(const fl &a, int k) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = k * a.l[j];
  return o;
}
HD __forceinline__ fl norm_times(const fl &a, int k) {
  int64_t v[9];
#pragma unroll
  for (int j = 0; j < 9; j++) v[j] = (int64_t)k * a.l[j] + (j < 8 ? HALF : 0);
  fl o;
#pragma unroll
  for (int j = 0; j < 8; j++) o.l[j] = ((int32_t)v[j] & MASK) - HALF + (j ? (int32_t)(v[j - 1] >> 29) : 0);
  o.l[8] = (int32_t)v[8] + (int32_t)(v[7] >> 29);
  return o;
}
HD __forceinline__ fl norm(const fl &a) {
  fl o;
  int32_t h[8];
#pragma unroll
  for (int j = 0; j < 8; j++) h[j] = (a.l[j] + HALF) >> 29;
#pragma unroll
  for (int j = 0; j < 8; j++) o.l[j] = a.l[j] - (h[j] << 29) + (j ? h[j - 1] : 0);
  o.l[8] = a.l[8] + h[7];
  return o;
}

// columns 9 .. 17, each of the lower eight with 2^28 added, as centred limbs
HD __forceinline__ fl centred(const int64_t *c) {
  fl o;
  int64_t carry = 0;
#pragma unroll
  for (int j = 0; j < 8; j++) {
    const int64_t v = c[9 + j] + carry;
    o.l[j] = ((int32_t)v & MASK) - HALF;
    carry = v >> 29;
  }
  o.l[8] = (int32_t)(c[17] + carry);
  return o;
}

// k a + b minus its rounded quotient by p (one unit, within 0.51 p, for |k a + b| below 2^9 p): the
// quotient from the top limb, of which p has 3171406; the limbs below it move that by less than 8
HD __forceinline__ fl reduce(const fl &a, int k, const fl &b) {
  const int32_t q = (int32_t)__builtin_rintf((float)(k * a.l[8] + b.l[8]) * (1.0f / 3171406.0f));
  int64_t v[9];
#pragma unroll
  for (int j = 0; j < 9; j++) v[j] = (int64_t)k * a.l[j] + (b.l[j] + (j < 8 ? HALF : 0)) + (int64_t)-q * (int32_t)FpP::M29[j];
  fl o;
#pragma unroll
  for (int j = 0; j < 8; j++) o.l[j] = ((int32_t)v[j] & MASK) - HALF + (j ? (int32_t)(v[j - 1] >> 29) : 0);
  o.l[8] = (int32_t)v[8] + (int32_t)(v[7] >> 29);
  return o;
}

// (sum_n a_n b_n) 2^{-261} mod p, N products and one reduction.  Written row by row in this order
// because a multiply-add that needs the one before it issues at half the rate.
template <int N> HD __forceinline__ fl dot(const fl *const *a, const fl *const *b) {
  int64_t c[18];
#pragma unroll
  for (int k = 0; k < 18; k++) c[k] = k >= 9 && k < 17 ? HALF : 0;
#pragma unroll
  for (int n = 0; n < N; n++)
#pragma unroll
    for (int j = 0; j < 9; j++) c[j] += (int64_t)a[n]->l[0] * b[n]->l[j];
#pragma unroll
  for (int k = 0; k < 9; k++) {
    LANE_ORDER();
    const uint32_t t = (uint32_t)c[k] * FpP::INV29;
    LANE_ORDER();
    if (k < 8) {
#pragma unroll
      for (int n = 0; n < N; n++)
#pragma unroll
        for (int j = 0; j < 9; j++) c[k + 1 + j] += (int64_t)a[n]->l[k + 1] * b[n]->l[j];
    }
    LANE_ORDER();
    const int32_t m = (int32_t)(t << 3) >> 3;
#pragma unroll
    for (int j = 0; j < 9; j++) c[k + j] += (int64_t)m * (int32_t)FpP::M29[j];
    LANE_ORDER();
    c[k + 1] += c[k] >> 29;
  }
  return centred(c);
}
// a^2 2^{-261}: each product of two limbs once (limbs within three units)
HD __forceinline__ fl sqr(const fl &a) {
  int64_t c[18];
#pragma unroll
  for (int k = 0; k < 18; k++) c[k] = k >= 9 && k < 17 ? HALF : 0;
  int32_t d[9];
#pragma unroll
  for (int j = 0; j < 9; j++) d[j] = 2 * a.l[j];
#pragma unroll
  for (int j = 0; j < 9; j++) c[j] += (int64_t)a.l[0] * (j ? d[j] : a.l[0]);
#pragma unroll
  for (int k = 0; k < 9; k++) {
    LANE_ORDER();
    const uint32_t t = (uint32_t)c[k] * FpP::INV29;
    LANE_ORDER();
#pragma unroll
    for (int j = k + 1; j < 9; j++) c[k + 1 + j] += (int64_t)a.l[k + 1] * (j > k + 1 ? d[j] : a.l[j]);
    LANE_ORDER();
    const int32_t m = (int32_t)(t << 3) >> 3;
#pragma unroll
    for (int j = 0; j < 9; j++) c[k + j] += (int64_t)m * (int32_t)FpP::M29[j];
    LANE_ORDER();
    c[k + 1] += c[k] >> 29;
  }
  return centred(c);
}
HD __forceinline__ fl mul(const fl &a, const fl &b) {
  const fl *x[1] = {&a}, *y[1] = {&b};
  return dot<1>(x, y);
}
// a b + c d
HD __forceinline__ fl mul2(const fl &a, const fl &b, const fl &c, const fl &d) {
  const fl *x[2] = {&a, &c}, *y[2] = {&b, &d};
  return dot<2>(x, y);
}
HD __forceinline__ fl mul4(const fl &a, const fl &b, const fl &c, const fl &d, const fl &e, const fl &f, const fl &g, const fl &h) {
  const fl *x[4] = {&a, &c, &e, &g}, *y[4] = {&b, &d, &f, &h};
  return dot<4>(x, y);
}
// the sum of six products
HD __forceinline__ fl dot6(const fl *const *a, const fl *const *b) { return dot<6>(a, b); }

// a packed element (limbs in [0, 2^29), two units; value below 32 p), and back (of a value below 16 p,
// which leaves y + p in (0, 2 p); the kernels' are below p), canonical
HD __forceinline__ fl in(const fe &x) {
  uint32_t w[9];
  r29::split<5>(x, w);
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = (int32_t)w[j];
  return o;
}
// 2^261 mod p, and a packed element below 0.7 p with centred limbs (a formula takes one factor of each
// product as large as `in` leaves it, not both)
HD __forceinline__ fl small_one() {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = bn::P_ONE29[j];
  return o;
}
HD __forceinline__ fl in_small(const fe &x) { return mul(in(x), small_one()); }
HD __forceinline__ fe out(const fl &x) {
  fl k;  // 2^256
#pragma unroll
  for (int j = 0; j < 9; j++) k.l[j] = j == 8 ? 1 << 24 : 0;
  const fl y = mul(x, k);
  uint32_t t[9];
  int32_t carry = 0;
#pragma unroll
  for (int j = 0; j < 9; j++) {  // y + p
    const int32_t v = y.l[j] + (int32_t)FpP::M29[j] + carry;
    t[j] = j < 8 ? (uint32_t)(v & MASK) : (uint32_t)v;
    carry = v >> 29;
  }
  fe o;
#pragma unroll
  for (int w = 0; w < 8; w++) {
    const int b = 32 * w, j = b / 29, s = b % 29;
    uint32_t v = t[j] >> s;
    if (j + 1 < 9) v |= t[j + 1] << (29 - s);
    if (s > 26 && j + 2 < 9) v |= t[j + 2] << (58 - s);
    o.l[w] = v;
  }
  f_reduce_once<FpP>(o);
  return o;
}

}  // namespace lane
