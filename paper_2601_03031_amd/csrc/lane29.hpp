// Base-field arithmetic and group law for one lane per element where throughput decides: the
// packed layout (field.hpp) packs, reduces and unpacks around every product, a third of its
// instructions, and the Jacobian formulas test for exceptional cases at every addition.
//
// Numbers are 9 signed limbs of 29 bits with the factor 2^261 (a packed element times 32).  A
// product leaves its limbs centred, in [-2^28, 2^28); sums and differences are limb by limb.  With the
// limbs of the factors of product n within A_n 2^28 and B_n 2^28 (one "unit": 2^28), a sum of products
// with one reduction keeps its 64-bit columns below 2^63 if the A_n B_n add up to at most 12:
// 9 sum A_n B_n + 18 (the reduction's) < 128 = 2^63 / 2^56.  Its value is below 0.5 p + sum |a_n b_n| /
// 169 p, so that no sum of a formula needs a reduction by p: with one point's coordinates below 2 p and
// the other's below 2 p, or below 32 p and affine, those of the sum are below 2 p.
//
// The group law is the complete one for y^2 = x^3 + b (J. Renes, C. Costello, L. Batina, "Complete
// addition formulas for prime order elliptic curves", 2016): homogeneous coordinates, the identity
// (0 : 1 : 0) and no exceptional case in groups of odd order.
#pragma once
#include "curve.hpp"
#include "glv.hpp"

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

// a packed element (limbs in [0, 2^29), two units; value below 32 p), and back (of a value below 8 p),
// canonical
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
  for (int j = 0; j < 9; j++) {  // y + p in (0.4 p, 1.6 p)
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

// ---------------------------------------------------------------- the two coordinate fields
// mul, mul2 (a b + c d), add, sub, neg, norm, times, and b3: 3 b x with limbs of one unit
struct G1 {
  using T = fl;
  using O = OpsG1;
  static HD __forceinline__ T in(const fe &x) { return lane::in(x); }
  static HD __forceinline__ fe out(const T &x) { return lane::out(x); }
  static HD __forceinline__ T zero() { return T{}; }
  static HD __forceinline__ T some() { return T{{1}}; }  // an element that is not zero
  static HD __forceinline__ T add(const T &a, const T &b) { return lane::add(a, b); }
  static HD __forceinline__ T sub(const T &a, const T &b) { return lane::sub(a, b); }
  static HD __forceinline__ T neg(const T &a) { return lane::neg(a); }
  static HD __forceinline__ T neg_if(const T &a, uint32_t m) { return lane::neg_if(a, m); }
  static HD __forceinline__ T norm(const T &a) { return lane::norm(a); }
  static HD __forceinline__ T times(const T &a, int k) { return lane::times(a, k); }
  static HD __forceinline__ T mul(const T &a, const T &b) { return lane::mul(a, b); }
  static HD __forceinline__ T mul2(const T &a, const T &b, const T &c, const T &d) { return lane::mul2(a, b, c, d); }
  static HD __forceinline__ T sqr(const T &a) { return lane::sqr(a); }
  static HD __forceinline__ T norm_times(const T &a, int k) { return lane::norm_times(a, k); }
  static HD __forceinline__ T b3(const T &a) { return lane::norm_times(a, 9); }
  static HD __forceinline__ fe inv(const fe &a) { return fp_inv_fast(a); }
};
struct fl2 {
  fl c0, c1;
};
struct G2 {
  using T = fl2;
  using O = OpsG2;
  static HD __forceinline__ T in(const fp2 &x) { return {lane::in(x.c0), lane::in(x.c1)}; }
  static HD __forceinline__ T in_small(const fp2 &x) { return {lane::in_small(x.c0), lane::in_small(x.c1)}; }
  static HD __forceinline__ fp2 out(const T &x) { return {lane::out(x.c0), lane::out(x.c1)}; }
  static HD __forceinline__ T zero() { return T{}; }
  static HD __forceinline__ T some() { return T{{{1}}, {}}; }
  static HD __forceinline__ T add(const T &a, const T &b) { return {lane::add(a.c0, b.c0), lane::add(a.c1, b.c1)}; }
  static HD __forceinline__ T sub(const T &a, const T &b) { return {lane::sub(a.c0, b.c0), lane::sub(a.c1, b.c1)}; }
  static HD __forceinline__ T neg(const T &a) { return {lane::neg(a.c0), lane::neg(a.c1)}; }
  static HD __forceinline__ T neg_if(const T &a, uint32_t m) { return {lane::neg_if(a.c0, m), lane::neg_if(a.c1, m)}; }
  static HD __forceinline__ T norm(const T &a) { return {lane::norm(a.c0), lane::norm(a.c1)}; }
  static HD __forceinline__ T times(const T &a, int k) { return {lane::times(a.c0, k), lane::times(a.c1, k)}; }
  static HD __forceinline__ T mul(const T &a, const T &b) {
    return {lane::mul2(a.c0, b.c0, lane::neg(a.c1), b.c1), lane::mul2(a.c0, b.c1, a.c1, b.c0)};
  }
  static HD __forceinline__ T mul2(const T &a, const T &b, const T &c, const T &d) {
    return {lane::mul4(a.c0, b.c0, lane::neg(a.c1), b.c1, c.c0, d.c0, lane::neg(c.c1), d.c1),
            lane::mul4(a.c0, b.c1, a.c1, b.c0, c.c0, d.c1, c.c1, d.c0)};
  }
  static HD __forceinline__ T sqr(const T &a) {
    return {lane::mul(lane::add(a.c0, a.c1), lane::sub(a.c0, a.c1)), lane::mul(lane::add(a.c0, a.c0), a.c1)};
  }
  static HD __forceinline__ T norm_times(const T &a, int k) { return {lane::norm_times(a.c0, k), lane::norm_times(a.c1, k)}; }
  static HD __forceinline__ fp2 inv(const fp2 &a) { return f2_inv(a); }
  static HD __forceinline__ T b3(const T &a) {
    T k;
#pragma unroll
    for (int j = 0; j < 9; j++) {
      k.c0.l[j] = bn::TWIST_3B29[0][j];
      k.c1.l[j] = bn::TWIST_3B29[1][j];
    }
    return mul(a, k);
  }
};

// ---------------------------------------------------------------- group law
template <class L> struct pt {
  typename L::T X, Y, Z;
};
template <class L> HD __forceinline__ pt<L> identity() { return {L::zero(), L::some(), L::zero()}; }

// the second half of an addition, from t0 = X1 X2, t1 = Y1 Y2, t3 = X1 Y2 + X2 Y1, t4 = Y1 Z2 + Y2 Z1
// (limbs within two units), y = 3b (X1 Z2 + X2 Z1), z = 3b Z1 Z2
template <class L>
HD __forceinline__ pt<L> add_tail(const typename L::T &t0, const typename L::T &t1, const typename L::T &t3, const typename L::T &t4,
                                  const typename L::T &y, const typename L::T &z) {
  using T = typename L::T;
  const T s = L::norm(L::add(t1, z)), d = L::sub(t1, z), t = L::times(t0, 3);
  return {L::mul2(t3, d, L::neg(t4), y), L::mul2(y, t, s, d), L::mul2(s, t4, t, t3)};
}
template <class L> HD __forceinline__ pt<L> add(const pt<L> &p, const pt<L> &q) {
  return add_tail<L>(L::mul(p.X, q.X), L::mul(p.Y, q.Y), L::mul2(p.X, q.Y, p.Y, q.X), L::mul2(p.Y, q.Z, p.Z, q.Y),
                     L::b3(L::mul2(p.X, q.Z, p.Z, q.X)), L::b3(L::mul(p.Z, q.Z)));
}
// p + (x, y, 1)
template <class L> HD __forceinline__ pt<L> madd(const pt<L> &p, const typename L::T &x, const typename L::T &y) {
  return add_tail<L>(L::mul(p.X, x), L::mul(p.Y, y), L::mul2(p.X, y, p.Y, x), L::add(p.Y, L::mul(p.Z, y)),
                     L::b3(L::add(p.X, L::mul(p.Z, x))), L::b3(p.Z));
}
template <class L> HD __forceinline__ pt<L> dbl(const pt<L> &p) {
  using T = typename L::T;
  const T t0 = L::sqr(p.Y), t1 = L::mul(p.Y, p.Z), t2 = L::b3(L::sqr(p.Z)), t3 = L::mul(p.X, p.Y);
  const T n = L::norm(L::sub(t0, L::times(t2, 3))), e = L::norm_times(t0, 8);
  return {L::mul(n, L::times(t3, 2)), L::mul2(e, t2, n, L::add(t0, t2)), L::mul(e, t1)};
}
// the affine point, packed; zeros for the identity
template <class L> HD __forceinline__ aff<typename L::O> to_aff(const pt<L> &p) {
  using O = typename L::O;
  const typename O::T z = L::out(p.Z);
  if (O::is_zero(z)) return aff_inf<O>();
  const typename L::T zi = L::in(L::inv(z));
  return {L::out(L::mul(p.X, zi)), L::out(L::mul(p.Y, zi))};
}
// to Jacobian coordinates, packed: (X Z, Y Z^2, Z)
template <class L> HD __forceinline__ jac<typename L::O> to_jac(const pt<L> &p) {
  const typename L::T yz = L::mul(p.Y, p.Z);
  return {L::out(L::mul(p.X, p.Z)), L::out(L::mul(yz, p.Z)), L::out(p.Z)};
}

// ---------------------------------------------------------------- scalar multiplication
// k P on G1 with the split k = k_0 + k_1 lam (glv.hpp): the table of d_0 B_0 + d_1 B_1, d_j < 4, two
// doublings and at most one addition per two bits.  The table's 15 points are in the caller's
// memory: T.put(e, point), T.get<G1>(e), 0 < e < 16.
template <class Tab> HD __forceinline__ pt<G1> mul_lane(const g1_aff &P, const glv::Dec &d, const Tab &T) {
  if (aff_is_inf(P) || d.nbits == 0) return identity<G1>();
  const fl x = in_small(P.x), y = in_small(P.y), x1 = mul(x, in(fe_const(bn::GLV_BETA))), one = small_one();
  const fl y0 = d.neg & 1 ? neg(y) : y, y1 = d.neg & 2 ? neg(y) : y;
#pragma unroll 1
  for (int s = 1; s <= 4; s *= 4) {  // the multiples of B_0, of B_1
    const fl &bx = s == 1 ? x : x1, &by = s == 1 ? y0 : y1;
    pt<G1> t = {bx, by, one};
    T.put(s, t);
#pragma unroll 1
    for (int m = 2; m <= 3; m++) {
      t = madd<G1>(t, bx, by);
      T.put(m * s, t);
    }
  }
#pragma unroll 1
  for (int e = 5; e < 16; e++)
    if (e & 3) T.put(e, add<G1>(T.template get<G1>(e & 12), T.template get<G1>(e & 3)));
  const int n = (int)(d.nbits + 1) / 2;
  pt<G1> acc = T.template get<G1>((int)glv::digit2(d, (uint32_t)(n - 1)));
#pragma unroll 1
  for (int w = n - 2; w >= 0; w--) {
#pragma unroll 1
    for (int i = 0; i < 2; i++) acc = dbl<G1>(acc);
    const uint32_t dg = glv::digit2(d, (uint32_t)w);
    if (dg) acc = add<G1>(acc, T.template get<G1>((int)dg));
  }
  return acc;
}

}  // namespace lane
