// Group laws and scalar multiplications on one-lane limbs (lane29.hpp), over any element type V that has
// its operations: fl in the kernels; both lanes of a pair, and bounds of limbs and values, in the host's checks.
//
// The group law is the complete one for y^2 = x^3 + b (J. Renes, C. Costello, L. Batina, "Complete
// addition formulas for prime order elliptic curves", 2016): homogeneous coordinates, the identity
// (0 : 1 : 0) and no exceptional case in groups of odd order.
#pragma once
#include "lane29.hpp"
#include "glv.hpp"

namespace lane {

// an element from 9 limbs
template <class V> HD __forceinline__ V const29(const int32_t *c);
template <> HD __forceinline__ fl const29<fl>(const int32_t *c) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = c[j];
  return o;
}
static constexpr int32_t UNIT29[9] = {1};  // an element that is not zero

// ---------------------------------------------------------------- the two coordinate fields
// mul, mul2 (a b + c d), add, sub, neg, norm, times, and b3: 3 b x with limbs of one unit
template <class V> struct G1of {
  using T = V;
  using O = OpsG1;
  static HD __forceinline__ T in(const fe &x) { return lane::in(x); }
  static HD __forceinline__ fe out(const T &x) { return lane::out(x); }
  static HD __forceinline__ T zero() { return T{}; }
  static HD __forceinline__ T some() { return const29<V>(UNIT29); }
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
using G1 = G1of<fl>;
template <class V> struct over2 {
  V c0, c1;
};
template <class V> struct G2of {
  using T = over2<V>;
  using O = OpsG2;
  static HD __forceinline__ T in(const fp2 &x) { return {lane::in(x.c0), lane::in(x.c1)}; }
  static HD __forceinline__ T in_small(const fp2 &x) { return {lane::in_small(x.c0), lane::in_small(x.c1)}; }
  static HD __forceinline__ fp2 out(const T &x) { return {lane::out(x.c0), lane::out(x.c1)}; }
  static HD __forceinline__ T zero() { return T{}; }
  static HD __forceinline__ T some() { return {const29<V>(UNIT29), V{}}; }
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
    return mul(a, T{const29<V>(bn::TWIST_3B29[0]), const29<V>(bn::TWIST_3B29[1])});
  }
};
using G2 = G2of<fl>;

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
// doublings and at most one addition per two bits.  x, y: P (not the identity), x1: beta x, all with limbs of
// one unit; one: 2^261.  The table's 15 points are in the caller's memory: T.put(e, point), T.get<L>(e),
// 0 < e < 16.
template <class V, class Tab>
HD __forceinline__ pt<G1of<V>> mul_table(const V &x, const V &y, const V &x1, const V &one, const glv::Dec &d, const Tab &T) {
  using L = G1of<V>;
  const V y0 = L::neg_if(y, d.neg & 1), y1 = L::neg_if(y, d.neg >> 1 & 1);
#pragma unroll 1
  for (int s = 1; s <= 4; s *= 4) {  // the multiples of B_0, of B_1
    const V &bx = s == 1 ? x : x1, &by = s == 1 ? y0 : y1;
    pt<L> t = {bx, by, one};
    T.put(s, t);
#pragma unroll 1
    for (int m = 2; m <= 3; m++) {
      t = madd<L>(t, bx, by);
      T.put(m * s, t);
    }
  }
#pragma unroll 1
  for (int e = 5; e < 16; e++)
    if (e & 3) T.put(e, add<L>(T.template get<L>(e & 12), T.template get<L>(e & 3)));
  const int n = (int)(d.nbits + 1) / 2;
  pt<L> acc = T.template get<L>((int)glv::digit2(d, (uint32_t)(n - 1)));
#pragma unroll 1
  for (int w = n - 2; w >= 0; w--) {
#pragma unroll 1
    for (int i = 0; i < 2; i++) acc = dbl<L>(acc);
    const uint32_t dg = glv::digit2(d, (uint32_t)w);
    if (dg) acc = add<L>(acc, T.template get<L>((int)dg));
  }
  return acc;
}
template <class Tab> HD __forceinline__ pt<G1> mul_lane(const g1_aff &P, const glv::Dec &d, const Tab &T) {
  if (aff_is_inf(P) || d.nbits == 0) return identity<G1>();
  const fl x = in_small(P.x);
  return mul_table(x, in_small(P.y), mul(x, in(fe_const(bn::GLV_BETA))), small_one(), d, T);
}

}  // namespace lane
