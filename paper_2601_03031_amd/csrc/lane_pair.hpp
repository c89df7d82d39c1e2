// G2 and pairings on two lanes (lane29.hpp's limbs), lane p of them with component p of every element of
// F_p2 (p = 0, 1): the state of a pairing, 24 elements of F_p, then fits the registers of its lanes, and a
// product in F_p2 is one sum of two products in each.  Sums of products over F_p2 have one reduction, so
// that F_p6 products and the product by a line are taken by their definition (a third of the reductions that
// the forms with fewer products need, and no sums before or after).
//
// V is what a lane holds: fl in the kernels, where p is the lane's own bit; both lanes' elements in the host's
// checks.  other(a): the other lane's; pick(p, a, b): a in lane 1, b in lane 0.
#pragma once
#include "lane_group.hpp"
#include "gls.hpp"

namespace lane {

// P: the type of p, own(): this lane's; limbs, words: the component of a constant (words: a packed one)
template <class V> struct Lane;
#ifdef __HIPCC__
template <> struct Lane<fl> {
  using P = bool;
  static __device__ __forceinline__ P own() { return threadIdx.x & 1; }
  static __device__ __forceinline__ fl limbs(P p, const int32_t (*c)[9]) {
    fl o;
#pragma unroll
    for (int j = 0; j < 9; j++) o.l[j] = c[p][j];
    return o;
  }
  static __device__ __forceinline__ fl words(P p, const uint32_t *w0, const uint32_t *w1) { return in_small(fe_const(p ? w1 : w0)); }
};
__device__ __forceinline__ fl other(const fl &a) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = __builtin_amdgcn_mov_dpp(a.l[j], 0xB1, 0xF, 0xF, true);
  return o;
}
__device__ __forceinline__ fl pick(bool p, const fl &a, const fl &b) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = p ? a.l[j] : b.l[j];
  return o;
}
#define PAIR __device__
#else
#define PAIR
#endif

// a second factor b as both lanes use it: a b = own(a) x + other(a) y, with (x, y) = (b_0, -b_1) in lane
// 0 and (b_0, b_1) in lane 1
template <class V> struct fac {
  V x, y;
};
template <class V, class P> PAIR __forceinline__ fac<V> factor(P p, const V &b) {
  const V o = other(b);
  return {pick(p, o, b), pick(p, b, neg(o))};
}
// sums of one, two and three products a b, the other lane's a given
template <class V> PAIR __forceinline__ V prod(const V &a, const V &ao, const fac<V> &b) { return mul2(a, b.x, ao, b.y); }
template <class V> PAIR __forceinline__ V prod2(const V &a, const V &ao, const fac<V> &b, const V &c, const V &co, const fac<V> &d) {
  return mul4(a, b.x, ao, b.y, c, d.x, co, d.y);
}
template <class V> PAIR __forceinline__ V prod3(const V &a, const V &ao, const fac<V> &b, const V &c, const V &co, const fac<V> &d, const V &e,
                                    const V &eo, const fac<V> &f) {
  const V *x[6] = {&a, &ao, &c, &co, &e, &eo}, *y[6] = {&b.x, &b.y, &d.x, &d.y, &f.x, &f.y};
  return dot6(x, y);
}
template <class V, class P> PAIR __forceinline__ V mul2_(P p, const V &a, const V &b) { return prod(a, other(a), factor(p, b)); }
// a^2: (a_0 + a_1)(a_0 - a_1) in lane 0, 2 a_1 a_0 in lane 1
template <class V, class P> PAIR __forceinline__ V sqr2_(P p, const V &a) {
  const V o = other(a);
  return mul(add(a, pick(p, a, o)), pick(p, o, sub(a, o)));
}
// k a + b, a - b and (9 + i) a, reduced: limbs of one unit, within 0.51 p
template <class V> PAIR __forceinline__ V red(const V &a, int k, const V &b) { return reduce(a, k, b); }
template <class V> PAIR __forceinline__ V red_sub(const V &a, const V &b) { return reduce(b, -1, a); }
template <class V, class P> PAIR __forceinline__ V xi(P p, const V &a) {
  const V o = other(a);
  return red(a, 9, pick(p, o, neg(o)));
}

template <class V> struct six {
  V c[3];  // over 1, v, v^2
};
// a b in F_p6 (limbs of one unit)
template <class V, class P> PAIR __forceinline__ six<V> mul6(P p, const six<V> &a, const six<V> &b) {
  const V o0 = other(a.c[0]), o1 = other(a.c[1]), o2 = other(a.c[2]);
  const fac<V> b0 = factor(p, b.c[0]), b1 = factor(p, b.c[1]), b2 = factor(p, b.c[2]);
  const fac<V> x1 = factor(p, xi(p, b.c[1])), x2 = factor(p, xi(p, b.c[2]));
  return {{prod3(a.c[0], o0, b0, a.c[1], o1, x2, a.c[2], o2, x1), prod3(a.c[0], o0, b1, a.c[1], o1, b0, a.c[2], o2, x2),
           prod3(a.c[0], o0, b2, a.c[1], o1, b1, a.c[2], o2, b0)}};
}
template <class V> struct twelve {
  six<V> a, b;  // a + b w, w^2 = v
};
// f^2 = (a + b)(a + v b) - t - v t + 2 t w, t = a b
template <class V, class P> PAIR __forceinline__ void sqr12(P p, twelve<V> &f) {
  six<V> x = f.a, y = f.b, t = {}, r = {};
#pragma unroll 1
  for (int k = 0; k < 2; k++) {  // (one copy of the product's code for both)
    r = mul6(p, x, y);
    if (k == 0) {
      t = r;
      const V v0 = xi(p, f.b.c[2]);
#pragma unroll
      for (int i = 0; i < 3; i++) {
        x.c[i] = red(f.a.c[i], 1, f.b.c[i]);
        y.c[i] = red(f.a.c[i], 1, i ? f.b.c[i - 1] : v0);
      }
    }
  }
  const V t0 = xi(p, t.c[2]);
#pragma unroll
  for (int i = 0; i < 3; i++) {
    f.a.c[i] = red_sub(sub(r.c[i], t.c[i]), i ? t.c[i - 1] : t0);
    f.b.c[i] = red(t.c[i], 2, V{});
  }
}
// f g = t0 + v t1 + (t2 - t0 - t1) w, t0 = a a', t1 = b b', t2 = (a + b)(a' + b')
template <class V, class P> PAIR __forceinline__ twelve<V> mul12(P p, const twelve<V> &f, const twelve<V> &g) {
  six<V> x = f.a, y = g.a, t[3] = {};
#pragma unroll 1
  for (int k = 0; k < 3; k++) {
    const six<V> r = mul6(p, x, y);
    if (k == 0) {
      t[0] = r;
      x = f.b;
      y = g.b;
    } else if (k == 1) {
      t[1] = r;
#pragma unroll
      for (int i = 0; i < 3; i++) {
        x.c[i] = red(f.a.c[i], 1, f.b.c[i]);
        y.c[i] = red(g.a.c[i], 1, g.b.c[i]);
      }
    } else {
      t[2] = r;
    }
  }
  const V v0 = xi(p, t[1].c[2]);
  twelve<V> o;
#pragma unroll
  for (int i = 0; i < 3; i++) {
    o.a.c[i] = red(t[0].c[i], 1, i ? t[1].c[i - 1] : v0);
    o.b.c[i] = red_sub(sub(t[2].c[i], t[0].c[i]), t[1].c[i]);
  }
  return o;
}
// f (l0 + l1 w + l3 w^3)
template <class V, class P> PAIR __forceinline__ void mul_line(P p, twelve<V> &f, const V &l0, const V &l1, const V &l3) {
  const fac<V> c0 = factor(p, l0), c1 = factor(p, l1), c3 = factor(p, l3), x1 = factor(p, xi(p, l1)), x3 = factor(p, xi(p, l3));
  const V *a = f.a.c, *b = f.b.c;
  const V ao[3] = {other(a[0]), other(a[1]), other(a[2])}, bo[3] = {other(b[0]), other(b[1]), other(b[2])};
  twelve<V> r;
  r.a.c[0] = prod3(a[0], ao[0], c0, b[1], bo[1], x3, b[2], bo[2], x1);
  r.a.c[1] = prod3(a[1], ao[1], c0, b[0], bo[0], c1, b[2], bo[2], x3);
  r.a.c[2] = prod3(a[2], ao[2], c0, b[0], bo[0], c3, b[1], bo[1], c1);
  r.b.c[0] = prod3(b[0], bo[0], c0, a[0], ao[0], c1, a[2], ao[2], x3);
  r.b.c[1] = prod3(b[1], bo[1], c0, a[0], ao[0], c3, a[1], ao[1], c1);
  r.b.c[2] = prod3(b[2], bo[2], c0, a[1], ao[1], c3, a[2], ao[2], c1);
  f = r;
}

// G2 with a lane for each component of its coordinates (lane_group.hpp's laws on the lane's own)
template <class V> struct G2pairOf {
  using T = V;
  static PAIR __forceinline__ typename Lane<V>::P p() { return Lane<V>::own(); }
  static PAIR __forceinline__ T zero() { return T{}; }
  static PAIR __forceinline__ T some() { return pick(p(), T{}, const29<V>(UNIT29)); }
  static PAIR __forceinline__ T one() { return pick(p(), T{}, const29<V>(bn::P_ONE29)); }
  static PAIR __forceinline__ T add(const T &a, const T &b) { return lane::add(a, b); }
  static PAIR __forceinline__ T sub(const T &a, const T &b) { return lane::sub(a, b); }
  static PAIR __forceinline__ T neg(const T &a) { return lane::neg(a); }
  static PAIR __forceinline__ T norm(const T &a) { return lane::norm(a); }
  static PAIR __forceinline__ T times(const T &a, int k) { return lane::times(a, k); }
  static PAIR __forceinline__ T norm_times(const T &a, int k) { return lane::norm_times(a, k); }
  static PAIR __forceinline__ T mul(const T &a, const T &b) { return mul2_(p(), a, b); }
  static PAIR __forceinline__ T mul2(const T &a, const T &b, const T &c, const T &d) {
    return prod2(a, other(a), factor(p(), b), c, other(c), factor(p(), d));
  }
  static PAIR __forceinline__ T sqr(const T &a) { return sqr2_(p(), a); }
  static PAIR __forceinline__ T b3(const T &a) { return mul(a, Lane<V>::limbs(p(), bn::TWIST_3B29)); }
};

// psi(x, y): the conjugates times constants
template <class V, class P> PAIR __forceinline__ void frobenius(P p, V &x, V &y) {
  x = mul2_(p, pick(p, neg(x), x), Lane<V>::words(p, bn::FROB1_2_0, bn::FROB1_2_1));
  y = mul2_(p, pick(p, neg(y), y), Lane<V>::words(p, bn::FROB1_3_0, bn::FROB1_3_1));
}

// k Q on G2 with the split k = sum_j k_j lam^j (gls.hpp): the table of the 15 subset sums of
// sign(k_j) psi^j(Q), a doubling and at most one addition per bit.  x, y: this lane's components of Q, with
// limbs of one unit; inf and d are the same in both lanes.  The table as for mul_table
template <class V, class Tab> PAIR __forceinline__ pt<G2pairOf<V>> mul_pair(V x, V y, bool inf, const gls::Dec &d, const Tab &T) {
  using L = G2pairOf<V>;
  if (inf || d.nbits == 0) return identity<L>();
  const auto p = L::p();
#pragma unroll 1
  for (int j = 0; j < 4; j++) {
    if (j) frobenius(p, x, y);
    const V s = neg_if(y, d.neg >> j & 1);
    T.put(1 << j, pt<L>{x, s, L::one()});
#pragma unroll 1
    for (int e = 1; e < 1 << j; e++) T.put(e + (1 << j), madd<L>(T.template get<L>(e), x, s));
  }
  const int n = (int)d.nbits;
  pt<L> acc = T.template get<L>((int)gls::digit(d, (uint32_t)(n - 1)));
#pragma unroll 1
  for (int t = n - 2; t >= 0; t--) {
    acc = dbl<L>(acc);
    const uint32_t dg = gls::digit(d, (uint32_t)t);
    if (dg) acc = add<L>(acc, T.template get<L>((int)dg));
  }
  return acc;
}

template <class V> struct point {
  V X, Y, Z;  // homogeneous
};
// T = 2 T and the tangent at T at P: l0 = 2YZ yP, l1 = -3X^2 xP, l3 = Y^2 - 3b'Z^2, all up to a factor in
// F_p2, which the final exponentiation removes
template <class V, class P> PAIR __forceinline__ void tangent(P p, point<V> &T, const V &xP, const V &yP, const V &b3, V &l0, V &l1, V &l3) {
  const V XX = sqr2_(p, T.X), YY = sqr2_(p, T.Y), E = mul2_(p, sqr2_(p, T.Z), b3);
  const V XY = mul2_(p, T.X, T.Y), YZ = mul2_(p, T.Y, T.Z);
  const fac<V> fY = factor(p, YY);
  l0 = mul(times(YZ, 2), yP);
  l1 = mul(times(XX, -3), xP);
  l3 = red_sub(YY, E);
  T.X = mul2_(p, times(XY, 2), red(E, -3, YY));
  T.Y = red_sub(sqr2_(p, red(E, 3, YY)), mul2_(p, red(E, 12, V{}), E));
  const V z = red(YZ, 8, V{});
  T.Z = prod(z, other(z), fY);
}
// T = T + (x, y) and the line through both at P
template <class V, class P> PAIR __forceinline__ void chord(P p, point<V> &T, const V &x, const V &y, const V &xP, const V &yP, V &l0, V &l1, V &l3) {
  const V Zo = other(T.Z);
  const fac<V> fx = factor(p, x), fy = factor(p, y);
  const V th = red_sub(T.Y, prod(T.Z, Zo, fy)), la = red_sub(T.X, prod(T.Z, Zo, fx));
  const V tho = other(th), lao = other(la);
  l0 = mul(la, yP);
  l1 = mul(neg(th), xP);
  l3 = prod2(th, tho, fx, neg(la), neg(lao), fy);
  const fac<V> D = factor(p, sqr2_(p, la));
  const V E = prod(la, lao, D), F = prod(T.Z, Zo, factor(p, sqr2_(p, th))), G = prod(T.X, other(T.X), D);
  const V H = red(G, -2, add(E, F));
  const fac<V> fE = factor(p, neg(E));
  T.X = prod(la, lao, factor(p, H));
  T.Y = prod2(th, tho, factor(p, red_sub(G, H)), T.Y, other(T.Y), fE);
  T.Z = prod(neg(T.Z), neg(Zo), fE);
}

// The Miller value of (P, Q) up to factors that the final exponentiation removes: over the non-adjacent
// form of 6u + 2 (d_65 = 1 starts T = Q; d_64 = 0), a doubling in each step, then with a digit an addition; the
// last two steps add pi(Q) and -pi^2(Q).  Neither point is the identity
template <class V, class P> PAIR __forceinline__ twelve<V> miller_pair(P p, const V &xP, const V &yP, const V &x, const V &y) {
  const V one = G2pairOf<V>::one(), zero = V{}, b3 = Lane<V>::limbs(p, bn::TWIST_3B29);
  point<V> T = {x, y, one};
  twelve<V> f = {{{one, zero, zero}}, {{zero, zero, zero}}};
  V sx = x, sy = y;
#pragma unroll 1
  for (int s = 64, add = 0; s >= -2;) {
    V l0, l1, l3;
    if (!add && s >= 0) {
      if (s != 64) sqr12(p, f);
      tangent(p, T, xP, yP, b3, l0, l1, l3);
    } else {
      V cx = sx, cy = sy;
      if (s < 0) {
        // the next Frobenius image, and its negative the second time
        frobenius(p, sx, sy);
        cx = sx;
        cy = s == -2 ? neg(sy) : sy;
      } else if (bn::ATE_NAF_NEG >> s & 1) {
        cy = neg(cy);
      }
      chord(p, T, cx, cy, xP, yP, l0, l1, l3);
    }
    mul_line(p, f, l0, l1, l3);
    add = !add && s >= 0 && s < 64 && ((bn::ATE_NAF_POS | bn::ATE_NAF_NEG) >> s & 1);
    if (!add) s--;
  }
  return f;
}

}  // namespace lane
