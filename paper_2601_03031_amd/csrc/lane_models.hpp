// What the host's checks run the one-lane formulas (lane_group.hpp, lane_pair.hpp) on in place of fl:
//   Both<S>  the elements of both lanes of a pair;
//   Bnd      bounds of an element: |limbs| within u 2^28, |value| within v p.  Every operation records how
//            near its columns come to 2^63, its 32-bit limbs to 2^31 and the arguments of `reduce` to 2^9 p, and
//            a data-dependent choice takes the larger of its sides.
#pragma once
#include <cmath>
#include "lane29.hpp"

namespace lane {

// ---------------------------------------------------------------- bounds
struct Bnd {
  double u, v;
};
namespace bounds {
struct Worst {
  double column, limb, reduced, packed;  // fractions of what is allowed; of p for a value packed (below 2)
};
inline Worst worst;
inline void see(double &w, double x) { w = std::fmax(w, x); }
static constexpr double TOP = 3171406.0;       // floor(p / 2^232)
static constexpr double SHRINK = 1.0 / 169.2;  // p / 2^261, rounded up
static constexpr double EPS = 1.0 / (1 << 24);
// the top limb: of the value, less what the lower limbs take from it
inline double top(const Bnd &a) { return (a.v * (TOP + 1) + a.u + 1) / (1 << 28); }
inline double unit(const Bnd &a) { return std::fmax(a.u, top(a)); }
inline Bnd limbs(const Bnd &a) {
  see(worst.limb, unit(a) / 8);
  return a;
}
inline Bnd product(double columns, double value) {
  // and the reduction's 9 products of a centred quotient limb with a limb of p, a carry, a half
  see(worst.column, (9 * columns + 18 + EPS) / 128);
  return limbs({1, 0.5 + EPS + value * SHRINK});
}
}  // namespace bounds

inline Bnd join(const Bnd &a, const Bnd &b) { return {std::fmax(a.u, b.u), std::fmax(a.v, b.v)}; }
inline Bnd add(const Bnd &a, const Bnd &b) { return bounds::limbs({a.u + b.u, a.v + b.v}); }
inline Bnd sub(const Bnd &a, const Bnd &b) { return add(a, b); }
inline Bnd neg(const Bnd &a) { return a; }
inline Bnd neg_if(const Bnd &a, uint32_t) { return a; }
inline Bnd times(const Bnd &a, int k) { return bounds::limbs({std::abs(k) * a.u, std::abs(k) * a.v}); }
inline Bnd norm(const Bnd &a) {
  bounds::see(bounds::worst.limb, (bounds::unit(a) + 1) / 8);
  return {1 + (a.u + 1) * bounds::EPS, a.v};
}
inline Bnd norm_times(const Bnd &a, int k) { return bounds::limbs({1 + (std::abs(k) * a.u + 1) * bounds::EPS, std::abs(k) * a.v}); }
inline Bnd reduce(const Bnd &a, int k, const Bnd &b) {
  const double v = std::abs(k) * a.v + b.v, u = std::abs(k) * a.u + b.u;
  bounds::see(bounds::worst.reduced, v / 512);
  bounds::see(bounds::worst.limb, (b.u + 1) / 8);
  bounds::see(bounds::worst.limb, (std::abs(k) * bounds::top(a) + bounds::top(b)) / 8);
  // the quotient: rounded, in single precision (three roundings), from the top limb, which the lower limbs move by u
  return bounds::limbs({1 + (u + 1024) * bounds::EPS, 0.5 + 512 * 3 * bounds::EPS + (u + 1) / bounds::TOP});
}
inline Bnd mul(const Bnd &a, const Bnd &b) { return bounds::product(bounds::unit(a) * bounds::unit(b), a.v * b.v); }
inline Bnd sqr(const Bnd &a) {
  bounds::see(bounds::worst.limb, 2 * bounds::unit(a) / 8);
  return mul(a, a);
}
template <int N> Bnd sum_of(const Bnd *const *a, const Bnd *const *b) {
  double c = 0, v = 0;
  for (int i = 0; i < N; i++) {
    c += bounds::unit(*a[i]) * bounds::unit(*b[i]);
    v += a[i]->v * b[i]->v;
  }
  return bounds::product(c, v);
}
inline Bnd mul2(const Bnd &a, const Bnd &b, const Bnd &c, const Bnd &d) {
  const Bnd *x[2] = {&a, &c}, *y[2] = {&b, &d};
  return sum_of<2>(x, y);
}
inline Bnd mul4(const Bnd &a, const Bnd &b, const Bnd &c, const Bnd &d, const Bnd &e, const Bnd &f, const Bnd &g, const Bnd &h) {
  const Bnd *x[4] = {&a, &c, &e, &g}, *y[4] = {&b, &d, &f, &h};
  return sum_of<4>(x, y);
}
inline Bnd dot6(const Bnd *const *a, const Bnd *const *b) { return sum_of<6>(a, b); }
// a packed element below p, taken to limbs (`in`, `in_small`) and a value packed (`fl`'s `out`)
inline Bnd packed() { return {2, 32}; }
inline void pack(const Bnd &x) {
  // times 2^256 = 5.3 p, whose one limb is 2^24; to this p is added, and one p taken off
  const Bnd y = mul(x, Bnd{1.0 / 16, 5.3});
  bounds::see(bounds::worst.packed, 1 + y.v);
  bounds::see(bounds::worst.limb, (bounds::unit(y) + 2) / 8);
}

// ---------------------------------------------------------------- both lanes of a pair
struct Lanes {};  // the lanes' bits: 0 and 1
template <class S> struct Both {
  S l[2];
};
template <class S> Both<S> add(const Both<S> &a, const Both<S> &b) { return {{add(a.l[0], b.l[0]), add(a.l[1], b.l[1])}}; }
template <class S> Both<S> sub(const Both<S> &a, const Both<S> &b) { return {{sub(a.l[0], b.l[0]), sub(a.l[1], b.l[1])}}; }
template <class S> Both<S> neg(const Both<S> &a) { return {{neg(a.l[0]), neg(a.l[1])}}; }
template <class S> Both<S> neg_if(const Both<S> &a, uint32_t m) { return {{neg_if(a.l[0], m), neg_if(a.l[1], m)}}; }
template <class S> Both<S> norm(const Both<S> &a) { return {{norm(a.l[0]), norm(a.l[1])}}; }
template <class S> Both<S> times(const Both<S> &a, int k) { return {{times(a.l[0], k), times(a.l[1], k)}}; }
template <class S> Both<S> norm_times(const Both<S> &a, int k) { return {{norm_times(a.l[0], k), norm_times(a.l[1], k)}}; }
template <class S> Both<S> reduce(const Both<S> &a, int k, const Both<S> &b) {
  return {{reduce(a.l[0], k, b.l[0]), reduce(a.l[1], k, b.l[1])}};
}
template <class S> Both<S> mul(const Both<S> &a, const Both<S> &b) { return {{mul(a.l[0], b.l[0]), mul(a.l[1], b.l[1])}}; }
template <class S> Both<S> mul2(const Both<S> &a, const Both<S> &b, const Both<S> &c, const Both<S> &d) {
  return {{mul2(a.l[0], b.l[0], c.l[0], d.l[0]), mul2(a.l[1], b.l[1], c.l[1], d.l[1])}};
}
template <class S>
Both<S> mul4(const Both<S> &a, const Both<S> &b, const Both<S> &c, const Both<S> &d, const Both<S> &e, const Both<S> &f, const Both<S> &g,
             const Both<S> &h) {
  Both<S> o;
  for (int i = 0; i < 2; i++) o.l[i] = mul4(a.l[i], b.l[i], c.l[i], d.l[i], e.l[i], f.l[i], g.l[i], h.l[i]);
  return o;
}
template <class S> Both<S> dot6(const Both<S> *const *a, const Both<S> *const *b) {
  Both<S> o;
  for (int i = 0; i < 2; i++) {
    const S *x[6], *y[6];
    for (int n = 0; n < 6; n++) {
      x[n] = &a[n]->l[i];
      y[n] = &b[n]->l[i];
    }
    o.l[i] = dot6(x, y);
  }
  return o;
}
template <class S> Both<S> join(const Both<S> &a, const Both<S> &b) { return {{join(a.l[0], b.l[0]), join(a.l[1], b.l[1])}}; }
template <class S> Both<S> other(const Both<S> &a) { return {{a.l[1], a.l[0]}}; }
template <class S> Both<S> pick(Lanes, const Both<S> &a, const Both<S> &b) { return {{b.l[0], a.l[1]}}; }

}  // namespace lane

#include "lane_group.hpp"
#include "lane_pair.hpp"

namespace lane {

template <> inline Bnd const29<Bnd>(const int32_t *c) {
  Bnd o = {0, 0};
  double t = 0;  // the value in units of 2^232
  for (int j = 0; j < 9; j++) {
    o.u = std::fmax(o.u, std::fabs((double)c[j]) / (1 << 28));
    t = t / (1 << 29) + c[j];
  }
  o.v = std::fabs(t) / bounds::TOP;
  return o;
}
template <> inline Both<fl> const29<Both<fl>>(const int32_t *c) { return {{const29<fl>(c), const29<fl>(c)}}; }
template <> inline Both<Bnd> const29<Both<Bnd>>(const int32_t *c) { return {{const29<Bnd>(c), const29<Bnd>(c)}}; }
inline fl small_word(const fl *, const uint32_t *w) { return in_small(fe_const(w)); }
inline Bnd small_word(const Bnd *, const uint32_t *) { return mul(packed(), const29<Bnd>(bn::P_ONE29)); }
template <class S> struct Lane<Both<S>> {
  using P = Lanes;
  static P own() { return {}; }
  static Both<S> limbs(P, const int32_t (*c)[9]) { return {{const29<S>(c[0]), const29<S>(c[1])}}; }
  static Both<S> words(P, const uint32_t *w0, const uint32_t *w1) { return {{small_word((S *)nullptr, w0), small_word((S *)nullptr, w1)}}; }
};

// larger of two points' or elements' bounds
template <class V> over2<V> join(const over2<V> &a, const over2<V> &b) { return {join(a.c0, b.c0), join(a.c1, b.c1)}; }
template <class L> pt<L> join(const pt<L> &a, const pt<L> &b) { return {join(a.X, b.X), join(a.Y, b.Y), join(a.Z, b.Z)}; }

// a table that keeps each point, and one that keeps bounds of them all
template <class Point> struct Kept {
  Point *t;
  template <class L> void put(int e, const pt<L> &v) const { t[e] = v; }
  template <class L> pt<L> get(int e) const { return t[e]; }
};
template <class Point> struct Joined {
  Point *t;
  template <class L> void put(int, const pt<L> &v) const { *t = join(*t, v); }
  template <class L> pt<L> get(int) const { return *t; }
};

}  // namespace lane
