// G2 scalar multiplication on the engine: k Q (+ A) with the GLS split k = sum_j k_j lam^j, the
// signed bases B_j = sign(k_j) psi^j(Q), a table of the 15 subset sums, and one doubling plus at
// most one table addition per bit of max |k_j| (65 bits).  The programs work on the curve
// y^2 = x^3 + 4 + 5i, isomorphic to the twist; the accumulator T is in homogeneous coordinates
// (each component the sum of G2_SUM slots) and the formulas are complete: no case is
// exceptional, the identity is (0 : 1 : 0).  The bits' programs run as one list of calls.  The
// control code is shared by the device (DevCtx, all lanes of the workgroup) and the host model
// (HostCtx).
#pragma once
#include "slp.hpp"
#include "gls.hpp"

namespace g2m {
using slp::f29;
static constexpr int NT = 24, NS = 4;  // slots of T, and of a component
static_assert(slp::G2_T_2_1_3 - slp::G2_T_0_0_0 == NT - 1, "T: four slots a component");

// T = the point in the 6 slots at src (homogeneous, on the isomorphic curve)
template <class Ctx> __host__ __device__ inline void load(Ctx &c, int src) {
  for (int i = c.lane(); i < NT; i += c.lanes()) c.S[slp::G2_T_0_0_0 + i] = c.S[i % NS ? slp::G2_CBASE : src + i / NS];
  c.sync();
}

// T = the identity
template <class Ctx> __host__ __device__ inline void load_identity(Ctx &c) {
  for (int i = c.lane(); i < NT; i += c.lanes()) c.S[slp::G2_T_0_0_0 + i] = c.S[slp::G2_CBASE + (i == 2 * NS)];
  c.sync();
}

// Q (affine, on the twist) must be in slots xQ, yQ and the constants (0, then 1, first) loaded.
// Leaves k Q in T.
template <class Ctx> __host__ __device__ inline void mul(Ctx &c, const gls::Dec &dec, bool qinf) {
  f29 *S = c.S;
  if (qinf || dec.nbits == 0) {
    load_identity(c);
    return;
  }
  c.run(slp::PROG_G2_BASES, 0, 0, 0);
  for (int i = c.lane(); i < 8; i += c.lanes()) {
    const int j = i >> 1, y = slp::G2_B0_y_0 + 4 * j + (i & 1);
    if (dec.neg >> j & 1) S[y] = slp::neg29(S[y]);
  }
  c.sync();
  c.run(slp::PROG_G2_TABLE, 0, 0, 0);
  const int n = (int)dec.nbits - 1;  // bits below the top one, a call each
  load(c, slp::G2_TB1_0 + 6 * ((int)gls::digit(dec, (uint32_t)n) - 1));
  for (int e = c.lane(); e < n; e += c.lanes()) {
    const int d = (int)gls::digit(dec, (uint32_t)(n - 1 - e));
    c.cl[e] = d ? slp::call(slp::PROG_G2_DBL_ADD, 0, slp::G2_TB1_0 + 6 * (d - 1)) : slp::call(slp::PROG_G2_DBL);
  }
  c.run_list(0, n);
}

// coordinate component i (0..5) of T
template <class Ctx> __host__ __device__ inline f29 coord(const Ctx &c, int i) {
  const f29 *t = c.S + slp::G2_T_0_0_0 + NS * i;
  return slp::add29(slp::add29(t[0], t[1]), slp::add29(t[2], t[3]));
}

// ---- Jacobian sums (the MSMs' partial sums, on the twist itself): J += A, A the Jacobian point
// at abase (ainf when it is the identity); inf says whether J is the identity, and is updated.
// An addition that meets equal x-coordinates (H = 0) is resolved exactly.
template <class Ctx> __host__ __device__ inline void add_jac(Ctx &c, bool &inf, int abase, bool ainf) {
  if (ainf) return;
  auto copy = [&]() {
    for (int i = c.lane(); i < 6; i += c.lanes()) c.S[slp::G2_J_0 + i] = c.S[abase + i];
    c.sync();
  };
  if (inf) {
    copy();
    inf = false;
    return;
  }
  c.run(slp::PROG_G2_JADD, 0, abase, 0);
  const bool h = slp::zero29(c.S[slp::G2_H_0]) && slp::zero29(c.S[slp::G2_H_1]);
  if (!h) return;
  const bool dbl = slp::zero29(c.S[slp::G2_RR_0]) && slp::zero29(c.S[slp::G2_RR_1]);
  c.sync();
  if (dbl) {
    copy();
    c.run(slp::PROG_G2_JDBL, 0, 0, 0);
  } else {
    inf = true;
  }
}

}  // namespace g2m
