// G1 scalar multiplication on the engine: k P (+ A) with the GLV split k = k_0 + k_1 lam
// (glv.hpp), the signed bases B0 = sign(k_0) P and B1 = sign(k_1) phi(P), phi(x, y) = (beta x, y),
// the 15-entry table of d0 B0 + d1 B1 (0 <= d0, d1 < 4) and one program of two doublings plus an
// addition per 2-bit window (two doublings alone for a zero window).  The accumulator T is in
// homogeneous coordinates (each the sum of G1_SUM slots) and the formulas are complete: no case
// is exceptional, the identity is (0 : 1 : 0).  The windows' programs run as one list of calls.
// The control code is shared by the device (DevCtx) and the host model (HostCtx).
#pragma once
#include "slp.hpp"
#include "glv.hpp"

namespace g1m {
using slp::f29;
static constexpr int NT = 6;  // slots of T
static_assert(slp::G1_T_2_1 - slp::G1_T_0_0 == NT - 1, "T: two slots a coordinate");

// T = the point in the 3 slots at src (homogeneous)
template <class Ctx> __host__ __device__ inline void load(Ctx &c, int src) {
  for (int i = c.lane(); i < NT; i += c.lanes()) c.S[slp::G1_T_0_0 + i] = c.S[i & 1 ? slp::G1_CBASE : src + (i >> 1)];
  c.sync();
}

// T = the identity
template <class Ctx> __host__ __device__ inline void load_identity(Ctx &c) {
  for (int i = c.lane(); i < NT; i += c.lanes()) c.S[slp::G1_T_0_0 + i] = c.S[slp::G1_CBASE + (i == 2)];
  c.sync();
}

// P (affine) must be in slots xP, yP and the constants (0, then 1, first) loaded.  Leaves k P in
// T.
template <class Ctx> __host__ __device__ inline void mul(Ctx &c, const glv::Dec &dec, bool pinf) {
  f29 *S = c.S;
  if (pinf || dec.nbits == 0) {
    load_identity(c);
    return;
  }
  c.run(slp::PROG_G1_PHI, 0, 0, 0);
  if (c.lane() == 0) {
    f29 y = S[slp::G1_yP];
    S[slp::G1_B1_y] = (dec.neg & 2) ? slp::neg29(y) : y;
    S[slp::G1_yP] = (dec.neg & 1) ? slp::neg29(y) : y;
  }
  c.sync();
  c.run(slp::PROG_G1_TABLE, 0, 0, 0);
  const int W = (int)(dec.nbits + 1) / 2 - 1;  // windows below the top one, a call each
  load(c, slp::G1_TB1_0 + 3 * ((int)glv::digit2(dec, (uint32_t)W) - 1));
  for (int e = c.lane(); e < W; e += c.lanes()) {
    const int d = (int)glv::digit2(dec, (uint32_t)(W - 1 - e));
    c.cl[e] = d ? slp::call(slp::PROG_G1_DBL2_ADD, 0, slp::G1_TB1_0 + 3 * (d - 1)) : slp::call(slp::PROG_G1_DBL2);
  }
  c.run_list(0, W);
}

// T += A for an affine A: its coordinates go to xP, yP (whose values are spent)
template <class Ctx> __host__ __device__ inline void add_affine(Ctx &c, const f29 &x, const f29 &y) {
  if (c.lane() == 0) {
    c.S[slp::G1_xP] = x;
    c.S[slp::G1_yP] = y;
  }
  c.run(slp::PROG_G1_MADD, 0, 0, 0);
}

// coordinate i (0..2) of T
template <class Ctx> __host__ __device__ inline f29 coord(const Ctx &c, int i) {
  return slp::add29(c.S[slp::G1_T_0_0 + 2 * i], c.S[slp::G1_T_0_0 + 2 * i + 1]);
}

}  // namespace g1m
