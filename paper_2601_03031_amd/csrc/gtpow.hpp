// Exponentiation in the cyclotomic subgroup of F_p12 (G_T) on the wave-cooperative
// engine, with the 4-dimensional split of the exponent: G_T has order r and the p-power
// Frobenius acts on it as exponentiation by lam = p mod r, so with k = sum_j k_j lam^j
// (mod r), |k_j| < 2^65 (the decomposition used for G2), g^k = prod_j frob^j(g)^{k_j}.
// A negative k_j takes the conjugate (the inverse in the cyclotomic subgroup).  The 15
// products of subsets of the four bases form a table; then one cyclotomic squaring and
// at most one table product per bit of max |k_j|.  Control code shared by the device
// (DevCtx) and the host model (HostCtx).
#pragma once
#include "slp.hpp"
#include "gls.hpp"

namespace gtp {

// buffers of 12 slots at fb + 12 b: 0 the input, 1..15 the table, 16 and 17 the
// accumulator
static constexpr int NBUF = 18;

template <class Ctx> __host__ __device__ inline void copy12(Ctx &c, int dst, int src) {
  for (int i = c.lane(); i < 12; i += c.lanes()) c.S[dst + i] = c.S[src + i];
  c.sync();
}

// g^k for g (cyclotomic) in buffer 0 and k given by its decomposition; returns the buffer
// holding the result, or -1 when k = 0 (the result is 1).  The signed Frobenius images, then
// one list of calls: the 11 table products and a call per bit (a squaring, with a product
// where the digit is not zero), the accumulator alternating between its two buffers.
template <class Ctx> __host__ __device__ inline int pow_cyc(Ctx &c, const gls::Dec &dec, int fb) {
  auto B = [fb](int b) { return (uint16_t)(fb + 12 * b); };
  if (dec.nbits == 0) return -1;
  const int n = (int)dec.nbits - 1;  // bits below the top one
  const int top = (int)gls::digit(dec, (uint32_t)n);
  if (c.lane() == 0) {
    // image j to buffer 2^j; where k_j is negative by way of buffer 16, for the conjugate
    int e = 0;
    for (int j = 0; j < 4; j++) {
      const bool neg = dec.neg >> j & 1;
      const int dst = neg && j ? 16 : 1 << j;
      if (j == 1) c.cl[e++] = slp::call(slp::PROG_F12_FROB1, B(0), B(0), B(dst));
      if (j == 2) c.cl[e++] = slp::call(slp::PROG_F12_FROB2, B(0), B(0), B(dst));
      if (j == 3) c.cl[e++] = slp::call(slp::PROG_F12_FROB3, B(0), B(0), B(dst));
      if (neg) c.cl[e++] = slp::call(slp::PROG_F12_CONJ, B(j ? 16 : 0), B(j ? 16 : 0), B(1 << j));
    }
  }
  if (!(dec.neg & 1)) copy12(c, B(1), B(0));
  c.sync();
  c.run_list(0, 3 + __builtin_popcount(dec.neg & 15u));
  const int HEAD = 11;
  for (int e = c.lane(); e < HEAD + n; e += c.lanes()) {
    if (e < HEAD) {
      int d = e + 3;  // the e-th of 3, 5, 6, 7, 9, .. 15
      d += d >= 4;
      d += d >= 8;
      const int lo = d & -d;
      c.cl[e] = slp::call(slp::PROG_F12_MUL, B(d - lo), B(lo), B(d));
    } else {
      const int i = e - HEAD, d = (int)gls::digit(dec, (uint32_t)(n - 1 - i));
      const int src = i == 0 ? top : 17 - (i & 1), dst = 16 + (i & 1);
      c.cl[e] = d ? slp::call(slp::PROG_F12_CSQR_MUL, B(src), B(d), B(dst)) : slp::call(slp::PROG_F12_CSQR, B(src), B(src), B(dst));
    }
  }
  c.run_list(0, HEAD + n);
  return n == 0 ? top : 17 - (n & 1);
}

}  // namespace gtp
