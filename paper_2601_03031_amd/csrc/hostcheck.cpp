// Host build of the device arithmetic headers (field, tower, curve, pairing, hash),
// exported with canonical big-endian byte encodings so CPU tests can compare the
// GPU path's arithmetic with the oracle before any kernel runs.  This is a test
// harness for the HIP code path; the library itself never runs it.
#include <cstring>
#include "field.hpp"
#include "tower.hpp"
#include "curve.hpp"
#include "pairing.hpp"
#include "hash.hpp"
#include "slp.hpp"
#include "lane_models.hpp"
#include "gls.hpp"
#include "g2mul.hpp"
#include "gtpow.hpp"
#include "g1mul.hpp"
#include "oa_terms.hpp"
#include "proof_grid.hpp"

#define API extern "C" __attribute__((visibility("default")))

template <class F> static fe rd(const uint8_t *b) {
  fe a;
  for (int i = 0; i < 8; i++)
    a.l[7 - i] = ((uint32_t)b[4 * i] << 24) | ((uint32_t)b[4 * i + 1] << 16) | ((uint32_t)b[4 * i + 2] << 8) | b[4 * i + 3];
  return f_to_mont<F>(a);
}
template <class F> static void wr(uint8_t *b, const fe &m) {
  fe a = f_from_mont<F>(m);
  for (int i = 0; i < 8; i++) {
    uint32_t w = a.l[7 - i];
    b[4 * i] = w >> 24; b[4 * i + 1] = w >> 16; b[4 * i + 2] = w >> 8; b[4 * i + 3] = w;
  }
}
static fp2 rd2(const uint8_t *b) { return {rd<FpP>(b), rd<FpP>(b + 32)}; }
static void wr2(uint8_t *b, const fp2 &a) { wr<FpP>(b, a.c0); wr<FpP>(b + 32, a.c1); }
static fp12 rd12(const uint8_t *b) {
  fp12 f;
  fp6 *h[2] = {&f.c0, &f.c1};
  for (int a = 0; a < 2; a++) {
    fp2 *q[3] = {&h[a]->c0, &h[a]->c1, &h[a]->c2};
    for (int c = 0; c < 3; c++) *q[c] = rd2(b + 384 / 2 * a + 64 * c);
  }
  return f;
}
static void wr12(uint8_t *b, const fp12 &f) {
  const fp6 *h[2] = {&f.c0, &f.c1};
  for (int a = 0; a < 2; a++) {
    const fp2 *q[3] = {&h[a]->c0, &h[a]->c1, &h[a]->c2};
    for (int c = 0; c < 3; c++) wr2(b + 192 * a + 64 * c, *q[c]);
  }
}
static g1_aff rdg1(const uint8_t *b) { return {rd<FpP>(b), rd<FpP>(b + 32)}; }
static void wrg1(uint8_t *b, const g1_aff &p) { wr<FpP>(b, p.x); wr<FpP>(b + 32, p.y); }
static g2_aff rdg2(const uint8_t *b) { return {rd2(b), rd2(b + 64)}; }
static void wrg2(uint8_t *b, const g2_aff &p) { wr2(b, p.x); wr2(b + 64, p.y); }
static void canon_scalar(uint32_t k[8], const uint8_t *b) {
  for (int i = 0; i < 8; i++)
    k[7 - i] = ((uint32_t)b[4 * i] << 24) | ((uint32_t)b[4 * i + 1] << 16) | ((uint32_t)b[4 * i + 2] << 8) | b[4 * i + 3];
}

// Modular inverse by the binary extended GCD with batched steps (after T. Pornin,
// "Optimized Binary GCD for Modular Inversion", 2020).  Invariants: x u = a and x v = b
// (mod m), starting from a = x, b = m, u = 1, v = 0.  Each outer round takes 30 binary-GCD
// steps (if a is odd: order a >= b by a swap, a -= b; then a /= 2) on 64-bit
// approximations of a and b (their low 30 bits, exact, and the top 34 bits of the longer
// one), recording the steps as a 2 x 2 integer matrix, and then applies the matrix to the
// full a, b (an exact division by 2^30) and to u, v (a Montgomery division by 2^30 mod m).
// It ends when a = 0, so b = gcd = 1 and v = x^{-1}.  All values depend only on the input,
// so a wave-uniform input keeps the whole computation on the scalar unit.
namespace bingcd {

DEV int bitlen(const fe &a) {
  for (int i = 7; i >= 0; i--)
    if (a.l[i]) return 32 * i + 32 - __builtin_clz(a.l[i]);
  return 0;
}

// 64-bit approximation: low 30 bits of a, then the 34 bits of a below bit n
DEV uint64_t approx(const fe &a, int n) {
  uint64_t lo = a.l[0] & 0x3fffffffu;
  if (n <= 64) return (uint64_t)a.l[0] | ((uint64_t)a.l[1] << 32);
  int s = n - 34, w = s >> 5, sh = s & 31;
  // words w, w + 1, w + 2 (zero past the top) picked by selects: an index into the limbs
  // would put the element in scratch memory
  uint32_t a0 = 0, a1 = 0, a2 = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    a0 = i == w ? a.l[i] : a0;
    a1 = i == w + 1 ? a.l[i] : a1;
    a2 = i == w + 2 ? a.l[i] : a2;
  }
  uint64_t v = (uint64_t)a0 >> sh;
  v |= (uint64_t)a1 << (32 - sh);
  if (sh > 30) v |= (uint64_t)a2 << (64 - sh);
  return lo | ((v & 0x3ffffffffull) << 30);
}

// (f a + g b) / 2^30 (exact) as a signed value: magnitude in r, returns true if negative
DEV bool lin_shift(const fe &a, const fe &b, int32_t f, int32_t g, fe &r) {
  uint32_t t[9];
  int64_t acc = 0;
  for (int i = 0; i < 8; i++) {
    acc += (int64_t)a.l[i] * f;
    t[i] = (uint32_t)acc;
    acc >>= 32;
  }
  t[8] = (uint32_t)acc;
  int64_t top = acc;
  acc = 0;
  for (int i = 0; i < 8; i++) {
    acc += (int64_t)t[i] + (int64_t)b.l[i] * g;
    t[i] = (uint32_t)acc;
    acc >>= 32;
  }
  top += acc;
  // top: the signed value of bits 256.. ; shift the 9-limb value right by 30
  uint32_t w8 = (uint32_t)top;
  for (int i = 0; i < 8; i++) r.l[i] = (t[i] >> 30) | ((i < 7 ? t[i + 1] : w8) << 2);
  bool neg = top < 0;
  if (neg) {
    uint64_t c = 1;
    for (int i = 0; i < 8; i++) {
      c += (uint32_t)~r.l[i];
      r.l[i] = (uint32_t)c;
      c >>= 32;
    }
  }
  return neg;
}

// (f u + g v) / 2^30 mod m for u, v in [0, m), |f|, |g| <= 2^30; result in [0, m)
template <class F> DEV fe mont_shift(const fe &u, const fe &v, int32_t f, int32_t g) {
  uint32_t t[8];
  int64_t acc = 0;
  uint32_t w[8];
  for (int i = 0; i < 8; i++) {
    acc += (int64_t)u.l[i] * f;
    w[i] = (uint32_t)acc;
    acc >>= 32;
  }
  int64_t top = acc;
  acc = 0;
  for (int i = 0; i < 8; i++) {
    acc += (int64_t)w[i] + (int64_t)v.l[i] * g;
    w[i] = (uint32_t)acc;
    acc >>= 32;
  }
  top += acc;
  // add q m with q = -t m^{-1} mod 2^30, making the low 30 bits zero
  uint32_t q = (w[0] * F::INV) & 0x3fffffffu;
  acc = 0;
  for (int i = 0; i < 8; i++) {
    acc += (int64_t)w[i] + (int64_t)q * F::M[i];
    t[i] = (uint32_t)acc;
    acc >>= 32;
  }
  top += acc;
  fe r;
  uint32_t w8 = (uint32_t)top;
  for (int i = 0; i < 8; i++) r.l[i] = (t[i] >> 30) | ((i < 7 ? t[i + 1] : w8) << 2);
  int64_t hi = top >> 30;   // the shifted value is r + hi 2^256, in (-2m, 3m)
  // normalise into [0, m): add m while negative, subtract m while >= m
  for (int k = 0; k < 2; k++) {
    if (hi < 0) {
      uint64_t c = 0;
      for (int i = 0; i < 8; i++) {
        c += (uint64_t)r.l[i] + F::M[i];
        r.l[i] = (uint32_t)c;
        c >>= 32;
      }
      hi += (int64_t)c;
    }
  }
  for (int k = 0; k < 2; k++) {
    uint32_t d[8];
    int64_t bw = 0;
    for (int i = 0; i < 8; i++) {
      int64_t x = (int64_t)r.l[i] - F::M[i] + bw;
      d[i] = (uint32_t)x;
      bw = x >> 32;
    }
    if (hi + bw >= 0) {
      for (int i = 0; i < 8; i++) r.l[i] = d[i];
      hi += bw;
    }
  }
  return r;
}

// x^{-1} mod m for 0 < x < m (x canonical, not in Montgomery form); false if the step
// budget ran out (never expected: 2 len(m) - 1 steps suffice for the exact algorithm)
template <class F> DEV bool inverse(const fe &x, fe &out, int *rounds = nullptr) {
  fe a = x, b = fe_const(F::M), u = fe_zero(), v = fe_zero();
  u.l[0] = 1;
  int it = 0;
  for (; it < 40; it++) {
    if (fe_is_zero(a)) break;
    int na = bitlen(a), nb = bitlen(b);
    int n = na > nb ? na : nb;
    uint64_t xa = approx(a, n), xb = approx(b, n);
    // |f|, |g| <= 2^j after j steps; the step is written without branches on 32-bit
    // halves so that a uniform input stays on the scalar unit
    uint32_t alo = (uint32_t)xa, ahi = (uint32_t)(xa >> 32);
    uint32_t blo = (uint32_t)xb, bhi = (uint32_t)(xb >> 32);
    int32_t f0 = 1, g0 = 0, f1 = 0, g1 = 1;
    for (int j = 0; j < 30; j++) {
      uint32_t odd = alo & 1u;
      uint32_t lt = (uint32_t)(ahi < bhi) | ((uint32_t)(ahi == bhi) & (uint32_t)(alo < blo));
      uint32_t sw = 0u - (odd & lt), od = 0u - odd;
      uint32_t t;
      t = (alo ^ blo) & sw; alo ^= t; blo ^= t;
      t = (ahi ^ bhi) & sw; ahi ^= t; bhi ^= t;
      int32_t ts;
      ts = (f0 ^ f1) & (int32_t)sw; f0 ^= ts; f1 ^= ts;
      ts = (g0 ^ g1) & (int32_t)sw; g0 ^= ts; g1 ^= ts;
      uint32_t sl = blo & od, sh = bhi & od;
      uint32_t nlo = alo - sl;
      ahi = ahi - sh - (uint32_t)(alo < sl);
      alo = nlo;
      f0 -= f1 & (int32_t)od;
      g0 -= g1 & (int32_t)od;
      alo = (alo >> 1) | (ahi << 31);
      ahi >>= 1;
      f1 *= 2;
      g1 *= 2;
    }
    fe a2, b2;
    if (lin_shift(a, b, f0, g0, a2)) { f0 = -f0; g0 = -g0; }
    if (lin_shift(a, b, f1, g1, b2)) { f1 = -f1; g1 = -g1; }
    fe u2 = mont_shift<F>(u, v, f0, g0), v2 = mont_shift<F>(u, v, f1, g1);
    a = a2; b = b2; u = u2; v = v2;
  }
  fe one = fe_zero();
  one.l[0] = 1;
  out = v;
  if (rounds) *rounds = it;
  return fe_is_zero(a) && fe_eq(b, one);
}

}  // namespace bingcd

// x^e (canonical, big-endian) by the windowed power on loose limbs
API int hc_pow_fixed(int which, const uint8_t *x, const uint8_t *e, uint8_t *out) {
  uint32_t w[8];
  canon_scalar(w, e);
  if (which == 0) wr<FpP>(out, f_pow_fixed<FpP>(rd<FpP>(x), w));
  else wr<FpR>(out, f_pow_fixed<FpR>(rd<FpR>(x), w));
  return 0;
}

// batched binary GCD on a canonical integer 0 < x < m (which 0: p, 1: r): x^{-1} mod m
// (big-endian 32 bytes) and the number of outer rounds; returns 1 if it converged
API int hc_bingcd(int which, const uint8_t *x, uint8_t *out, int *rounds) {
  fe a, r;
  for (int i = 0; i < 8; i++) {
    const uint8_t *q = x + 28 - 4 * i;
    a.l[i] = (uint32_t)q[0] << 24 | (uint32_t)q[1] << 16 | (uint32_t)q[2] << 8 | q[3];
  }
  bool ok = which == 0 ? bingcd::inverse<FpP>(a, r, rounds) : bingcd::inverse<FpR>(a, r, rounds);
  for (int i = 0; i < 8; i++) {
    uint8_t *q = out + 28 - 4 * i;
    q[0] = (uint8_t)(r.l[i] >> 24); q[1] = (uint8_t)(r.l[i] >> 16); q[2] = (uint8_t)(r.l[i] >> 8); q[3] = (uint8_t)r.l[i];
  }
  return ok ? 1 : 0;
}

// op: 0 add 1 sub 2 mul 3 inv(Fermat) 4 inv(binary) 5 half
API int hc_field(int which, int op, const uint8_t *a, const uint8_t *b, uint8_t *out) {
  if (which == 0) {
    fe x = rd<FpP>(a), y = rd<FpP>(b), z;
    switch (op) {
      case 0: z = fp_add(x, y); break;
      case 1: z = fp_sub(x, y); break;
      case 2: z = fp_mul(x, y); break;
      case 3: z = fp_inv(x); break;
      case 4: z = fp_inv_fast(x); break;
      case 5: z = fp_half(x); break;
      default: return -1;
    }
    wr<FpP>(out, z);
  } else {
    fe x = rd<FpR>(a), y = rd<FpR>(b), z;
    switch (op) {
      case 0: z = fr_add(x, y); break;
      case 1: z = fr_sub(x, y); break;
      case 2: z = fr_mul(x, y); break;
      case 3: z = fr_inv(x); break;
      case 4: z = fr_inv_fast(x); break;
      case 5: z = f_half<FpR>(x); break;
      default: return -1;
    }
    wr<FpR>(out, z);
  }
  return 0;
}

// op: 0 mul 1 sqr 2 inv 3 final_exp 4 frob1 5 frob2 6 frob3 7 cyclo_sqr 8 cyclo_pow_u
API int hc_fp12(int op, const uint8_t *a, const uint8_t *b, uint8_t *out) {
  fp12 x = rd12(a), y = rd12(b), z;
  switch (op) {
    case 0: z = f12_mul(x, y); break;
    case 1: z = f12_sqr(x); break;
    case 2: z = f12_inv(x); break;
    case 3: z = f12_final_exp(x); break;
    case 4: z = f12_frob1(x); break;
    case 5: z = f12_frob2(x); break;
    case 6: z = f12_frob3(x); break;
    case 7: z = f12_cyclo_sqr(x); break;
    case 8: z = f12_cyclo_pow_u(x); break;
    default: return -1;
  }
  wr12(out, z);
  return 0;
}

API int hc_fp2(int op, const uint8_t *a, const uint8_t *b, uint8_t *out) {
  fp2 x = rd2(a), y = rd2(b), z;
  switch (op) {
    case 0: z = f2_mul(x, y); break;
    case 1: z = f2_sqr(x); break;
    case 2: z = f2_inv(x); break;
    case 3: z = f2_mul_xi(x); break;
    default: return -1;
  }
  wr2(out, z);
  return 0;
}

// op: 0 add 1 dbl 2 scalar mul (k canonical BE in b) 3 madd
API int hc_g1(int op, const uint8_t *a, const uint8_t *b, uint8_t *out) {
  g1_aff P = rdg1(a);
  if (op == 2) {
    uint32_t k[8];
    canon_scalar(k, b);
    wrg1(out, jac_to_aff(scalar_mul(P, k)));
    return 0;
  }
  g1_aff Q = rdg1(b);
  if (op == 0) wrg1(out, jac_to_aff(jac_add(jac_from_aff(P), jac_from_aff(Q))));
  else if (op == 1) wrg1(out, jac_to_aff(jac_dbl(jac_from_aff(P))));
  else if (op == 3) wrg1(out, jac_to_aff(jac_madd(jac_from_aff(P), Q)));
  else return -1;
  return 0;
}

API int hc_g2(int op, const uint8_t *a, const uint8_t *b, uint8_t *out) {
  g2_aff P = rdg2(a);
  if (op == 2) {
    uint32_t k[8];
    canon_scalar(k, b);
    wrg2(out, jac_to_aff(scalar_mul(P, k)));
    return 0;
  }
  if (op == 4) { wrg2(out, g2_frobenius(P)); return 0; }
  g2_aff Q = rdg2(b);
  if (op == 0) wrg2(out, jac_to_aff(jac_add(jac_from_aff(P), jac_from_aff(Q))));
  else if (op == 1) wrg2(out, jac_to_aff(jac_dbl(jac_from_aff(P))));
  else if (op == 3) wrg2(out, jac_to_aff(jac_madd(jac_from_aff(P), Q)));
  else return -1;
  return 0;
}

API int hc_pairing(const uint8_t *P, const uint8_t *Q, uint8_t *out) {
  wr12(out, f12_final_exp(miller_loop(rdg1(P), rdg2(Q))));
  return 0;
}

API void hc_h2f(const char *dst, const uint8_t *msg, uint64_t len, uint8_t *out) {
  sha::Hasher h;
  sha::xmd_begin(h);
  h.bytes(msg, (int)len);
  wr<FpR>(out, sha::xmd_finish_fr(h, dst));
}

// the cooperative form used by the challenge kernels (one lane here): msg (len bytes, at
// most 1024) after Z_pad
API void hc_h2f_coop(const char *dst, const uint8_t *msg, uint64_t len, uint8_t *out) {
  static uint32_t w[16 + 256 + 32], t2[16], sched[sha::SCHED_WORDS];
  for (uint64_t i = 0; i < len; i++) sha::put_byte(w, 64 + (uint32_t)i, msg[i]);
  wr<FpR>(out, sha::xmd_fr_coop(sha::Coop{0, 1, sched}, w, (uint32_t)len, dst, t2));
}

// SHA-256 through the cooperative form (len at most 1024)
API void hc_sha256_coop(const uint8_t *msg, uint64_t len, uint8_t *out) {
  static uint32_t w[256 + 32], sched[sha::SCHED_WORDS];
  for (uint64_t i = 0; i < len; i++) sha::put_byte(w, (uint32_t)i, msg[i]);
  uint32_t o[8];
  sha::sha_coop(sha::Coop{0, 1, sched}, w, (uint32_t)len, o);
  for (int i = 0; i < 8; i++) {
    out[4 * i] = o[i] >> 24; out[4 * i + 1] = o[i] >> 16; out[4 * i + 2] = o[i] >> 8; out[4 * i + 3] = o[i];
  }
}

API void hc_sha256(const uint8_t *msg, uint64_t len, uint8_t *out) {
  sha::Hasher h;
  h.init();
  h.bytes(msg, (int)len);
  uint32_t o[8];
  h.final(o);
  for (int i = 0; i < 8; i++) { out[4 * i] = o[i] >> 24; out[4 * i + 1] = o[i] >> 16; out[4 * i + 2] = o[i] >> 8; out[4 * i + 3] = o[i]; }
}

API void hc_merkle_leaf(const uint8_t m[32], const uint8_t c[64], uint8_t out[32]) {
  uint32_t mw[8], cw[16], o[8];
  for (int i = 0; i < 8; i++) mw[i] = ((uint32_t)m[4 * i] << 24) | ((uint32_t)m[4 * i + 1] << 16) | ((uint32_t)m[4 * i + 2] << 8) | m[4 * i + 3];
  for (int i = 0; i < 16; i++) cw[i] = ((uint32_t)c[4 * i] << 24) | ((uint32_t)c[4 * i + 1] << 16) | ((uint32_t)c[4 * i + 2] << 8) | c[4 * i + 3];
  sha::merkle_leaf(o, mw, cw);
  for (int i = 0; i < 8; i++) { out[4 * i] = o[i] >> 24; out[4 * i + 1] = o[i] >> 16; out[4 * i + 2] = o[i] >> 8; out[4 * i + 3] = o[i]; }
}

API void hc_merkle_node(const uint8_t l[32], const uint8_t r[32], uint8_t out[32]) {
  uint32_t lw[8], rw[8], o[8];
  for (int i = 0; i < 8; i++) {
    lw[i] = ((uint32_t)l[4 * i] << 24) | ((uint32_t)l[4 * i + 1] << 16) | ((uint32_t)l[4 * i + 2] << 8) | l[4 * i + 3];
    rw[i] = ((uint32_t)r[4 * i] << 24) | ((uint32_t)r[4 * i + 1] << 16) | ((uint32_t)r[4 * i + 2] << 8) | r[4 * i + 3];
  }
  sha::merkle_node(o, lw, rw);
  for (int i = 0; i < 8; i++) { out[4 * i] = o[i] >> 24; out[4 * i + 1] = o[i] >> 16; out[4 * i + 2] = o[i] >> 8; out[4 * i + 3] = o[i]; }
}


// ---- the wave-cooperative engine's programs through the host model of the interpreter
static void ld_consts(slp::f29 *S, int base, const uint32_t (*C)[9], int n) {
  for (int c = 0; c < n; c++) {
    for (int j = 0; j < 9; j++) S[base + c].l[j] = C[c][j];
    S[base + c].l[9] = S[base + c].l[10] = S[base + c].l[11] = 0;
  }
}

// Miller loop of the engine (before the final exponentiation)
API int hc_slp_miller(const uint8_t *P, const uint8_t *Q, uint8_t *out) {
  static slp::f29 S[slp::ML_NSLOT];
  g1_aff p = rdg1(P);
  g2_aff q = rdg2(Q);
  const fe in[6] = {p.x, p.y, q.x.c0, q.x.c1, q.y.c0, q.y.c1};
  for (int k = 0; k < 6; k++) S[slp::ML_xP + k] = slp::to29(in[k]);
  ld_consts(S, slp::ML_CBASE, slp::ML_CONSTS, slp::ML_NCONST);
  slp::run_host(S, slp::PROG_ML, 0, 0, 0);
  fp12 f;
  fe *fw = reinterpret_cast<fe *>(&f);
  for (int k = 0; k < 12; k++) fw[k] = slp::from29(slp::canon29(S[slp::ML_f_0 + k]));
  wr12(out, f);
  return 0;
}

// final exponentiation (op 0) or F_p12 product of a and b (op 1) on the engine
API int hc_slp_f12(int op, const uint8_t *a, const uint8_t *b, uint8_t *out) {
  fp12 x = rd12(a), y = rd12(b), f;
  const fe *xw = reinterpret_cast<const fe *>(&x), *yw = reinterpret_cast<const fe *>(&y);
  fe *fw = reinterpret_cast<fe *>(&f);
  if (op == 1) {
    static slp::f29 S[slp::F12_NSLOT + 36];
    auto buf = [](int k) { return slp::F12_NSLOT + 12 * k; };
    for (int k = 0; k < 12; k++) { S[buf(0) + k] = slp::to29(xw[k]); S[buf(1) + k] = slp::to29(yw[k]); }
    ld_consts(S, slp::F12_CBASE, slp::F12_CONSTS, slp::F12_NCONST);
    slp::run_host(S, slp::PROG_F12_MUL, buf(0), buf(1), buf(2));
    for (int k = 0; k < 12; k++) fw[k] = slp::from29(slp::canon29(S[buf(2) + k]));
  } else {
    static slp::f29 S[slp::FE_NSLOT];
    for (int k = 0; k < 12; k++) S[slp::FE_X_0 + k] = slp::to29(xw[k]);
    ld_consts(S, slp::FE_CBASE, slp::FE_CONSTS, slp::FE_NCONST);
    slp::run_host(S, slp::PROG_FE_NORM, 0, 0, 0);
    S[slp::FE_tinv] = slp::to29(fp_inv_fast(slp::from29(slp::canon29(S[slp::FE_t]))));
    slp::run_host(S, slp::PROG_FE_REST, 0, 0, 0);
    for (int k = 0; k < 12; k++) fw[k] = slp::from29(slp::canon29(S[slp::FE_D_0 + k]));
  }
  wr12(out, f);
  return 0;
}


// radix-2^29 lane arithmetic on raw integers (big-endian 32 bytes, below 2p):
// ops 0 and 3: sum_i k_i x_i mod p (almost reduced, then canonical); op 1: Montgomery
// product a b 2^{-261} (canonical); ops 2 and 4: the almost-reduced linear combination itself
// plus p (it is signed, within p of zero)
static fe rd_raw(const uint8_t *b) {
  fe a;
  for (int i = 0; i < 8; i++)
    a.l[7 - i] = ((uint32_t)b[4 * i] << 24) | ((uint32_t)b[4 * i + 1] << 16) | ((uint32_t)b[4 * i + 2] << 8) | b[4 * i + 3];
  return a;
}
static void wr_raw(uint8_t *b, const fe &a) {
  for (int i = 0; i < 8; i++) {
    uint32_t w = a.l[7 - i];
    b[4 * i] = w >> 24; b[4 * i + 1] = w >> 16; b[4 * i + 2] = w >> 8; b[4 * i + 3] = w;
  }
}
API int hc_slp_lane(int op, int n, const int *k, const uint8_t *xs, uint8_t *out) {
  if (op == 1) {
    slp::f29 r = slp::canon29(slp::mont29(slp::to29(rd_raw(xs)), slp::to29(rd_raw(xs + 32))));
    wr_raw(out, slp::from29(r));
    return 0;
  }
  int64_t acc[9] = {};
  for (int i = 0; i < n; i++) {
    slp::f29 x = slp::to29(rd_raw(xs + 32 * i));
    for (int j = 0; j < 9; j++) acc[j] += (int64_t)k[i] * (int32_t)x.l[j];
  }
  slp::f29 r = slp::red29(acc);
  if (op == 2 || op == 4)
    for (int j = 0; j < 9; j++) r.l[j] += slp::P29[j];
  wr_raw(out, slp::from29(op == 2 || op == 4 ? slp::norm29(r) : slp::canon29(r)));
  return 0;
}


// ---- host model of the 8-lane field layout (field_wide.hpp), lane for lane: element limbs
// g = 0..7 as an array, the cross-lane steps written out (ds_swizzle broadcasts of limb k,
// DPP shifts by one limb, the ballot carry-lookahead).  Raw Montgomery limbs in and out, no
// conversions, so that the range of every output can be checked at the inputs' extremes and
// compared bit for bit with the device (vc_diag_field's raw modes).
namespace w8 {
struct V { uint32_t v[8]; };
static void shdn(const uint32_t *x, uint32_t *o) { for (int g = 0; g < 8; g++) o[g] = g < 7 ? x[g + 1] : 0u; }
static void shup(const uint32_t *x, uint32_t *o) { for (int g = 0; g < 8; g++) o[g] = g ? x[g - 1] : 0u; }
// carry into each lane from per-lane generate/propagate flags, and the carry out of lane 7,
// exactly as wchain(): C = ((g|p) + g) ^ (g|p) ^ g over the lanes 0..6, lane 7's own flags
// decide the carry out
static uint32_t g_active = 0xFF;  // lanes taking part in the ballots (all 8 in the library)
static void chain(const bool *gen, const bool *prop, uint32_t *cin, bool &out) {
  uint32_t G = 0, P = 0;
  for (int g = 0; g < 8; g++) { G |= (uint32_t)gen[g] << g; P |= (uint32_t)prop[g] << g; }
  G &= g_active;  // a ballot sees only active lanes
  P &= g_active;
  uint32_t gg = G & 0x7f, pp = P & 0x7f, a = gg | pp;
  uint32_t C = (a + gg) ^ a ^ gg;
  for (int g = 0; g < 8; g++) cin[g] = (C >> g) & 1u;
  out = (((G >> 7) & 1u) | (((P >> 7) & 1u) & ((C >> 7) & 1u))) != 0;
}
static void reduce(const uint32_t *M, const uint32_t *s, uint32_t *o) {  // s - m if s >= m
  bool gen[8], prop[8], bout;
  uint32_t bin[8];
  for (int g = 0; g < 8; g++) { gen[g] = s[g] < M[g]; prop[g] = s[g] == M[g]; }
  chain(gen, prop, bin, bout);
  for (int g = 0; g < 8; g++) o[g] = bout ? s[g] : s[g] - M[g] - bin[g];
}
static void add(const uint32_t *M, const uint32_t *a, const uint32_t *b, uint32_t *o) {
  uint32_t lo[8], cin[8], t[8];
  bool gen[8], prop[8], out;
  for (int g = 0; g < 8; g++) {
    uint64_t s = (uint64_t)a[g] + b[g];
    lo[g] = (uint32_t)s;
    gen[g] = (s >> 32) != 0;
    prop[g] = lo[g] == 0xFFFFFFFFu;
  }
  chain(gen, prop, cin, out);
  for (int g = 0; g < 8; g++) t[g] = lo[g] + cin[g];
  reduce(M, t, o);
}
static void sub(const uint32_t *M, const uint32_t *a, const uint32_t *b, uint32_t *o) {
  bool gen[8], prop[8], bout, out;
  uint32_t bin[8], d[8], lo[8], cin[8];
  for (int g = 0; g < 8; g++) { gen[g] = a[g] < b[g]; prop[g] = a[g] == b[g]; }
  chain(gen, prop, bin, bout);
  for (int g = 0; g < 8; g++) {
    d[g] = a[g] - b[g] - bin[g];
    uint64_t s = (uint64_t)d[g] + (bout ? M[g] : 0u);
    lo[g] = (uint32_t)s;
    gen[g] = (s >> 32) != 0;
    prop[g] = lo[g] == 0xFFFFFFFFu;
  }
  chain(gen, prop, cin, out);
  for (int g = 0; g < 8; g++) o[g] = lo[g] + cin[g];
}
static void mul(const uint32_t *M, uint32_t INV, const uint32_t *a, const uint32_t *b, uint32_t *o) {
  uint32_t t[8] = {0}, c[8] = {0};
  for (int j = 0; j < 8; j++) {
    uint64_t X[8], Y[8];
    uint32_t ylo[8], yd[8];
    for (int g = 0; g < 8; g++) X[g] = (uint64_t)a[g] * b[j] + t[g];
    uint32_t m = (uint32_t)X[0] * INV;
    for (int g = 0; g < 8; g++) { Y[g] = (uint64_t)m * M[g] + (uint32_t)X[g]; ylo[g] = (uint32_t)Y[g]; }
    shdn(ylo, yd);
    for (int g = 0; g < 8; g++) {
      uint64_t s = (uint64_t)yd[g] + (X[g] >> 32) + (Y[g] >> 32) + c[g];
      t[g] = (uint32_t)s;
      c[g] = (uint32_t)(s >> 32);
    }
  }
  uint32_t cu[8], lo[8], cin[8], r[8];
  bool gen[8], prop[8], out;
  shup(c, cu);
  for (int g = 0; g < 8; g++) {
    uint64_t f = (uint64_t)t[g] + cu[g];
    lo[g] = (uint32_t)f;
    gen[g] = (f >> 32) != 0;
    prop[g] = lo[g] == 0xFFFFFFFFu;
  }
  chain(gen, prop, cin, out);
  for (int g = 0; g < 8; g++) r[g] = lo[g] + cin[g];
  reduce(M, r, o);
}
}  // namespace w8

// the lanes of a group that take part in the ballots (0xFF: all; the library's kernels keep
// every group whole)
API void hc_wide_active(uint32_t mask) { w8::g_active = mask & 0xFF; }

// op 0 mul, 1 add, 2 sub on raw little-endian limbs (32 bytes each); which 0: p, 1: r
API int hc_wide_raw(int which, int op, const uint8_t *a, const uint8_t *b, uint8_t *out) {
  const uint32_t *M = which ? bn::R_MOD : bn::P_MOD;
  const uint32_t INV = which ? bn::R_INV : bn::P_INV;
  uint32_t x[8], y[8], z[8];
  memcpy(x, a, 32);
  memcpy(y, b, 32);
  switch (op) {
    case 0: w8::mul(M, INV, x, y, z); break;
    case 1: w8::add(M, x, y, z); break;
    case 2: w8::sub(M, x, y, z); break;
    default: return -1;
  }
  memcpy(out, z, 32);
  return 0;
}

// GLS decomposition of a canonical scalar (big-endian 32 bytes): out = 4 signed 128-bit
// two's-complement values (little-endian 16 bytes each) and the bit length
API int hc_gls(const uint8_t *kb, uint8_t *out, uint32_t *nbits) {
  fe k = rd_raw(kb);
  gls::Dec d = gls::decompose(k.l);
  for (int j = 0; j < 4; j++) {
    uint32_t m[4] = {d.mag[j][0], d.mag[j][1], d.mag[j][2], 0};
    if (d.neg >> j & 1) {
      uint64_t cy = 1;
      for (int w = 0; w < 4; w++) { uint64_t t = (uint64_t)(uint32_t)~m[w] + cy; m[w] = (uint32_t)t; cy = t >> 32; }
    }
    for (int w = 0; w < 4; w++)
      for (int b = 0; b < 4; b++) out[16 * j + 4 * w + b] = (uint8_t)(m[w] >> (8 * b));
  }
  *nbits = d.nbits;
  return 0;
}


// ---- scalar multiplications on the engine's host model, results affine (zeros = identity)
static fe out29(const slp::f29 &x) { return slp::from29(slp::canon29(x)); }

struct HostG2 {
  slp::f29 S[slp::G2_NSLOT];
  slp::HostCtx c{S};
  void begin(const g2_aff &Q) {
    ld_consts(S, slp::G2_CBASE, slp::G2_CONSTS, slp::G2_NCONST);
    const fe *q = reinterpret_cast<const fe *>(&Q);
    for (int i = 0; i < 4; i++) S[slp::G2_xQ_0 + i] = slp::to29(q[i]);
  }
  void mul(const g2_aff &Q, const gls::Dec &dec) {
    begin(Q);
    g2m::mul(c, dec, aff_is_inf(Q));
  }
  // 2^{16 m} Q in T
  void dbl_mult(const g2_aff &Q, int m) {
    begin(Q);
    if (aff_is_inf(Q)) g2m::load_identity(c);
    else c.run(slp::PROG_G2_LOAD, 0, 0, 0);
    for (int i = 0; i < 16 * m; i++) c.run(slp::PROG_G2_DBL, 0, 0, 0);
  }
  void add_affine(const g2_aff &A) {
    if (aff_is_inf(A)) return;
    const fe *a = reinterpret_cast<const fe *>(&A);
    for (int i = 0; i < 4; i++) S[slp::G2_xQ_0 + i] = slp::to29(a[i]);
    c.run(slp::PROG_G2_MADD, 0, 0, 0);
  }
  // T += the homogeneous point p
  void add_hom(const fe *p) {
    for (int i = 0; i < 6; i++) S[slp::G2_TB1_0 + i] = slp::to29(p[i]);
    c.run(slp::PROG_G2_ADD, 0, slp::G2_TB1_0, 0);
  }
  void hom(fe *p) {
    for (int i = 0; i < 6; i++) p[i] = out29(g2m::coord(c, i));
  }
  g2_aff aff() {
    c.run(slp::PROG_G2_NORM, 0, 0, 0);
    const fe t = out29(S[slp::G2_t]);
    g2_aff r = {};
    if (fe_is_zero(t)) return r;
    S[slp::G2_tinv] = slp::to29(fp_inv_fast(t));
    c.run(slp::PROG_G2_AFF, 0, 0, 0);
    for (int i = 0; i < 4; i++) reinterpret_cast<fe *>(&r)[i] = out29(S[slp::G2_ax_0 + i]);
    return r;
  }
};

struct HostG1 {
  slp::f29 S[slp::G1_NSLOT];
  slp::HostCtx c{S};
  void begin(const g1_aff &P) {
    ld_consts(S, slp::G1_CBASE, slp::G1_CONSTS, slp::G1_NCONST);
    S[slp::G1_xP] = slp::to29(P.x);
    S[slp::G1_yP] = slp::to29(P.y);
  }
  void mul(const g1_aff &P, const glv::Dec &dec) {
    begin(P);
    g1m::mul(c, dec, aff_is_inf(P));
  }
  // 2^{32 m} P in T
  void dbl_mult(const g1_aff &P, int m) {
    begin(P);
    S[slp::G1_TB1_0] = slp::to29(P.x);
    S[slp::G1_TB1_0 + 1] = slp::to29(P.y);
    S[slp::G1_TB1_0 + 2] = slp::to29(f_one<FpP>());
    if (aff_is_inf(P)) g1m::load_identity(c);
    else g1m::load(c, slp::G1_TB1_0);
    for (int i = 0; i < 16 * m; i++) c.run(slp::PROG_G1_DBL2, 0, 0, 0);
  }
  void add_affine(const g1_aff &A) {
    if (!aff_is_inf(A)) g1m::add_affine(c, slp::to29(A.x), slp::to29(A.y));
  }
  void add_hom(const fe *p) {
    for (int i = 0; i < 3; i++) S[slp::G1_TB1_0 + i] = slp::to29(p[i]);
    c.run(slp::PROG_G1_ADD, 0, slp::G1_TB1_0, 0);
  }
  void hom(fe *p) {
    for (int i = 0; i < 3; i++) p[i] = out29(g1m::coord(c, i));
  }
  g1_aff aff() {
    const fe z = out29(g1m::coord(c, 2));
    g1_aff r = {};
    if (fe_is_zero(z)) return r;
    S[slp::G1_tinv] = slp::to29(fp_inv_fast(z));
    c.run(slp::PROG_G1_AFF, 0, 0, 0);
    r.x = out29(S[slp::G1_ax]);
    r.y = out29(S[slp::G1_ay]);
    return r;
  }
};

// k Q + A (A may be null); k canonical 32 bytes big-endian
API int hc_g2_mul(const uint8_t *Qb, const uint8_t *kb, const uint8_t *Ab, uint8_t *out) {
  static HostG2 h;
  fe k = rd_raw(kb);
  h.mul(rdg2(Qb), gls::decompose(k.l));
  if (Ab) h.add_affine(rdg2(Ab));
  wrg2(out, h.aff());
  return 0;
}

// k P + A (A may be null)
API int hc_g1_mul_engine(const uint8_t *Pb, const uint8_t *kb, const uint8_t *Ab, uint8_t *out) {
  static HostG1 h;
  fe k = rd_raw(kb);
  h.mul(rdg1(Pb), glv::decompose(k.l));
  if (Ab) h.add_affine(rdg1(Ab));
  wrg1(out, h.aff());
  return 0;
}

// k P as the sum over t < 4 of chunk_t(k) (2^{32 t} P): the split used to run the four parts in
// parallel
API int hc_g1_mul_split(const uint8_t *Pb, const uint8_t *kb, uint8_t *out) {
  static HostG1 h;
  g1_aff P = rdg1(Pb);
  fe k = rd_raw(kb);
  glv::Dec dec = glv::decompose(k.l);
  g1_jac acc = jac_inf<OpsG1>(), Pt = jac_from_aff(P);
  for (int t = 0; t < 4; t++) {
    if (t)
      for (int i = 0; i < 32; i++) Pt = jac_dbl(Pt);
    h.mul(jac_to_aff(Pt), glv::chunk(dec, t));
    acc = jac_madd(acc, h.aff());
  }
  wrg1(out, jac_to_aff(acc));
  return 0;
}

// The split fold, as the GPU runs it: multiples 2^{32 t} P by repeated double doublings, the four
// chunked multiplications into homogeneous partials, then their sum plus A (affine; may be null
// or the identity).
API int hc_fold_split_g1(const uint8_t *Pb, const uint8_t *kb, const uint8_t *Ab, uint8_t *out) {
  static HostG1 h;
  g1_aff P = rdg1(Pb);
  fe k = rd_raw(kb);
  glv::Dec dec = glv::decompose(k.l);
  fe part[4][3];
  for (int t = 0; t < 4; t++) {
    h.dbl_mult(P, t);
    const g1_aff base = h.aff();
    h.mul(base, glv::chunk(dec, t));
    h.hom(part[t]);
  }
  g1m::load_identity(h.c);
  for (int t = 0; t < 4; t++) h.add_hom(part[t]);
  if (Ab) h.add_affine(rdg1(Ab));
  wrg1(out, h.aff());
  return 0;
}

// the same for G2: multiples 2^{16 t} Q, bits [16 t, 16 t + w_t) of the GLS split
API int hc_fold_split_g2(const uint8_t *Qb, const uint8_t *kb, const uint8_t *Ab, uint8_t *out) {
  static HostG2 h;
  g2_aff Q = rdg2(Qb);
  fe k = rd_raw(kb);
  gls::Dec dec = gls::decompose(k.l);
  fe part[4][6];
  for (int t = 0; t < 4; t++) {
    h.dbl_mult(Q, t);
    const g2_aff base = h.aff();
    h.mul(base, gls::chunk(dec, 16 * t, t < 3 ? 16 : 17));
    h.hom(part[t]);
  }
  g2m::load_identity(h.c);
  for (int t = 0; t < 4; t++) h.add_hom(part[t]);
  if (Ab) h.add_affine(rdg2(Ab));
  wrg2(out, h.aff());
  return 0;
}

// g^k as the product over t < 4 of pow(g^{2^{16 t}}, chunk of bits [16 t, 16 t + w_t)) with
// w_t = 16 (t < 3) or 17, on the engine (host model)
API int hc_gt_pow_split(const uint8_t *gb, const uint8_t *kb, uint8_t *out) {
  static slp::f29 S[slp::F12_NSLOT + 12 * gtp::NBUF];
  fp12 g = rd12(gb), acc = f12_one();
  fe k = rd_raw(kb);
  gls::Dec dec = gls::decompose(k.l);
  const fe *gw = reinterpret_cast<const fe *>(&g);
  ld_consts(S, slp::F12_CBASE, slp::F12_CONSTS, slp::F12_NCONST);
  for (int i = 0; i < 12; i++) S[slp::F12_NSLOT + i] = slp::to29(gw[i]);
  slp::HostCtx c{S};
  const int b0 = slp::F12_NSLOT, b17 = slp::F12_NSLOT + 12 * 17;
  for (int t = 0; t < 4; t++) {
    if (t) {
      for (int i = 0; i < 16; i++) {
        slp::run_host(S, slp::PROG_F12_CSQR, b0, b0, b17);
        for (int q = 0; q < 12; q++) S[b0 + q] = S[b17 + q];
      }
    }
    slp::f29 base[12];
    for (int q = 0; q < 12; q++) base[q] = S[b0 + q];
    int r = gtp::pow_cyc(c, gls::chunk(dec, 16 * t, t < 3 ? 16 : 17), slp::F12_NSLOT);
    if (r >= 0) {
      fp12 part;
      fe *pw = reinterpret_cast<fe *>(&part);
      for (int q = 0; q < 12; q++) pw[q] = slp::from29(slp::canon29(S[slp::F12_NSLOT + 12 * r + q]));
      acc = f12_mul(acc, part);
    }
    for (int q = 0; q < 12; q++) S[b0 + q] = base[q];
  }
  wr12(out, acc);
  return 0;
}

// g^k on the engine (host model) for g in the cyclotomic subgroup, k canonical (32 bytes
// big-endian) through the 4-dimensional Frobenius split
API int hc_gt_pow_cyc(const uint8_t *gb, const uint8_t *kb, uint8_t *out) {
  static slp::f29 S[slp::F12_NSLOT + 12 * gtp::NBUF];
  fp12 g = rd12(gb);
  const fe *gw = reinterpret_cast<const fe *>(&g);
  for (int i = 0; i < 12; i++) S[slp::F12_NSLOT + i] = slp::to29(gw[i]);
  ld_consts(S, slp::F12_CBASE, slp::F12_CONSTS, slp::F12_NCONST);
  fe k = rd_raw(kb);
  gls::Dec dec = gls::decompose(k.l);
  slp::HostCtx c{S};
  int r = gtp::pow_cyc(c, dec, slp::F12_NSLOT);
  fp12 f;
  fe *fw = reinterpret_cast<fe *>(&f);
  for (int i = 0; i < 12; i++)
    fw[i] = r < 0 ? (i == 0 ? f_one<FpP>() : fe_zero()) : slp::from29(slp::canon29(S[slp::F12_NSLOT + 12 * r + i]));
  wr12(out, f);
  return 0;
}

// Montgomery products (MUL operations) in the engine's programs, for the work model
// (9.. : G1 phi + table, two doublings + addition, two doublings, mixed addition, to affine;
// cyclotomic squaring; the three Frobenius maps):
// 0 Miller loop (whole sequence), 1 final exponentiation (whole sequence, without the
// one-lane inversion), 2 G2 signed bases (to the isomorphic curve), 3 G2 table, 4 G2 doubling, 5 G2 addition,
// 6 G2 mixed addition, 7 G2 to affine (norm + affine), 8 F_p12 product
static uint64_t prog_muls(int prog) {
  uint64_t n = 0;
  for (int v = 0; v < 4; v++)
    for (uint32_t d = slp::PROGS[prog].d[v]; d; d = slp::blk_word(slp::OPS, d, 0, 1))
      for (int i = 0; i < slp::blk_ops(d); i++) n += slp::term_coef(slp::blk_word(slp::OPS, d, 2 * i, 0)) == 1;
  return n;
}
API uint64_t hc_engine_muls(int which) {
  switch (which) {
    case 0: return prog_muls(slp::PROG_ML);
    case 1: return prog_muls(slp::PROG_FE_NORM) + prog_muls(slp::PROG_FE_REST);
    case 2: return prog_muls(slp::PROG_G2_BASES);
    case 3: return prog_muls(slp::PROG_G2_TABLE);
    case 4: return prog_muls(slp::PROG_G2_DBL);
    case 5: return prog_muls(slp::PROG_G2_DBL_ADD) - prog_muls(slp::PROG_G2_DBL);
    case 6: return prog_muls(slp::PROG_G2_MADD);
    case 7: return prog_muls(slp::PROG_G2_NORM) + prog_muls(slp::PROG_G2_AFF);
    case 8: return prog_muls(slp::PROG_F12_MUL);
    case 9: return prog_muls(slp::PROG_G1_PHI) + prog_muls(slp::PROG_G1_TABLE);
    case 10: return prog_muls(slp::PROG_G1_DBL2_ADD);
    case 11: return prog_muls(slp::PROG_G1_DBL2);
    case 12: return prog_muls(slp::PROG_G1_MADD);
    case 13: return prog_muls(slp::PROG_G1_AFF);
    case 14: return prog_muls(slp::PROG_F12_CSQR);
    case 15: return prog_muls(slp::PROG_F12_FROB1) + prog_muls(slp::PROG_F12_FROB2) + prog_muls(slp::PROG_F12_FROB3);
    case 16: return prog_muls(slp::PROG_G1_ADD);
  }
  return 0;
}


// The one-lane group law: sum of n affine points as mixed additions of the first m to the identity,
// of the others to the identity, and the two sums added
template <class L, class A> static A lane_sum(const A *p, int n, int m) {
  lane::pt<L> s[2] = {lane::identity<L>(), lane::identity<L>()};
  for (int i = 0; i < n; i++)
    if (!aff_is_inf(p[i])) s[i >= m] = lane::madd<L>(s[i >= m], L::in(p[i].x), L::in(p[i].y));
  return jac_to_aff(lane::to_jac<L>(lane::add<L>(s[0], s[1])));
}
// k P by the one-lane multiplication
API int hc_lane_mul(const uint8_t *Pb, const uint8_t *kb, uint8_t *out) {
  const fe k = rd_raw(kb);
  lane::pt<lane::G1> tab[16];
  wrg1(out, lane::to_aff<lane::G1>(lane::mul_lane(rdg1(Pb), glv::decompose(k.l), lane::Kept<lane::pt<lane::G1>>{tab})));
  return 0;
}
API int hc_lane_sum(int grp, const uint8_t *pts, int n, int m, uint8_t *out) {
  if (grp == 0) {
    g1_aff p[64];
    for (int i = 0; i < n; i++) p[i] = rdg1(pts + 64 * i);
    wrg1(out, lane_sum<lane::G1>(p, n, m));
  } else {
    g2_aff p[64];
    for (int i = 0; i < n; i++) p[i] = rdg2(pts + 128 * i);
    wrg2(out, lane_sum<lane::G2>(p, n, m));
  }
  return 0;
}

// k P on G1 with the GLV split k = k_0 + k_1 lam: bases B0 = sign(k_0) P and
// B1 = sign(k_1) phi(P), phi(x, y) = (beta x, y); joint 2-bit windows d0 + 4 d1 over the
// table d0 B0 + d1 B1 (Jacobian), two doublings and at most one addition per window
static g1_jac g1_mul_glv(const g1_aff &P, const glv::Dec &d) {
  if (aff_is_inf(P) || d.nbits == 0) return jac_inf<OpsG1>();
  g1_aff B0 = P, B1 = {fp_mul(P.x, fe_const(bn::GLV_BETA)), P.y};
  if (d.neg & 1) B0 = aff_neg(B0);
  if (d.neg & 2) B1 = aff_neg(B1);
  g1_jac T[16];
  T[0] = jac_inf<OpsG1>();
  T[1] = jac_from_aff(B0);
  T[2] = jac_dbl(T[1]);
  T[3] = jac_madd(T[2], B0);
  T[4] = jac_from_aff(B1);
  T[8] = jac_dbl(T[4]);
  T[12] = jac_madd(T[8], B1);
  for (int d1 = 1; d1 < 4; d1++)
    for (int d0 = 1; d0 < 4; d0++) T[d0 + 4 * d1] = jac_add(T[4 * d1], T[d0]);
  int nw = (int)(d.nbits + 1) / 2;
  g1_jac acc = T[glv::digit2(d, (uint32_t)(nw - 1))];
  for (int w = nw - 2; w >= 0; w--) {
    acc = jac_dbl(jac_dbl(acc));
    uint32_t dg = glv::digit2(d, (uint32_t)w);
    if (dg) acc = jac_add(acc, T[dg]);
  }
  return acc;
}

// k P on G1 through the GLV split (host build of the device formulas); P, out affine BE
API int hc_g1_mul_glv(const uint8_t *Pb, const uint8_t *kb, uint8_t *out, uint8_t *dec_out) {
  fe k = rd_raw(kb);
  glv::Dec d = glv::decompose(k.l);
  if (dec_out) memcpy(dec_out, &d, sizeof d);
  wrg1(out, jac_to_aff(g1_mul_glv(rdg1(Pb), d)));
  return 0;
}

#ifdef VC_COUNT_MULS
// Field multiplications (F_p or F_r, Montgomery) performed by one operation of the
// GPU path's formulas: 0 Miller loop, 1 final exponentiation, 2 G1 scalar mul
// (254-bit scalar), 3 G2 scalar mul, 4 G1 add, 5 G1 mixed add, 6 G2 add, 7 G2 mixed
// add, 8 G1 doubling, 9 G2 doubling, 10 F_p12 mul, 11 Jacobian->affine G1 (excluding
// the binary-GCD inversion), 12 Jacobian->affine G2, 13 F_p12 squaring (general).
API uint64_t hc_count(int op) {
  uint8_t gb1[64], gb2[128];
  g1_aff G1 = {fe_const(bn::G1X), fe_const(bn::G1Y)};
  g2_aff G2 = {{fe_const(bn::G2X0), fe_const(bn::G2X1)}, {fe_const(bn::G2Y0), fe_const(bn::G2Y1)}};
  (void)gb1; (void)gb2;
  uint32_t k[8] = {0x9e3779b9u, 0x7f4a7c15u, 0xf39cc060u, 0x5cedc834u, 0x1082276bu, 0xf3a27251u, 0xbe8e7a8bu, 0x2a9d0c3fu};
  g1_jac P1 = jac_dbl(jac_from_aff(G1));
  g2_jac P2 = jac_dbl(jac_from_aff(G2));
  g1_aff A1 = jac_to_aff(P1);
  g2_aff A2 = jac_to_aff(P2);
  fp12 f = miller_loop(G1, G2);
  uint64_t &c = fmul_counter();
  c = 0;
  switch (op) {
    case 0: (void)miller_loop(A1, A2); break;
    case 1: (void)f12_final_exp(f); break;
    case 2: (void)scalar_mul(G1, k); break;
    case 3: (void)scalar_mul(G2, k); break;
    case 4: (void)jac_add(P1, jac_dbl(P1)); break;
    case 5: (void)jac_madd(jac_dbl(P1), G1); break;
    case 6: (void)jac_add(P2, jac_dbl(P2)); break;
    case 7: (void)jac_madd(jac_dbl(P2), G2); break;
    case 8: (void)jac_dbl(P1); break;
    case 9: (void)jac_dbl(P2); break;
    case 10: (void)f12_mul(f, f); break;
    case 11: (void)jac_to_aff(P1); break;
    case 12: (void)jac_to_aff(P2); break;
    case 13: (void)f12_sqr(f); break;
    default: return 0;
  }
  uint64_t n = c;
  // subtract the set-up work done inside the measured expression
  c = 0;
  switch (op) {
    case 4: (void)jac_dbl(P1); break;
    case 5: (void)jac_dbl(P1); break;
    case 6: (void)jac_dbl(P2); break;
    case 7: (void)jac_dbl(P2); break;
    default: break;
  }
  return n - c;
}
#endif

// the index map of the terms taken one round ahead (oa_terms.hpp): term id as (a, v, out)
API void hc_oa_term(uint64_t id, uint64_t K, uint64_t nb, uint64_t q, uint64_t *out) {
  oat::Term t = oat::term(id, K, nb, q);
  out[0] = t.a;
  out[1] = t.v;
  out[2] = t.out;
}

// the launch grid of a workgroup for each of N proofs
API void hc_proof_grid(uint64_t N, uint32_t *xy) {
  const ProofGrid g = proof_grid(N);
  xy[0] = g.x;
  xy[1] = g.y;
}

// a batch of 30 division steps: delta, the low words of f (odd) and g -> the matrix u, v, q, r and delta after it
API void hc_divsteps_batch(int32_t delta, uint32_t f, uint32_t g, int32_t *out) {
  const divsteps::Mat t = divsteps::batch(delta, f, g);
  out[0] = t.u; out[1] = t.v; out[2] = t.q; out[3] = t.r;
  out[4] = delta;
}

// ---------------------------------------------------------------- two lanes a point, a pairing
typedef lane::Both<lane::fl> Pair;
typedef lane::G2pairOf<Pair> G2lanes;
static Pair pair_in(const fp2 &x) { return {{lane::in_small(x.c0), lane::in_small(x.c1)}}; }
static fp2 pair_out(const Pair &x) { return {lane::out(x.l[0]), lane::out(x.l[1])}; }
static bool is_inf2(const g2_aff &q) { return aff_is_inf(q); }

// k Q + A on G2 by a pair of lanes (A the identity: left out)
API int hc_pair_mul(const uint8_t *Qb, const uint8_t *kb, const uint8_t *Ab, uint8_t *out) {
  const fe k = rd_raw(kb);
  const g2_aff Q = rdg2(Qb), A = rdg2(Ab);
  lane::pt<G2lanes> tab[16];
  lane::pt<G2lanes> t = lane::mul_pair(pair_in(Q.x), pair_in(Q.y), is_inf2(Q), gls::decompose(k.l), lane::Kept<lane::pt<G2lanes>>{tab});
  if (!is_inf2(A)) t = lane::madd<G2lanes>(t, pair_in(A.x), pair_in(A.y));
  const fp2 z = pair_out(t.Z);
  if (f2_is_zero(z)) {
    wrg2(out, aff_inf<OpsG2>());
    return 0;
  }
  const fp2 zi = f2_inv(z);
  const Pair zl = {{lane::in(zi.c0), lane::in(zi.c1)}};
  wrg2(out, {pair_out(G2lanes::mul(t.X, zl)), pair_out(G2lanes::mul(t.Y, zl))});
  return 0;
}
// the product of n Miller values by pairs of lanes (before the final exponentiation)
API int hc_pair_miller(const uint8_t *Pb, const uint8_t *Qb, int n, uint8_t *out) {
  lane::twelve<Pair> f;
  for (int i = 0; i < n; i++) {
    const g1_aff P = rdg1(Pb + 64 * i);
    const g2_aff Q = rdg2(Qb + 128 * i);
    const lane::fl x = lane::in_small(P.x), y = lane::in_small(P.y);
    const lane::twelve<Pair> g = lane::miller_pair(lane::Lanes{}, Pair{{x, x}}, Pair{{y, y}}, pair_in(Q.x), pair_in(Q.y));
    f = i ? lane::mul12(lane::Lanes{}, f, g) : g;
  }
  fp12 o;
  fe *w = reinterpret_cast<fe *>(&o);
  for (int q = 0; q < 6; q++)
    for (int p = 0; p < 2; p++) w[2 * q + p] = lane::out((q < 3 ? f.a.c[q] : f.b.c[q - 3]).l[p]);
  wr12(out, o);
  return 0;
}

// ---------------------------------------------------------------- bounds of the lane kernels' limbs and values
// Runs the kernels' formulas on bounds; w: how near the worst column, limb, argument of `reduce` come to
// what they may be (1), the largest value packed, plus p (2), and the largest coordinate of a point.  Returns whether sums of any length stay within
// the bounds found (the others' steps are run one by one).
namespace {
using lane::Bnd;
template <class L> struct Bounds {
  typedef lane::pt<L> pt;
  // grows acc by step until that adds less than EPS, widens it a little and looks whether step keeps within
  template <class F> static bool closed(pt &acc, F step) {
    for (int i = 0; i < 200; i++) acc = lane::join(acc, step(acc));
    const pt wide = widened(acc);
    acc = wide;
    return within(step(wide), wide);
  }
  static Bnd widen(const Bnd &a) { return {a.u * (1 + 1e-6), a.v * (1 + 1e-6)}; }
  static lane::over2<Bnd> widen(const lane::over2<Bnd> &a) { return {widen(a.c0), widen(a.c1)}; }
  static lane::Both<Bnd> widen(const lane::Both<Bnd> &a) { return {{widen(a.l[0]), widen(a.l[1])}}; }
  static pt widened(const pt &a) { return {widen(a.X), widen(a.Y), widen(a.Z)}; }
  static bool le(const Bnd &a, const Bnd &b) { return a.u <= b.u && a.v <= b.v; }
  static bool le(const lane::over2<Bnd> &a, const lane::over2<Bnd> &b) { return le(a.c0, b.c0) && le(a.c1, b.c1); }
  static bool le(const lane::Both<Bnd> &a, const lane::Both<Bnd> &b) { return le(a.l[0], b.l[0]) && le(a.l[1], b.l[1]); }
  static bool within(const pt &a, const pt &b) { return le(a.X, b.X) && le(a.Y, b.Y) && le(a.Z, b.Z); }
};
double widest;
void largest(const Bnd &a) { widest = std::fmax(widest, a.v); }
void largest(const lane::over2<Bnd> &a) { largest(a.c0); largest(a.c1); }
void largest(const lane::Both<Bnd> &a) { largest(a.l[0]); largest(a.l[1]); }
template <class L> void largest(const lane::pt<L> &t) { largest(t.X); largest(t.Y); largest(t.Z); }
void pack(const lane::over2<Bnd> &a) { pack(a.c0); pack(a.c1); }
void pack(const lane::Both<Bnd> &a) { pack(a.l[0]); pack(a.l[1]); }
// what follows: packed as it is, to Jacobian form, to affine form (z: a packed inverse)
template <class L> void results(const lane::pt<L> &t, const typename L::T &z) {
  largest(t);
  pack(t.X); pack(t.Y); pack(t.Z);
  pack(L::mul(t.X, t.Z)); pack(L::mul(L::mul(t.Y, t.Z), t.Z));
  pack(L::mul(t.X, z)); pack(L::mul(t.Y, z));
}
// a multi-scalar multiplication: mixed additions of packed points, then sums of sums
template <class L> bool msm_bounds(const typename L::T &a) {
  typedef lane::pt<L> pt;
  pt acc = lane::identity<L>();
  const bool ok = Bounds<L>::closed(acc, [&](const pt &t) { return lane::join(lane::madd<L>(t, a, a), lane::add<L>(t, t)); });
  results<L>(acc, a);
  return ok;
}
}  // namespace

API int hc_lane_bounds(int which, double *w) {
  lane::bounds::worst = {};
  widest = 0;
  const Bnd in = lane::packed(), one = lane::const29<Bnd>(bn::P_ONE29), small = lane::mul(in, one);
  bool ok = true;
  if (which == 0) {
    ok = msm_bounds<lane::G1of<Bnd>>(in);
  } else if (which == 1) {
    ok = msm_bounds<lane::G2of<Bnd>>({in, in});
  } else if (which == 2) {
    // a multiplication, a packed point added (the folds), sums of up to 64 (the terms)
    typedef lane::G1of<Bnd> L;
    glv::Dec d;
    memset(&d, 0xff, sizeof d);
    d.nbits = 128;
    lane::pt<L> tab = {}, t = lane::mul_table(small, small, lane::mul(small, in), one, d, lane::Joined<lane::pt<L>>{&tab});
    results<L>(lane::madd<L>(t, in, in), in);
    for (int i = 0; i < 6; i++) t = lane::join(t, lane::add<L>(t, t));
    results<L>(t, in);
  } else if (which == 3) {
    typedef lane::Both<Bnd> V;
    typedef lane::G2pairOf<V> L;
    gls::Dec d;
    memset(&d, 0xff, sizeof d);
    d.nbits = 96;
    const V s = {{small, small}};
    lane::pt<L> tab = {}, t = lane::mul_pair(s, s, false, d, lane::Joined<lane::pt<L>>{&tab});
    t = lane::join(t, lane::madd<L>(t, s, s));
    largest(t);
    pack(t.Z);
    pack(L::mul(t.X, V{{in, in}}));
    pack(L::mul(t.Y, V{{in, in}}));
  } else {
    typedef lane::Both<Bnd> V;
    const V s = {{small, small}};
    lane::twelve<V> f = lane::miller_pair(lane::Lanes{}, s, s, s, s);
    for (int i = 0; i < 5; i++) f = lane::mul12(lane::Lanes{}, f, f);
    for (int q = 0; q < 3; q++) {
      pack(f.a.c[q]);
      pack(f.b.c[q]);
    }
  }
  const lane::bounds::Worst &b = lane::bounds::worst;
  w[0] = b.column; w[1] = b.limb; w[2] = b.reduced; w[3] = b.packed; w[4] = widest;
  return ok;
}

// sum_n a_n b_n 2^{-261}, six products of 9 limbs each; k a + b less its quotient by p
API void hc_lane_dot6(const int32_t *a, const int32_t *b, int32_t *o) {
  lane::fl x[6], y[6];
  const lane::fl *px[6], *py[6];
  for (int n = 0; n < 6; n++) {
    x[n] = lane::const29<lane::fl>(a + 9 * n);
    y[n] = lane::const29<lane::fl>(b + 9 * n);
    px[n] = &x[n];
    py[n] = &y[n];
  }
  const lane::fl r = lane::dot6(px, py);
  memcpy(o, r.l, sizeof r.l);
}
API void hc_lane_reduce(const int32_t *a, int k, const int32_t *b, int32_t *o) {
  const lane::fl r = lane::reduce(lane::const29<lane::fl>(a), k, lane::const29<lane::fl>(b));
  memcpy(o, r.l, sizeof r.l);
}
// the canonical residue of an engine slot's limbs, and of the sum of four
API void hc_canon29(const int32_t *l, uint8_t *out) {
  slp::f29 x = {};
  for (int j = 0; j < 9; j++) x.l[j] = (uint32_t)l[j];
  wr<FpP>(out, slp::from29(slp::canon29(x)));
}
API void hc_red29(const int64_t *c, int32_t *o) {
  const slp::f29 r = slp::red29(c);
  for (int j = 0; j < 9; j++) o[j] = (int32_t)r.l[j];
}

// operations of program prog (0 .. 8: the group laws' that write the accumulator) that write a slot of T
// and are neither products nor copies of 0 or 1; -1 for another number
API int hc_sums_into_T(int prog) {
  static const int g1[] = {slp::PROG_G1_DBL2, slp::PROG_G1_DBL2_ADD, slp::PROG_G1_MADD, slp::PROG_G1_ADD},
                   g2[] = {slp::PROG_G2_DBL, slp::PROG_G2_DBL_ADD, slp::PROG_G2_MADD, slp::PROG_G2_ADD, slp::PROG_G2_LOAD};
  if (prog < 0 || prog >= 9) return -1;
  const bool two = prog >= 4;
  const int first = two ? slp::G2_T_0_0_0 : slp::G1_T_0_0, n = two ? g2m::NT : g1m::NT;
  const slp::Call c = slp::call(two ? g2[prog - 4] : g1[prog]);
  int sums = 0;
  for (int v = 0; v < 4; v++)
    for (uint32_t d = c.d[v]; d; d = slp::blk_word(slp::OPS, d, 0, 1))
      for (int i = 0; i < slp::blk_ops(d); i++) {
        const uint32_t head = slp::blk_word(slp::OPS, d, 2 * i, 0);
        const int dst = (int)(slp::term_addr(head, c.rel) / 48);
        if (dst < first || dst >= first + n || slp::term_coef(head) == 1) continue;
        int terms = 0, consts = 0;  // (a copy of the constant 0 or 1, the first two)
        for (int h = 0; h < 2; h++)
          for (int t = 0; t < slp::blk_terms(d); t++) {
            const uint32_t w = slp::blk_word(slp::OPS, d, 2 * i + h, 2 + t);
            const int src = (int)(slp::term_addr(w, c.rel) / 48), base = two ? slp::G2_CBASE : slp::G1_CBASE;
            terms += slp::term_coef(w) != 0;
            consts += slp::term_coef(w) == 1 && (src == base || src == base + 1);
          }
        if (terms != 1 || consts != 1) sums++;
      }
  return sums;
}
