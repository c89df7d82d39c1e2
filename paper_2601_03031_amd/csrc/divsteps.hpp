// Modular inverse by batches of 30 division steps (D. J. Bernstein, B.-Y. Yang, "Fast constant-time
// gcd computation and modular inversion", 2019; here in variable time, the inputs are public).
// From f = m, g = x, delta = 1 a division step maps (delta, f, g) to
//   (1 - delta, g, (g - f) / 2)         if delta > 0 and g is odd,
//   (1 + delta, f, (g + (g mod 2) f) / 2)  otherwise;
// 741 of them bring g to 0 and f to +-1 for 256-bit inputs.  The steps of a batch depend on the
// low 30 bits of f and g alone; their product, a 2 x 2 matrix t / 2^30 with row sums |u| + |v| <=
// 2^30, is then applied to f and g (exactly) and, modulo m, to d and e with f = d x, g = e x.
// With delta at or below 0 the next 1 - delta steps swap nothing, whatever g's bits are: together they add
// w f to g, w = -g / f mod 2^n, n = 1 - delta, and halve n times.  After them delta is above 0; then an even g is halved,
// and an odd one swaps.  A swap's (f, g) -> (g, -f) and the run without one that follows it, of 1 + delta steps, are one
// combination, g -> w g - f with w = f / g mod 2^(1 + delta), and its halvings one shift with those of the even g's.
// Numbers are 9 signed limbs of 30 bits, the lower 8 in [0, 2^30).  d and e are not reduced on the
// way: with the multiple of m taken in [-2^29, 2^29) each batch adds at most m / 2 to them.
#pragma once
#include <cstdint>

#ifndef __HIPCC__
#define __host__
#define __device__
#define __forceinline__ inline
#endif

namespace divsteps {

static constexpr int NL = 9, BATCHES = 25;
static constexpr uint32_t MASK = 0x3fffffffu;

struct Mat {
  int32_t u, v, q, r;
};

// limb i of the 256-bit integer x
__host__ __device__ constexpr int32_t limb30(const uint32_t *x, int i) {
  const int w = 30 * i >> 5, s = 30 * i & 31;
  uint32_t v = x[w] >> s;
  if (s > 2 && w + 1 < 8) v |= x[w + 1] << (32 - s);
  return (int32_t)(v & MASK);
}

// the low bits of f or g within a batch, and its coefficients of the f and g that the batch began with
// (times 2 for each step so far)
struct Low {
  uint32_t x, f, g;
};

// x / f mod 2^n, for odd f and 0 < n < 32.  f is its own inverse mod 8 (odd squares are 1 there), and Newton's
// step for 1 / f doubles the bits that are right.
__host__ __device__ __forceinline__ uint32_t quotient(uint32_t x, uint32_t f, int n) {
  uint32_t inv = f * (2 - f * f);
  for (int right = 6; right < n; right *= 2) inv *= 2 - f * inv;
  return x * inv & ((1u << n) - 1);
}

// 30 steps from the low bits of f (odd) and g
__host__ __device__ __forceinline__ Mat batch(int32_t &delta, uint32_t flow, uint32_t glow) {
  Low f = {flow, 1, 0}, g = {glow, 0, 1};
  int left = 30;
  if (delta <= 0) {  // the rest of a run that the batch before began
    const uint32_t w = quotient(0u - g.x, f.x, 1 - delta < left ? 1 - delta : left);
    g = {g.x + w * f.x, w * f.f, 1 + w * f.g};
  }
  for (;;) {
    const int halved = __builtin_ctz(g.x | 1u << left);  // (at most the steps that are left)
    g.x >>= halved;
    f.f <<= halved;
    f.g <<= halved;
    delta += halved;
    left -= halved;
    if (left == 0) return {(int32_t)f.f, (int32_t)f.g, (int32_t)g.f, (int32_t)g.g};
    const uint32_t w = quotient(f.x, g.x, 1 + delta < left ? 1 + delta : left);
    const Low was = f;
    f = g;
    g = {w * f.x - was.x, w * f.f - was.f, w * f.g - was.g};
    delta = -delta;
  }
}

// o = (a x + b y + k m) / 2^30, with k (masked by kmask) the multiple that makes the low limb zero.
// On the f, g rows the low limb of a x + b y is zero already and kmask is 0.
template <class F>
__host__ __device__ __forceinline__ void row(const int32_t *x, const int32_t *y, int32_t a, int32_t b, int32_t kmask, int32_t *o) {
  int64_t c = (int64_t)a * x[0] + (int64_t)b * y[0];
  // F::INV = -1 / m mod 2^32; the multiple as a signed 30-bit number
  const int32_t k = (int32_t)(((uint32_t)c * F::INV) << 2) >> 2 & kmask;
  c += (int64_t)k * limb30(F::M, 0);
  c >>= 30;
#pragma unroll
  for (int i = 1; i < NL; i++) {
    c += (int64_t)a * x[i] + (int64_t)b * y[i] + (int64_t)k * limb30(F::M, i);
    o[i - 1] = (int32_t)((uint32_t)c & MASK);
    c >>= 30;
  }
  o[NL - 1] = (int32_t)c;
}

// d (-d with neg), within 2^9 m, as a canonical integer of 8 words
template <class F> __host__ __device__ __forceinline__ void finish(const int32_t *d, bool neg, uint32_t *out) {
  // d = q m + rest, |rest| <= 0.6 m, q from the top limb (14 bits of m lie there)
  const float est = (float)d[NL - 1] * (1.0f / (float)limb30(F::M, NL - 1));
  const int32_t q = (int32_t)(est + (est < 0 ? -0.5f : 0.5f));
  const int32_t sg = neg ? -1 : 1, k = 1 - sg * q;
  uint32_t t[NL];
  int64_t c = 0;
#pragma unroll
  for (int i = 0; i < NL; i++) {
    c += (int64_t)sg * d[i] + (int64_t)k * limb30(F::M, i);
    t[i] = (uint32_t)c & MASK;
    c >>= 30;
  }
#pragma unroll
  for (int w = 0; w < 8; w++) {
    const int b = 32 * w, j = b / 30, s = b % 30;
    uint32_t v = t[j] >> s | t[j + 1] << (30 - s);
    if (s > 28 && j + 2 < NL) v |= t[j + 2] << (60 - s);
    out[w] = v;
  }
  // within (0.4 m, 1.6 m): one subtraction
  uint32_t r[8];
  int64_t bw = 0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    bw += (int64_t)out[i] - F::M[i];
    r[i] = (uint32_t)bw;
    bw >>= 32;
  }
#pragma unroll
  for (int i = 0; i < 8; i++) out[i] = bw < 0 ? out[i] : r[i];
}

// x^{-1} mod m of the integer 0 < x < m, one lane by itself
template <class F> __host__ __device__ __forceinline__ void inverse(const uint32_t *x, uint32_t *out) {
  int32_t f[NL], g[NL], d[NL], e[NL], delta = 1;
#pragma unroll
  for (int i = 0; i < NL; i++) {
    f[i] = limb30(F::M, i);
    g[i] = limb30(x, i);
    d[i] = 0;
    e[i] = i == 0;
  }
  for (int b = 0; b < BATCHES; b++) {
    int32_t any = 0;
#pragma unroll
    for (int i = 0; i < NL; i++) any |= g[i];
    if (any == 0) break;
    const Mat t = batch(delta, (uint32_t)f[0], (uint32_t)g[0]);
    int32_t n0[NL], n1[NL];
    row<F>(f, g, t.u, t.v, 0, n0);
    row<F>(f, g, t.q, t.r, 0, n1);
#pragma unroll
    for (int i = 0; i < NL; i++) { f[i] = n0[i]; g[i] = n1[i]; }
    row<F>(d, e, t.u, t.v, -1, n0);
    row<F>(d, e, t.q, t.r, -1, n1);
#pragma unroll
    for (int i = 0; i < NL; i++) { d[i] = n0[i]; e[i] = n1[i]; }
  }
  finish<F>(d, f[NL - 1] < 0, out);
}

#ifdef __HIPCC__
// The same for an x that is equal in every lane of a fully active wavefront: the steps of a batch
// run on the scalar unit, and lanes 0 .. 3 of each four hold f, g, d and e, so that one pass of the
// vector unit over 9 limbs applies the matrix to all four.  About 19 us (a final exponentiation,
// which has one, 0.360 -> 0.322 ms); a binary GCD all on the scalar unit took 57.
template <class F> __device__ __forceinline__ void inverse_uniform(const uint32_t *x, uint32_t *out) {
  const int p = threadIdx.x & 3;
  const int32_t kmask = p & 2 ? -1 : 0;
  int32_t own[NL], delta = 1;
#pragma unroll
  for (int i = 0; i < NL; i++) own[i] = p == 0 ? limb30(F::M, i) : p == 1 ? limb30(x, i) : p == 3 ? (i == 0) : 0;
#pragma unroll 1
  for (int b = 0; b < BATCHES; b++) {
    const uint32_t f0 = __builtin_amdgcn_readlane(own[0], 0), g0 = __builtin_amdgcn_readlane(own[0], 1);
    if (g0 == 0) {
      int32_t any = 0;
#pragma unroll
      for (int i = 0; i < NL; i++) any |= own[i];
      if (__builtin_amdgcn_readlane(any, 1) == 0) break;
    }
    const Mat t = batch(delta, f0, g0);
    int32_t other[NL], o[NL];
#pragma unroll
    for (int i = 0; i < NL; i++) other[i] = __builtin_amdgcn_mov_dpp(own[i], 0xB1, 0xF, 0xF, true);  // lane ^ 1
    // even rows: u own + v other; odd rows: r own + q other
    row<F>(own, other, p & 1 ? t.r : t.u, p & 1 ? t.q : t.v, kmask, o);
#pragma unroll
    for (int i = 0; i < NL; i++) own[i] = o[i];
  }
  int32_t d[NL];
#pragma unroll
  for (int i = 0; i < NL; i++) d[i] = __builtin_amdgcn_readlane(own[i], 2);
  finish<F>(d, __builtin_amdgcn_readlane(own[NL - 1], 0) < 0, out);
}
#endif

}  // namespace divsteps
