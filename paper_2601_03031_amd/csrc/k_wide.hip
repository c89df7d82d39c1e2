// Kernels in the wide layout (field_wide.hpp): 8 lanes per field element, so one
// 64-lane block serves 8 independent point sums.  These are short dependent chains
// whose count of independent items per launch is far below the lane count of the chip.
//
// Memory layouts are the same as everywhere else (32-byte little-endian field
// elements, points as consecutive elements): lane g of a group loads limb g.
#define VC_WIDE 1
#include <hip/hip_runtime.h>
#include "field.hpp"
#include "tower.hpp"
#include "curve.hpp"
#include "kernels.h"

#define TPBW 64
#define GPB (TPBW / 8)  // groups (elements) per block

namespace prof {
void begin(const char *name, hipStream_t st);
void end(hipStream_t st);
void name_last(const char *name);
}  // namespace prof
namespace dbg {
bool on();
void check(const char *name, hipStream_t st);
}  // namespace dbg

static inline unsigned nblkw(uint64_t n) { return (unsigned)((n + GPB - 1) / GPB); }
__device__ __forceinline__ uint64_t wgid() { return (uint64_t)blockIdx.x * GPB + (threadIdx.x >> 3); }

// element idx of a type made of n field elements, lane g taking limb g of each
template <class T> __device__ __forceinline__ T wld(const void *base, uint64_t idx) {
  constexpr int n = sizeof(T) / 4;
  T r;
  uint32_t *rv = reinterpret_cast<uint32_t *>(&r);
  const uint32_t *src = static_cast<const uint32_t *>(base) + idx * (uint64_t)n * 8 + wg();
#pragma unroll
  for (int k = 0; k < n; k++) rv[k] = src[k * 8];
  return r;
}
template <class T> __device__ __forceinline__ void wst(void *base, uint64_t idx, const T &v) {
  constexpr int n = sizeof(T) / 4;
  const uint32_t *rv = reinterpret_cast<const uint32_t *>(&v);
  uint32_t *dst = static_cast<uint32_t *>(base) + idx * (uint64_t)n * 8 + wg();
#pragma unroll
  for (int k = 0; k < n; k++) dst[k * 8] = rv[k];
}

// W of every job at level d: segment s = x 2^d + p (reduced at in + s stride) is W_x[2^d - 1 + p]
__global__ void __launch_bounds__(TPBW) kw_w_aff(const S2Job *J, uint32_t G, const void *in, uint64_t stride, uint32_t d) {
  uint64_t s = wgid();
  if (s >= ((uint64_t)G << d)) return;
  const uint64_t x = s >> d, p = s & ((1ull << d) - 1);
  g1_aff a = jac_to_aff(wld<g1_jac>(in, s * stride));
  wst(J[x].W, (1ull << d) - 1 + p, a);
}

// ---------------------------------------------------------------- sums
template <class O>
__global__ void __launch_bounds__(TPBW) kw_jac_step(void *data, uint64_t nseg, uint64_t stride, uint64_t len, uint64_t s) {
  uint64_t per = (len + 2 * s - 1) / (2 * s);
  uint64_t id = wgid();
  if (id >= nseg * per) return;
  uint64_t g = id / per, q = id % per;
  uint64_t a = 2 * s * q, b = a + s;
  if (b >= len) return;
  jac<O> x = wld<jac<O>>(data, g * stride + a), y = wld<jac<O>>(data, g * stride + b);
  wst(data, g * stride + a, jac_add(x, y));
}

template <class O>
__global__ void __launch_bounds__(TPBW) kw_jac_to_aff(const void *in, uint64_t stride, uint64_t n, void *out,
                                                     uint64_t ostride) {
  uint64_t i = wgid();
  if (i >= n) return;
  wst(out, i * ostride, jac_to_aff(wld<jac<O>>(in, i * stride)));
}

// out[s] = affine(sum_{q < len} data[s len + q])
__global__ void __launch_bounds__(TPBW) kw_sum_g1(const void *data, uint64_t nseg, uint64_t len, void *out) {
  uint64_t s = wgid();
  if (s >= nseg) return;
  g1_jac acc = wld<g1_jac>(data, s * len);
  for (uint64_t q = 1; q < len; q++) acc = jac_add(acc, wld<g1_jac>(data, s * len + q));
  wst(out, s, jac_to_aff(acc));
}

// C_j of every job of a batched commit: the sum of its nslice MSM block results, affine, into
// the job's commitment and into the packed array Cp (entry k0 + j)
__global__ void __launch_bounds__(TPBW) kw_commit_sums(const CJob *J, uint32_t n, uint64_t total, void *Cp) {
  uint64_t i = wgid();
  if (i >= total) return;
  uint32_t lo = 0, hi = n;  // the job holding packed entry i
  while (hi - lo > 1) {
    uint32_t mid = (lo + hi) / 2;
    if (J[mid].k0 <= i) lo = mid;
    else hi = mid;
  }
  const CJob &c = J[lo];
  const uint64_t j = i - c.k0;
  g1_jac acc = wld<g1_jac>(c.part, j * c.nslice);
  for (uint64_t q = 1; q < c.nslice; q++) acc = jac_add(acc, wld<g1_jac>(c.part, j * c.nslice + q));
  g1_aff a = jac_to_aff(acc);
  wst(c.Cj, j, a);
  wst(Cp, i, a);
}

__global__ void __launch_bounds__(TPBW) kw_dlevel(const S2Job *J, uint32_t G, uint64_t K, uint32_t h) {
  uint64_t w = wgid();
  if (w >= G * (K >> h)) return;
  g1_aff *D = J[w / (K >> h)].D;
  w %= K >> h;
  uint64_t off = 2 * K - ((2 * K) >> h), offc = 2 * K - ((2 * K) >> (h - 1));
  g1_aff l = wld<g1_aff>(D, offc + 2 * w), r = wld<g1_aff>(D, offc + 2 * w + 1);
  wst(D, off + w, jac_to_aff(jac_madd(jac_from_aff(l), r)));
}


// ---------------------------------------------------------------- diagnostics
// field operation on canonical inputs (limbs), for the layout self-test:
// op 0 mul, 1 add, 2 sub, 3 half, 4 inverse, 5 square; F_p if which == 0, F_r if 1;
// which 2 (F_p) / 3 (F_r): ops 0-2 on raw Montgomery limbs, no conversion either way
__global__ void __launch_bounds__(TPBW) kw_diag_field(int which, int op, const void *a, const void *b, uint64_t n,
                                                     void *out) {
  uint64_t i = wgid();
  if (i >= n) return;
  fe x = wld<fe>(a, i), y = wld<fe>(b, i), r;
  if (which >= 2) {
    // raw Montgomery limbs in and out (ops 0 mul, 1 add, 2 sub), to check the range of results
    if (which == 2) r = op == 0 ? f_mul<FpP>(x, y) : op == 1 ? f_add<FpP>(x, y) : f_sub<FpP>(x, y);
    else r = op == 0 ? f_mul<FpR>(x, y) : op == 1 ? f_add<FpR>(x, y) : f_sub<FpR>(x, y);
  } else if (which == 0) {
    x = f_to_mont<FpP>(x);
    y = f_to_mont<FpP>(y);
    switch (op) {
      case 0: r = fp_mul(x, y); break;
      case 1: r = fp_add(x, y); break;
      case 2: r = fp_sub(x, y); break;
      case 3: r = fp_half(x); break;
      case 4: r = fp_inv(x); break;
      default: r = fp_sqr(x); break;
    }
    r = f_from_mont<FpP>(r);
  } else {
    x = f_to_mont<FpR>(x);
    y = f_to_mont<FpR>(y);
    switch (op) {
      case 0: r = fr_mul(x, y); break;
      case 1: r = fr_add(x, y); break;
      case 2: r = fr_sub(x, y); break;
      case 3: r = f_half<FpR>(x); break;
      case 4: r = fr_inv(x); break;
      default: r = f_sqr<FpR>(x); break;
    }
    r = f_from_mont<FpR>(r);
  }
  wst(out, i, r);
}

// ---------------------------------------------------------------- launchers
namespace klw {
#define LW(kern, n, ...)                                                                     \
  do {                                                                                       \
    prof::begin(#kern, st);                                                                  \
    hipLaunchKernelGGL(kern, dim3(nblkw(n)), dim3(TPBW), 0, st, __VA_ARGS__);                \
    prof::end(st);                                                                           \
    prof::name_last(#kern);                                                                  \
    if (dbg::on()) dbg::check(#kern, st);                                                    \
  } while (0)

void w_aff(const S2Job *J, uint32_t G, const void *in, uint64_t stride, uint32_t d, hipStream_t st) {
  LW(kw_w_aff, (uint64_t)G << d, J, G, in, stride, d);
}
void g1_reduce(void *data, uint64_t nseg, uint64_t stride, uint64_t len, hipStream_t st) {
  for (uint64_t s = 1; s < len; s <<= 1) {
    uint64_t per = (len + 2 * s - 1) / (2 * s);
    LW(kw_jac_step<OpsG1>, nseg * per, data, nseg, stride, len, s);
  }
}
void g1_to_aff(const void *in, uint64_t stride, uint64_t n, void *out, uint64_t ostride, hipStream_t st) {
  LW(kw_jac_to_aff<OpsG1>, n, in, stride, n, out, ostride);
}
void sum_g1(const void *data, uint64_t nseg, uint64_t len, void *out, hipStream_t st) { LW(kw_sum_g1, nseg, data, nseg, len, out); }
void commit_sums(const CJob *J, uint32_t n, uint64_t total, void *Cp, hipStream_t st) {
  if (total) LW(kw_commit_sums, total, J, n, total, Cp);
}
void dlevel(const S2Job *J, uint32_t G, uint64_t K, uint32_t h, hipStream_t st) {
  LW(kw_dlevel, G * (K >> h), J, G, K, h);
}
void diag_field(int which, int op, const void *a, const void *b, uint64_t n, void *out, hipStream_t st) {
  LW(kw_diag_field, n, which, op, a, b, n, out);
}
}  // namespace klw
