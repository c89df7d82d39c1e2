// Kernels on the workgroup-cooperative engine (slp.hpp): Miller loops, F_p12 product trees,
// the final exponentiation, scalar multiplications and powers, one workgroup of two wavefronts
// per pairing / product / element.
#include "kcommon.hpp"
#include "slp.hpp"
#include "g2mul.hpp"
#include "gtpow.hpp"
#include "g1mul.hpp"
#include "oa_terms.hpp"

// every program family but the final exponentiation's is scheduled for the same number of
// wavefronts, so that a kernel may run several of them
#define SLP_W 2
#define SLP_T (64 * SLP_W)
#define FE_T (64 * slp::FE_WAVES)
static_assert(slp::ML_WAVES == SLP_W && slp::F12_WAVES == SLP_W && slp::G1_WAVES == SLP_W && slp::G2_WAVES == SLP_W,
              "programs scheduled for another workgroup size");
typedef slp::DevCtx<SLP_W> Ctx;
typedef slp::DevCtx<SLP_W, true> CtxInline;  // for kernels with one place that runs calls
// slots of a kernel that runs only some of a family's programs (the tables' take the most)
constexpr int most(int a, int b = 0, int c = 0, int d = 0) {
  const int x = a > b ? a : b, y = c > d ? c : d;
  return x > y ? x : y;
}
constexpr int G1_DBL_SLOTS = most(slp::G1_DBL2_SLOTS, slp::G1_AFF_SLOTS);
constexpr int G2_AFF_ALL_SLOTS = most(slp::G2_NORM_SLOTS, slp::G2_AFF_SLOTS);
constexpr int G2_DBL_ALL_SLOTS = most(slp::G2_DBL_SLOTS, slp::G2_LOAD_SLOTS, G2_AFF_ALL_SLOTS);
// the call list of a workgroup in LDS
#define CALL_LIST() __shared__ slp::Call calls_sh[slp::MAX_CALLS + 1]

namespace {

__device__ __forceinline__ bool g1_inf(const g1_aff &P) { return fe_is_zero(P.x) && fe_is_zero(P.y); }
__device__ __forceinline__ bool g2_inf(const g2_aff &Q) {
  return fe_is_zero(Q.x.c0) && fe_is_zero(Q.x.c1) && fe_is_zero(Q.y.c0) && fe_is_zero(Q.y.c1);
}

using slp::f29;

template <int NCONST, int T = SLP_T>
__device__ __forceinline__ void load_consts(f29 *S, int base, const uint32_t (*C)[9]) {
  for (int c = threadIdx.x; c < NCONST; c += T) {
    f29 v;
#pragma unroll
    for (int j = 0; j < 9; j++) v.l[j] = C[c][j];
    v.l[9] = v.l[10] = v.l[11] = 0;
    S[base + c] = v;
  }
}

// Miller loop of e(P, Q) into dst (12 coefficients); identity inputs give 1.
__device__ __forceinline__ void miller_one(CtxInline c, const g1_aff *P, const g2_aff *Q, fp12 *dst) {
  f29 *S = c.S;
  const int t = threadIdx.x;
  fe *out = reinterpret_cast<fe *>(dst);
  if (g1_inf(*P) || g2_inf(*Q)) {
    if (t < 12) out[t] = t == 0 ? f_one<FpP>() : fe_zero();
    return;
  }
  if (t < 2) S[slp::ML_xP + t] = slp::to29(t ? P->y : P->x);
  else if (t < 6) {
    const fe *q = reinterpret_cast<const fe *>(Q);
    S[slp::ML_xP + t] = slp::to29(q[t - 2]);  // xQ.0, xQ.1, yQ.0, yQ.1
  }
  load_consts<slp::ML_NCONST>(S, slp::ML_CBASE, slp::ML_CONSTS);
  c.run(slp::PROG_ML, 0, 0, 0);
  if (t < 12) out[t] = slp::from29(slp::canon29(S[slp::ML_f_0 + t]));
}

}  // namespace

// out[i] = Miller(P[i sp], Q[i sq])
__global__ void __launch_bounds__(SLP_T, 4) ks_miller(const g1_aff *P, uint64_t sp, const g2_aff *Q, uint64_t sq, uint64_t n,
                                                  fp12 *out) {
  __shared__ f29 S[slp::ML_NSLOT];
  __shared__ slp::Call calls_sh[1];
  uint64_t i = blockIdx.x;
  if (i >= n) return;
  miller_one(CtxInline{S, calls_sh}, P + i * sp, Q + i * sq, out + i);
}

// side 0 (L) pairs A[h+i] with V[i], side 1 (R) A[i] with V[h+i]; F[(2k+side) K/2 + i]
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_miller(const g1_aff *A, const g2_aff *V, uint64_t K, uint64_t nb, uint64_t h,
                                                     fp12 *F) {
  CHAIN_PRIORITY();
  __shared__ f29 S[slp::ML_NSLOT];
  __shared__ slp::Call calls_sh[1];
  uint64_t id = blockIdx.x;
  if (id >= nb * 2 * h) return;
  uint64_t k = id / (2 * h), r = id % (2 * h), side = r / h, i = r % h;
  const g1_aff *P = A + (side ? k * K + i : k * K + h + i);
  const g2_aff *Q = V + (side ? k * K + h + i : k * K + i);
  miller_one(CtxInline{S, calls_sh}, P, Q, F + (k * 2 + side) * (K / 2) + i);
}

// Of the n workgroups that meet at a counter, the last to arrive returns true (and resets it);
// what the others wrote before is visible to it.  The fences are one lane's, between barriers:
// each writes back or drops cache lines, and with both wavefronts issuing them a launch of 2^15
// F_p12 products took 1.19 ms against 0.46 ms with one wavefront a workgroup.
__device__ bool last_arrival(uint32_t *cnt, uint32_t n, uint32_t *flag) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    const uint32_t old = atomicAdd(cnt, 1u);
    if (old == n - 1) {
      *cnt = 0;
      __threadfence();
    }
    *flag = old == n - 1;
  }
  __syncthreads();
  return *flag != 0;
}

#define F12_BUF(b) ((uint16_t)(slp::F12_NSLOT + 12 * (b)))

// Product of each segment data[g stride + 0 .. len) into data[g stride] in one launch: a
// workgroup per pair of the first level; of two sibling nodes, the workgroup that finishes
// second climbs to the parent (arrival counters as in k_jac_tree).
__global__ void __launch_bounds__(SLP_T, 4) ks_f12_tree(fp12 *data, uint64_t nseg, uint64_t stride, uint64_t len, uint32_t *cnt) {
  CHAIN_PRIORITY();
  __shared__ f29 S[slp::F12_NSLOT + 36];
  __shared__ uint32_t arrived;
  __shared__ slp::Call calls_sh[1];
  CtxInline cx{S, calls_sh};
  uint64_t per = (len + 1) / 2;
  uint64_t id = blockIdx.x;
  if (id >= nseg * per) return;
  uint64_t g = id / per, q = id % per;
  fp12 *seg = data + g * stride;
  uint32_t *c = cnt + g * tree_counters(len);
  const int t = threadIdx.x;
  uint64_t s = 1, n = per, cb = 0;
  for (;;) {
    uint64_t a = 2 * s * q, b = a + s;
    if (b < len) {
      fe *da = reinterpret_cast<fe *>(seg + a);
      const fe *db = reinterpret_cast<const fe *>(seg + b);
      if (t < 12) {
        S[slp::F12_NSLOT + t] = slp::to29(da[t]);
        S[slp::F12_NSLOT + 12 + t] = slp::to29(db[t]);
      }
      __syncthreads();
      cx.run(slp::PROG_F12_MUL, F12_BUF(0), F12_BUF(1), F12_BUF(2));
      if (t < 12) da[t] = slp::from29(slp::canon29(S[slp::F12_NSLOT + 24 + t]));
    }
    if (n == 1) return;
    uint64_t nn = (n + 1) / 2, qp = q >> 1;
    if ((q ^ 1) < n) {
      if (!last_arrival(&c[cb + qp], 2, &arrived)) return;
    }
    cb += nn;
    q = qp;
    n = nn;
    s *= 2;
  }
}

// Final exponentiation of one F_p12 element: the norm, one inversion in F_p and the rest, on
// four wavefronts (the chain of squarings is a product level each, and the products gathered
// beside it fill the other lanes: 274 levels on four wavefronts, some 350 on two).
__device__ __forceinline__ void fe_job(const fp12 *in, fp12 *out) {
  __shared__ f29 S[slp::FE_NSLOT];
  __shared__ slp::Call calls_sh[1];
  slp::DevCtx<slp::FE_WAVES, true> c{S, calls_sh};
  int t = threadIdx.x;
  const fe *src = reinterpret_cast<const fe *>(in);
  if (t < 12) S[slp::FE_X_0 + t] = slp::to29(src[t]);
  load_consts<slp::FE_NCONST, FE_T>(S, slp::FE_CBASE, slp::FE_CONSTS);
#pragma unroll 1
  for (int part = 0; part < 2; part++) {
    c.run(part ? slp::PROG_FE_REST : slp::PROG_FE_NORM, 0, 0, 0);
    if (!part) c.invert(slp::FE_tinv, S[slp::FE_t]);
  }
  fe *dst = reinterpret_cast<fe *>(out);
  if (t < 12) dst[t] = slp::from29(slp::canon29(S[slp::FE_D_0 + t]));
}

// f^((p^12 - 1)/r), a workgroup per input; input s at in[s in_stride], output to
// (s odd ? out1 : out0)[(s >> 1) ostride]
__global__ void __launch_bounds__(FE_T, 4) ks_final_exp(const fp12 *in, uint64_t in_stride, uint64_t n, fp12 *out0, fp12 *out1,
                                                       uint64_t ostride) {
  CHAIN_PRIORITY();
  uint64_t s = blockIdx.x;
  if (s >= n) return;
  fe_job(in + s * in_stride, ((s & 1) ? out1 : out0) + (s >> 1) * ostride);
}

// ---------------------------------------------------------------- G2 scalar multiplications
__device__ __forceinline__ fe out29(const f29 &x) { return slp::from29(slp::canon29(x)); }

// T (homogeneous) to affine coordinates of the twist, zeros for the identity
__device__ void g2_store_aff(Ctx c, g2_aff *oaff) {
  const int t = threadIdx.x;
  fe *o = reinterpret_cast<fe *>(oaff);
  c.run(slp::PROG_G2_NORM, 0, 0, 0);
  if (!c.invert(slp::G2_tinv, c.S[slp::G2_t])) {
    if (t < 4) o[t] = fe_zero();
    return;
  }
  c.run(slp::PROG_G2_AFF, 0, 0, 0);
  if (t < 4) o[t] = out29(c.S[slp::G2_ax_0 + t]);
}
// T as six field elements (homogeneous, on the isomorphic curve), in the place of a g2_jac
__device__ void g2_store_hom(Ctx c, g2_jac *out) {
  const int t = threadIdx.x;
  if (t < 6) reinterpret_cast<fe *>(out)[t] = out29(g2m::coord(c, t));
}

// T += A for an affine A of the twist: its coordinates go to xQ, yQ (whose values are spent)
__device__ void g2_add_affine(Ctx c, const g2_aff *A) {
  if (g2_inf(*A)) return;
  const int t = threadIdx.x;
  if (t < 4) c.S[slp::G2_xQ_0 + t] = slp::to29(reinterpret_cast<const fe *>(A)[t]);
  c.run(slp::PROG_G2_MADD, 0, 0, 0);
}

// T = k Q + A on the engine (A optional).  With lo >= 0 only bits [lo, lo + width) of the GLS
// split of k are applied (gls::chunk).
__device__ void g2_job(Ctx c, gls::Dec *dec, const g2_aff *Q, const fe *k_mont, const g2_aff *A, int lo = -1, int width = 0) {
  const int t = threadIdx.x;
  if (t == 0) {
    fe kc = f_from_mont<FpR>(*k_mont);
    gls::Dec d = gls::decompose(kc.l);
    *dec = lo < 0 ? d : gls::chunk(d, lo, width);
  }
  if (t >= 64 && t < 68) c.S[slp::G2_xQ_0 + t - 64] = slp::to29(reinterpret_cast<const fe *>(Q)[t - 64]);
  load_consts<slp::G2_NCONST>(c.S, slp::G2_CBASE, slp::G2_CONSTS);
  __syncthreads();
  g2m::mul(c, *dec, g2_inf(*Q));
  if (A) g2_add_affine(c, A);
}

// terms q_m h_m of the KZG proof of v_l with every multiplication split in four parts (bits
// [16 p, 16 p + 16) of the GLS split, 17 for p = 3) on the multiples hm[3 m + p - 1] =
// 2^{16 p} h_m made at setup: S2[4 id + p] (homogeneous) for term id = k (2K - 2) + m
__global__ void __launch_bounds__(SLP_T, 4) ks_kzg_terms_split(const g2_aff *h, const g2_aff *hm, const fe *Qc, uint64_t K,
                                                           uint64_t nb, g2_jac *S2) {
  CHAIN_PRIORITY();
  __shared__ f29 S[slp::G2_NSLOT];
  CALL_LIST();
  Ctx c{S, calls_sh};
  __shared__ gls::Dec dec;
  uint64_t n = 2 * K - 2;
  uint64_t id = blockIdx.x;
  if (id >= 4 * nb * n) return;
  uint64_t term = id >> 2, m = term % n;
  int part = (int)(id & 3);
  g2_job(c, &dec, part ? hm + 3 * m + part - 1 : h + m, Qc + term, nullptr, 16 * part, part < 3 ? 16 : 17);
  g2_store_hom(c, S2 + id);
}

// ---------------------------------------------------------------- G_T exponentiation
// out = in^k (k in Montgomery F_r form; kc: 16 words of LDS), square-and-multiply.  The input may be any
// element: one of the cyclotomic subgroup, as every pairing value is (x^{p^4} x = x^{p^2}: two Frobenius
// maps and a product), takes its squarings, half as long as the general ones, and the non-adjacent form of
// k, as its inverse is its conjugate: a power 0.70 ms for 1.03
__device__ void gt_pow_job(Ctx c, const fp12 *in, const fe *k_mont, uint32_t *kc, fp12 *out) {
  f29 *S = c.S;
  const int t = threadIdx.x;
  const fe *src = reinterpret_cast<const fe *>(in);
  if (t < 12) S[F12_BUF(0) + t] = slp::to29(src[t]);
  if (t == 0) {
    fe kcan = f_from_mont<FpR>(*k_mont);
    for (int w = 0; w < 8; w++) kc[w] = kcan.l[w];
  }
  load_consts<slp::F12_NCONST>(S, slp::F12_CBASE, slp::F12_CONSTS);
  __syncthreads();
  c.run(slp::PROG_F12_FROB2, F12_BUF(0), F12_BUF(0), F12_BUF(1));
  c.run(slp::PROG_F12_FROB2, F12_BUF(1), F12_BUF(1), F12_BUF(2));
  c.run(slp::PROG_F12_MUL, F12_BUF(2), F12_BUF(0), F12_BUF(3));
  bool same = true;
  if (t < 12) {
    const f29 x = slp::canon29(S[F12_BUF(1) + t]), y = slp::canon29(S[F12_BUF(3) + t]);
    for (int i = 0; i < 9; i++) same = same && x.l[i] == y.l[i];
  }
  const bool cyc = __syncthreads_and(same);
  if (cyc) c.run(slp::PROG_F12_CONJ, F12_BUF(0), F12_BUF(0), F12_BUF(3));
  // the digits: +1 where a bit of kc[0 .. 8) is set, -1 of kc[8 .. 16); the non-adjacent form is (3k - k) / 2
  // digit by digit
  if (t == 0) {
    uint32_t h[9], carry = 0;
    for (int w = 0; w < 8; w++) {
      const uint64_t v = 3ull * kc[w] + carry;
      h[w] = (uint32_t)v;
      carry = (uint32_t)(v >> 32);
    }
    h[8] = 0;  // 3 k is below 2^256
    for (int w = 0; w < 8; w++) {
      const uint32_t k0 = kc[w], k1 = w < 7 ? kc[w + 1] : 0, p0 = h[w] & ~k0, p1 = h[w + 1] & ~k1, n0 = k0 & ~h[w], n1 = k1 & ~h[w + 1];
      kc[8 + w] = cyc ? n0 >> 1 | n1 << 31 : 0;
      if (cyc) kc[w] = p0 >> 1 | p1 << 31;
    }
  }
  __syncthreads();
  int top = -1;
  for (int b = 255; b >= 0; b--)
    if ((kc[b >> 5] >> (b & 31)) & 1) { top = b; break; }
  fe *dst = reinterpret_cast<fe *>(out);
  if (top < 0) {
    if (t < 12) dst[t] = t == 0 ? f_one<FpP>() : fe_zero();
    return;
  }
  const int sqr = cyc ? slp::PROG_F12_CSQR : slp::PROG_F12_SQR, sqr_mul = cyc ? slp::PROG_F12_CSQR_MUL : slp::PROG_F12_SQR_MUL;
  // a call per bit below the top one (a squaring, with a product where the digit is not zero),
  // the accumulator alternating between buffers 1 and 2; buffer 0 holds the base, 3 its conjugate
#pragma unroll 1
  for (int first = 0; first < top; first += slp::MAX_CALLS) {
    const int n = top - first < slp::MAX_CALLS ? top - first : slp::MAX_CALLS;
    for (int e = t; e < n; e += SLP_T) {
      const int i = first + e, bit = top - 1 - i, src = i == 0 ? 0 : 2 - (i & 1), dst = 1 + (i & 1);
      const bool one = kc[bit >> 5] >> (bit & 31) & 1, minus = kc[8 + (bit >> 5)] >> (bit & 31) & 1;
      c.cl[e] = one || minus ? slp::call(sqr_mul, F12_BUF(src), F12_BUF(minus ? 3 : 0), F12_BUF(dst))
                    : slp::call(sqr, F12_BUF(src), F12_BUF(src), F12_BUF(dst));
    }
    c.run_list(0, n);
  }
  const int acc = top == 0 ? 0 : 2 - (top & 1);
  if (t < 12) dst[t] = slp::from29(slp::canon29(S[F12_BUF(acc) + t]));
}

// ---------------------------------------------------------------- G1 scalar multiplications
// T (homogeneous) to affine, zeros for the identity
__device__ void g1_store_aff(Ctx c, g1_aff *oaff) {
  const int t = threadIdx.x;
  fe *o = reinterpret_cast<fe *>(oaff);
  if (!c.invert(slp::G1_tinv, g1m::coord(c, 2))) {
    if (t < 2) o[t] = fe_zero();
    return;
  }
  c.run(slp::PROG_G1_AFF, 0, 0, 0);
  if (t < 2) o[t] = out29(c.S[t ? slp::G1_ay : slp::G1_ax]);
}
// T as three field elements (homogeneous), in the place of a g1_jac
__device__ void g1_store_hom(Ctx c, g1_jac *out) {
  const int t = threadIdx.x;
  if (t < 3) reinterpret_cast<fe *>(out)[t] = out29(g1m::coord(c, t));
}

// T = k P + A on the engine (A optional).  With chunk >= 0 only that 32-bit part of the GLV split
// of k is applied (glv::chunk).
__device__ void g1_job(Ctx c, glv::Dec *dec, const g1_aff *P, const fe *k_mont, const g1_aff *A, int chunk = -1) {
  const int t = threadIdx.x;
  if (t == 0) {
    fe kc = f_from_mont<FpR>(*k_mont);
    glv::Dec d = glv::decompose(kc.l);
    *dec = chunk < 0 ? d : glv::chunk(d, chunk);
  }
  if (t >= 64 && t < 66) c.S[slp::G1_xP + t - 64] = slp::to29(t == 65 ? P->y : P->x);
  load_consts<slp::G1_NCONST>(c.S, slp::G1_CBASE, slp::G1_CONSTS);
  __syncthreads();
  g1m::mul(c, *dec, g1_inf(*P));
  if (A && !g1_inf(*A)) g1m::add_affine(c, slp::to29(A->x), slp::to29(A->y));
}

// out[i] = k_i P_i, affine, a workgroup per point
__global__ void __launch_bounds__(SLP_T, 4) ks_g1_mul(const g1_aff *P, const fe *k, uint64_t n, g1_aff *out) {
  __shared__ f29 S[slp::G1_NSLOT];
  CALL_LIST();
  __shared__ glv::Dec dec;
  Ctx c{S, calls_sh};
  const uint64_t i = blockIdx.x;
  if (i >= n) return;
  g1_job(c, &dec, P + i, k + i, nullptr);
  g1_store_aff(c, out + i);
}

// The powers and multiples of a verification in one launch, a workgroup each: X[i]^{kx_i} of n3
// elements of F_p12, k_i Q on G2 of n2 scalars (one base), k_i P_i on G1 of n1 points, the longest
// first.  At 2^16 entries in batches of 256 (16, 1 and 276 of them) 0.71 ms, the time of a power;
// one after another, the multiples with 8 lanes a field element, they took 1.0 + 3.2 + 1.5 ms.
__global__ void __launch_bounds__(SLP_T, 4) ks_mults(const fp12 *X, const fe *kx, uint64_t n3, fp12 *outx, const g2_aff *Q,
                                                     const fe *kq, uint64_t n2, g2_aff *outq, const g1_aff *P, const fe *kp,
                                                     uint64_t n1, g1_aff *outp) {
  __shared__ f29 S[most(slp::G1_NSLOT, slp::G2_NSLOT, slp::F12_NSLOT + 48)];
  CALL_LIST();
  __shared__ glv::Dec d1;
  __shared__ gls::Dec d2;
  __shared__ uint32_t kc[16];
  Ctx c{S, calls_sh};
  uint64_t i = blockIdx.x;
  if (i < n3) {
    gt_pow_job(c, X + i, kx + i, kc, outx + i);
  } else if ((i -= n3) < n2) {
    g2_job(c, &d2, Q, kq + i, nullptr);
    g2_store_aff(c, outq + i);
  } else if ((i -= n2) < n1) {
    g1_job(c, &d1, P + i, kp + i, nullptr);
    g1_store_aff(c, outp + i);
  }
}

// ---------------------------------------------------------------- group sums on the engine
// Sum of each segment data[g stride + 0 .. len) of points into data[g stride] in one launch: a
// workgroup per pair of the first level; of two sibling nodes, the workgroup that finishes
// second climbs to the parent (arrival counters as in ks_f12_tree).  HOM: homogeneous points of
// the engine's multiplications (G1, or G2 on the isomorphic curve), an addition two levels and
// never exceptional; otherwise Jacobian G2 points of the twist (the MSM's), the identity any
// point with Z = 0.
template <bool G2, bool HOM>
__global__ void __launch_bounds__(SLP_T, 4) ks_pt_tree(void *data, uint64_t nseg, uint64_t stride, uint64_t len, uint32_t *cnt) {
  if (G2) CHAIN_PRIORITY();
  else AHEAD_PRIORITY();
  constexpr int NC = G2 ? 6 : 3;  // coordinates (F_p elements) per point
  __shared__ f29 S[!G2 ? slp::G1_ADD_SLOTS : HOM ? slp::G2_ADD_SLOTS : most(slp::G2_JADD_SLOTS, slp::G2_JDBL_SLOTS)];
  __shared__ slp::Call calls_sh[HOM ? 1 : slp::MAX_CALLS + 1];
  slp::DevCtx<SLP_W, HOM> cx{S, calls_sh};
  __shared__ uint32_t arrived;
  uint64_t per = (len + 1) / 2;
  uint64_t id = blockIdx.x;
  if (id >= nseg * per) return;
  uint64_t g = id / per, q = id % per;
  fe *seg = reinterpret_cast<fe *>(data) + g * stride * NC;
  uint32_t *c = cnt + g * tree_counters(len);
  const int t = threadIdx.x;
  const int A0 = G2 ? slp::G2_TB1_0 : slp::G1_TB1_0, B0 = A0 + NC;
  if (G2) load_consts<slp::G2_NCONST>(S, slp::G2_CBASE, slp::G2_CONSTS);
  else load_consts<slp::G1_NCONST>(S, slp::G1_CBASE, slp::G1_CONSTS);
  uint64_t s = 1, n = per, cb = 0;
  for (;;) {
    uint64_t a = 2 * s * q, b = a + s;
    if (b < len) {
      fe *da = seg + a * NC;
      const fe *db = seg + b * NC;
      if (HOM) {
        if (t < 2 * NC) S[A0 + t] = slp::to29(t < NC ? da[t] : db[t - NC]);
        __syncthreads();
        if constexpr (G2) {
          g2m::load(cx, A0);
          cx.run(slp::PROG_G2_ADD, 0, B0, 0);
          if (t < NC) da[t] = out29(g2m::coord(cx, t));
        } else {
          g1m::load(cx, A0);
          cx.run(slp::PROG_G1_ADD, 0, B0, 0);
          if (t < NC) da[t] = out29(g1m::coord(cx, t));
        }
      } else if (!(fe_is_zero(db[4]) && fe_is_zero(db[5]))) {
        bool inf = fe_is_zero(da[4]) && fe_is_zero(da[5]);
        if (t < NC) {
          S[slp::G2_J_0 + t] = slp::to29(da[t]);
          S[A0 + t] = slp::to29(db[t]);
        }
        __syncthreads();
        g2m::add_jac(cx, inf, A0, false);
        if (t < NC) da[t] = inf ? ((t == 0 || t == 2) ? f_one<FpP>() : fe_zero()) : out29(S[slp::G2_J_0 + t]);
      }
    }
    if (n == 1) return;
    uint64_t nn = (n + 1) / 2, qp = q >> 1;
    if ((q ^ 1) < n) {
      if (!last_arrival(&c[cb + qp], 2, &arrived)) return;
    }
    cb += nn;
    q = qp;
    n = nn;
    s *= 2;
  }
}

// (i odd ? out1 : out0)[(i >> 1) ostride] = the homogeneous point in[i stride] in affine
// coordinates, a workgroup per point
template <bool G2>
__global__ void __launch_bounds__(SLP_T, 4) ks_hom_to_aff(const void *in, uint64_t stride, uint64_t n, void *out0, void *out1,
                                                         uint64_t ostride) {
  CHAIN_PRIORITY();
  constexpr int NC = G2 ? 6 : 3;
  __shared__ f29 S[G2 ? G2_AFF_ALL_SLOTS : slp::G1_AFF_SLOTS];
  CALL_LIST();
  Ctx c{S, calls_sh};
  const uint64_t i = blockIdx.x;
  if (i >= n) return;
  const int t = threadIdx.x, A0 = G2 ? slp::G2_TB1_0 : slp::G1_TB1_0;
  if (t < NC) S[A0 + t] = slp::to29((reinterpret_cast<const fe *>(in) + i * stride * NC)[t]);
  void *out = i & 1 ? out1 : out0;
  if (G2) {
    load_consts<slp::G2_NCONST>(S, slp::G2_CBASE, slp::G2_CONSTS);
    __syncthreads();
    g2m::load(c, A0);
    g2_store_aff(c, reinterpret_cast<g2_aff *>(out) + (i >> 1) * ostride);
  } else {
    load_consts<slp::G1_NCONST>(S, slp::G1_CBASE, slp::G1_CONSTS);
    __syncthreads();
    g1m::load(c, A0);
    g1_store_aff(c, reinterpret_cast<g1_aff *>(out) + (i >> 1) * ostride);
  }
}

// ---------------------------------------------------------------- Step 1 rounds, fused
// Round-1 (direct) G1 terms on the engine: b_L[i] A_R[i] (side 0) and b_R[i] A_L[i] (side 1)
// into S[(2k + side) (K / 2) + i] (homogeneous)
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_g1terms(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t h,
                                                      g1_jac *Sout) {
  AHEAD_PRIORITY();
  __shared__ f29 S[slp::G1_NSLOT];
  CALL_LIST();
  Ctx c{S, calls_sh};
  __shared__ glv::Dec d1;
  uint64_t id = blockIdx.x;
  if (id >= nb * 2 * h) return;
  uint64_t k = id / (2 * h), r = id % (2 * h), side = r / h, i = r % h;
  g1_job(c, &d1, A + (side ? k * K + i : k * K + h + i), B + (side ? k * K + h + i : k * K + i), nullptr);
  g1_store_hom(c, Sout + (k * 2 + side) * (K / 2) + i);
}

template <int A_, int B_> struct imax { static constexpr int v = A_ > B_ ? A_ : B_; };

// The fold of round j (Eq. folding) for every batch: blocks [0, nb h) fold G1 and b,
// blocks [nb h, 2 nb h) fold G2.  Aout[i] = Ain[i] + x Ain[h + i], Bout[i] = Bin[i] +
// x^{-1} Bin[h + i], Vout[i] = Vin[i] + x^{-1} Vin[h + i].
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_fold(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout, const g2_aff *Vin,
                                                   g2_aff *Vout, const fe *X, const fe *Xinv, uint64_t K, uint64_t nb,
                                                   uint64_t h, uint32_t j, uint32_t lK) {
  CHAIN_PRIORITY();
  __shared__ f29 S[imax<slp::G1_NSLOT, slp::G2_NSLOT>::v];
  CALL_LIST();
  Ctx c{S, calls_sh};
  __shared__ glv::Dec d1;
  __shared__ gls::Dec d2;
  uint64_t id = blockIdx.x;
  if (id >= 2 * nb * h) return;
  bool g2 = id >= nb * h;
  if (g2) id -= nb * h;
  uint64_t k = id / h, i = id % h, slot = k * lK + (j - 1);
  if (g2) {
    g2_job(c, &d2, Vin + k * K + h + i, Xinv + slot, Vin + k * K + i);
    g2_store_aff(c, Vout + k * K + i);
    return;
  }
  if (threadIdx.x == 32) Bout[k * K + i] = fr_add(Bin[k * K + i], fr_mul(Bin[k * K + h + i], Xinv[slot]));
  g1_job(c, &d1, Ain + k * K + h + i, X + slot, Ain + k * K + i);
  g1_store_aff(c, Aout + k * K + i);
}

// The next round's terms (oa_terms.hpp): the Miller loops into F[out], a workgroup per term
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_pterms(const g1_aff *A, const g2_aff *V, uint64_t K, uint64_t nb, uint64_t q,
                                                     fp12 *F) {
  CHAIN_PRIORITY();
  __shared__ f29 S[slp::ML_NSLOT];
  __shared__ slp::Call calls_sh[1];
  uint64_t id = blockIdx.x;
  if (id >= nb * 8 * q) return;
  oat::Term tm = oat::term(id, K, nb, q);
  miller_one(CtxInline{S, calls_sh}, A + tm.a, V + tm.v, F + tm.out);
}

// The G1 terms b[v] A[a] of the next round into S1[out] (homogeneous), a workgroup per term
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_g1terms_next(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t q,
                                                           g1_jac *S1) {
  AHEAD_PRIORITY();
  __shared__ f29 S[slp::G1_NSLOT];
  CALL_LIST();
  Ctx c{S, calls_sh};
  __shared__ glv::Dec d1;
  uint64_t id = blockIdx.x;
  if (id >= nb * 8 * q) return;
  oat::Term tm = oat::term(id, K, nb, q);
  g1_job(c, &d1, A + tm.a, B + tm.v, nullptr);
  g1_store_hom(c, S1 + tm.out);
}

// ---------------------------------------------------------------- cyclotomic G_T powers
#define GTP_SLOTS (slp::F12_NSLOT + 12 * gtp::NBUF)

// ---------------------------------------------------------------- split multiplications
// Multiples for the time-split multiplications: M[3 s + m - 1] = G[s]^{2^{16 m}} (cyclotomic
// squarings), a workgroup per (s, m), m = 1, 2, 3
__global__ void __launch_bounds__(SLP_T, 4) ks_gt_sqr_mults(const fp12 *G, uint64_t n, fp12 *M) {
  CHAIN_PRIORITY();
  __shared__ f29 S[slp::F12_NSLOT + 24];
  CALL_LIST();
  CtxInline c{S, calls_sh};
  uint64_t id = blockIdx.x;
  if (id >= 3 * n) return;
  uint64_t s = id / 3, m = id % 3 + 1;
  const int t = threadIdx.x;
  const fe *src = reinterpret_cast<const fe *>(G + s);
  if (t < 12) S[F12_BUF(0) + t] = slp::to29(src[t]);
  load_consts<slp::F12_NCONST>(S, slp::F12_CBASE, slp::F12_CONSTS);
  __syncthreads();
  for (int e = t; e < 16 * (int)m; e += SLP_T)
    c.cl[e] = slp::call(slp::PROG_F12_CSQR, F12_BUF(e & 1), F12_BUF(e & 1), F12_BUF(1 - (e & 1)));
  c.run_list(0, 16 * (int)m);  // an even number of squarings: the result is in buffer 0
  fe *dst = reinterpret_cast<fe *>(M + 3 * s + m - 1);
  if (t < 12) dst[t] = slp::from29(slp::canon29(S[F12_BUF(0) + t]));
}

// point s of a segmented list: P[(s / seg) segstride + s % seg]
__device__ __forceinline__ uint64_t seg_index(uint64_t s, uint64_t seg, uint64_t segstride) {
  return (s / seg) * segstride + s % seg;
}

// prog n times on the same slots
__device__ void repeat(Ctx c, int prog, int n) {
  for (int e = threadIdx.x; e < n; e += SLP_T) c.cl[e] = slp::call(prog);
  c.run_list(0, n);
}

// 2^{32 m} P (affine) by 16 m double doublings on the engine
__device__ void g1_dbl_mult(Ctx c, const g1_aff *P, int m, g1_aff *o) {
  const int t = threadIdx.x;
  load_consts<slp::G1_NCONST>(c.S, slp::G1_CBASE, slp::G1_CONSTS);
  if (t >= 64 && t < 67) c.S[slp::G1_TB1_0 + t - 64] = slp::to29(t == 66 ? f_one<FpP>() : t == 65 ? P->y : P->x);
  __syncthreads();
  if (g1_inf(*P)) g1m::load_identity(c);
  else g1m::load(c, slp::G1_TB1_0);
  repeat(c, slp::PROG_G1_DBL2, 16 * m);
  g1_store_aff(c, o);
}

// 2^{16 m} Q (affine) by 16 m doublings on the engine
__device__ void g2_dbl_mult(Ctx c, const g2_aff *Q, int m, g2_aff *o) {
  const int t = threadIdx.x;
  load_consts<slp::G2_NCONST>(c.S, slp::G2_CBASE, slp::G2_CONSTS);
  if (t >= 64 && t < 68) c.S[slp::G2_xQ_0 + t - 64] = slp::to29(reinterpret_cast<const fe *>(Q)[t - 64]);
  __syncthreads();
  if (g2_inf(*Q)) g2m::load_identity(c);
  else c.run(slp::PROG_G2_LOAD, 0, 0, 0);
  repeat(c, slp::PROG_G2_DBL, 16 * m);
  g2_store_aff(c, o);
}

// 2^{32 m} P (affine) for a homogeneous P (m = 0: P itself), on the engine
__device__ void g1_hom_mult_aff(Ctx c, const g1_jac *P, int m, g1_aff *o) {
  const int t = threadIdx.x;
  load_consts<slp::G1_NCONST>(c.S, slp::G1_CBASE, slp::G1_CONSTS);
  if (t >= 64 && t < 67) c.S[slp::G1_TB1_0 + t - 64] = slp::to29(reinterpret_cast<const fe *>(P)[t - 64]);
  __syncthreads();
  g1m::load(c, slp::G1_TB1_0);
  repeat(c, slp::PROG_G1_DBL2, 16 * m);
  g1_store_aff(c, o);
}

// M[3 s + m - 1] = 2^{16 m} Q_s (affine), Q_s as in seg_index, a workgroup per (s, m), m = 1, 2, 3
__global__ void __launch_bounds__(SLP_T, 4) ks_g2_dbl_mults(const g2_aff *Q, uint64_t seg, uint64_t segstride, uint64_t n,
                                                        g2_aff *M) {
  __shared__ f29 S[G2_DBL_ALL_SLOTS];
  CALL_LIST();
  Ctx c{S, calls_sh};
  uint64_t id = blockIdx.x;
  if (id >= 3 * n) return;
  uint64_t s = id / 3, m = id % 3 + 1;
  g2_dbl_mult(c, Q + seg_index(s, seg, segstride), (int)m, M + 3 * s + m - 1);
}

// the multiples of a round's arrays in one launch: blocks [0, 3 n1) M1[3 s + m - 1] =
// 2^{32 m} P_s (G1, P_s at seg_index(s, seg1, segstride)), blocks [3 n1, 3 (n1 + n2))
// M2[3 s + m - 1] = 2^{16 m} Q_s (G2, seg2)
__global__ void __launch_bounds__(SLP_T, 4) ks_fold_mults(const g1_aff *P, uint64_t seg1, uint64_t n1, const g2_aff *Q,
                                                      uint64_t seg2, uint64_t n2, uint64_t segstride, g1_aff *M1,
                                                      g2_aff *M2) {
  CHAIN_PRIORITY();
  __shared__ f29 S[most(G1_DBL_SLOTS, G2_DBL_ALL_SLOTS)];
  CALL_LIST();
  Ctx c{S, calls_sh};
  uint64_t id = blockIdx.x;
  if (id >= 3 * (n1 + n2)) return;
  bool g2 = id >= 3 * n1;
  if (g2) id -= 3 * n1;
  uint64_t s = id / 3, m = id % 3 + 1;
  if (g2) g2_dbl_mult(c, Q + seg_index(s, seg2, segstride), (int)m, M2 + 3 * s + m - 1);
  else g1_dbl_mult(c, P + seg_index(s, seg1, segstride), (int)m, M1 + 3 * s + m - 1);
}

// T = the sum of the four parts at J (homogeneous) and A (affine, optional)
__device__ void g1_sum_parts(Ctx c, const g1_jac *J, const g1_aff *A) {
  const int t = threadIdx.x;
  if (t < 12) c.S[slp::G1_TB1_0 + t] = slp::to29(reinterpret_cast<const fe *>(J)[t]);
  const bool has_a = A && !g1_inf(*A);
  if (has_a && t >= 64 && t < 66) c.S[slp::G1_xP + t - 64] = slp::to29(t == 65 ? A->y : A->x);
  __syncthreads();
  g1m::load(c, slp::G1_TB1_0);
  if (t < 4) c.cl[t] = t < 3 ? slp::call(slp::PROG_G1_ADD, 0, slp::G1_TB1_0 + 3 * (t + 1)) : slp::call(slp::PROG_G1_MADD);
  c.run_list(0, has_a ? 4 : 3);
}

// The fold of round j with every multiplication split in four parts run in parallel (M1
// covers the whole arrays, M1[3 (k 2h + i') + p - 1] for index i' of batch k; M2 the halves,
// M2[3 (k h + i) + p - 1] for V[h + i]):
// blocks [0, 4 nb h): part p of x A[h + i] on the base 2^{32 p} A[h + i] (M1, p > 0) with
// the p-th 32-bit chunk of the GLV split of x into J1[4 s + p]; blocks [4 nb h, 8 nb h):
// part p of x^{-1} V[h + i] on 2^{16 p} V[h + i] (M2) with bits [16 p, 16 p + 16) (17 for
// p = 3) of the GLS split into J2[4 s + p] (s = k h + i).  The last part to finish adds the
// four partial results and A[i] (V[i]) and writes the affine result; part 0 of G1 also
// folds b.  Same results as ks_oa_fold.
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_fold_split(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout,
                                                         const g2_aff *Vin, g2_aff *Vout, const fe *X, const fe *Xinv,
                                                         const g1_aff *M1, const g2_aff *M2, g1_jac *J1, g2_jac *J2,
                                                         uint32_t *cnt, uint64_t K, uint64_t nb, uint64_t h, uint32_t j,
                                                         uint32_t lK) {
  CHAIN_PRIORITY();
  __shared__ f29 S[imax<slp::G1_NSLOT, slp::G2_NSLOT>::v];
  CALL_LIST();
  Ctx c{S, calls_sh};
  __shared__ glv::Dec d1;
  __shared__ gls::Dec d2;
  __shared__ uint32_t flag;
  uint64_t id = blockIdx.x, n = nb * h;
  if (id >= 8 * n) return;
  const int t = threadIdx.x;
  bool g2 = id >= 4 * n;
  if (g2) id -= 4 * n;
  uint64_t s = id >> 2, k = s / h, i = s % h, slot = k * lK + (j - 1);
  int part = (int)(id & 3);
  if (!g2) {
    if (part == 0 && t == 32) Bout[k * K + i] = fr_add(Bin[k * K + i], fr_mul(Bin[k * K + h + i], Xinv[slot]));
    g1_job(c, &d1, part ? M1 + 3 * (k * 2 * h + h + i) + part - 1 : Ain + k * K + h + i, X + slot, nullptr, part);
    g1_store_hom(c, J1 + 4 * s + part);
    if (!last_arrival(cnt + s, 4, &flag)) return;
    g1_sum_parts(c, J1 + 4 * s, Ain + k * K + i);
    g1_store_aff(c, Aout + k * K + i);
    return;
  }
  g2_job(c, &d2, part ? M2 + 3 * s + part - 1 : Vin + k * K + h + i, Xinv + slot, nullptr, 16 * part, part < 3 ? 16 : 17);
  g2_store_hom(c, J2 + 4 * s + part);
  if (!last_arrival(cnt + n + s, 4, &flag)) return;
  // sum of the parts (in the table slots) and V[i]
  if (t < 24) S[slp::G2_TB1_0 + t] = slp::to29(reinterpret_cast<const fe *>(J2 + 4 * s)[t]);
  __syncthreads();
  g2m::load(c, slp::G2_TB1_0);
  if (t < 3) c.cl[t] = slp::call(slp::PROG_G2_ADD, 0, slp::G2_TB1_0 + 6 * (t + 1));
  c.run_list(0, 3);
  g2_add_affine(c, Vin + k * K + i);
  g2_store_aff(c, Vout + k * K + i);
}

// The G1 terms b[v] A[a] of the next round (oa_terms.hpp, arrays of length 4q) with each
// multiplication split in four parts: part p on the multiple M[3 (k 4q + a') + p - 1] =
// 2^{32 p} A[k K + a'] (p > 0) with the p-th 32-bit chunk of the GLV split of b[v], into
// J[4 term + p]; the last part to finish writes the sum to S1[out] (homogeneous)
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_g1terms_split(const g1_aff *A, const fe *B, const g1_aff *M, uint64_t K,
                                                            uint64_t nb, uint64_t q, g1_jac *J, uint32_t *cnt, g1_jac *S1) {
  AHEAD_PRIORITY();
  __shared__ f29 S[slp::G1_NSLOT];
  CALL_LIST();
  Ctx c{S, calls_sh};
  __shared__ glv::Dec d1;
  __shared__ uint32_t flag;
  uint64_t id = blockIdx.x;
  if (id >= 4 * nb * 8 * q) return;
  uint64_t term = id >> 2, k = term / (8 * q);
  int part = (int)(id & 3);
  oat::Term tm = oat::term(term, K, nb, q);
  g1_job(c, &d1, part ? M + 3 * (k * 4 * q + (tm.a - k * K)) + part - 1 : A + tm.a, B + tm.v, nullptr, part);
  g1_store_hom(c, J + 4 * term + part);
  if (!last_arrival(cnt + term, 4, &flag)) return;
  g1_sum_parts(c, J + 4 * term, nullptr);
  g1_store_hom(c, S1 + tm.out);
}

// The x-dependent part of a round taken ahead, each multiplication split in four parts run
// in parallel: for s < 4 nb and part p < 4, k_s = (s odd ? k_odd : k_even)[(s >> 2) kstride];
// blocks [0, 16 nb): PE[4 s + p] = (PX[s]^{2^{16 p}})^{chunk_p}, the Frobenius split of k_s
// restricted to bits [16 p, 16 p + 16) (17 bits for p = 3); blocks [16 nb, 32 nb):
// PM[4 s + p] = chunk_p(k_s) (2^{32 p} PX1[s]) (homogeneous).  Multiples come from
// ks_gt_sqr_mults and ks_g1_dbl_mults (PXm, PX1m).
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_combine_split(const fp12 *PX, const fp12 *PXm, const g1_aff *PX1,
                                                            const g1_aff *PX1m, const fe *k_even, const fe *k_odd,
                                                            uint64_t kstride, uint64_t nb, fp12 *PE, g1_jac *PM) {
  CHAIN_PRIORITY();
  __shared__ f29 S[imax<GTP_SLOTS, slp::G1_NSLOT>::v];
  CALL_LIST();
  Ctx c{S, calls_sh};
  __shared__ gls::Dec dec;
  __shared__ glv::Dec d1;
  uint64_t id = blockIdx.x;
  if (id >= 32 * nb) return;
  const int t = threadIdx.x;
  bool g1 = id >= 16 * nb;
  if (g1) id -= 16 * nb;
  uint64_t s = id >> 2;
  int part = (int)(id & 3);
  const fe *k = (s & 1 ? k_odd : k_even) + (s >> 2) * kstride;
  if (g1) {
    g1_job(c, &d1, part ? PX1m + 3 * s + part - 1 : PX1 + s, k, nullptr, part);
    g1_store_hom(c, PM + 4 * s + part);
    return;
  }
  if (t == 0) {
    fe kc = f_from_mont<FpR>(*k);
    dec = gls::chunk(gls::decompose(kc.l), 16 * part, part < 3 ? 16 : 17);
  }
  const fe *src = reinterpret_cast<const fe *>(part ? PXm + 3 * s + part - 1 : PX + s);
  if (t < 12) S[F12_BUF(0) + t] = slp::to29(src[t]);
  load_consts<slp::F12_NCONST>(S, slp::F12_CBASE, slp::F12_CONSTS);
  __syncthreads();
  int r = gtp::pow_cyc(c, dec, slp::F12_NSLOT);
  fe *dst = reinterpret_cast<fe *>(PE + 4 * s + part);
  if (t < 12) dst[t] = r < 0 ? (t == 0 ? f_one<FpP>() : fe_zero()) : slp::from29(slp::canon29(S[F12_BUF(r) + t]));
}

// Both parts of L_j, R_j from the combine, in one launch.  Blocks [0, 2 nb):
// (side ? R : L)[k lK] = U[2k + side] prod_{g in {2 side, 2 side + 1}, p < 4} P[4 (4k + g) + p]
// (G_T); blocks [2 nb, 4 nb): the G1 parts U1[2k + side] + sum of the 8 homogeneous parts
// P1[4 (4k + 2 side) + i], affine, into L1 / R1.  (The G1 side as Jacobian sums on single lanes
// with a per-lane inversion held the launch at 0.19 ms.)
__global__ void __launch_bounds__(SLP_T, 4) ks_oa_combine8(const fp12 *U, const fp12 *P, const g1_aff *U1, const g1_jac *P1,
                                                       uint64_t nb, fp12 *L, fp12 *R, g1_aff *L1, g1_aff *R1, uint64_t lK) {
  CHAIN_PRIORITY();
  __shared__ f29 S[imax<slp::F12_NSLOT + 12 * 11, slp::G1_NSLOT>::v];
  CALL_LIST();
  Ctx c{S, calls_sh};
  uint64_t id = blockIdx.x;
  if (id >= 4 * nb) return;
  const int t = threadIdx.x;
  const bool g1 = id >= 2 * nb;
  if (g1) id -= 2 * nb;
  const uint64_t k = id / 2, side = id % 2;
  if (g1) {
    // the 8 parts in table slots, U1 in xP, yP
    const fe *p = reinterpret_cast<const fe *>(P1 + 4 * (4 * k + 2 * side));
    if (t < 24) S[slp::G1_TB1_0 + t] = slp::to29(p[t]);
    const bool has_u = !g1_inf(U1[id]);
    if (has_u && t >= 64 && t < 66) S[slp::G1_xP + t - 64] = slp::to29(t == 65 ? U1[id].y : U1[id].x);
    load_consts<slp::G1_NCONST>(S, slp::G1_CBASE, slp::G1_CONSTS);
    __syncthreads();
    g1m::load(c, slp::G1_TB1_0);
    if (t < 8) c.cl[t] = t < 7 ? slp::call(slp::PROG_G1_ADD, 0, slp::G1_TB1_0 + 3 * (t + 1)) : slp::call(slp::PROG_G1_MADD);
    c.run_list(0, has_u ? 8 : 7);
    g1_store_aff(c, (side ? R1 : L1) + k * lK);
    return;
  }
  // buffers 0 and 1 the product (alternating, U first), 2..9 the powers
  const fe *u = reinterpret_cast<const fe *>(U + id), *pp = reinterpret_cast<const fe *>(P + 4 * (4 * k + 2 * side));
  for (int i = t; i < 12 * 9; i += SLP_T) S[i < 12 ? F12_BUF(0) + i : F12_BUF(1) + i] = slp::to29(i < 12 ? u[i] : pp[i - 12]);
  load_consts<slp::F12_NCONST>(S, slp::F12_CBASE, slp::F12_CONSTS);
  if (t < 8) c.cl[t] = slp::call(slp::PROG_F12_MUL, F12_BUF(t & 1), F12_BUF(2 + t), F12_BUF(1 - (t & 1)));
  c.run_list(0, 8);
  fe *dst = reinterpret_cast<fe *>((side ? R : L) + k * lK);
  if (t < 12) dst[t] = slp::from29(slp::canon29(S[F12_BUF(0) + t]));
}

// final exponentiations of two strided lists: job s < n0 takes in0[s st0] to out0[s], the
// others in1[(s - n0) st1] to out1[s - n0]
__global__ void __launch_bounds__(FE_T, 4) ks_final_exp2(const fp12 *in0, uint64_t st0, uint64_t n0, fp12 *out0,
                                                        const fp12 *in1, uint64_t st1, uint64_t n1, fp12 *out1) {
  CHAIN_PRIORITY();
  uint64_t s = blockIdx.x;
  if (s >= n0 + n1) return;
  fe_job(s < n0 ? in0 + s * st0 : in1 + (s - n0) * st1, s < n0 ? out0 + s : out1 + (s - n0));
}

// The reduced G1 groups of the terms taken ahead (oa_terms.hpp, segment sums in PS) made
// ready for the combine: blocks [0, 2 nb): U group (2k + side) to PU1 (affine); blocks
// [2 nb, 18 nb): XY group s = 4k + g as PX1[s] (affine, m = 0) and PX1m[3 s + m - 1] =
// 2^{32 m} PX1[s] (m = 1..3)
__global__ void __launch_bounds__(SLP_T, 4) ks_g1_finish(const g1_jac *PS, uint64_t nb, uint64_t q, g1_aff *PU1, g1_aff *PX1,
                                                     g1_aff *PX1m) {
  AHEAD_PRIORITY();
  __shared__ f29 S[G1_DBL_SLOTS];
  CALL_LIST();
  Ctx c{S, calls_sh};
  uint64_t id = blockIdx.x;
  if (id >= 18 * nb) return;
  if (id < 2 * nb) {
    g1_hom_mult_aff(c, PS + id * 2 * q, 0, PU1 + id);
    return;
  }
  id -= 2 * nb;
  uint64_t s = id >> 2;
  int m = (int)(id & 3);
  g1_hom_mult_aff(c, PS + nb * 4 * q + s * q, m, m ? PX1m + 3 * s + m - 1 : PX1 + s);
}

namespace ks {
void miller(const g1_aff *P, uint64_t sp, const g2_aff *Q, uint64_t sq, uint64_t n, fp12 *out, hipStream_t st) {
  if (n) LAUNCH(ks_miller, dim3((unsigned)n), dim3(SLP_T), 0, P, sp, Q, sq, n, out);
}
void oa_miller(const g1_aff *A, const g2_aff *V, uint64_t K, uint64_t nb, uint64_t h, fp12 *F, hipStream_t st) {
  LAUNCH(ks_oa_miller, dim3((unsigned)(nb * 2 * h)), dim3(SLP_T), 0, A, V, K, nb, h, F);
}
void f12_reduce(fp12 *data, uint64_t nseg, uint64_t stride, uint64_t len, uint32_t *cnt, hipStream_t st) {
  if (len > 1) LAUNCH(ks_f12_tree, dim3((unsigned)(nseg * ((len + 1) / 2))), dim3(SLP_T), 0, data, nseg, stride, len, cnt);
}
void final_exp(const fp12 *in, uint64_t stride, uint64_t n, fp12 *out0, fp12 *out1, uint64_t ostride, hipStream_t st) {
  if (!out1) {  // every output to out0[s ostride]
    out1 = out0 + ostride;
    ostride *= 2;
  }
  if (n) LAUNCH(ks_final_exp, dim3((unsigned)n), dim3(FE_T), 0, in, stride, n, out0, out1, ostride);
}
void oa_fold(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout, const g2_aff *Vin, g2_aff *Vout, const fe *X,
             const fe *Xinv, uint64_t K, uint64_t nb, uint64_t h, uint32_t j, uint32_t lK, hipStream_t st) {
  LAUNCH(ks_oa_fold, dim3((unsigned)(2 * nb * h)), dim3(SLP_T), 0, Ain, Bin, Aout, Bout, Vin, Vout, X, Xinv, K, nb, h, j, lK);
}
void oa_pterms(const g1_aff *A, const g2_aff *V, uint64_t K, uint64_t nb, uint64_t q, fp12 *F, hipStream_t st) {
  LAUNCH(ks_oa_pterms, dim3((unsigned)(nb * 8 * q)), dim3(SLP_T), 0, A, V, K, nb, q, F);
}
void gt_sqr_mults(const fp12 *G, uint64_t n, fp12 *M, hipStream_t st) {
  if (n) LAUNCH(ks_gt_sqr_mults, dim3((unsigned)(3 * n)), dim3(SLP_T), 0, G, n, M);
}
void g1_finish(const g1_jac *PS, uint64_t nb, uint64_t q, g1_aff *PU1, g1_aff *PX1, g1_aff *PX1m, hipStream_t st) {
  LAUNCH(ks_g1_finish, dim3((unsigned)(18 * nb)), dim3(SLP_T), 0, PS, nb, q, PU1, PX1, PX1m);
}
void oa_g1terms_next(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t q, g1_jac *S1, hipStream_t st) {
  LAUNCH(ks_oa_g1terms_next, dim3((unsigned)(nb * 8 * q)), dim3(SLP_T), 0, A, B, K, nb, q, S1);
}
void oa_g1terms_split(const g1_aff *A, const fe *B, const g1_aff *M, uint64_t K, uint64_t nb, uint64_t q, g1_jac *J,
                      uint32_t *cnt, g1_jac *S1, hipStream_t st) {
  LAUNCH(ks_oa_g1terms_split, dim3((unsigned)(4 * nb * 8 * q)), dim3(SLP_T), 0, A, B, M, K, nb, q, J, cnt, S1);
}
void fold_mults(const g1_aff *P, uint64_t seg1, uint64_t n1, const g2_aff *Q, uint64_t seg2, uint64_t n2, uint64_t segstride,
                g1_aff *M1, g2_aff *M2, hipStream_t st) {
  if (n1 + n2)
    LAUNCH(ks_fold_mults, dim3((unsigned)(3 * (n1 + n2))), dim3(SLP_T), 0, P, seg1, n1, Q, seg2, n2, segstride, M1, M2);
}
void oa_fold_split(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout, const g2_aff *Vin, g2_aff *Vout, const fe *X,
                   const fe *Xinv, const g1_aff *M1, const g2_aff *M2, g1_jac *J1, g2_jac *J2, uint32_t *cnt, uint64_t K,
                   uint64_t nb, uint64_t h, uint32_t j, uint32_t lK, hipStream_t st) {
  LAUNCH(ks_oa_fold_split, dim3((unsigned)(8 * nb * h)), dim3(SLP_T), 0, Ain, Bin, Aout, Bout, Vin, Vout, X, Xinv, M1, M2, J1,
         J2, cnt, K, nb, h, j, lK);
}
void oa_combine_split(const fp12 *PX, const fp12 *PXm, const g1_aff *PX1, const g1_aff *PX1m, const fe *k_even,
                      const fe *k_odd, uint64_t kstride, uint64_t nb, fp12 *PE, g1_jac *PM, hipStream_t st) {
  LAUNCH(ks_oa_combine_split, dim3((unsigned)(32 * nb)), dim3(SLP_T), 0, PX, PXm, PX1, PX1m, k_even, k_odd, kstride, nb, PE,
         PM);
}
void oa_combine8(const fp12 *U, const fp12 *P, const g1_aff *U1, const g1_jac *P1, uint64_t nb, fp12 *L, fp12 *R, g1_aff *L1,
                 g1_aff *R1, uint64_t lK, hipStream_t st) {
  LAUNCH(ks_oa_combine8, dim3((unsigned)(4 * nb)), dim3(SLP_T), 0, U, P, U1, P1, nb, L, R, L1, R1, lK);
}
void final_exp2(const fp12 *in0, uint64_t st0, uint64_t n0, fp12 *out0, const fp12 *in1, uint64_t st1, uint64_t n1, fp12 *out1,
                hipStream_t st) {
  if (n0 + n1) LAUNCH(ks_final_exp2, dim3((unsigned)(n0 + n1)), dim3(FE_T), 0, in0, st0, n0, out0, in1, st1, n1, out1);
}
void g1_tree(g1_jac *data, uint64_t nseg, uint64_t stride, uint64_t len, uint32_t *cnt, hipStream_t st) {
  if (len > 1) LAUNCH((ks_pt_tree<false, true>), dim3((unsigned)(nseg * ((len + 1) / 2))), dim3(SLP_T), 0, data, nseg, stride, len, cnt);
}
void g2_tree(g2_jac *data, uint64_t nseg, uint64_t stride, uint64_t len, bool hom, uint32_t *cnt, hipStream_t st) {
  const dim3 grid((unsigned)(nseg * ((len + 1) / 2)));
  if (len > 1 && hom) LAUNCH((ks_pt_tree<true, true>), grid, dim3(SLP_T), 0, data, nseg, stride, len, cnt);
  else if (len > 1) LAUNCH((ks_pt_tree<true, false>), grid, dim3(SLP_T), 0, data, nseg, stride, len, cnt);
}
void g1_hom_to_aff(const g1_jac *in, uint64_t stride, uint64_t n, g1_aff *out0, g1_aff *out1, uint64_t ostride, hipStream_t st) {
  if (n) LAUNCH(ks_hom_to_aff<false>, dim3((unsigned)n), dim3(SLP_T), 0, in, stride, n, out0, out1, ostride);
}
void g2_hom_to_aff(const g2_jac *in, uint64_t stride, uint64_t n, g2_aff *out, uint64_t ostride, hipStream_t st) {
  if (n) LAUNCH(ks_hom_to_aff<true>, dim3((unsigned)n), dim3(SLP_T), 0, in, stride, n, out, out + ostride, 2 * ostride);
}
void oa_g1terms(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t h, g1_jac *S, hipStream_t st) {
  LAUNCH(ks_oa_g1terms, dim3((unsigned)(nb * 2 * h)), dim3(SLP_T), 0, A, B, K, nb, h, S);
}
void kzg_terms_split(const g2_aff *h, const g2_aff *hm, const fe *Qc, uint64_t K, uint64_t nb, g2_jac *S2, hipStream_t st) {
  LAUNCH(ks_kzg_terms_split, dim3((unsigned)(4 * nb * (2 * K - 2))), dim3(SLP_T), 0, h, hm, Qc, K, nb, S2);
}
void g2_dbl_mults(const g2_aff *Q, uint64_t seg, uint64_t segstride, uint64_t n, g2_aff *M, hipStream_t st) {
  if (n) LAUNCH(ks_g2_dbl_mults, dim3((unsigned)(3 * n)), dim3(SLP_T), 0, Q, seg, segstride, n, M);
}
void g1_mul(const g1_aff *P, const fe *k, uint64_t n, g1_aff *out, void *tab, hipStream_t st) {
  if (n > MUL_MAX) kn::g1_mul(P, 0, k, n, out, tab, st);
  else if (n) LAUNCH(ks_g1_mul, dim3((unsigned)n), dim3(SLP_T), 0, P, k, n, out);
}
void mults(const fp12 *X, const fe *kx, uint64_t n3, fp12 *outx, const g2_aff *Q, const fe *kq, uint64_t n2, g2_aff *outq,
           const g1_aff *P, const fe *kp, uint64_t n1, g1_aff *outp, void *tab, hipStream_t st) {
  const bool many1 = n1 > MUL_MAX, many2 = n2 > MUL_MAX;
  if (many1) kn::g1_mul(P, 0, kp, n1, outp, tab, st);
  if (many2) kn::g2_mul(Q, 1, kq, n2, outq, tab, st);
  const uint64_t m1 = many1 ? 0 : n1, m2 = many2 ? 0 : n2;
  if (n3 + m2 + m1)
    LAUNCH(ks_mults, dim3((unsigned)(n3 + m2 + m1)), dim3(SLP_T), 0, X, kx, n3, outx, Q, kq, m2, outq, P, kp, m1, outp);
}
}  // namespace ks
