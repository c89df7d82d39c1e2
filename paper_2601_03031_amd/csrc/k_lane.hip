// Scalar multiplications on one lane per element (lane29.hpp): the direct rounds of open-all, where
// there are points enough to give every SIMD a wavefront of 64 of them, and those that no chain
// waits for.
//
// A lane's table of 15 multiples (1.7 KB) is in memory of the caller's workspace, a slot for each
// workgroup; a launch has at most as many workgroups as stay resident (two wavefronts on each SIMD, by
// their registers: kn::TABLE_SLOTS) and each takes blocks of 64 in turn.  As an array of the lane's own
// it would be scratch memory, which the runtime keeps for every hardware queue and for every lane
// that the device could hold: 0.8 GB a queue, 12 GB on sixteen, that no workspace or budget counts.
#define VC_INLINE_HELPERS 1
#include "kcommon.hpp"
#include "lane_group.hpp"
#include "lane_pair.hpp"
#include "oa_terms.hpp"

#define LT 64  // threads of a workgroup: one wavefront, so that they spread over the SIMDs

namespace {

using lane::pt;
typedef lane::G1 L1_;
using lane::mul_lane;

// The lane's table: points of 27 words in seven 16-byte pieces, the same piece of the 64 lanes side by side
struct Table {
  uint4 *at;
  __device__ explicit Table(void *mem) : at(static_cast<uint4 *>(mem) + (uint64_t)blockIdx.x * (kn::TABLE_SLOT_BYTES / 16) + threadIdx.x) {}
  template <class L> __device__ __forceinline__ void put(int e, const pt<L> &t) const {
    uint4 *p = at + (e - 1) * (7 * LT);
    uint32_t w[28];
#pragma unroll
    for (int j = 0; j < 9; j++) {
      w[j] = t.X.l[j];
      w[9 + j] = t.Y.l[j];
      w[18 + j] = t.Z.l[j];
    }
    w[27] = 0;
#pragma unroll
    for (int q = 0; q < 7; q++) p[q * LT] = uint4{w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
  }
  template <class L> __device__ __forceinline__ pt<L> get(int e) const {
    const uint4 *p = at + (e - 1) * (7 * LT);
    uint32_t w[28];
#pragma unroll
    for (int q = 0; q < 7; q++) {
      const uint4 v = p[q * LT];
      w[4 * q] = v.x;
      w[4 * q + 1] = v.y;
      w[4 * q + 2] = v.z;
      w[4 * q + 3] = v.w;
    }
    pt<L> t;
#pragma unroll
    for (int j = 0; j < 9; j++) {
      t.X.l[j] = w[j];
      t.Y.l[j] = w[9 + j];
      t.Z.l[j] = w[18 + j];
    }
    return t;
  }
};
static_assert(kn::TABLE_SLOT_BYTES == 15 * 7 * 16 * LT, "15 points of seven 16-byte pieces a lane");

// the blocks of 64 threads' work that a workgroup takes in turn
#define FOR_BLOCKS(id, n) for (uint64_t id = (uint64_t)blockIdx.x * LT + threadIdx.x, n_ = (n); id - threadIdx.x < n_; id += (uint64_t)gridDim.x * LT)

// the sum of `per` consecutive lanes' points, in the first of them
__device__ __forceinline__ pt<L1_> sum_groups(pt<L1_> t, pt<L1_> *sh, uint32_t per) {
  sh[threadIdx.x] = t;
  __syncthreads();
#pragma unroll 1
  for (uint32_t s = 1; s < per; s *= 2) {
    const bool on = threadIdx.x % (2 * s) == 0;
    if (on) t = lane::add<L1_>(t, sh[threadIdx.x + s]);
    __syncthreads();
    if (on) sh[threadIdx.x] = t;
    __syncthreads();
  }
  return t;
}
// homogeneous, packed, in the place of a Jacobian point
__device__ __forceinline__ g1_jac hom(const pt<L1_> &t) { return {lane::out(t.X), lane::out(t.Y), lane::out(t.Z)}; }

}  // namespace

// A_j = A_L o A_R^{x_j}, b_j = b_L + b_R / x_j; x_j enters through its GLV split (per batch)
__global__ void __launch_bounds__(LT, 2) kn_oa_fold_g1(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout, const fe *Xinv,
                                                    const glv::Dec *dec, uint64_t K, uint64_t nb, uint64_t h, uint32_t j,
                                                    uint32_t lK, void *tab) {
  const Table T(tab);
  FOR_BLOCKS(id, nb * h) {
    if (id >= nb * h) return;
    const uint64_t k = id / h, i = id % h;
    pt<L1_> t = mul_lane(Ain[k * K + h + i], dec[k], T);
    const g1_aff l = Ain[k * K + i];
    if (!aff_is_inf(l)) t = lane::madd<L1_>(t, lane::in(l.x), lane::in(l.y));
    Aout[k * K + i] = lane::to_aff<L1_>(t);
    Bout[k * K + i] = fr_add(Bin[k * K + i], fr_mul(Bin[k * K + h + i], Xinv[k * lK + (j - 1)]));
  }
}

// the G1 terms of <A_R, b_L> (side 0) and <A_L, b_R> (side 1), the sums of `per` consecutive ones
// (per divides h and LT): S[(2 k + side) (K / 2) + i / per], homogeneous
__global__ void __launch_bounds__(LT, 2) kn_oa_g1terms(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t h,
                                                    uint32_t per, g1_jac *S, void *tab) {
  __shared__ pt<L1_> sh[LT];
  const Table T(tab);
  FOR_BLOCKS(id, nb * 2 * h) {
    const bool live = id < nb * 2 * h;
    const uint64_t k = id / (2 * h), r = id % (2 * h), side = r / h, i = r % h;
    pt<L1_> t = lane::identity<L1_>();
    if (live) {
      const fe c = f_from_mont<FpR>(B[side ? k * K + h + i : k * K + i]);
      t = mul_lane(A[side ? k * K + i : k * K + h + i], glv::decompose(c.l), T);
    }
    t = sum_groups(t, sh, per);
    if (live && threadIdx.x % per == 0) S[(k * 2 + side) * (K / 2) + i / per] = hom(t);
  }
}

// the same for the G1 terms b[v] A[a] taken a round ahead (oa_terms.hpp; per divides q and LT): the
// groups' sums at the start of each group's place in S1
__global__ void __launch_bounds__(LT, 2) kn_oa_g1terms_next(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t q,
                                                         uint32_t per, g1_jac *S1, void *tab) {
  __shared__ pt<L1_> sh[LT];
  const Table T(tab);
  FOR_BLOCKS(id, nb * 8 * q) {
    const bool live = id < nb * 8 * q;
    const oat::Term tm = oat::term(live ? id : 0, K, nb, q);
    pt<L1_> t = lane::identity<L1_>();
    if (live) {
      const fe c = f_from_mont<FpR>(B[tm.v]);
      t = mul_lane(A[tm.a], glv::decompose(c.l), T);
    }
    t = sum_groups(t, sh, per);
    const uint64_t len = id % (8 * q) < 4 * q ? 2 * q : q, at = tm.out % len;  // (both areas hold whole groups)
    if (live && threadIdx.x % per == 0) S1[tm.out - at + at / per] = hom(t);
  }
}

// out[i] = k_i P_i (P_0 with broadcast), affine
__device__ __forceinline__ g1_aff mul_aff(const g1_aff &P, const fe &k_mont, const Table &T) {
  const fe c = f_from_mont<FpR>(k_mont);
  return lane::to_aff<L1_>(mul_lane(P, glv::decompose(c.l), T));
}
__global__ void __launch_bounds__(LT, 2) kn_g1_mul(const g1_aff *P, int broadcast, const fe *k, uint64_t n, g1_aff *out, void *tab) {
  const Table T(tab);
  FOR_BLOCKS(i, n)
    if (i < n) out[i] = mul_aff(P[broadcast ? 0 : i], k[i], T);
}

// HyperEval terms (canonical differences of the folded table g* times PST keys) of every job:
// term r of level d of job x goes to S[(d G + x) M / 2 + r], Jacobian
__global__ void __launch_bounds__(LT, 2) kn_hyper_terms(const S2Job *J, uint32_t G, uint64_t K, const g1_aff *ek, uint64_t M,
                                                     uint32_t lM, g1_jac *S, void *tab) {
  const Table T(tab);
  const uint64_t per = M / 2;
  FOR_BLOCKS(id, G * lM * per) {
    if (id >= G * lM * per) return;
    const uint64_t x = id / (lM * per);
    const fe *g = J[x].Y + (2 * K - 2) * M;  // g*, the root row of the y-tree
    const uint32_t d = (uint32_t)(id / per % lM);
    const uint64_t r = id % per, half = 1ull << (lM - d - 1), p = r / half, c = r % half;
    const fe q = fr_sub(g[p * (2 * half) + half + c], g[p * (2 * half) + c]);
    S[(d * G + x) * per + r] = lane::to_jac<L1_>(mul_lane(ek[half - 1 + c], glv::decompose(q.l), T));
  }
}

// the D-tree's leaves D_j = rho_j C_j of every job
__global__ void __launch_bounds__(LT, 2) kn_d_leaves(const S2Job *J, uint32_t G, uint64_t K, void *tab) {
  const Table T(tab);
  FOR_BLOCKS(id, G * K) {
    if (id >= G * K) return;
    const S2Job &jb = J[id / K];
    const uint64_t j = id % K;
    jb.D[j] = mul_aff(jb.Cj[j], jb.rho[j], T);
  }
}

// ---------------------------------------------------------------- two lanes a point, a pairing
namespace {

using lane::fl;
using lane::pick;
typedef lane::G2pairOf<fl> G2pair;

__device__ __forceinline__ fe other_fe(const fe &a) {
  fe o;
#pragma unroll
  for (int j = 0; j < 8; j++) o.l[j] = __builtin_amdgcn_mov_dpp(a.l[j], 0xB1, 0xF, 0xF, true);
  return o;
}
// this lane's components of the affine point; zeros for the identity
__device__ __forceinline__ void to_aff_pair(const pt<G2pair> &t, fe &x, fe &y) {
  const fe z = lane::out(t.Z), zo = other_fe(z), n = fp_add(fp_sqr(z), fp_sqr(zo));
  x = y = fe_zero();
  if (fe_is_zero(n)) return;  // (a sum of two squares is zero for zeros only: -1 is no square)
  const fe w = fp_mul(z, fp_inv_fast(n));
  const fl zi = lane::in(G2pair::p() ? fp_neg(w) : w);
  x = lane::out(G2pair::mul(t.X, zi));
  y = lane::out(G2pair::mul(t.Y, zi));
}
// c in both lanes of a pair (the other lane's is read whatever this one's is: both are active then)
__device__ __forceinline__ bool both(bool c) {
  const int o = __builtin_amdgcn_mov_dpp((int)c, 0xB1, 0xF, 0xF, true);
  return (int)c & o;
}

}  // namespace

// v_j = v_L o v_R^{1/x_j}, two lanes a point (half the chain and half the state of one lane a point: 16384
// of them 1.5 ms for 2.5); Vout may be Vin
__global__ void __launch_bounds__(LT, 2) kn_oa_fold_g2(const g2_aff *Vin, g2_aff *Vout, const fe *Xinv, uint64_t K, uint64_t nb,
                                                    uint64_t h, uint32_t j, uint32_t lK, void *tab) {
  const Table T(tab);
  const bool p = G2pair::p();
  FOR_BLOCKS(lid, 2 * nb * h) {
    const uint64_t id = lid >> 1;
    if (id >= nb * h) return;
    const uint64_t k = id / h, i = id % h;
    const fe c = f_from_mont<FpR>(Xinv[k * lK + (j - 1)]);
    const fe *r = reinterpret_cast<const fe *>(Vin + k * K + h + i), *l = reinterpret_cast<const fe *>(Vin + k * K + i);
    const fe rx = r[p], ry = r[2 + p], lx = l[p], ly = l[2 + p];
    pt<G2pair> t = lane::mul_pair(lane::in_small(rx), lane::in_small(ry), both(fe_is_zero(rx) && fe_is_zero(ry)), gls::decompose(c.l), T);
    if (!both(fe_is_zero(lx) && fe_is_zero(ly))) t = lane::madd<G2pair>(t, lane::in_small(lx), lane::in_small(ly));
    fe x, y;
    to_aff_pair(t, x, y);
    fe *o = reinterpret_cast<fe *>(Vout + k * K + i);
    o[p] = x;
    o[2 + p] = y;
  }
}

// out[i] = k_i P_i (P_0 with broadcast) on G2, two lanes a point
__global__ void __launch_bounds__(LT, 2) kn_g2_mul(const g2_aff *P, int broadcast, const fe *k, uint64_t n, g2_aff *out, void *tab) {
  const Table T(tab);
  const bool p = G2pair::p();
  FOR_BLOCKS(lid, 2 * n) {
    const uint64_t i = lid >> 1;
    if (i >= n) return;
    const fe c = f_from_mont<FpR>(k[i]);
    const fe *q = reinterpret_cast<const fe *>(P + (broadcast ? 0 : i));
    const fe qx = q[p], qy = q[2 + p];
    fe x, y;
    to_aff_pair(lane::mul_pair(lane::in_small(qx), lane::in_small(qy), both(fe_is_zero(qx) && fe_is_zero(qy)), gls::decompose(c.l), T), x, y);
    fe *o = reinterpret_cast<fe *>(out + i);
    o[p] = x;
    o[2 + p] = y;
  }
}

// Miller values of the direct rounds: side 0 (L) pairs A[h + i] with V[i], side 1 (R) A[i] with V[h + i];
// the products of `per` consecutive ones (per divides h and LT / 2) into F[(2 k + side) K / 2 + i / per],
// equal to the engine's up to factors that the final exponentiation removes.  Bound by the
// multiply-adds: 32768 pairings, a wavefront for each SIMD, 2.5 ms; with 8 lanes an element they
// took 19, and half as many 9.
__global__ void __launch_bounds__(LT) kn_oa_miller(const g1_aff *A, const g2_aff *V, uint64_t K, uint64_t nb, uint64_t h,
                                                   uint32_t per, fp12 *F) {
  const uint64_t id = ((uint64_t)blockIdx.x * LT + threadIdx.x) >> 1;
  if (id >= nb * 2 * h) return;
  const bool p = threadIdx.x & 1;
  const uint64_t k = id / (2 * h), r = id % (2 * h), side = r / h, i = r % h;
  const g1_aff P = A[side ? k * K + i : k * K + h + i];
  const fe *Q = reinterpret_cast<const fe *>(V + (side ? k * K + h + i : k * K + i));
  const fe qx = Q[p], qy = Q[2 + p];
  // the identity in either place: 1
  const bool qz = both(fe_is_zero(qx) && fe_is_zero(qy));
  const bool none = aff_is_inf(P) || qz;
  const fl xP = lane::in_small(P.x), yP = lane::in_small(P.y), x = lane::in_small(qx), y = lane::in_small(qy);
  lane::twelve<fl> f = lane::miller_pair(p, xP, yP, x, y);
  const fl one = G2pair::one(), zero = {};
#pragma unroll
  for (int q = 0; q < 3; q++) {
    f.a.c[q] = pick(none, q == 0 ? one : zero, f.a.c[q]);
    f.b.c[q] = pick(none, zero, f.b.c[q]);
  }
  // (groups of `per` pairings do not cross wavefronts; lanes that are not the first of theirs go along)
#pragma unroll 1
  for (uint32_t d = 1; d < per; d *= 2) {
    lane::twelve<fl> g;
#pragma unroll
    for (int q = 0; q < 3; q++)
#pragma unroll
      for (int e = 0; e < 9; e++) {
        g.a.c[q].l[e] = __shfl_down(f.a.c[q].l[e], 2 * d);
        g.b.c[q].l[e] = __shfl_down(f.b.c[q].l[e], 2 * d);
      }
    f = lane::mul12(p, f, g);
  }
  if (id % per) return;
  fe *out = reinterpret_cast<fe *>(F + (k * 2 + side) * (K / 2) + i / per);
#pragma unroll
  for (int q = 0; q < 6; q++) out[2 * q + p] = lane::out(q < 3 ? f.a.c[q] : f.b.c[q - 3]);
}

namespace kn {
#define LN(kern, n, ...) LAUNCH(kern, dim3((unsigned)(((n) + LT - 1) / LT)), dim3(LT), 0, __VA_ARGS__)
// with a table for each workgroup
#define LNT(kern, n, ...) LAUNCH(kern, dim3((unsigned)table_slots(n)), dim3(LT), 0, __VA_ARGS__)

uint64_t oa_g1terms(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t h, g1_jac *S, void *tab, hipStream_t st) {
  if (nb * 2 * h < LANE_MIN) {
    ks::oa_g1terms(A, B, K, nb, h, S, st);
    return h;
  }
  const uint32_t per = h < LT ? (uint32_t)h : LT;
  LNT(kn_oa_g1terms, nb * 2 * h, A, B, K, nb, h, per, S, tab);
  return h / per;
}
uint64_t oa_g1terms_next(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t q, g1_jac *S1, void *tab, hipStream_t st) {
  if (nb * 8 * q < LANE_MIN) {
    ks::oa_g1terms_next(A, B, K, nb, q, S1, st);
    return 1;
  }
  const uint32_t per = q < LT ? (uint32_t)q : LT;
  LNT(kn_oa_g1terms_next, nb * 8 * q, A, B, K, nb, q, per, S1, tab);
  return per;
}
void oa_fold_g1(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout, const fe *Xinv, const glv::Dec *dec, uint64_t K,
                uint64_t nb, uint64_t h, uint32_t j, uint32_t lK, void *tab, hipStream_t st) {
  LNT(kn_oa_fold_g1, nb * h, Ain, Bin, Aout, Bout, Xinv, dec, K, nb, h, j, lK, tab);
}
void oa_fold_g2(const g2_aff *Vin, g2_aff *Vout, const fe *Xinv, uint64_t K, uint64_t nb, uint64_t h, uint32_t j, uint32_t lK,
                void *tab, hipStream_t st) {
  LNT(kn_oa_fold_g2, 2 * nb * h, Vin, Vout, Xinv, K, nb, h, j, lK, tab);
}
uint64_t oa_miller(const g1_aff *A, const g2_aff *V, uint64_t K, uint64_t nb, uint64_t h, fp12 *F, hipStream_t st) {
  const uint32_t per = h < LT / 2 ? (uint32_t)h : LT / 2;
  LN(kn_oa_miller, nb * 4 * h, A, V, K, nb, h, per, F);
  return h / per;
}
void g1_mul(const g1_aff *P, int bc, const fe *k, uint64_t n, g1_aff *out, void *tab, hipStream_t st) {
  if (n) LNT(kn_g1_mul, n, P, bc, k, n, out, tab);
}
void g2_mul(const g2_aff *P, int bc, const fe *k, uint64_t n, g2_aff *out, void *tab, hipStream_t st) {
  if (n) LNT(kn_g2_mul, 2 * n, P, bc, k, n, out, tab);
}
void hyper_terms(const S2Job *J, uint32_t G, uint64_t K, const g1_aff *ek, uint64_t M, uint32_t lM, g1_jac *S, void *tab, hipStream_t st) {
  LNT(kn_hyper_terms, G * lM * (M / 2), J, G, K, ek, M, lM, S, tab);
}
void d_leaves(const S2Job *J, uint32_t G, uint64_t K, void *tab, hipStream_t st) { LNT(kn_d_leaves, G * K, J, G, K, tab); }
}  // namespace kn
