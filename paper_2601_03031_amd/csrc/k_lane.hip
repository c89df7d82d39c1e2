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
#include "lane29.hpp"
#include "gls.hpp"
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

// ---------------------------------------------------------------- Miller loops
// Two lanes a pairing, lane p of them with component p of every element of F_p2 (p = 0, 1): the state of
// a pairing, 24 elements of F_p, then fits the registers of its lanes, and a product in F_p2 is one
// sum of two products in each.  Sums of products over F_p2 have one reduction, so that F_p6 products
// and the product by a line are taken by their definition (a third of the reductions that the forms
// with fewer products need, and no sums before or after).
namespace {

using lane::fl;

__device__ __forceinline__ fl other(const fl &a) {  // the other lane's
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = __builtin_amdgcn_mov_dpp(a.l[j], 0xB1, 0xF, 0xF, true);
  return o;
}
__device__ __forceinline__ fl pick(bool c, const fl &a, const fl &b) {
  fl o;
#pragma unroll
  for (int j = 0; j < 9; j++) o.l[j] = c ? a.l[j] : b.l[j];
  return o;
}
// a second factor b as both lanes use it: a b = own(a) x + other(a) y, with (x, y) = (b_0, -b_1) in lane
// 0 and (b_0, b_1) in lane 1
struct fac {
  fl x, y;
};
__device__ __forceinline__ fac factor(bool p, const fl &b) {
  const fl o = other(b);
  return {pick(p, o, b), pick(p, b, lane::neg(o))};
}
// sums of one, two and three products a b, the other lane's a given
__device__ __forceinline__ fl prod(const fl &a, const fl &ao, const fac &b) { return lane::mul2(a, b.x, ao, b.y); }
__device__ __forceinline__ fl prod2(const fl &a, const fl &ao, const fac &b, const fl &c, const fl &co, const fac &d) {
  return lane::mul4(a, b.x, ao, b.y, c, d.x, co, d.y);
}
__device__ __forceinline__ fl prod3(const fl &a, const fl &ao, const fac &b, const fl &c, const fl &co, const fac &d, const fl &e,
                                    const fl &eo, const fac &f) {
  const fl *x[6] = {&a, &ao, &c, &co, &e, &eo}, *y[6] = {&b.x, &b.y, &d.x, &d.y, &f.x, &f.y};
  return lane::dot<6>(x, y);
}
__device__ __forceinline__ fl mul2_(bool p, const fl &a, const fl &b) { return prod(a, other(a), factor(p, b)); }
// a^2: (a_0 + a_1)(a_0 - a_1) in lane 0, 2 a_1 a_0 in lane 1
__device__ __forceinline__ fl sqr2_(bool p, const fl &a) {
  const fl o = other(a);
  return lane::mul(lane::add(a, pick(p, a, o)), pick(p, o, lane::sub(a, o)));
}
// k a + b, a - b and (9 + i) a, reduced: limbs of one unit, within 0.51 p
__device__ __forceinline__ fl red(const fl &a, int k, const fl &b) { return lane::reduce(a, k, b); }
__device__ __forceinline__ fl red_sub(const fl &a, const fl &b) { return lane::reduce(b, -1, a); }
__device__ __forceinline__ fl xi(bool p, const fl &a) {
  const fl o = other(a);
  return red(a, 9, pick(p, o, lane::neg(o)));
}

struct six {
  fl c[3];  // over 1, v, v^2
};
// a b in F_p6 (limbs of one unit)
__device__ __forceinline__ six mul6(bool p, const six &a, const six &b) {
  const fl o0 = other(a.c[0]), o1 = other(a.c[1]), o2 = other(a.c[2]);
  const fac b0 = factor(p, b.c[0]), b1 = factor(p, b.c[1]), b2 = factor(p, b.c[2]);
  const fac x1 = factor(p, xi(p, b.c[1])), x2 = factor(p, xi(p, b.c[2]));
  return {{prod3(a.c[0], o0, b0, a.c[1], o1, x2, a.c[2], o2, x1), prod3(a.c[0], o0, b1, a.c[1], o1, b0, a.c[2], o2, x2),
           prod3(a.c[0], o0, b2, a.c[1], o1, b1, a.c[2], o2, b0)}};
}
struct twelve {
  six a, b;  // a + b w, w^2 = v
};
// f^2 = (a + b)(a + v b) - t - v t + 2 t w, t = a b
__device__ __forceinline__ void sqr12(bool p, twelve &f) {
  six x = f.a, y = f.b, t = {}, r = {};
#pragma unroll 1
  for (int k = 0; k < 2; k++) {  // (one copy of the product's code for both)
    r = mul6(p, x, y);
    if (k == 0) {
      t = r;
      const fl v0 = xi(p, f.b.c[2]);
#pragma unroll
      for (int i = 0; i < 3; i++) {
        x.c[i] = red(f.a.c[i], 1, f.b.c[i]);
        y.c[i] = red(f.a.c[i], 1, i ? f.b.c[i - 1] : v0);
      }
    }
  }
  const fl t0 = xi(p, t.c[2]);
#pragma unroll
  for (int i = 0; i < 3; i++) {
    f.a.c[i] = red_sub(lane::sub(r.c[i], t.c[i]), i ? t.c[i - 1] : t0);
    f.b.c[i] = red(t.c[i], 2, fl{});
  }
}
// f g = t0 + v t1 + (t2 - t0 - t1) w, t0 = a a', t1 = b b', t2 = (a + b)(a' + b')
__device__ __forceinline__ twelve mul12(bool p, const twelve &f, const twelve &g) {
  six x = f.a, y = g.a, t[3] = {};
#pragma unroll 1
  for (int k = 0; k < 3; k++) {
    const six r = mul6(p, x, y);
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
  const fl v0 = xi(p, t[1].c[2]);
  twelve o;
#pragma unroll
  for (int i = 0; i < 3; i++) {
    o.a.c[i] = red(t[0].c[i], 1, i ? t[1].c[i - 1] : v0);
    o.b.c[i] = red_sub(lane::sub(t[2].c[i], t[0].c[i]), t[1].c[i]);
  }
  return o;
}
// f (l0 + l1 w + l3 w^3)
__device__ __forceinline__ void mul_line(bool p, twelve &f, const fl &l0, const fl &l1, const fl &l3) {
  const fac c0 = factor(p, l0), c1 = factor(p, l1), c3 = factor(p, l3), x1 = factor(p, xi(p, l1)), x3 = factor(p, xi(p, l3));
  const fl *a = f.a.c, *b = f.b.c;
  const fl ao[3] = {other(a[0]), other(a[1]), other(a[2])}, bo[3] = {other(b[0]), other(b[1]), other(b[2])};
  twelve r;
  r.a.c[0] = prod3(a[0], ao[0], c0, b[1], bo[1], x3, b[2], bo[2], x1);
  r.a.c[1] = prod3(a[1], ao[1], c0, b[0], bo[0], c1, b[2], bo[2], x3);
  r.a.c[2] = prod3(a[2], ao[2], c0, b[0], bo[0], c3, b[1], bo[1], c1);
  r.b.c[0] = prod3(b[0], bo[0], c0, a[0], ao[0], c1, a[2], ao[2], x3);
  r.b.c[1] = prod3(b[1], bo[1], c0, a[0], ao[0], c3, a[1], ao[1], c1);
  r.b.c[2] = prod3(b[2], bo[2], c0, a[1], ao[1], c3, a[2], ao[2], c1);
  f = r;
}

// G2 with a lane for each component of its coordinates (lane29.hpp's group law on the lane's own)
struct G2pair {
  using T = fl;
  static __device__ __forceinline__ bool p() { return threadIdx.x & 1; }
  static __device__ __forceinline__ T zero() { return T{}; }
  static __device__ __forceinline__ T some() { return T{{!p()}}; }
  static __device__ __forceinline__ T one() { return pick(p(), T{}, lane::small_one()); }
  static __device__ __forceinline__ T add(const T &a, const T &b) { return lane::add(a, b); }
  static __device__ __forceinline__ T sub(const T &a, const T &b) { return lane::sub(a, b); }
  static __device__ __forceinline__ T neg(const T &a) { return lane::neg(a); }
  static __device__ __forceinline__ T norm(const T &a) { return lane::norm(a); }
  static __device__ __forceinline__ T times(const T &a, int k) { return lane::times(a, k); }
  static __device__ __forceinline__ T norm_times(const T &a, int k) { return lane::norm_times(a, k); }
  static __device__ __forceinline__ T mul(const T &a, const T &b) { return mul2_(p(), a, b); }
  static __device__ __forceinline__ T mul2(const T &a, const T &b, const T &c, const T &d) {
    return prod2(a, other(a), factor(p(), b), c, other(c), factor(p(), d));
  }
  static __device__ __forceinline__ T sqr(const T &a) { return sqr2_(p(), a); }
  static __device__ __forceinline__ T b3(const T &a) {
    T k;
#pragma unroll
    for (int j = 0; j < 9; j++) k.l[j] = bn::TWIST_3B29[p()][j];
    return mul(a, k);
  }
};

// k Q on G2 with the split k = sum_j k_j lam^j (gls.hpp): the table of the 15 subset sums of
// sign(k_j) psi^j(Q), a doubling and at most one addition per bit.  x, y: this lane's components of Q;
// inf and d are the same in both lanes
__device__ __forceinline__ pt<G2pair> mul_pair(const fe &qx, const fe &qy, bool inf, const gls::Dec &d, const Table &T) {
  if (inf || d.nbits == 0) return lane::identity<G2pair>();
  const bool p = G2pair::p();
  fl x = lane::in_small(qx), y = lane::in_small(qy);
  const fl kx = lane::in_small(fe_const(p ? bn::FROB1_2_1 : bn::FROB1_2_0)), ky = lane::in_small(fe_const(p ? bn::FROB1_3_1 : bn::FROB1_3_0));
#pragma unroll 1
  for (int j = 0; j < 4; j++) {
    if (j) {
      x = mul2_(p, pick(p, lane::neg(x), x), kx);
      y = mul2_(p, pick(p, lane::neg(y), y), ky);
    }
    const fl s = pick(d.neg >> j & 1, lane::neg(y), y);
    T.put(1 << j, pt<G2pair>{x, s, G2pair::one()});
#pragma unroll 1
    for (int e = 1; e < 1 << j; e++) T.put(e + (1 << j), lane::madd<G2pair>(T.get<G2pair>(e), x, s));
  }
  const int n = (int)d.nbits;
  pt<G2pair> acc = T.get<G2pair>((int)gls::digit(d, (uint32_t)(n - 1)));
#pragma unroll 1
  for (int t = n - 2; t >= 0; t--) {
    acc = lane::dbl<G2pair>(acc);
    const uint32_t dg = gls::digit(d, (uint32_t)t);
    if (dg) acc = lane::add<G2pair>(acc, T.get<G2pair>((int)dg));
  }
  return acc;
}
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

struct point {
  fl X, Y, Z;  // homogeneous
};
// T = 2 T and the tangent at T at P: l0 = 2YZ yP, l1 = -3X^2 xP, l3 = Y^2 - 3b'Z^2, all up to a factor in
// F_p2, which the final exponentiation removes
__device__ __forceinline__ void tangent(bool p, point &T, const fl &xP, const fl &yP, const fl &b3, fl &l0, fl &l1, fl &l3) {
  const fl XX = sqr2_(p, T.X), YY = sqr2_(p, T.Y), E = mul2_(p, sqr2_(p, T.Z), b3);
  const fl XY = mul2_(p, T.X, T.Y), YZ = mul2_(p, T.Y, T.Z);
  const fac fY = factor(p, YY);
  l0 = lane::mul(lane::times(YZ, 2), yP);
  l1 = lane::mul(lane::times(XX, -3), xP);
  l3 = red_sub(YY, E);
  T.X = mul2_(p, lane::times(XY, 2), red(E, -3, YY));
  T.Y = red_sub(sqr2_(p, red(E, 3, YY)), mul2_(p, red(E, 12, fl{}), E));
  const fl z = red(YZ, 8, fl{});
  T.Z = prod(z, other(z), fY);
}
// T = T + (x, y) and the line through both at P
__device__ __forceinline__ void chord(bool p, point &T, const fl &x, const fl &y, const fl &xP, const fl &yP, fl &l0, fl &l1, fl &l3) {
  const fl Zo = other(T.Z);
  const fac fx = factor(p, x), fy = factor(p, y);
  const fl th = red_sub(T.Y, prod(T.Z, Zo, fy)), la = red_sub(T.X, prod(T.Z, Zo, fx));
  const fl tho = other(th), lao = other(la);
  l0 = lane::mul(la, yP);
  l1 = lane::mul(lane::neg(th), xP);
  l3 = prod2(th, tho, fx, lane::neg(la), lane::neg(lao), fy);
  const fac D = factor(p, sqr2_(p, la));
  const fl E = prod(la, lao, D), F = prod(T.Z, Zo, factor(p, sqr2_(p, th))), G = prod(T.X, other(T.X), D);
  const fl H = red(G, -2, lane::add(E, F));
  const fac fE = factor(p, lane::neg(E));
  T.X = prod(la, lao, factor(p, H));
  T.Y = prod2(th, tho, factor(p, red_sub(G, H)), T.Y, other(T.Y), fE);
  T.Z = prod(lane::neg(T.Z), lane::neg(Zo), fE);
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
    pt<G2pair> t = mul_pair(rx, ry, both(fe_is_zero(rx) && fe_is_zero(ry)), gls::decompose(c.l), T);
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
    to_aff_pair(mul_pair(qx, qy, both(fe_is_zero(qx) && fe_is_zero(qy)), gls::decompose(c.l), T), x, y);
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
  fl one = lane::small_one(), zero = {};
  one = pick(p, zero, one);
  fl b3;
#pragma unroll
  for (int j = 0; j < 9; j++) b3.l[j] = bn::TWIST_3B29[p][j];
  point T = {x, y, one};
  twelve f = {{{one, zero, zero}}, {{zero, zero, zero}}};
  // over the non-adjacent form of 6u + 2 (d_65 = 1 starts T = Q; d_64 = 0), a doubling in each step, then
  // with a digit an addition; the last two steps add pi(Q) and -pi^2(Q)
  fl sx = x, sy = y;
#pragma unroll 1
  for (int s = 64, add = 0; s >= -2;) {
    fl l0, l1, l3;
    if (!add && s >= 0) {
      if (s != 64) sqr12(p, f);
      tangent(p, T, xP, yP, b3, l0, l1, l3);
    } else {
      fl cx = sx, cy = sy;
      if (s < 0) {
        // the next Frobenius image, and its negative the second time
        const fl kx = lane::in_small(fe_const(p ? bn::FROB1_2_1 : bn::FROB1_2_0)), ky = lane::in_small(fe_const(p ? bn::FROB1_3_1 : bn::FROB1_3_0));
        sx = cx = mul2_(p, pick(p, lane::neg(sx), sx), kx);
        sy = cy = mul2_(p, pick(p, lane::neg(sy), sy), ky);
        if (s == -2) cy = lane::neg(cy);
      } else if (bn::ATE_NAF_NEG >> s & 1) {
        cy = lane::neg(cy);
      }
      chord(p, T, cx, cy, xP, yP, l0, l1, l3);
    }
    mul_line(p, f, l0, l1, l3);
    add = !add && s >= 0 && s < 64 && ((bn::ATE_NAF_POS | bn::ATE_NAF_NEG) >> s & 1);
    if (!add) s--;
  }
#pragma unroll
  for (int q = 0; q < 3; q++) {
    f.a.c[q] = pick(none, q == 0 ? one : zero, f.a.c[q]);
    f.b.c[q] = pick(none, zero, f.b.c[q]);
  }
  // (groups of `per` pairings do not cross wavefronts; lanes that are not the first of theirs go along)
#pragma unroll 1
  for (uint32_t d = 1; d < per; d *= 2) {
    twelve g;
#pragma unroll
    for (int q = 0; q < 3; q++)
#pragma unroll
      for (int e = 0; e < 9; e++) {
        g.a.c[q].l[e] = __shfl_down(f.a.c[q].l[e], 2 * d);
        g.b.c[q].l[e] = __shfl_down(f.b.c[q].l[e], 2 * d);
      }
    f = mul12(p, f, g);
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
