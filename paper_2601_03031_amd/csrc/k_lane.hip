// Scalar multiplications on one lane per element (lane29.hpp): the direct rounds of open-all, where
// there are points enough to give every SIMD a wavefront of 64 of them, and those that no chain
// waits for.
#define VC_INLINE_HELPERS 1
#include "kcommon.hpp"
#include "lane29.hpp"

#define LT 64  // threads of a workgroup: one wavefront, so that they spread over the SIMDs

namespace {

using lane::pt;
typedef lane::G1 L1_;
typedef lane::G2 L2_;
using lane::mul_lane;

}  // namespace

// A_j = A_L o A_R^{x_j}, b_j = b_L + b_R / x_j; x_j enters through its GLV split (per batch)
__global__ void __launch_bounds__(LT) kn_oa_fold_g1(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout, const fe *Xinv,
                                                    const glv::Dec *dec, uint64_t K, uint64_t nb, uint64_t h, uint32_t j,
                                                    uint32_t lK) {
  const uint64_t id = (uint64_t)blockIdx.x * LT + threadIdx.x;
  if (id >= nb * h) return;
  const uint64_t k = id / h, i = id % h;
  pt<L1_> t = mul_lane(Ain[k * K + h + i], dec[k]);
  const g1_aff l = Ain[k * K + i];
  if (!aff_is_inf(l)) t = lane::madd<L1_>(t, lane::in(l.x), lane::in(l.y));
  Aout[k * K + i] = lane::to_aff<L1_>(t);
  Bout[k * K + i] = fr_add(Bin[k * K + i], fr_mul(Bin[k * K + h + i], Xinv[k * lK + (j - 1)]));
}

// the G1 terms of <A_R, b_L> (side 0) and <A_L, b_R> (side 1), the sums of `per` consecutive ones
// (per divides h and LT): S[(2 k + side) (K / 2) + i / per], homogeneous
__global__ void __launch_bounds__(LT) kn_oa_g1terms(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t h,
                                                    uint32_t per, g1_jac *S) {
  __shared__ pt<L1_> sh[LT];
  const uint64_t id = (uint64_t)blockIdx.x * LT + threadIdx.x;
  const bool live = id < nb * 2 * h;
  const uint64_t k = id / (2 * h), r = id % (2 * h), side = r / h, i = r % h;
  pt<L1_> t = lane::identity<L1_>();
  if (live) {
    const fe c = f_from_mont<FpR>(B[side ? k * K + h + i : k * K + i]);
    t = mul_lane(A[side ? k * K + i : k * K + h + i], glv::decompose(c.l));
  }
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
  if (live && threadIdx.x % per == 0) S[(k * 2 + side) * (K / 2) + i / per] = {lane::out(t.X), lane::out(t.Y), lane::out(t.Z)};
}

// v_j = v_L o v_R^{1/x_j}; Vout may be Vin
__global__ void __launch_bounds__(LT) kn_oa_fold_g2(const g2_aff *Vin, g2_aff *Vout, const fe *Xinv, uint64_t K, uint64_t nb,
                                                    uint64_t h, uint32_t j, uint32_t lK) {
  const uint64_t id = (uint64_t)blockIdx.x * LT + threadIdx.x;
  if (id >= nb * h) return;
  const uint64_t k = id / h, i = id % h;
  const fe c = f_from_mont<FpR>(Xinv[k * lK + (j - 1)]);
  pt<L2_> t = mul_lane(Vin[k * K + h + i], gls::decompose(c.l));
  const g2_aff l = Vin[k * K + i];
  if (!aff_is_inf(l)) t = lane::madd<L2_>(t, L2_::in(l.x), L2_::in(l.y));
  Vout[k * K + i] = lane::to_aff<L2_>(t);
}

// out[i] = k_i P_i (P_0 with broadcast), affine
template <class L, class Dec>
__device__ __forceinline__ aff<typename L::O> mul_aff(const aff<typename L::O> &P, const fe &k_mont, Dec (*split)(const uint32_t *)) {
  const fe c = f_from_mont<FpR>(k_mont);
  return lane::to_aff<L>(mul_lane(P, split(c.l)));
}
__global__ void __launch_bounds__(LT) kn_g1_mul(const g1_aff *P, int broadcast, const fe *k, uint64_t n, g1_aff *out) {
  const uint64_t i = (uint64_t)blockIdx.x * LT + threadIdx.x;
  if (i < n) out[i] = mul_aff<L1_>(P[broadcast ? 0 : i], k[i], glv::decompose);
}
__global__ void __launch_bounds__(LT) kn_g2_mul(const g2_aff *P, int broadcast, const fe *k, uint64_t n, g2_aff *out) {
  const uint64_t i = (uint64_t)blockIdx.x * LT + threadIdx.x;
  if (i < n) out[i] = mul_aff<L2_>(P[broadcast ? 0 : i], k[i], gls::decompose);
}

// HyperEval terms (canonical differences of the folded table g* times PST keys) of every job:
// term r of level d of job x goes to S[(d G + x) M / 2 + r], Jacobian
__global__ void __launch_bounds__(LT) kn_hyper_terms(const S2Job *J, uint32_t G, uint64_t K, const g1_aff *ek, uint64_t M,
                                                     uint32_t lM, g1_jac *S) {
  uint64_t id = (uint64_t)blockIdx.x * LT + threadIdx.x;
  const uint64_t per = M / 2;
  if (id >= G * lM * per) return;
  const uint64_t x = id / (lM * per);
  const fe *g = J[x].Y + (2 * K - 2) * M;  // g*, the root row of the y-tree
  id %= lM * per;
  const uint32_t d = (uint32_t)(id / per);
  const uint64_t r = id % per, half = 1ull << (lM - d - 1), p = r / half, c = r % half;
  const fe q = fr_sub(g[p * (2 * half) + half + c], g[p * (2 * half) + c]);
  S[(d * G + x) * per + r] = lane::to_jac<L1_>(mul_lane(ek[half - 1 + c], glv::decompose(q.l)));
}

// the D-tree's leaves D_j = rho_j C_j of every job
__global__ void __launch_bounds__(LT) kn_d_leaves(const S2Job *J, uint32_t G, uint64_t K) {
  const uint64_t id = (uint64_t)blockIdx.x * LT + threadIdx.x;
  if (id >= G * K) return;
  const S2Job &jb = J[id / K];
  const uint64_t j = id % K;
  jb.D[j] = mul_aff<L1_>(jb.Cj[j], jb.rho[j], glv::decompose);
}

namespace kn {
#define LN(kern, n, ...) LAUNCH(kern, dim3((unsigned)(((n) + LT - 1) / LT)), dim3(LT), 0, __VA_ARGS__)
// Multiplications from which a launch is given to single lanes.  A lane's chain is the longest (G1
// 0.9 to 1.1 ms, G2 2.4, whatever the number up to 65536, a wavefront for each SIMD), but it does the least work
// for it: with 8 lanes a field element 65536 G1 terms took 7.5 ms and 32768 G2 folds 9.4, and none
// less than 1.7.  The engine's workgroup for each takes 0.4 ms (G1) to 0.7 (a fold) up to 2048 of them, and
// 1.5 ms for 8192 terms, with the whole chip.
static constexpr uint64_t LANE_MIN = 4096;

uint64_t oa_g1terms(const g1_aff *A, const fe *B, uint64_t K, uint64_t nb, uint64_t h, g1_jac *S, hipStream_t st) {
  if (nb * 2 * h < LANE_MIN) {
    ks::oa_g1terms(A, B, K, nb, h, S, st);
    return h;
  }
  const uint32_t per = h < LT ? (uint32_t)h : LT;
  LN(kn_oa_g1terms, nb * 2 * h, A, B, K, nb, h, per, S);
  return h / per;
}
bool fold_lanes(uint64_t nb, uint64_t h) { return nb * h >= LANE_MIN; }
void oa_fold_g1(const g1_aff *Ain, const fe *Bin, g1_aff *Aout, fe *Bout, const fe *Xinv, const glv::Dec *dec, uint64_t K,
                uint64_t nb, uint64_t h, uint32_t j, uint32_t lK, hipStream_t st) {
  LN(kn_oa_fold_g1, nb * h, Ain, Bin, Aout, Bout, Xinv, dec, K, nb, h, j, lK);
}
void oa_fold_g2(const g2_aff *Vin, g2_aff *Vout, const fe *Xinv, uint64_t K, uint64_t nb, uint64_t h, uint32_t j, uint32_t lK,
                hipStream_t st) {
  LN(kn_oa_fold_g2, nb * h, Vin, Vout, Xinv, K, nb, h, j, lK);
}
void g1_mul(const g1_aff *P, int bc, const fe *k, uint64_t n, g1_aff *out, hipStream_t st) {
  if (n) LN(kn_g1_mul, n, P, bc, k, n, out);
}
void g2_mul(const g2_aff *P, int bc, const fe *k, uint64_t n, g2_aff *out, hipStream_t st) {
  if (n) LN(kn_g2_mul, n, P, bc, k, n, out);
}
void hyper_terms(const S2Job *J, uint32_t G, uint64_t K, const g1_aff *ek, uint64_t M, uint32_t lM, g1_jac *S, hipStream_t st) {
  LN(kn_hyper_terms, G * lM * (M / 2), J, G, K, ek, M, lM, S);
}
void d_leaves(const S2Job *J, uint32_t G, uint64_t K, hipStream_t st) { LN(kn_d_leaves, G * K, J, G, K); }
}  // namespace kn
