// Kernels of VC.Verify for one opening proof (appendix C; section 3 FC.BVerify with the
// faster verifier; section 4.2 for the Merkle and folding parts):
//   kv_decode      point decompression and range checks, one thread per proof element
//   kv_chains      Fiat-Shamir replay (r_i, x_j, z, rho_j), f_v(z), Merkle path, y*
//   kv_jobs        b_l, the multiplication and power jobs
//   kv_assemble    point sums and the pairs of the three pairing checks
//   kv_compare     the final equalities
// Scalar multiplications, G_T exponentiations, Miller loops and final exponentiations
// run in the shared kernels (the engine's, and single lanes' for more than 2048 multiplications).
#include "kcommon.hpp"
#include "verify.h"

namespace {

__device__ fe rd_be(const uint8_t *b) {
  fe a;
  for (int i = 0; i < 8; i++)
    a.l[7 - i] = ((uint32_t)b[4 * i] << 24) | ((uint32_t)b[4 * i + 1] << 16) | ((uint32_t)b[4 * i + 2] << 8) | b[4 * i + 3];
  return a;
}

__device__ bool lt_words(const fe &a, const uint32_t *m) {
  for (int i = 7; i >= 0; i--)
    if (a.l[i] != m[i]) return a.l[i] < m[i];
  return false;
}

// canonical y > (p - 1)/2
__device__ bool larger(const fe &ymont) { return !lt_words(f_from_mont<FpP>(ymont), bn::P_HALF) && !fe_eq(f_from_mont<FpP>(ymont), fe_const(bn::P_HALF)); }

// a^((p - 3) / 4): times a, a square root of a or (p = 3 mod 4, -1 no square) of -a
__device__ __attribute__((noinline)) fe pow_sqrt(const fe &a) { return f_pow_fixed<FpP>(a, bn::P_SQRT_EXP); }

// A compressed point: of G1 (32 bytes: x, flag 0x80 identity, 0x40 y > (p - 1)/2) into *o1, or of G2
// (64 bytes: x.c0 || x.c1, the sign that of y.c1, or of y.c0 when y.c1 = 0) into *o2.  One path for
// both, as the lanes of a wavefront hold points of both kinds: the root of G1's x^3 + 3 and that of
// the norm of G2's right side are the same call.  Bound by its two powers, chains of 312 products
// each: the items of a proof of 276 points take 0.38 ms; with a branch for each kind of item and a
// bit at a time, three powers and an inverse on G2, they took 2.4.
//
// On G2 with a = a0 + a1 i, s = sqrt(a0^2 + a1^2), t = (a0 + s) / 2 and w = t^((p-3)/4): x0 = w t has
// x0^2 = +-t and 1 / x0 = +-w, so that with the upper sign x0 + (a1 / 2 x0) i is a root, and with the
// lower sign, where (a0 - s) / 2 = -a1^2 / 4t is the square, a1 / 2 x0 + x0 i is.  The square is
// checked at the end.
__device__ bool decompress(const uint8_t *b, bool g2, g1_aff *o1, g2_aff *o2) {
  const int len = g2 ? 64 : 32;
  const bool inf = b[0] & 0x80, big = b[0] & 0x40;
  if (g2) *o2 = {f2_zero(), f2_zero()};
  else *o1 = {fe_zero(), fe_zero()};
  if (inf) {
    uint32_t any = b[0] & 0x7f;
    for (int i = 1; i < len; i++) any |= b[i];
    return any == 0;
  }
  fe x0 = rd_be(b), x1 = fe_zero();
  x0.l[7] &= 0x3fffffffu;
  if (g2) x1 = rd_be(b + 32);
  if (!lt_words(x0, bn::P_MOD) || !lt_words(x1, bn::P_MOD)) return false;
  x0 = f_to_mont<FpP>(x0);
  fp2 rhs = {fe_zero(), fe_zero()};
  fe a;
  if (g2) {
    x1 = f_to_mont<FpP>(x1);
    const fp2 x = {x0, x1};
    rhs = f2_add(f2_mul(f2_sqr(x), x), f2_const(bn::TWIST_B0, bn::TWIST_B1));
    a = fe_is_zero(rhs.c1) ? rhs.c0 : fp_add(fp_sqr(rhs.c0), fp_sqr(rhs.c1));
  } else {
    a = fp_add(fp_mul(fp_sqr(x0), x0), f_mul_small<FpP>(f_one<FpP>(), 3));
  }
  const fe s = fp_mul(pow_sqrt(a), a);
  const bool square = fe_eq(fp_sqr(s), a);
  if (!g2) {
    if (!square) return false;
    *o1 = {x0, larger(s) != big ? fp_neg(s) : s};
    return true;
  }
  fp2 y;
  if (fe_is_zero(rhs.c1)) {
    y = square ? fp2{s, fe_zero()} : fp2{fe_zero(), s};
  } else {
    if (!square) return false;
    const fe t = fp_half(fp_add(rhs.c0, s)), w = pow_sqrt(t), r = fp_mul(w, t);
    const bool plus = fe_eq(fp_sqr(r), t);
    fe h = fp_mul(fp_half(rhs.c1), w);
    if (!plus) h = fp_neg(h);
    y = plus ? fp2{r, h} : fp2{h, r};
  }
  const fp2 chk = f2_sqr(y);
  if (!fe_eq(chk.c0, rhs.c0) || !fe_eq(chk.c1, rhs.c1)) return false;
  const bool l = fe_is_zero(y.c1) ? larger(y.c0) : larger(y.c1);
  *o2 = {{x0, x1}, l != big ? f2_neg(y) : y};
  return true;
}

// One item of a serialized proof and where it goes.  A lane first finds its item and then decodes
// it, so that lanes with items of different origin decode together; an F_p12 element is 12 items.
enum { IT_ZERO1, IT_ZERO, IT_G1, IT_G2, IT_FP, IT_FR, IT_FR_LE };  // IT_ZERO1, IT_ZERO: zeros for a point of G1, a scalar
struct Item {
  int kind, bad;  // bad: the flag raised when the bytes are none
  const uint8_t *src;
  void *dst;
};
__device__ Item item(int kind, const uint8_t *src, void *dst, int bad = VFLAG_BAD_PROOF) { return {kind, bad, src, dst}; }
// coefficient k of an F_p12 element
__device__ Item item_gt(const uint8_t *src, fp12 *dst, uint32_t k, int bad = VFLAG_BAD_PROOF) {
  return {IT_FP, bad, src + 32 * k, reinterpret_cast<fe *>(dst) + k};
}
__device__ void decode_item(const Item &it, int *flags) {
  bool ok = true;
  if (it.kind == IT_G1 || it.kind == IT_G2) {
    ok = decompress(it.src, it.kind == IT_G2, (g1_aff *)it.dst, (g2_aff *)it.dst);
  } else if (it.kind == IT_ZERO1) {
    *(g1_aff *)it.dst = {fe_zero(), fe_zero()};
  } else if (it.kind == IT_ZERO) {
    *(fe *)it.dst = fe_zero();
  } else if (it.kind == IT_FP) {
    const fe v = rd_be(it.src);
    ok = lt_words(v, bn::P_MOD);
    *(fe *)it.dst = f_to_mont<FpP>(v);
  } else {
    fe v;
    if (it.kind == IT_FR) v = rd_be(it.src);
    else
      for (int i = 0; i < 8; i++)
        v.l[i] = (uint32_t)it.src[4 * i] | (uint32_t)it.src[4 * i + 1] << 8 | (uint32_t)it.src[4 * i + 2] << 16 |
                 (uint32_t)it.src[4 * i + 3] << 24;
    ok = lt_words(v, bn::R_MOD);
    *(fe *)it.dst = f_to_mont<FpR>(v);
  }
  if (!ok) atomicOr(flags, it.bad);
}

}  // namespace

// one thread per item of proof blockIdx.y (layout of the serialized proof, vc_proof_get): the G2
// points first (the longest), then the G1 points, then the field elements
__device__ __host__ uint32_t kv_items(uint32_t t, uint32_t l, uint32_t lM) { return 2 + (t + 3 * l + 1 + lM) + (25 * l + 13); }
__global__ void __launch_bounds__(TPB) kv_decode(const VCtx *cs) {
  const VCtx &c = cs[blockIdx.y];
  uint32_t id = (uint32_t)gtid();
  const uint32_t t = c.t, l = c.lK, lM = c.lM;
  if (id >= kv_items(t, l, lM)) return;
  // block commitments, rounds, A_l v_l pi_v, D-tree siblings with their y, W
  const uint8_t *rounds = c.proof + 32 * t, *tail = rounds + 832ull * l, *dy = tail + 160, *w = dy + 64ull * l;
  Item it;
  if (id < 2) it = item(IT_G2, tail + 32 + 64 * id, id ? c.piv : c.vl);
  else if ((id -= 2) < t) it = item(IT_G1, c.proof + 32 * id, c.blk + id);
  else if ((id -= t) < 2 * l) it = item(IT_G1, rounds + 832ull * (id / 2) + (id % 2 ? 800 : 384), (id % 2 ? c.Rg1 : c.Lg1) + id / 2);
  else if ((id -= 2 * l) < 1) it = item(IT_G1, tail, c.Al);
  // (a sub-array proof has no Step 2 items and no entry: zeros)
  else if ((id -= 1) < l) it = item(c.fc_only ? IT_ZERO1 : IT_G1, dy + 64 * id, c.Dsib + id);
  else if ((id -= l) < lM) it = item(c.fc_only ? IT_ZERO1 : IT_G1, w + 32 * id, c.Wp + id);
  else if ((id -= lM) < 24 * l) {
    const uint32_t r = id / 24, side = id / 12 % 2;
    it = item_gt(rounds + 832ull * r + 416 * side, (side ? c.Rgt : c.Lgt) + r, id % 12);
  } else if ((id -= 24 * l) < l) it = item(c.fc_only ? IT_ZERO : IT_FR, dy + 64 * id + 32, c.ysib + id);
  else if ((id -= l) < 12) it = item_gt(c.Cb, c.C, id, VFLAG_BAD_INPUT);
  else it = item(c.fc_only ? IT_ZERO : IT_FR_LE, c.mib, c.mi, VFLAG_BAD_INPUT);
  decode_item(it, c.flags);
}

// Fiat-Shamir replay, the three chains that do not depend on one another in a workgroup each
// (blockIdx.x; blockIdx.y: the proof):
//   0  the challenges x_j with their inverses, z and f_v(z);
//   1  the chunk digests, sigma and the batching coefficients r_u;
//   2  the Merkle path, rho_j and y*.
// Bound by the first, a chain of l hashes of 17 blocks: 0.43 ms at 2^16 entries in batches of 256, 2.0
// when a workgroup did the three in turn, with an inverse in each round.
static constexpr uint32_t MAX_CHUNKS = 1024;  // t <= 32768 (K of log N <= 30)
// words of shared memory: sigma's message (a prefix of 392 bytes and the tag, the digests, padding),
// then a chunk's message and schedules for each wavefront
static constexpr uint32_t SIGMA_WORDS = (392 + 32 + 32 * MAX_CHUNKS + 72) / 4, CHUNK_WORDS = 32 * 18 + 18;
static constexpr uint32_t CHAIN_WORDS = SIGMA_WORDS + 4 * (CHUNK_WORDS + sha::SCHED_WORDS);

// x_1 .. x_l = H2F(FC-X, x_{j-1} || L_gt || L_g1 || R_gt || R_g1) and their inverses, then z =
// H2F(FC-Z, x_l || v_l) in all lanes, f_v(z) = prod_j (1 + x_j^{-1} z^{2^{l-j+1}}) in lane 0; the
// workgroup hashes together.  lds: 512 + SCHED_WORDS words
template <class C> __device__ fe challenge_chain(const C &c, uint32_t l, uint32_t *lds, fe *fz) {
  const int tid = threadIdx.x;
  uint32_t *msg = lds + sha::SCHED_WORDS, *t2 = msg + 16 + 8 + 2 * (96 + 16) + 32;
  const sha::Coop cp{tid, 256, lds};
  for (uint32_t j = 0; j < l; j++) {
    const int pre = j > 0 ? 8 : 0;
    const int e = j > 0 ? tid - 1 : tid;
    if (j > 0 && tid == 0) sha::put_words<FpR>(msg + 16, c.x[j - 1]);
    if (e >= 0 && e < 28) {
      int side = e / 14, q = e % 14;
      const fe *src = q < 12 ? reinterpret_cast<const fe *>(side ? c.Rgt + j : c.Lgt + j) + q
                             : reinterpret_cast<const fe *>(side ? c.Rg1 + j : c.Lg1 + j) + (q - 12);
      sha::put_words<FpP>(msg + 16 + pre + 112 * side + 8 * q, *src);
    }
    __syncthreads();
    const fe x = sha::xmd_fr_coop(cp, msg, 4 * (pre + 224), DSTR_FC_X, t2);
    if (tid == 0) {
      if (fe_is_zero(x)) atomicOr(c.flags, VFLAG_BAD_PROOF);
      c.x[j] = x;
    }
    __syncthreads();
  }
  if (tid == 0) sha::put_words<FpR>(msg + 16, c.x[l - 1]);
  if (tid >= 1 && tid <= 4) sha::put_words<FpP>(msg + 24 + 8 * (tid - 1), reinterpret_cast<const fe *>(c.vl)[tid - 1]);
  for (uint32_t j = tid; j < l; j += 256) c.xinv[j] = f_inv_fast<FpR>(c.x[j], bn::R_R3);
  __syncthreads();
  const fe z = sha::xmd_fr_coop(cp, msg, 160, DSTR_FC_Z, t2);
  if (tid == 0) {
    fe f = f_one<FpR>(), zp = fr_mul(z, z);  // z^{2^1}
    for (int j = (int)l; j >= 1; j--) {      // exponent 2^{l-j+1}: j = l first
      f = fr_mul(f, fr_add(f_one<FpR>(), fr_mul(c.xinv[j - 1], zp)));
      zp = fr_mul(zp, zp);
    }
    *fz = f;
  }
  return z;
}

__global__ void __launch_bounds__(256) kv_chains(const VCtx *cs) {
  const VCtx &c = cs[blockIdx.y];
  const int tid = threadIdx.x;
  const uint32_t t = c.t, l = c.lK;
  __shared__ uint32_t lds[CHAIN_WORDS];
  __shared__ uint32_t sigma[8];
  if (blockIdx.x == 0) {
    const fe z = challenge_chain(c, l, lds, c.fz);
    if (tid == 0) c.ms[t + 2 * l + 3] = z;
  } else if (blockIdx.x == 1) {
    // sigma = H(FC-R || C || t || digests of 32-entry chunks); a wavefront per chunk
    const int wave = tid / 64, lane = tid % 64;
    uint32_t *msg = lds + SIGMA_WORDS + wave * (CHUNK_WORDS + sha::SCHED_WORDS);
    const sha::Coop cw{lane, 64, msg + CHUNK_WORDS};
    const uint32_t nch = (t + 31) / 32, dl = (uint32_t)sha::cstrlen(DSTR_FC_R);
    for (uint32_t q = wave; q < nch; q += 4) {
      const uint32_t n = t - 32 * q < 32 ? t - 32 * q : 32, u = 32 * q + lane;
      if (lane < (int)n) {
        const uint64_t a = c.lo + u;
        msg[18 * lane] = (uint32_t)(a >> 32);
        msg[18 * lane + 1] = (uint32_t)a;
        sha::put_words<FpP>(msg + 18 * lane + 2, c.blk[u].x);
        sha::put_words<FpP>(msg + 18 * lane + 10, c.blk[u].y);
      }
      cw.sync();
      uint32_t dig[8];
      sha::sha_coop(cw, msg, 72u * n, dig);
      // byte lane of the digest (every lane has it)
      uint32_t v = 0;
      for (int w = 0; w < 8; w++) v = lane / 4 == w ? dig[w] : v;
      if (lane < 32) sha::put_byte(lds, dl + 392 + 32 * q + lane, v >> (24 - 8 * (lane & 3)));
    }
    if ((uint32_t)tid < dl) sha::put_byte(lds, tid, (uint8_t)DSTR_FC_R[tid]);
    if (tid >= 64 && tid < 76) sha::put_field_bytes<FpP>(lds, dl + 32 * (tid - 64), reinterpret_cast<const fe *>(c.C)[tid - 64]);
    if (tid >= 128 && tid < 136) sha::put_byte(lds, dl + 384 + (tid - 128), tid < 132 ? 0 : (t >> (8 * (135 - tid))) & 0xff);
    __syncthreads();
    uint32_t sg[8];
    sha::sha_coop(sha::Coop{tid, 256, lds + SIGMA_WORDS}, lds, dl + 392 + 32 * nch, sg);
    if (tid == 0)
      for (int w = 0; w < 8; w++) sigma[w] = sg[w];
    __syncthreads();
    // r_u = H2F(FC-R, sigma || u)
    for (uint32_t u = tid; u < t; u += 256) {
      sha::Hasher hs;
      sha::xmd_begin(hs);
      for (int w = 0; w < 8; w++) hs.word(sigma[w]);
      hs.u64(u);
      c.r[u] = sha::xmd_finish_fr(hs, DSTR_FC_R);
    }
  } else if (c.fc_only) {
    if (tid == 0) {
      c.ms[t + 2 * l + 1] = fe_zero();
      c.ms[t + 2 * l + 2] = fe_zero();
    }
  } else {
    // Merkle path of leaf i = SHA-256(0x00 || m_i || C_j) up to the root
    uint32_t *msg = lds + sha::SCHED_WORDS, *t2 = msg + 16 + 12 * 8 + 8 + 2 + 32;
    if (tid == 64) {
      const g1_aff &Cj = c.blk[c.j - c.lo];
      uint32_t mw[8], cw[16], node[8];
      fe mc = f_from_mont<FpR>(*c.mi);
      fe cx = f_from_mont<FpP>(Cj.x), cy = f_from_mont<FpP>(Cj.y);
      for (int q = 0; q < 8; q++) { mw[q] = mc.l[7 - q]; cw[q] = cx.l[7 - q]; cw[8 + q] = cy.l[7 - q]; }
      sha::merkle_leaf(node, mw, cw);
      uint64_t pos = c.N + c.i;
      for (uint32_t h = 0; h < c.L; h++, pos >>= 1) {
        uint32_t sib[8];
        const uint8_t *sb = c.mpath + 32 * h;
        for (int q = 0; q < 8; q++)
          sib[q] = ((uint32_t)sb[4 * q] << 24) | ((uint32_t)sb[4 * q + 1] << 16) | ((uint32_t)sb[4 * q + 2] << 8) | sb[4 * q + 3];
        uint32_t o[8];
        if (pos & 1) sha::merkle_node(o, sib, node);
        else sha::merkle_node(o, node, sib);
        for (int q = 0; q < 8; q++) node[q] = o[q];
      }
      for (int q = 0; q < 8; q++) msg[16 + 96 + q] = node[q];
      msg[16 + 104] = (uint32_t)(c.j >> 32);
      msg[16 + 105] = (uint32_t)c.j;
    }
    if (tid < 12) sha::put_words<FpP>(msg + 16 + 8 * tid, reinterpret_cast<const fe *>(c.C)[tid]);
    __syncthreads();
    const fe rho = sha::xmd_fr_coop(sha::Coop{tid, 256, lds}, msg, 4 * 106, DSTR_RHO, t2);
    if (tid == 0) {
      fe ystar = fr_mul(rho, *c.mi);
      for (uint32_t h = 0; h < l; h++) ystar = fr_add(ystar, c.ysib[h]);
      c.ms[t + 2 * l + 1] = rho;
      c.ms[t + 2 * l + 2] = ystar;
    }
  }
}

// b_l = sum_u r_u prod_k (x_k^{-1})^{bit_{l-k}(a_u)} as a tree of per-thread partial sums, and the
// multiplication and power jobs, a workgroup per proof
__global__ void __launch_bounds__(256) kv_jobs(const VCtx *cs) {
  const VCtx &c = cs[blockIdx.x];
  const int tid = threadIdx.x;
  const uint32_t t = c.t, l = c.lK;
  __shared__ fe part[256];
  fe acc = fe_zero();
  for (uint32_t u = tid; u < t; u += 256) {
    fe term = c.r[u];
    for (uint32_t k = 1; k <= l; k++)
      if (((c.lo + u) >> (l - k)) & 1) term = fr_mul(term, c.xinv[k - 1]);
    acc = fr_add(acc, term);
  }
  part[tid] = acc;
  __syncthreads();
  for (int sft = 128; sft > 0; sft >>= 1) {
    if (tid < sft) part[tid] = fr_add(part[tid], part[tid + sft]);
    __syncthreads();
  }
  // G1 multiplication jobs: r_u blk_u; x_j Lg1_j; x_j^{-1} Rg1_j; b_l A_l; rho C_j; y* g1; z g1
  // (the last three scalars are there already); then (g1, 0) up to the stride of the job arrays
  const g1_aff g1 = {fe_const(bn::G1X), fe_const(bn::G1Y)};
  for (uint32_t q = tid; q < c.nmul; q += 256) {
    g1_aff base = g1;
    fe k = fe_zero();
    bool set = true;
    if (q < t) {
      base = c.blk[q]; k = c.r[q];
    } else if (q < t + 2 * l) {
      uint32_t j = (q - t) / 2;
      if ((q - t) % 2 == 0) { base = c.Lg1[j]; k = c.x[j]; }
      else { base = c.Rg1[j]; k = c.xinv[j]; }
    } else if (q == t + 2 * l) {
      base = *c.Al; k = part[0];
    } else if (q < t + 2 * l + 4) {
      if (q == t + 2 * l + 1) base = c.blk[c.j - c.lo];
      set = false;
    }
    c.mb[q] = base;
    if (set) c.ms[q] = k;
  }
  // G_T jobs: L_j^{x_j}, R_j^{1/x_j}
  for (uint32_t q = tid; q < 2 * l; q += 256) {
    c.gts[q] = (q % 2 == 0) ? c.x[q / 2] : c.xinv[q / 2];
    c.gtb[q] = (q % 2 == 0) ? c.Lgt[q / 2] : c.Rgt[q / 2];
  }
}

// point sums and pairing inputs, three workgroups per proof (blockIdx.y), as none of the points needs
// another:
//   0  the sum of the t + 2l products, as a tree of per-thread partial sums;
//   1  the first pair of the Step 2 check;
//   2  the points of the other pairs, a thread each.
// 0.16 ms at 2^16 entries in batches of 256, two thirds of it the tree; 0.78 with one thread for all but
// the tree.
__global__ void __launch_bounds__(256) kv_assemble(const VCtx *cs) {
  const VCtx &c = cs[blockIdx.y];
  const int tid = threadIdx.x;
  const uint32_t t = c.t, l = c.lK, lM = c.lM;
  // pairs: (A_l, v_l) | (beta g1 - z g1, pi_v), (-g1, v_l - f_v(z) g2) | (D* - y* g1, -g2), (W_d, s'_d g2)
  const g1_aff g1 = {fe_const(bn::G1X), fe_const(bn::G1Y)};
  const g2_aff g2 = {f2_const(bn::G2X0, bn::G2X1), f2_const(bn::G2Y0, bn::G2Y1)};
  if (blockIdx.x == 0) {
    __shared__ g1_jac sh[256];
    g1_jac acc = jac_inf<OpsG1>();
    for (uint32_t u = tid; u < t + 2 * l; u += 256) acc = jac_madd(acc, c.mo[u]);
    sh[tid] = acc;
    __syncthreads();
    for (int sft = 128; sft > 0; sft >>= 1) {
      if (tid < sft) sh[tid] = jac_add(sh[tid], sh[tid + sft]);
      __syncthreads();
    }
    // G_T product C prod L^x R^{1/x} gathers in gto[0..2l] with C last
    for (uint32_t q = tid; q < 2 * l; q += 256) c.gto[q] = c.gtp[q];
    if (tid == 0) {
      *c.Cg1 = jac_to_aff(sh[0]);
      *c.bA = c.mo[t + 2 * l];
      c.gto[2 * l] = *c.C;
    }
  } else if (blockIdx.x == 1) {
    if (tid == 0) {
      g1_jac D = jac_from_aff(c.mo[t + 2 * l + 1]);
      for (uint32_t h = 0; h < l; h++) D = jac_madd(D, c.Dsib[h]);
      c.pp[3] = jac_to_aff(jac_madd(D, aff_neg(c.mo[t + 2 * l + 2])));
      c.pq[3] = aff_neg(g2);
    } else if (tid == 64) {
      c.pp[0] = *c.Al; c.pq[0] = *c.vl;
      c.pp[1] = jac_to_aff(jac_madd(jac_from_aff(*c.g1beta), aff_neg(c.mo[t + 2 * l + 3])));
      c.pq[1] = *c.piv;
    }
  } else {
    // thread 0: v_l - f_v(z) g2; thread 1 + d: s'_d g2, that is s_var g2 or, with bit var of a, less g2
    for (uint32_t q = tid; q < 1 + lM; q += 256) {
      const uint32_t d = q - 1, var = lM - 1 - d;
      const bool sub = q == 0 || ((uint64_t)c.a >> var & 1);
      g2_aff Q = q == 0 ? *c.vl : c.vk[var];
      const g2_aff S = q == 0 ? *c.fzg2 : g2;
      if (sub) Q = jac_to_aff(jac_madd(jac_from_aff(Q), aff_neg(S)));
      if (q == 0) {
        c.pp[2] = aff_neg(g1); c.pq[2] = Q;
      } else {
        c.pp[4 + d] = c.Wp[d]; c.pq[4 + d] = Q;
      }
    }
  }
}

// the final equalities, a thread per proof
__global__ void __launch_bounds__(64) kv_compare(const VCtx *cs, uint32_t n) {
  uint64_t p = gtid();
  if (p >= n) return;
  const VCtx &c = cs[p];
  fp12 one;
  fe *o = reinterpret_cast<fe *>(&one);
  for (int k = 0; k < 12; k++) o[k] = k == 0 ? f_one<FpP>() : fe_zero();
  auto eq12 = [](const fp12 &a, const fp12 &b) {
    const fe *x = reinterpret_cast<const fe *>(&a), *y = reinterpret_cast<const fe *>(&b);
    bool e = true;
    for (int k = 0; k < 12; k++) e = e && fe_eq(x[k], y[k]);
    return e;
  };
  bool ok = eq12(c.E[0], c.gto[0]) && eq12(c.E[1], one) && eq12(c.E[2], one) && fe_eq(c.bA->x, c.Cg1->x) &&
            fe_eq(c.bA->y, c.Cg1->y);
  if (c.cj_expect) {
    const g1_aff &cj = c.blk[c.j - c.lo];
    ok = ok && fe_eq(cj.x, c.cj_expect->x) && fe_eq(cj.y, c.cj_expect->y);
  }
  if (ok) atomicOr(c.flags, VFLAG_ACCEPT);
}

// the three final exponentiations' inputs of every proof side by side (products of the pairs
// 0, 1..2 and 3..), so that one launch takes them all: G[3 p + r] = F[p npair + {0, 1, 3}[r]]
__global__ void __launch_bounds__(TPB) kv_fe_gather(const fp12 *F, uint64_t npair, uint32_t n, fp12 *G) {
  uint64_t id = gtid();
  if (id >= 3ull * n) return;
  uint64_t p = id / 3, r = id % 3;
  G[id] = F[p * npair + (r == 2 ? 3 : r)];
}

namespace kv {
void fe_gather(const fp12 *F, uint64_t npair, uint32_t n, fp12 *G, hipStream_t st) { L1(kv_fe_gather, 3ull * n, F, npair, n, G); }
void decode(const VCtx *cs, uint32_t n, uint32_t tmax, uint32_t lK, uint32_t lM, hipStream_t st) {
  LAUNCH(kv_decode, dim3(nblk(kv_items(tmax, lK, lM)), n), dim3(TPB), 0, cs);
}
void transcript(const VCtx *cs, uint32_t n, hipStream_t st) {
  LAUNCH(kv_chains, dim3(3, n), dim3(256), 0, cs);
  LAUNCH(kv_jobs, dim3(n), dim3(256), 0, cs);
}
void assemble(const VCtx *cs, uint32_t n, hipStream_t st) { LAUNCH(kv_assemble, dim3(3, n), dim3(256), 0, cs); }
void compare(const VCtx *cs, uint32_t n, hipStream_t st) {
  LAUNCH(kv_compare, dim3((n + 63) / 64), dim3(64), 0, cs, n);
}
}  // namespace kv

// ------------------------------------------------------------------ every proof at once
// Serialization of all N proofs (the wire format of vc_proof_get) and their verification in
// one pass: items that honest proofs share (the block and FC proof of a batch, the D-tree
// siblings, the W commitments) are compared byte for byte with the proof that represents
// them and decoded once; the PST checks (section 4.2 Step 2, appendix C) of all proofs are
// combined with random 128-bit weights delta_i into one product of l_M + 1 pairings:
//   e(sum_i delta_i (D*_i - y*_i g1 + sum_d a_{i,var d} W_{i,d}), -g2) prod_d e(sum_i delta_i W_{i,d}, vk_{var d}) = 1
// with var d = l_M - 1 - d.  The FC part (FC.BVerify with the faster verifier) is the same
// for every proof of a batch and is checked once per batch by the one-proof verifier.
namespace {

__device__ uint64_t pl_bm(const PLayout &y) { return (uint64_t)y.b * y.M; }
__device__ uint64_t pl_batch(const PLayout &y, uint64_t i) { return i / pl_bm(y); }
__device__ uint32_t pl_t(const PLayout &y, uint64_t k) { return k == y.nb - 1 ? y.t_last : y.b; }
// byte offset of proof i
__device__ uint64_t pl_off(const PLayout &y, uint64_t i) {
  uint64_t k = pl_batch(y, i), bm = pl_bm(y);
  return k * bm * y.len_full + (i - k * bm) * (k == y.nb - 1 ? y.len_last : y.len_full);
}
// start of the Step 2 part (after block, rounds and tail) in a proof of batch k
__device__ uint64_t pl_step2(const PLayout &y, uint64_t k) { return 32ull * pl_t(y, k) + 832ull * y.lK + 160; }

__device__ int ilog2(uint64_t v) {
  int r = 0;
  while (v >>= 1) r++;
  return r;
}
// heap index n of a D-tree sibling (levels h < lK of K >> h nodes) to (h, s)
__device__ void d_node(uint64_t n, uint64_t K, uint32_t &h, uint64_t &s) {
  h = 0;
  while (n >= (K >> h)) { n -= K >> h; h++; }
  s = n;
}
// heap index w of a W commitment to depth d and prefix p
__device__ void w_node(uint64_t w, uint32_t &d, uint64_t &p) {
  d = (uint32_t)ilog2(w + 1);
  p = w + 1 - (1ull << d);
}

}  // namespace

// Serialization.  A proof is a row of 32-byte units (t block commitments, 26 for a round, 5 of the tail,
// then a D sibling and its y for each level, W, the Merkle path), and most are those of other proofs: the
// block and FC proof are a batch's, a D sibling that of 2^h subvectors, a W that of a prefix.  kps_first
// encodes each such unit once, in the first proof that carries it; kps_copy, a workgroup per proof, takes
// them from there and turns the y and the digests around.  Bound by the writes: 1.07 GB (2^16 proofs,
// b = 256) in 0.31 ms; with a thread encoding each item in place, a byte at a time, 2.0.
namespace {

struct unit32 {
  uint32_t w[8];
};
__device__ __forceinline__ unit32 swapped(const uint32_t *v, bool rev) {  // big-endian words, in the order given or reversed
  unit32 o;
#pragma unroll
  for (int q = 0; q < 8; q++) o.w[q] = __builtin_bswap32(v[rev ? 7 - q : q]);
  return o;
}
__device__ unit32 unit_fe(const fe &mont) {
  const fe c = f_from_mont<FpP>(mont);
  return swapped(c.l, true);
}
__device__ unit32 unit_g1(const g1_aff &p) {
  unit32 o = {};
  if (aff_is_inf(p)) {
    o.w[0] = 0x80;
    return o;
  }
  o = unit_fe(p.x);
  if (larger(p.y)) o.w[0] |= 0x40;
  return o;
}
// half 0: x.c0 with the flags, 1: x.c1
__device__ unit32 unit_g2(const g2_aff &p, int half) {
  unit32 o = {};
  if (aff_is_inf(p)) {
    if (!half) o.w[0] = 0x80;
    return o;
  }
  o = unit_fe(half ? p.x.c1 : p.x.c0);
  if (!half && (fe_is_zero(p.y.c1) ? larger(p.y.c0) : larger(p.y.c1))) o.w[0] |= 0x40;
  return o;
}
// ALIGNED: to and from 16-byte boundaries, else a byte at a time
template <bool ALIGNED> __device__ __forceinline__ void put_unit(uint8_t *o, const unit32 &u) {
  if (ALIGNED) {
    reinterpret_cast<uint4 *>(o)[0] = uint4{u.w[0], u.w[1], u.w[2], u.w[3]};
    reinterpret_cast<uint4 *>(o)[1] = uint4{u.w[4], u.w[5], u.w[6], u.w[7]};
  } else {
    for (int q = 0; q < 32; q++) o[q] = (uint8_t)(u.w[q >> 2] >> (8 * (q & 3)));
  }
}
template <bool ALIGNED> __device__ __forceinline__ unit32 get_unit(const uint8_t *b) {
  unit32 u = {};
  if (ALIGNED) {
    const uint4 x = reinterpret_cast<const uint4 *>(b)[0], y = reinterpret_cast<const uint4 *>(b)[1];
    u = {{x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w}};
  } else {
    for (int q = 0; q < 32; q++) u.w[q >> 2] |= (uint32_t)b[q] << (8 * (q & 3));
  }
  return u;
}

}  // namespace

// one thread per unit that proofs share: the b + 26 l + 5 of a batch, the 2K - 2 D siblings, the M - 1 W
template <bool ALIGNED> __global__ void __launch_bounds__(TPB) kps_first(PSCtx c) {
  const PLayout &y = c.y;
  const uint64_t l = y.lK, pre = y.b + 26 * l + 5, nD = 2 * y.K - 2, nW = y.M - 1;
  uint64_t id = gtid();
  if (id >= y.nb * pre + nD + nW) return;
  unit32 u;
  uint8_t *o;
  if (id < y.nb * pre) {
    const uint64_t k = id / pre, t = pl_t(y, k);
    uint64_t q = id % pre;
    if (q >= t + 26 * l + 5) return;  // (the last batch may be shorter)
    o = c.out + pl_off(y, k * pl_bm(y)) + 32 * q;
    if (q < t) {
      u = unit_g1(c.Cj[k * y.b + q]);
    } else if ((q -= t) < 26 * l) {
      const uint64_t s = k * l + q / 26, e = q % 26, side = e / 13, f = e % 13;
      if (f < 12) u = unit_fe(reinterpret_cast<const fe *>((side ? c.Rgt : c.Lgt) + s)[f]);
      else u = unit_g1((side ? c.Rg1 : c.Lg1)[s]);
    } else if ((q -= 26 * l) == 0) {
      u = unit_g1(c.Al[k]);
    } else {
      u = unit_g2(q < 3 ? c.vl[k] : c.piv[k], (int)(q - 1) & 1);
    }
  } else if ((id -= y.nb * pre) < nD) {
    uint32_t h;
    uint64_t s;
    d_node(id, y.K, h, s);
    const uint64_t i = ((s ^ 1) << h) * y.M;
    o = c.out + pl_off(y, i) + pl_step2(y, pl_batch(y, i)) + 64 * h;
    u = unit_g1(c.D[id]);
  } else {
    id -= nD;
    uint32_t d;
    uint64_t p;
    w_node(id, d, p);
    const uint64_t i = p << (y.lM - d);
    o = c.out + pl_off(y, i) + pl_step2(y, 0) + 64 * l + 32 * d;
    u = unit_g1(c.W[id]);
  }
  put_unit<ALIGNED>(o, u);
}

// proof of this workgroup (proof_grid)
__device__ __forceinline__ uint64_t proof_id() { return ((uint64_t)blockIdx.y << 16) + blockIdx.x; }

// every other unit, a workgroup per proof
template <bool ALIGNED> __global__ void __launch_bounds__(256) kps_copy(PSCtx c) {
  const PLayout &y = c.y;
  const uint64_t i = proof_id(), k = pl_batch(y, i), j = i / y.M, a = i % y.M, first = k * pl_bm(y);
  const uint32_t t = pl_t(y, k), l = y.lK, pre = t + 26 * l + 5, n = pre + 2 * l + y.lM + y.L;
  uint8_t *o = c.out + pl_off(y, i);
  const uint8_t *f = c.out + pl_off(y, first);
  for (uint32_t q = threadIdx.x; q < n; q += 256) {
    unit32 u;
    uint32_t v = q;
    if (v < pre) {
      if (i == first) continue;
      u = get_unit<ALIGNED>(f + 32 * q);
    } else if ((v -= pre) < 2 * l) {
      const uint32_t h = v >> 1;
      if (v & 1) {
        const uint64_t node = 2 * y.K - ((2 * y.K) >> h) + ((j >> h) ^ 1);
        u = swapped(c.Y[node * y.M + a].l, true);  // stored canonical
      } else {
        const uint64_t r = ((j >> h) << h) * y.M;
        if (r == i) continue;
        u = get_unit<ALIGNED>(c.out + pl_off(y, r) + pl_step2(y, pl_batch(y, r)) + 64 * h);
      }
    } else if ((v -= 2 * l) < y.lM) {
      const uint64_t r = (a >> (y.lM - v)) << (y.lM - v);
      if (r == i) continue;
      u = get_unit<ALIGNED>(c.out + pl_off(y, r) + pl_step2(y, 0) + 64ull * l + 32 * v);
    } else {
      v -= y.lM;
      u = swapped(c.tree + 8 * (((y.N + i) >> v) ^ 1), false);
    }
    put_unit<ALIGNED>(o + 32ull * q, u);
  }
}

// shared items, one thread each: K block commitments, 2K - 2 D-tree siblings, M - 1 W, C (12
// coefficients)
__global__ void __launch_bounds__(TPB) kva_decode(VACtx c) {
  const PLayout &y = c.y;
  uint64_t id = gtid(), K = y.K;
  const uint64_t nD = 2 * K - 2, nW = y.M - 1;
  if (id >= K + nD + nW + 12) return;
  Item it;
  if (id < K) {
    const uint64_t k = id / y.b;
    it = item(IT_G1, c.proofs + pl_off(y, k * pl_bm(y)) + 32 * (id - k * y.b), c.Cj + id);
  } else if ((id -= K) < nD) {
    uint32_t h;
    uint64_t s;
    d_node(id, K, h, s);
    uint64_t j = (s ^ 1) << h, i = j * y.M;
    it = item(IT_G1, c.proofs + pl_off(y, i) + pl_step2(y, pl_batch(y, i)) + 64 * h, c.Dn + id);
  } else if ((id -= nD) < nW) {
    uint32_t d;
    uint64_t p;
    w_node(id, d, p);
    uint64_t i = p << (y.lM - d);
    it = item(IT_G1, c.proofs + pl_off(y, i) + pl_step2(y, 0) + 64ull * y.lK + 32 * d, c.Wn + id);
  } else {
    it = item_gt(c.Cb, c.C, (uint32_t)(id - nW), VFLAG_BAD_INPUT);
  }
  decode_item(it, c.flags);
}

// the root of every proof's Merkle path from its leaf (m_i, C_j), one thread per proof
__global__ void __launch_bounds__(TPB) kva_roots(VACtx c) {
  const PLayout &y = c.y;
  uint64_t i = gtid();
  if (i >= y.N) return;
  uint64_t j = i / y.M;
  fe m;
  for (int q = 0; q < 8; q++) {
    const uint8_t *b = c.m + 32 * i + 4 * q;
    m.l[q] = (uint32_t)b[0] | ((uint32_t)b[1] << 8) | ((uint32_t)b[2] << 16) | ((uint32_t)b[3] << 24);
  }
  if (!lt_words(m, bn::R_MOD)) atomicOr(c.flags, VFLAG_BAD_INPUT);
  fe cx = f_from_mont<FpP>(c.Cj[j].x), cy = f_from_mont<FpP>(c.Cj[j].y);
  uint32_t mw[8], cw[16], node[8];
  for (int q = 0; q < 8; q++) { mw[q] = m.l[7 - q]; cw[q] = cx.l[7 - q]; cw[8 + q] = cy.l[7 - q]; }
  sha::merkle_leaf(node, mw, cw);
  const uint8_t *path = c.proofs + pl_off(y, i) + pl_step2(y, pl_batch(y, i)) + 64ull * y.lK + 32ull * y.lM;
  uint64_t pos = y.N + i;
  for (uint32_t h = 0; h < y.L; h++, pos >>= 1) {
    uint32_t sib[8], o[8];
    for (int q = 0; q < 8; q++) {
      const uint8_t *sb = path + 32 * h + 4 * q;
      sib[q] = ((uint32_t)sb[0] << 24) | ((uint32_t)sb[1] << 16) | ((uint32_t)sb[2] << 8) | sb[3];
    }
    if (pos & 1) sha::merkle_node(o, sib, node);
    else sha::merkle_node(o, node, sib);
    for (int q = 0; q < 8; q++) node[q] = o[q];
  }
  for (int q = 0; q < 8; q++) c.root[8 * i + q] = node[q];
}

// rho_j from C and the root of proof 0, one thread per j
__global__ void __launch_bounds__(64) kva_rho(VACtx c) {
  uint64_t j = gtid();
  if (j >= c.y.K) return;
  sha::Hasher hr;
  sha::xmd_begin(hr);
  hr.gt(*c.C);
  for (int q = 0; q < 8; q++) hr.word(c.root[q]);
  hr.u64(j);
  c.rho[j] = sha::xmd_finish_fr(hr, DSTR_RHO);
}

// a workgroup per proof: its block, FC proof, D-tree siblings and W against the proofs that
// represent them (16-byte words; every proof starts on a 32-byte boundary)
__global__ void __launch_bounds__(256) kva_same(VACtx c) {
  const PLayout &y = c.y;
  __shared__ int diff;
  const uint64_t i = proof_id();
  const int t = threadIdx.x;
  if (t == 0) diff = 0;
  __syncthreads();
  uint64_t k = pl_batch(y, i), j = i / y.M, a = i % y.M, i0 = k * pl_bm(y);
  const uint4 *P = reinterpret_cast<const uint4 *>(c.proofs + pl_off(y, i));
  bool d = false;
  if (i != i0) {
    const uint4 *R = reinterpret_cast<const uint4 *>(c.proofs + pl_off(y, i0));
    uint64_t n16 = pl_step2(y, k) / 16;
    for (uint64_t q = t; q < n16; q += 256) {
      uint4 u = P[q], v = R[q];
      d |= u.x != v.x || u.y != v.y || u.z != v.z || u.w != v.w;
    }
  }
  // item x < lK: D-tree sibling of level x; lK <= x < lK + lM: W of depth x - lK (two words each)
  uint32_t nit = y.lK + y.lM;
  if ((uint32_t)t < 2 * nit) {
    uint32_t x = t / 2, half = t % 2;
    uint64_t ir, ofs_i, ofs_r;
    if (x < y.lK) {
      ir = ((j >> x) << x) * y.M;
      ofs_i = pl_step2(y, k) + 64ull * x;
      ofs_r = pl_step2(y, pl_batch(y, ir)) + 64ull * x;
    } else {
      uint32_t dd = x - y.lK;
      ir = (a >> (y.lM - dd)) << (y.lM - dd);
      ofs_i = pl_step2(y, k) + 64ull * y.lK + 32ull * dd;
      ofs_r = pl_step2(y, 0) + 64ull * y.lK + 32ull * dd;
    }
    if (ir != i) {
      uint4 u = reinterpret_cast<const uint4 *>(c.proofs + pl_off(y, i) + ofs_i)[half];
      uint4 v = reinterpret_cast<const uint4 *>(c.proofs + pl_off(y, ir) + ofs_r)[half];
      d |= u.x != v.x || u.y != v.y || u.z != v.z || u.w != v.w;
    }
  }
  if (d) atomicOr(&diff, 1);
  __syncthreads();
  if (t == 0) c.odd[i] = diff ? 1 : 0;
}

// one thread per proof: y*_i = rho_j m_i + sum of the y siblings, the weight delta_i =
// H(seed, i) (128 bits), and delta_i, delta_i y*_i (zero for a proof left to the one-proof
// verifier, which joins the list)
__global__ void __launch_bounds__(TPB) kva_proof(VACtx c) {
  const PLayout &y = c.y;
  uint64_t i = gtid();
  if (i >= y.N) return;
  bool odd = c.odd[i] != 0;
  for (int q = 0; q < 8; q++) odd = odd || c.root[8 * i + q] != c.root[q];
  uint64_t j = i / y.M;
  fe m;
  for (int q = 0; q < 8; q++) {
    const uint8_t *b = c.m + 32 * i + 4 * q;
    m.l[q] = (uint32_t)b[0] | ((uint32_t)b[1] << 8) | ((uint32_t)b[2] << 16) | ((uint32_t)b[3] << 24);
  }
  fe ys = fr_mul(c.rho[j], f_to_mont<FpR>(m));
  const uint8_t *s2 = c.proofs + pl_off(y, i) + pl_step2(y, pl_batch(y, i));
  for (uint32_t h = 0; h < y.lK; h++) {
    fe v = rd_be(s2 + 64 * h + 32);
    if (!lt_words(v, bn::R_MOD)) atomicOr(c.flags, VFLAG_BAD_PROOF);
    ys = fr_add(ys, f_to_mont<FpR>(v));
  }
  sha::Hasher hs;
  hs.init();
  hs.str(DSTR_VALL);
  hs.bytes(c.seed, 32);
  hs.u64(i);
  uint32_t dg[8];
  hs.final(dg);
  fe w = fe_zero();
  for (int q = 0; q < 4; q++) w.l[3 - q] = dg[q];
  w = f_to_mont<FpR>(w);
  if (odd) {
    uint32_t at = atomicAdd(c.oddcnt, 1u);
    c.oddlist[at] = i;  // at < N: one entry per proof at most
    w = fe_zero();
  }
  c.delta[i] = w;
  c.dy[i] = fr_mul(w, ys);
}

// sums of the weights: per row j (over a), per column a (over j), and of delta_i y*_i;
// workgroups [0, K) rows, [K, K + M) columns, K + M the total
__global__ void __launch_bounds__(256) kva_sums(VACtx c) {
  const PLayout &y = c.y;
  __shared__ fe sh[256];
  uint64_t g = blockIdx.x;
  const int t = threadIdx.x;
  fe acc = fe_zero();
  if (g < y.K) {
    for (uint64_t a = t; a < y.M; a += 256) acc = fr_add(acc, c.delta[g * y.M + a]);
  } else if (g < y.K + y.M) {
    uint64_t a = g - y.K;
    for (uint64_t j = t; j < y.K; j += 256) acc = fr_add(acc, c.delta[j * y.M + a]);
  } else {
    for (uint64_t i = t; i < y.N; i += 256) acc = fr_add(acc, c.dy[i]);
  }
  sh[t] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) sh[t] = fr_add(sh[t], sh[t + s]);
    __syncthreads();
  }
  if (t == 0) {
    if (g < y.K) c.rowsum[g] = sh[0];
    else if (g < y.K + y.M) c.colsum[g - y.K] = sh[0];
    else *c.sy = sh[0];
  }
}

// the multiplication terms, one thread each.  Segment 0 (3K + M - 2 terms), paired with -g2:
// rho_j Delta_j C_j; (sum of Delta over the subvectors whose sibling is D node (h, s)) D;
// (sum of the column weights over the upper half of W's range) W; -(sum delta y*) g1.
// Segment 1 + d (2^d terms), paired with vk_{l_M - 1 - d}: (sum over W's range) W.
__global__ void __launch_bounds__(TPB) kva_terms(VACtx c) {
  const PLayout &y = c.y;
  const uint64_t K = y.K, M = y.M, T0 = 3 * K + M - 2;
  uint64_t id = gtid();
  if (id >= T0 + M - 1) return;
  g1_aff base;
  fe k = fe_zero();
  if (id < K) {
    base = c.Cj[id];
    k = fr_mul(c.rho[id], c.rowsum[id]);
  } else if (id < 3 * K - 2) {
    uint64_t n = id - K, s;
    uint32_t h;
    d_node(n, K, h, s);
    base = c.Dn[n];
    uint64_t j0 = (s ^ 1) << h;
    for (uint64_t j = j0; j < j0 + (1ull << h); j++) k = fr_add(k, c.rowsum[j]);
  } else if (id < T0 - 1 || id >= T0) {
    bool upper = id < T0;
    uint64_t w = upper ? id - (3 * K - 2) : id - T0, p;
    uint32_t d;
    w_node(w, d, p);
    base = c.Wn[w];
    uint64_t len = 1ull << (y.lM - d), lo = p * len + (upper ? len / 2 : 0), hi = (p + 1) * len;
    for (uint64_t a = lo; a < hi; a++) k = fr_add(k, c.colsum[a]);
  } else {
    base = {fe_const(bn::G1X), fe_const(bn::G1Y)};
    k = fr_sub(fe_zero(), *c.sy);
  }
  c.bases[id] = base;
  c.scal[id] = k;
}

// a workgroup per segment: the sum of its products, and the pairing inputs
__global__ void __launch_bounds__(256) kva_segsum(VACtx c) {
  const PLayout &y = c.y;
  __shared__ g1_jac sh[256];
  const uint64_t T0 = 3 * y.K + y.M - 2;
  uint32_t g = blockIdx.x;
  if (g > y.lM) return;
  const int t = threadIdx.x;
  uint64_t lo = g == 0 ? 0 : T0 + (1ull << (g - 1)) - 1, len = g == 0 ? T0 : 1ull << (g - 1);
  g1_jac acc = jac_inf<OpsG1>();
  for (uint64_t q = t; q < len; q += 256) acc = jac_madd(acc, c.prod[lo + q]);
  sh[t] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) sh[t] = jac_add(sh[t], sh[t + s]);
    __syncthreads();
  }
  if (t == 0) {
    c.pp[g] = jac_to_aff(sh[0]);
    g2_aff g2 = {f2_const(bn::G2X0, bn::G2X1), f2_const(bn::G2Y0, bn::G2Y1)};
    c.pq[g] = g == 0 ? aff_neg(g2) : c.vk[y.lM - g];  // segment 1 + d: vk_{l_M - 1 - d}
  }
}

__global__ void __launch_bounds__(64) kva_check(VACtx c) {
  if (gtid() != 0) return;
  const fe *e = reinterpret_cast<const fe *>(c.E);
  bool one = fe_eq(e[0], f_one<FpP>());
  for (int q = 1; q < 12; q++) one = one && fe_is_zero(e[q]);
  if (one) atomicOr(c.flags, VFLAG_ACCEPT);
}

namespace kva {
uint64_t nterms(const VACtx &c) { return 3 * c.y.K + 2 * c.y.M - 3; }
void serialize(const PSCtx &c, hipStream_t st) {
  const uint64_t n = c.y.nb * (c.y.b + 26ull * c.y.lK + 5) + 2 * c.y.K - 2 + c.y.M - 1;
  const ProofGrid g = proof_grid(c.y.N);
  if (reinterpret_cast<uintptr_t>(c.out) & 15) {
    L1(kps_first<false>, n, c);
    LAUNCH(kps_copy<false>, dim3(g.x, g.y), dim3(256), 0, c);
  } else {
    L1(kps_first<true>, n, c);
    LAUNCH(kps_copy<true>, dim3(g.x, g.y), dim3(256), 0, c);
  }
}
void decode(const VACtx &c, hipStream_t st) { L1(kva_decode, 3 * c.y.K + c.y.M + 9, c); }
void roots(const VACtx &c, hipStream_t st) { L1(kva_roots, c.y.N, c); }
void rho(const VACtx &c, hipStream_t st) { LAUNCH(kva_rho, dim3((unsigned)((c.y.K + 63) / 64)), dim3(64), 0, c); }
void same(const VACtx &c, hipStream_t st) {
  const ProofGrid g = proof_grid(c.y.N);
  LAUNCH(kva_same, dim3(g.x, g.y), dim3(256), 0, c);
}
void proof(const VACtx &c, hipStream_t st) { L1(kva_proof, c.y.N, c); }
void sums(const VACtx &c, hipStream_t st) { LAUNCH(kva_sums, dim3((unsigned)(c.y.K + c.y.M + 1)), dim3(256), 0, c); }
void terms(const VACtx &c, hipStream_t st) { L1(kva_terms, nterms(c), c); }
void segsum(const VACtx &c, hipStream_t st) { LAUNCH(kva_segsum, dim3(c.y.lM + 1), dim3(256), 0, c); }
void check(const VACtx &c, hipStream_t st) { LAUNCH(kva_check, dim3(1), dim3(64), 0, c); }
}  // namespace kva

// ------------------------------------------------------------------ evaluation proof at a point
// Verifier of the evaluation proof (section 4.3): FC.BVerify of C_F = <C, T(r_L)> on the dense
// query b = r_0 T (faster verifier), then PC.Verify of F at r_R:
//   e(C_F - y g1, g2) = prod_d e(W_d, (s_var - r_var) g2),  var = l_M - 1 - d.
// The pairs and the final equalities are laid out as for one opening proof (kv_compare).

// one thread per item: v_l, pi_v, then C_F, the rounds' points, A_l and W, then the rounds' and C's
// coefficients, y and the point
__device__ __host__ uint32_t kve_items(uint32_t l, uint32_t lM, uint32_t L) { return 2 + (1 + 2 * l + 1 + lM) + (24 * l + 1 + 12 + L); }
__global__ void __launch_bounds__(TPB) kve_decode(VECtx c) {
  uint32_t id = (uint32_t)gtid();
  const uint32_t l = c.lK, lM = c.lM;
  if (id >= kve_items(l, lM, c.L)) return;
  const uint8_t *rounds = c.proof + 32, *tail = rounds + 832ull * l;
  Item it;
  if (id < 2) it = item(IT_G2, tail + 32 + 64 * id, id ? c.piv : c.vl);
  else if ((id -= 2) < 1) it = item(IT_G1, c.proof, c.CF);
  else if ((id -= 1) < 2 * l) it = item(IT_G1, rounds + 832ull * (id / 2) + (id % 2 ? 800 : 384), (id % 2 ? c.Rg1 : c.Lg1) + id / 2);
  else if ((id -= 2 * l) < 1) it = item(IT_G1, tail, c.Al);
  else if ((id -= 1) < lM) it = item(IT_G1, tail + 192 + 32 * id, c.W + id);
  else if ((id -= lM) < 24 * l) {
    const uint32_t r = id / 24, side = id / 12 % 2;
    it = item_gt(rounds + 832ull * r + 416 * side, (side ? c.Rgt : c.Lgt) + r, id % 12);
  } else if ((id -= 24 * l) < 1) it = item(IT_FR, tail + 160, c.y);
  else if ((id -= 1) < 12) it = item_gt(c.Cb, c.C, id, VFLAG_BAD_INPUT);
  else it = item(IT_FR_LE, c.rle + 32 * (id - 12), c.r + (id - 12), VFLAG_BAD_INPUT);
  decode_item(it, c.flags);
}

// r_0 (thread 0), the challenges x_j, z, f_v(z), b_l = r_0 sum_j T_j prod_k (x_k^{-1})^{bit_{l-k}(j)}
// as a tree, and the jobs (one workgroup)
__global__ void __launch_bounds__(256) kve_transcript(VECtx c) {
  const int tid = threadIdx.x;
  const uint32_t l = c.lK, lM = c.lM;
  __shared__ fe part[256];
  __shared__ fe s_r0, s_z;
  __shared__ uint32_t lds[sha::SCHED_WORDS + 512];
  if (tid == 0) {
    sha::Hasher hs;
    hs.init();
    hs.str(DSTR_EVAL);
    hs.gt(*c.C);
    for (int k = (int)c.L - 1; k >= 0; k--) hs.field<FpR>(c.r[k]);
    hs.g1(*c.CF);
    uint32_t sigma[8];
    hs.final(sigma);
    sha::Hasher hx;
    sha::xmd_begin(hx);
    for (int w = 0; w < 8; w++) hx.word(sigma[w]);
    hx.u64(0);
    s_r0 = sha::xmd_finish_fr(hx, DSTR_EVAL);
  }
  const fe z = challenge_chain(c, l, lds, c.g2s);
  if (tid == 0) s_z = z;
  __syncthreads();
  fe acc = fe_zero();
  for (uint64_t j = tid; j < c.K; j += 256) {
    fe term = c.T[j];
    for (uint32_t k = 1; k <= l; k++)
      if ((j >> (l - k)) & 1) term = fr_mul(term, c.xinv[k - 1]);
    acc = fr_add(acc, term);
  }
  part[tid] = acc;
  __syncthreads();
  for (int sft = 128; sft > 0; sft >>= 1) {
    if (tid < sft) part[tid] = fr_add(part[tid], part[tid + sft]);
    __syncthreads();
  }
  const g1_aff g1 = {fe_const(bn::G1X), fe_const(bn::G1Y)};
  for (uint32_t q = tid; q < 2 * l + 4; q += 256) {
    g1_aff base = g1;
    fe k;
    if (q < 2 * l) {
      uint32_t j = q / 2;
      if (q % 2 == 0) { base = c.Lg1[j]; k = c.x[j]; }
      else { base = c.Rg1[j]; k = c.xinv[j]; }
    } else if (q == 2 * l) {
      base = *c.Al; k = fr_mul(s_r0, part[0]);
    } else if (q == 2 * l + 1) {
      base = *c.CF; k = s_r0;
    } else if (q == 2 * l + 2) {
      k = *c.y;
    } else {
      k = s_z;
    }
    c.mb[q] = base;
    c.ms[q] = k;
  }
  for (uint32_t d = tid; d < lM; d += 256) c.g2s[1 + d] = c.r[lM - 1 - d];
  for (uint32_t q = tid; q < 2 * l; q += 256) {
    c.gts[q] = (q % 2 == 0) ? c.x[q / 2] : c.xinv[q / 2];
    c.gtb[q] = (q % 2 == 0) ? c.Lgt[q / 2] : c.Rgt[q / 2];
  }
}

// point sums and the pairs, a thread for each point (blockIdx.x 0: on G1, 1: on G2)
__global__ void __launch_bounds__(256) kve_assemble(VECtx c) {
  const uint32_t l = c.lK, lM = c.lM, tid = threadIdx.x;
  const g1_aff g1 = {fe_const(bn::G1X), fe_const(bn::G1Y)};
  const g2_aff g2 = {f2_const(bn::G2X0, bn::G2X1), f2_const(bn::G2Y0, bn::G2Y1)};
  // pairs: (A_l, v_l) | (beta g1 - z g1, pi_v), (-g1, v_l - f_v(z) g2) | (C_F - y g1, -g2), (W_d, (s - r)_var g2)
  if (blockIdx.x == 0) {
    if (tid == 0) {
      g1_jac acc = jac_from_aff(c.mo[2 * l + 1]);  // r_0 C_F
      for (uint32_t u = 0; u < 2 * l; u++) acc = jac_madd(acc, c.mo[u]);
      *c.Cg1 = jac_to_aff(acc);
      *c.bA = c.mo[2 * l];
    } else if (tid == 64 || tid == 65) {
      const bool p0 = tid == 65;
      c.pp[p0 ? 3 : 1] = jac_to_aff(jac_madd(jac_from_aff(p0 ? *c.CF : *c.g1beta), aff_neg(c.mo[2 * l + (p0 ? 2 : 3)])));
      c.pq[p0 ? 3 : 1] = p0 ? aff_neg(g2) : *c.piv;
    } else if (tid == 128) {
      c.pp[0] = *c.Al; c.pq[0] = *c.vl;
      c.gto[2 * l] = *c.C;
    }
    for (uint32_t q = tid; q < 2 * l; q += 256) c.gto[q] = c.gtp[q];
    return;
  }
  for (uint32_t q = tid; q < 1 + lM; q += 256) {
    const g2_aff Q = jac_to_aff(jac_madd(jac_from_aff(q == 0 ? *c.vl : c.vk[lM - q]), aff_neg(c.g2o[q])));
    c.pp[q == 0 ? 2 : 3 + q] = q == 0 ? aff_neg(g1) : c.W[q - 1];
    c.pq[q == 0 ? 2 : 3 + q] = Q;
  }
}

namespace kve {
void decode(const VECtx &c, hipStream_t st) { L1(kve_decode, kve_items(c.lK, c.lM, c.L), c); }
void transcript(const VECtx &c, hipStream_t st) { LAUNCH(kve_transcript, dim3(1), dim3(256), 0, c); }
void assemble(const VECtx &c, hipStream_t st) { LAUNCH(kve_assemble, dim3(2), dim3(256), 0, c); }
}  // namespace kve

// ------------------------------------------------------------------ all sub-array proofs at once
// A workgroup per subvector j: its proof against the first proof of its batch (16-byte words;
// honest proofs of a batch are equal), and entry j of its block against the commitment
// recomputed from m_j.  Proofs that differ join the list checked alone.
__global__ void __launch_bounds__(256) ksa_check(const uint8_t *proofs, uint64_t K, uint32_t b, uint64_t nb,
                                                 uint64_t len_full, uint64_t len_last, const g1_aff *Cre,
                                                 uint64_t *oddlist, uint32_t *oddcnt, int *flags) {
  __shared__ int diff;
  uint64_t j = blockIdx.x;
  if (j >= K) return;
  const int t = threadIdx.x;
  uint64_t k = j / b, j0 = k * b, len = k == nb - 1 ? len_last : len_full;
  const uint8_t *P = proofs + k * (uint64_t)b * len_full + (j - j0) * len;
  const uint8_t *R = proofs + k * (uint64_t)b * len_full;
  if (t == 0) diff = 0;
  __syncthreads();
  bool d = false;
  if (j != j0) {
    const uint4 *p4 = reinterpret_cast<const uint4 *>(P), *r4 = reinterpret_cast<const uint4 *>(R);
    for (uint64_t q = t; q < len / 16; q += 256) {
      uint4 u = p4[q], v = r4[q];
      d |= u.x != v.x || u.y != v.y || u.z != v.z || u.w != v.w;
    }
  }
  if (d) atomicOr(&diff, 1);
  __syncthreads();
  if (t != 0) return;
  g1_aff e;
  bool ok = decompress(P + 32 * (j - j0), false, &e, nullptr);
  if (!ok || !fe_eq(e.x, Cre[j].x) || !fe_eq(e.y, Cre[j].y)) atomicOr(flags, VFLAG_BAD_PROOF);
  if (diff) oddlist[atomicAdd(oddcnt, 1u)] = j;
}

namespace ksa {
void check(const uint8_t *proofs, uint64_t K, uint32_t b, uint64_t nb, uint64_t len_full, uint64_t len_last,
           const g1_aff *Cre, uint64_t *oddlist, uint32_t *oddcnt, int *flags, hipStream_t st) {
  LAUNCH(ksa_check, dim3((unsigned)K), dim3(256), 0, proofs, K, b, nb, len_full, len_last, Cre, oddlist, oddcnt, flags);
}
}  // namespace ksa
