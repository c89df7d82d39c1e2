// Workgroup-cooperative straight-line-program engine (device only, packed field layout).
//
// A workgroup of a few wavefronts runs programs generated by gen_slp.py: sequences of levels,
// each a set of independent base-field operations on field elements held in LDS slots.  A pair
// of lanes executes an operation, 32 operations a wavefront:
//   MUL  dst = (sum_i k_i x_i) (sum_i l_i y_i)   each lane forms one factor, the lanes exchange
//                                                them and form the product
//   LIN  dst = sum_i k_i x_i                     each lane sums half of the terms
// so additions feeding a product are folded into the product's lanes.  Slots hold field
// elements as 9 limbs of 29 bits: every term and every partial product is one 32 x 32
// multiply-add into a 64-bit column.  A level ends in a barrier; within a level no operation
// writes a slot that another one reads, so the wavefronts need none in between.
//
// What bounds it: a level's time is the instruction stream of one wavefront (about 4 cycles an
// instruction; the Montgomery product alone is 231 of them, 0.39 us), so a level is split
// where it is free of dependences: the two factors of a product run on two lanes, a level's
// operations on as many wavefronts (SIMDs) as it takes.
#pragma once
#include "field.hpp"
#include "slp_progs.hpp"

namespace slp {

// A slot: 9 limbs of 29 bits (little-endian, normalized), the same integer as the
// 8 x 32-bit Montgomery form used elsewhere (R = 2^256); words 9..11 pad to 48 bytes.
struct alignas(16) f29 {
  uint32_t l[12];
};
#define SLP_M29 0x1fffffffu

__host__ __device__ __forceinline__ f29 to29(const fe &x) {
  f29 r;
#pragma unroll
  for (int j = 0; j < 9; j++) {
    int b = 29 * j, w = b >> 5, s = b & 31;
    uint32_t v = x.l[w] >> s;
    if (s > 3 && w + 1 < 8) v |= x.l[w + 1] << (32 - s);
    r.l[j] = v & SLP_M29;
  }
  r.l[9] = r.l[10] = r.l[11] = 0;
  return r;
}

__host__ __device__ __forceinline__ fe from29(const f29 &x) {
  fe r;
#pragma unroll
  for (int w = 0; w < 8; w++) {
    int b = 32 * w, j = b / 29, s = b % 29;
    uint32_t v = x.l[j] >> s;
    if (j + 1 < 9) v |= x.l[j + 1] << (29 - s);
    if (s > 26 && j + 2 < 9) v |= x.l[j + 2] << (58 - s);
    r.l[w] = v;
  }
  return r;
}

// Values in slots are signed and "almost reduced": |x| < 1.2 p, limbs 0..7 signed and within 2^30 +
// 2^18 ("loose": a sum's slot adds two reduced halves limb by limb, each in [-2^17, 2^29 + 2^17]), the top
// limb signed.  Only kernel outputs are made canonical.  So no offset is carried through the sums, a
// negation is the negated limbs, and the carries of a sum are taken once, all columns side by side.
//
// red29: V = sum c_j 2^{29 j} minus its rounded quotient by p.  The coefficient magnitudes of
// a sum add up to less than 2^15, so every column is below 2^45 + 2^33 (V below 2^16 p).  The
// quotient is estimated in single precision from the top column: the columns below it move V / p
// by less than 0.021, the dropped low bits by 2^-13, the roundings by less than 0.01 for
// quotients below 2^16.  The sum with 1.5 2^23 rounds it to the nearest integer, so
// |V - q p| < 0.54 p.
__host__ __device__ __forceinline__ int32_t neg_quotient29(int64_t top) {
  const float magic = 12582912.0f;
  const float f = __builtin_fmaf((float)(int32_t)(top >> 8), INVP240, magic);
  return (int32_t)(0x4B400000u - __builtin_bit_cast(uint32_t, f));
}
__host__ __device__ __forceinline__ f29 red29(const int64_t *c) {
  const int32_t nq = neg_quotient29(c[8]);
  f29 o;
  int64_t v[8];
#pragma unroll
  for (int j = 0; j < 8; j++) v[j] = c[j] + (int64_t)nq * (int32_t)P29[j];
  o.l[8] = (uint32_t)c[8] + (uint32_t)nq * P29[8] + (uint32_t)(v[7] >> 29);
#pragma unroll
  for (int j = 0; j < 8; j++) o.l[j] = ((uint32_t)v[j] & SLP_M29) + (j ? (uint32_t)(v[j - 1] >> 29) : 0u);
  o.l[9] = o.l[10] = o.l[11] = 0;
  return o;
}

// the same value with limbs 0..7 in [0, 2^29)
__host__ __device__ __forceinline__ f29 norm29(const f29 &x) {
  f29 o;
  int32_t carry = 0;
#pragma unroll
  for (int j = 0; j < 8; j++) {
    const int32_t v = (int32_t)x.l[j] + carry;
    o.l[j] = (uint32_t)v & SLP_M29;
    carry = v >> 29;
  }
  o.l[8] = x.l[8] + (uint32_t)carry;
  o.l[9] = o.l[10] = o.l[11] = 0;
  return o;
}

// x + y (limbs 0..7 in [0, 2^29) again) for slots that products write, the constants 0 and 1, and sums of
// such; -x limb by limb (limbs are signed)
__host__ __device__ __forceinline__ f29 add29(const f29 &x, const f29 &y) {
  f29 o;
#pragma unroll
  for (int j = 0; j < 12; j++) o.l[j] = x.l[j] + y.l[j];
  return norm29(o);
}
__host__ __device__ __forceinline__ f29 neg29(const f29 &x) {
  f29 o;
#pragma unroll
  for (int j = 0; j < 12; j++) o.l[j] = 0u - x.l[j];
  return o;
}

// canonical residue of an almost-reduced value or a sum of up to four products (in (-2p, 5p)):
// x + 2p lies in (0, 7p), and 4p, 2p and p are taken off where they fit.  Limbs of x within 2^30 + 2^18:
// those of 2p are below 0.89 2^30, and the sums below 2^31
__host__ __device__ __forceinline__ f29 canon29(const f29 &x) {
  f29 y = x;
#pragma unroll
  for (int j = 0; j < 9; j++) y.l[j] += 2 * P29[j];
  y = norm29(y);
#pragma unroll
  for (int k = 2; k >= 0; k--) {
    f29 d = y;
#pragma unroll
    for (int j = 0; j < 9; j++) d.l[j] -= P29[j] << k;
    d = norm29(d);
    if ((int32_t)d.l[8] >= 0) y = d;
  }
  return y;
}
__host__ __device__ inline bool zero29(const f29 &x) {
  const f29 c = canon29(x);
  uint32_t t = 0;
  for (int j = 0; j < 9; j++) t |= c.l[j];
  return t == 0;
}

// keeps the instructions written before it ahead of those written after it
#ifdef __HIP_DEVICE_COMPILE__
#define SLP_ORDER() __builtin_amdgcn_sched_barrier(0)
#else
#define SLP_ORDER()
#endif

// Montgomery product with radix 2^29 over 9 limbs: a b 2^{-261} mod p for almost-reduced a and
// b, result in (-0.01 p, 1.01 p) with limbs 0..7 in [0, 2^29).  Products go into signed 64-bit
// columns without carries (the factors are reductions, limbs below 2^29 + 2^17, and each column
// stays below 2^62.5); the reduction clears one column at a time.  The order is fixed row by row: a multiply-add that needs the one before it issues
// after 8 cycles instead of 4, and left to itself the compiler sums each column in one
// dependent chain to save registers (1512 cycles a product against 930 in this order).
__host__ __device__ __forceinline__ f29 mont29(const f29 &a, const f29 &b) {
  int64_t c[18];
#pragma unroll
  for (int k = 0; k < 18; k++) c[k] = 0;
#pragma unroll
  for (int j = 0; j < 9; j++) c[j] = (int64_t)(int32_t)a.l[0] * (int32_t)b.l[j];
#pragma unroll
  for (int k = 0; k < 9; k++) {
    SLP_ORDER();
    const uint32_t t = (uint32_t)c[k] * PINV29;
    SLP_ORDER();
    if (k < 8) {
#pragma unroll
      for (int j = 0; j < 9; j++) c[k + 1 + j] += (int64_t)(int32_t)a.l[k + 1] * (int32_t)b.l[j];
    }
    SLP_ORDER();
    const int32_t m = (int32_t)(t & SLP_M29);
#pragma unroll
    for (int j = 0; j < 9; j++) c[k + j] += (int64_t)m * (int32_t)P29[j];
    SLP_ORDER();
    c[k + 1] += c[k] >> 29;
  }
  f29 o;
  int64_t carry = 0;
#pragma unroll
  for (int j = 0; j < 8; j++) {
    const int64_t v = c[9 + j] + carry;
    o.l[j] = (uint32_t)v & SLP_M29;
    carry = v >> 29;
  }
  o.l[8] = (uint32_t)(c[17] + carry);
  o.l[9] = o.l[10] = o.l[11] = 0;
  return o;
}

// Segment bases in bytes packed 16 bits apiece: bits [16 s, 16 s + 16) hold the base of segment
// s (segment 0 is absolute, so its base is 0).  Segments are 0..3.
__host__ __device__ __forceinline__ uint64_t seg_bases(uint32_t bx, uint32_t by, uint32_t bd) {
  return ((uint64_t)(bx * 48u) << 16) | ((uint64_t)(by * 48u) << 32) | ((uint64_t)(bd * 48u) << 48);
}

// byte address of the slot that term t names: its segment's base is one shift of the packed
// bases (bits 26..29 of a term are zero, so t >> 26 is 16 times the segment)
__host__ __device__ __forceinline__ uint32_t term_off(uint32_t t) { return (t & 0xfffu) << 4; }
__host__ __device__ __forceinline__ uint32_t term_addr(uint32_t t, uint64_t rel) {
  return term_off(t) + ((uint32_t)(rel >> (t >> 26)) & 0xffffu);
}

// signed 13-bit coefficient at bits 12..24 of a term
__host__ __device__ __forceinline__ int term_coef(uint32_t t) { return (int)(t << 7) >> 19; }

// a block descriptor's fields (gen_slp.py OpTable)
static constexpr uint32_t BLK_OFF = (1u << 19) - 1, BLK_T2 = 1u << 19, BLK_T4 = 1u << 20, BLK_T6 = 1u << 21,
                          BLK_T10 = 1u << 22, BLK_SEG = 1u << 23, BLK_MUL = 1u << 30, BLK_LIN = 1u << 31;
__host__ __device__ __forceinline__ int blk_ops(uint32_t d) { return (int)(d >> 24 & 63u); }
__host__ __device__ __forceinline__ int blk_terms(uint32_t d) {
  return d & BLK_T10 ? 14 : d & BLK_T6 ? 10 : d & BLK_T4 ? 6 : d & BLK_T2 ? 4 : 2;
}
// word i of lane l's record of the block
__host__ __device__ __forceinline__ uint32_t blk_word(const uint32_t *ops, uint32_t d, int l, int i) {
  return ops[4 * (d & BLK_OFF) + 256 * (i >> 2) + 4 * l + (i & 3)];
}

// One call of a sequence: the program's first descriptors (one per wavefront) and the packed
// segment bases
struct alignas(16) Call {
  uint32_t d[4];
  uint64_t rel, pad;
};
__host__ __device__ __forceinline__ Call call(int prog, int x = 0, int y = 0, int d = 0) {
  const ProgDesc &p = PROGS[prog];
  return Call{{p.d[0], p.d[1], p.d[2], p.d[3]}, seg_bases(x, y, d), 0};
}

static constexpr int MAX_CALLS = 128;

#ifdef __HIPCC__
typedef __attribute__((address_space(3))) f29 lds_f29;
typedef __attribute__((address_space(3))) Call lds_call;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;

// the 9 limbs of the slot at an LDS address (slots are 16-byte aligned)
__device__ __forceinline__ void get_slot(uint32_t addr, uint32_t *x) {
  const lds_u32x4 *p = (const lds_u32x4 *)(uintptr_t)addr;
  const u32x4 a = p[0], b = p[1];
  x[8] = ((const lds_u32 *)p)[8];
#pragma unroll
  for (int j = 0; j < 4; j++) {
    x[j] = a[j];
    x[4 + j] = b[j];
  }
}
__device__ __forceinline__ void put_slot(uint32_t addr, const f29 &r) {
  lds_u32x4 *p = (lds_u32x4 *)(uintptr_t)addr;
  p[0] = u32x4{r.l[0], r.l[1], r.l[2], r.l[3]};
  p[1] = u32x4{r.l[4], r.l[5], r.l[6], r.l[7]};
  ((lds_u32 *)p)[8] = r.l[8];
}

// the other lane's value of a pair
__device__ __forceinline__ uint32_t partner(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);  // quad_perm [1, 0, 3, 2]
}

// End of a level: the wavefront's slot writes are done, then the workgroup's.  (Operations
// fetched ahead stay in flight: the barrier waits for LDS only.)
template <int NW> __device__ __forceinline__ void level_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if (NW > 1) __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// base: the slots' LDS address; rel: the segment bases with it added
template <int N, bool SEG>
__device__ __forceinline__ void add_terms(uint32_t base, const uint32_t *w, uint64_t rel, int64_t *acc) {
  uint32_t x[N][9];
#pragma unroll
  for (int i = 0; i < N; i++) get_slot(SEG ? term_addr(w[i], rel) : term_off(w[i]) + base, x[i]);
#pragma unroll
  for (int i = 0; i < N; i++) {
    const int k = term_coef(w[i]);
    SLP_ORDER();
#pragma unroll
    for (int j = 0; j < 9; j++) acc[j] += (int64_t)k * (int32_t)x[i][j];
  }
  SLP_ORDER();
}
// the loads of up to six terms issue back to back, so that their latencies overlap; unused
// terms name slot 0 with coefficient 0
template <bool SEG>
__device__ __forceinline__ void add_record(uint32_t base, uint32_t d, const uint32_t *w, uint64_t rel, int64_t *acc) {
  if (!(d & BLK_T2)) {
    add_terms<2, SEG>(base, w + 2, rel, acc);
  } else if (!(d & BLK_T4)) {
    add_terms<4, SEG>(base, w + 2, rel, acc);
  } else {
    add_terms<6, SEG>(base, w + 2, rel, acc);
    if (d & BLK_T6) {
      add_terms<4, SEG>(base, w + 8, rel, acc);
      if (d & BLK_T10) add_terms<4, SEG>(base, w + 12, rel, acc);
    }
  }
}

// One wavefront's operations of a level (block descriptor d, this lane's record w); lanes past
// the block's operations do not come here.
__device__ __forceinline__ void run_block(uint32_t base, uint32_t d, const uint32_t *w, uint64_t rel) {
  const bool mul = term_coef(w[0]) == 1;
  const uint32_t dst = term_addr(w[0], rel);
  int64_t acc[9];
#pragma unroll
  for (int j = 0; j < 9; j++) acc[j] = 0;
  if (d & BLK_SEG) add_record<true>(base, d, w, rel, acc);
  else add_record<false>(base, d, w, rel, acc);
  f29 r = red29(acc);
  if (d & BLK_LIN) {
    if (!mul) {  // the sum of both lanes' halves
#pragma unroll
      for (int j = 0; j < 9; j++) r.l[j] += partner(r.l[j]);
    }
  }
  if (d & BLK_MUL) {
    f29 o;
#pragma unroll
    for (int j = 0; j < 9; j++) o.l[j] = partner(r.l[j]);
    if (mul) r = mont29(r, o);
  }
  if (!(threadIdx.x & 1)) put_slot(dst, r);
}

// Runs the calls cl[0 .. n), n > 0 (LDS), on the slots at LDS address `base` with all
// wavefronts of the workgroup.
//
// Records are fetched one level ahead, across calls too: a level's record names the next
// level's block, the last one's is 0, and a call's entry (read from LDS a call ahead) names
// the first.  The loop is written for the fewest scalar instructions, since one wavefront
// issues about one instruction in four cycles whatever its kind.
template <int NW> __device__ __forceinline__ void run_calls(uint32_t base, uint32_t list, int n) {
  static_assert(NW == 2 || NW == 4, "a call entry holds up to four descriptors");
  base = __builtin_amdgcn_readfirstlane(base);
  list = __builtin_amdgcn_readfirstlane(list);
  n = __builtin_amdgcn_readfirstlane(n);
  const uint32_t lane = threadIdx.x & 63, half = lane >> 1;
  const uint32_t wave4 = threadIdx.x >> 6 << 2;  // where this wavefront's descriptor is in an entry
  const uint32_t end = list + 32u * n;
  const uint64_t base4 = base * 0x0001000100010001ull;
  uint32_t n_ent = list;  // entry after the next level's call
  uint32_t ahead_d = *(const lds_u32 *)(uintptr_t)(list + wave4);  // that entry
  u32x2 ahead_rel = *(const lds_u32x2 *)(uintptr_t)(list + 16);
  uint32_t nd = 0;     // the next level: descriptor,
  uint64_t n_rel = 0;  // segment bases
  auto next_call = [&]() {
    nd = __builtin_amdgcn_readfirstlane(ahead_d);
    n_rel = base4 + (__builtin_amdgcn_readfirstlane(ahead_rel[0]) | (uint64_t)__builtin_amdgcn_readfirstlane(ahead_rel[1]) << 32);
    n_ent += 32;
    if (n_ent < end) {
      ahead_d = *(const lds_u32 *)(uintptr_t)(n_ent + wave4);
      ahead_rel = *(const lds_u32x2 *)(uintptr_t)(n_ent + 16);
    }
  };
  // (all 64 lanes read, those past the block's operations to no effect; straight into the
  // registers that the level reads, since a move of a loaded word here would wait for it)
  auto load = [&](u32x4 *nw) {
    const char *o = (const char *)OPS + (((nd & BLK_OFF) << 4) + (lane << 4));
    nw[0] = *(const u32x4 *)o;
    if (nd & BLK_T2) {
      nw[1] = *(const u32x4 *)(o + 1024);
      if (nd & BLK_T6) {
        nw[2] = *(const u32x4 *)(o + 2048);
        if (nd & BLK_T10) nw[3] = *(const u32x4 *)(o + 3072);
      }
    }
  };
  // one level from cw, the next fetched to nw; true at the end of the run
  auto step = [&](const u32x4 *cw, u32x4 *nw) -> bool {
    uint32_t w[LANE_TERMS_MAX + 2];
#pragma unroll
    for (int i = 0; i < LANE_TERMS_MAX + 2; i++) w[i] = cw[i >> 2][i & 3];
    const uint32_t d = nd;
    const uint64_t rel = n_rel;
    nd = __builtin_amdgcn_readfirstlane(w[1]);
    if (!nd && n_ent < end) next_call();
    if (nd) load(nw);
    if (half < (uint32_t)blk_ops(d)) run_block(base, d, w, rel);
    level_sync<NW>();
    return nd == 0;
  };
  u32x4 wa[4] = {}, wb[4] = {};
  next_call();
  load(wa);
  while (!step(wa, wb) && !step(wb, wa)) {}
}

// the same as a function: called, it saves and restores some sixty vector registers a lane in
// scratch memory
template <int NW> __device__ __noinline__ void run_calls_fn(uint32_t base, uint32_t list, int n) { run_calls<NW>(base, list, n); }

// Device context for control code shared with the host model: the workgroup's slots and a list
// of calls in LDS.  (cl: MAX_CALLS entries for lists and one more for single calls; a context in
// line that only runs single calls has one entry.)  A kernel
// with one place that runs calls has the engine in line, one with several calls it: with the
// call's scratch traffic a launch of 2^15 F_p12 products took 1.98 ms, in line it takes a
// quarter of that.
template <int NW, bool INLINE = false> struct DevCtx {
  f29 *S;
  Call *cl;
  __device__ int lane() const { return threadIdx.x; }
  __device__ int lanes() const { return 64 * NW; }
  __device__ void sync() { __syncthreads(); }
  // calls cl[first .. n)
  __device__ void run_list(int first, int n) {
    __syncthreads();
    if (first >= n) return;
    const uint32_t base = (uint32_t)(uintptr_t)(lds_f29 *)S, list = (uint32_t)(uintptr_t)((lds_call *)cl + first);
    if (INLINE) run_calls<NW>(base, list, n - first);
    else run_calls_fn<NW>(base, list, n - first);
  }
  // slot dst = the inverse of v (the same in all lanes; 0 for 0), by division steps on the scalar
  // unit; false if v is 0
  __device__ bool invert(int dst, const f29 &v) {
    const fe r = f_inv_uniform<FpP>(from29(canon29(v)), bn::P_R3);
    if (threadIdx.x == 0) S[dst] = to29(r);
    __syncthreads();
    return !fe_is_zero(r);
  }
  __device__ void run(int prog, int bx, int by, int bd) {
    // (the list's extra entry; a context in line has no other)
    const int e = INLINE ? 0 : MAX_CALLS;
    __syncthreads();
    if (threadIdx.x == 0) cl[e] = call(prog, bx, by, bd);
    run_list(e, e + 1);
  }
};
#endif

// Host model: every operation of a level reads before any writes.
inline void run_host(f29 *S, const Call &c) {
  const uint64_t rel = c.rel;
  f29 r[128];
  uint32_t dst[128];
  uint32_t d[4] = {c.d[0], c.d[1], c.d[2], c.d[3]};
  while (d[0]) {
    int n = 0;
    for (int v = 0; v < 4 && d[v]; v++) {
      const int T = blk_terms(d[v]);
      for (int i = 0; i < blk_ops(d[v]); i++, n++) {
        int64_t acc[2][9];
        for (int h = 0; h < 2; h++) {
          for (int j = 0; j < 9; j++) acc[h][j] = 0;
          for (int t = 0; t < T; t++) {
            const uint32_t w = blk_word(OPS, d[v], 2 * i + h, 2 + t);
            const f29 &x = S[term_addr(w, rel) / 48];
            for (int j = 0; j < 9; j++) acc[h][j] += (int64_t)term_coef(w) * (int32_t)x.l[j];
          }
        }
        const uint32_t head = blk_word(OPS, d[v], 2 * i, 0);
        r[n] = red29(acc[0]);
        const f29 o = red29(acc[1]);
        if (term_coef(head) == 1) r[n] = mont29(r[n], o);
        else
          for (int j = 0; j < 9; j++) r[n].l[j] += o.l[j];
        dst[n] = term_addr(head, rel) / 48;
      }
      d[v] = blk_word(OPS, d[v], 0, 1);
    }
    for (int i = 0; i < n; i++) S[dst[i]] = r[i];
  }
}

inline void run_host(f29 *S, int prog, int bx, int by, int bd) { run_host(S, call(prog, bx, by, bd)); }

struct HostCtx {
  f29 *S;
  int l = 0;
  Call list[MAX_CALLS + 1];
  Call *cl = list;
  void run(int prog, int bx, int by, int bd) { run_host(S, prog, bx, by, bd); }
  void sync() {}
  int lane() const { return l; }
  int lanes() const { return 1; }
  void run_list(int first, int n) {
    for (int e = first; e < n; e++) run_host(S, cl[e]);
  }
};

}  // namespace slp
