"""FlexProofs commit + OpenAll on one MI355X: benchmark.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline] [--no-extra]

A step is one pass of the whole hot path over one seeded synthetic vector:
VC.Commit (PST commitments of the K subvectors, FC commitment) and VC.OpenAll
(all ceil(K/b) FC batch proofs, the Merkle tree, the randomized folding tree and
HyperEval on g*).  The workload is N = 2^16 with b = log^2 N = 256 and uniform
32-bit entries (the paper's headline all-proofs configuration); `value` is the
median all-N-proofs (OpenAll) time in ms.  The N = 2^20, b = 400 full-width
workload and the commitment MSM rate are reported under "extra".

Per-kernel durations come from HIP events recorded by the library on its launch
stream during the timed steps; the roofline object is for the kernel with the
largest share of the timed region.
"""
from __future__ import annotations

import argparse
import ctypes
import json
import os
import statistics
import sys
import time

# hardware queues for the library's streams (as the package sets it), before any device use
if int(os.environ.get("GPU_MAX_HW_QUEUES", "4") or 4) < 16:
    os.environ["GPU_MAX_HW_QUEUES"] = "16"

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "all-N-proofs time (ms) at N=2^16,b=log²N and N=2^20; MSM points/s"
PEAK_MAD_TOPS = 256 * 64 * 2.4e9 / 2 / 1e12   # v_mad_u64_u32 issues at half rate: 19.66 T multiply-adds/s
PEAK_HBM_GBS = 8000.0
MADS_PER_FMUL = 136                        # the price of a field multiplication: an 8x32-bit CIOS product
                                           # (64 + 64 + 8; the kernels' own, on 9x29-bit limbs, have 81 + 81)
AHEAD_MAX_PAIRS = 4096                     # the library's switch to next-round terms (batches x K)
AHEAD_FEW_PAIRS, AHEAD_FEW_BATCHES = 1024, 4
# HBM bytes per launch from rocprofv3 FETCH_SIZE / WRITE_SIZE, scaled by a reference copy
# (profiles/ks_final_exp2_n16_b256_hbm_counters.md): of the programs those kernels run now
TRAFFIC_BYTES = {"ks_final_exp2": round((4600.9 * 2.000 + 2.2 * 1.000) * 1024),
                 "ks_oa_pterms": round((7445.6 * 2.000 + 910.5 * 1.000) * 1024)}
# additions of the reduction of a block's buckets: with 128 buckets the two sums of each (128), the suffix
# sums (7 x 128 - 127) and their sum (127); with 256 places the suffix sums (8 x 256 - 255) and their sum (255)
REDUCE_128, REDUCE_256 = 128 + 769 + 127, 1793 + 255
FOLD_SPLIT_MAX = 256                       # folds of at most this many pairs run split in four parts
DIRECT_MIN = 512                           # rounds of more pairs than this run direct in the ahead mode
KZG_SPLIT_MAX = 8192                       # KZG proofs of at most this many split jobs run split
LANE_MILLER_MIN = 4096                     # direct-round Miller loops of this many pairs run two lanes a pairing
LANE_MIN = 4096                            # direct-round terms and folds of this many run on single lanes


def takes_ahead(nb, K):
    return nb * K <= AHEAD_MAX_PAIRS and (nb <= AHEAD_FEW_BATCHES or nb * K <= AHEAD_FEW_PAIRS)


def op_costs():
    """Field multiplications per operation: formulas of the one-lane and eight-lane layouts
    (host build count) and the engine's programs (Montgomery products in the tables)."""
    L = ctypes.CDLL(os.path.join(ROOT, "paper_2601_03031_amd", "lib", "libvc_hostcheck.so"))
    L.hc_count.restype = ctypes.c_uint64
    L.hc_engine_muls.restype = ctypes.c_uint64
    names = ["miller", "final_exp", "g1_mul", "g2_mul", "g1_add", "g1_madd", "g2_add", "g2_madd",
             "g1_dbl", "g2_dbl", "f12_mul", "g1_to_aff", "g2_to_aff"]
    c = {n: int(L.hc_count(i)) for i, n in enumerate(names)}
    e = [int(L.hc_engine_muls(i)) for i in range(17)]
    c["e_miller"], c["e_final_exp"], c["e_f12_mul"] = e[0], e[1], e[8]
    # GLS scalar multiplication on G2: psi images, table, then per bit of the 65-bit
    # split scalars one doubling and (with probability 15/16) one table addition
    c["e_g2_mul"] = e[2] + e[3] + 64 * e[4] + 60 * e[5]
    c["e_g2_madd"], c["e_g2_to_aff"] = e[6], e[7]
    # GLV scalar multiplication on G1 (128-bit split scalars in 2-bit joint windows): table,
    # then per window two doublings and (with probability 15/16) an addition
    c["e_g1_mul"] = e[9] + 60 * e[10] + 4 * e[11]
    c["e_g1_madd"], c["e_g1_to_aff"] = e[12], e[13]
    # G_T power through the 4-dimensional split (65-bit): Frobenius images, 11 table
    # products, then per bit one cyclotomic squaring and (15/16) one product
    c["e_gt_pow"] = e[15] + 11 * e[8] + 64 * e[14] + 60 * e[8]
    c["e_g1_tab"], c["e_g1_dbl2"], c["e_csqr"], c["e_gt_tab"] = e[9], e[11], e[14], e[15] + 11 * e[8]
    c["e_g1_add"], c["e_g2_add"], c["e_g2_dbl"] = e[16], e[5], e[4]
    # one of the four parts of a split multiplication: G1 on a 32-bit chunk (16 windows),
    # G2 on a 16-bit chunk (16 bits); then the last part adds the four partial results and A
    c["e_g1_part"] = e[9] + 15 * e[10] + e[11]
    c["e_g2_part"] = e[2] + e[3] + 16 * e[4] + 15 * e[5]
    c["f12_sqr"] = int(L.hc_count(13))
    return c


MILLER_SQUARINGS = 63   # F_p12 squarings of the Miller loop over 6u+2 (its 65-bit NAF-free binary form)


def fc_support_terms(K, lo, t):
    """non-zero terms of the sparse G1 parts <A_R, b_L> and <A_L, b_R> over the rounds of one
    FC batch opening whose exponent vector b is supported on [lo, lo + t) (section 3, Eq. (b)
    and (folding)): the support folds to {s mod h} each round"""
    sup, n, h = set(range(lo, lo + t)), 0, K
    while h > 1:
        h //= 2
        n += sum(1 for s in sup if s < 2 * h)   # every support index meets one side of the round
        sup = {s % h for s in sup}
    return n


def method_work(L, b, limbs, c):
    """Algorithmic field multiplications of the method (the operation counts of the paper's
    algorithms at this size: commit MSM, FC.Commit, Protocol 1 Step 1 with round 1's pairings
    shared by all batches, Step 2), priced with the one-lane formulas of the library (host
    build count): a multi-pairing of h pairs costs h Miller loops without their F_p12
    squarings plus one set of squarings; an MSM of n terms over fixed bases with 8-bit windows
    costs one mixed addition per non-zero digit and a running-sum bucket reduction
    (2 x 255 additions per bucket set); every other MSM is priced as its scalar
    multiplications.  Returns per-phase and per-kernel totals."""
    import numpy as np
    lK, lM = L // 2, L - L // 2
    K, M, N = 1 << lK, 1 << lM, 1 << L
    nb = (K + b - 1) // b
    sq = MILLER_SQUARINGS * c["f12_sqr"]
    pair = c["miller"] - sq
    mpair = lambda h: h * pair + sq               # one multi-pairing of h pairs
    nz_digits = int(np.count_nonzero(np.ascontiguousarray(limbs).view(np.uint8)))
    S = min(M, 8192 // (4 if int(limbs[:, 1:].max()) == 0 else 32))
    msm = nz_digits * c["g1_madd"] + K * ((M + S - 1) // S) * 510 * c["g1_add"]
    fc_commit = mpair(K) + c["final_exp"]
    rounds = [(j, K >> j) for j in range(1, lK + 1)]
    # Miller work and final exponentiations per round (round 1 shared by every batch)
    miller = {j: (2 * mpair(h) if j == 1 else nb * 2 * mpair(h)) for j, h in rounds}
    fexp = {j: (2 if j == 1 else 2 * nb) * c["final_exp"] for j, h in rounds}
    sparse = sum(fc_support_terms(K, k * b, min(b, K - k * b)) for k in range(nb)) * c["g1_mul"]
    fold_g1 = sum(nb * h for _, h in rounds) * (c["g1_mul"] + c["g1_madd"])
    fold_g2 = sum(nb * h for _, h in rounds) * (c["g2_mul"] + c["g2_madd"])
    nq = 2 * K - 2   # the KZG quotient's terms: a G2 MSM over the fixed SRS points h_m
    kzg = nb * (nq * 32 * 255 // 256 * c["g2_madd"] + -(-nq // 32) * 510 * c["g2_add"])
    step2 = K * c["g1_mul"] + (K - 1) * c["g1_add"] + lM * (M // 2) * c["g1_mul"] + N
    phases = {"commit_msm": msm, "fc_commit": fc_commit, "step1_miller": sum(miller.values()),
              "step1_final_exp": sum(fexp.values()), "step1_sparse_g1": sparse, "step1_fold_g1": fold_g1,
              "step1_fold_g2": fold_g2, "step1_kzg": kzg, "step2": step2}
    # attribution to the kernels that carry each part of the work in the library's schedule
    ahead = lK >= 2 and takes_ahead(nb, K)
    j0 = 2
    while j0 < lK and nb * (K >> j0) > DIRECT_MIN:
        j0 += 1
    direct = [j for j, _ in rounds if not ahead or j < j0]
    taken = [j for j, _ in rounds if ahead and j >= j0]
    by_kernel = {"k_msm_slices<lane::G1>": msm, "ks_miller": mpair(K),
                 "ks_oa_pterms": sum(miller[j] for j in taken),
                 "ks_final_exp2": sum(fexp[j] for j in taken),
                 "ks_final_exp": sum(fexp[j] for j in direct) + c["final_exp"]}
    wide = [j for j in direct if (1 if j == 1 else nb) * (K >> j) >= LANE_MILLER_MIN]
    by_kernel["kn_oa_miller"] = sum(miller[j] for j in wide)
    by_kernel["ks_oa_miller"] = sum(miller[j] for j in direct if j not in wide)
    return {"phases": phases, "open_all": sum(v for k, v in phases.items() if k not in ("commit_msm", "fc_commit")),
            "commit": msm + fc_commit, "by_kernel": {k: v for k, v in by_kernel.items() if v}}


def msm_work(limbs, K, M):
    """What the library's commit MSM executes: nonzero digits (mixed additions) and the additions of its
    blocks' reductions.  Entries of 256 bits take signed digits (a byte of the entry plus 128 in every
    byte, less 128) into 128 buckets with two sums each, 32-bit ones bytes into 255 buckets; a block sums
    up to 8 slices of a row (a power of two that leaves 1024 blocks) before it reduces them."""
    import numpy as np
    limbs = np.ascontiguousarray(limbs)
    full = int(limbs[:, 1:].max()) != 0
    S = min(M, 8192 // (32 if full else 4))
    nslice = -(-M // S)
    g = 1
    while g < 8 and nslice % (2 * g) == 0 and K * nslice // (2 * g) >= 1024:
        g *= 2
    if not full:
        return int(np.count_nonzero(limbs.view(np.uint8))), K * nslice // g * REDUCE_256
    add, carry, nz = np.uint64(0x8080808080808080), np.zeros(len(limbs), dtype=np.uint64), 0
    for q in range(4):
        t = limbs[:, q] + add
        c = t < add
        t = t + carry
        carry = (c | (t < carry)).astype(np.uint64)
        nz += int(np.count_nonzero(t.view(np.uint8) != 128))
    return nz, K * nslice // g * REDUCE_128


def work_model(L, b, limbs, costs):
    """Algorithmic field multiplications per kernel over one step (commit + open-all)."""
    lK, lM = L // 2, L - L // 2
    K, M, N = 1 << lK, 1 << lM, 1 << L
    nb = (K + b - 1) // b
    rounds = [K >> j for j in range(1, lK + 1)]
    digits, adds = msm_work(limbs, K, M)
    g1_fold = costs["e_g1_mul"] + costs["e_g1_madd"] + costs["e_g1_to_aff"]
    g2_fold = costs["e_g2_mul"] + costs["e_g2_madd"] + costs["e_g2_to_aff"]
    nq = 2 * K - 2
    w = {
        "k_msm_slices<lane::G1>": digits * costs["g1_madd"] + adds * costs["g1_add"],
        "ks_miller": K * costs["e_miller"],
        "kn_hyper_terms": lM * (M // 2) * costs["g1_mul"],
    }
    # KZG proof: with few terms, split multiplications; otherwise a G2 MSM over 8-bit windows
    # of the fixed SRS points (about 255/256 of the (term, window) pairs have a nonzero signed digit;
    # slices of 32 bases, or of 256 where those give 512 blocks); then the engine tree over the
    # partial sums
    if 4 * nb * nq <= KZG_SPLIT_MAX:
        w["ks_kzg_terms_split"] = 4 * nb * nq * costs["e_g2_part"]
        w["(ks_pt_tree<true, true>)"] = nb * (4 * nq - 1) * costs["e_g2_add"]
    else:
        slices = -(-nq // (256 if nb * -(-nq // 256) >= 512 else 32))
        group = 1
        while group < 8 and slices % (2 * group) == 0 and nb * slices // (2 * group) >= 1024:
            group *= 2
        w["k_msm_slices<lane::G2>"] = ((nb * nq * 32 * 255 // 256) * costs["g2_madd"]
                                       + nb * slices // group * REDUCE_128 * costs["g2_add"])
        w["(ks_pt_tree<true, false>)"] = nb * (slices - 1) * costs["e_g2_add"]
    if lK >= 2 and takes_ahead(nb, K):
        # rounds j < j0 direct (the device is full), rounds j >= j0 from terms of the arrays of
        # round j - 1 (q = K >> j)
        j0 = 2
        while j0 < lK and nb * (K >> j0) > DIRECT_MIN:
            j0 += 1
        direct = [K >> j for j in range(1, j0)]
        nbr = lambda h: 1 if h == K // 2 else nb   # round 1's pairings are computed once for all batches
        qs = [K >> j for j in range(j0, lK + 1)]
        split = [nb * h for h in rounds if nb * h <= FOLD_SPLIT_MAX]
        whole = [nb * h for h in rounds if nb * h > FOLD_SPLIT_MAX]
        g1_sum = 3 * costs["e_g1_add"] + costs["e_g1_madd"] + costs["e_g1_to_aff"]
        g2_sum = 3 * costs["e_g2_add"] + costs["e_g2_madd"] + costs["e_g2_to_aff"]
        w.update({
            "ks_oa_miller": sum(nbr(h) * 2 * h for h in direct) * costs["e_miller"],
            "ks_oa_g1terms": sum(nb * 2 * h for h in direct if nb * 2 * h < LANE_MIN) * costs["e_g1_mul"],
            "kn_oa_g1terms": sum(nb * 2 * h for h in direct if nb * 2 * h >= LANE_MIN) * costs["g1_mul"],
            "ks_final_exp": (sum(2 * nbr(h) for h in direct) + 1) * costs["e_final_exp"],
            "ks_f12_tree": (K - 1 + sum(2 * nbr(h) * (h - 1) for h in direct)
                            + sum(2 * nb * (2 * q - 1) + 4 * nb * (q - 1) for q in qs)) * costs["e_f12_mul"],
            "(ks_pt_tree<false, true>)": (sum(2 * nb * (h - 1) for h in direct)
                                   + sum(2 * nb * (2 * q - 1) + 4 * nb * (q - 1) for q in qs)) * costs["e_g1_add"],
            "ks_oa_fold": sum(whole) * (g1_fold + g2_fold),
            "ks_oa_fold_split": sum(split) * (4 * costs["e_g1_part"] + g1_sum + 4 * costs["e_g2_part"] + g2_sum),
            # multiples 2^{32m} (G1, 16m double doublings) and 2^{16m} (G2, 16m doublings), m = 1..3,
            # of the whole arrays of the split rounds
            "ks_fold_mults": sum(split) * (2 * (96 * costs["e_g1_dbl2"] + 3 * costs["e_g1_to_aff"])
                                           + 96 * costs["e_g2_dbl"] + 3 * costs["e_g2_to_aff"]),
            "ks_oa_pterms": sum(nb * 8 * q for q in qs) * costs["e_miller"],
            "ks_oa_g1terms_split": sum(nb * 8 * (K >> (j + 1)) * (4 * costs["e_g1_part"] + 3 * costs["e_g1_add"])
                                       for j in range(j0 - 1, lK) if nb * (K >> j) <= FOLD_SPLIT_MAX),
            "ks_oa_g1terms_next": sum(nb * 8 * (K >> (j + 1)) * costs["e_g1_mul"]
                                      for j in range(j0 - 1, lK) if nb * (K >> j) > FOLD_SPLIT_MAX),
            "ks_final_exp2": len(qs) * 6 * nb * costs["e_final_exp"],
            # the G1 groups to affine form, with their multiples 2^{32m} (16m double doublings)
            "ks_g1_finish": len(qs) * (2 * nb * costs["e_g1_to_aff"]
                                       + 4 * nb * (96 * costs["e_g1_dbl2"] + 4 * costs["e_g1_to_aff"])),
            # four-part split multiplications: the whole work plus three more tables each
            "ks_oa_combine_split": len(qs) * 4 * nb * (costs["e_gt_pow"] + 3 * costs["e_gt_tab"]
                                                       + costs["e_g1_mul"] + 3 * costs["e_g1_tab"]),
            "ks_oa_combine8": len(qs) * 2 * nb * (8 * costs["e_f12_mul"] + 7 * costs["g1_add"] + costs["g1_madd"]
                                                  + costs["g1_to_aff"]),
            "ks_gt_sqr_mults": len(qs) * 4 * nb * 96 * costs["e_csqr"],
        })
    else:
        nbr = lambda h: 1 if h == K // 2 else nb   # round 1's pairings are computed once for all batches
        wide = [h for h in rounds if nbr(h) * h >= LANE_MILLER_MIN]
        w.update({
            "ks_oa_miller": sum(nbr(h) * 2 * h for h in rounds if h not in wide) * costs["e_miller"],
            "kn_oa_miller": sum(nbr(h) * 2 * h for h in wide) * costs["miller"],
            "ks_final_exp": (sum(2 * nbr(h) for h in rounds) + 1) * costs["e_final_exp"],
            "ks_f12_tree": (K - 1 + sum(2 * nbr(h) * (h - 1) for h in rounds)) * costs["e_f12_mul"],
            "kn_oa_fold_g2": sum(nb * h for h in rounds if nb * h >= LANE_MIN) * g2_fold,
            "kn_oa_fold_g1": sum(nb * h for h in rounds if nb * h >= LANE_MIN) * g1_fold,
            "ks_oa_fold": sum(nb * h for h in rounds if nb * h < LANE_MIN) * (g1_fold + g2_fold),
            "kn_oa_g1terms": sum(nb * 2 * h for h in rounds if nb * 2 * h >= LANE_MIN) * costs["g1_mul"],
            "ks_oa_g1terms": sum(nb * 2 * h for h in rounds if nb * 2 * h < LANE_MIN) * costs["e_g1_mul"],
        })
    return w


def mad_peak(V):
    """ALU peak for the roofline: the measured multiply-add rate (probe kernel in the library)
    when it exceeds the rate derived from the unit counts and clock"""
    try:
        measured = V.vc_diag_mad_rate(0)
    except Exception as e:  # noqa: BLE001 - the derived peak stands in
        log("mad probe failed: %s" % e)
        measured = 0.0
    if measured > PEAK_MAD_TOPS:
        return measured, "measured (vc_diag_mad_rate: v_mad_u64_u32 probe, 8 chains per lane)"
    return PEAK_MAD_TOPS, "derived: 256 CU x 64 lanes x 2.4 GHz / 2 (half-rate v_mad_u64_u32); probe %.2f" % measured


def fold_bytes(L):
    """HBM bytes the y-tree must move at least (section 4.2, Sub-protocol): read the N entries
    and the K randomizers rho_j, write every node of the (2K - 1) x M tree, 32 bytes each"""
    lK, lM = L // 2, L - L // 2
    K, M, N = 1 << lK, 1 << lM, 1 << L
    return 32 * (N + K + (2 * K - 1) * M)


def log(msg):
    print("[bench] " + msg, file=sys.stderr, flush=True)


def run_workload(V, torch, L, b, bits, seed, steps, warmup, profile="all"):
    """profile: None, "all" (every kernel launch bracketed by events) or one kernel name"""
    import numpy as np
    log("workload L=%d b=%d bits=%d seed=%d: setup" % (L, b, bits, seed))
    from paper_2601_03031_amd import inputs as I
    limbs = I.entries(1 << L, seed, bits)
    if bits == 32:
        m = torch.from_numpy(limbs[:, 0].astype(np.uint32).view(np.int32).copy()).cuda()
    else:
        m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
    pp = V.vc_setup(L, I.TRAPDOOR_SEED, 0)
    stream = torch.cuda.current_stream()
    for _ in range(warmup):
        cm = V.vc_commit(pp, m, bits, stream)
        pr = V.vc_open_all(pp, cm, b, stream)
        del pr, cm
    torch.cuda.synchronize()
    log("warmup done; timing %d steps" % steps)
    commit_ms, open_ms = [], []
    if profile:
        V.vc_profile_only(None if profile == "all" else profile)
        V.vc_profile_enable(True)
    t_all = time.perf_counter()
    for _ in range(steps):
        t0 = time.perf_counter()
        cm = V.vc_commit(pp, m, bits, stream)
        t1 = time.perf_counter()
        pr = V.vc_open_all(pp, cm, b, stream)
        t2 = time.perf_counter()
        commit_ms.append(1e3 * (t1 - t0))
        open_ms.append(1e3 * (t2 - t1))
        del pr, cm
    torch.cuda.synchronize()
    wall = time.perf_counter() - t_all
    prof = V.vc_profile_read() if profile else {}
    V.vc_profile_enable(False)
    V.vc_profile_only(None)
    return limbs, commit_ms, open_ms, prof, wall


# (executors, streams per executor, jobs per fused group[, ahead threshold]) of the batched-jobs
# runs: group 1 is one job per executor (vc_open_all_batch), larger groups fuse the jobs of one
# size; a threshold set on the executors overrides the library's choice (0: every Step 1 round
# direct; 4096: terms taken one round ahead up to 4096 batch-index pairs, whatever their number of batches;
# fused groups sharing the device run direct unless one is set)
BATCH_SETUPS = ((8, 2, 1), (16, 1, 1), (16, 1, 1, 0), (16, 1, 64), (16, 1, 64, 4096), (8, 2, 64))


def batched_jobs(V, torch, n_jobs=64, seed=5, setups=BATCH_SETUPS, reps=2, peak=PEAK_MAD_TOPS):
    """Batched jobs: n_jobs independent vectors, N = 2^L with L uniform in [8, 18] (seeded),
    b = min(L^2, K), uniform full-width entries, each committed once.  Open-all of every job
    one after another on one stream, against the batch call on ne executors of ns streams
    each, either one job per executor (g = 1, vc_open_all_batch) or the jobs of one size fused
    in groups of at most g (vc_open_all_grouped), ne groups at a time; the best of `reps`
    passes each.  The serialized proofs at the ends of every vector are compared with the
    one-job call's.  The commits are timed too: vc_commit of every job in turn against
    vc_commit_batch (all MSMs in one persistent launch, FC.Commit fused), with the MSM schedule
    autotuned for these sizes first; commit + open-all is reported for the sequential path, the
    executor pool and the fused form."""
    import numpy as np
    from paper_2601_03031_amd import inputs as I
    rng = np.random.default_rng(seed)
    Ls = [int(x) for x in rng.integers(8, 19, n_jobs)]
    log("batched jobs: %d vectors, L in [8, 18]: setup and commit" % n_jobs)
    params, jobs, fmul, fexec, ents = {}, [], 0, 0, []
    costs = op_costs()
    for i, L in enumerate(Ls):
        if L not in params:
            params[L] = V.vc_setup(L, I.TRAPDOOR_SEED, 0)
        pp = params[L]
        limbs = I.entries(1 << L, 1000 * seed + i, 256)
        # algorithmic field multiplications of this job's open-all (the method's counts), and
        # what the library executes for it
        fmul += method_work(L, min(L * L, pp.K), limbs, costs)["open_all"]
        w = work_model(L, min(L * L, pp.K), limbs, costs)
        fexec += sum(v for k, v in w.items() if k not in ("k_msm_slices<lane::G1>", "ks_miller"))
        m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
        ents.append((pp, m, 256))
        jobs.append((pp, V.vc_commit(pp, m, 256), min(L * L, pp.K)))
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    # commits: one after another, then batched (after the schedule is tuned for these sizes)
    t0 = time.perf_counter()
    V.vc_tune_msm(8, 18)
    tune_s = time.perf_counter() - t0

    def seq_commit():
        t0 = time.perf_counter()
        out = [V.vc_commit(pp, m, bits, stream) for pp, m, bits in ents]
        return 1e3 * (time.perf_counter() - t0), out

    def batch_commit():
        t0 = time.perf_counter()
        out = V.vc_commit_batch(ents, stream=stream)
        return 1e3 * (time.perf_counter() - t0), out

    gex = V.vc_exec_create(0, 1)
    gex.set_graphs(True)

    def graph_commit():  # the same on an executor that captures the chain once and replays it
        t0 = time.perf_counter()
        out = V.vc_commit_batch(ents, ex=gex, stream=stream)
        return 1e3 * (time.perf_counter() - t0), out

    seq_c_ms, seq_c = min((seq_commit() for _ in range(reps)), key=lambda r: r[0])
    bat_c_ms, bat_c = min((batch_commit() for _ in range(reps + 1)), key=lambda r: r[0])
    gra_c_ms, gra_c = min((graph_commit() for _ in range(reps + 1)), key=lambda r: r[0])
    for a, g, r, (_, cm, _) in zip(bat_c, gra_c, seq_c, jobs):
        if a.C != r.C or a.C != cm.C or g.C != r.C:
            raise RuntimeError("a batched commitment differs from the one-job call's")
    graph_stats = gex.graph_stats()
    del seq_c, bat_c, gra_c, gex
    log("batched jobs: commits one by one %.1f ms, batched %.1f ms, graph %.1f ms (tuning %.1f s)"
        % (seq_c_ms, bat_c_ms, gra_c_ms, tune_s))

    def sequential():
        t0 = time.perf_counter()
        out = [V.vc_open_all(pp, cm, b, stream) for pp, cm, b in jobs]
        return 1e3 * (time.perf_counter() - t0), out

    seq_ms, seq_out = min((sequential() for _ in range(reps)), key=lambda r: r[0])
    log("batched jobs: sequential %.1f ms" % seq_ms)
    res = {"jobs": n_jobs, "L_counts": {str(L): Ls.count(L) for L in sorted(set(Ls))},
           "proofs": sum(pp.N for pp, _, _ in jobs), "sequential_ms": round(seq_ms, 2), "batch_ms": {}}
    for st_ in setups:
        ne, ns, g = st_[:3]
        execs = [V.vc_exec_create(0, ns) for _ in range(ne)]
        thr = st_[3] if len(st_) > 3 else None
        for ex in execs:
            if thr is not None:
                ex.set_ahead(thr)
        best, out = None, None
        for _ in range(reps + 1):  # the first pass sizes every executor's workspace
            t0 = time.perf_counter()
            out = V.vc_open_all_batch(jobs, execs) if g == 1 else V.vc_open_all_grouped(jobs, execs, g)
            ms = 1e3 * (time.perf_counter() - t0)
            best = ms if best is None or ms < best else best
        for (pp, _, _), a, r in zip(jobs, out, seq_out):
            for i in (0, pp.N - 1):
                if V.vc_proof_get(a, i) != V.vc_proof_get(r, i):
                    raise RuntimeError("batched proof %d of a 2^%d job differs from the one-job call" % (i, pp.log_n))
        del out, execs
        key = "%dx%d" % (ne, ns) + ("" if g == 1 else "_g%d" % g) + \
            ("" if thr is None else "_direct" if thr == 0 else "_ahead%d" % thr)
        res["batch_ms"][key] = round(best, 2)
        log("batched jobs: %d executors x %d streams, groups of %d%s: %.1f ms"
            % (ne, ns, g, "" if thr is None else " (ahead threshold %d)" % thr, best))
    k_best = min(res["batch_ms"], key=lambda k: res["batch_ms"][k])
    res["speedup"] = round(seq_ms / res["batch_ms"][k_best], 2)
    res["best_setup"] = k_best
    pool = min((v for k, v in res["batch_ms"].items() if "_g" not in k), default=None)
    fused = min((v for k, v in res["batch_ms"].items() if "_g" in k), default=None)
    res["ahead_vs_direct_ms"] = {k: v for k, v in res["batch_ms"].items() if k.startswith("16x1")}
    res["commit_ms"] = {"sequential": round(seq_c_ms, 2), "batched": round(bat_c_ms, 2),
                        "batched_graph": round(gra_c_ms, 2), "graph_captures_replays": list(graph_stats),
                        "speedup": round(seq_c_ms / min(bat_c_ms, gra_c_ms), 2), "msm_tuning_s": round(tune_s, 2)}
    res["commit_plus_open_ms"] = {"sequential": round(seq_c_ms + seq_ms, 2),
                                  "pool": round(seq_c_ms + pool, 2) if pool else None,
                                  "fused": round(min(bat_c_ms, gra_c_ms) + fused, 2) if fused else None}
    if fused:
        res["commit_plus_open_ms"]["speedup_fused"] = round((seq_c_ms + seq_ms) / (min(bat_c_ms, gra_c_ms) + fused), 2)
    V.vc_tune_load(None)  # the rest of the run keeps the default schedule
    # device utilization: the jobs' algorithmic multiply-adds over the time, against the ALU peak
    tops = lambda f, ms: f * MADS_PER_FMUL / (ms / 1e3) / 1e12
    res["field_mults"] = int(fmul)
    res["executed_field_mults"] = int(fexec)
    res["alu_frac"] = {"sequential": round(tops(fmul, seq_ms) / peak, 5),
                       "batched": round(tops(fmul, res["batch_ms"][k_best]) / peak, 5),
                       "batched_executed": round(tops(fexec, res["batch_ms"][k_best]) / peak, 5)}
    res["hw_queues"] = int(os.environ.get("GPU_MAX_HW_QUEUES", "0") or 0)
    return res


SERVE_SETUPS = ((1, 6), (8, 2))           # (executors, streams): the one-job path, then the pool


def serving(V, torch, n_req=40, rate=8.0, seed=7, setups=SERVE_SETUPS, budget=64 << 30):
    """Serving loop: a seeded Poisson stream of n_req open-all requests (rate per second),
    N = 2^L with L uniform in [10, 20], b uniform in {1, L, L^2} within [1, K], 32-bit or
    full-width entries half and half, each vector committed beforehand.  The same stream is
    served by one executor of six streams (one request at a time, as vc_open_all) and by the
    pool; latency is submission to completion.  Proof 0 of every request must agree."""
    import numpy as np
    from paper_2601_03031_amd import inputs as I
    rng = np.random.default_rng(seed)
    reqs, t = [], 0.0
    for _ in range(n_req):
        t += float(rng.exponential(1.0 / rate))
        L = int(rng.integers(10, 21))
        K = 1 << (L // 2)
        b = int(rng.choice([x for x in (1, L, L * L) if x <= K]))
        bits = 32 if rng.random() < 0.5 else 256
        reqs.append((L, b, bits, t))
    log("serving: %d requests over %.1f s: setup and commit" % (n_req, t))
    params, cms = {}, []
    for i, (L, b, bits, _) in enumerate(reqs):
        if L not in params:
            params[L] = V.vc_setup(L, I.TRAPDOOR_SEED, 0)
        limbs = I.entries(1 << L, 7000 + i, bits)
        if bits == 32:
            m = torch.from_numpy(limbs[:, 0].astype(np.uint32).view(np.int32).copy()).cuda()
        else:
            m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
        cms.append(V.vc_commit(params[L], m, bits))
    torch.cuda.synchronize()
    proofs = sum(1 << L for L, _, _, _ in reqs)
    res = {"requests": n_req, "rate_per_s": rate, "span_s": round(t, 2), "proofs": proofs, "budget_bytes": budget,
           "b_counts": {k: sum(1 for L, b, _, _ in reqs if ("1" if b == 1 else "L" if b == L else "L^2") == k)
                        for k in ("1", "L", "L^2")},
           "setups": {}}
    first = None
    for ne, ns in setups:
        sv = V.vc_server_create(0, ne, ns, budget)
        t0 = time.perf_counter()
        tickets = []
        for (L, b, bits, arr), cm in zip(reqs, cms):
            dt = t0 + arr - time.perf_counter()
            if dt > 0:
                time.sleep(dt)
            tickets.append(sv.submit(params[L], cm, b))
        lat, p0 = [], []
        for tk in tickets:
            pr, (_, total) = sv.wait(tk)
            lat.append(total)
            p0.append(V.vc_proof_get(pr, 0))
            del pr
        wall = time.perf_counter() - t0
        held, peak, _ = sv.stats()
        del sv
        if first is None:
            first = p0
        elif p0 != first:
            raise RuntimeError("served proofs differ between executor setups")
        key = "%dx%d" % (ne, ns)
        res["setups"][key] = {"p50_ms": round(float(np.percentile(lat, 50)), 1),
                              "p99_ms": round(float(np.percentile(lat, 99)), 1),
                              "mean_ms": round(float(np.mean(lat)), 1), "wall_s": round(wall, 2),
                              "proofs_per_s": round(proofs / wall), "peak_held_bytes": int(peak)}
        log("serving %s: p50 %.0f ms, p99 %.0f ms, wall %.1f s" % (key, res["setups"][key]["p50_ms"],
                                                                   res["setups"][key]["p99_ms"], wall))
    return res


def verify_all_timing(V, torch, L=16, b=256, seed=2, reps=3):
    """Verification of all N proofs of the N = 2^L workload with batch size b (32-bit entries,
    seed 2): device serialization of the N proofs, then vc_verify_all (best of reps each), and
    the one-proof verifier on a few proofs for comparison."""
    import numpy as np
    from paper_2601_03031_amd import inputs as I
    limbs = I.entries(1 << L, seed, 32)
    pp = V.vc_setup(L, I.TRAPDOOR_SEED, 0)
    cm = V.vc_commit(pp, torch.from_numpy(limbs[:, 0].astype(np.uint32).view(np.int32).copy()).cuda(), 32)
    pr = V.vc_open_all(pp, cm, b)
    m = torch.frombuffer(bytearray(I.limbs_to_bytes(limbs)), dtype=torch.uint8).cuda()
    ser_ms, ver_ms, ser = [], [], None
    for r in range(reps):
        del ser
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ser = V.vc_proofs_serialize(pr)
        t1 = time.perf_counter()
        v, ns = V.vc_verify_all(pp, cm.C, b, m, ser, bytes([r]) * 32)
        t2 = time.perf_counter()
        if v != 1:
            raise RuntimeError("verify_all rejected the honest proofs")
        ser_ms.append(1e3 * (t1 - t0))
        ver_ms.append(1e3 * (t2 - t1))
    ints = I.limbs_to_ints(limbs)
    one = []
    for i in (0, 12345, 65535):
        proof = V.vc_proof_get(pr, i)
        t0 = time.perf_counter()
        if V.vc_verify(pp, cm.C, b, i, ints[i], proof) != 1:
            raise RuntimeError("vc_verify rejected an honest proof")
        one.append(1e3 * (time.perf_counter() - t0))
    n = 1 << L
    return {"N": n, "b": b, "serialized_bytes": int(ser.numel()), "serialize_ms": round(min(ser_ms), 3),
            "verify_all_ms": round(min(ver_ms), 3), "proofs_verified_per_s": round(n / (min(ver_ms) / 1e3)),
            "checked_alone": ns, "one_proof_verify_ms": round(statistics.median(one), 3)}


def subarray_timing(V, torch, cases=((16, 256, 32, 2), (20, 400, 256, 3)), reps=3):
    """OpenAll for sub-arrays (Step 1 alone) against the full open-all on the same commitment,
    best of reps each."""
    import numpy as np
    from paper_2601_03031_amd import inputs as I
    out = {}
    for L, b, bits, seed in cases:
        limbs = I.entries(1 << L, seed, bits)
        if bits == 32:
            m = torch.from_numpy(limbs[:, 0].astype(np.uint32).view(np.int32).copy()).cuda()
        else:
            m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
        pp = V.vc_setup(L, I.TRAPDOOR_SEED, 0)
        cm = V.vc_commit(pp, m, bits)
        st = torch.cuda.current_stream()
        times = {}
        for name, fn in (("subarrays_ms", V.vc_open_subarrays), ("open_all_ms", V.vc_open_all)):
            best = None
            for _ in range(reps + 1):  # the first call sizes the workspace
                t0 = time.perf_counter()
                pr = fn(pp, cm, b, st)
                ms = 1e3 * (time.perf_counter() - t0)
                del pr
                best = ms if best is None or ms < best else best
            times[name] = round(best, 3)
        out["n2^%d_b%d" % (L, b)] = times
    return out


def eval_timing(V, torch, cases=((16, 32, 2), (20, 256, 3)), reps=3):
    """Evaluation proof of f_m at a seeded random point (section 4.3), best of reps, after one
    call that sizes the workspace."""
    import random
    import numpy as np
    from paper_2601_03031_amd import inputs as I
    out = {}
    for L, bits, seed in cases:
        limbs = I.entries(1 << L, seed, bits)
        if bits == 32:
            m = torch.from_numpy(limbs[:, 0].astype(np.uint32).view(np.int32).copy()).cuda()
        else:
            m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
        pp = V.vc_setup(L, I.TRAPDOOR_SEED, 0)
        cm = V.vc_commit(pp, m, bits)
        rng = random.Random(seed)
        r = [rng.randrange(I.R) for _ in range(L)]
        best = None
        for _ in range(reps + 1):
            t0 = time.perf_counter()
            V.vc_eval_proof(pp, cm, r)
            ms = 1e3 * (time.perf_counter() - t0)
            best = ms if best is None or ms < best else best
        out["n2^%d" % L] = round(best, 3)
    return out


def c3_timing(V, torch, Ls=(22, 24), seed=3, warm_max=26):
    """Single-job open-all beyond 2^20 (Table 3's larger columns and the largest size that fits
    the device): b = log^2 N, full-width entries drawn on the device (uniform in [0, 2^253),
    seeded); setup, commit and open-all times, the open-all's own device bytes
    (vc_open_all_footprint) and the device memory in use after it returns.  Sizes up to
    2^warm_max are timed on a second pass, larger ones once (their first call is as fast)."""
    from paper_2601_03031_amd import inputs as I
    out = {}
    for L in Ls:
        N = 1 << L
        K = 1 << (L // 2)
        b = min(L * L, K)
        log("c3: N=2^%d b=%d: setup" % (L, b))
        t0 = time.perf_counter()
        pp = V.vc_setup(L, I.TRAPDOOR_SEED, 0)
        setup_s = time.perf_counter() - t0
        m = I.device_entries(N, seed)
        torch.cuda.synchronize()
        st = torch.cuda.current_stream()
        runs = []
        warm = L <= warm_max
        for r in range(2 if warm else 1):
            log("c3: N=2^%d commit + open-all, pass %d" % (L, r))
            t0 = time.perf_counter()
            cm = V.vc_commit(pp, m, 256, st)
            t1 = time.perf_counter()
            pr = V.vc_open_all(pp, cm, b, st)
            t2 = time.perf_counter()
            runs.append((1e3 * (t1 - t0), 1e3 * (t2 - t1)))
            free, total = torch.cuda.mem_get_info()
            if r + 1 < (2 if warm else 1):
                del pr, cm
        c_ms, o_ms = runs[-1]
        out["n2^%d_b%d" % (L, b)] = {
            "all_proofs_ms": round(o_ms, 2), "commit_ms": round(c_ms, 2), "setup_s": round(setup_s, 2),
            "first_call_ms": [round(x, 2) for x in runs[0]], "open_all_footprint_bytes": V.vc_open_all_footprint(pp, b),
            "device_bytes_in_use": int(total - free), "proofs": N,
            "proofs_per_s": round(N / (o_ms / 1e3))}
        log("c3: N=2^%d open-all %.1f ms, commit %.1f ms, %.1f GB in use" % (L, o_ms, c_ms, (total - free) / 1e9))
        del pr, cm, m, pp
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
    return out


def cpu_model():
    try:
        for ln in open("/proc/cpuinfo"):
            if ln.startswith("model name"):
                return ln.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(L, b, bits, seed, reps=5, reps1=2):
    """The oracle (plain C, OpenMP over independent units) on the host cores: one warm-up,
    then the median of `reps` OpenAll runs on all threads, and the median of `reps1` runs on
    one thread (the paper's setting), on the full workload's commitment."""
    import oracle as O
    log("cpu baseline (oracle) L=%d b=%d" % (L, b))
    from paper_2601_03031_amd import inputs as I
    limbs = I.entries(1 << L, seed, bits)
    threads = O.max_threads()
    pp = O.Params(L, I.TRAPDOOR_SEED)
    t0 = time.perf_counter()
    cm = O.Commitment(pp, I.limbs_to_bytes(limbs))
    commit_ms = 1e3 * (time.perf_counter() - t0)

    def runs(n):
        out = []
        for _ in range(n):
            t = time.perf_counter()
            op = O.Opening(cm, b)
            out.append(1e3 * (time.perf_counter() - t))
            del op
        return out

    runs(1)  # warm-up
    many = runs(reps)
    O.set_threads(1)
    one = runs(reps1)
    O.set_threads(threads)
    del cm, pp
    return {"value": round(statistics.median(many), 1), "unit": "ms", "cores": threads, "kind": "oracle",
            "sample": "the full N=2^%d, b=%d, %d-bit-entry workload: oracle OpenAll (all-N-proofs) time, "
                      "median of %d after a warm-up; one commitment (%.1f ms)" % (L, b, bits, reps, commit_ms),
            "runs_ms": [round(x, 1) for x in many], "mean_ms": round(statistics.mean(many), 1),
            "one_thread_ms": round(statistics.median(one), 1), "one_thread_runs": len(one),
            "cpu_model": cpu_model()}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extra", action="store_true")
    ap.add_argument("--batch-only", type=str, default="", metavar="SETUPS",
                    help="only run the batched-jobs comparison with these executors x streams[ x group] "
                         "setups (e.g. 4x6,16x1,16x1x64) and print its JSON")
    ap.add_argument("--batch-direct", action="store_true", help="with --batch-only: every Step 1 round direct")
    ap.add_argument("--serve-only", action="store_true", help="only run the serving-loop comparison")
    ap.add_argument("--only", choices=("verify_all", "eval", "subarrays"), default=None,
                    help="only run this extra measurement and print its JSON (for profiling)")
    ap.add_argument("--serve-rate", type=float, default=0, help="request rate per second of the serving stream")
    ap.add_argument("--serve-setups", type=str, default="", metavar="SETUPS",
                    help="executors x streams of the served runs (e.g. 1x6,4x6)")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MIB",
                    help="only copy MIB MiB device to device three times (reference kernel for the "
                         "FETCH_SIZE / WRITE_SIZE counters) and exit")
    ap.add_argument("--c3", type=str, default="", metavar="LOGNS",
                    help="only time single-job open-all at these log2 N (e.g. 22,24,26) and print its JSON")
    ap.add_argument("--mad-peak", action="store_true",
                    help="only measure the multiply-add peak with the library's probe kernel and exit")
    a = ap.parse_args()
    if a.mad_peak:
        import paper_2601_03031_amd as V
        r = V.vc_diag_mad_rate(0)
        print(json.dumps({"mad_per_s_T": round(r, 3), "derived_T": round(PEAK_MAD_TOPS, 3)}), flush=True)
        return
    if a.copy_calibration:
        import torch
        n = a.copy_calibration << 20
        src = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes": n, "copies": 3}), flush=True)
        return
    if a.gpus != 1:
        print("bench.py measures one GPU only: the single-GPU path is the build's scope "
              "(multi-GPU sharding is a design note, not built); run with --gpus 1", file=sys.stderr)
        sys.exit(2)
    import torch
    import paper_2601_03031_amd as V
    V.lib()
    if not torch.cuda.is_available():
        print("no GPU visible", file=sys.stderr)
        sys.exit(1)
    if a.c3:
        print(json.dumps(c3_timing(V, torch, [int(x) for x in a.c3.split(",")])), flush=True)
        return
    if a.only:
        fn = {"verify_all": lambda: verify_all_timing(V, torch), "eval": lambda: eval_timing(V, torch),
              "subarrays": lambda: subarray_timing(V, torch)}[a.only]
        print(json.dumps(fn()), flush=True)
        return
    if a.serve_only:
        kw = {}
        if a.serve_rate:
            kw["rate"] = a.serve_rate
        if a.serve_setups:
            kw["setups"] = [tuple(int(v) for v in x.split("x")) for x in a.serve_setups.split(",")]
        print(json.dumps(serving(V, torch, **kw)), flush=True)
        return
    if a.batch_only:
        setups = [tuple(int(v) for v in x.split("x")) + ((1,) if x.count("x") == 1 else ()) for x in a.batch_only.split(",")]
        if a.batch_direct:
            setups = [s_ + (0,) for s_ in setups]
        print(json.dumps(batched_jobs(V, torch, setups=setups)), flush=True)
        return

    L, b, bits, seed = 16, 256, 32, 2
    # per-kernel table from a separate pass with every launch bracketed by events (the
    # events cost host time and would perturb the timed steps); it names the dominant kernel
    psteps = 2
    limbs, _, _, prof, _ = run_workload(V, torch, L, b, bits, seed, psteps, a.warmup)
    total_prof = sum(ms for _, ms in prof.values())
    dname = max(prof.items(), key=lambda kv: kv[1][1])[0]
    # timed steps: only the dominant kernel's launches carry events (its average duration)
    _, commit_ms, open_ms, pdom, wall = run_workload(V, torch, L, b, bits, seed, a.steps, a.warmup, profile=dname)
    dcount, dms = pdom.get(dname, (0, 0.0))
    costs = op_costs()
    work = work_model(L, b, limbs, costs)
    method = method_work(L, b, limbs, costs)
    peak, peak_src = mad_peak(V)
    roofline = None
    if dcount and (dname in method["by_kernel"] or dname in work):
        # algorithmic work: the method's operation counts (method_work) where the kernel carries a
        # part of them, else what the kernel executes; the executed work is reported beside it
        basis = "method" if dname in method["by_kernel"] else "executed"
        fm = method["by_kernel"].get(dname, work.get(dname, 0))
        per_launch_fmul = fm / (dcount / a.steps)
        avg_s = dms / dcount / 1e3
        achieved = per_launch_fmul * MADS_PER_FMUL / avg_s / 1e12
        exec_per_launch = work.get(dname, 0) / (dcount / a.steps)
        roofline = {"bound": "alu", "kernel": dname, "achieved": round(achieved, 5), "peak": round(peak, 3),
                    "unit": "T mad/s", "frac": round(achieved / peak, 6), "traffic": TRAFFIC_BYTES.get(dname),
                    "work_basis": basis, "per_launch_field_mults": int(per_launch_fmul),
                    "mads_per_field_mult": MADS_PER_FMUL, "avg_launch_ms": round(dms / dcount, 4),
                    "launches_per_step": dcount / a.steps, "peak_source": peak_src,
                    "peak_derived": round(PEAK_MAD_TOPS, 3),
                    "executed_field_mults_per_launch": int(exec_per_launch),
                    "executed_frac": round(exec_per_launch * MADS_PER_FMUL / avg_s / 1e12 / peak, 6)}
    kernels = {k: {"launches": c // psteps, "ms_per_step": round(ms / psteps, 4),
                   "share": round(ms / total_prof, 4) if total_prof else None}
               for k, (c, ms) in sorted(prof.items(), key=lambda kv: -kv[1][1])}
    msm_ms = (prof.get("k_msm_slices<lane::G1>", (0, 0))[1] + prof.get("kw_sum_g1", (0, 0))[1]) / psteps
    tops = lambda fm, ms: fm * MADS_PER_FMUL / (ms / 1e3) / 1e12   # 10^12 multiply-adds per second
    open_med = statistics.median(open_ms)
    extra = {"commit_ms": round(statistics.median(commit_ms), 3),
             "open_ms_all": [round(x, 3) for x in open_ms],
             "open_ms_mean": round(statistics.mean(open_ms), 3),
             "msm_points_per_s": round((1 << L) / (msm_ms / 1e3)) if msm_ms else None,
             "msm_points_per_s_commit_wall": round((1 << L) / (statistics.median(commit_ms) / 1e3)),
             "method_field_mults": {k: int(v) for k, v in method["phases"].items()},
             "fractions": {"open_all_n2^16_b256": round(tops(method["open_all"], open_med) / peak, 6)},
             "kernels": kernels}
    if not a.no_extra:
        L2, b2 = 20, 400
        n2 = max(1, min(a.steps, 2))
        limbs2, _, _, p2, _ = run_workload(V, torch, L2, b2, 256, 3, 1, 1)
        _, c2, o2, _, _ = run_workload(V, torch, L2, b2, 256, 3, n2, 1, profile=None)
        method2 = method_work(L2, b2, limbs2, costs)
        msm2 = p2.get("k_msm_slices<lane::G1>", (0, 0))[1] + p2.get("kw_sum_g1", (0, 0))[1]
        fbytes = fold_bytes(L2)
        fold_k = sorted(k for k in p2 if k.startswith("k_ytree"))
        fold_ms = sum(p2[k][1] for k in fold_k)
        fold_gbs = fbytes / (fold_ms / 1e3) / 1e9 if fold_ms else None
        extra["n2^20_b400"] = {"all_proofs_ms": round(statistics.median(o2), 3), "commit_ms": round(statistics.median(c2), 3),
                               "msm_points_per_s": round((1 << L2) / (msm2 / 1e3)) if msm2 else None,
                               "msm_points_per_s_commit_wall": round((1 << L2) / (statistics.median(c2) / 1e3)),
                               "method_field_mults": {k: int(v) for k, v in method2["phases"].items()}}
        fr = extra["fractions"]
        fr["open_all_n2^20_b400"] = round(tops(method2["open_all"], statistics.median(o2)) / peak, 6)
        if msm2:
            # the commit MSM kernels alone (sorted-digit bucket accumulation, then the slice sums)
            fr["msm_n2^20"] = {"frac": round(tops(method2["phases"]["commit_msm"], msm2) / peak, 5),
                               "kernel_ms": round(msm2, 4), "field_mults": int(method2["phases"]["commit_msm"])}
        # the y-tree passes (Step 2 folding of the randomized rows) against HBM bandwidth: timed
        # alone on the device (vc_diag_fold), and as they ran inside the profiled open-all
        # beside the Step 1 kernels (their events then include waits for compute units)
        from paper_2601_03031_amd import inputs as I
        for Lf in (20, 24):
            ppf = V.vc_setup(Lf, I.TRAPDOOR_SEED, 0)
            cmf = V.vc_commit(ppf, I.device_entries(1 << Lf, 3), 256)
            alone = V.vc_diag_fold(cmf)
            fb = fold_bytes(Lf)
            gbs = fb / (alone / 1e3) / 1e9
            fr["fold_n2^%d" % Lf] = {"GB_per_s": round(gbs, 1), "frac_of_hbm": round(gbs / PEAK_HBM_GBS, 5),
                                      "bytes": fb, "kernel_ms": round(alone, 4), "timing": "alone (vc_diag_fold)"}
            del cmf, ppf
        if fold_gbs:
            fr["fold_n2^20"]["in_open_all"] = {"GB_per_s": round(fold_gbs, 1), "kernel_ms": round(fold_ms, 4),
                                              "kernels": fold_k}
        # batch-size sweep (one timed step each): all-N-proofs ms and the whole-open-all fraction
        sweep, sweep_fr = {}, {}
        for (Ls, bs, bits_s, seed_s) in ((16, 1, 32, 2), (16, 16, 32, 2), (20, 20, 256, 3), (20, 1, 256, 3)):
            lim_s, cs_, os_, _, _ = run_workload(V, torch, Ls, bs, bits_s, seed_s, 1, 1, profile=False)
            sweep["n2^%d_b%d" % (Ls, bs)] = round(os_[0], 3)
            sweep_fr["open_all_n2^%d_b%d" % (Ls, bs)] = round(
                tops(method_work(Ls, bs, lim_s, costs)["open_all"], os_[0]) / peak, 6)
        extra["b_sweep_all_proofs_ms"] = sweep
        fr.update(sweep_fr)
        extra["batched_64_jobs"] = batched_jobs(V, torch, peak=peak)
        extra["serving"] = serving(V, torch)
        extra["serving_16_per_s"] = serving(V, torch, rate=16.0)
        extra["subarrays"] = subarray_timing(V, torch)
        extra["eval_proof_ms"] = eval_timing(V, torch)
        extra["verify_all_n2^16"] = {"b256": verify_all_timing(V, torch, b=256), "b1": verify_all_timing(V, torch, b=1)}
        # single-job open-all at Table 3's larger sizes and at the largest that fits the device
        torch.cuda.empty_cache()
        try:
            extra["c3_single_job"] = c3_timing(V, torch, (22, 24, 30))
        except Exception as e:  # noqa: BLE001 - reported in the line, the other figures stand
            extra["c3_single_job"] = {"error": str(e)}
    cpu = None
    if not a.no_cpu_baseline:
        cpu = cpu_baseline(L, b, bits, seed)
    line = {"metric": METRIC, "value": round(statistics.median(open_ms), 3), "unit": "ms", "n_gpus": 1,
            "steps": a.steps, "warmup": a.warmup,
            "ms_per_step": round(statistics.median([c + o for c, o in zip(commit_ms, open_ms)]), 3),
            "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
            "dtype": "u32 limbs: exact 254-bit F_p/F_r (BN254)",
            "data": "synthetic", "config": {"workload": "N=2^16 commit + open-all, b=log^2 N=256, uniform 32-bit entries "
                                            "(seed 2), BN254", "N": 1 << L, "b": b, "entry_bits": bits},
            "roofline": roofline, "cpu_baseline": cpu, "extra": extra}
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
