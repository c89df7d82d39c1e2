"""Workloads by which the framework's speed is followed: what a user has it do, through the
package's public calls.

listed() names the cases, draw(rng) gives more of the same ranges, prepare(case, seed) makes
what a program holds before the call (the keys, the entries, for a verifier the proofs),
run(state) is one pass, work(case) the least work of a pass.  Every output is bytes (encoded
group elements, proofs, verdicts), exact for its inputs.

The kinds of case:
  commit      vc_commit of one vector, its subvector commitments and C read back;
  open        vc_open_all on a committed vector, all N proofs written out;
  jobs        many small vectors at once: vc_commit_batch, vc_open_all_grouped, all proofs;
  subarrays   vc_open_subarrays, one proof of each batch (they are the same within a batch);
  eval        vc_eval_proof at a random point;
  verify      vc_verify on a few single proofs, for some seeds one of them for another entry;
  verify_all  vc_verify_all on all N proofs, one to three of them altered.
"""
import random
import weakref

import numpy as np
import torch

import paper_2601_03031_amd as V
from paper_2601_03031_amd import inputs as I

# field multiplications of one operation of the scheme (BN254): a Miller loop, a final
# exponentiation, a G1 multiplication, a G2 multiplication, a mixed G1 addition
MILLER, FINAL, MUL1, MUL2, MADD = 8511, 7342, 2000, 4900, 11
MAD = 136  # 32-bit multiply-adds of a field multiplication


def listed():
    return [
        # the least a prover asks for: a vector of 256 entries (the lower end of the batched
        # jobs); launches and one short chain of kernels count
        {"name": "commit_2e8", "op": "commit", "log_n": 8, "bits": 256},
        # the commitment that goes before the headline open-all: 32-bit entries
        {"name": "commit_2e16_u32", "op": "commit", "log_n": 16, "bits": 32},
        # a large commitment of full-width entries: multi-scalar multiplication throughput
        {"name": "commit_2e20", "op": "commit", "log_n": 20, "bits": 256},
        # sixteen small vectors served together, of uneven sizes
        {"name": "jobs_16", "op": "jobs", "count": 16, "lo": 8, "hi": 12},
        # the smallest workload of the benchmark: N = 2^10, a batch for every subvector
        {"name": "open_2e10_b1", "op": "open", "log_n": 10, "b": 1, "bits": 256},
        # the headline: N = 2^16, b = log^2 N, one batch, a chain of dependent rounds
        {"name": "open_2e16_b256", "op": "open", "log_n": 16, "b": 256, "bits": 32},
        # b = 2 log N on an odd log N, so that K < M and the last batch is a short one
        {"name": "open_2e17_b34", "op": "open", "log_n": 17, "b": 34, "bits": 256},
        # a batch for every subvector, shortest proofs: 256 batches fill the device
        {"name": "open_2e16_b1", "op": "open", "log_n": 16, "b": 1, "bits": 32},
        # a large vector opened at b = log^2 N, by sub-arrays
        {"name": "subarrays_2e20_b400", "op": "subarrays", "log_n": 20, "b": 400, "bits": 256},
        # a large vector's evaluation proof (the scheme used inside a proof system)
        {"name": "eval_2e20", "op": "eval", "log_n": 20, "bits": 256},
        # a light client that checks the proofs it got, one by one
        {"name": "verify_2e16_b256", "op": "verify", "log_n": 16, "b": 256, "count": 2},
        # an auditor that checks all of them, a few altered
        {"name": "verify_all_2e14_b128", "op": "verify_all", "log_n": 14, "b": 128},
    ]


def draw(rng):
    op = rng.choice(["commit", "commit", "jobs", "open", "open", "open", "subarrays", "eval", "verify", "verify_all"])
    bits = rng.choice([32, 256])
    if op == "commit":
        return {"op": op, "log_n": rng.randint(8, 20), "bits": bits}
    if op == "jobs":
        lo = rng.randint(7, 10)
        return {"op": op, "count": rng.randint(3, 16), "lo": lo, "hi": rng.randint(lo, 12)}
    if op == "eval":
        return {"op": op, "log_n": rng.randint(8, 20), "bits": bits}
    if op == "verify_all":
        log_n = rng.randint(8, 14)
    elif op == "subarrays":
        log_n = rng.randint(10, 20)
    elif op == "open":
        log_n = rng.randint(8, 17)
    else:
        log_n = rng.randint(8, 16)
    K = 1 << (log_n // 2)
    # 1, 2 log N, log^2 N, or any size between; at most about 64 batches of 2^17's K = 256
    lo = max(1, K * K >> 16, K * K >> (14 if op == "subarrays" else 16))
    b = rng.choice([lo, 2 * log_n, log_n * log_n, int(lo * (K / lo) ** rng.random())])
    case = {"op": op, "log_n": log_n, "b": max(lo, min(b, K))}
    if op in ("open", "subarrays"):
        case["bits"] = bits
    if op == "verify":
        case["count"] = rng.randint(1, 3)
    return case


# A program keeps one set of keys for a size, and one pool of executors, and uses them for all
# vectors: the states of a case that are alive together share them.
_keys = weakref.WeakValueDictionary()
_pools = weakref.WeakValueDictionary()


class _Pool:
    def __init__(self, n):
        self.execs = [V.vc_exec_create(0, 1) for _ in range(n)]


def _params(log_n):
    pp = _keys.get(log_n)
    if pp is None:
        pp = _keys[log_n] = V.vc_setup(log_n, I.TRAPDOOR_SEED, 0)
    return pp


def _pool(n):
    p = _pools.get(n)
    if p is None:
        p = _pools[n] = _Pool(n)
    return p


def _entries(n, seed, bits):
    """n entries on the device: 32-bit integers, or 32-byte little-endian values below r."""
    if bits == 256:
        return I.device_entries(n, seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randint(0, 2**32, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)


def _sizes(case):
    """log N of each vector of a jobs case, spread evenly over its range."""
    lo, hi, n = case["lo"], case["hi"], case["count"]
    return [lo + (hi - lo + 1) * i // n for i in range(n)]


def _u8(data):
    return np.frombuffer(data, dtype=np.uint8)


def prepare(case, seed):
    op = case["op"]
    if op == "jobs":
        sizes = _sizes(case)
        return {"op": op, "pool": _pool(8),
                "jobs": [(_params(L), _entries(1 << L, seed * 64 + i, 256), 256) for i, L in enumerate(sizes)],
                "b": [max(1, min(L * L, 1 << (L // 2))) for L in sizes]}
    L = case["log_n"]
    pp = _params(L)
    bits = case.get("bits", 256)
    m = _entries(pp.N, seed, bits)
    st = {"op": op, "pp": pp, "m": m, "bits": bits, "b": case.get("b", 0)}
    if op == "commit":
        return st
    st["cm"] = V.vc_commit(pp, m, bits)
    if op in ("open", "subarrays"):
        return st
    rng = random.Random(seed)
    if op == "eval":
        st["point"] = [rng.randrange(I.R) for _ in range(L)]
        return st
    b = case["b"]
    pr = V.vc_open_all(pp, st["cm"], b)
    if op == "verify":
        st["proofs"] = []
        for k in range(case["count"]):
            i = rng.randrange(pp.N)
            value = int.from_bytes(m[32 * i:32 * i + 32].cpu().numpy().tobytes(), "little")
            proof = V.vc_proof_get(pr, i)
            if k == seed % (case["count"] + 1):  # another entry than the one committed
                value = (value + 1) % I.R
            st["proofs"].append((i, value, proof))
        return st
    st["all"] = V.vc_proofs_serialize(pr)
    st["seed"] = rng.randbytes(32)
    offs = V.proof_offsets(pp, b)
    for i in rng.sample(range(1, pp.N), 1 + seed % 3):  # a Merkle path's last byte
        st["all"][offs[i + 1] - 1] ^= 1
    return st


def run(st):
    op = st["op"]
    if op == "commit":
        cm = V.vc_commit(st["pp"], st["m"], st["bits"])
        return [_u8(cm.C), _u8(cm.export("Cj"))]
    if op == "open":
        return V.vc_proofs_serialize(V.vc_open_all(st["pp"], st["cm"], st["b"]))
    if op == "jobs":
        execs = st["pool"].execs
        cms = V.vc_commit_batch(st["jobs"], execs[0])
        prs = V.vc_open_all_grouped([(j[0], cm, b) for j, cm, b in zip(st["jobs"], cms, st["b"])], execs, 64)
        return [[_u8(cm.C) for cm in cms], [V.vc_proofs_serialize(pr) for pr in prs]]
    if op == "subarrays":
        pr = V.vc_open_subarrays(st["pp"], st["cm"], st["b"])
        firsts = list(range(0, st["pp"].K, st["b"]))
        return _u8(b"".join(V.vc_subarray_proof_get(pr, j) for j in firsts))
    if op == "eval":
        return _u8(V.vc_eval_proof(st["pp"], st["cm"], st["point"]))
    if op == "verify":
        return [V.vc_verify(st["pp"], st["cm"].C, st["b"], i, value, proof) for i, value, proof in st["proofs"]]
    return list(V.vc_verify_all(st["pp"], st["cm"].C, st["b"], st["m"], st["all"], st["seed"]))


def _commit_muls(L, bits):
    N, K = 1 << L, 1 << (L // 2)
    return N * (bits // 8) * MADD + K * MILLER + FINAL


def _step1_muls(L, b):
    """The FC batch proofs: for each batch 2K pairings' Miller loops, the folds, the sums and
    the KZG proof, and two final exponentiations a round."""
    lK = L // 2
    K = 1 << lK
    nb = -(-K // b)
    return nb * (2 * K * MILLER + 2 * lK * FINAL + K * (3 * MUL1 + MUL2) + 2 * K * MUL2)


def work(case):
    op = case["op"]
    if op == "jobs":
        parts = [{"op": o, "log_n": L, "b": max(1, min(L * L, 1 << (L // 2))), "bits": 256}
                 for L in _sizes(case)
                 for o in ("commit", "open")]
        ws = [work(p) for p in parts]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    L, b, bits = case["log_n"], case.get("b", 0), case.get("bits", 256)
    lK = L // 2
    lM = L - lK
    N, K, M = 1 << L, 1 << lK, 1 << lM
    entry = bits // 8
    keys = 64 * M + 128 * K
    if op == "commit":
        muls, size = _commit_muls(L, bits), N * entry + keys + 64 * K + 384
    elif op == "open":
        proof = 32 * min(b, K) + lK * 832 + 160 + 64 * lK + 32 * lM + 32 * L
        muls = _step1_muls(L, b) + 4 * N + (2 * K + M) * MUL1
        size = 32 * N + keys + 64 * K + N * proof
    elif op == "subarrays":
        muls, size = _step1_muls(L, b), keys + 64 * K + -(-K // b) * (32 * min(b, K) + lK * 832 + 160)
    elif op == "eval":
        muls, size = _step1_muls(L, K) + N + (K + M) * MUL1, 32 * N + keys + 64 * K + 832 * lK + 32 * lM + 224
    elif op == "verify":
        n = case["count"]
        muls = n * ((min(b, K) + 2 * lK) * MUL1 + (lM + 4) * MILLER + 3 * FINAL + 2 * lK * 5000)
        size = n * (32 * min(b, K) + lK * 832 + 160 + 64 * lK + 32 * lM + 32 * L + 384) + keys
    else:
        nb = -(-K // b)
        muls = nb * ((min(b, K) + 2 * lK) * MUL1 + 3 * MILLER + 2 * FINAL + 2 * lK * 5000) + (3 * K + 2 * M) * MUL1
        muls += (lM + 1) * MILLER + FINAL
        size = N * (32 * min(b, K) + lK * 832 + 160 + 64 * lK + 32 * lM + 32 * L + 32) + keys
    return {"bytes": size, "flops": 2 * MAD * muls}


def exact(case, seed):
    """Every output is bytes or a whole number: there is nothing to compare in 64 bits."""
    return None
