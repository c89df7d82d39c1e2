"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, byte for byte.

Every group element, field element, challenge, Merkle node and serialized proof is
unique given the inputs (exact arithmetic, canonical encodings), so the bar is
bit-exact equality.  Inputs come from the shared seeded generators; the oracle
never sees anything the GPU produced.
"""
import os
import sys

import numpy as np
import pytest

import oracle as O
from paper_2601_03031_amd import inputs as I

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SEED = I.TRAPDOOR_SEED


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def vc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_03031_amd as V
    V.lib()
    return V


def dev_entries(limbs: np.ndarray):
    return torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()


def dev_u32(v: np.ndarray):
    return torch.from_numpy(v.astype(np.uint32).view(np.int32).copy()).cuda()


# oracle objects of the large workloads, shared by the tests that check the same vector
# (an oracle commitment at N = 2^20 takes tens of seconds); keyed by (L, seed, bits[, b])
_ORACLE = {}


def oracle_commitment(L, seed, bits, limbs):
    key = (L, seed, bits)
    if key not in _ORACLE:
        opp = O.Params(L, SEED)
        _ORACLE[key] = (opp, O.Commitment(opp, I.limbs_to_bytes(limbs)))
    return _ORACLE[key]


def oracle_opening(L, seed, bits, limbs, b):
    key = (L, seed, bits, b)
    if key not in _ORACLE:
        _ORACLE[key] = O.Opening(oracle_commitment(L, seed, bits, limbs)[1], b)
    return _ORACLE[key]


class Case:
    """one workload run through both paths"""

    def __init__(self, V, L, b, seed=1, bits=256, zero=False):
        self.L, self.b = L, b
        say("case L=%d b=%d seed=%d bits=%d zero=%s" % (L, b, seed, bits, zero))
        N = 1 << L
        if zero:
            limbs = np.zeros((N, 4), dtype=np.uint64)
            self.opp = O.Params(L, SEED)
            self.ocm = O.Commitment(self.opp, I.limbs_to_bytes(limbs))
            self.oop = O.Opening(self.ocm, b)
        else:
            limbs = I.entries(N, seed, bits)
            self.opp, self.ocm = oracle_commitment(L, seed, bits, limbs)
            self.oop = oracle_opening(L, seed, bits, limbs, b) if L == 20 else O.Opening(self.ocm, b)
        self.m = I.limbs_to_ints(limbs)
        say("  oracle done; GPU setup/commit/open_all")
        self.gpp = V.vc_setup(L, SEED, 0)
        if bits == 32:
            self.gcm = V.vc_commit(self.gpp, dev_u32(limbs[:, 0].astype(np.uint32)), 32)
        else:
            self.gcm = V.vc_commit(self.gpp, dev_entries(limbs), 256)
        self.gpr = V.vc_open_all(self.gpp, self.gcm, b)
        torch.cuda.synchronize()
        say("  GPU done")


def compare_all(V, cs: Case, proofs="all"):
    pp = cs.opp
    for k in range(pp.lM + 1):
        assert cs.gpp.export("ek", k) == pp.export("ek", k), ("ek", k)
    for w in ("vk", "h", "g1beta"):
        assert cs.gpp.export(w) == pp.export(w), w
    assert cs.gcm.export("Cj") == b"".join(cs.ocm.Cj)
    assert cs.gcm.C == cs.ocm.C and cs.gcm.export("C") == cs.ocm.C
    for k in range(cs.oop.nb):
        for w in ("fc_x", "fc_rounds", "fc_tail"):
            assert cs.gpr.export(w, k) == cs.oop.export(w, k), (w, k)
    for w in ("merkle", "rho", "y", "D", "W"):
        assert cs.gpr.export(w) == cs.oop.export(w), w
    idx = range(pp.N) if proofs == "all" else proofs
    for i in idx:
        assert V.vc_proof_get(cs.gpr, i) == cs.oop.proof(i), ("proof", i)


@pytest.mark.parametrize("L,b", [(4, 1), (4, 4), (5, 3), (6, 2), (6, 8)])
def test_open_all_bit_exact_small(vc, L, b):
    cs = Case(vc, L, b, seed=L)
    compare_all(vc, cs)


def test_open_all_u32_entries(vc):
    cs = Case(vc, 6, 3, seed=2, bits=32)
    compare_all(vc, cs)


def test_zero_vector(vc):
    cs = Case(vc, 4, 2, zero=True)
    compare_all(vc, cs)


def test_n1024_b1_all_arrays(vc):
    """N = 2^10, b = 1: the small full workload (32 FC batches, 5 rounds each)."""
    cs = Case(vc, 10, 1, seed=1)
    compare_all(vc, cs, proofs=[0, 1, 31, 32, 511, 512, 1000, 1023])


def test_rejects_bad_input(vc):
    pp = vc.vc_setup(4, SEED, 0)
    bad = np.zeros((16, 4), dtype=np.uint64)
    r_limbs = [(I.R >> (64 * k)) & (2**64 - 1) for k in range(4)]
    bad[3] = np.array(r_limbs, dtype=np.uint64)  # entry == r
    with pytest.raises(vc.VCError) as e:
        vc.vc_commit(pp, dev_entries(bad), 256)
    assert e.value.code == vc.VC_EINVAL
    good = I.entries(16, 5)
    cm = vc.vc_commit(pp, dev_entries(good), 256)
    for b in (0, 5):
        with pytest.raises(vc.VCError) as e:
            vc.vc_open_all(pp, cm, b)
        assert e.value.code == vc.VC_EINVAL


@pytest.mark.parametrize("L,b", [(5, 2), (8, 16)])
def test_params_load_oracle_srs(vc, L, b):
    """An externally made SRS: the oracle's keys from a trapdoor seed no device setup uses,
    loaded with vc_params_load; the keys read back unchanged, and commit + open-all on them
    equal the oracle's on the same keys, every array and every proof."""
    other = b"external-srs".ljust(32, b"\0")
    say("params load: L=%d b=%d" % (L, b))
    opp = O.Params(L, other)
    srs = b"".join([opp.export("ek", k) for k in range(L - L // 2 + 1)] +
                   [opp.export("vk"), opp.export("h"), opp.export("g1beta")])
    gpp = vc.vc_params_load(srs, 0)
    assert gpp.log_n == L and gpp.srs_bytes() == srs
    limbs = I.entries(1 << L, 40 + L)
    ocm = O.Commitment(opp, I.limbs_to_bytes(limbs))
    oop = O.Opening(ocm, b)
    gcm = vc.vc_commit(gpp, dev_entries(limbs), 256)
    assert gcm.C == ocm.C and gcm.export("Cj") == b"".join(ocm.Cj)
    gpr = vc.vc_open_all(gpp, gcm, b)
    for k in range(oop.nb):
        for w in ("fc_x", "fc_rounds", "fc_tail"):
            assert gpr.export(w, k) == oop.export(w, k), (w, k)
    for w in ("merkle", "rho", "y", "D", "W"):
        assert gpr.export(w) == oop.export(w), w
    for i in range(1 << L):
        assert vc.vc_proof_get(gpr, i) == oop.proof(i), i


def test_params_load_rejects(vc):
    """Lengths that fit no size, a coordinate >= p and a point moved off its curve."""
    srs = vc.vc_setup(4, SEED, 0).srs_bytes()
    for bad_len in (srs[:-1], srs + b"\0" * 32, b""):
        with pytest.raises(vc.VCError) as e:
            vc.vc_params_load(bad_len, 0)
        assert e.value.code == vc.VC_EINVAL
    P = O.P
    big = bytearray(srs)
    big[0:32] = P.to_bytes(32, "big")  # x of ek_0[0] = p
    off = bytearray(srs)
    y = int.from_bytes(off[32:64], "big")
    off[32:64] = ((y + 1) % P).to_bytes(32, "big")  # y of ek_0[0] + 1: off the curve
    h0 = 64 * (2 * 4 - 1) + 128 * 2  # first h point (L = 4: M = 4, log M = 2)
    off2 = bytearray(srs)
    x = int.from_bytes(off2[h0:h0 + 32], "big")
    off2[h0:h0 + 32] = ((x + 1) % P).to_bytes(32, "big")  # a G2 point off the twist
    for bad in (big, off, off2):
        with pytest.raises(vc.VCError) as e:
            vc.vc_params_load(bytes(bad), 0)
        assert e.value.code == vc.VC_EINVAL
    assert vc.vc_params_load(srs, 0).srs_bytes() == srs


@pytest.mark.parametrize("L,b", [(8, 1), (8, 16), (14, 1)])
def test_zero_challenge_is_reported(vc, L, b):
    """A zero Fiat-Shamir challenge (section 3, FC.BOpen: the fold needs x_j^{-1}) ends the
    open-all with VC_ECHALLENGE.  Forced from the host in the first and the last round, in the
    rounds taken one ahead (L = 8) and the direct ones (2^14, b = 1); the one-job and the
    batch call both report it, and the same executor then opens the vector as before."""
    say("zero challenge: L=%d b=%d" % (L, b))
    pp = vc.vc_setup(L, SEED, 0)
    N, lK = 1 << L, L // 2
    cm = vc.vc_commit(pp, dev_entries(I.entries(N, 11)), 256)
    ref = vc.vc_open_all(pp, cm, b)
    want = [vc.vc_proof_get(ref, i) for i in (0, N - 1)]
    del ref
    ex = vc.vc_exec_create(0, 6)
    try:
        for rnd in (1, lK):
            vc.vc_test_zero_challenge(rnd)
            with pytest.raises(vc.VCError) as e:
                vc.vc_open_all(pp, cm, b)
            assert e.value.code == vc.VC_ECHALLENGE
            with pytest.raises(vc.VCError) as e:
                vc.vc_open_all_batch([(pp, cm, b), (pp, cm, b)], [ex])
            assert e.value.code == vc.VC_ECHALLENGE
    finally:
        vc.vc_test_zero_challenge(0)
    got = vc.vc_open_all_batch([(pp, cm, b)], [ex])[0]
    assert [vc.vc_proof_get(got, i) for i in (0, N - 1)] == want
    again = vc.vc_open_all(pp, cm, b)
    assert [vc.vc_proof_get(again, i) for i in (0, N - 1)] == want


@pytest.mark.parametrize("L,b", [(8, 16), (10, 3), (12, 1), (16, 256)])
def test_direct_rounds_equal_rounds_ahead(vc, L, b):
    """Step 1 with every round direct (an executor with vc_exec_set_ahead(0): the paper's
    order) gives the same bytes as the default schedule, which takes terms one round ahead
    at these sizes but (12, 1), direct by default (Eq. (folding): the lookahead only regroups
    the same pairings; test_gpu_lanes.py has schedules that go direct first and then ahead)."""
    say("direct rounds: L=%d b=%d" % (L, b))
    pp = vc.vc_setup(L, SEED, 0)
    N = 1 << L
    cm = vc.vc_commit(pp, dev_entries(I.entries(N, 90 + L)), 256)
    ref = vc.vc_open_all(pp, cm, b)
    ex = vc.vc_exec_create(0, 6)
    ex.set_ahead(0)
    got = vc.vc_open_all_ex(pp, cm, b, ex)
    for k in range((pp.K + b - 1) // b):
        for w in ("fc_x", "fc_rounds", "fc_tail"):
            assert got.export(w, k) == ref.export(w, k), (w, k)
    for w in ("merkle", "rho", "y", "D", "W"):
        assert got.export(w) == ref.export(w), w
    for i in (0, N // 2 + 1, N - 1):
        assert vc.vc_proof_get(got, i) == vc.vc_proof_get(ref, i), i


def sample_indices(N, M, b, seed, extra=()):
    """edges of the first and last batch and block, plus seeded random positions"""
    rng = np.random.default_rng(seed)
    K = N // M
    base = {0, 1, M - 1, M, N - 1, N - M, min(b, K - 1) * M, ((K - 1) // b) * b * M}
    base |= set(int(x) for x in rng.integers(0, N, 24))
    return sorted(i for i in base | set(extra) if 0 <= i < N)


def test_full_n16_b256_u32(vc):
    """The benchmark workload (N = 2^16, b = log^2 N = 256, uniform 32-bit entries, seed 2):
    every exported array, and sampled serialized proofs, byte for byte."""
    cs = Case(vc, 16, 256, seed=2, bits=32)
    compare_all(vc, cs, proofs=sample_indices(1 << 16, 256, 256, 2))


def test_n16_b16_u32(vc):
    cs = Case(vc, 16, 16, seed=2, bits=32)
    compare_all(vc, cs, proofs=sample_indices(1 << 16, 256, 16, 3))


def test_full_n20_b400(vc):
    """N = 2^20, b = log^2 N = 400 (3 batches, the last with 224 entries), full-width entries
    (seed 3): every exported array and sampled proofs."""
    cs = Case(vc, 20, 400, seed=3, bits=256)
    compare_all(vc, cs, proofs=sample_indices(1 << 20, 1024, 400, 4))


def test_n14_b1_direct_wide_sampled(vc):
    """N = 2^14, b = 1: 128 batches fill the device, so the rounds run direct, the first ones
    (at least 4096 pairs) with the Miller loops and G2 folds on the wide layout.  Sampled
    proofs against the oracle's one-proof-at-a-time construction and its verifier."""
    L, b = 14, 1
    say("case L=14 b=1 (direct rounds, sampled)")
    limbs = I.entries(1 << L, 7, 256)
    ints = I.limbs_to_ints(limbs)
    gpp = vc.vc_setup(L, SEED, 0)
    gcm = vc.vc_commit(gpp, dev_entries(limbs), 256)
    gpr = vc.vc_open_all(gpp, gcm, b)
    torch.cuda.synchronize()
    opp = O.Params(L, SEED)
    m_le = I.limbs_to_bytes(limbs)
    for i in (0, 129, 8191, 16383):
        proof = vc.vc_proof_get(gpr, i)
        assert proof == O.naive_proof(opp, m_le, b, i), i
        assert O.verify(opp, gcm.C, b, i, ints[i], proof) == 1, i


def dev_le32(limbs: np.ndarray):
    """the entries as N x 32 little-endian bytes on the device (what the verifiers read)"""
    return torch.frombuffer(bytearray(I.limbs_to_bytes(limbs)), dtype=torch.uint8).cuda()


def verify_every_proof(V, gpp, gcm, gpr, b, limbs):
    """all N proofs serialized on the device and checked by vc_verify_all (the random-weight
    combination of every PST check plus the FC check of every batch)"""
    ser = V.vc_proofs_serialize(gpr)
    v, alone = V.vc_verify_all(gpp, gcm.C, b, dev_le32(limbs), ser, bytes(range(32)))
    say("  verify_all over %d proofs: %d (%d checked alone)" % (gpp.N, v, alone))
    assert v == 1
    del ser
    torch.cuda.empty_cache()


@pytest.mark.timeout(900)
def test_full_n16_b1_u32(vc):
    """N = 2^16, b = 1 (256 FC batches, the device-full direct rounds with wide Miller loops
    and G2 folds), 32-bit entries (seed 2): every batch's fc_x / fc_rounds / fc_tail and every
    Step-2 array against the oracle's whole OpenAll, sampled serialized proofs, and every
    proof through the GPU verifier."""
    cs = Case(vc, 16, 1, seed=2, bits=32)
    compare_all(vc, cs, proofs=sample_indices(1 << 16, 256, 1, 5, extra=(129 * 256, 200 * 256 + 77)))
    verify_every_proof(vc, cs.gpp, cs.gcm, cs.gpr, 1, I.entries(1 << 16, 2, 32))


@pytest.mark.timeout(900)
def test_full_n20_b20(vc):
    """N = 2^20, b = 20 (52 FC batches, the last with t = 4), full-width entries (seed 3):
    every batch's FC arrays and every Step-2 array against the oracle's whole OpenAll;
    sampled proofs including the first and last of the short batch and of middle batches;
    every proof through the GPU verifier."""
    cs = Case(vc, 20, 20, seed=3, bits=256)
    M = 1024
    extra = (1020 * M, 1020 * M + 1, 1023 * M + 1023, 500 * M, 519 * M + 1023, 260 * M + 5, 279 * M)
    compare_all(vc, cs, proofs=sample_indices(1 << 20, M, 20, 6, extra=extra))
    verify_every_proof(vc, cs.gpp, cs.gcm, cs.gpr, 20, I.entries(1 << 20, 3, 256))


@pytest.mark.timeout(900)
def test_n20_b1_blocks(vc):
    """N = 2^20, b = 1 (1024 FC batches): the oracle's whole OpenAll is beyond a test here, so
    34 batches spread over the range (first and last included) are computed by the oracle's
    Step 1 for those blocks alone and compared whole; the Step-2 arrays (which do not depend
    on b) against the oracle's OpenAll at b = 400; sampled proofs against the one-proof-at-a-
    time construction; every proof through the GPU verifier."""
    L, b = 20, 1
    say("case L=20 b=1 (34 whole batches)")
    limbs = I.entries(1 << L, 3, 256)
    ints = I.limbs_to_ints(limbs)
    gpp = vc.vc_setup(L, SEED, 0)
    gcm = vc.vc_commit(gpp, dev_entries(limbs), 256)
    gpr = vc.vc_open_all(gpp, gcm, b)
    torch.cuda.synchronize()
    say("  GPU done; oracle commit")
    opp, ocm = oracle_commitment(L, 3, 256, limbs)
    m_le = I.limbs_to_bytes(limbs)
    assert gcm.export("Cj") == b"".join(ocm.Cj) and gcm.C == ocm.C
    ks = sorted(set([0, 1, 2, 511, 512, 1022, 1023] + [int(x) for x in np.linspace(3, 1021, 27)]))
    assert len(ks) >= 32
    say("  oracle Step 1 for %d blocks" % len(ks))
    blocks = ocm.open_blocks(b, ks)
    for k, blk in zip(ks, blocks):
        for w in ("fc_x", "fc_rounds", "fc_tail"):
            assert gpr.export(w, k) == blk[w], (w, k)
    say("  oracle Step 2 (OpenAll at b = 400)")
    oop = oracle_opening(L, 3, 256, limbs, 400)
    for w in ("merkle", "rho", "y", "D", "W"):
        assert gpr.export(w) == oop.export(w), w
    for i in (0, 1023, 777777, (1 << 20) - 1):
        proof = vc.vc_proof_get(gpr, i)
        assert proof == O.naive_proof(opp, m_le, b, i), i
        assert O.verify(opp, gcm.C, b, i, ints[i], proof) == 1, i
    verify_every_proof(vc, gpp, gcm, gpr, b, limbs)


@pytest.mark.timeout(1200)
def test_n22_b484_beyond_2_20(vc):
    """N = 2^22 (K = M = 2048, past the shared-memory KZG quotient and the 1024-entry
    batches), b = log^2 N = 484 (5 batches, the last with 112 entries), full-width entries
    (seed 3): every exported array against the oracle's OpenAll, sampled proofs byte for
    byte and through the oracle's verifier, one proof against the oracle's one-proof-at-a-time
    construction."""
    L, b = 22, 484
    cs = Case(vc, L, b, seed=3, bits=256)
    N, M = 1 << L, 2048
    idx = sample_indices(N, M, b, 7, extra=(4 * b * M, 4 * b * M + 111 * M + M - 1))
    compare_all(vc, cs, proofs=idx)
    limbs = I.entries(N, 3, 256)
    for i in idx[:6]:
        assert O.verify(cs.opp, cs.gcm.C, b, i, cs.m[i], vc.vc_proof_get(cs.gpr, i)) == 1, i
    i = N - 1
    assert vc.vc_proof_get(cs.gpr, i) == O.naive_proof(cs.opp, I.limbs_to_bytes(limbs), b, i)


def test_setup_size_limits(vc):
    with pytest.raises(vc.VCError) as e:
        vc.vc_setup(31, SEED, 0)
    assert e.value.code == vc.VC_EINVAL
    with pytest.raises(vc.VCError) as e:
        vc.vc_setup(1, SEED, 0)
    assert e.value.code == vc.VC_EINVAL
