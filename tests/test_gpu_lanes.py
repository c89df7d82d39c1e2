"""Open-alls whose rounds take the kernels on single lanes and on pairs of lanes."""
import numpy as np
import pytest

import oracle as O
from paper_2601_03031_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEED = I.TRAPDOOR_SEED


@pytest.fixture(scope="module")
def vc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_03031_amd as V
    V.lib()
    return V


def to_device(limbs):
    return torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()


@pytest.mark.parametrize("rows", [(), (3, 64, 127)])
def test_identity_commitments(vc, rows):
    """2^14 entries, b = 1, all of them zero but those of a few subvectors: the commitments of the others are
    the identity, in both places of the Miller loops, terms and folds of rounds 1 and 2 (8192 and 4096 pairs,
    on lanes) and of the rounds on the engine; every array of every batch as the oracle's."""
    L, b = 14, 1
    print("identity commitments, rows", rows, flush=True)
    N, M = 1 << L, 1 << 7
    limbs = np.zeros((N, 4), dtype=np.uint64)
    src = I.entries(N, 141, 256)
    for j in rows:
        limbs[j * M:(j + 1) * M] = src[j * M:(j + 1) * M]
    ocm = O.Commitment(O.Params(L, SEED), I.limbs_to_bytes(limbs))
    oop = O.Opening(ocm, b)
    print("  oracle done", flush=True)
    pp = vc.vc_setup(L, SEED, 0)
    cm = vc.vc_commit(pp, to_device(limbs), 256)
    assert cm.export("Cj") == b"".join(ocm.Cj) and cm.C == ocm.C
    pr = vc.vc_open_all(pp, cm, b)
    for k in range(oop.nb):
        for w in ("fc_x", "fc_rounds", "fc_tail"):
            assert pr.export(w, k) == oop.export(w, k), (w, k)
    for w in ("merkle", "rho", "y", "D", "W"):
        assert pr.export(w) == oop.export(w), w
    for i in (0, 3 * M + 1, 64 * M, N - 1):
        assert vc.vc_proof_get(pr, i) == oop.proof(i), i


def same_step1(vc, pp, got, ref):
    for k in range((pp.K + got.b - 1) // got.b):
        for w in ("fc_x", "fc_rounds", "fc_tail"):
            assert got.export(w, k) == ref.export(w, k), (w, k)


@pytest.mark.parametrize("L,b,bound", [(8, 16, 4096), (10, 3, 4096), (12, 1, 4096), (14, 4, 4096), (16, 256, 4096), (16, 128, None), (18, 128, None)])
def test_rounds_ahead_equal_direct_rounds(vc, L, b, bound):
    """Rounds taken ahead (a caller's bound of 4096 pairs, or None: the default rule, which takes them ahead
    at these sizes) give the same bytes as direct rounds (a bound of 0).  (12, 1) and (14, 4) go
    direct first and then ahead; their first terms ahead are 4096, sums of 8 and of 16 by lanes, and those of
    (18, 128) sums of 64; (16, 128) has 1024, on the engine."""
    print("rounds ahead L=%d b=%d bound=%s" % (L, b, bound), flush=True)
    pp = vc.vc_setup(L, SEED, 0)
    cm = vc.vc_commit(pp, I.device_entries(1 << L, 180 + L), 256)
    direct, other = vc.vc_exec_create(0, 6), vc.vc_exec_create(0, 6)
    direct.set_ahead(0)
    if bound is not None:
        other.set_ahead(bound)
    ref = vc.vc_open_all_ex(pp, cm, b, direct)
    got = vc.vc_open_all_ex(pp, cm, b, other)
    same_step1(vc, pp, got, ref)
    for w in ("merkle", "rho", "D", "W"):
        assert got.export(w) == ref.export(w), w
    for i in (0, pp.N // 2 + 1, pp.N - 1):
        assert vc.vc_proof_get(got, i) == vc.vc_proof_get(ref, i), i


def test_blocks_in_turn(vc):
    """2^18 entries, b = 1: the terms and G2 folds of round 1 have 262144 lanes, twice as many as the launch's
    workgroups, and the G1 folds 131072, as many: every proof verifies."""
    L, b = 18, 1
    print("blocks in turn L=%d" % L, flush=True)
    pp = vc.vc_setup(L, SEED, 0)
    m = I.device_entries(1 << L, 188)
    cm = vc.vc_commit(pp, m, 256)
    proofs = vc.vc_proofs_serialize(vc.vc_open_all(pp, cm, b))
    assert vc.vc_verify_all(pp, cm.C, b, m, proofs, bytes(range(32))) == (1, pp.K)


@pytest.mark.parametrize("L,b", [(12, 1), (14, 2), (14, 3)])
def test_direct_rounds_at_the_lines(vc, L, b):
    """Direct rounds at the lines where lanes take over from the engine (4096): (12, 1) has 4096 terms in round 1
    and 2048 folds, (14, 2) 8192 terms, 4096 folds and, in round 2, 4096 terms; (14, 3) has 43 batches, 5504 and
    2752 terms and 2752 folds, blocks that hold parts of two batches.  Every array of Step 1 as the oracle's."""
    print("direct rounds L=%d b=%d" % (L, b), flush=True)
    limbs = I.entries(1 << L, 200 + 10 * L + b, 256)
    ocm = O.Commitment(O.Params(L, SEED), I.limbs_to_bytes(limbs))
    oop = O.Opening(ocm, b)
    print("  oracle done", flush=True)
    pp = vc.vc_setup(L, SEED, 0)
    cm = vc.vc_commit(pp, to_device(limbs), 256)
    ex = vc.vc_exec_create(0, 6)
    ex.set_ahead(0)
    pr = vc.vc_open_all_ex(pp, cm, b, ex)
    assert oop.nb == -(-pp.K // b)
    same_step1(vc, pp, pr, oop)
    for i in (0, pp.N - 1):
        assert vc.vc_proof_get(pr, i) == oop.proof(i), i
