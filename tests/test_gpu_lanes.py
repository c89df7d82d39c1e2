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
