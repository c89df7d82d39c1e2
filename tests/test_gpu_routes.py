"""Sizes on both sides of the lines where the dispatch goes from one kernel to another."""
import ctypes as C
import random

import numpy as np
import pytest

import oracle as O
from paper_2601_03031_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_03031_amd as V
    V.lib()
    return V


@pytest.mark.parametrize("L,b", [(14, 2), (14, 1)])
def test_verify_products(vc, L, b):
    """One check of every batch: 64 (20 products each, 1280) and 128 batches (19 each, 2432), the
    multiplications on the engine and on single lanes (from 2049 on).  The proofs verify; a byte changed in a
    round's point of one batch (an invalid encoding or another point) does not."""
    print("verify_all L=%d b=%d" % (L, b), flush=True)
    limbs = I.entries(1 << L, 77 + b, 256)
    m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
    pp = vc.vc_setup(L, I.TRAPDOOR_SEED, 0)
    cm = vc.vc_commit(pp, m, 256)
    pr = vc.vc_open_all(pp, cm, b)
    proofs = vc.vc_proofs_serialize(pr)
    le = m.reshape(-1)
    seed = bytes(random.Random(5).randrange(256) for _ in range(32))
    assert vc.vc_verify_all(pp, cm.C, b, le, proofs, seed)[0] == 1
    bad = proofs.clone()
    bad[32 * b + 384 + 20] ^= 1  # L_g1 of round 1 of the first batch
    assert vc.vc_verify_all(pp, cm.C, b, le, bad, seed)[0] == 0


@pytest.mark.parametrize("b", [31, 33, 64])
def test_verify_chunks(vc, b):
    """Batches whose last chunk of 32 block commitments is short, one over, or full (2^12 entries,
    64 subvectors): a proof of the first and of the last batch verifies, with another entry it does
    not."""
    L = 12
    print("verify L=%d b=%d" % (L, b), flush=True)
    limbs = I.entries(1 << L, 90 + b, 256)
    ints = I.limbs_to_ints(limbs)
    m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
    pp = vc.vc_setup(L, I.TRAPDOOR_SEED, 0)
    cm = vc.vc_commit(pp, m, 256)
    pr = vc.vc_open_all(pp, cm, b)
    for i in (0, (1 << L) - 1):
        proof = vc.vc_proof_get(pr, i)
        assert vc.vc_verify(pp, cm.C, b, i, ints[i], proof) == 1, i
        assert vc.vc_verify(pp, cm.C, b, i, ints[i] ^ 1, proof) == 0, i


@pytest.mark.parametrize("L", [4, 7])
def test_msm_digits(vc, L):
    """Entries whose bytes are 0, 1, 0x7f, 0x80, 0x81 and 0xff, alone and in runs (the signed digits' ends
    and their carries), and those next to 0 and r: every C_j and C as the oracle's."""
    print("msm digits L=%d" % L, flush=True)
    N = 1 << L
    runs = [int.from_bytes(bytes([0x2f] + [b] * 31), "big") for b in (0x00, 0x01, 0x7f, 0x80, 0x81, 0xff)]
    vals = runs + [0, 1, 127, 128, 129, 255, 256, O.R - 1, O.R - 128, O.R - 129, 1 << 253, (1 << 248) - 1, (1 << 128) - 1]
    vals += [0x80 << 8 * i for i in range(31)] + [0x7f80 << 8 * i for i in range(30)]
    vals = [v % O.R for v in (vals * (N // len(vals) + 1))[:N]] if len(vals) < N else vals[:N]
    limbs = np.frombuffer(b"".join(v.to_bytes(32, "little") for v in vals), dtype=np.uint64).reshape(N, 4).copy()
    ocm = O.Commitment(O.Params(L, I.TRAPDOOR_SEED), I.limbs_to_bytes(limbs))
    m = torch.from_numpy(limbs.view(np.uint8).reshape(-1).copy()).cuda()
    cm = vc.vc_commit(vc.vc_setup(L, I.TRAPDOOR_SEED, 0), m, 256)
    assert cm.export("Cj") == b"".join(ocm.Cj)
    assert cm.C == ocm.C


@pytest.mark.parametrize("L,b", [(5, 3), (8, 16), (7, 1)])
def test_serialize(vc, L, b):
    """All proofs in one launch equal the proofs gathered one by one (a short last batch, one batch, a batch
    per subvector), to a 16-byte boundary and to one that is not."""
    print("serialize L=%d b=%d" % (L, b), flush=True)
    limbs = I.entries(1 << L, 60 + b, 256)
    m = torch.from_numpy(np.ascontiguousarray(limbs).view(np.uint8).reshape(-1).copy()).cuda()
    pp = vc.vc_setup(L, I.TRAPDOOR_SEED, 0)
    pr = vc.vc_open_all(pp, vc.vc_commit(pp, m, 256), b)
    want = b"".join(vc.vc_proof_get(pr, i) for i in range(1 << L))
    assert bytes(vc.vc_proofs_serialize(pr).cpu().numpy().tobytes()) == want
    buf = torch.zeros(len(want) + 64, dtype=torch.uint8, device="cuda")
    n = C.c_uint64(0)
    assert vc.lib().vc_proofs_serialize(pr.ptr, C.c_void_p(buf.data_ptr() + 5), len(want), C.byref(n)) == 0
    out = buf.cpu().numpy().tobytes()
    assert n.value == len(want) and out[5:5 + len(want)] == want
    assert not any(out[:5]) and not any(out[5 + len(want):])


def test_serialize_two_dimensions(vc):
    """2^17 proofs: the workgroups of the second half lie in the grid's second dimension.  All proofs
    verify, and some of both halves equal the proofs gathered one by one."""
    L, b = 17, 256
    print("serialize L=%d b=%d" % (L, b), flush=True)
    m = I.device_entries(1 << L, 171)
    pp = vc.vc_setup(L, I.TRAPDOOR_SEED, 0)
    cm = vc.vc_commit(pp, m, 256)
    pr = vc.vc_open_all(pp, cm, b)
    proofs = vc.vc_proofs_serialize(pr)
    offs = vc.proof_offsets(pp, b)
    for i in (0, 1, 65535, 65536, 65537, 100003, 131071):
        assert proofs[offs[i]:offs[i + 1]].cpu().numpy().tobytes() == vc.vc_proof_get(pr, i), i
    assert vc.vc_verify_all(pp, cm.C, b, m, proofs, bytes(range(32))) == (1, 1)  # (its one batch)
