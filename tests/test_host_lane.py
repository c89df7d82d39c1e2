"""The one-lane limbs and complete additions of the throughput kernels on the host build, against the
oracle's group law."""
import ctypes as C
import os
import random

import pytest

import oracle as O

HC_PATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_03031_amd", "lib",
                       "libvc_hostcheck.so")


@pytest.fixture(scope="module")
def hc():
    if not os.path.exists(HC_PATH):
        from paper_2601_03031_amd import build as B
        B.build_hostcheck()
    return C.CDLL(HC_PATH)


@pytest.mark.parametrize("grp", [0, 1])
def test_sums(hc, grp):
    """Two sums of points, one added to the other: random points, the same point over and over (mixed
    additions that double), a point and its opposite (the identity inside and at the end), identities
    among the inputs, equal and opposite sums."""
    gen = O.generators()[grp]
    op, size = ((O.g1_op, 64), (O.g2_op, 128))[grp]
    rng = random.Random(700 + grp)
    rnd = lambda: op("mul", gen, O.be32(rng.randrange(1, O.R)))
    inf = bytes(size)
    a, b = rnd(), rnd()
    na = op("neg", a)
    lists = [([rnd() for _ in range(12)], 5), ([a] * 9, 4), ([a] * 8, 4), ([a, na], 2), ([a, na, b], 2), ([a, b, a, b], 2),
             ([a, b, na, op("neg", b)], 2), ([inf, a, inf], 1), ([inf, inf], 1), ([a], 1), ([a], 0), ([], 0),
             ([a, a, na, na, a], 3), ([rnd() for _ in range(40)], 40)]
    for pts, m in lists:
        want = inf
        for p in pts:
            want = op("add", want, p)
        o = C.create_string_buffer(size)
        hc.hc_lane_sum(grp, b"".join(pts), len(pts), m, o)
        assert o.raw == want, (len(pts), m)


def test_multiplication(hc):
    """k P on G1 over the split of k: the scalars at the ends, those whose split has one part only or
    negative parts, and random ones; the identity."""
    gen = O.generators()[0]
    rng = random.Random(710)
    rnd = lambda: O.g1_op("mul", gen, O.be32(rng.randrange(1, O.R)))
    P = rnd()
    ks = [0, 1, 2, 3, 4, 5, 15, 16, 17, O.R - 1, O.R - 2, 1 << 64, (1 << 64) - 1, 1 << 127, O.R >> 1]
    cases = [(P, k) for k in ks] + [(bytes(64), 5)] + [(rnd(), rng.randrange(O.R)) for _ in range(300)]
    for p, k in cases:
        o = C.create_string_buffer(64)
        hc.hc_lane_mul(p, O.be32(k), o)
        assert o.raw == (O.g1_op("mul", p, O.be32(k)) if any(p) else bytes(64)), k
