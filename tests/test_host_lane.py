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


def value(limbs):
    return sum(v << 29 * j for j, v in enumerate(limbs))


def top_of(v):
    """the top limb that leaves the value near v p with the other limbs near zero"""
    return int(v * O.P) >> 232


def test_pair_multiplication(hc):
    """k Q + A on G2 by two lanes: scalars at the ends and random ones, the identity in either place."""
    gen = O.generators()[1]
    rng = random.Random(720)
    rnd = lambda: O.g2_op("mul", gen, O.be32(rng.randrange(1, O.R)))
    inf = bytes(128)
    Q = rnd()
    cases = [(Q, k, inf) for k in (0, 1, 2, 3, O.R - 1, O.R - 2, 1 << 64, (1 << 66) - 1, O.R >> 1)]
    cases += [(inf, 5, inf), (inf, 5, Q), (Q, 0, Q), (Q, 1, Q), (Q, O.R - 1, Q), (Q, 2, O.g2_op("neg", Q))]
    cases += [(rnd(), rng.randrange(O.R), rnd()) for _ in range(60)]
    for q, k, a in cases:
        o = C.create_string_buffer(128)
        hc.hc_pair_mul(q, O.be32(k), a, o)
        want = O.g2_op("mul", q, O.be32(k)) if any(q) and k else inf
        assert o.raw == O.g2_op("add", want, a), k


@pytest.mark.parametrize("n", [1, 2, 5])
def test_pair_miller(hc, n):
    """The product of n Miller values by two lanes each: the pairing after the final exponentiation."""
    g1, g2 = O.generators()
    rng = random.Random(730 + n)
    for _ in range(3):
        P = [O.g1_op("mul", g1, O.be32(rng.randrange(1, O.R))) for _ in range(n)]
        Q = [O.g2_op("mul", g2, O.be32(rng.randrange(1, O.R))) for _ in range(n)]
        f, e = C.create_string_buffer(384), C.create_string_buffer(384)
        hc.hc_pair_miller(b"".join(P), b"".join(Q), n, f)
        assert hc.hc_fp12(3, f.raw, f.raw, e) == 0
        assert e.raw == O.pairing(P, Q)


@pytest.mark.parametrize("which", ["msm on G1", "msm on G2", "multiplication on G1", "multiplication on G2 by two lanes", "Miller loop"])
def test_bounds(hc, which):
    """The formulas run on bounds of limbs and values: no column reaches 2^63, no limb 2^31, no argument of a
    reduction 2^9 p, every value packed lies within p of zero (one subtraction makes it canonical), and
    sums of any length keep within the bounds found, coordinates below p."""
    w = (C.c_double * 5)()
    closed = hc.hc_lane_bounds(("msm on G1", "msm on G2", "multiplication on G1", "multiplication on G2 by two lanes",
                                "Miller loop").index(which), w)
    print(which, list(w))
    column, limb, reduced, packed, coordinate = w
    assert closed and column < 1 and limb < 1 and reduced < 1 and packed < 2 and coordinate < 1


def test_products_at_the_bound(hc):
    """Six products whose factors' limbs are as large as twelve units allow (sqrt 2 each, and two by one), of
    all signs: exact, with centred limbs and a value below 0.5 p + sum |a b| / 169 p."""
    rng = random.Random(740)
    inv = pow(1 << 261, -1, O.P)
    for units in ((1.414, 1.414), (2.0, 1.0)):
        for signs in range(40):
            def limbs(u):
                m = int(u * (1 << 28))
                f = (lambda: m) if signs == 0 else (lambda: -m) if signs == 1 else (lambda: rng.choice((m, -m)))
                return [f() for _ in range(8)] + [rng.choice((1, -1)) * top_of(1.9)]
            a, b = [limbs(units[0]) for _ in range(6)], [limbs(units[1]) for _ in range(6)]
            o = (C.c_int32 * 9)()
            hc.hc_lane_dot6((C.c_int32 * 54)(*sum(a, [])), (C.c_int32 * 54)(*sum(b, [])), o)
            got, want = value(list(o)), sum(value(x) * value(y) for x, y in zip(a, b))
            assert (got - want * inv) % O.P == 0
            assert all(-(1 << 28) <= v < 1 << 28 for v in o[:8])
            assert abs(got) <= (0.5 + 1e-6) * O.P + sum(abs(value(x) * value(y)) for x, y in zip(a, b)) / (1 << 261)


def test_reduction_at_the_bound(hc):
    """k a + b up to 2^9 p: the value modulo p, within 0.51 p, limbs of one unit."""
    rng = random.Random(750)
    for k in (-3, -2, -1, 1, 2, 3, 8, 9, 12):
        for v in (0, 0.499, 0.5, 0.501, 1, 7.5, 20, 31.9):
            for _ in range(6):
                lim = lambda t, u: [rng.choice((1, -1)) * int(u * (1 << 28)) for _ in range(8)] + [rng.choice((1, -1)) * top_of(t)]
                a, b = lim(v, 1), lim(v, 2)
                o = (C.c_int32 * 9)()
                hc.hc_lane_reduce((C.c_int32 * 9)(*a), k, (C.c_int32 * 9)(*b), o)
                got = value(list(o))
                assert (got - k * value(a) - value(b)) % O.P == 0
                assert abs(got) < 0.51 * O.P and all(abs(x) <= (1 << 28) + (1 << 12) for x in o[:8])


def test_engine_slots_at_the_bound(hc):
    """The engine's loose limbs at their ends: a sum's slot (two reduced halves, limbs to 2^30 + 2^18 either
    way) made canonical, and a reduction of columns whose coefficients add up to 2^15 on such limbs."""
    rng = random.Random(760)
    ends = ((1 << 30) + (1 << 18), -(1 << 30) - (1 << 18), (1 << 29) + (1 << 17), 0, -1)
    for t in range(300):
        l = [(ends[t] if t < len(ends) else rng.choice(ends)) for _ in range(8)]
        # a value in (-2p, 5p) with these lower limbs
        top = rng.choice([top_of(v) for v in (-1.1, -0.5, 0, 0.5, 1.2, 2.5, 4.5)])
        l.append(top - (value(l) >> 232))
        out = C.create_string_buffer(32)
        hc.hc_canon29((C.c_int32 * 9)(*l), out)
        # (slots hold Montgomery residues with the factor 2^256; written out without it)
        assert int.from_bytes(out.raw, "big") == value(l) * pow(1 << 256, -1, O.P) % O.P, l
    for t in range(300):
        k = (1 << 15) - 1
        c = [k * rng.choice(ends[:2]) for _ in range(8)] + [rng.choice((1, -1)) * rng.randrange(int(k * 1.2 * O.P) >> 232)]
        o = (C.c_int32 * 9)()
        hc.hc_red29((C.c_int64 * 9)(*c), o)
        got = value(list(o))
        assert (got - value(c)) % O.P == 0 and abs(got) < 0.54 * O.P
        assert all(-(1 << 17) - 1 <= v <= (1 << 29) + (1 << 17) for v in o[:8])


def test_accumulators_are_products(hc):
    """The slots whose sums are taken outside the programs (the accumulator's, up to four a component) are
    written by products, with limbs below 2^29, or hold 0 or 1."""
    assert [hc.hc_sums_into_T(i) for i in range(9)] == [0] * 9
