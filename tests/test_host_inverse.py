"""The modular inverse by batched division steps and the windowed power on loose limbs, on the host
build, against Python's."""
import ctypes as C
import os
import random

import pytest

import oracle as O

HC_PATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_03031_amd", "lib",
                       "libvc_hostcheck.so")
P, R = O.P, O.R


@pytest.fixture(scope="module")
def hc():
    if not os.path.exists(HC_PATH):
        from paper_2601_03031_amd import build as B
        B.build_hostcheck()
    return C.CDLL(HC_PATH)


@pytest.mark.parametrize("which,mod", [(0, P), (1, R)])
def test_inverse(hc, which, mod):
    """Small and large values, powers of two (runs of zero bits longer than a batch), values next to
    multiples of them, and the zero that maps to zero."""
    rng = random.Random(900 + which)
    vals = [0, 1, 2, 3, 62, 63, mod - 1, mod - 2, mod // 2, mod // 2 + 1, mod // 3]
    vals += [1 << s for s in (29, 30, 31, 60, 64, 90, 128, 240, 253)]
    vals += [(1 << s) + d for s in (30, 60, 120, 250) for d in (-1, 1)]
    vals += [rng.randrange(mod) for _ in range(300)] + [rng.randrange(1 << 40) for _ in range(40)]
    for x in vals:
        o = C.create_string_buffer(32)
        hc.hc_field(which, 4, O.be32(x), O.be32(x), o)
        assert int.from_bytes(o.raw, "big") == (pow(x, -1, mod) if x else 0), x


@pytest.mark.parametrize("which,mod", [(0, P), (1, R)])
def test_pow_fixed(hc, which, mod):
    """Exponents of one bit, runs of ones and zeros, windows cut off at bit 0; bases at the ends of
    the range."""
    rng = random.Random(910 + which)
    exps = [1, 2, 3, 5, 15, 16, 17, 30, (1 << 255) | 1, (1 << 256) - 1, 1 << 255, (P - 3) // 4, mod - 2]
    exps += [rng.randrange(1, 1 << 256) for _ in range(10)]
    for x in [0, 1, mod - 1, 2, (1 << 253) % mod] + [rng.randrange(mod) for _ in range(5)]:
        for e in exps:
            o = C.create_string_buffer(32)
            hc.hc_pow_fixed(which, O.be32(x), O.be32(e), o)
            assert int.from_bytes(o.raw, "big") == pow(x, e, mod), (x, e)


def division_steps(n, delta, f, g):
    """n division steps by their definition: 2^n times the matrix that takes f and g to theirs, and delta"""
    u, v, q, r = 1, 0, 0, 1
    for _ in range(n):
        if delta > 0 and g & 1:
            delta, f, g, u, v, q, r = 1 - delta, g, (g - f) // 2, 2 * q, 2 * r, q - u, r - v
        else:
            b = g & 1
            delta, g, u, v, q, r = 1 + delta, (g + b * f) // 2, 2 * u, 2 * v, q + b * u, r + b * v
    return [u, v, q, r], delta


def test_batch(hc):
    """A batch's matrix and delta are those of 30 single steps: every small delta, runs without a swap as
    long as the batch and longer, g zero, even or all ones."""
    rng = random.Random(920)
    out = (C.c_int32 * 5)()
    deltas = list(range(-40, 41)) + [1] * 200
    for delta in deltas:
        for g in (0, 1, 2, 1 << 29, 1 << 30, 0xffffffff, 0x3fffffff, rng.getrandbits(32), rng.getrandbits(32) << 7 & 0xffffffff):
            f = rng.getrandbits(32) | 1
            hc.hc_divsteps_batch(C.c_int32(delta), C.c_uint32(f), C.c_uint32(g), out)
            assert (list(out[:4]), out[4]) == division_steps(30, delta, f, g), (delta, f, g)
