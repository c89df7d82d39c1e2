"""Generate slp_progs.hpp: straight-line programs (SLPs) over F_p for the
workgroup-cooperative engine in slp.hpp.

A program is a dataflow graph of base-field operations, produced by running the
formulas of the BN254 tower, the twist and the pairing on tracer values.  The
scheduler packs it into levels of independent operations; a workgroup executes a level
per step, a pair of lanes per operation (32 operations per wavefront).  Operations:
  MUL  dst = (sum_i k_i x_i) (sum_i l_i y_i)        (Montgomery product; a lane per factor)
  LIN  dst = sum_i k_i x_i  (mod p)                 (half of the terms per lane)
Linear combinations are kept symbolic by the tracer and materialised only where a
product or an output needs them, so chains of additions fuse into few LIN operations.
Slots are field elements in LDS.  An operand names a 2-bit segment and a 10-bit offset:
segment 0 is absolute, segments 1..3 are bases the caller sets before running a
relocatable program.

Programs:
  * the Miller loop of the optimal ate pairing, whole: the loop follows the non-adjacent form
    of 6u + 2; the closing additions use pi(Q) and -pi^2(Q);
  * the final exponentiation, whole but for its inversion in F_p;
  * F_p12 operations (relocatable: X in segment 1, Y in segment 2, D in segment 3): product,
    squarings, Frobenius powers, conjugate;
  * G1 and G2 scalar multiplication steps.

Run:  python gen_slp.py > slp_progs.hpp      (the build does this)
      python gen_slp.py --check              (run every program on random inputs
                                              against plain polynomial arithmetic)
"""
from __future__ import annotations

import random
import sys

U = 0x44E992B44A6909F1
P = 36 * U**4 + 36 * U**3 + 24 * U**2 + 6 * U + 1
R = 36 * U**4 + 36 * U**3 + 18 * U**2 + 6 * U + 1
RMONT = 1 << 256
SEG_SHIFT = 10         # a slot field: segment | offset
WAVE_OPS = 32          # operations of a level that one wavefront executes
KMAX = 127

OP_NOP, OP_MUL, OP_LIN = 0, 1, 2


# ============================================================================ tracer
LANE_TERMS = (2, 4, 6, 10, 14)  # terms that a lane sums (padded up to one of these; a record is
                                # whole groups of four words, two of them head and chain)
# Trace-time limits (set per program by build_all from TRACE_LIMITS): terms of a linear
# operation and terms of one factor of a product
NTERM = 16


class Prog:
    """SSA values: ('in', name) | ('const', x) | ('lin', terms) | ('mul', termsA, termsB);
    terms are tuples of (value id, small integer coefficient)"""

    def __init__(self, name):
        self.name = name
        self.vals = []
        self.inputs = {}
        self.outputs = {}
        self.consts = {}
        self.memo = {}
        self.zero = self.const(0)

    def new(self, node):
        key = node if node[0] in ("lin", "mul") else None
        if key is not None and key in self.memo:
            return self.memo[key]
        self.vals.append(node)
        v = len(self.vals) - 1
        if key is not None:
            self.memo[key] = v
        return v

    def inp(self, name):
        v = self.new(("in", name))
        self.inputs[name] = v
        return F(self, {v: 1})

    def const(self, x):
        x %= P
        if x not in self.consts:
            self.consts[x] = self.new(("const", x))
        return self.consts[x]

    def fconst(self, x):
        return F(self, {self.const(x): 1})

    def out(self, name, f):
        self.outputs[name] = f.atom()


def canon(terms):
    return tuple(sorted((k, c) for k, c in terms.items() if c != 0))


class F:
    """a base-field value: a small-integer linear combination of atoms (value ids)"""
    __slots__ = ("p", "t")

    def __init__(self, p, terms):
        self.p = p
        self.t = {k: c for k, c in terms.items() if c != 0}

    def _lin(self, o, s):
        t = dict(self.t)
        for k, c in o.t.items():
            t[k] = t.get(k, 0) + s * c
        return F(self.p, t)

    def __add__(self, o):
        return self._lin(o, 1)

    def __sub__(self, o):
        return self._lin(o, -1)

    def __neg__(self):
        return F(self.p, {k: -c for k, c in self.t.items()})

    def scale(self, k):
        return F(self.p, {a: c * k for a, c in self.t.items()})

    def __mul__(self, o):
        if not self.t or not o.t:
            return F(self.p, {})
        A, B = operand_terms(self.p, self.t), operand_terms(self.p, o.t)
        a, b = canon(A), canon(B)
        if b < a:
            a, b = b, a
        return F(self.p, {self.p.new(("mul", a, b)): 1})

    def sqr(self):
        return self * self

    def mul(self, o):
        return self * o

    def atom(self):
        if not self.t:
            return self.p.zero
        if len(self.t) == 1:
            (k, c), = self.t.items()
            if c == 1:
                return k
        a = materialise(self.p, self.t)
        self.t = {a: 1}
        return a


SIDE = 8


def operand_terms(p, t):
    """a factor of a product: coefficients within [-KMAX, KMAX], at most SIDE terms"""
    t = fit_coeffs(p, dict(t))
    if len(t) > SIDE:
        t = {materialise(p, t): 1}
    return t


def fit_coeffs(p, t):
    """rewrite terms whose coefficient exceeds KMAX through an intermediate LIN"""
    for k, c in list(t.items()):
        if abs(c) > KMAX:
            s = 1 if c > 0 else -1
            a = abs(c)
            f1 = next((d for d in range(KMAX, 1, -1) if a % d == 0 and a // d <= KMAX), None)
            del t[k]
            if f1:
                v = p.new(("lin", ((k, f1),)))
                t[v] = t.get(v, 0) + s * (a // f1)
            else:
                v = p.new(("lin", ((k, KMAX),)))
                t[v] = t.get(v, 0) + s * (a // KMAX)
                if a % KMAX:
                    t[k] = t.get(k, 0) + s * (a % KMAX)
            return fit_coeffs(p, {kk: cc for kk, cc in t.items() if cc})
    return t


def materialise(p, terms):
    """LIN operations computing sum c_k x_k, NTERM terms per operation, shallow tree"""
    t = fit_coeffs(p, {k: c for k, c in terms.items() if c != 0})
    if not t:
        return p.zero
    if len(t) == 1:
        (k, c), = t.items()
        if c == 1:
            return k
    items = sorted(t.items(), key=lambda kc: (-abs(kc[1]), kc[0]))
    if len(items) <= NTERM:
        return p.new(("lin", canon(dict(items))))
    n = len(items)
    g = -(-(n - NTERM) // (NTERM - 1))          # sub-sums needed
    raw = items[:NTERM - g]
    rest = items[NTERM - g:]
    subs = []
    per = -(-len(rest) // g)
    for i in range(0, len(rest), per):
        subs.append((materialise(p, dict(rest[i:i + per])), 1))
    return p.new(("lin", canon(dict(raw + subs))))


# ============================================================================ tower
def zero2(p):
    return F2(F(p, {}), F(p, {}))


class F2:
    __slots__ = ("c0", "c1")

    def __init__(self, c0, c1):
        self.c0, self.c1 = c0, c1

    def __add__(s, o):
        return F2(s.c0 + o.c0, s.c1 + o.c1)

    def __sub__(s, o):
        return F2(s.c0 - o.c0, s.c1 - o.c1)

    def __neg__(s):
        return F2(-s.c0, -s.c1)

    def scale(s, k):
        return F2(s.c0.scale(k), s.c1.scale(k))

    def is_zero(s):
        return not s.c0.t and not s.c1.t

    def mul(s, o, kara=False):
        if s.is_zero() or o.is_zero():
            return zero2(s.c0.p)
        a0, a1, b0, b1 = s.c0, s.c1, o.c0, o.c1
        if kara:
            v0, v1 = a0 * b0, a1 * b1
            return F2(v0 - v1, (a0 + a1) * (b0 + b1) - v0 - v1)
        return F2(a0 * b0 - a1 * b1, a0 * b1 + a1 * b0)

    def sqr(s):
        a0, a1 = s.c0, s.c1
        return F2((a0 + a1) * (a0 - a1), (a0 * a1).scale(2))

    def mul_fp(s, x):
        return F2(s.c0 * x, s.c1 * x)

    def mul_xi(s):  # (9 + i)(a0 + a1 i) = (9 a0 - a1) + (a0 + 9 a1) i
        return F2(s.c0.scale(9) - s.c1, s.c0 + s.c1.scale(9))

    def conj(s):
        return F2(s.c0, -s.c1)

    def mul_const(s, c):
        p = s.c0.p
        k0, k1 = c[0] % P, c[1] % P
        r0, r1 = F(p, {}), F(p, {})
        if k0:
            g = p.fconst(k0)
            r0 = r0 + s.c0 * g
            r1 = r1 + s.c1 * g
        if k1:
            g = p.fconst(k1)
            r0 = r0 - s.c1 * g
            r1 = r1 + s.c0 * g
        return F2(r0, r1)


class F6:
    __slots__ = ("c",)

    def __init__(self, c0, c1, c2):
        self.c = (c0, c1, c2)

    def __add__(s, o):
        return F6(*(x + y for x, y in zip(s.c, o.c)))

    def __sub__(s, o):
        return F6(*(x - y for x, y in zip(s.c, o.c)))

    def __neg__(s):
        return F6(*(-x for x in s.c))

    def mul(s, o, kara2=True):
        a0, a1, a2 = s.c
        b0, b1, b2 = o.c
        v0, v1, v2 = a0.mul(b0, kara2), a1.mul(b1, kara2), a2.mul(b2, kara2)
        c0 = v0 + ((a1 + a2).mul(b1 + b2, kara2) - v1 - v2).mul_xi()
        c1 = (a0 + a1).mul(b0 + b1, kara2) - v0 - v1 + v2.mul_xi()
        c2 = (a0 + a2).mul(b0 + b2, kara2) - v0 + v1 - v2
        return F6(c0, c1, c2)

    def mul_v(s):  # v (c0 + c1 v + c2 v^2) = xi c2 + c0 v + c1 v^2
        return F6(s.c[2].mul_xi(), s.c[0], s.c[1])


class F12:
    __slots__ = ("a", "b")

    def __init__(self, a, b):
        self.a, self.b = a, b

    def coeffs(self):  # memory order c0.c0.c0, c0.c0.c1, ..., c1.c2.c1
        out = []
        for h in (self.a, self.b):
            for q in h.c:
                out += [q.c0, q.c1]
        return out

    @staticmethod
    def of(cs):
        f2 = [F2(cs[2 * j], cs[2 * j + 1]) for j in range(6)]
        return F12(F6(*f2[:3]), F6(*f2[3:]))

    def mul(s, o, kara2=True):
        t0, t1 = s.a.mul(o.a, kara2), s.b.mul(o.b, kara2)
        c1 = (s.a + s.b).mul(o.a + o.b, kara2) - t0 - t1
        return F12(t0 + t1.mul_v(), c1)

    def sqr(s, kara2=True):
        # complex squaring over F_p6: t = a b, c0 = (a + b)(a + v b) - t - v t, c1 = 2t
        a, b = s.a, s.b
        t = a.mul(b, kara2)
        m = (a + b).mul(a + b.mul_v(), kara2)
        return F12(m - t - t.mul_v(), t + t)

    def conj(s):
        return F12(s.a, -s.b)


# ============================================================================ constants
def f2mul_int(a, b):
    return ((a[0] * b[0] - a[1] * b[1]) % P, (a[0] * b[1] + a[1] * b[0]) % P)


def f2pow_int(a, e):
    r = (1, 0)
    while e:
        if e & 1:
            r = f2mul_int(r, a)
        a = f2mul_int(a, a)
        e >>= 1
    return r


def f2inv_int(a):
    n = pow(a[0] * a[0] + a[1] * a[1], -1, P)
    return (a[0] * n % P, -a[1] * n % P)


XI = (9, 1)
TWIST_B = f2mul_int((3, 0), f2inv_int(XI))     # b' = 3 / xi
B3 = f2mul_int((3, 0), TWIST_B)                # 3 b'
B9 = f2mul_int((9, 0), TWIST_B)                # 9 b'
GAM1 = [f2pow_int(XI, k * (P - 1) // 6) for k in range(6)]
GAM2 = [f2pow_int(XI, k * (P * P - 1) // 6) for k in range(6)]
GAM3 = [f2pow_int(XI, k * (P**3 - 1) // 6) for k in range(6)]
assert all(g[1] == 0 for g in GAM2)
FROB_TX, FROB_TY = GAM1[2], GAM1[3]            # twist Frobenius: (conj(x) tx, conj(y) ty)
FROB2_TX = f2pow_int(XI, (P * P - 1) // 3)
FROB2_TY = f2pow_int(XI, (P * P - 1) // 2)
assert FROB2_TX[1] == 0 and FROB2_TY[1] == 0


def frob12(f, e):
    """f^{p^e}, e = 1, 2, 3: the F_p2 coefficient of w^k (k = 2q + h) maps to conj^e(c) gamma_e[k]"""
    p = f.a.c[0].c0.p
    out = []
    for h, half in enumerate((f.a, f.b)):
        for q, c in enumerate(half.c):
            k = 2 * q + h
            if e & 1:
                c = c.conj()
            if k == 0:
                out.append(c)
            elif e == 2:
                g = p.fconst(GAM2[k][0])
                out.append(F2(c.c0 * g, c.c1 * g))
            else:
                out.append(c.mul_const(GAM1[k] if e == 1 else GAM3[k]))
    return F12(F6(*out[:3]), F6(*out[3:]))


# ============================================================================ pairing formulas
def line_dbl(T, xP, yP):
    """T = (X, Y, Z, U) homogeneous projective on y^2 = x^3 + b' with U = 3 b' Z carried along, so
    that 3 b' Z^2 = Z U is ready in the first product level.  Returns 2T (scaled by 4)
    and the tangent at T evaluated at P up to an F_p2 factor, as (l0, l1, l3) meaning
    l0 + l1 w + l3 w^3:  l0 = 2YZ yP, l1 = -3X^2 xP, l3 = Y^2 - 3b'Z^2."""
    X, Y, Z, U = T
    XX, YY, E = X.sqr(), Y.sqr(), Z.mul(U)
    XY, YZ, YU = X.mul(Y), Y.mul(Z), Y.mul(U)
    X3 = XY.mul(YY - E.scale(3)).scale(2)  # 2 XY (Y^2 - 9b'Z^2)
    Y3 = (YY + E.scale(3)).sqr() - E.sqr().scale(12)
    Z3 = YY.mul(YZ).scale(8)               # 8 Y^3 Z
    U3 = YY.mul(YU).scale(8)
    l0 = YZ.scale(2).mul_fp(yP)
    l1 = XX.scale(-3).mul_fp(xP)
    l3 = YY - E
    return (X3, Y3, Z3, U3), (l0, l1, l3)


def line_add(T, Q, xP, yP):
    """T projective as above, Q = (xQ, yQ) affine: T + Q and the line through T and Q at P:
    l0 = lam yP, l1 = -theta xP, l3 = theta xQ - lam yQ  (theta = Y - yQ Z, lam = X - xQ Z)."""
    X, Y, Z, U = T
    xQ, yQ = Q
    th = Y - yQ.mul(Z)
    la = X - xQ.mul(Z)
    C, D = th.sqr(), la.sqr()
    E2 = la.mul(D)
    F2_ = Z.mul(C)
    G2 = X.mul(D)
    H2 = E2 + F2_ - G2.scale(2)
    X3 = la.mul(H2)
    Y3 = th.mul(G2 - H2) - Y.mul(la).mul(D)
    Z3 = Z.mul(la).mul(D)
    U3 = U.mul(la).mul(D)
    l0 = la.mul_fp(yP)
    l1 = (-th).mul_fp(xP)
    l3 = th.mul(xQ) - la.mul(yQ)
    return (X3, Y3, Z3, U3), (l0, l1, l3)


def line_to_f12(l):
    """l0 + l1 w + l3 w^3 = (l0, 0, 0) + (l1, l3, 0) w"""
    l0, l1, l3 = l
    z = zero2(l0.c0.p)
    return F12(F6(l0, z, z), F6(l1, l3, z))


def sparse01(x, b0, b1, kara2=True):
    """(x0 + x1 v + x2 v^2)(b0 + b1 v)"""
    x0, x1, x2 = x.c
    v0, v1 = x0.mul(b0, kara2), x1.mul(b1, kara2)
    c0 = v0 + x2.mul(b1, kara2).mul_xi()
    c1 = (x0 + x1).mul(b0 + b1, kara2) - v0 - v1
    c2 = x2.mul(b0, kara2) + v1
    return F6(c0, c1, c2)


def mul_by_line(f, l, kara2=True):
    """f (a + b w) with a = (l0, 0, 0), b = (l1, l3, 0)"""
    l0, l1, l3 = l
    f0, f1 = f.a, f.b
    t0 = F6(*(c.mul(l0, kara2) for c in f0.c))
    t1 = sparse01(f1, l1, l3, kara2)
    m = sparse01(f0 + f1, l0 + l1, l3, kara2)
    return F12(t0 + t1.mul_v(), m - t0 - t1)


def line_mul_line(la, lb):
    """(a0 + a1 w + a3 w^3)(b0 + b1 w + b3 w^3), w^6 = xi:
    w^0: a0b0; w^1: a0b1 + a1b0; w^2: a1b1; w^3: a0b3 + a3b0; w^4: a1b3 + a3b1; w^6 -> xi: a3b3"""
    a0, a1, a3 = la
    b0, b1, b3 = lb
    p = a0.c0.p
    z = zero2(p)
    t00, t11, t33 = a0.mul(b0), a1.mul(b1), a3.mul(b3)
    c = {0: t00 + t33.mul_xi(), 1: a0.mul(b1) + a1.mul(b0), 2: t11, 3: a0.mul(b3) + a3.mul(b0),
         4: a1.mul(b3) + a3.mul(b1), 5: z}
    # w^k, k = 2q + h  ->  (h, q)
    h0 = F6(c[0], c[2], c[4])
    h1 = F6(c[1], c[3], c[5])
    return F12(h0, h1)


def twist_frob(Q):
    xQ, yQ = Q
    return (xQ.conj().mul_const(FROB_TX), yQ.conj().mul_const(FROB_TY))


def twist_frob2_neg(Q):
    xQ, yQ = Q
    p = xQ.c0.p
    gx, gy = p.fconst(FROB2_TX[0]), p.fconst(-FROB2_TY[0])
    return (F2(xQ.c0 * gx, xQ.c1 * gx), F2(yQ.c0 * gy, yQ.c1 * gy))


def naf(k):
    d = []
    while k:
        if k & 1:
            z = 2 - (k % 4)
            k -= z
        else:
            z = 0
        d.append(z)
        k //= 2
    return d[::-1]


ATE = 6 * U + 2
ATE_NAF = naf(ATE)          # most significant first, leading digit 1


# ============================================================================ programs
def f2_in(p, name):
    return F2(p.inp(name + ".0"), p.inp(name + ".1"))


def f12_in(p, name):
    return F12.of([p.inp("%s.%d" % (name, k)) for k in range(12)])


def f2_out(p, name, v):
    p.out(name + ".0", v.c0)
    p.out(name + ".1", v.c1)


def f12_out(p, name, f):
    for k, c in enumerate(f.coeffs()):
        p.out("%s.%d" % (name, k), c)


def line_in(p, name):
    return tuple(f2_in(p, "%s.%d" % (name, k)) for k in range(3))


def line_out(p, name, l):
    for k, c in enumerate(l):
        f2_out(p, "%s.%d" % (name, k), c)


def pt_in(p, name):
    return tuple(f2_in(p, "%s.%s" % (name, c)) for c in "XYZ")


def pt_out(p, name, T):
    for c, v in zip("XYZ", T):
        f2_out(p, "%s.%s" % (name, c), v)


def miller_programs():
    """The Miller loop over the NAF digits of 6u + 2 and the closing additions of pi(Q) and
    -pi^2(Q) as one program: the scheduler then overlaps the chain of the twist point with the
    chain of the accumulator across the whole loop."""
    p = Prog("ml")
    xP, yP = p.inp("xP"), p.inp("yP")
    Q = (f2_in(p, "xQ"), f2_in(p, "yQ"))
    nQ = (Q[0], -Q[1])
    T = (Q[0], Q[1], F2(p.fconst(1), p.fconst(0)), F2(p.fconst(B3[0]), p.fconst(B3[1])))
    f = None
    for d in ATE_NAF[1:]:
        if f is not None:
            f = f.sqr()
        T, l1 = line_dbl(T, xP, yP)
        if d:
            T, l2 = line_add(T, Q if d == 1 else nQ, xP, yP)
            m = line_mul_line(l1, l2)
            f = m if f is None else f.mul(m)
        else:
            f = line_to_f12(l1) if f is None else mul_by_line(f, l1)
    T, la = line_add(T, twist_frob(Q), xP, yP)
    _, lb = line_add(T, twist_frob2_neg(Q), xP, yP)
    f12_out(p, "f", f.mul(line_mul_line(la, lb)))
    return {p.name: p}


MILLER_STATE = ["xP", "yP", "xQ.0", "xQ.1", "yQ.0", "yQ.1"] + ["f.%d" % k for k in range(12)]


def cyclo_sqr(X, L=None):
    """Granger-Scott squaring of a cyclotomic element over the three F_p4 pairs
    (w^0, w^3), (w^1, w^4), (w^2, w^5), with s = w^3, s^2 = xi.  L: the same element, from
    which the terms outside the products are taken (X by default)."""
    L = L or X
    def by_w(X):
        a, b = X.a, X.b
        return {0: a.c[0], 2: a.c[1], 4: a.c[2], 1: b.c[0], 3: b.c[1], 5: b.c[2]}   # by power of w
    g, z = by_w(X), by_w(L)

    def fp4_sqr(x, y):  # (x + y s)^2 with s^2 = xi: (x^2 + xi y^2, 2xy)
        t0, t1 = x.sqr(), y.sqr()
        return t0 + t1.mul_xi(), (x + y).sqr() - t0 - t1

    t0, t1 = fp4_sqr(g[0], g[3])
    n0 = t0.scale(3) - z[0].scale(2)
    n1 = t1.scale(3) + z[3].scale(2)
    t0, t1 = fp4_sqr(g[1], g[4])
    t2, t3 = fp4_sqr(g[2], g[5])
    n4 = t0.scale(3) - z[2].scale(2)
    n5 = t1.scale(3) + z[5].scale(2)
    t0 = t3.mul_xi()
    n2 = t0.scale(3) + z[1].scale(2)
    n3 = t2.scale(3) - z[4].scale(2)
    h = {0: n0, 3: n1, 1: n2, 4: n3, 2: n4, 5: n5}
    return F12(F6(h[0], h[2], h[4]), F6(h[1], h[3], h[5]))


def materialised(X):
    """X with every coefficient a value of its own; X's own expressions stay as they are"""
    return F12.of([F(c.p, {F(c.p, dict(c.t)).atom(): 1}) if c.t else c for c in X.coeffs()])


def f12_programs():
    progs = {}

    def mk(name, fn, n_in):
        p = Prog(name)
        X = f12_in(p, "X")
        args = [X] + ([f12_in(p, "Y")] if n_in == 2 else [])
        f12_out(p, "D", fn(*args))
        progs[name] = p

    mk("f12_mul", lambda X, Y: X.mul(Y), 2)
    mk("f12_sqr", lambda X: X.sqr(), 1)
    mk("f12_sqr_mul", lambda X, Y: X.sqr().mul(Y), 2)
    mk("f12_csqr", cyclo_sqr, 1)
    mk("f12_csqr_mul", lambda X, Y: cyclo_sqr(X).mul(Y), 2)
    mk("f12_frob1", lambda X: frob12(X, 1), 1)
    mk("f12_frob2", lambda X: frob12(X, 2), 1)
    mk("f12_frob3", lambda X: frob12(X, 3), 1)
    mk("f12_conj", lambda X: X.conj(), 1)
    return progs


# the exponents of the final exponentiation's hard part: (p^4 - p^2 + 1)/r = l0 + l1 p + l2 p^2 + p^3
# with l2 = 6u^2 + 1, l1 = -36u^3 - 18u^2 - 12u + 1, l0 = l1 - (2 l2 + 6u + 1)
HARD_L1N, HARD_L2, HARD_L3 = 36 * U**3 + 18 * U**2 + 12 * U - 1, 6 * U**2 + 1, 6 * U + 1
assert (P**4 - P**2 + 1) // R == -HARD_L1N - 2 * HARD_L2 - HARD_L3 - HARD_L1N * P + HARD_L2 * P**2 + P**3


def final_exp_programs():
    """The final exponentiation f^((p^12 - 1)/r) in two programs around one inversion in F_p
    (input X, result D, both absolute slots).

    fe_norm: n6 = X conj(X) = a^2 - v b^2 in F_p6; the F_p6 inverse of n6 is (A, B, C) / n2 with
    A = c0^2 - xi c1 c2, B = xi c2^2 - c0 c1, C = c1^2 - c0 c2, n2 = c0 A + xi (c2 B + c1 C);
    t = n2 conj(n2) in F_p.

    fe_rest, from tinv = t^{-1}: the easy part f = (conj(X) X^{-1})^{p^2 + 1}, with n6^{-1} =
    (A, B, C) conj(n2) tinv and conj(X) X^{-1} = conj(X)^2 n6^{-1}; then the hard part from the
    lowest digit up: one chain of squarings f^{2^i}, and f^{-l1}, f^{l2}, f^{6u + 1} gathered
    beside it over the signed digits of their exponents (a negative digit takes the conjugate,
    the inverse in the cyclotomic subgroup).  The chain is 193 squarings, a product level each:
    a squaring's factors are sums of the products before it, and its coefficients are also
    made values in the level beside, for the linear terms of the next and for the products."""
    progs = {}
    p = Prog("fe_norm")
    X = f12_in(p, "X")
    n6 = X.a.mul(X.a) - X.b.mul(X.b).mul_v()
    c0, c1, c2 = n6.c
    A = c0.sqr() - c1.mul(c2).mul_xi()
    B = c2.sqr().mul_xi() - c0.mul(c1)
    C = c1.sqr() - c0.mul(c2)
    n2 = c0.mul(A) + (c2.mul(B) + c1.mul(C)).mul_xi()
    for nm, v in (("nA", A), ("nB", B), ("nC", C), ("n2", n2)):
        f2_out(p, nm, v)
    p.out("t", n2.c0 * n2.c0 + n2.c1 * n2.c1)
    progs[p.name] = p

    p = Prog("fe_rest")
    X = f12_in(p, "X")
    A, B, C, n2 = (f2_in(p, nm) for nm in ("nA", "nB", "nC", "n2"))
    n2i = n2.conj().mul_fp(p.inp("tinv"))
    n6i = F6(A.mul(n2i), B.mul(n2i), C.mul(n2i))
    cx2 = X.conj().sqr()
    e = F12(cx2.a.mul(n6i), cx2.b.mul(n6i))
    f = materialised(frob12(e, 2).mul(e))
    digits = [naf(x)[::-1] for x in (HARD_L1N, HARD_L2, HARD_L3)]
    n = max(len(d) for d in digits)
    s, z, acc = f, f, [None, None, None]
    for i in range(n):
        for k in range(3):
            d = digits[k][i] if i < len(digits[k]) else 0
            if d:
                v = z if d > 0 else z.conj()
                acc[k] = v if acc[k] is None else materialised(acc[k].mul(v))
        if i + 1 < n:
            s = cyclo_sqr(s, z)
            z = materialised(s)
    a1, a2, a3 = acc                                  # f^{-l1}, f^{l2}, f^{6u + 1}
    t0 = a1.mul(cyclo_sqr(a2).mul(a3))                # f^{-l0}
    r1 = t0.conj().mul(frob12(a1.conj(), 1))
    r2 = frob12(a2, 2).mul(frob12(f, 3))
    f12_out(p, "D", r1.mul(r2))
    progs[p.name] = p
    return progs


FE_STATE = (["X.%d" % k for k in range(12)] + ["D.%d" % k for k in range(12)] + ["t", "tinv"]
            + ["%s.%d" % (nm, k) for nm in ("nA", "nB", "nC", "n2") for k in (0, 1)])

# ============================================================================ G2 scalar multiplication (GLS)
# psi(x, y) = (conj(x) tx, conj(y) ty) acts on G2 as multiplication by lam = p mod r = 6u^2.
# A scalar k is split as k = sum_j k_j lam^j (mod r), |k_j| < 2^65, with the reduced lattice
# basis below (rows b satisfy b0 + b1 lam + b2 lam^2 + b3 lam^3 = 0 mod r) and Babai rounding
# with the constants G (c_i = floor(k G_i / 2^256), k_j = [j = 0] k - sum_i c_i b_ij).
GLS_B = [[2 * U + 1, 0, 2 * U, 1], [2 * U, U + 1, -U, U], [U + 1, U, U, -2 * U], [2 * U + 1, -U, -(U + 1), -U]]


def gls_constants():
    from fractions import Fraction
    n = 4
    M = [[Fraction(x) for x in row] + [Fraction(int(i == j)) for j in range(n)] for i, row in enumerate(GLS_B)]
    for c in range(n):
        piv = next(r for r in range(c, n) if M[r][c] != 0)
        M[c], M[piv] = M[piv], M[c]
        pv = M[c][c]
        M[c] = [x / pv for x in M[c]]
        for r in range(n):
            if r != c and M[r][c] != 0:
                f = M[r][c]
                M[r] = [a - f * b for a, b in zip(M[r], M[c])]
    alpha = M[0][n:]
    G = [round(a * 2**256) for a in alpha]
    assert all(0 <= g < 2**192 for g in G)
    return G


def gls_decompose(k):
    G = gls_constants()
    c = [(k * g) >> 256 for g in G]
    return [(k if j == 0 else 0) - sum(c[i] * GLS_B[i][j] for i in range(4)) for j in range(4)]


def j_dbl(T):
    X, Y, Z = T
    A, B = X.sqr(), Y.sqr()
    C = B.sqr()
    D = ((X + B).sqr() - A - C).scale(2)
    E = A.scale(3)
    X3 = E.sqr() - D.scale(2)
    Y3 = E.mul(D - X3) - C.scale(8)
    Z3 = Y.mul(Z).scale(2)
    return (X3, Y3, Z3)


def j_add(T1, T2):
    """add-2007-bl; returns the sum and (H, r): H = 0 means equal x, then r = 0 means equal points"""
    X1, Y1, Z1 = T1
    X2, Y2, Z2 = T2
    Z1Z1, Z2Z2 = Z1.sqr(), Z2.sqr()
    U1, U2 = X1.mul(Z2Z2), X2.mul(Z1Z1)
    S1, S2 = Y1.mul(Z2).mul(Z2Z2), Y2.mul(Z1).mul(Z1Z1)
    H = U2 - U1
    I = H.scale(2).sqr()
    J = H.mul(I)
    rr = (S2 - S1).scale(2)
    V = U1.mul(I)
    X3 = rr.sqr() - J - V.scale(2)
    Y3 = rr.mul(V - X3) - S1.mul(J).scale(2)
    Z3 = ((Z1 + Z2).sqr() - Z1Z1 - Z2Z2).mul(H)
    return (X3, Y3, Z3), H, S2 - S1


def jac_in(p, name):
    return tuple(F2(p.inp("%s.%d" % (name, 2 * c)), p.inp("%s.%d" % (name, 2 * c + 1))) for c in range(3))


def jac_out(p, name, T):
    for c, v in enumerate(T):
        p.out("%s.%d" % (name, 2 * c), v.c0)
        p.out("%s.%d" % (name, 2 * c + 1), v.c1)


# Scalar multiplications run on homogeneous coordinates with the complete formulas for
# y^2 = x^3 + b (J. Renes, C. Costello, L. Batina, "Complete addition formulas for prime order
# elliptic curves", 2016, algorithms 7 and 9): two product levels for an addition and two for
# a doubling (Jacobian formulas take five and three), and no exceptional cases in the groups of
# odd order r.  b3 multiplies by 3b.
def rcb_add(P1, P2, b3):
    X1, Y1, Z1 = P1
    X2, Y2, Z2 = P2
    t0, t1, t2 = X1.mul(X2), Y1.mul(Y2), Z1.mul(Z2)
    t3 = X1.mul(Y2) + X2.mul(Y1)
    t4 = Y1.mul(Z2) + Y2.mul(Z1)
    y3 = b3(X1.mul(Z2) + X2.mul(Z1))
    t0 = t0.scale(3)
    t2 = b3(t2)
    z3, t1 = t1 + t2, t1 - t2
    return (t3.mul(t1) - t4.mul(y3), y3.mul(t0) + t1.mul(z3), z3.mul(t4) + t0.mul(t3))


def rcb_dbl(P1, b3):
    X, Y, Z = P1
    t0, t1, t2, t3 = Y.sqr(), Y.mul(Z), Z.sqr(), X.mul(Y)
    t2 = b3(t2)
    n = t0 - t2.scale(3)
    return (n.mul(t3).scale(2), t2.mul(t0).scale(8) + n.mul(t0 + t2), t0.mul(t1).scale(8))


# A point between two programs is kept as sums: each coordinate a fixed number of slots whose
# sum it is, so that a program ends in its last products and not in a level of additions.
def sums_in(p, name, n):
    f = p.inp("%s.0" % name)
    for i in range(1, n):
        f = f + p.inp("%s.%d" % (name, i))
    return f


def sums_out(p, name, f, n):
    """f as n slots: its products with their coefficients taken into a factor; more terms than
    slots are added up in the last one"""
    t = sorted(f.t.items())
    vs = []
    for k, (v, c) in enumerate(t):
        if k == n - 1 and len(t) > n:
            vs.append(F(p, dict(t[k:])).atom())
            break
        if c == 1:
            vs.append(v)
            continue
        node = p.vals[v]
        if node[0] == "mul":
            for x, y in ((1, 2), (2, 1)):  # the factor with the smaller coefficients takes c
                if all(abs(c * k_) <= KMAX for _, k_ in node[x]):
                    break
            else:
                x = None
            if x:
                g = tuple((i, c * k_) for i, k_ in node[x])
                A, B = (g, node[y]) if g <= node[y] else (node[y], g)
                vs.append(p.new(("mul", A, B)))
                continue
        vs.append(F(p, {v: c}).atom())
    vs += [p.zero] * (n - len(vs))
    for i, v in enumerate(vs):
        p.outputs["%s.%d" % (name, i)] = v


# G2 works on y^2 = x^3 + b'' with b'' = 4 + 5i, isomorphic to the twist by (x, y) ->
# (u^2 x, u^3 y), u^6 = b''/b', so that the formulas' 3b'' is a pair of small integers.
def sixth_root(r):
    """some u in F_p2 with u^6 = r"""
    n = P * P - 1
    m = n
    while m % 2 == 0:
        m //= 2
    while m % 3 == 0:
        m //= 3
    x0 = f2pow_int(r, pow(6, -1, m))
    k = 2
    while True:
        g = f2pow_int((k, 1), m)
        if f2pow_int(g, n // m // 2) != (1, 0) and f2pow_int(g, n // m // 3) != (1, 0):
            break
        k += 1
    x = x0
    for _ in range(n // m):
        if f2pow_int(x, 6) == r:
            return x
        x = f2mul_int(x, g)
    raise ValueError("no sixth root")


G2_BPP = (4, 5)
G2_U = sixth_root(f2mul_int(G2_BPP, f2inv_int(f2mul_int(B3, (pow(3, -1, P), 0)))))
G2_U2 = f2mul_int(G2_U, G2_U)
G2_U3 = f2mul_int(G2_U2, G2_U)
G2_UI = f2inv_int(G2_U)


def f2conj_int(a):
    return (a[0], -a[1] % P)


# psi on the isomorphic curve: (conj(x) tx, conj(y) ty) with the constants carried over
G2_TX = f2mul_int(FROB_TX, f2mul_int(G2_U2, f2inv_int(f2conj_int(G2_U2))))
G2_TY = f2mul_int(FROB_TY, f2mul_int(G2_U3, f2inv_int(f2conj_int(G2_U3))))


def b3_g2(a):  # (12 + 15 i) a
    c0, c1 = 3 * G2_BPP[0], 3 * G2_BPP[1]
    return F2(a.c0.scale(c0) - a.c1.scale(c1), a.c1.scale(c0) + a.c0.scale(c1))


def b3_g1(a):  # b = 3
    return a.scale(9)


G2_SUM, G1_SUM = 4, 2  # slots of a coordinate's component between two programs


def pt2_in(p, name, n=G2_SUM):
    return tuple(F2(sums_in(p, "%s.%d.0" % (name, c), n), sums_in(p, "%s.%d.1" % (name, c), n)) for c in range(3))


def pt2_out(p, name, T):
    for c, v in enumerate(T):
        sums_out(p, "%s.%d.0" % (name, c), v.c0, G2_SUM)
        sums_out(p, "%s.%d.1" % (name, c), v.c1, G2_SUM)


def g2_programs():
    progs = {}

    def done(p):
        progs[p.name] = p

    # Q and its psi images on the isomorphic curve, each from Q by one constant a coordinate:
    # psi^j(x) = conj^j(x) kx
    p = Prog("g2_bases")
    x, y = f2_in(p, "xQ"), f2_in(p, "yQ")
    kx, ky = G2_U2, G2_U3
    for j in range(4):
        if j:
            x, y = x.conj(), y.conj()
            kx, ky = f2mul_int(f2conj_int(kx), G2_TX), f2mul_int(f2conj_int(ky), G2_TY)
        f2_out(p, "B%d.x" % j, x.mul_const(kx))
        f2_out(p, "B%d.y" % j, y.mul_const(ky))
    done(p)
    # table TB[d] = sum_{j in d} B_j, the caller's signs on the y
    p = Prog("g2_table")
    one = F2(p.fconst(1), p.fconst(0))
    TB = {}
    for j in range(4):
        TB[1 << j] = (f2_in(p, "B%d.x" % j), f2_in(p, "B%d.y" % j), one)
    for d in range(1, 16):
        lo = d & -d if bin(d).count("1") < 4 else 3
        if d != lo:
            TB[d] = rcb_add(TB[d - lo], TB[lo], b3_g2)
    for d in range(1, 16):
        jac_out(p, "TB%d" % d, TB[d])
    done(p)
    p = Prog("g2_dbl")
    pt2_out(p, "T", rcb_dbl(pt2_in(p, "T"), b3_g2))
    done(p)
    p = Prog("g2_dbl_add")
    pt2_out(p, "T", rcb_add(rcb_dbl(pt2_in(p, "T"), b3_g2), jac_in(p, "A"), b3_g2))
    done(p)
    p = Prog("g2_add")
    pt2_out(p, "T", rcb_add(pt2_in(p, "T"), jac_in(p, "A"), b3_g2))
    done(p)
    # T += (xQ, yQ) of the twist
    p = Prog("g2_madd")
    pt2_out(p, "T", rcb_add(pt2_in(p, "T"), (f2_in(p, "xQ").mul_const(G2_U2), f2_in(p, "yQ").mul_const(G2_U3),
                                             F2(p.fconst(1), p.fconst(0))), b3_g2))
    done(p)
    # T = (xQ, yQ) of the twist
    p = Prog("g2_load")
    pt2_out(p, "T", (f2_in(p, "xQ").mul_const(G2_U2), f2_in(p, "yQ").mul_const(G2_U3), F2(p.fconst(1), p.fconst(0))))
    done(p)
    # to affine coordinates of the twist: t = N(Z); then x = X conj(Z) t^{-1} u^{-2}, y likewise
    p = Prog("g2_norm")
    Z = pt2_in(p, "T")[2]
    p.out("t", Z.c0 * Z.c0 + Z.c1 * Z.c1)
    done(p)
    p = Prog("g2_aff")
    X, Y, Z = pt2_in(p, "T")
    ti = p.inp("tinv")
    Zi = Z.conj().mul_fp(ti)
    f2_out(p, "ax", X.mul_const(f2mul_int(G2_UI, G2_UI)).mul(Zi))
    f2_out(p, "ay", Y.mul_const(f2mul_int(f2mul_int(G2_UI, G2_UI), G2_UI)).mul(Zi))
    done(p)
    # Jacobian coordinates on the twist (the sums of the MSMs): doubling and addition, which
    # reports equal x-coordinates (H = 0), then equal points (RR = 0)
    p = Prog("g2_jdbl")
    jac_out(p, "J", j_dbl(jac_in(p, "J")))
    done(p)
    p = Prog("g2_jadd")
    T, H, r = j_add(jac_in(p, "J"), jac_in(p, "A"))
    jac_out(p, "J", T)
    f2_out(p, "H", H)
    f2_out(p, "RR", r)
    done(p)
    return progs


# G1 (y^2 = x^3 + 3 over F_p) on the engine: GLV with phi(x, y) = (beta x, y)
GLV_BETA = 0x59E26BCEA0D48BACD4F263F1ACDB5C4F5763473177FFFFFE
GLV_LAM = 0xB3C4D79D41A917585BFC41088D8DAAA78B17EA66B99C90DD


def g1_in(p, name):
    return tuple(p.inp("%s.%d" % (name, c)) for c in range(3))


def pt1_in(p, name):
    return tuple(sums_in(p, "%s.%d" % (name, c), G1_SUM) for c in range(3))


def pt1_out(p, name, T):
    for c, v in enumerate(T):
        sums_out(p, "%s.%d" % (name, c), v, G1_SUM)


def g1_programs():
    progs = {}

    def done(p):
        progs[p.name] = p

    p = Prog("g1_phi")
    p.out("B1.x", p.inp("xP") * p.fconst(GLV_BETA))
    done(p)
    # table TB[d0 + 4 d1] = d0 B0 + d1 B1 for the joint 2-bit windows; B0 in (xP, yP), B1 in
    # (B1.x, B1.y), signs applied by the caller
    p = Prog("g1_table")
    one = p.fconst(1)
    TB = {1: (p.inp("xP"), p.inp("yP"), one), 4: (p.inp("B1.x"), p.inp("B1.y"), one)}
    for d in (1, 4):
        TB[2 * d] = rcb_dbl(TB[d], b3_g1)
        TB[3 * d] = rcb_add(TB[2 * d], TB[d], b3_g1)
    for d1 in (1, 2, 3):
        for d0 in (1, 2, 3):
            TB[d0 + 4 * d1] = rcb_add(TB[4 * d1], TB[d0], b3_g1)
    for d in range(1, 16):
        for c, v in enumerate(TB[d]):
            p.out("TB%d.%d" % (d, c), v)
    done(p)
    p = Prog("g1_dbl2")
    pt1_out(p, "T", rcb_dbl(rcb_dbl(pt1_in(p, "T"), b3_g1), b3_g1))
    done(p)
    p = Prog("g1_dbl2_add")
    pt1_out(p, "T", rcb_add(rcb_dbl(rcb_dbl(pt1_in(p, "T"), b3_g1), b3_g1), g1_in(p, "A"), b3_g1))
    done(p)
    p = Prog("g1_add")
    pt1_out(p, "T", rcb_add(pt1_in(p, "T"), g1_in(p, "A"), b3_g1))
    done(p)
    # T += (xP, yP)
    p = Prog("g1_madd")
    pt1_out(p, "T", rcb_add(pt1_in(p, "T"), (p.inp("xP"), p.inp("yP"), p.fconst(1)), b3_g1))
    done(p)
    p = Prog("g1_aff")
    X, Y, Z = pt1_in(p, "T")
    zi = p.inp("tinv")
    p.out("ax", X * zi)
    p.out("ay", Y * zi)
    done(p)
    return progs


G1_STATE = (["T.%d.%d" % (c, k) for c in range(3) for k in range(G1_SUM)] + ["xP", "yP", "B1.x", "B1.y", "tinv"]
            + ["TB%d.%d" % (d, k) for d in range(1, 16) for k in range(3)] + ["ax", "ay"])


G2_STATE = (["T.%d.%d.%d" % (c, h, k) for c in range(3) for h in (0, 1) for k in range(G2_SUM)]
            + ["xQ.0", "xQ.1", "yQ.0", "yQ.1", "t", "tinv"]
            + ["B%d.%s.%d" % (j, c, k) for j in range(4) for c in "xy" for k in (0, 1)]
            + ["TB%d.%d" % (d, k) for d in range(1, 16) for k in range(6)]
            + ["J.%d" % k for k in range(6)] + ["H.0", "H.1", "RR.0", "RR.1", "ax.0", "ax.1", "ay.0", "ay.1"])


# ============================================================================ scheduling
def operands(v):
    if v[0] == "mul":
        return tuple(k for k, _ in v[1]) + tuple(k for k, _ in v[2])
    if v[0] == "lin":
        return tuple(k for k, _ in v[1])
    return ()


# Cost of a level in ns of the interpreter (measured on gfx950): a fixed part, a part per
# term of the longest lane record, the Montgomery product of a level with products.
LEVEL_BASE, LEVEL_TERM, LEVEL_MUL = 430, 25, 520


def lane_terms(v):
    """terms of an operation's longer lane record (before padding)"""
    if v[0] == "mul":
        return max(len(v[1]), len(v[2]))
    return -(-len(v[1]) // 2)


def pad_terms(n):
    return next(t for t in LANE_TERMS if n <= t)


def levels_cost(p, levels):
    c = 0
    for ops in levels:
        t = max(pad_terms(lane_terms(p.vals[i])) for i in ops)
        mul = any(p.vals[i][0] == "mul" for i in ops)
        c += LEVEL_BASE + LEVEL_TERM * t + (LEVEL_MUL if mul else 0)
    return c


def schedule(p, lanes):
    """The cheapest of the stage schedules below (as early / as late as possible) and the
    list schedules."""
    if len(p.vals) > 4000:  # a whole Miller loop or exponentiation
        cand = [schedule_list(p, lanes, bias, window) for bias in (0, 200) for window in (3000, 8000)]
    else:
        cand = [schedule_phases(p, lanes, late=False), schedule_phases(p, lanes, late=True)]
        cand += [schedule_list(p, lanes, bias) for bias in (0, 100, 200, 300, -150)]
    return min(cand, key=lambda c: levels_cost(p, c[0]))


def schedule_list(p, lanes, bias=0, window=1 << 30):
    """List scheduling by the longest remaining path (products and additions weighted by the
    cost of their levels).  A level either runs the ready operations, or additions alone: the
    latter when the additions lead the critical path and the products can wait for a shorter
    level (bias shifts that choice).  Operations whose remaining path is shorter than the
    longest one by more than `window` wait: a chain that could run far ahead would hold slots."""
    vals = p.vals
    n = len(vals)
    live = [False] * n
    stack = list(p.outputs.values())
    while stack:
        i = stack.pop()
        if live[i]:
            continue
        live[i] = True
        stack.extend(operands(vals[i]))
    is_op = [live[i] and vals[i][0] in ("mul", "lin") for i in range(n)]
    wl = LEVEL_BASE + 4 * LEVEL_TERM
    wm = wl + LEVEL_MUL
    h = [0] * n
    users = [[] for _ in range(n)]
    need = [0] * n
    for i in range(n):
        if is_op[i]:
            for a in set(operands(vals[i])):
                if is_op[a]:
                    users[a].append(i)
                    need[i] += 1
    for i in reversed(range(n)):
        if is_op[i]:
            h[i] = (wm if vals[i][0] == "mul" else wl) + max([h[u] for u in users[i]] + [0])
    ready = [i for i in range(n) if is_op[i] and need[i] == 0]
    levels = []
    level_of = [-1] * n
    while ready:
        top = max(h[i] for i in ready)
        cand = sorted((i for i in ready if h[i] >= top - window), key=lambda i: (-h[i], i))
        muls = [i for i in cand if vals[i][0] == "mul"]
        lins = [i for i in cand if vals[i][0] == "lin"]
        hm = h[muls[0]] if muls else -1
        hl = h[lins[0]] if lins else -1
        if muls and (not lins or max(hm, hl - wl + wm) < max(hl, hm + wl) + bias):
            pick = cand[:lanes]
        else:
            pick = lins[:lanes] or muls[:lanes]
        L = len(levels)
        levels.append(sorted(pick))
        for i in pick:
            level_of[i] = L
        ready = [i for i in ready if level_of[i] < 0]
        for i in pick:
            for u in users[i]:
                need[u] -= 1
                if need[u] == 0:
                    ready.append(u)
    return levels, level_of, live


def schedule_phases(p, lanes, late=False):
    """Stage scheduling: a product's stage is its multiplicative depth (products on the
    longest path from the inputs), so all products of one depth share one level (split
    only beyond the lane count).  Additions run in a phase between two product levels,
    levelised by their depth within the phase: the phase right after the products they
    depend on, or (late) the last phase before their first use, so that additions that
    only feed outputs or later products share levels that exist anyway."""
    vals = p.vals
    n = len(vals)
    live = [False] * n
    stack = list(p.outputs.values())
    while stack:
        i = stack.pop()
        if live[i]:
            continue
        live[i] = True
        stack.extend(operands(vals[i]))
    is_op = [live[i] and vals[i][0] in ("mul", "lin") for i in range(n)]
    md = [0] * n      # multiplicative depth
    ld = [0] * n      # depth in additions since the last product
    for i in range(n):
        if not is_op[i]:
            continue
        ops_ = [a for a in operands(vals[i]) if is_op[a]]
        if vals[i][0] == "mul":
            md[i] = 1 + max([md[a] for a in ops_] + [0])
            ld[i] = 0
        else:
            m = max([md[a] for a in ops_] + [0])
            md[i] = m
            ld[i] = 1 + max([ld[a] for a in ops_ if md[a] == m] + [0])
    # a product at depth k must follow the additions of phase k-1 that feed it
    maxd = max([md[i] for i in range(n) if is_op[i]] + [0])
    phase = list(md)
    if late:
        users = [[] for _ in range(n)]
        for i in range(n):
            if is_op[i]:
                for a in set(operands(vals[i])):
                    users[a].append(i)
        outset = set(p.outputs.values())
        for i in reversed(range(n)):
            if not (is_op[i] and vals[i][0] == "lin"):
                continue
            lim = maxd if i in outset else 1 << 30
            for c in users[i]:
                lim = min(lim, md[c] - 1 if vals[c][0] == "mul" else phase[c])
            assert md[i] <= lim < 1 << 30
            phase[i] = lim
        for i in range(n):
            if is_op[i] and vals[i][0] == "lin":
                ld[i] = 1 + max([ld[a] for a in operands(vals[i])
                                 if is_op[a] and vals[a][0] == "lin" and phase[a] == phase[i]] + [0])
    buckets = {}
    for i in range(n):
        if not is_op[i]:
            continue
        if vals[i][0] == "mul":
            key = (md[i] - 1, 1 << 20)          # after phase md-1 additions
        else:
            key = (phase[i], ld[i])
        buckets.setdefault(key, []).append(i)
    levels = []
    level_of = [-1] * n
    for key in sorted(buckets):
        ops_ = sorted(buckets[key])
        for k in range(0, len(ops_), lanes):
            L = len(levels)
            levels.append(ops_[k:k + lanes])
            for i in ops_[k:k + lanes]:
                level_of[i] = L
    return levels, level_of, live


def compile_prog(p, io_slot, const_slot, temp_base, temp_limit, lanes):
    """Schedule p and assign slots.  io_slot(name) gives the encoded slot of an input or
    output name (an output with the name of an input replaces it), const_slot(x) the slot
    of a constant.  Returns (levels of encoded op tuples, highest temp slot used + 1).
    The wavefronts of a level run apart: an operation never writes a slot that an operation
    of the same level reads."""
    levels, level_of, live = schedule(p, lanes)
    vals = p.vals
    n = len(vals)
    nlev = len(levels)
    slot = [None] * n
    for name, v in p.inputs.items():
        slot[v] = io_slot(name)
    for x, v in p.consts.items():
        slot[v] = const_slot(x)
    last = [-1] * n
    for i in range(n):
        if level_of[i] >= 0:
            for a in operands(vals[i]):
                last[a] = max(last[a], level_of[i])
    outs = {}
    for name, v in p.outputs.items():
        outs.setdefault(v, []).append(name)
    for v in outs:
        last[v] = nlev
    # last read of the value held in each io slot at entry
    held_read = {}
    for name, v in p.inputs.items():
        held_read[io_slot(name)] = last[v]
    free = list(range(temp_limit - 1, temp_base - 1, -1))
    busy = []
    used = temp_base
    copies = []
    for i in sorted((i for i in range(n) if level_of[i] >= 0), key=lambda i: (level_of[i], i)):
        L = level_of[i]
        keep = []
        for rl, s in busy:
            (free if rl < L else keep).append(s if rl < L else (rl, s))
        busy = keep
        names = outs.get(i, [])
        # write in place when this is the only output of the value and the slot's entry
        # value is not read after this level
        if len(names) == 1 and held_read.get(io_slot(names[0]), -1) < L:
            slot[i] = io_slot(names[0])
            continue
        if not free:
            raise RuntimeError("%s: out of temp slots" % p.name)
        s = free.pop()
        used = max(used, s + 1)
        slot[i] = s
        busy.append((last[i], s))
        for nm in names:
            copies.append((nm, i))
    # outputs that are inputs or constants of the program, or that share a value
    for v, names in outs.items():
        if level_of[v] < 0:
            for nm in names:
                if slot[v] != io_slot(nm):
                    copies.append((nm, v))
    enc = []
    for ops in levels:
        row = []
        for i in ops:
            v = vals[i]
            if v[0] == "mul":
                row.append((OP_MUL, slot[i], len(v[1]), tuple((slot[k], c) for k, c in v[1] + v[2])))
            else:
                row.append((OP_LIN, slot[i], len(v[1]), tuple((slot[k], c) for k, c in v[1])))
        enc.append(row)
    # copies of inputs and constants share the last level, where its operations do not read
    # their destinations; the others follow in a level of their own
    early = [(nm, v) for nm, v in copies if level_of[v] < 0 and enc and held_read.get(io_slot(nm), -1) < nlev - 1]
    early = early[:max(0, lanes - len(enc[-1]))] if enc else []
    if early:
        enc[-1] = enc[-1] + [(OP_LIN, io_slot(nm), 1, ((slot[v], 1),)) for nm, v in early]
        copies = [c for c in copies if c not in early]
    if copies:
        row = [(OP_LIN, io_slot(nm), 1, ((slot[v], 1),)) for nm, v in copies]
        for k in range(0, len(row), lanes):
            enc.append(row[k:k + lanes])
    for row in enc:
        reads = set(s_ for op in row for s_, c in op[3] if c)
        writes = [op[1] for op in row]
        assert len(set(writes)) == len(writes) and not reads & set(writes), p.name
    return enc, used


# ============================================================================ kernels
class Kernel:
    """programs that share one LDS slot map: named state slots, constants, temps"""

    def __init__(self, name, progs, state, segs=None, waves=2):
        self.name = name
        self.waves = waves
        lanes = WAVE_OPS * waves
        self.state = {nm: i for i, nm in enumerate(state)}
        self.segs = segs or {}
        consts = sorted(set(x for p in progs.values() for x in p.consts) | {0, 1})
        self.cbase = len(state)
        self.cslot = {x: self.cbase + k for k, x in enumerate(consts)}
        self.consts = consts
        self.tbase = self.cbase + len(consts)
        self.progs = {}
        self.used = {}  # slots up to the highest one that a program uses
        self.ntemps = self.tbase
        for nm, p in progs.items():
            enc, used = compile_prog(p, self.io_slot, lambda x: self.cslot[x % P], self.tbase, 1 << SEG_SHIFT, lanes)
            self.progs[nm] = enc
            self.used[nm] = used
            self.ntemps = max(self.ntemps, used)
        self.nslots = self.ntemps

    def io_slot(self, name):
        head = name.split(".")[0]
        if head in self.segs:
            seg = self.segs[head]
            assert 1 <= seg <= 3  # the interpreter packs the bases of segments 1..3 only
            off = int(name.split(".")[1])
            return (seg << SEG_SHIFT) | off
        return self.state[name]


def encode_term(s, c):
    """32-bit term: offset of the slot in its segment in 16-byte units (bits 0..11; a slot is
    48 bytes), signed coefficient (bits 12..24), segment (bits 30..31)"""
    off = 3 * (s & ((1 << SEG_SHIFT) - 1))
    assert 0 <= s < 4 << SEG_SHIFT and off < 4096 and -4096 <= c < 4096
    return off | ((c & 0x1fff) << 12) | ((s >> SEG_SHIFT) << 30)


def lane_records(op):
    """the two lanes' records of an operation: kind, destination (encoded as a term, the kind
    in place of the coefficient) and the terms.  A product's first factor is scaled by 32,
    which turns the radix-2^261 Montgomery product into the R = 2^256 one; a sum's terms are
    dealt to both lanes."""
    kind, dst, na, terms = op
    if kind == OP_MUL:
        A, B = [(s, 32 * c) for s, c in terms[:na]], list(terms[na:])
    else:
        A, B = list(terms[0::2]), list(terms[1::2])
    # columns and quotients of the interpreter are bounded for coefficient magnitudes that add up
    # to less than 2^15
    assert sum(abs(c) for _, c in A) < 32768 and sum(abs(c) for _, c in B) < 32768
    head = encode_term(dst, kind)
    return [[head] + [encode_term(s, c) for s, c in t] for t in (A, B)]


def level_blocks(row, waves):
    """the operations of a level dealt to the wavefronts: products first (most terms first),
    then the sums, those in wavefronts of their own while there are any; returns a list of
    operations for each wavefront"""
    def nt(op):
        return max(op[2], len(op[3]) - op[2]) if op[0] == OP_MUL else -(-len(op[3]) // 2)
    muls = sorted((op for op in row if op[0] == OP_MUL), key=nt, reverse=True)
    lins = sorted((op for op in row if op[0] == OP_LIN), key=nt, reverse=True)
    wm, wl = -(-len(muls) // WAVE_OPS), -(-len(lins) // WAVE_OPS)
    out = [[] for _ in range(waves)]
    if muls and lins and wm + wl <= waves:
        for k, op in enumerate(muls):
            out[k // WAVE_OPS].append(op)
        for k, op in enumerate(lins):
            out[wm + k // WAVE_OPS].append(op)
    else:
        for k, op in enumerate(muls + lins):
            out[k // WAVE_OPS].append(op)
    return out


class OpTable:
    """The wavefronts' operations of all levels ("blocks").  A block is a record per lane: head,
    the descriptor of the wavefront's next level (0 at the program's end), the terms, padded to
    groups of four words.  Groups lie 64 lanes apart (1 KB), so that a fetch is one 16-byte load
    per group at fixed offsets; blocks of the same number of groups share a row of 64 lanes.
    A block without operations still has one record, for the next descriptor.

    A descriptor: bits 0..18 offset of the block in units of four words, 19 / 20 / 21 / 22 more than 2 / 4 / 6 / 10 terms, 23 any
    term or destination in segments 1..3, 24..29 operations, 30 any product, 31 any sum."""

    def __init__(self):
        self.words = [0] * 256       # row 0 is not used: no descriptor is 0
        self.rows = {}               # groups -> [first word of the open row, lanes taken]

    def add(self, ops, nxt):
        recs = [r for op in ops for r in lane_records(op)] or [[0]]
        T = pad_terms(max(len(r) - 1 for r in recs))
        G = (T + 2 + 3) // 4
        row = self.rows.get(G)
        if row is None or row[1] + len(recs) > 64:
            row = self.rows[G] = [len(self.words), 0]
            self.words += [0] * (256 * G)
        base = row[0] + 4 * row[1]
        row[1] += len(recs)
        for l, r in enumerate(recs):
            r = [r[0], nxt] + r[1:] + [0] * (4 * G - 1 - len(r))
            for g in range(G):
                self.words[base + 256 * g + 4 * l:base + 256 * g + 4 * l + 4] = r[4 * g:4 * g + 4]
        d = base // 4
        assert base % 4 == 0 and d < 1 << 19 and len(ops) <= WAVE_OPS
        d |= (T > 2) << 19 | (T > 4) << 20 | (T > 6) << 21 | (T > 10) << 22
        d |= any(s_ >> SEG_SHIFT for op in ops for s_ in [op[1]] + [t[0] for t in op[3]]) << 23
        d |= len(ops) << 24
        d |= any(op[0] == OP_MUL for op in ops) << 30 | any(op[0] == OP_LIN for op in ops) << 31
        return d

    def finish(self):
        self.words += [0] * (256 * 4)  # a fetch reads all 64 lanes of its rows
        return self.words


TRACE_LIMITS = tuple((nt, sd) for nt in (8, 12, 20, 28) for sd in (4, 6, 10, 14))


WHOLE_LIMITS = ((12, 6), (20, 6), (12, 10), (20, 10), (28, 10))


def cheapest(make, waves, limits=TRACE_LIMITS):
    """trace every program under each (NTERM, SIDE) limit and keep, per program, the trace
    whose schedule costs least"""
    global NTERM, SIDE
    best = {}
    saved = NTERM, SIDE
    for nt, sd in limits:
        NTERM, SIDE = nt, sd
        for nm, p in make().items():
            c = levels_cost(p, schedule(p, WAVE_OPS * waves)[0])
            if nm not in best or c < best[nm][0]:
                best[nm] = (c, p)
    NTERM, SIDE = saved
    return {nm: p for nm, (c, p) in best.items()}


# wavefronts of a workgroup, by kernel family
ML_WAVES, FE_WAVES, F12_WAVES, G2_WAVES, G1_WAVES = 2, 4, 2, 2, 2

_BUILT = []


def build_all():
    if not _BUILT:
        mk = Kernel("ml", cheapest(miller_programs, ML_WAVES, WHOLE_LIMITS), MILLER_STATE, waves=ML_WAVES)
        ek = Kernel("fe", cheapest(final_exp_programs, FE_WAVES, WHOLE_LIMITS), FE_STATE, waves=FE_WAVES)
        fk = Kernel("f12", cheapest(f12_programs, F12_WAVES), [], segs={"X": 1, "Y": 2, "D": 3}, waves=F12_WAVES)
        gk = Kernel("g2", cheapest(g2_programs, G2_WAVES), G2_STATE, segs={"A": 2}, waves=G2_WAVES)
        g1k = Kernel("g1", cheapest(g1_programs, G1_WAVES), G1_STATE, segs={"A": 2}, waves=G1_WAVES)
        _BUILT.append((mk, ek, fk, gk, g1k))
    return _BUILT[0]


# ============================================================================ emission
def limbs(x):
    return [(x >> (32 * i)) & 0xFFFFFFFF for i in range(8)]


M29 = (1 << 29) - 1


def limbs29(x):
    return [(x >> (29 * i)) & M29 for i in range(9)]


def emit_radix():
    """constants of the radix-2^29 lane arithmetic"""
    o = []
    o.append("static constexpr uint32_t P29[9] = {%s};" % ", ".join("0x%08xu" % v for v in limbs29(P)))
    o.append("static constexpr uint32_t PINV29 = 0x%08xu;  // -p^{-1} mod 2^29" % ((-pow(P, -1, 1 << 29)) % (1 << 29)))
    assert P >> 232 < (1 << 29)
    o.append("static constexpr float INVP240 = %.9gf;  // 2^240 / p" % (float(2**240) / P))
    return o


def emit(kernels):
    o = []
    w = o.append
    w("// Generated by gen_slp.py -- straight-line programs for the wave-cooperative engine.")
    w("#pragma once")
    w("#include <cstdint>")
    w("namespace slp {")
    for line in emit_radix():
        w(line)
    table = OpTable()
    descs = []
    for k in kernels:
        w("// kernel %s: %d slots (%d state, %d constants)" % (k.name, k.nslots, len(k.state), len(k.consts)))
        assert k.nslots <= 1 << SEG_SHIFT  # absolute slots are offsets in segment 0
        w("static constexpr int %s_NSLOT = %d;" % (k.name.upper(), k.nslots))
        w("static constexpr int %s_CBASE = %d;" % (k.name.upper(), k.cbase))
        w("static constexpr int %s_NCONST = %d;" % (k.name.upper(), len(k.consts)))
        w("static constexpr int %s_WAVES = %d;" % (k.name.upper(), k.waves))
        assert k.waves in (2, 4)
        for nm, s in k.state.items():
            w("static constexpr int %s_%s = %d;" % (k.name.upper(), nm.replace(".", "_"), s))
        for nm, enc in k.progs.items():
            nxt = [0] * k.waves
            for row in reversed(enc):  # last level first: a level names the next one
                for v, ops in enumerate(level_blocks(row, k.waves)):
                    nxt[v] = table.add(ops, nxt[v])
            w("static constexpr int PROG_%s = %d, %s_SLOTS = %d;" % (nm.upper(), len(descs), nm.upper(), k.used[nm]))
            descs.append((nm, nxt + [0] * (4 - k.waves)))
    w("// a program: descriptors of its first level, one per wavefront")
    w("struct ProgDesc { uint32_t d[4]; };")
    w("static constexpr ProgDesc PROGS[%d] = {" % len(descs))
    for nm, d in descs:
        w("  {{0x%xu, 0x%xu, 0x%xu, 0x%xu}},  // %s" % (*d, nm))
    w("};")
    w("static constexpr int LANE_TERMS_MAX = %d;" % max(LANE_TERMS))
    words = table.finish()
    w("__device__ const uint32_t OPS[%d] __attribute__((aligned(64))) = {" % len(words))
    for k0 in range(0, len(words), 16):
        w("  %s," % ", ".join("0x%xu" % x for x in words[k0:k0 + 16]))
    w("};")
    for k in kernels:
        w("__device__ const uint32_t %s_CONSTS[%d][9] = {" % (k.name.upper(), len(k.consts)))
        for x in k.consts:
            w("  {%s}," % ", ".join("0x%08xu" % v for v in limbs29(x * RMONT % P)))
        w("};")
    G = gls_constants()
    w("// GLS decomposition on G2: lattice basis rows (signed) and rounding constants G_i")
    w("static constexpr int64_t GLS_B_NEG[4][4] = {%s};" % ", ".join(
        "{%s}" % ", ".join("%d" % (1 if x < 0 else 0) for x in row) for row in GLS_B))
    w("static constexpr uint64_t GLS_B_ABS[4][4] = {%s};" % ", ".join(
        "{%s}" % ", ".join("0x%xull" % abs(x) for x in row) for row in GLS_B))
    w("static constexpr uint32_t GLS_G[4][6] = {%s};" % ", ".join(
        "{%s}" % ", ".join("0x%08xu" % ((g >> (32 * i)) & 0xFFFFFFFF) for i in range(6)) for g in G))
    w("}  // namespace slp")
    return "\n".join(o) + "\n"


# ============================================================================ checks
def run_levels(levels, S, segbase=(0, 0, 0, 0)):
    def res(x):
        return segbase[x >> SEG_SHIFT] + (x & ((1 << SEG_SHIFT) - 1)) if x >> SEG_SHIFT else x
    for row in levels:
        out = []
        for kind, dst, na, terms in row:
            if kind == OP_MUL:
                a = sum(c * S[res(s)] for s, c in terms[:na])
                b = sum(c * S[res(s)] for s, c in terms[na:])
                out.append((res(dst), a * b % P))
            else:
                out.append((res(dst), sum(c * S[res(s)] for s, c in terms) % P))
        for d, v in out:
            S[d] = v


# plain reference: F_p12 as F_p2[w] / (w^6 - xi); coefficient j = 3h + q is w^{2q + h}
def ref_from_mem(cs):
    poly = [None] * 6
    for j in range(6):
        h, q = divmod(j, 3)
        poly[2 * q + h] = (cs[2 * j] % P, cs[2 * j + 1] % P)
    return poly


def ref_to_mem(poly):
    cs = [0] * 12
    for k in range(6):
        q, h = divmod(k, 2)
        j = 3 * h + q
        cs[2 * j], cs[2 * j + 1] = poly[k]
    return cs


def ref_mul(a, b):
    acc = [(0, 0)] * 11
    for i in range(6):
        for j in range(6):
            t = f2mul_int(a[i], b[j])
            acc[i + j] = ((acc[i + j][0] + t[0]) % P, (acc[i + j][1] + t[1]) % P)
    out = list(acc[:6])
    for k in range(6, 11):
        t = f2mul_int(acc[k], XI)
        out[k - 6] = ((out[k - 6][0] + t[0]) % P, (out[k - 6][1] + t[1]) % P)
    return out


def ref_pow(a, e):
    r = [(1, 0)] + [(0, 0)] * 5
    while e:
        if e & 1:
            r = ref_mul(r, a)
        a = ref_mul(a, a)
        e >>= 1
    return r


def ref_conj(a):  # w -> -w
    return [(c[0], c[1]) if k % 2 == 0 else ((-c[0]) % P, (-c[1]) % P) for k, c in enumerate(a)]


def ref_frob(a):
    """x -> x^p: coefficient k gets conj(c) gamma1[k]"""
    return [f2mul_int((c[0], (-c[1]) % P), GAM1[k]) for k, c in enumerate(a)]


def ref_inv(a):
    return ref_pow(a, P**12 - 2)


def ref_miller(xP, yP, Q):
    """affine Miller loop of the optimal ate pairing, lines in the w-polynomial form"""
    def add_aff(T, S):
        (x1, y1), (x2, y2) = T, S
        if T == S:
            lam = f2mul_int(f2mul_int((3, 0), f2mul_int(x1, x1)), f2inv_int(f2mul_int((2, 0), y1)))
        else:
            lam = f2mul_int(((y2[0] - y1[0]) % P, (y2[1] - y1[1]) % P), f2inv_int(((x2[0] - x1[0]) % P, (x2[1] - x1[1]) % P)))
        x3 = ((f2mul_int(lam, lam)[0] - x1[0] - x2[0]) % P, (f2mul_int(lam, lam)[1] - x1[1] - x2[1]) % P)
        t = f2mul_int(lam, ((x1[0] - x3[0]) % P, (x1[1] - x3[1]) % P))
        y3 = ((t[0] - y1[0]) % P, (t[1] - y1[1]) % P)
        # line yP - lam xP w + (lam x1 - y1) w^3
        l = [(0, 0)] * 6
        l[0] = (yP, 0)
        lx = f2mul_int(lam, (xP, 0))
        l[1] = ((-lx[0]) % P, (-lx[1]) % P)
        m = f2mul_int(lam, x1)
        l[3] = ((m[0] - y1[0]) % P, (m[1] - y1[1]) % P)
        return (x3, y3), l
    f = [(1, 0)] + [(0, 0)] * 5
    T = Q
    negQ = (Q[0], (0, 0) if Q[1] == (0, 0) else ((-Q[1][0]) % P, (-Q[1][1]) % P))
    for d in ATE_NAF[1:]:
        f = ref_mul(f, f)
        T, l = add_aff(T, T)
        f = ref_mul(f, l)
        if d:
            T, l = add_aff(T, Q if d == 1 else negQ)
            f = ref_mul(f, l)
    Q1 = (f2mul_int((Q[0][0], (-Q[0][1]) % P), FROB_TX), f2mul_int((Q[1][0], (-Q[1][1]) % P), FROB_TY))
    Q2 = (f2mul_int(Q[0], FROB2_TX), f2mul_int(Q[1], ((-FROB2_TY[0]) % P, 0)))
    T, l = add_aff(T, Q1)
    f = ref_mul(f, l)
    T, l = add_aff(T, Q2)
    f = ref_mul(f, l)
    return f


def check():
    rng = random.Random(5)
    mk, ek, fk, gk, g1k = build_all()
    for k in (mk, ek, fk, gk, g1k):
        for nm, enc in k.progs.items():
            nmul = sum(1 for r in enc for op in r if op[0] == OP_MUL)
            nmlev = sum(1 for r in enc if any(op[0] == OP_MUL for op in r))
            print("%-22s levels %4d  mul-levels %3d  MUL %5d  LIN %5d  width %2d" %
                  (nm, len(enc), nmlev, nmul, sum(len(r) for r in enc) - nmul, max(len(r) for r in enc)),
                  file=sys.stderr)
        print("kernel %s: %d slots, %d wavefronts" % (k.name, k.nslots, k.waves), file=sys.stderr)
    # F_p12 programs against the polynomial reference
    base = {"X": fk.nslots, "Y": fk.nslots + 12, "D": fk.nslots + 24}
    seg = (0, base["X"], base["Y"], base["D"], 0, 0, 0, 0)
    for trial in range(3):
        S = [rng.randrange(P) for _ in range(fk.nslots + 36)]
        for x, s in fk.cslot.items():
            S[s] = x
        X = S[base["X"]:base["X"] + 12]
        Y = S[base["Y"]:base["Y"] + 12]
        rx, ry = ref_from_mem(X), ref_from_mem(Y)
        cyc = ref_mul(ref_conj(rx), ref_inv(rx))
        cyc = ref_mul(ref_frob(ref_frob(cyc)), cyc)        # cyclotomic element
        want = {"f12_mul": ref_mul(rx, ry), "f12_frob1": ref_frob(rx), "f12_frob2": ref_frob(ref_frob(rx)),
                "f12_frob3": ref_frob(ref_frob(ref_frob(rx))), "f12_conj": ref_conj(rx),
                "f12_sqr": ref_mul(rx, rx), "f12_sqr_mul": ref_mul(ref_mul(rx, rx), ry)}
        for nm, wv in want.items():
            S2 = list(S)
            run_levels(fk.progs[nm], S2, seg)
            got = S2[base["D"]:base["D"] + 12]
            assert got == ref_to_mem(wv), nm
        # cyclotomic squaring on a cyclotomic input
        S2 = list(S)
        S2[base["X"]:base["X"] + 12] = ref_to_mem(cyc)
        run_levels(fk.progs["f12_csqr"], S2, seg)
        assert S2[base["D"]:base["D"] + 12] == ref_to_mem(ref_mul(cyc, cyc)), "csqr"
        S2 = list(S)
        S2[base["X"]:base["X"] + 12] = ref_to_mem(cyc)
        run_levels(fk.progs["f12_csqr_mul"], S2, seg)
        assert S2[base["D"]:base["D"] + 12] == ref_to_mem(ref_mul(ref_mul(cyc, cyc), ry)), "csqr_mul"
    print("F_p12 programs ok", file=sys.stderr)
    S = [0] * ek.nslots
    for x, sl in ek.cslot.items():
        S[sl] = x
    fin = [rng.randrange(P) for _ in range(12)]
    for k in range(12):
        S[ek.state["X.%d" % k]] = fin[k]
    run_levels(ek.progs["fe_norm"], S)
    S[ek.state["tinv"]] = pow(S[ek.state["t"]], -1, P)
    run_levels(ek.progs["fe_rest"], S)
    got = [S[ek.state["D.%d" % k]] for k in range(12)]
    assert got == ref_to_mem(ref_pow(ref_from_mem(fin), (P**12 - 1) // R)), "final exponentiation"
    print("final exponentiation ok", file=sys.stderr)
    # Miller loop: the program vs the affine reference, compared after the
    # final exponentiation (the two differ by factors in proper subfields)
    g2 = ((10857046999023057135944570762232829481370756359578518086990519993285655852781,
           11559732032986387107991004021392285783925812861821192530917403151452391805634),
          (8495653923123431417604973247489272438418190587263600148770280649306958101930,
           4082367875863433681332203403145435568316851327593401208105741076214120093531))
    xP, yP = 1, 2
    S = [0] * mk.nslots
    for x, s in mk.cslot.items():
        S[s] = x
    st = mk.state
    S[st["xP"]], S[st["yP"]] = xP, yP
    S[st["xQ.0"]], S[st["xQ.1"]], S[st["yQ.0"]], S[st["yQ.1"]] = g2[0][0], g2[0][1], g2[1][0], g2[1][1]
    run_levels(mk.progs["ml"], S)
    f = ref_from_mem([S[st["f.%d" % k]] for k in range(12)])
    g = ref_miller(xP, yP, g2)
    e = (P**12 - 1) // R
    assert ref_pow(f, e) == ref_pow(g, e), "Miller loop"
    print("Miller loop ok", file=sys.stderr)
    check_g2(gk, rng)
    check_g1(g1k, rng)


def f2add(a, b):
    return ((a[0] + b[0]) % P, (a[1] + b[1]) % P)


def f2sub(a, b):
    return ((a[0] - b[0]) % P, (a[1] - b[1]) % P)


def aff_add(A, B):
    """affine addition on the twist (None = identity)"""
    if A is None:
        return B
    if B is None:
        return A
    if A[0] == B[0]:
        if f2add(A[1], B[1]) == (0, 0):
            return None
        lam = f2mul_int(f2mul_int((3, 0), f2mul_int(A[0], A[0])), f2inv_int(f2mul_int((2, 0), A[1])))
    else:
        lam = f2mul_int(f2sub(B[1], A[1]), f2inv_int(f2sub(B[0], A[0])))
    x3 = f2sub(f2sub(f2mul_int(lam, lam), A[0]), B[0])
    return (x3, f2sub(f2mul_int(lam, f2sub(A[0], x3)), A[1]))


def aff_mul(A, k):
    R_ = None
    for bit in bin(k)[2:]:
        R_ = aff_add(R_, R_)
        if bit == "1":
            R_ = aff_add(R_, A)
    return R_


G2GEN = ((10857046999023057135944570762232829481370756359578518086990519993285655852781,
          11559732032986387107991004021392285783925812861821192530917403151452391805634),
         (8495653923123431417604973247489272438418190587263600148770280649306958101930,
          4082367875863433681332203403145435568316851327593401208105741076214120093531))


def check_g2(gk, rng):
    lam = P % R
    st = gk.state
    def setsum(S, pt):  # T from affine on the isomorphic curve, the sums split at random
        x, y = (0, 0), (1, 0)
        z = (0, 0)
        if pt is not None:
            x, y, z = f2mul_int(pt[0], G2_U2), f2mul_int(pt[1], G2_U3), (1, 0)
        for c, v in enumerate((x, y, z)):
            for h in (0, 1):
                r = [rng.randrange(P) for _ in range(G2_SUM - 1)]
                for k, w in enumerate(r + [(v[h] - sum(r)) % P]):
                    S[st["T.%d.%d.%d" % (c, h, k)]] = w
    def aff(X, Y, Z, iso=True):
        if Z == (0, 0):
            return None
        zi = f2inv_int(Z)
        x, y = f2mul_int(X, zi), f2mul_int(Y, zi)
        ui2 = f2mul_int(G2_UI, G2_UI)
        return (f2mul_int(x, ui2), f2mul_int(y, f2mul_int(ui2, G2_UI)))
    def getsum(S):
        v = [tuple(sum(S[st["T.%d.%d.%d" % (c, h, k)]] for k in range(G2_SUM)) % P for h in (0, 1)) for c in range(3)]
        return aff(*v)
    def gettab(S, d):
        v = [S[st["TB%d.%d" % (d, k)]] % P for k in range(6)]
        return aff((v[0], v[1]), (v[2], v[3]), (v[4], v[5]))
    for trial in range(2):
        Q = aff_mul(G2GEN, rng.randrange(1, R))
        S = [0] * gk.nslots
        for x, sl in gk.cslot.items():
            S[sl] = x
        S[st["xQ.0"]], S[st["xQ.1"]], S[st["yQ.0"]], S[st["yQ.1"]] = Q[0][0], Q[0][1], Q[1][0], Q[1][1]
        run_levels(gk.progs["g2_bases"], S)
        run_levels(gk.progs["g2_table"], S)
        for d in range(1, 16):
            want = None
            for j in range(4):
                if d >> j & 1:
                    want = aff_add(want, aff_mul(Q, pow(lam, j, R)))
            assert gettab(S, d) == want, ("table", d)
        for A in (Q, aff_mul(Q, 7), None):
            setsum(S, A)
            run_levels(gk.progs["g2_dbl"], S)
            A2 = aff_add(A, A)
            assert getsum(S) == A2, "dbl"
            base = st["TB5.0"]
            setsum(S, A)
            run_levels(gk.progs["g2_dbl_add"], S, (0, 0, base, 0))
            assert getsum(S) == aff_add(A2, gettab(S, 5)), "dbl_add"
        for A in (Q, None, gettab(S, 5), (gettab(S, 5)[0], ((-gettab(S, 5)[1][0]) % P, (-gettab(S, 5)[1][1]) % P))):
            setsum(S, A)
            run_levels(gk.progs["g2_add"], S, (0, 0, st["TB5.0"], 0))
            assert getsum(S) == aff_add(A, gettab(S, 5)), "add"
            run_levels(gk.progs["g2_madd"], S)
            want = aff_add(aff_add(A, gettab(S, 5)), Q)
            assert getsum(S) == want, "madd"
        run_levels(gk.progs["g2_norm"], S)
        S[st["tinv"]] = pow(S[st["t"]], -1, P)
        run_levels(gk.progs["g2_aff"], S)
        assert ((S[st["ax.0"]], S[st["ax.1"]]), (S[st["ay.0"]], S[st["ay.1"]])) == want, "aff"
        run_levels(gk.progs["g2_load"], S)
        assert getsum(S) == Q, "load"
        # the Jacobian programs
        def setj(name, pt):
            for k, v in enumerate((*pt[0], *pt[1], 1, 0)):
                S[st["%s.%d" % (name, k)]] = v
        def getj():
            v = [S[st["J.%d" % k]] % P for k in range(6)]
            X, Y, Z = (v[0], v[1]), (v[2], v[3]), (v[4], v[5])
            zi = f2inv_int(Z)
            zi2 = f2mul_int(zi, zi)
            return (f2mul_int(X, zi2), f2mul_int(Y, f2mul_int(zi2, zi)))
        setj("J", Q)
        run_levels(gk.progs["g2_jdbl"], S)
        assert getj() == aff_add(Q, Q), "jdbl"
        setj("TB1", Q)
        run_levels(gk.progs["g2_jadd"], S, (0, 0, st["TB1.0"], 0))
        assert getj() == aff_add(aff_add(Q, Q), Q), "jadd"
        setj("J", Q)
        run_levels(gk.progs["g2_jadd"], S, (0, 0, st["TB1.0"], 0))
        assert S[st["H.0"]] % P == 0 and S[st["H.1"]] % P == 0 and S[st["RR.0"]] % P == 0 and S[st["RR.1"]] % P == 0
    # decomposition
    for k in [0, 1, R - 1] + [rng.randrange(R) for _ in range(2000)]:
        kj = gls_decompose(k)
        assert (sum(kj[j] * pow(lam, j, R) for j in range(4)) - k) % R == 0 and max(abs(x) for x in kj) < 2**65
    print("G2 programs and GLS decomposition ok", file=sys.stderr)


def g1_aff_add(A, B):
    if A is None:
        return B
    if B is None:
        return A
    if A[0] == B[0]:
        if (A[1] + B[1]) % P == 0:
            return None
        l = 3 * A[0] * A[0] * pow(2 * A[1], -1, P) % P
    else:
        l = (B[1] - A[1]) * pow(B[0] - A[0], -1, P) % P
    x = (l * l - A[0] - B[0]) % P
    return (x, (l * (A[0] - x) - A[1]) % P)


def g1_aff_mul(A, k):
    R_ = None
    for bit in bin(k)[2:]:
        R_ = g1_aff_add(R_, R_)
        if bit == "1":
            R_ = g1_aff_add(R_, A)
    return R_


def check_g1(g1k, rng):
    st = g1k.state
    def setsum(S, pt):
        for c, v in enumerate((0, 1, 0) if pt is None else (pt[0], pt[1], 1)):
            r = rng.randrange(P)
            S[st["T.%d.0" % c]], S[st["T.%d.1" % c]] = r, (v - r) % P
    def aff(X, Y, Z):
        if Z % P == 0:
            return None
        zi = pow(Z, -1, P)
        return (X * zi % P, Y * zi % P)
    def getsum(S):
        return aff(*((S[st["T.%d.0" % c]] + S[st["T.%d.1" % c]]) % P for c in range(3)))
    def gettab(S, d):
        return aff(*(S[st["TB%d.%d" % (d, k)]] for k in range(3)))
    for trial in range(3):
        Pt = g1_aff_mul((1, 2), rng.randrange(1, R))
        S = [0] * g1k.nslots
        for x, sl in g1k.cslot.items():
            S[sl] = x
        S[st["xP"]], S[st["yP"]] = Pt
        run_levels(g1k.progs["g1_phi"], S)
        assert (S[st["B1.x"]] % P, Pt[1]) == g1_aff_mul(Pt, GLV_LAM), "phi"
        S[st["B1.y"]] = Pt[1]
        run_levels(g1k.progs["g1_table"], S)
        for d in range(1, 16):
            want = g1_aff_add(g1_aff_mul(Pt, d & 3), g1_aff_mul(Pt, (d >> 2) * GLV_LAM % R)) if d & 3 else \
                g1_aff_mul(Pt, (d >> 2) * GLV_LAM % R)
            assert gettab(S, d) == want, ("table", d)
        T7 = gettab(S, 7)
        for A in (Pt, T7, (T7[0], -T7[1] % P), None):
            A4 = None if A is None else g1_aff_mul(A, 4)
            setsum(S, A)
            run_levels(g1k.progs["g1_dbl2"], S)
            assert getsum(S) == A4, "dbl2"
            setsum(S, A)
            run_levels(g1k.progs["g1_dbl2_add"], S, (0, 0, st["TB7.0"], 0))
            assert getsum(S) == g1_aff_add(A4, T7), "dbl2_add"
            setsum(S, A)
            run_levels(g1k.progs["g1_add"], S, (0, 0, st["TB7.0"], 0))
            assert getsum(S) == g1_aff_add(A, T7), "add"
            run_levels(g1k.progs["g1_madd"], S)
            want = g1_aff_add(g1_aff_add(A, T7), Pt)
            assert getsum(S) == want, "madd"
        S[st["tinv"]] = pow(S[st["T.2.0"]] + S[st["T.2.1"]], -1, P)
        run_levels(g1k.progs["g1_aff"], S)
        assert (S[st["ax"]] % P, S[st["ay"]] % P) == want, "aff"
    print("G1 programs ok", file=sys.stderr)


if __name__ == "__main__":
    if "--check" in sys.argv:
        check()
    else:
        sys.stdout.write(emit(list(build_all())))
