"""Generate constants.hpp: BN254 constants for the HIP kernels, derived here from
the curve parameter u with Python integers (no tables copied from elsewhere).

Run:  python gen_constants.py > constants.hpp
"""
import sys

U = 0x44E992B44A6909F1
P = 36 * U**4 + 36 * U**3 + 24 * U**2 + 6 * U + 1
R = 36 * U**4 + 36 * U**3 + 18 * U**2 + 6 * U + 1
RM = 1 << 256


def limbs(x, n=8):
    return [(x >> (32 * i)) & 0xFFFFFFFF for i in range(n)]


def arr(name, x, n=8):
    return "static constexpr uint32_t %s[%d] = {%s};" % (name, n, ", ".join("0x%08xu" % v for v in limbs(x, n)))


def mont(x, m=P):
    return x * RM % m


# F_p2 arithmetic with i^2 = -1
def f2mul(a, b):
    return ((a[0] * b[0] - a[1] * b[1]) % P, (a[0] * b[1] + a[1] * b[0]) % P)


def f2pow(a, e):
    r = (1, 0)
    while e:
        if e & 1:
            r = f2mul(r, a)
        a = f2mul(a, a)
        e >>= 1
    return r


def f2inv(a):
    n = pow(a[0] * a[0] + a[1] * a[1], -1, P)
    return (a[0] * n % P, -a[1] * n % P)


def f2conj(a):
    return (a[0], -a[1] % P)


XI = (9, 1)
out = []
w = out.append
w("// Generated by gen_constants.py -- BN254 constants for the HIP kernels.")
w("#pragma once")
w("#include <cstdint>")
w("namespace bn {")
w(arr("P_MOD", P))
w("static constexpr uint32_t P_INV = 0x%08xu;  // -p^{-1} mod 2^32" % ((-pow(P, -1, 1 << 32)) % (1 << 32)))
w("static constexpr uint32_t P_MOD29[9] = {%s};  // radix 2^29" % ", ".join("0x%08xu" % ((P >> (29 * i)) & 0x1fffffff) for i in range(9)))
w("static constexpr uint32_t P_INV29 = 0x%08xu;  // -p^{-1} mod 2^29" % ((-pow(P, -1, 1 << 29)) % (1 << 29)))
w("static constexpr uint32_t R_MOD29[9] = {%s};" % ", ".join("0x%08xu" % ((R >> (29 * i)) & 0x1fffffff) for i in range(9)))
w("static constexpr uint32_t R_INV29 = 0x%08xu;" % ((-pow(R, -1, 1 << 29)) % (1 << 29)))
w(arr("P_ONE", mont(1)))
w(arr("P_R2", RM * RM % P))
w(arr("P_MINUS_2", P - 2))
w(arr("P_SQRT_EXP", (P - 3) // 4))
w(arr("P_HALF", (P - 1) // 2))
w(arr("R_MOD", R))
w("static constexpr uint32_t R_INV = 0x%08xu;  // -r^{-1} mod 2^32" % ((-pow(R, -1, 1 << 32)) % (1 << 32)))
w(arr("R_ONE", mont(1, R)))
w(arr("R_R2", RM * RM % R))
w(arr("R_MINUS_2", R - 2))
w(arr("R_R3", RM**3 % R))
w(arr("P_R3", RM**3 % P))
w(arr("R_R1", RM % R))  # 2^256 mod r
# twist constant b' = 3 / xi
bt = f2mul((3, 0), f2inv(XI))
w(arr("TWIST_B0", mont(bt[0])))
w(arr("TWIST_B1", mont(bt[1])))


def centred29(x):
    """radix 2^29, limbs 0 .. 7 in [-2^28, 2^28)"""
    v = []
    for i in range(9):
        d = x & 0x1fffffff
        if i < 8 and d >= 1 << 28:
            d -= 1 << 29
        v.append(d if i < 8 else x)
        x = (x - d) >> 29
    return "{%s}" % ", ".join(map(str, v))


# for the one-lane formulas, with factor 2^261: 1 and 3 b'
w("static constexpr int32_t P_ONE29[9] = %s;" % centred29(2**261 % P))
w("static constexpr int32_t TWIST_3B29[2][9] = {%s};" % ", ".join(centred29(3 * c * 2**261 % P) for c in bt))
# Frobenius coefficients: gamma1[k] = xi^{k(p-1)/6}, gamma2[k] = xi^{k(p^2-1)/6} (in F_p),
# gamma3[k] = xi^{k(p^3-1)/6}
g1 = [f2pow(XI, k * (P - 1) // 6) for k in range(6)]
g2 = [f2pow(XI, k * (P * P - 1) // 6) for k in range(6)]
g3 = [f2pow(XI, k * (P**3 - 1) // 6) for k in range(6)]
for k in range(6):
    assert g2[k][1] == 0
for k in range(1, 6):
    w(arr("FROB1_%d_0" % k, mont(g1[k][0])))
    w(arr("FROB1_%d_1" % k, mont(g1[k][1])))
    w(arr("FROB2_%d" % k, mont(g2[k][0])))
    w(arr("FROB3_%d_0" % k, mont(g3[k][0])))
    w(arr("FROB3_%d_1" % k, mont(g3[k][1])))
# twist Frobenius: psi^-1 pi psi (x, y) = (conj(x) xi^{(p-1)/3}, conj(y) xi^{(p-1)/2})
tx, ty = f2pow(XI, (P - 1) // 3), f2pow(XI, (P - 1) // 2)
assert tx == g1[2] and ty == g1[3]
# optimal ate loop 6u+2 and the final-exponent parameter u
w("static constexpr uint64_t ATE_LOOP = 0x%xull;  // low 64 bits of 6u+2 (bit 64 set)" % ((6 * U + 2) & (2**64 - 1)))
assert (6 * U + 2) >> 64 == 1
# its non-adjacent form: 22 nonzero digits against 37 set bits; the top digit is d_65 = 1 and
# d_64 = 0, so the digits d_0 .. d_63 are two masks (+1 and -1)
naf, k = [], 6 * U + 2
while k:
    z = (2 - k % 4) if k & 1 else 0
    naf.append(z)
    k = (k - z) // 2
assert len(naf) == 66 and naf[65] == 1 and naf[64] == 0
assert sum(d << i for i, d in enumerate(naf)) == 6 * U + 2
assert all(naf[i] == 0 or naf[i + 1] == 0 for i in range(65))
w("static constexpr uint64_t ATE_NAF_POS = 0x%xull;  // digits +1 of the NAF of 6u+2 below d_64 (d_65 = 1, d_64 = 0)"
  % sum(1 << i for i in range(64) if naf[i] == 1))
w("static constexpr uint64_t ATE_NAF_NEG = 0x%xull;  // digits -1" % sum(1 << i for i in range(64) if naf[i] == -1))
w("static constexpr uint64_t BN_U = 0x%xull;" % U)
# G1, G2 generators (Montgomery)
w(arr("G1X", mont(1)))
w(arr("G1Y", mont(2)))
G2X = (10857046999023057135944570762232829481370756359578518086990519993285655852781,
       11559732032986387107991004021392285783925812861821192530917403151452391805634)
G2Y = (8495653923123431417604973247489272438418190587263600148770280649306958101930,
       4082367875863433681332203403145435568316851327593401208105741076214120093531)
w(arr("G2X0", mont(G2X[0])))
w(arr("G2X1", mont(G2X[1])))
w(arr("G2Y0", mont(G2Y[0])))
w(arr("G2Y1", mont(G2Y[1])))
# check the hard part of the final exponent decomposes exactly
lam = [-36 * U**3 - 30 * U**2 - 18 * U - 2, -36 * U**3 - 18 * U**2 - 12 * U + 1, 6 * U**2 + 1, 1]
assert sum(l * P**k for k, l in enumerate(lam)) == (P**4 - P**2 + 1) // R
# GLV on G1: phi(x, y) = (beta x, y) acts as multiplication by lam (beta^3 = 1 in F_p,
# lam^2 + lam + 1 = 0 mod r); the pair is fixed by checking phi(g1) = lam g1 in the tests.
# Reduced basis of {(a, b): a + b lam = 0 mod r} and Babai rounding constants
# G_i = round(alpha_i 2^256) with alpha = the first row of the inverse basis.
GLV_BETA = 0x59E26BCEA0D48BACD4F263F1ACDB5C4F5763473177FFFFFE
GLV_LAM = 0xB3C4D79D41A917585BFC41088D8DAAA78B17EA66B99C90DD
assert pow(GLV_BETA, 3, P) == 1 and (GLV_LAM * GLV_LAM + GLV_LAM + 1) % R == 0
GLV_B = [[-(2 * U + 1), 6 * U * U + 2 * U], [-(6 * U * U + 4 * U + 1), -(2 * U + 1)]]
for row in GLV_B:
    assert (row[0] + row[1] * GLV_LAM) % R == 0
_det = GLV_B[0][0] * GLV_B[1][1] - GLV_B[0][1] * GLV_B[1][0]
_alpha = [GLV_B[1][1], -GLV_B[0][1]]  # first row of the inverse times det
GLV_G = [(a * 2**256 + _det // 2) // _det if _det > 0 else -((a * 2**256 - _det // 2) // -_det) for a in _alpha]
w(arr("GLV_BETA", mont(GLV_BETA)))
w("static constexpr uint32_t GLV_B_NEG[2][2] = {%s};" % ", ".join(
    "{%s}" % ", ".join("%d" % (1 if x < 0 else 0) for x in row) for row in GLV_B))
w("static constexpr uint32_t GLV_B_ABS[2][2][4] = {%s};" % ", ".join(
    "{%s}" % ", ".join("{%s}" % ", ".join("0x%08xu" % ((abs(x) >> (32 * i)) & 0xFFFFFFFF) for i in range(4)) for x in row)
    for row in GLV_B))
w("static constexpr uint32_t GLV_G_NEG[2] = {%s};" % ", ".join("%d" % (1 if g < 0 else 0) for g in GLV_G))
w("static constexpr uint32_t GLV_G_ABS[2][5] = {%s};" % ", ".join(
    "{%s}" % ", ".join("0x%08xu" % ((abs(g) >> (32 * i)) & 0xFFFFFFFF) for i in range(5)) for g in GLV_G))
assert all(abs(g) < 2**160 for g in GLV_G)
w("}  // namespace bn")
sys.stdout.write("\n".join(out) + "\n")
