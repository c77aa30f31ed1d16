"""Generate qlskum_erfc_coeffs.h: polynomial coefficients of the scaled
complementary error function and of the exponential used by the flux
kernels.

For y >= 0 write t = c / (c + y) in (0, 1] and
    erfc(y) = exp(-y^2) * t * R(t),    R(t) = erfc(y) exp(y^2) / t,
where R is smooth on [0, 1] (R(0) = 1 / (c sqrt(pi))).  R is interpolated
at Chebyshev points of u = 2t - 1 = (c - y)/(c + y) in 50-digit arithmetic
(mpmath) and the Chebyshev series is converted exactly to monomials in u
before rounding, so the kernels evaluate it by Horner's rule (one fma per
term; the monomial coefficients sum to about 1 in magnitude, so the
conversion costs no accuracy).
FP64: c = 3.5, 23 terms (max relative error 2.7e-16 in double);
FP32: c = 2, 11 terms.

For |y| <= 1 (the range of S = u_e sqrt(beta) below local Mach ~1.2) the
FP32 path uses a shorter form: erf(y) = y P(y^2) with P the near-minimax
polynomial of erf(sqrt(u)) / sqrt(u) on u in [0, 1] from mpmath's Chebyshev
fit, 6 coefficients (fit error 4.1e-8).
For |y| <= 1.25 (local Mach below ~1.5) the FP64 flux kernel uses the same
form, erf(y)/2 = y P(y^2) with 14 coefficients on u in [0, 1.25^2] (fit error
1.1e-18).
Exponential (FP64): exp(r) on |r| <= ln2/2 by the degree-11 polynomial of
mpmath's Chebyshev fit (fit error 3.2e-18; with the two-part reduction
x = k ln2 + r, 1.4e-16 relative in double), and ln2 split into a double and
its remainder.
Run from this directory:
    python gen_erfc.py > qlskum_erfc_coeffs.h
"""
import mpmath as mp

mp.mp.dps = 50


def coeffs(c, n, nodes=80):
    """Chebyshev interpolation coefficients of R on [-1, 1] in u, truncated
    to n terms (series sum_k a_k T_k(u))."""
    c = mp.mpf(c)

    def R(t):
        if t == 0:
            return 1 / (c * mp.sqrt(mp.pi))
        y = c / t - c
        return mp.erfc(y) * mp.exp(y * y) / t

    th = [mp.pi * (j + mp.mpf(1) / 2) / nodes for j in range(nodes)]
    fx = [R((mp.cos(a) + 1) / 2) for a in th]
    out = [2 * mp.fsum(fx[j] * mp.cos(k * th[j]) for j in range(nodes)) / nodes for k in range(n)]
    out[0] /= 2
    return out


def monomial(cheb):
    """Exact conversion of sum_k a_k T_k(u) to sum_k m_k u^k."""
    n = len(cheb)
    T = [[mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]]
    for k in range(2, n):
        a = [mp.mpf(0)] + [2 * v for v in T[k - 1]]
        b = T[k - 2] + [mp.mpf(0)] * (len(a) - len(T[k - 2]))
        T.append([x - y for x, y in zip(a, b)])
    m = [mp.mpf(0)] * n
    for j in range(n):
        for k, v in enumerate(T[j]):
            m[k] += cheb[j] * v
    return m


def small(n):
    def f(u):
        if u == 0:
            return 2 / mp.sqrt(mp.pi)
        return mp.erf(mp.sqrt(u)) / mp.sqrt(u)
    return mp.chebyfit(f, [0, 1], n)  # highest power first


def small64(edge, n):
    def f(u):
        if u == 0:
            return 1 / mp.sqrt(mp.pi)
        return mp.erf(mp.sqrt(u)) / (2 * mp.sqrt(u))
    return mp.chebyfit(f, [0, mp.mpf(edge) ** 2], n)  # highest power first


def exp_poly(deg):
    half = mp.log(2) / 2
    return mp.chebyfit(mp.exp, [-half, half], deg + 1)[::-1]  # lowest power first


def main():
    m64 = monomial(coeffs("3.5", 23))
    e64 = exp_poly(11)
    ln2 = mp.log(2)
    ln2_hi = mp.mpf(float(ln2))
    m32 = monomial(coeffs(2, 11))
    p32 = small(6)
    print("// Generated by gen_erfc.py: monomial coefficients (lowest power first)")
    print("// of R(t) = erfc(y) exp(y^2) / t,  t = c / (c + y),  in u = 2t - 1.")
    print("#pragma once")
    print("namespace ql {")
    print("constexpr double kErfcC64 = 3.5;")
    print(f"constexpr int kErfcN64 = {len(m64)};")
    print("constexpr double kErfcPoly64[kErfcN64] = {")
    for v in m64:
        print(f"    {mp.nstr(v, 20, min_fixed=0, max_fixed=0)},")
    print("};")
    print("constexpr float kErfcC32 = 2.0f;")
    print(f"constexpr int kErfcN32 = {len(m32)};")
    print("constexpr float kErfcPoly32[kErfcN32] = {")
    for v in m32:
        print(f"    {mp.nstr(v, 12, min_fixed=0, max_fixed=0)}f,")
    print("};")
    print("// erf(y) = y P(y^2) for |y| <= 1, P highest power first")
    print(f"constexpr int kErfP32N = {len(p32)};")
    print("constexpr float kErfP32[kErfP32N] = {")
    for v in p32:
        print(f"    {mp.nstr(v, 12, min_fixed=0, max_fixed=0)}f,")
    print("};")
    p64 = small64("1.25", 14)
    print("// erf(y) / 2 = y P(y^2) for |y| <= kErfNear64, P highest power first")
    print("constexpr double kErfNear64 = 1.25;")
    print(f"constexpr int kErfN64 = {len(p64)};")
    print("constexpr double kErfPoly64[kErfN64] = {")
    for v in p64:
        print(f"    {mp.nstr(v, 20, min_fixed=0, max_fixed=0)},")
    print("};")
    print("// exp(r) = sum_k e_k r^k for |r| <= ln2/2 (lowest power first); ln2 = hi + lo")
    print(f"constexpr double kLog2e = {mp.nstr(1 / ln2, 20, min_fixed=0, max_fixed=0)};")
    print(f"constexpr double kLn2Hi = {mp.nstr(ln2_hi, 20, min_fixed=0, max_fixed=0)};")
    print(f"constexpr double kLn2Lo = {mp.nstr(ln2 - ln2_hi, 20, min_fixed=0, max_fixed=0)};")
    print(f"constexpr int kExpN64 = {len(e64)};")
    print("constexpr double kExpPoly64[kExpN64] = {")
    for v in e64:
        print(f"    {mp.nstr(v, 20, min_fixed=0, max_fixed=0)},")
    print("};")
    print("}  // namespace ql")


if __name__ == "__main__":
    main()
