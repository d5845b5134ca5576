"""Generate the FP64 coefficients of the real-space pair kernels (realspace.hip).

erfc(x) exp(x^2) on [0, 6.5]: Chebyshev interpolant of degree 19 in y, the affine map of 4 / (4 + x)
onto [-1, 1]; (2^f - 1) / f on [-1/2, 1/2]: Chebyshev interpolant of degree 10.  Both in 60-digit
arithmetic, as powers of y and f.  Run: python fit_fp64.py  (prints the coefficients, lowest order
first, and the largest relative errors)."""
import mpmath as mp

mp.mp.dps = 60
XMAX, K = mp.mpf("6.5"), mp.mpf(4)


def powers(f, a, b, n):
    """Powers of y in [-1, 1] of the degree-n Chebyshev interpolant of f on [a, b]."""
    th = [mp.pi * (k + mp.mpf(1) / 2) / (n + 1) for k in range(n + 1)]
    v = [f((a + b) / 2 + (b - a) / 2 * mp.cos(t)) for t in th]
    c = [sum(vk * mp.cos(j * t) for vk, t in zip(v, th)) * 2 / (n + 1) for j in range(n + 1)]
    c[0] /= 2
    t0, t1 = [mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]
    out = [c[0]] + [mp.mpf(0)] * n
    for j in range(1, n + 1):
        for i, q in enumerate(t1):
            out[i] += c[j] * q
        t2 = [mp.mpf(0)] + [2 * q for q in t1]
        for i, q in enumerate(t0):
            t2[i] -= q
        t0, t1 = t1, t2
    return out


def erfcx(x):
    return mp.erfc(x) * mp.exp(x * x)


def erfc_poly():
    a, b = K / (K + XMAX), mp.mpf(1)
    return powers(lambda t: erfcx(K / t - K), a, b, 19), 2 * K / (b - a), -(a + b) / (b - a)


def exp2_poly():
    def f(z):
        return (mp.mpf(2) ** z - 1) / z if abs(z) > mp.mpf(10) ** -20 else mp.log(2)
    return [q * mp.mpf(2) ** i for i, q in enumerate(powers(f, mp.mpf(-0.5), mp.mpf(0.5), 10))]


if __name__ == "__main__":
    p, scale, shift = erfc_poly()
    print("kErfcYScale", repr(float(scale)), "kErfcYShift", repr(float(shift)))
    print("kErfcPoly", [float(q) for q in p])
    x = [XMAX * i / 300 for i in range(301)]
    print("error", mp.nstr(max(abs(mp.polyval(p[::-1], scale / (K + v) + shift) / erfcx(v) - 1) for v in x), 3))
    q = exp2_poly()
    print("kExp2Poly", [float(v) for v in q])
    z = [mp.mpf(i) / 200 - mp.mpf(1) / 2 for i in range(201)]
    print("error", mp.nstr(max(abs((1 + v * mp.polyval(q[::-1], v)) / mp.mpf(2) ** v - 1) for v in z), 3))
