"""The FP32 erfc used by the real-space pair kernels (coefficients read from the kernel source)
against scipy's scaled complementary error function, evaluated in FP32 as on the GPU."""
import os
import re

import numpy as np
from scipy.special import erfc, erfcx

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2011_01207_amd", "csrc",
                   "realspace.hip")


def kernel_coefficients():
    body = open(SRC).read()
    body = body[body.index("d_erfc_g(float x, float gauss)"):]
    body = body[:body.index("return p * gauss;")]
    first = float(re.search(r"float p = ([-0-9.e+]+)f;", body).group(1))
    rest = [float(v) for v in re.findall(r"fmaf\(p, t, ([-0-9.e+]+)f\)", body)]
    return [first] + rest   # highest order first


def test_fp32_erfc_relative_error():
    coef = np.array(kernel_coefficients(), dtype=np.float32)
    assert len(coef) == 10
    x = np.linspace(0.0, 4.5, 200001).astype(np.float32)
    t0 = (np.float32(1.0) / (np.float32(1.0) + np.float32(0.5) * x)).astype(np.float32)
    # the kernel takes t from the hardware reciprocal (within 1 ulp): check t and its neighbours
    for t in (t0, np.nextafter(t0, np.float32(0.0)), np.nextafter(t0, np.float32(2.0))):
        p = np.full_like(t, coef[0])
        for cval in coef[1:]:
            p = (p * t + cval).astype(np.float32)
        rel = np.abs(p.astype(np.float64) - erfcx(x.astype(np.float64))) / erfcx(x.astype(np.float64))
        assert rel.max() < 6e-7
        # with the Gaussian factor: erfc itself to FP32-level relative accuracy
        e = p.astype(np.float64) * np.exp(-x.astype(np.float64) ** 2)
        assert np.max(np.abs(e - erfc(x.astype(np.float64))) / erfc(x.astype(np.float64))) < 6e-7


def kernel_table(name):
    m = re.search(r"constexpr double %s\[\d+\] = \{([^}]*)\};" % name, open(SRC).read())
    return [float(v) for v in m.group(1).replace("\n", " ").split(",")]


def kernel_horner(coef, x):
    """The value and a bound on its rounding: 2 n u sum |c_k| |x|^k."""
    p = np.full_like(x, coef[-1])
    for c in coef[-2::-1]:
        p = p * x + c
    return p, 2 * len(coef) * 2.0 ** -53 * sum(abs(c) * np.abs(x) ** k for k, c in enumerate(coef))


def test_fp64_erfc_and_exp2_polynomials():
    """The FP64 polynomials at their rounding bounds (and a few units of scipy's own), the erfc also
    past the end of its fit, where the Gaussian makes it nothing beside a field."""
    body = open(SRC).read()
    scale, shift = (float(v) for v in re.search(
        r"kErfcYScale = ([-0-9.]+), kErfcYShift = ([-0-9.]+);", body).groups())
    x = np.linspace(0.0, 6.5, 100001)
    p, bound = kernel_horner(kernel_table("kErfcPoly"), scale / (4.0 + x) + shift)
    assert np.all(np.abs(p - erfcx(x)) <= bound + 4e-15 * erfcx(x))
    far = np.linspace(6.5, 40.0, 1001)
    p, _ = kernel_horner(kernel_table("kErfcPoly"), scale / (4.0 + far) + shift)
    assert np.all(np.abs(p - erfcx(far)) * np.exp(-far ** 2) < 1e-20)
    f = np.linspace(-0.5, 0.5, 100001)
    q, bound = kernel_horner([1.0] + kernel_table("kExp2Poly"), f)
    assert np.all(np.abs(q - np.exp2(f)) <= bound + 4e-16)
