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


def test_fp64_pair_functions_against_exact(tmp_path):
    """2^x, 1/sqrt and the erfc of the FP32 tiles' FP64 pairs, compiled for the host from the kernel source
    (the hardware's estimates at 24 bits), in units of 2^-53: one rounding for the first two, with a tenth for
    what it rounds; three for erfc up to 3.8 (the Gaussian's, the product's, and what P's inner steps leave)."""
    import ctypes
    import subprocess

    import mpmath as mp
    mp.mp.dps = 40
    body = open(SRC).read()
    body = body[body.index("constexpr double kExp2Poly"):body.index("__device__ __forceinline__ float d_length")]
    (tmp_path / "f.cpp").write_text("""
#include <cmath>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
#define __builtin_amdgcn_rsq(x) ((double)(1.0f / sqrtf((float)(x))))
""" + body + """
extern "C" void run(int n, const double* x, double* o)
{
    for (int i = 0; i < n; ++i, o += 3) {
        o[0] = d_exp2(-x[i] * x[i]);
        o[1] = d_rsqrt(x[i]);
        o[2] = erfc_fit(x[i]);
    }
}
""")
    subprocess.check_call(["g++", "-O2", "-mfma", "-ffp-contract=off", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                           str(tmp_path / "f.cpp"), "-o", str(tmp_path / "f.so")])
    x = np.concatenate([np.random.default_rng(5).uniform(0.0, 3.8, 3000), 10.0 ** -np.arange(1.0, 9.0)])
    out = np.empty((len(x), 3))
    run = ctypes.CDLL(str(tmp_path / "f.so")).run
    run(len(x), ctypes.c_void_p(x.ctypes.data), ctypes.c_void_p(out.ctypes.data))
    for v, o in zip(x, out):
        z = mp.mpf(float(v))
        exact = mp.mpf(2) ** mp.mpf(float(-v * v)), 1 / mp.sqrt(z), mp.erfc(z)
        for f, units, ref in zip(o, (1.1, 1.1, 3.0), exact):
            assert abs(mp.mpf(float(f)) / ref - 1) <= units * mp.mpf(2) ** -53, (v, units)
    # where 2^x ends: an argument beyond any int, zero, and a denormal
    ends = np.array([1e200, 40.0, 32.0])
    run(3, ctypes.c_void_p(ends.ctypes.data), ctypes.c_void_p(out.ctypes.data))
    assert list(out[:3, 0]) == [0.0, 0.0, 2.0 ** -1024]
