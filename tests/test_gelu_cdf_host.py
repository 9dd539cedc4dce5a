"""The normal CDF of the bf16 GELU epilogues (pf_gelu.h) in fp32 against
float64, on the CPU: bf16 outputs hide its error, so the header itself is
compiled for the host, with the correctly rounded reciprocal and exponential
in the place of the hardware's (each within one unit in the last place).

Bounds.  The CDF must be as good as the form 0.5 (1 + erf) with the library
erff, which measures 7.4e-8 .. 8.0e-8 on the device over |x| <= 2 .. 6 (1 + erf
rounds by up to 2^-24, erf is off by about 1.5 x 2^-24; half of both): 1.25 x
2^-24 = 7.45e-8.  The derivative adds x times the density (at most 0.25,
near x = 1) with four roundings of 2^-24 of it (two factors, the exponential, and
the exponent's two of x^2 / 2 = 0.5 each), another 2^-24, and one rounding of a sum
up to 1.13, a third.  Over the activations of a network, |x| <= 0.5 .. 3, the
2-norm error of gelu and its derivative is at most 4.1e-8, the library erff
form's own.  The negative tail keeps its relative accuracy where 1 + erf
cancels: the fit's 4e-7 and a few units of 2^-24, plus the rounding of the
exponent x^2 / 2 log2 e (two roundings of up to 2^-24 of it, at |x| = 10 2 x 50 x
2^-24 = 6e-6)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
from scipy.special import erfc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cmath>
#define __builtin_amdgcn_rcpf(x) (float)(1.0 / (double)(x))
#define __builtin_amdgcn_exp2f(x) (float)std::exp2((double)(x))
#include "pf_gelu.h"
extern "C" void eval(int n, const float *x, float *cdf, float *g, float *d) {
  for (int i = 0; i < n; ++i) {
    float e;
    cdf[i] = pf::normal_cdf(x[i], e);
    g[i] = pf::gelu_fast(x[i]);
    d[i] = pf::gelu_grad_fast(x[i]);
  }
}
"""


@pytest.fixture(scope="module")
def gelu(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("needs g++ and the HIP headers")
    d = tmp_path_factory.mktemp("gelu")
    src, lib = str(d / "gelu.cpp"), str(d / "gelu.so")
    with open(src, "w") as f:
        f.write(SRC)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-w",
                        "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "paper_2112_00029_amd", "csrc"), src, "-o", lib],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    f = ctypes.CDLL(lib).eval

    def run(x):
        x = np.ascontiguousarray(x, np.float32)
        out = [np.empty_like(x) for _ in range(3)]
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        f(ctypes.c_int(x.size), p(x), *map(p, out))
        x = x.astype(np.float64)
        with np.errstate(all="ignore"):
            cdf = 0.5 * erfc(-x / np.sqrt(2))
            ref = (cdf, x * cdf, cdf + x * np.exp(-0.5 * x * x) / np.sqrt(2 * np.pi))
        return [(a.astype(np.float64), b) for a, b in zip(out, ref)]
    return run


@pytest.mark.parametrize("lim", [0.5, 1.0, 2.0, 3.0, 6.0])
def test_errors_are_those_of_the_erf_form(gelu, lim):
    (cdf, c), (g, gr), (d, dr) = gelu(np.linspace(-lim, lim, 400001))
    assert np.abs(cdf - c).max() <= 1.25 * 2.0 ** -24
    assert np.abs(d - dr).max() <= 3 * 2.0 ** -24
    for got, ref in ((g, gr), (d, dr)):
        assert np.linalg.norm(got - ref) <= 4.1e-8 * np.linalg.norm(ref)


def test_negative_tail_keeps_its_relative_accuracy(gelu):
    x = np.linspace(-10, -1.25, 400001)
    (cdf, c), _g, _d = gelu(x)
    # The fit; 1 / (1 + p |x|), products and sums that matter, the exponential.
    bound = 4.2e-7 + 6 * 2.0 ** -24 + 2 * (x * x / 2 * np.log2(np.e)) * np.log(2) * 2.0 ** -24
    i = int(np.argmax(np.abs(cdf - c) / c - bound))
    assert (np.abs(cdf - c) <= bound * c).all(), (x[i], abs(cdf[i] - c[i]) / c[i], bound[i])


def test_branch_points_and_specials(gelu):
    """Both sides of |x| = 1.25, where the form changes, zeros and overflow."""
    e = np.float32(1.25)
    x = np.array([np.nextafter(e, 0), e, np.nextafter(e, 2), -np.nextafter(e, 0), -e,
                  -np.nextafter(e, 2), 0.0, -0.0, 30.0, -30.0, 1e20, -1e20, 3e38, -3e38], np.float32)
    (cdf, c), (g, gr), (d, dr) = gelu(x)
    assert np.abs(cdf - c).max() <= 1.25 * 2.0 ** -24
    assert np.abs(d - dr).max() <= 3 * 2.0 ** -24
    assert (np.abs(g - gr) <= 1.25 * 2.0 ** -24 * np.minimum(np.abs(x), 2) + 2.0 ** -24 * np.abs(gr)
            + 2.0 ** -126).all()  # (a tail below 2^-126 flushes)
    assert all(np.isnan(v[0]).all() for v in gelu(np.array([np.nan])))
