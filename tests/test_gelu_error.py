"""The GELU of the bf16 kernels' forward epilogues against 64 bits: no less accurate, anywhere, than z = a/2 (1 + erff(a / sqrt 2)) and
its derivative with an exponential of its own, the form that the fp32 kernels use.  Host build of the device function."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
from scipy.special import erf, erfc

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2501_17086_amd", "csrc")
SRC = """
#include "gelu.h"
static float step(float x, int n) { return n == 0 ? x : std::nextafterf(x, n > 0 ? HUGE_VALF : -HUGE_VALF); }
extern "C" void run(const float* a, float* z, float* dz, long n, int e, int r) {
  for (long i = 0; i < n; ++i)
    hbp::gelu_pair(a[i], z[i], dz[i], [e](float x) { return step((float)std::exp2((double)x), e); },
                   [r](float x) { return step((float)(1.0 / (double)x), r); });
}
"""
# between the places where either form changes behaviour: both tails, both sides of 5/4 and of 0
BANDS = ((-14, -6), (-6, -4), (-4, -2), (-2, -1.25), (-1.25, -1), (-1, -0.25), (-0.25, 0), (0, 0.25), (0.25, 1), (1, 1.25), (1.25, 2),
         (2, 4), (4, 14))


@pytest.fixture(scope="module")
def gelu(tmp_path_factory):
    d = tmp_path_factory.mktemp("gelu")
    (d / "gelu.cpp").write_text(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-shared", "-fPIC", f"-I{CSRC}", str(d / "gelu.cpp"), "-o",
                    str(d / "gelu.so")], check=True)
    lib = ctypes.CDLL(str(d / "gelu.so"))

    def run(a, e, r):
        z, dz = np.empty_like(a), np.empty_like(a)
        p = lambda t: t.ctypes.data_as(ctypes.c_void_p)
        lib.run(p(a), p(z), p(dz), ctypes.c_long(a.size), e, r)
        return z, dz
    return run


def _step(x, n):
    return x if n == 0 else np.nextafter(x, np.float32(np.inf if n > 0 else -np.inf))


def _erf_form(a, r, e):
    """erff and the exponential within one unit in the last place (r, e = -1, 0, 1), every operation rounded to 32 bits."""
    f = np.float32
    one = f(1) + _step(erf((a * f(0.7071067811865475)).astype(np.float64)).astype(f), r)
    ex = _step(np.exp2((f(-0.5) * a * a * f(1.4426950408889634)).astype(np.float64)).astype(f), e)
    return f(0.5) * a * one, f(0.5) * one + a * ex * f(0.3989422804014327)


def test_no_less_accurate_than_the_erf_form(gelu):
    a = np.unique(np.concatenate([np.linspace(-14, 14, 400001), np.linspace(-1.5, 1.5, 400001), np.geomspace(1e-6, 14, 40001),
                                  -np.geomspace(1e-6, 14, 40001)]).astype(np.float32))
    a = a[a != 0]
    x = a.astype(np.float64)
    phi = 0.5 * erfc(-x / np.sqrt(2))
    z, dz = x * phi, phi + x * np.exp(-0.5 * x * x) / np.sqrt(2 * np.pi)

    def errors(got):
        ez, ed = np.abs(got[0] - z), np.abs(got[1] - dz)
        return [(ez[m].max(), (ez[m] / np.abs(z[m])).max(), ed[m].max()) for lo, hi in BANDS for m in [(a >= lo) & (a < hi)]]

    worst = lambda runs: np.max([errors(r) for r in runs], axis=0)
    got = worst([gelu(a, e, r) for e in (-1, 0, 1) for r in (-1, 0, 1)])
    bound = worst([_erf_form(a, r, e) for r in (-1, 0, 1) for e in (-1, 0, 1)])
    assert (got <= bound).all(), list(zip(BANDS, got, bound))


def test_ends_of_the_range(gelu):
    a = np.array([0.0, -0.0, 20.0, -20.0, 1e20, np.inf, np.nan], np.float32)
    z, dz = gelu(a, 0, 0)
    assert np.array_equal(z[:3], [0, 0, 20]) and np.array_equal(dz[:3], [0.5, 0.5, 1])
    assert abs(z[3]) < 1e-37 and abs(dz[3]) < 1e-37
    assert z[4] == a[4] and dz[4] == 1 and z[5] == np.inf and np.isnan(z[6]) and np.isnan(dz[6])
