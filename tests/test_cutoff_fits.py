"""The float64 near field's fitted constants (csrc/cutoff_fits.h) against multiprecision values, at the errors that the
header states."""
import os
import re

import numpy as np
import pytest

mp = pytest.importorskip("mpmath")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TEXT = open(os.path.join(ROOT, "paper_1106_5273_amd", "csrc", "cutoff_fits.h")).read()


def _list(name):
    return [float(v) for v in re.search(name + r"\[\d+\] = \{([^}]*)\}", TEXT).group(1).split(",")]


def _num(name):
    return float(re.search(r"#define %s (\S+)" % name, TEXT).group(1))


def _horner(c, t):
    r = mp.mpf(0)
    for q in reversed(c):
        r = r * t + mp.mpf(q)
    return r


def _p(a, x):
    return mp.gammainc(mp.mpf(a), 0, x, regularized=True)


def test_series_below_the_split():
    with mp.workdps(40):
        c, top = _list("VFMM64_M2_C"), mp.mpf(_num("VFMM64_XSPLIT"))
        for i in range(1, 200):
            x = top * i / 199
            want = _p(2.5, x) * mp.exp(x) / x ** mp.mpf(2.5)
            assert abs(_horner(c, x) / want - 1) <= 6e-17
            # the sum for 3/2 from it
            assert abs((x * _horner(c, x) + 1 / mp.gamma(2.5)) / (_p(1.5, x) * mp.exp(x) / x ** mp.mpf(1.5)) - 1) <= 6e-17


def test_complement_above_the_split():
    with mp.workdps(40):
        c = _list("VFMM64_PE_C")
        lo, hi = mp.mpf(_num("VFMM64_XSPLIT")), mp.mpf(_num("VFMM64_XMAX"))
        for i in range(200):
            x = lo + (hi - lo) * i / 199
            u = 1 / mp.sqrt(x)
            pe = _horner(c, mp.mpf(_num("VFMM64_PE_SCALE")) * u + mp.mpf(_num("VFMM64_PE_SHIFT")))
            p3 = 1 - mp.exp(-x) * (u * pe + 2 / mp.sqrt(mp.pi) / u)
            assert abs(p3 / _p(1.5, x) - 1) <= 2e-17
            p5 = p3 - 4 / (3 * mp.sqrt(mp.pi)) * x ** mp.mpf(1.5) * mp.exp(-x)
            assert abs(p5 / _p(2.5, x) - 1) <= 2e-17
        assert 1 - _p(1.5, hi) < 1 - _p(2.5, hi) <= 2.0 ** -53  # 1 in double beyond


def test_two_parts_of_ln_2():
    hi, lo = _num("VFMM64_LN2_HI"), _num("VFMM64_LN2_LO")
    with mp.workdps(60):
        assert abs(mp.mpf(hi) + mp.mpf(lo) - mp.log(2)) <= mp.mpf(2) ** -92
        for n in (1, 1155, 4095):
            assert mp.mpf(n * hi) == n * mp.mpf(hi)  # exact products
    assert np.float64(hi) * 2.0 ** 40 == np.floor(np.float64(hi) * 2.0 ** 40)
