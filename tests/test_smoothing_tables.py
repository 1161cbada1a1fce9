"""The fitted tables of the double near field hold their stated errors.

csrc/smoothing_coeffs.h states an error bound with each fit; it has to hold for
the table as stored, evaluated by Horner's rule in double (grids other than the
generator's: within 1.5 times the stated maximum).
"""
import math
import os
import re

import mpmath as mp
import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_10749_amd", "csrc")
with open(os.path.join(CSRC, "smoothing_coeffs.h")) as f:
    HEADER = f.read()


def table(name):
    body = re.search(name + r"\[\d+\] = \{([^}]*)\}", HEADER).group(1)
    return [float(v) for v in body.split(",")]


def define(name):
    return float(re.search(rf"#define {name} ([0-9.]+)", HEADER).group(1))


def stated(pattern):
    return float(re.search(pattern, HEADER).group(1))


def horner(c, x):
    a = np.full_like(x, c[-1])
    for v in reversed(c[:-1]):
        a = a * x + v
    return a


def test_the_stated_errors_hold_for_the_stored_tables():
    rng = np.random.default_rng(7)
    rho = np.concatenate([np.linspace(0.49, 7.19, 2111), rng.uniform(0.49, 7.2, 2000)])
    bound = stated(r"double, max rel\. error ([0-9.e-]+)\)")
    t = 1.0 / (1.0 + define("SDBIE_ERFCX_P") * rho)
    g = horner(table("kERFCX_F64"), t)
    with mp.workdps(40):
        e = max(abs(mp.mpf(float(a)) / (mp.erfc(mp.mpf(float(r))) * mp.exp(mp.mpf(float(r)) ** 2)) - 1)
                for a, r in zip(g, rho))
    print(f"erfcx: {float(e):.2e}, stated {bound:.1e}")
    assert e < 1.5 * bound

    bound = stated(r"kERFCXW_F64\[j\] t\^j is erfc\(rho\) to ([0-9.e-]+) \(absolute")
    t = 1.0 / (1.0 + define("SDBIE_ERFCXW_P") * rho)
    g = horner(table("kERFCXW_F64"), t)
    with mp.workdps(40):
        e = max(abs(mp.mpf(float(a)) * mp.exp(-mp.mpf(float(r)) ** 2) - mp.erfc(mp.mpf(float(r))))
                for a, r in zip(g, rho))
    print(f"weighted erfc: {float(e):.2e}, stated {bound:.1e}")
    assert e < 1.5 * bound

    bound = stated(r"e\^y on \|y\| <= ln\(2\)/2 to ([0-9.e-]+) \(relative")
    h = 0.5 * math.log(2.0)
    y = np.concatenate([np.linspace(-h, h, 2111), rng.uniform(-h, h, 2000)])
    a = horner(table("kEXP_F64"), y)
    with mp.workdps(40):
        e = max(abs(mp.mpf(float(v)) / mp.exp(mp.mpf(float(u))) - 1) for v, u in zip(a, y))
    print(f"exp: {float(e):.2e}, stated {bound:.1e}")
    assert e < 1.5 * bound
