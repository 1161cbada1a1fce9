"""The short smoothing of the symmetric passes loses no accuracy.

near_factors_sym forms s_1 .. s_4 with fewer operations than near_factors (the
one-direction passes): weighted erfc fit, e^y of 12 terms, folded constants.
Both are emulated here operation by operation, fma by fma, in double against 60
digits; the expressions of the short form are read from csrc/pair_kernels.hip.
Bars: over the whole range and over each part of it the root mean square error
within 1.1 of the former's, over the whole range the largest within 1.25 (the
largest of a few thousand rounding errors scatters by about that much).
"""
import math
import os
import re

import mpmath as mp
import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_10749_amd", "csrc")
with open(os.path.join(CSRC, "smoothing_coeffs.h")) as f:
    HEADER = f.read()
with open(os.path.join(CSRC, "pair_kernels.hip")) as f:
    KERNELS = f.read()
SYM = KERNELS[KERNELS.index("void near_factors_sym("):KERNELS.index("void near_factors_n(")]


def table(name, text=HEADER):
    body = re.search(name + r"\[\d+\] = \{([^}]*)\}", text).group(1)
    return [float(eval(v.strip())) for v in body.split(",")]  # numbers and quotients of numbers


def define(name):
    return float(re.search(rf"#define {name} ([0-9.]+)", HEADER).group(1))


def expression(pattern):
    """The C expression that the pattern's group matches in near_factors_sym, for eval()."""
    text = " ".join(re.search(pattern, SYM, re.S).group(1).split()).replace("[u]", "")
    return compile(text, text, "eval")


def fma(a, b, c):
    return float(mp.mpf(a) * mp.mpf(b) + mp.mpf(c))  # exact in 300 bits, rounded once


def horner(c, x):
    a = c[-1]
    for v in reversed(c[:-1]):
        a = fma(a, x, v)
    return a


def hardware_rcp(v):
    return float(np.float32(1.0 / v))  # v_rcp_f64 is good to about a float


LOG2E, LN2, LN2_LO = 1.44269504088896340736, 0.693147180559945309417, 2.319046813846299558e-17
C = 1.128379167095512573896  # 2 / sqrt(pi)
TABS = {"taylor": table("kExpTaylor", KERNELS), "erfcx": table("kERFCX_F64"), "exp": table("kEXP_F64"),
        "erfcw": table("kERFCXW_F64"), "p": define("SDBIE_ERFCX_P"), "pw": define("SDBIE_ERFCXW_P")}
Y = expression(r"y\[u\] = (fma\(n\[u\], kLn2, .*?);")
Y_LOW = expression(r"if \(K3 \|\| K4\) y\[u\] = (.*?);") if "kLn2Lo" in SYM else None
PREFACTORS = {m[0]: expression(rf"{m[0]} = (kTwoOverSqrtPi[^,;]*)[,;]")
              for m in re.findall(r"(\w+) = (kTwoOverSqrtPi[^,;]*)", SYM)}
FACTORS = [expression(rf"k{k}\[u\] \*=\s*c \? (.*?) : 1\.0;") for k in (1, 2, 3, 4)]


def former(rho):
    """near_factors, the closed forms"""
    x = rho * rho
    n = float(np.rint(x * LOG2E))
    r = fma(-n, LN2_LO, fma(-n, LN2, x))
    e = math.ldexp(horner(TABS["taylor"], -r), -int(n))
    v = fma(TABS["p"], rho, 1.0)
    t = hardware_rcp(v)
    for _ in range(2):
        t = fma(fma(-v, t, 1.0), t, t)
    ef = fma(-e, horner(TABS["erfcx"], t), 1.0)
    ce = C * rho * e
    third = ce * (1.0 / 3.0)
    return (fma(-third, fma(2.0, x, -5.0), ef), fma(third, fma(2.0, x, -3.0), ef),
            fma(-third, fma(fma(4.0, x, -14.0), x, 3.0), ef),
            fma(-(ce * (1.0 / 9.0)), fma(fma(fma(8.0, x, -36.0), x, 6.0), x, 9.0), ef))


def short(rho):
    """near_factors_sym, the closed forms"""
    x = rho * rho
    names = {"fma": fma, "x": x, "n": float(np.rint(x * LOG2E)), "kLn2": LN2, "kLn2Lo": LN2_LO, "kTwoOverSqrtPi": C,
             "rho": rho}
    v = fma(TABS["pw"], rho, 1.0)
    h = hardware_rcp(v)
    d = fma(-v, h, 1.0)
    t = fma(h, fma(d, d, d), h)
    names["y"] = eval(Y, names)
    out = []
    for k in (1, 2, 3, 4):
        if k == 3 and Y_LOW:
            names["y"] = eval(Y_LOW, names)
        e = names["e"] = math.ldexp(horner(TABS["exp"], names["y"]), -int(names["n"]))
        names["ef"] = fma(-e, horner(TABS["erfcw"], t), 1.0)
        for name, value in PREFACTORS.items():
            names[name] = eval(value, names)
        out.append(eval(FACTORS[k - 1], names))
    return out


def exact(rho):
    r = mp.mpf(rho)
    x = r * r
    ef, ce = mp.erf(r), 2 / mp.sqrt(mp.pi) * r * mp.exp(-x)
    return (ef - ce * (2 * x - 5) / 3, ef + ce * (2 * x - 3) / 3, ef - ce * ((4 * x - 14) * x + 3) / 3,
            ef - ce * (((8 * x - 36) * x + 6) * x + 9) / 9)


def smoothing_errors(rhos):
    err = np.empty((2, 4, len(rhos)))
    with mp.workprec(300):
        for i, rho in enumerate(rhos):
            ref = exact(rho)
            for f, form in enumerate((former, short)):
                for k, v in enumerate(form(rho)):
                    err[f, k, i] = float((mp.mpf(v) - ref[k]) / ref[k])
    return np.abs(err)


def test_short_smoothing_is_as_accurate_as_the_closed_forms():
    rng = np.random.default_rng(11)
    rhos = np.concatenate([rng.uniform(0.5, 1.2, 1500), rng.uniform(0.5, 7.1, 1500)])
    parts = {"all": rhos}
    for lo, hi in ((0.5, 0.8), (0.8, 1.2), (1.2, 1.8), (1.8, 2.5), (2.5, 7.1)):
        parts[f"{lo} .. {hi}"] = rng.uniform(lo, hi, 1000)
    bad = []
    for name, r in parts.items():
        err = smoothing_errors([float(v) for v in r])
        for k in range(4):
            (a, b), (ra, rb) = err[:, k].max(axis=1), np.sqrt((err[:, k] ** 2).mean(axis=1))
            print(f"{name}: s_{k + 1} largest {a:.2e} -> {b:.2e}, rms {ra:.2e} -> {rb:.2e} ({rb / ra:.3f})")
            if not (rb < 1.1 * ra and (name != "all" or b < 1.25 * a)):
                bad.append((name, k + 1))
    assert not bad
