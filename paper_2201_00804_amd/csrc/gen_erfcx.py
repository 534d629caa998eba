"""Writes erfcx_fit.h: Chebyshev fits of the scaled complementary error
function erfcx(x) = exp(x^2) erfc(x) on 0 <= x <= XMAX, used by the pair
kernels as erfc(x) = exp(-x^2) erfcx(x) with the exp(-x^2) the Ewald
recursion computes anyway.

The variable is t = 1 / (1 + P x) mapped to u in [-1, 1]; the series is a
least-squares fit in relative error at Chebyshev nodes of u, against
scipy.special.erfcx.  Beyond XMAX the kernels clamp x (erfc(6) = 2e-17, so
the clamped value is off by a relative factor below x / XMAX on numbers
under 2e-17).  The FP64 series is also written as powers of u, and with it
the polynomial q of exp(r) = 1 + r + r^2 q(r), |r| <= ln(2) / 2, fitted the
same way to the sum of r^k / (k + 2)!.

    python paper_2201_00804_amd/csrc/gen_erfcx.py   # rewrites erfcx_fit.h
"""
import os

import numpy as np
from numpy.polynomial import chebyshev as C
from scipy.special import erfcx, factorial

XMAX = 6.0
FITS = {"double": (16, 0.2), "float": (8, 0.8)}   # degree, P
EXP_DEG = 9
HERE = os.path.dirname(os.path.abspath(__file__))


def fit(deg, p, npts=6000):
    t0 = 1.0 / (1.0 + p * XMAX)
    k = np.arange(npts)
    u = np.cos(np.pi * (k + 0.5) / npts)
    t = t0 + (1.0 - t0) * 0.5 * (u + 1.0)
    y = erfcx((1.0 / t - 1.0) / p)
    c, *_ = np.linalg.lstsq(C.chebvander(u, deg) / y[:, None], np.ones_like(y), rcond=None)
    xs = np.linspace(0.0, XMAX, 400001)
    ts = 1.0 / (1.0 + p * xs)
    rel = np.abs(C.chebval(2.0 * (ts - t0) / (1.0 - t0) - 1.0, c) / erfcx(xs) - 1.0)
    return t0, c, float(rel.max())


def fit_exp(deg, npts=6000):
    h = 0.5 * np.log(2.0)
    k = np.arange(npts)
    u = np.cos(np.pi * (k + 0.5) / npts)
    y = sum((h * u) ** m / factorial(m + 2) for m in range(20))
    c = C.cheb2poly(C.chebfit(u, y, deg)) / h ** np.arange(deg + 1)
    r = (h * np.linspace(-1.0, 1.0, 200001)).astype(np.longdouble)
    q = sum(np.longdouble(v) * r ** m for m, v in enumerate(c))
    return c, float(np.abs((1 + r + r * r * q) / np.exp(r) - 1).max())


def array(name, c):
    return [f"constexpr double {name}[{len(c)}] = {{"] + [f"    {float(v)!r}," for v in c] + \
        ["};", ""]


def main():
    lines = ["// Generated by gen_erfcx.py: Chebyshev series of erfcx(x) = exp(x^2) erfc(x)",
             f"// on 0 <= x <= {XMAX} in u = 2 (t - t0) / (1 - t0) - 1, t = 1 / (1 + p x).",
             "#pragma once", "", "namespace sibfa {", "",
             f"constexpr double kErfcxMax = {XMAX!r};", ""]
    for ty, (deg, p) in FITS.items():
        t0, c, err = fit(deg, p)
        sfx = "f" if ty == "float" else ""
        name = "F32" if ty == "float" else "F64"
        lines += [f"// largest relative error of the fit on [0, {XMAX}]: {err:.2e}",
                  f"constexpr int kErfcxDeg{name} = {deg};",
                  f"constexpr {ty} kErfcxP{name} = {p!r}{sfx};",
                  f"constexpr {ty} kErfcxT0{name} = {float(t0)!r}{sfx};",
                  f"constexpr {ty} kErfcxC{name}[{deg + 1}] = {{"]
        lines += [f"    {float(v)!r}{sfx}," for v in c]
        lines += ["};", ""]
        print(f"{ty}: degree {deg}, p {p}, max relative error {err:.2e}")
        if name == "F64":
            lines += ["// the same series as powers of u"] + array("kErfcxMF64", C.cheb2poly(c))
    c, err = fit_exp(EXP_DEG)
    lines += ["// exp(r) = 1 + r + r^2 q(r), |r| <= ln(2) / 2: powers of r of q;",
              f"// largest relative error {err:.1e}",
              f"constexpr int kExpDeg = {EXP_DEG};"] + array("kExpQ", c)
    lines += ["}  // namespace sibfa", ""]
    with open(os.path.join(HERE, "erfcx_fit.h"), "w") as f:
        f.write("\n".join(lines))


if __name__ == "__main__":
    main()
