"""Writes hair_fastmath_coef.h: polynomial coefficients of the shading kernels' arcsine and
arctangent and hyperbolic tangent, and the 8-point Gauss-Legendre rule with the refraction
constants of its nodes.

    python paper_2405_10565_amd/csrc/gen_fastmath.py [--check]

Fits (float64, Lawson's iteratively reweighted least squares toward the minimax fit, on
Chebyshev nodes):
  asin(z) = z + z^3 P(z^2)     z in [0, 1/2], P of degree 4, relative error of asin < 1e-8
  asin(z) = z + z^3 W(z^2)     z in [0, 0.68], W of degree 7, relative error of asin < 1e-8
  atan(a) = a Q(a^2)           a in [0, 1],   Q of degree 8, absolute error < 1e-8
                               (written as Q / 2 and as Q / 2 pi: half the angle, and turns)
  tanh(x) = x + x^3 H(x^2)     x in [0, 5/8], H of degree 4, relative error of tanh < 1e-8
The kernels reduce |x| > 1/2 by asin(x) = pi/2 - 2 asin(sqrt((1 - x) / 2)) and atan2 to
[0, 1] by octant symmetry.  --check only verifies that the header on disk is current.
"""
from __future__ import annotations

import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "hair_fastmath_coef.h")


def lawson(f, lo, hi, deg, weight, iters=60, n=4000):
    """Weighted minimax polynomial fit by Lawson's algorithm; returns (coefficients, max error)."""
    x = lo + (hi - lo) * (1 - np.cos(np.pi * (np.arange(n) + 0.5) / n)) / 2
    y, w = f(x), weight(x)
    V = np.vander(x, deg + 1, increasing=True)
    lw = np.full(n, 1.0 / n)
    for _ in range(iters):
        sw = np.sqrt(lw) * w
        c, *_ = np.linalg.lstsq(V * sw[:, None], y * sw, rcond=None)
        e = np.abs(V @ c - y) * w
        lw = lw * e
        lw /= lw.sum()
    return c, float((np.abs(V @ c - y) * w).max())


def coefficients():
    p, ep = lawson(lambda t: (np.arcsin(np.sqrt(t)) - np.sqrt(t)) / t ** 1.5, 1e-12, 0.25, 4, lambda t: t)
    q, eq = lawson(lambda t: np.arctan(np.sqrt(t)) / np.sqrt(t), 1e-12, 1.0, 8, np.sqrt)
    aw, eaw = lawson(lambda t: (np.arcsin(np.sqrt(t)) - np.sqrt(t)) / t ** 1.5, 1e-12, 0.68 ** 2, 7, lambda t: t)
    h, eh = lawson(lambda t: (np.tanh(np.sqrt(t)) - np.sqrt(t)) / t ** 1.5, 1e-12, 0.625 ** 2, 4, lambda t: t)
    x, w = (v[4:] for v in np.polynomial.legendre.leggauss(8))
    return {"asin_p": p, "asin_err": ep, "atan_q": q, "atan_err": eq, "asin_w": aw, "asin_w_err": eaw,
            "tanh_h": h, "tanh_err": eh, "gl_x": x, "gl_w": w,
            "gl_gamma_o": np.arcsin(x), "gl_cos_gamma_o": np.sqrt((1 - x) * (1 + x))}


def fmt(v, suffix="f"):
    return ", ".join(f"{float(c):.17g}{suffix}" for c in v)


def render() -> str:
    c = coefficients()
    return f"""// Generated by gen_fastmath.py (same folder); do not edit by hand.
#pragma once

namespace hair {{

// asin(z) = z + z^3 P(z^2) on [0, 1/2]; P ascending, relative error {c['asin_err']:.1e}
constexpr float kAsinP[5] = {{{fmt(c['asin_p'])}}};
// atan(a) = a Q(a^2) on [0, 1]; Q ascending, absolute error {c['atan_err']:.1e}; as Q / 2 and Q / 2 pi
constexpr float kAtanHalfQ[9] = {{{fmt(c['atan_q'] / 2)}}};
constexpr float kAtanTurnsQ[9] = {{{fmt(c['atan_q'] / (2 * np.pi))}}};
// asin(z) = z + z^3 W(z^2) on [0, 0.68]; W ascending, relative error {c['asin_w_err']:.1e}
constexpr float kAsinW[8] = {{{fmt(c['asin_w'])}}};
// tanh(x) = x + x^3 H(x^2) on [0, 5/8]; H ascending, relative error {c['tanh_err']:.1e}
constexpr float kTanhH[5] = {{{fmt(c['tanh_h'])}}};

// 8-point Gauss-Legendre rule on [-1, 1]: its nodes h_k > 0 (the rule is symmetric), weights, and at
// each node the incidence angle gamma_o = asin(h_k) and cos(gamma_o) = sqrt(1 - h_k^2).
constexpr float kGLx[4] = {{{fmt(c['gl_x'])}}};
constexpr float kGLw[4] = {{{fmt(c['gl_w'])}}};
constexpr double kGLgo[4] = {{{fmt(c['gl_gamma_o'], '')}}};
constexpr float kGLcgo[4] = {{{fmt(c['gl_cos_gamma_o'])}}};

}}  // namespace hair
"""


def main():
    text = render()
    if "--check" in sys.argv:
        cur = open(OUT).read() if os.path.exists(OUT) else ""
        if cur != text:
            print("hair_fastmath_coef.h is out of date; run gen_fastmath.py")
            sys.exit(1)
        return
    with open(OUT, "w") as f:
        f.write(text)
    print(OUT)


if __name__ == "__main__":
    main()
