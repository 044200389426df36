"""Fit the rational approximations used by the FP32 SOV loop and write
fp32_math_coeffs.h next to this file.

Two functions are approximated by ratios of polynomials:

  R = Phi(-a) exp(a^2/2) = erfcx(a / sqrt 2) / 2 as a function of v = kappa a,
      kappa = sqrt(log2(e) / 2), for a in [0, 40]; degree (4, 5), positive
      coefficients (the ratio decays like 1/(a sqrt(2 pi)) as the true R does).
      With v in hand, exp(-a^2/2) = 2^(-v^2), so the loop scales its rows by
      kappa once and never multiplies a^2 by log2(e)/2.
  z = -Phi^{-1}(q) for q in (0, 1/2] as a function of s = sqrt(-log2 q) in
      [1, 34] (s = 1 at q = 1/2; sqrt(-2 log q) = sqrt(2 log 2) s); degree (5, 4).
  The same z for s in [34, 1100], degree (3, 2): the loop's split path, whose
      log2 q carries an exponent kept outside the FP32 number (down to -2^20),
      uses it beyond s = 34 (relative error weights).

The fit is Lawson's iteratively reweighted least squares on the linearised
problem P(x) - f(x) Q(x) = 0 (a standard route to near-minimax rational
approximations), with relative error weights for R and absolute error for z.
Targets come from scipy.special.erfcx and from a high-precision Newton solve
of log Phi(-z) = -s^2/2 with mpmath.

Run: python fit_fp32_math.py   (development-time only; the header is committed)
"""
from __future__ import annotations

import os

import mpmath
import numpy as np
from scipy.special import erfcx

S0 = float(np.sqrt(2.0 * np.log(2.0)))      # s at q = 1/2


def z_of_s(s: float) -> float:
    mpmath.mp.dps = 40
    s = mpmath.mpf(s)
    target = -s * s / 2
    if s > 3:
        z = s - mpmath.log(2 * mpmath.pi * s * s) / (2 * s)
    else:
        z = mpmath.sqrt(2) * mpmath.erfinv(1 - 2 * mpmath.exp(target))
    for _ in range(60):
        f = mpmath.log(mpmath.ncdf(-z)) - target
        fp = -mpmath.npdf(z) / mpmath.ncdf(-z)
        dz = f / fp
        z -= dz
        if abs(dz) < mpmath.mpf(10) ** -30:
            break
    return float(z)


def lawson(x, y, n, m, weight, iters=80):
    V = np.vander(x, max(n, m) + 1, increasing=True)
    w = np.ones_like(x) / len(x)
    best = None
    for _ in range(iters):
        A = np.hstack([V[:, :n + 1], -y[:, None] * V[:, 1:m + 1]])
        sw = np.sqrt(w) * weight
        c, *_ = np.linalg.lstsq(A * sw[:, None], y * sw, rcond=None)
        p = c[:n + 1]
        q = np.concatenate([[1.0], c[n + 1:]])
        err = (V[:, :n + 1] @ p / (V[:, :m + 1] @ q) - y) * weight
        e = float(np.max(np.abs(err)))
        if best is None or e < best[0]:
            best = (e, p, q)
        w = np.maximum(w * np.abs(err) / np.sum(w * np.abs(err)), 1e-15)
    return best


def eval_f32(p, q, x):
    x32 = np.asarray(x, dtype=np.float32)
    P = np.zeros_like(x32)
    Q = np.zeros_like(x32)
    for c in np.asarray(p, dtype=np.float32)[::-1]:
        P = P * x32 + c
    for c in np.asarray(q, dtype=np.float32)[::-1]:
        Q = Q * x32 + c
    return (P / Q).astype(np.float64)


def main():
    here = os.path.dirname(os.path.abspath(__file__))
    mpmath.mp.dps = 40
    kappa = float(mpmath.sqrt(1 / (2 * mpmath.log(2))))
    a = np.concatenate([np.linspace(0, 6, 1500), np.linspace(6, 40, 800)])
    ra = 0.5 * erfcx(a / np.sqrt(2.0))
    eR, pR, qR = lawson(kappa * a, ra, 4, 5, 1.0 / ra, iters=300)
    aa = np.linspace(0, 40, 200001)
    rr = 0.5 * erfcx(aa / np.sqrt(2.0))
    eR32 = float(np.max(np.abs(eval_f32(pR, qR, np.float32(kappa) * aa) - rr) / rr))

    s = np.concatenate([np.linspace(S0, 4, 400), np.linspace(4, 40, 400)])
    z = np.array([z_of_s(v) for v in s])
    x = s / S0
    eZ, pZ, qZ = lawson(x, z, 5, 4, np.ones_like(s))
    eZ32 = float(np.max(np.abs(eval_f32(pZ, qZ, x) - z) / np.maximum(z, 0.05)))
    xw = np.concatenate([np.linspace(34.0, 100.0, 400), np.linspace(100.0, 1100.0, 400)])
    zw = np.array([z_of_s(v * S0) for v in xw])
    eW, pW, qW = lawson(xw, zw, 3, 2, 1.0 / zw, iters=150)
    xxw = np.linspace(34.0, 1100.0, 2000)
    eW32 = float(np.max(np.abs(eval_f32(pW, qW, xxw) - np.array([z_of_s(v * S0) for v in xxw])) /
                        np.array([z_of_s(v * S0) for v in xxw])))
    assert np.all(pR > 0) and np.all(qR > 0) and np.all(qZ > 0) and np.all(qW > 0)

    def arr(name, v):
        body = ", ".join(float(np.float32(c)).hex() + "f" for c in v)
        return f"static constexpr float {name}[{len(v)}] = {{{body}}};\n"

    with open(os.path.join(here, "fp32_math_coeffs.h"), "w") as f:
        f.write("// Generated by fit_fp32_math.py; do not edit.\n")
        f.write("// R = erfcx(a/sqrt2)/2 ~= P(v)/Q(v), v = kappa a, a in [0, 40]:"
                f" max rel err {eR:.2e} (fp64 eval), {eR32:.2e} (fp32 eval).\n")
        f.write("// z = -Phi^-1(q) ~= P(s)/Q(s), s = sqrt(-log2 q):"
                f" max abs err {eZ:.2e} (fp64), rel {eZ32:.2e} (fp32).\n")
        f.write("// z for s in [34, 1100] ~= P(s)/Q(s):"
                f" max rel err {eW:.2e} (fp64), {eW32:.2e} (fp32).\n")
        f.write("#pragma once\n")
        f.write(f"static constexpr double kPhiScale = {kappa!r};   // kappa = sqrt(log2(e) / 2)\n")
        f.write(arr("kRP", pR) + arr("kRQ", qR) + arr("kZP", pZ) + arr("kZQ", qZ))
        f.write(arr("kZPW", pW) + arr("kZQW", qW))
    print("R", eR, eR32, "z", eZ, eZ32, "z wide", eW, eW32)


if __name__ == "__main__":
    main()
