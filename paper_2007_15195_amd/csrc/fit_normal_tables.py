"""Write normal_tables.h and normal_tables_f32.h next to this file. normal_tables.h: node values of the normal quantile
and CDF for the FP64 loops (device_nodes_f64.h), computed in 40-digit
arithmetic (mpmath).

Quantile nodes: q in [2^-15, 1/2] is cut into octaves of 128 equal cells; the
node of a cell is its midpoint q_i, and holds z_i = -Phi^{-1}(q_i) and
1 / phi(z_i). One more cell holds q = 1/2 exactly (the first of the octave
above). CDF nodes: a_i = i / 128, i = -1088 .. 1088 (|a| <= 8.5), each holding
Phi(a_i) and phi(a_i).

normal_tables_f32.h, for the FP32 loop (qmc_f32.h): the quantile
z = -Phi^{-1}(q) on q in [2^-15, 1/2] as one quadratic per cell of 32 per
octave, (c0, c1, c2, midpoint), minimax in absolute error, each coefficient
rounded to FP32 before the lower ones are fitted; and the coefficients of
log2 Phi(-v / kappa), v in [0, 4.7], kappa = sqrt(log2(e) / 2), a polynomial of
degree 8 by Lawson's reweighted least squares: relative error of Phi up to
v = 3.41 (Phi = 2^-15, below which the loop takes the ratio instead), absolute
beyond. Its leading coefficient is negative, so
2^poly falls to 0 beyond the fitted range.

Run: python fit_normal_tables.py   (development-time only; the header is committed)
"""
from __future__ import annotations

import os

import mpmath
import numpy as np

mpmath.mp.dps = 40

OCTAVES, PER_OCTAVE = 14, 128
PER_UNIT, A_MAX = 128, 8.5


def quantile(q):
    """-Phi^{-1}(q), q in (0, 1/2 + 2^-8)."""
    return mpmath.sqrt(2) * mpmath.erfinv(1 - 2 * mpmath.mpf(q))


def pairs():
    for o in range(-1 - OCTAVES, 0):
        for j in range(PER_OCTAVE if o < -1 else 1):
            z = quantile(mpmath.mpf(2) ** o * (1 + (mpmath.mpf(j) + mpmath.mpf(1) / 2) / PER_OCTAVE))
            yield z, 1 / mpmath.npdf(z)
    n = int(A_MAX * PER_UNIT)
    for i in range(-n, n + 1):
        a = mpmath.mpf(i) / PER_UNIT
        yield mpmath.ncdf(a), mpmath.npdf(a)


def main():
    rows = [f"{float(a)!r}, {float(b)!r}," for a, b in pairs()]
    nq = OCTAVES * PER_OCTAVE + 1
    out = ["// Generated by fit_normal_tables.py; do not edit.",
           "// Nodes of the normal quantile (-Phi^{-1}(q_i), 1 / phi) and, after them, of the CDF (Phi(a_i), phi(a_i)).",
           "#pragma once", "", "namespace vecchia {", "",
           f"constexpr int kNinvNodes = {nq};",
           f"constexpr int kPhiNodes = {len(rows) - nq};",
           f"constexpr int kPhiMid = {(len(rows) - nq) // 2};   // the node of a = 0",
           "constexpr int kNormNodes = kNinvNodes + kPhiNodes;", "",
           "#if defined(__HIPCC__)", "static __device__", "#else", "static", "#endif",
           "const double kNormNodeTable[2 * kNormNodes] = {"]
    for k in range(0, len(rows), 2):
        out.append("    " + " ".join(rows[k:k + 2]))
    out += ["};", "", "}  // namespace vecchia", ""]
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "normal_tables.h")
    with open(path, "w") as f:
        f.write("\n".join(out))


OCTAVES32, PER_OCTAVE32 = 14, 32
KAPPA = mpmath.sqrt(1 / (2 * mpmath.log(2)))


def minimax(A, f, w, iters=40):
    """Lawson's reweighted least squares of A c = f in the weighted maximum norm."""
    W = w.copy()
    for _ in range(iters):
        c = np.linalg.lstsq(A * W[:, None], f * W, rcond=None)[0]
        e = np.abs(A @ c - f) * w
        W = W * np.maximum(e / e.max(), 1e-3) ** 0.3
        W /= W.max()
    return c


def rounded(cols, f, w):
    """Coefficients of the columns (highest power first), each rounded to FP32 before the rest are fitted."""
    out, rest = [], f.copy()
    for k in range(len(cols)):
        c = np.float32(minimax(np.stack(cols[k:], axis=1), rest, w)[0])
        out.append(c)
        rest = rest - float(c) * cols[k]
    return out


def cells32():
    for o in range(-1 - OCTAVES32, 0):
        for j in range(PER_OCTAVE32 if o < -1 else 1):
            lo, hi = 2.0 ** o * (1 + j / PER_OCTAVE32), 2.0 ** o * (1 + (j + 1) / PER_OCTAVE32)
            mid = (lo + hi) / 2
            d = np.cos((2 * np.arange(15) + 1) * np.pi / 30) * (hi - lo) / 2
            z = np.array([float(quantile(mpmath.mpf(float(mid + v)))) for v in d])
            c2, c1, c0 = rounded([d * d, d, np.ones_like(d)], z, np.ones_like(d))
            yield c0, c1, c2, np.float32(mid)


def tail_poly(n=8, vmax=4.7, vfull=3.41):
    v = (1 - np.cos(np.linspace(0, np.pi, 1201))) / 2 * vmax
    g = np.array([float(mpmath.log(mpmath.ncdf(-mpmath.mpf(float(x)) / KAPPA), 2)) for x in v])
    w = np.maximum(np.minimum(1.0, 2.0 ** (g - np.interp(vfull, v, g))), 1e-9)
    c = minimax(np.vander(v, n + 1, increasing=True), g, w, 80)
    assert c[n] < 0
    return [np.float32(x) for x in c]


def main32():
    hexf = lambda x: float(x).hex() + "f"
    rows = ["{" + ", ".join(hexf(x) for x in r) + "}," for r in cells32()]
    out = ["// Generated by fit_normal_tables.py; do not edit.",
           "// FP32 quantile cells (c0, c1, c2, midpoint) and log2 Phi(-v / kappa) (increasing powers).",
           "#pragma once", "", "namespace vecchia {", "",
           f"constexpr int kQuantCells = {len(rows)};",
           "static __device__ const float kQuantTable[kQuantCells][4] = {"]
    out += ["    " + r for r in rows] + ["};"]
    c = tail_poly()
    out += [f"constexpr float kTailPoly[{len(c)}] = {{" + ", ".join(hexf(x) for x in c) + "};", "", "}  // namespace vecchia", ""]
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "normal_tables_f32.h"), "w") as f:
        f.write("\n".join(out))


if __name__ == "__main__":
    main()
    main32()
