"""Write normal_tables.h next to this file: node values of the normal quantile
and CDF for the FP64 loops (device_nodes_f64.h), computed in 40-digit
arithmetic (mpmath).

Quantile nodes: q in [2^-15, 1/2] is cut into octaves of 128 equal cells; the
node of a cell is its midpoint q_i, and holds z_i = -Phi^{-1}(q_i) and
1 / phi(z_i). One more cell holds q = 1/2 exactly (the first of the octave
above). CDF nodes: a_i = i / 128, i = -1088 .. 1088 (|a| <= 8.5), each holding
Phi(a_i) and phi(a_i).

Run: python fit_normal_tables.py   (development-time only; the header is committed)
"""
from __future__ import annotations

import os

import mpmath

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


if __name__ == "__main__":
    main()
