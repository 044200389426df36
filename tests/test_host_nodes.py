"""The FP64 loops' node-table normal quantile and CDF (csrc/device_nodes_f64.h), built for the host by g++, against
40-digit values (mpmath): cell and octave edges, node midpoints, the ends of both ranges. One unit of rounding in the
node, one in the result and the truncated series give 3 * 2^-53 relative; near q = 1/2, where z -> 0, 2^-58 absolute."""
import os
import shutil
import subprocess

import numpy as np
import pytest

mpmath = pytest.importorskip("mpmath")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_15195_amd", "csrc")


def _inputs(which):
    rng = np.random.default_rng(5)
    if which == "q":
        edges = np.array([2.0 ** o * (1 + j / 128) for o in range(-15, -1) for j in (0, 1, 64, 127)])
        x = np.concatenate([rng.uniform(2.0 ** -15, 0.5, 800), 2.0 ** -rng.uniform(1, 15, 800), edges,
                            np.nextafter(edges[1:], 0), [0.5, np.nextafter(0.5, 0), 2.0 ** -15]])
        return np.clip(x, 2.0 ** -15, 0.5)
    half = (np.arange(-1088, 1088) + 0.5) / 128            # farthest from a node
    return np.concatenate([rng.uniform(-8.5, 8.5, 800), rng.standard_normal(600), half[::5], [-8.5, 8.5, 0.0, 1e-300]])


@pytest.mark.parametrize("which", ["q", "c"])
def test_node_tables_against_40_digits(which, tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "nodes")
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-mfma", "-I", CSRC,
                        os.path.join(ROOT, "tests", "host_sanitize", "nodes64_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-500:]
    xs = _inputs(which)
    out = subprocess.run([exe], input="".join(f"{which} {float(x)!r}\n" for x in xs), capture_output=True, text=True,
                         timeout=120)
    got = [float(v) for v in out.stdout.split()]
    assert len(got) == len(xs)
    mpmath.mp.dps = 40
    for x, g in zip(xs, got):
        x = mpmath.mpf(float(x))
        ref = mpmath.sqrt(2) * mpmath.erfinv(1 - 2 * x) if which == "q" else mpmath.ncdf(x)
        assert abs(mpmath.mpf(g) - ref) <= 3 * mpmath.mpf(2) ** -53 * abs(ref) + (mpmath.mpf(2) ** -58 if which == "q" else 0), float(x)
