"""The FP32 loop's own functions through the test hooks, elementwise against SciPy: the inner factors' tail 2^p(|v|), the
rare path's factor and quantile, the table's quantile, and arguments far beyond any ratio's fitted range (a nearly
singular block scales a limit by up to 1e8).

Bounds: the tail is held to the ratio's (2e-6 relative plus the exponent's FP32 rounding twice), beyond its range to
5e-11 absolute; the rare factor to the split path's; a quantile from log2 q to the main rational's 5e-6 (of its value or,
below 0.05, of that) plus what the factor's error moves it by, at most as much relative; the table's to the quadratics'
1.5e-7 and three roundings of numbers below 4.1, 2^-22 each."""
import math

import numpy as np
import pytest
from scipy.special import log_ndtr, ndtr, ndtri, ndtri_exp

from tests.gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu

KAPPA = math.sqrt(1.0 / (2.0 * math.log(2.0)))
LN2 = math.log(2.0)


def _probe(name, x_np):
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    x = torch.tensor(x_np, dtype=torch.float64, device="cuda")
    out = torch.empty((len(x_np), 3), dtype=torch.float64, device="cuda")
    V.vecchia_probe_math(getattr(V, "VECCHIA_PROBE_" + name), x, out)
    torch.cuda.synchronize()
    v = (np.asarray(x_np) * KAPPA).astype(np.float32).astype(np.float64)
    return out.cpu().numpy(), v


def _exponent(v):
    return 2.0 * LN2 * np.minimum(v * v, 1048576.0) * 2.0 ** -24


def test_inner_factor_tail():
    lim = 3.41 / KAPPA
    o, v = _probe("TAIL_F32", np.concatenate([np.linspace(-lim, lim, 700_000), [0.0, -0.0]]))
    rel = np.abs(o[:, 0] / ndtr(-np.abs(v) / KAPPA) - 1.0)
    print("FP32 inner tail: max rel %.2e, rms %.2e" % (rel.max(), np.sqrt(np.mean(rel ** 2))))
    assert np.all(rel <= 2e-6 + _exponent(v))
    o, v = _probe("TAIL_F32", np.concatenate([np.linspace(lim, 60.0, 200_000), np.logspace(1.5, 30, 200_000), [math.inf]]))
    assert np.all(np.abs(o[:, 0] - ndtr(-v / KAPPA)) <= 5e-11)
    assert np.isnan(_probe("TAIL_F32", [math.nan])[0][0, 0])


def test_rare_path_factor_and_quantile():
    t = np.concatenate([np.linspace(-1000.0, -3.9, 400_000), np.linspace(-4.5, 9.0, 200_000)])
    o, v = _probe("RARE_F32", t)
    te = v / KAPPA
    err = np.abs(np.log(o[:, 1]) + o[:, 2] * LN2 - log_ndtr(te))
    print("FP32 rare path: max |log err| of the factor %.2e" % err.max())
    assert np.all(err <= 2e-6 + _exponent(v))
    want = -ndtri_exp(log_ndtr(te) - LN2)
    d = np.abs(o[:, 0] - want) / np.maximum(want, 0.05)
    print("FP32 rare path: max rel err of the quantile %.2e" % d.max())
    assert np.all(d <= 2 * 5e-6)


@pytest.mark.parametrize("t", [1e4, 1e6, 4e7, 1e8, 1e10, 1e13, 1e19])
def test_arguments_beyond_the_fitted_range(t):
    o, _ = _probe("PHI_F32", [-t, t])
    assert np.array_equal(o[:, 0], [0.0, 0.0])
    o, _ = _probe("RARE_F32", [-t, t])
    assert np.all(np.isfinite(o))
    assert 0.0 < o[0, 1] < 1.0 and o[0, 2] == -1048576.0           # the exponent stops at -2^20
    assert abs(o[0, 0] / -ndtri_exp(-1048576.0 * LN2) - 1.0) <= 1e-4
    assert o[1, 1] == 1.0 and o[1, 2] == 0.0 and abs(o[1, 0]) <= 1e-6
    for what in ("PHI_F32", "RARE_F32"):
        assert np.all(np.isnan(_probe(what, [math.nan])[0][0, :2]))


def test_quantile_from_the_table():
    q = np.concatenate([np.logspace(math.log10(2.0 ** -15), math.log10(0.5), 400_000), np.linspace(0.3, 0.5, 100_000),
                        [2.0 ** -15, 0.5]])
    q = np.clip(q, 2.0 ** -15, 0.5)
    o, _ = _probe("NINV_F32", q)
    err = np.abs(o[:, 0] + ndtri(o[:, 1]))
    print("FP32 quantile from the table: max abs err %.2e" % err.max())
    assert err.max() <= 1.5e-7 + 3 * 2.0 ** -22
