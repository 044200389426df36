"""The full-dimension estimate where its value is NaN (a covariance that is not positive definite, a NaN threshold) or
exactly -inf (a limit of -inf, or one whose square overflows): the two are told apart, whichever Cholesky panel or
dimension block holds the cause and however ragged the point tiles are."""
import math

import numpy as np
import pytest

from tests.gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _full(S, b, N, R):
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    plan = V.vecchia_plan_from_cov(S, 1)
    out = torch.empty(2, dtype=torch.float64, device="cuda")
    V.vecchia_full_logcdf(plan, torch.tensor(b, device="cuda"), V.make_qmc(N, R, 2, V.VECCHIA_FP64), out)
    torch.cuda.synchronize()
    V.vecchia_plan_destroy(plan)
    return out.cpu().numpy()


def _cov(D):
    return 0.5 * np.eye(D) + 0.5


@pytest.mark.parametrize("N,R", [(1, 1), (16, 2), (100, 3), (1500, 10)])
@pytest.mark.parametrize("D,bad", [(1, 0), (20, 0), (20, 13), (20, 19), (150, 5), (150, 40), (150, 149)])
def test_indefinite_covariance_gives_nan(D, bad, N, R):
    S = _cov(D)
    S[bad, bad] = -1.0
    assert np.all(np.isnan(_full(S, np.ones(D), N, R)))
    b = np.ones(D)
    b[D // 2] = -math.inf
    assert np.isnan(_full(S, b, N, R)[0])


@pytest.mark.parametrize("N,R", [(1, 1), (100, 3), (1500, 10)])
@pytest.mark.parametrize("D,i", [(20, 0), (20, 19), (150, 0), (150, 77), (150, 149)])
def test_zero_probability_and_nan_thresholds(D, i, N, R):
    b = np.ones(D)
    for v in (-math.inf, -1e160):
        b[i] = v
        out = _full(_cov(D), b, N, R)
        assert out[0] == -math.inf
    b[i] = math.nan
    assert np.isnan(_full(_cov(D), b, N, R)[0])
    b[i] = math.inf
    assert np.isfinite(_full(_cov(D), b, N, R)[0])
