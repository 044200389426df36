"""FP32 terms whose conditioning set holds two sites 1e-8 to 3e-8 apart: the second site's limit is scaled by up to 1e8,
where the polynomials of the FP32 CDF ratio leave FP32's range. Against FP64 terms, with the bound of the FP32 kernels'
other tests (2e-5 of a term's size or, for a small one, of 1): a lane whose scaled limit is that far below zero has a
factor that is 0 in any precision, one as far above it a factor of 1. Where both limits of the pair are close to each
other, FP32's rounding of y times 1e8 decides which lanes those are, so there only finite values are asked for."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _terms(V, torch, plan, x_np, precision):
    x = torch.tensor(x_np, dtype=torch.float64, device="cuda")
    out = torch.empty(2, dtype=torch.float64, device="cuda")
    terms = torch.empty((V.plan_n_terms(plan), 2), dtype=torch.float64, device="cuda")
    V.vecchia_logcdf(plan, x, V.make_qmc(1000, 4, 5, precision), out, terms=terms)
    torch.cuda.synchronize()
    return terms.cpu().numpy()[:, 0]


@pytest.mark.parametrize("dx", [1e-8, 2e-8, 3e-8, -1e-8, -3e-8])
@pytest.mark.parametrize("first,second,exact", [(3.0, -2.0, True), (-2.0, 3.0, True), (3.0, 2.0, False), (2.0, 2.5, False)])
def test_fp32_terms_conditioned_on_a_close_pair(dx, first, second, exact):
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    locs = np.array([[0.0, 0.0], [dx, 0.0], [0.5, 0.5], [0.2, 0.9], [0.7, 0.1]])
    plan = V.vecchia_plan(locs, W.ORDER_GIVEN, 4, V.make_cov(V.VECCHIA_COV_MATERN, 1.5, 1.0, 1.0, 0.0), perm=np.arange(5))
    x = np.array([first, second, 1.0, 1.0, 1.0])
    got, want = (_terms(V, torch, plan, x, p)[2:] for p in (V.VECCHIA_FP32_LOOP, V.VECCHIA_FP64))
    V.vecchia_plan_destroy(plan)
    assert np.all(np.isfinite(got)), got
    if exact:
        assert np.all(np.abs(got - want) <= 2e-5 * np.maximum(1.0, np.abs(want))), (got, want)


@pytest.mark.parametrize("p", [1, 2, 3])
def test_fp32_plan_and_joint_terms_with_a_close_pair(p):
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    locs = np.random.default_rng(1).random((30, 2))
    locs[1] = locs[0] + [1e-8, 0.0]
    cov = V.make_cov(V.VECCHIA_COV_MATERN, 1.5, 1.0, 1.0, 1e-16)
    plan = (V.vecchia_plan(locs, W.ORDER_GIVEN, 8, cov, perm=np.arange(30)) if p == 1
            else V.vecchia_plan_block(locs, W.ORDER_GIVEN, 8, p, cov, perm=np.arange(30)))
    x = np.full(30, 2.0)
    x[:2] = 3.0, -1.0
    got, want = (_terms(V, torch, plan, x, q) for q in (V.VECCHIA_FP32_LOOP, V.VECCHIA_FP64))
    V.vecchia_plan_destroy(plan)
    assert np.all(np.abs(got - want) <= 2e-5 * np.maximum(1.0, np.abs(want))), (got, want)
