"""The FP32 QMC kernels at the sizes where their launch can go wrong: chain lengths at the edges of the kernel sizes
(even numbers and 63; 4, 8, .., 60, 63 for joint blocks) and of the register-held lattice state (24 steps), point
counts below, at and above a wave and a chunk, and thresholds for which no, few and many lanes leave the fast forms.
Against FP64 terms, elementwise: a factor and a quantile are each good to about 5e-7, at most 63 of them enter a term,
and an exponential covariance amplifies them little, so 2e-5 of a term's size or, for a small one, of 1. Then launches
that several chain lengths share against a launch per length (bit for bit: an item does not depend on its launch)."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


def _terms(V, torch, plan, x_np, q, profile=False):
    x = torch.tensor(x_np, dtype=torch.float64, device="cuda")
    out = torch.empty(2, dtype=torch.float64, device="cuda")
    terms = torch.empty((V.plan_n_terms(plan), 2), dtype=torch.float64, device="cuda")
    if profile:
        V.vecchia_profile_enable(1)
    try:
        V.vecchia_logcdf(plan, x, q, out, terms=terms)
        torch.cuda.synchronize()
    finally:
        if profile:
            V.vecchia_profile_enable(0)
            V.vecchia_profile_reset()
    return out.cpu().numpy(), terms.cpu().numpy()


def _check(got, want):
    on = np.isfinite(want)     # a term whose every product underflows is -inf in both
    assert np.array_equal(got[~on], want[~on])
    d = np.abs(got[on] - want[on])
    assert np.all(d <= 2e-5 * np.maximum(1.0, np.abs(want[on]))), (d.max(), int(np.argmax(d)))


@pytest.mark.parametrize("m,n_points,n_shifts", [(1, 1, 2), (2, 63, 3), (3, 64, 2), (12, 65, 2), (13, 130, 2), (24, 2049, 2),
                                                 (25, 64, 2), (32, 65, 2), (33, 64, 2), (49, 65, 2), (63, 70, 2)])
@pytest.mark.parametrize("mean_x,sd_x", [(1.2, 0.1), (-1.5, 0.1), (0.0, 4.0)])
def test_fp32_terms_at_kernel_edges(m, n_points, n_shifts, mean_x, sd_x):
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    inst = W.small_random_instance(m + 9, m, 700 + m, nu=0.5, rho=0.3, n_points=n_points, n_shifts=n_shifts,
                                   mean_x=mean_x, sd_x=sd_x)
    plan = V.vecchia_plan(inst.locs, inst.ordering, m, inst.cov)
    got, want = (_terms(V, torch, plan, inst.x, V.make_qmc(n_points, n_shifts, 5, p))[1]
                 for p in (V.VECCHIA_FP32_LOOP, V.VECCHIA_FP64))
    V.vecchia_plan_destroy(plan)
    _check(got[:, 0], want[:, 0])


@pytest.mark.parametrize("m,p", [(1, 2), (1, 3), (2, 3), (3, 3), (7, 4), (9, 3), (30, 2), (31, 2)])
@pytest.mark.parametrize("mean_x,sd_x", [(1.2, 0.1), (0.0, 4.0)])
def test_fp32_block_terms_at_kernel_edges(m, p, mean_x, sd_x):
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    inst = W.small_random_instance(3 * m + 20, m, 800 + m, nu=0.5, rho=0.3, n_points=130, n_shifts=2, mean_x=mean_x, sd_x=sd_x)
    plan = V.vecchia_plan_block(inst.locs, inst.ordering, m, p, inst.cov)
    got, want = (_terms(V, torch, plan, inst.x, V.make_qmc(130, 2, 5, prec))[1]
                 for prec in (V.VECCHIA_FP32_LOOP, V.VECCHIA_FP64))
    V.vecchia_plan_destroy(plan)
    _check(got[:, 0], want[:, 0])


@pytest.mark.parametrize("D,m,p,n_points,precision", [(60, 5, 1, 300, "fp32"), (60, 30, 1, 300, "fp64"), (80, 7, 3, 200, "fp32"),
                                                      (2500, 20, 1, 8192, "fp32"), (900, 11, 1, 8192, "fp64")])
def test_shared_launches_equal_a_launch_per_chain_length(D, m, p, n_points, precision):
    # the timing hook launches every chain length by itself; the last two plans' longest chains have a launch of
    # their own either way and the shorter ones share it
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    inst = W.small_random_instance(D, m, 61, nu=1.5, rho=0.1, n_points=n_points, n_shifts=4)
    plan = (V.vecchia_plan(inst.locs, inst.ordering, m, inst.cov) if p == 1
            else V.vecchia_plan_block(inst.locs, inst.ordering, m, p, inst.cov))
    q = V.make_qmc(n_points, 4, 6, V.VECCHIA_FP32_LOOP if precision == "fp32" else V.VECCHIA_FP64)
    a, ta = _terms(V, torch, plan, inst.x, q)
    b, tb = _terms(V, torch, plan, inst.x, q, profile=True)
    V.vecchia_plan_destroy(plan)
    assert np.array_equal(ta, tb, equal_nan=True) and np.array_equal(a, b, equal_nan=True)
