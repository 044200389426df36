"""The FP64 QMC kernels at the sizes where their launch can go wrong: chain lengths at the edges of the kernel sizes
(every even number, 63), of the register-held lattice state (12 steps) and of the workgroup shapes (32, 52 steps); point
counts below, at and above a wave and a chunk; one shift and several. Against the oracle, elementwise."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests.gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n_points,n_shifts", [(1, 1, 2), (2, 63, 3), (3, 64, 2), (12, 65, 2), (13, 513, 1), (32, 130, 2),
                                                 (33, 64, 2), (52, 65, 2), (53, 40, 2), (63, 70, 2)])
@pytest.mark.parametrize("mean_x", [1.2, -1.5])
def test_fp64_terms_at_kernel_edges(m, n_points, n_shifts, mean_x):
    torch = torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    D = m + 9
    inst = W.small_random_instance(D, m, 500 + m, nu=0.5, rho=0.3, n_points=n_points, n_shifts=n_shifts, mean_x=mean_x)
    c = inst.cov
    ref = oracle.logcdf(inst.locs, inst.x, m, c.family, c.nu, c.sigma2, c.range, c.nugget, inst.ordering, n_points, n_shifts,
                        inst.qmc.seed)
    plan = V.vecchia_plan(inst.locs, inst.ordering, m, inst.cov)
    x = torch.tensor(inst.x, dtype=torch.float64, device="cuda")
    out = torch.empty(2, dtype=torch.float64, device="cuda")
    terms = torch.empty((D, 2), dtype=torch.float64, device="cuda")
    V.vecchia_logcdf(plan, x, V.make_qmc(n_points, n_shifts, inst.qmc.seed, V.VECCHIA_FP64), out, terms=terms)
    torch.cuda.synchronize()
    got = terms.cpu().numpy()
    V.vecchia_plan_destroy(plan)
    # parity bar of the FP64 path: 1e-10 per term (exponential blocks are well conditioned here)
    np.testing.assert_allclose(got[:, 0], ref["terms"][:, 0], rtol=0, atol=1e-10)
    if n_shifts > 1:
        np.testing.assert_allclose(got[:, 1], ref["terms"][:, 1], rtol=1e-7, atol=1e-10)
