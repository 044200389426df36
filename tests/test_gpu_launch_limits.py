"""Batches whose work items come near the 2^31 - 1 of one launch. Chain lengths with few items share the launch of the
next longer ones, and FP64 launches take plain and joint terms alike: a batch is refused only where the items of one
length of one kind pass the limit by themselves. Batches are created, not run (creation allocates nothing on the
device)."""
import numpy as np
import pytest

from tests.gpu_helpers import torch_cuda

pytestmark = pytest.mark.gpu

LIMIT = 2 ** 31 - 1


def _plain(V, D, m):
    """D - m terms conditioned on the first m variables, the first m on nothing."""
    return V.vecchia_plan_from_cov(np.eye(D), m, nbr=[[] if i < m else list(range(m)) for i in range(D)])


def _joint(V, D, m):
    return V.vecchia_plan_from_cov_block(np.eye(D), [(list(range(m)) + [i], m) for i in range(m, D)])


def _qmc(V, shifts, chunks, precision):
    return V.make_qmc(chunks * (2048 if precision == V.VECCHIA_FP32_LOOP else 512), shifts, 1, precision)


def _create(V, plans, qmcs):
    try:
        V.vecchia_batch_destroy(V.vecchia_batch_create(plans, qmcs))
        return True
    except V.VecchiaError:
        return False
    finally:
        for p in plans:
            V.vecchia_plan_destroy(p)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("short_terms", [5, 15])
def test_a_shared_launch_stays_within_the_limit(prec, short_terms):
    torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    p = V.VECCHIA_FP32_LOOP if prec == "fp32" else V.VECCHIA_FP64
    # two-step items: 1998 * 1024 * 1048 + 10 * 100 * 3325 = LIMIT - 951; one-step items: 100 a term
    long_items = 1998 * 1024 * 1048 + 10 * 100 * 3325
    assert long_items == LIMIT - 951
    plans = [_plain(V, 2000, 2), _plain(V, 12, 2), _plain(V, 1 + short_terms, 1)]
    assert _create(V, plans, [_qmc(V, 1024, 1048, p), _qmc(V, 100, 3325, p), _qmc(V, 10, 10, p)])


def test_plain_and_joint_fp64_terms_of_one_length_have_a_limit_each():
    torch_cuda()
    from paper_2007_15195_amd import vecchia as V
    q = _qmc(V, 1024, 1000, V.VECCHIA_FP64)   # 1200 * 1024 * 1000 items each, 2.46e9 together
    assert _create(V, [_plain(V, 1202, 2), _joint(V, 1202, 2)], [q, q])
    assert not _create(V, [_plain(V, 1202, 2), _plain(V, 1202, 2)], [q, q])
    assert not _create(V, [_joint(V, 1202, 2), _joint(V, 1202, 2)], [q, q])
