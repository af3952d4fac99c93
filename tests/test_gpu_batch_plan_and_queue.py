"""A batch's plan and its queued form side by side: the queued form's first
call must leave what the plan's numeric runs read (the rows' lists, placed in
an order that differs from one analysis to the next once there are several
chunks of 2048 rows), and a plan made after it must stand by itself."""
import numpy as np
import pytest

import oracle
from paper_2103_11991_amd import gen
from gpu_util import compare

pytestmark = pytest.mark.gpu


def _products():
    n, bwa, bwb = gen.batch_sizes(10, seed=3, lo=4000, hi=9000)
    return [(gen.banded_random(int(n[i]), int(bwa[i]), 3, 2 * i), gen.banded_random(int(n[i]), int(bwb[i]), 3, 2 * i + 1))
            for i in range(10)]


def _check(get, prods):
    import torch
    torch.cuda.synchronize()
    for i, (A, B) in enumerate(prods):
        rp, c, v = get(i)
        compare(A, B, rp.cpu().numpy().astype(np.int64), c.cpu().numpy(), v.cpu().numpy())


@pytest.mark.parametrize("plan_first", [True, False])
def test_numeric_runs_on_the_plan_after_a_queued_run(plan_first):
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMMBatch
    prods = _products()
    need = sum(int(oracle.row_nnz(A, B).sum()) for A, B in prods)
    batch = SpGEMMBatch([DeviceCsr.from_host(A) for A, _ in prods], [DeviceCsr.from_host(B) for _, B in prods])
    if plan_first:
        batch.plan()
    batch.run_queued(need)
    _check(batch.product_queued, prods)
    for numeric_only in (True, False, True):
        batch.run(numeric_only=numeric_only)
        _check(batch.product, prods)
        batch.run_queued(need)
        _check(batch.product_queued, prods)


def test_learned_sizes_without_a_predictor_are_refused():
    from paper_2103_11991_amd._lib import SpgError
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMMBatch
    A = gen.banded_random(300, 9, 1, 0)
    batch = SpGEMMBatch([DeviceCsr.from_host(A)], [DeviceCsr.from_host(A)], binning=1)
    for call in (batch.plan, lambda: batch.run_queued(10 ** 5)):
        with pytest.raises(SpgError) as e:
            call()
        assert e.value.status_name == "SPG_ERR_STATE"
