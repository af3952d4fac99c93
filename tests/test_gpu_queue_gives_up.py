"""A queued run whose waits end before their slots fill: the kernel ends, the
run is reported, and the next run on the same batch is whole again."""
import numpy as np
import pytest

import oracle
from paper_2103_11991_amd import gen
from gpu_util import compare

pytestmark = pytest.mark.gpu


def test_a_given_up_wait_is_reported_and_the_next_run_is_whole():
    import torch
    from paper_2103_11991_amd._lib import OPT, SpgError, spg_batch_set_option
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMMBatch
    prods = [(gen.banded_random(900, 24, 3, 2 * i), gen.banded_random(900, 24, 3, 2 * i + 1)) for i in range(8)]
    need = sum(int(oracle.row_nnz(A, B).sum()) for A, B in prods)
    batch = SpGEMMBatch([DeviceCsr.from_host(A) for A, _ in prods], [DeviceCsr.from_host(B) for _, B in prods])

    def whole():
        torch.cuda.synchronize()
        for i, (A, B) in enumerate(prods):
            rp, c, v = batch.product_queued(i)
            compare(A, B, rp.cpu().numpy().astype(np.int64), c.cpu().numpy(), v.cpu().numpy())
        batch.stats()

    batch.run_queued(need)
    whole()
    # 64 symbolic items for more workgroups than that: the others find their
    # numeric slots empty at their first look
    spg_batch_set_option(batch.b, OPT["queue_polls"], 0)
    batch.run_queued(need)
    for call in (lambda: batch.product_queued(0), batch.stats, lambda: batch.product_queued(0)):
        with pytest.raises(SpgError) as e:
            call()
        assert e.value.status_name == "SPG_ERR_HIP" and "given up" in str(e.value)
    spg_batch_set_option(batch.b, OPT["queue_polls"], 1 << 26)
    for _ in range(2):
        batch.run_queued(need)
        whole()


@pytest.mark.parametrize("value", [-1, (1 << 26) + 1])
def test_polls_out_of_range_are_refused(value):
    from paper_2103_11991_amd._lib import OPT, SpgError, spg_batch_set_option
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMMBatch
    A = DeviceCsr.from_host(gen.banded_random(300, 9, 1, 0))
    batch = SpGEMMBatch([A], [A])
    with pytest.raises(SpgError) as e:
        spg_batch_set_option(batch.b, OPT["queue_polls"], value)
    assert e.value.status_name == "SPG_ERR_ARG"
