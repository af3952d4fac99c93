"""One-wait symbolic phases of many rows of 512 to 16 thousand products, where
the tiers of 128 and of 512 lanes run in launches of their own or with the
next tier, by the average row; with every LDS limit's last tier."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare, run_gpu

pytestmark = pytest.mark.gpu


def _matrix(m, n, lo, hi, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(lo, hi + 1, size=m)
    ci = np.concatenate([rng.choice(n, size=int(l), replace=False) for l in lens])
    return gen.csr_from_rows_cols(m, n, np.repeat(np.arange(m), lens), ci,
                                  rng.integers(-2, 3, size=ci.size).astype(np.float64))


# rows on both sides of the rule's average products: 512, 4096, 2048 and 16384
@pytest.mark.parametrize("m", [1023, 1024, 1500])
@pytest.mark.parametrize("la,lb", [((10, 20), (20, 40)), ((20, 60), (20, 60)), ((60, 80), (50, 66)),
                                   ((100, 160), (30, 40)), ((200, 300), (60, 66)), ((200, 300), (70, 80))])
def test_average_rows(la, lb, m):
    A, B = _matrix(m, 700, *la, 1), _matrix(700, 1500, *lb, 2)
    rp, c, v, op = run_gpu(A, B)
    assert op.stats()["sym_waits"] == 1
    rows = [(0, 40), (m // 2, m // 2 + 40), (m - 40, m)]
    compare(A, B, rp, c, v, rows=rows, exact=True)
    assert rp[-1] == c.size


@pytest.mark.parametrize("limit", [1024, 2048, 4096, 8192, 16384, 32768])
@pytest.mark.parametrize("la,lb", [((20, 60), (20, 60)), ((100, 160), (40, 60))])
def test_last_tier_of_the_limit(la, lb, limit):
    A, B = _matrix(1100, 700, *la, 3), _matrix(700, 30000, *lb, 4)
    rp, c, v, op = run_gpu(A, B, lds_limit=limit)
    assert op.stats()["sym_waits"] == 1
    compare(A, B, rp, c, v, rows=[(0, 30), (1070, 1100)], exact=True)
