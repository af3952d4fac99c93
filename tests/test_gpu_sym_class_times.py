"""Times of the symbolic classes: a launch of several classes, as one-wait
calls make, counts in a class that has rows, and in one class only."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def _matrix(m, n, per_row, seed):
    rng = np.random.default_rng(seed)
    ci = np.concatenate([rng.choice(n, size=per_row, replace=False) for _ in range(m)])
    return gen.csr_from_rows_cols(m, n, np.repeat(np.arange(m), per_row), ci, np.ones(ci.size))


# rows of the direct classes 0, 4, 6 and 7, and of class 11 (two-level, second tier)
@pytest.mark.parametrize("binning", [2, 0])
@pytest.mark.parametrize("case", ["lap2d", (20, 30000, 20), (60, 30000, 40), (130, 1500, 40), (6, 200000, 8)])
def test_times_lie_in_classes_with_rows(case, binning):
    if case == "lap2d":
        A = B = gen.laplace2d_5pt(64)
    else:
        A, B = _matrix(1500, 700, case[0], 1), _matrix(700, case[1], case[2], 2)
    op = run_gpu(A, B, binning=binning, timing=1)[3]
    for _ in range(3):  # (the first call's times hold the loading of the kernels)
        op.symbolic()
    st = op.stats()
    rows, ms = st["sym_rows"], st["sym_class_ms"]
    assert st["sym_waits"] == 1 and sum(rows) > 0
    # a launch without rows keeps its own, shorter time
    assert max(t for r, t in zip(rows, ms) if r) > max(t for r, t in zip(rows, ms) if not r)
