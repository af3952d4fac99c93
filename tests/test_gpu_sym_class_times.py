"""Times of the symbolic classes: a launch of several classes, as one-wait
calls make, counts in a class that has rows, and in one class only."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def _long_rows():
    rng = np.random.default_rng(5)
    lens = rng.integers(100, 160, size=1500)
    ci = np.concatenate([rng.choice(700, size=int(l), replace=False) for l in lens])
    A = gen.csr_from_rows_cols(1500, 700, np.repeat(np.arange(1500), lens), ci, np.ones(ci.size))
    return A, gen.csr_from_rows_cols(700, 1500, np.repeat(np.arange(700), 40), rng.permuted(
        np.tile(np.arange(1500), (700, 1)), axis=1)[:, :40].ravel(), np.ones(28000))


@pytest.mark.parametrize("which,binning", [("lap2d", 2), ("lap2d", 0), ("long", 2), ("long", 0)])
def test_times_lie_in_classes_with_rows(which, binning):
    A, B = (gen.laplace2d_5pt(64),) * 2 if which == "lap2d" else _long_rows()
    op = run_gpu(A, B, binning=binning, timing=1)[3]
    for _ in range(3):  # (the first call's times hold the loading of the kernels)
        op.symbolic()
    st = op.stats()
    rows, ms = st["sym_rows"], st["sym_class_ms"]
    assert st["sym_waits"] == 1 and sum(rows) > 0
    # a launch without rows keeps its own, shorter time
    assert max(t for r, t in zip(rows, ms) if r) > max(t for r, t in zip(rows, ms) if not r)
