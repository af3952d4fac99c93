"""Global-path rows whose sparse neighbouring tiles are merged: columns and list
pairs of a group below, at and above its limits (2048 columns, 1024 pairs, 16
tiles), empty tiles, dense tiles between sparse ones, and both kinds of row
(more than 256 entries of A: one unit per tile).  Integer values: exact."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare, run_gpu

pytestmark = pytest.mark.gpu

W = 4096  # columns per tile


def _product(tiles, per_tile, stride, a_lens, dtype, seed=0, k=None):
    """B rows that each hold a part of `per_tile[t]` columns, `stride` apart, in tile t; A rows that take many."""
    rng = np.random.default_rng(seed)
    nb = 300
    k = k or tiles * W
    cols = np.concatenate([t * W + np.arange(c) * stride % W for t, c in enumerate(np.resize(per_tile, tiles))])
    cols = np.unique(cols[cols < k])
    keep = rng.random((nb, cols.size)) < 0.2
    keep[0] = True
    r, c = np.nonzero(keep)
    B = gen.csr_from_rows_cols(nb, k, r, cols[c], rng.integers(-3, 4, size=r.size).astype(dtype))
    lens = np.asarray(a_lens)
    ac = np.concatenate([np.sort(rng.choice(nb, size=int(x), replace=False)) for x in lens])
    A = gen.csr_from_rows_cols(lens.size, nb, np.repeat(np.arange(lens.size), lens), ac,
                               rng.integers(-3, 4, size=ac.size).astype(dtype))
    return A, B


LENS = [100, 200, 255, 256, 257, 300, 64, 0, 2, 250, 250]


def _check(A, B, tiles):
    """The LDS limit that still holds the symbolic table of the whole range, so that most rows' values do not fit."""
    limit = 1024
    while limit < tiles * W // 8:
        limit *= 2
    rp, c, v, op = run_gpu(A, B, lds_limit=limit)
    compare(A, B, rp, c, v, exact=True)
    st = op.stats()
    assert st["num_rows"][9] >= 6 and st["num_tiles"] == tiles and st["tile_fallback_rows"] == 0


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("tiles", [1, 2, 15, 16, 17, 33, 64, 65, 127, 128])
def test_tiles(tiles, dtype):
    A, B = _product(tiles, [300, 0, 0, 170, 400], 37, LENS, dtype, tiles, k=tiles * W - 5)
    _check(A, B, tiles)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("per_tile, stride", [
    ([128], 1), ([127, 128, 129], 1),         # 16 tiles of 128 columns: exactly 2048, and around it
    ([64], 33), ([63, 64, 65], 33),           # 16 tiles of 64 pairs: exactly 1024, and around it
    ([1024, 1023, 1, 0], 2), ([2047, 1, 1], 2), ([4096, 0, 3, 2, 0, 0, 2048], 1),
])
def test_limits_of_a_group(per_tile, stride, dtype):
    A, B = _product(60, per_tile, stride, LENS, dtype, 5)
    _check(A, B, 60)
