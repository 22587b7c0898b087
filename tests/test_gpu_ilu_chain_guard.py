"""Exact triangular solves of factors that the chain solve must not take or
must bound: rows whose columns are not in order."""
import numpy as np
import pytest
import torch

import workloads as W
from tests._gpu import DEV, dev, matrix

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxl():
    import paper_2006_16852_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(mxl):
    return mxl.Context(0)


def _banded(n, offsets, seed):
    """Diagonally dominant matrix with the given diagonals beside the main one."""
    rng = np.random.default_rng(seed)
    r = np.concatenate([np.arange(max(0, -o), min(n, n - o)) for o in (*offsets, 0)])
    c = np.concatenate([np.arange(max(0, -o), min(n, n - o)) + o for o in (*offsets, 0)])
    key = np.sort(r.astype(np.int64) * n + c)
    r, c = key // n, (key % n).astype(np.int32)
    v = rng.uniform(-1.0, 1.0, key.size)
    v[r == c] = np.bincount(r, weights=np.abs(v), minlength=n) + 1.0
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    return W.Csr(n, n, rp, c, v, "banded")


def _substitute(A, lu, r):
    """Both substitutions with every row's entries in their stored order,
    whichever side of the diagonal they stand on."""
    n, x = A.nrows, r.copy()
    rows = [range(A.row_ptr[i], A.row_ptr[i + 1]) for i in range(n)]
    for i in range(n):
        for q in rows[i]:
            if A.col[q] < i:
                x[i] = x[i] - lu[q] * x[A.col[q]]
    for i in reversed(range(n)):
        d = 0.0
        for q in rows[i]:
            if A.col[q] > i:
                x[i] = x[i] - lu[q] * x[A.col[q]]
            elif A.col[q] == i:
                d = lu[q]
        x[i] = x[i] / d
    return x


@pytest.mark.parametrize("swap", [(0, 1), (3, 4), (1, 3), (0, 4)])
def test_rows_out_of_order_take_the_levels(mxl, ctx, swap):
    """A pentadiagonal matrix with two entries of some rows exchanged, within
    a side of the diagonal and across it (the diagonal stays in the middle of
    its five entries, where it is found): solved by levels, as stored."""
    A = _banded(640, (-2, -1, 1, 2), 3)
    for i in range(40, 600, 7):
        a, b = A.row_ptr[i] + swap[0], A.row_ptr[i] + swap[1]
        A.col[[a, b]] = A.col[[b, a]]
        A.val[[a, b]] = A.val[[b, a]]
    P = mxl.ilu(matrix(mxl, ctx, A), sweeps=1)
    lu = P.info(factors=True)["lu"]
    r = W.uniform_vec(A.nrows, 5)
    z = torch.empty(A.nrows, dtype=torch.float64, device=DEV)
    P.apply(dev(r), z)
    assert np.array_equal(z.cpu().numpy(), _substitute(A, lu, r))


def test_column_outside_the_matrix_is_an_error(mxl, ctx):
    A = _banded(640, (-2, -1, 1, 2), 3)
    A.col[A.row_ptr[101] - 1] = 640 + 10_000_000
    with pytest.raises(mxl.MxlError) as e:
        mxl.ilu(matrix(mxl, ctx, A), sweeps=1)
    assert e.value.status == mxl.ERR_INVALID_MATRIX
