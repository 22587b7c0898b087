"""Rounding error of the CSR product as wrapped, against extended precision.

It sums every row with fused multiply-adds in short chains added pairwise.  The
yardstick is the error of W lanes a row (the vector variant with an explicit
width): the product nobody chose a variant for may not be less exact than the
one with a width of the mean row length.  Norms over thousands of rows of
random data vary by about one part in the root of their number; 4% covers that."""
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


def _lengths(lens, seed):
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens, np.int64)
    n = lens.size
    rp = np.concatenate([[0], np.cumsum(lens)])
    r = np.repeat(np.arange(n), lens)
    col = (np.arange(rp[-1]) - rp[r]) * n // lens[r]  # spread over the row, ascending
    return W.Csr(n, n, rp.astype(np.int32), col.astype(np.int32), rng.standard_normal(rp[-1]), "lengths")


N = 40_000
CASES = {
    "5pt": lambda: W.stencil_2d5(200),
    "7pt": lambda: W.aniso_3d7(34),
    "27pt": lambda: W.stencil_3d27(34),
    "equal_15": lambda: _lengths(np.full(N, 15), 1),
    "equal_40": lambda: _lengths(np.full(N, 40), 2),
    "equal_300": lambda: _lengths(np.full(9000, 300), 3),
    "40_and_2": lambda: _lengths(np.where(np.arange(N) % 7 == 0, 40, 2), 4),
    "mostly_empty": lambda: _lengths(np.where(np.arange(N) % 10 == 0, 60, 0), 5),
    "1_to_29": lambda: _lengths(np.random.default_rng(6).integers(1, 30, N), 6),
    "longer_than_a_run": lambda: _lengths(np.where(np.arange(N) % 40 == 0, 700, 3), 7),
}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", list(CASES))
def test_error_is_not_above_w_lanes_a_row(mxl, ctx, name, dtype):
    A = CASES[name]()
    f = np.float64 if dtype == torch.float64 else np.float32
    xh = W.uniform_vec(A.ncols, 9).astype(f)
    prod = A.val.astype(f).astype(np.longdouble) * xh.astype(np.longdouble)[A.col]
    full = np.diff(A.row_ptr) > 0
    want = np.zeros(A.nrows, np.longdouble)
    want[full] = np.add.reduceat(prod, A.row_ptr[:-1][full])
    M = matrix(mxl, ctx, A, dtype)
    w = 2
    while w < 64 and w < A.val.size / A.nrows:
        w *= 2
    err = {}
    for what, op in (("wrapped", M), ("lanes", M.convert("csr", variant=1, vector_width=w))):
        y = torch.empty(A.nrows, dtype=dtype, device=DEV)
        op.apply(dev(xh), y)
        err[what] = float(np.linalg.norm((y.cpu().numpy().astype(np.longdouble) - want).astype(np.float64)))
    assert err["wrapped"] <= 1.04 * err["lanes"], err


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("short", [3, 9])  # blocks of at most 320 and of 512 entries
def test_long_rows_of_row_blocks_equal_64_lanes(mxl, ctx, short, dtype):
    """A row that is a block of its own is swept by the whole wave, one entry a
    lane after another as with 64 lanes a row: the same bits."""
    lens = np.where(np.arange(3000) % 50 == 0, np.random.default_rng(1).integers(513, 4000, 3000), short)
    A = _lengths(lens, 8)
    M = matrix(mxl, ctx, A, dtype)
    x = dev(W.uniform_vec(A.ncols, 9), dtype)
    y = [torch.empty(A.nrows, dtype=dtype, device=DEV) for _ in range(2)]
    M.convert("csr", variant=mxl.CSR_STREAM).apply(x, y[0])
    M.convert("csr", variant=1, vector_width=64).apply(x, y[1])
    long = np.flatnonzero(lens > 512)
    assert np.array_equal(y[0].cpu().numpy()[long], y[1].cpu().numpy()[long])
