"""Exact triangular solves of factors that the chain solve must not take or
must bound: rows whose columns are not in order, and waits that end without
their operand."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle as O
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


def _set_wait_passes(mxl, P, passes):
    f = getattr(mxl.lib, "_ZN3mxl25ilu_chain_set_wait_passesEP6mxl_opl")  # no entry point of the ABI
    f.argtypes, f.restype = [C.c_void_p, C.c_int64], C.c_int
    assert f(P.h, passes) == 0


def test_a_solve_that_gives_up_is_an_error(mxl, ctx):
    """With no pass without progress allowed (the worker's first pass never finds a
    record), every group gives up at once: NaN comes out, the next synchronising
    call says so once, and with the ordinary limit the same handle solves again."""
    A = W.convdiff_3d7(19)
    M = matrix(mxl, ctx, A)
    P = mxl.ilu(M, sweeps=2)
    lu = P.info(factors=True)["lu"]
    r = W.uniform_vec(A.nrows, 5)
    z = torch.empty(A.nrows, dtype=torch.float64, device=DEV)
    S = mxl.solver("gmres", M, P, max_iters=200, reduction=1e-8)
    usual = (1 << 26) + 64 * A.nrows
    _set_wait_passes(mxl, P, 0)
    P.apply(dev(r), z)
    with pytest.raises(mxl.MxlError) as e:
        P.info()
    assert e.value.status == mxl.ERR_INTERNAL
    assert np.isnan(z.cpu().numpy()).any()
    P.info()  # reported once
    with pytest.raises(mxl.MxlError):
        S.solve(dev(r), torch.zeros_like(z))
    _set_wait_passes(mxl, P, usual)
    P.apply(dev(r), z)
    P.info()
    assert np.array_equal(z.cpu().numpy(), _substitute(A, lu, r))
    assert S.solve(dev(r), torch.zeros_like(z))["stop_reason"] == mxl.STOP_CONVERGED


@pytest.mark.parametrize("n,half", [(4, 30_000), (64, 400)])
def test_groups_that_wait_for_whole_chains(mxl, ctx, n, half):
    """Chains one after another: the first row of a chain needs the last row of
    the chain before it, so that every group waits for all earlier ones."""
    rows = n * half
    r = np.arange(rows)
    cut = r % half == 0
    pr = np.concatenate([r[~cut], r[cut][1:], r])
    pc = np.concatenate([r[~cut] - 1, r[cut][1:] - 2, r])
    key = np.sort(np.unique(np.concatenate([pr * rows + pc, pc * rows + pr])))
    rr, cc = key // rows, (key % rows).astype(np.int32)
    v = np.random.default_rng(1).uniform(-1, 1, key.size)
    v[rr == cc] = np.bincount(rr, weights=np.abs(v), minlength=rows) + 1.0
    A = W.Csr(rows, rows, np.concatenate([[0], np.cumsum(np.bincount(rr, minlength=rows))]).astype(np.int32), cc, v, "serial")
    P = mxl.ilu(matrix(mxl, ctx, A), sweeps=1)
    lu = P.info(factors=True)["lu"]
    b = W.uniform_vec(rows, 5)
    z = torch.empty(rows, dtype=torch.float64, device=DEV)
    P.apply(dev(b), z)
    P.info()
    assert np.array_equal(z.cpu().numpy(), O.ilu_apply(A, lu, b, mode=0, sweeps=0))


def _tridiagonal_with_wide_rows(n, extra):
    """One row with `extra` more entries before, one with as many behind the diagonal."""
    A = _banded(n, (-1, 1), 4)
    rng = np.random.default_rng(6)
    i, j = n - 3, 2
    r = np.repeat(np.arange(n, dtype=np.int64), A.row_lengths())
    add = np.concatenate([i * n + 10 * np.arange(1, extra + 1), j * n + 50 + 10 * np.arange(1, extra + 1)])
    key = np.concatenate([r * n + A.col, add])
    val = np.concatenate([A.val, rng.uniform(-0.01, 0.01, add.size)])
    o = np.argsort(key)
    key, val = key[o], val[o]
    r = key // n
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    return W.Csr(n, n, rp, (key % n).astype(np.int32), val, "wide_rows")


@pytest.mark.parametrize("extra", [1, 4, 5, 6, 12])
def test_padding_on_either_side_of_its_line(mxl, ctx, extra):
    """(2 extra + 2) slots a row against 4 nnz + 2 n: chains up to 5 extra
    entries, levels above; the same substitution either way."""
    A = _tridiagonal_with_wide_rows(6001, extra)
    P = mxl.ilu(matrix(mxl, ctx, A), sweeps=2)
    lu = P.info(factors=True)["lu"]
    r = W.uniform_vec(A.nrows, 5)
    z = torch.empty(A.nrows, dtype=torch.float64, device=DEV)
    P.apply(dev(r), z)
    assert np.array_equal(z.cpu().numpy(), O.ilu_apply(A, lu, r, mode=0, sweeps=0))


def test_one_wide_row_does_not_multiply_the_memory(mxl, ctx):
    A = _tridiagonal_with_wide_rows(500_000, 12)
    M = matrix(mxl, ctx, A)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    P = mxl.ilu(M, sweeps=0)
    used = before - torch.cuda.mem_get_info()[0]
    # factors 8 nnz, diagonal, work vectors and level lists: 44 bytes a row; rounding of the allocator
    assert used <= 8 * A.val.size + 44 * A.nrows + (32 << 20), used
    del P
