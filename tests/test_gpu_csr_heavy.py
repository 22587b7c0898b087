"""The CSR operator as wrapped on matrices with blocks of rows far above the
mean, which helper waves take in parts: products at the edges of the rule
(blocks just under and over it, a last block that is not full, a block ruled by
one row, parts without rows, more heavy blocks than helpers) against the FP64
oracle, and the fused dot of CG on such a matrix.

Tolerance per row: 1e-12 (FP64), 1e-5 (FP32) of |alpha| sum |a||x| + |beta||y|.
"""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests._gpu import DEV, assert_rows_close, dev, matrix, spmv_reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxl():
    import paper_2006_16852_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(mxl):
    return mxl.Context(0)


def _rows(lengths, ncols, seed):
    lengths = np.asarray(lengths, np.int64)
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lengths)])
    row = np.repeat(np.arange(lengths.size), lengths)
    col = (np.arange(rp[-1]) - rp[row]) * ncols // lengths[row]
    return W.Csr(lengths.size, ncols, rp.astype(np.int32), col.astype(np.int32), rng.uniform(-1, 1, rp[-1]), "heavy")


LENGTHS = {
    "cluster": [5] * 3000 + [400] * 200 + [5] * 3000,
    "cluster_in_the_last_block": [6] * 20_000 + [600] * 9,
    "first_rows_longer_than_a_run": [3000] * 40 + [6] * 20_000,
    # 64 rows a block, heavy above 2,560 (at most 5 entries a row) or 2,048
    "at_the_line": ([4, 5] * 20_000 + [40] * 64 + [40] * 63 + [41] + [5] * 65) * 2,
    "at_the_longer_line": [6] * 32 * 3000 + [64] * 32 + [65] * 32 + [6] * 32 * 50,
    # one row with a quarter of its block's entries and one just under
    "ruled_by_one_row": [6] * 6400 + [3000] + [150] * 31 + [6] * 640 + [1400] + [150] * 31 + [6] * 640,
    "empty_rows_in_a_heavy_block": [6] * 6400 + [0, 700, 0, 0, 700, 700, 0, 700] * 20 + [0] * 40 + [6] * 6400,
    "heavy_all_over": ([6] * 640 + [300] * 32) * 40,
    "few_rows": [5] * 30 + [300] * 30,
}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("name", list(LENGTHS))
def test_heavy_blocks(mxl, ctx, name, dtype):
    A = _rows(LENGTHS[name], 70_001, 11)
    op = matrix(mxl, ctx, A, dtype)
    rng = np.random.default_rng(7)
    x, y0 = rng.uniform(-1, 1, A.ncols), rng.uniform(-1, 1, A.nrows)
    fp32 = dtype == torch.float32
    for alpha, beta in [(1.0, 0.0), (0.5, -2.0)]:
        y = dev(y0, dtype) if beta else torch.full((A.nrows,), float("nan"), dtype=dtype, device=DEV)
        op.apply(dev(x, dtype), y, alpha, beta)
        want, bound = spmv_reference(A, x, alpha, beta, y0, fp32)
        assert_rows_close(y.cpu().numpy(), want, bound, 1e-5 if fp32 else 1e-12, f"{name} {alpha} {beta}")


def test_cg_with_heavy_blocks_tracks_the_oracle(mxl, ctx):
    """A Poisson matrix with a dense diagonal block of 300 rows: the fused dots of
    CG include the helpers' rows; two solves are equal bit for bit."""
    n, m, at = 20_000, 300, 7_000
    rng = np.random.default_rng(5)
    D = rng.uniform(-1, 1, (m, m))
    D = D + D.T
    rows, cols, vals = [], [], []
    for o in (-1, 1):
        i = np.arange(max(0, -o), min(n, n - o))
        i = i[~((i >= at) & (i < at + m) & (i + o >= at) & (i + o < at + m))]
        rows.append(i), cols.append(i + o), vals.append(np.full(i.size, -1.0))
    a, b = np.nonzero(~np.eye(m, dtype=bool))
    rows.append(a + at), cols.append(b + at), vals.append(D[a, b])
    r, c, v = np.concatenate(rows), np.concatenate(cols), np.concatenate(vals)
    s = np.bincount(r, weights=np.abs(v), minlength=n) + 0.05
    r, c, v = np.concatenate([r, np.arange(n)]), np.concatenate([c, np.arange(n)]), np.concatenate([v, s])
    o = np.lexsort((c, r))
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    A = W.Csr(n, n, rp, c[o].astype(np.int32), v[o], "dense_block")
    b = O.spmv(A, W.uniform_vec(n, 3))
    ref = O.pcg(A, b, dinv=O.jacobi_dinv(A)[0], reduction=1e-10)
    M = matrix(mxl, ctx, A)
    S = mxl.solver("cg", M, mxl.jacobi(M), max_iters=2000, reduction=1e-10)
    got = []
    for _ in range(2):
        x = torch.zeros(n, dtype=torch.float64, device=DEV)
        info = S.solve(dev(b), x)
        assert info["stop_reason"] == mxl.STOP_CONVERGED
        assert abs(info["iterations"] - ref["iterations"]) <= 2, (info["iterations"], ref["iterations"])
        got.append(x.cpu().numpy())
    assert np.array_equal(got[0], got[1])
    res = b - O.spmv(A, got[0])
    assert np.linalg.norm(res) <= 1.01e-10 * np.linalg.norm(b)
