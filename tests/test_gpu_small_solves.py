"""CG and BiCGSTAB in one workgroup at the edges of their register shapes (rows
128 | 512 | 1024 | 2048 | 4096, entries a row 5 | 8 | 32), against the FP64
oracle after three iterations from a nonzero guess.

The sums differ from the oracle's by their order only: three steps on matrices
of condition below 10 keep rounding (1e-16 a step) under 1e-12 of max |x|.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests._gpu import dev, matrix

pytestmark = pytest.mark.gpu


def _matrix(n, width, seed, spd, drop_diagonal=()):
    """Rows of at most `width` entries: a band of offsets, symmetric when spd,
    and a diagonal that dominates; rows in drop_diagonal store none."""
    rng = np.random.default_rng(seed)
    h = (width - 1) // 2
    off = sorted(rng.choice(np.arange(1, min(n, 4 * h + 2)), h, replace=False))
    rows, cols, vals = [], [], []
    for d in off:
        i = np.arange(n - d)
        a = rng.uniform(-1, 1, n - d)
        rows += [i, i + d]
        cols += [i + d, i]
        vals += [a, a if spd else rng.uniform(-1, 1, n - d)]
    if not spd and width % 2 == 0:  # the last entry of an even width, one-sided
        d = 4 * h + 3
        rows, cols, vals = rows + [np.arange(n - d)], cols + [np.arange(d, n)], vals + [rng.uniform(-1, 1, n - d)]
    keep = np.setdiff1d(np.arange(n), np.asarray(drop_diagonal, int))
    rows.append(keep)
    cols.append(keep)
    vals.append(np.full(keep.size, 2.0 * len(off) + 1.0) + rng.uniform(0, 1, keep.size))
    r, c, v = np.concatenate(rows), np.concatenate(cols), np.concatenate(vals)
    o = np.lexsort((c, r))
    r, c, v = r[o], c[o], v[o]
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    return W.Csr(n, n, rp, c.astype(np.int32), v, f"band{n}w{width}")


SHAPES = [(63, 8), (128, 8), (129, 5), (512, 8), (513, 5), (1024, 5), (1024, 8), (1025, 5), (700, 32),
          (1024, 31), (2048, 5), (2048, 8), (2049, 5), (4096, 5)]


def _compare(solver, ref_fn, A, prec, reduction=1e-300, steps=3):
    import paper_2006_16852_amd as mxl
    ctx = mxl.Context(0)
    M = matrix(mxl, ctx, A)
    b, x0 = W.uniform_vec(A.nrows, 3), W.uniform_vec(A.nrows, 5)
    S = mxl.solver(solver, M, mxl.jacobi(M) if prec else None, max_iters=steps, reduction=reduction, launch_mode=2)
    x = dev(x0)
    info = S.solve(dev(b), x)
    ref = ref_fn(A, b, x0=x0, dinv=O.jacobi_dinv(A)[0] if prec else None, max_iters=steps, reduction=reduction)
    print(f"[{solver} {A.name}] {info['iterations']} {ref['iterations']}", flush=True)
    assert info["stop_reason"] == ref["stop_reason"] and info["iterations"] == ref["iterations"]
    err = np.abs(x.cpu().numpy() - ref["x"]).max()
    assert err <= 1e-12 * max(1.0, np.abs(ref["x"]).max()), err


@pytest.mark.parametrize("n,width", SHAPES)
def test_cg_shapes(n, width):
    _compare("cg", O.pcg, _matrix(n, width, n + width, True), True)


@pytest.mark.parametrize("n,width", [s for s in SHAPES if (s[1] <= 5 or s[1] == 8 and s[0] <= 1024)])
def test_bicgstab_shapes(n, width):
    _compare("bicgstab", O.bicgstab, _matrix(n, width, n + width, False), True)


@pytest.mark.parametrize("n,width", [(90, 8), (600, 5), (1024, 8), (4000, 5)])
def test_rows_without_a_diagonal(n, width):
    """Such rows keep another entry in the slot that the diagonal has elsewhere."""
    A = _matrix(n, width, 7, False, drop_diagonal=[0, 5, n // 2, n - 1])
    _compare("bicgstab", O.bicgstab, A, False, steps=2)


@pytest.mark.parametrize("A", [W.stencil_3d27(12), W.stencil_2d5(70), W.stencil_2d5(90)], ids=lambda a: a.name)
def test_auto_beyond_the_register_shapes(A):
    """Up to 35,000 stored entries one workgroup, beyond one kernel per step."""
    import paper_2006_16852_amd as mxl
    ctx = mxl.Context(0)
    M = matrix(mxl, ctx, A)
    b = O.spmv(A, W.uniform_vec(A.nrows, 1))
    ref = O.pcg(A, b, dinv=O.jacobi_dinv(A)[0], reduction=1e-10, max_iters=5000)
    S = mxl.solver("cg", M, mxl.jacobi(M), max_iters=5000, reduction=1e-10)
    for _ in range(2):  # the second solve of a solver takes the route decided by the first
        x = dev(np.zeros(A.nrows))
        info = S.solve(dev(b), x)
        assert info["stop_reason"] == ref["stop_reason"]
        assert abs(info["iterations"] - ref["iterations"]) <= max(2, int(0.02 * ref["iterations"]))
        assert np.linalg.norm(b - O.spmv(A, x.cpu().numpy())) <= 1.01e-10 * np.linalg.norm(b)
