"""The batched solve by size classes (no schedule given): systems at the edges
of every class, wider than the register rows, larger than the largest class,
against the oracle's per-system PCG and against the persistent kernel."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests._gpu import DEV, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxl():
    import paper_2006_16852_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(mxl):
    return mxl.Context(0)


def _band(n, half, seed):
    """Symmetric, strictly dominant band with random gaps (so rows are padded)."""
    rng = np.random.default_rng(seed)
    rows, cols, vals = [], [], []
    for d in range(1, min(half, n - 1) + 1):
        a = np.arange(n - d)
        keep = rng.random(n - d) < 0.9
        a = a[keep]
        v = rng.standard_normal(a.size)
        rows += [a, a + d]
        cols += [a + d, a]
        vals += [v, v]
    r = np.concatenate(rows + [np.arange(n)])
    c = np.concatenate(cols + [np.arange(n)])
    v = np.concatenate(vals + [np.zeros(n)])
    v[-n:] = np.bincount(r, weights=np.abs(v), minlength=n) + 1.0
    o = np.lexsort((c, r))
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    return W.Csr(n, n, rp, c[o].astype(np.int32), v[o], f"band{n}_{half}")


def _batch(systems, seed=3):
    sp = np.concatenate([[0], np.cumsum([A.nrows for A in systems])]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum([A.nnz for A in systems])])
    rp = np.concatenate([A.row_ptr[:-1] + o for A, o in zip(systems, off)] + [[off[-1]]]).astype(np.int32)
    return W.Batch(len(systems), sp, rp, np.concatenate([A.col for A in systems]).astype(np.int32),
                   np.concatenate([A.val for A in systems]), W.uniform_vec(int(sp[-1]), seed))


def _solve(mxl, ctx, B, tuning=None, **crit):
    op = mxl.batch(ctx, B.sys_ptr, dev(B.sys_ptr), dev(B.row_ptr), dev(B.col), dev(B.val))
    b = dev(B.b)
    x = torch.full_like(b, 3.0)  # not read: every system starts from zero
    it = torch.zeros(B.nsys, dtype=torch.int32, device=DEV)
    rel = torch.zeros(B.nsys, dtype=torch.float64, device=DEV)
    st = torch.zeros(B.nsys, dtype=torch.uint8, device=DEV)
    op.solve(b, x, it, rel, st, tuning=tuning, **({"reduction": 1e-10} | crit))
    return [t.cpu().numpy() for t in (x, it, rel, st)]


SIZES = [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 1300]


@pytest.mark.parametrize("half", [1, 3, 13, 14], ids=["w3", "w7", "w27", "w29_rest"])
def test_class_edges(mxl, ctx, half):
    B = _batch([_band(n, half, 10 + k) for k, n in enumerate(SIZES)])
    ref = O.batch_pcg(B, reduction=1e-10)
    x, it, rel, st = _solve(mxl, ctx, B)
    assert np.all(st == 1) and np.all(np.abs(it - ref["iterations"]) <= 2)
    for s in range(B.nsys):
        r0, r1 = B.sys_ptr[s], B.sys_ptr[s + 1]
        r = B.b[r0:r1] - O.spmv(B.system(s), x[r0:r1])
        assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(B.b[r0:r1]), s


def test_same_stops_as_the_persistent_kernel(mxl, ctx):
    """Zero, NaN and Inf right-hand sides, an iteration limit and systems that
    break down stop as the persistent kernel stops them."""
    sys_ = [_band(n, 4, 40 + n) for n in (5, 64, 70, 200, 300, 600, 1000)]
    indef = _band(90, 2, 7)
    indef.val[:] = -indef.val  # negative definite: p.Ap < 0 in the first step
    B = _batch(sys_ + [indef])
    for s, v in ((1, 0.0), (2, np.nan), (3, np.inf)):
        B.b[B.sys_ptr[s]:B.sys_ptr[s + 1]] = v
    for crit in (dict(), dict(max_iters=3), dict(nonfinite_check=0, max_iters=5), dict(reduction=0.0, max_iters=4)):
        x1, it1, rel1, st1 = _solve(mxl, ctx, B, None, **crit)
        x2, it2, rel2, st2 = _solve(mxl, ctx, B, (256, 2, 0, 2), **crit)
        assert np.array_equal(st1, st2) and np.array_equal(it1, it2), (crit, st1, st2, it1, it2)
        assert np.array_equal(np.isnan(x1), np.isnan(x2)) and np.array_equal(np.isnan(rel1), np.isnan(rel2))


def test_large_entries_meet_the_criterion_by_its_root(mxl, ctx):
    """||b|| so large that its square leaves the range in which the criterion
    is compared on squares."""
    B = _batch([_band(100, 3, 5), _band(300, 3, 6)])
    B.b *= 1e148
    ref = O.batch_pcg(B, reduction=1e-10)
    x, it, rel, st = _solve(mxl, ctx, B)
    assert np.all(st == 1) and np.all(np.abs(it - ref["iterations"]) <= 2)
