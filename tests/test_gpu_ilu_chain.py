"""Exact triangular solves along chains of rows (runs of rows that depend on
their neighbour), at the edges of their plan: groups of chains cut short,
tiles of chains with and without skew, a numbering whose tiles would wait in
a circle, operands beyond a group's LDS places, rows wider than a record,
chains too short for the method.  Every row does the oracle's operations in
its order, so all of them equal the oracle bit for bit."""
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


def _from_pairs(n, pairs, seed, name):
    """Diagonally dominant matrix with the given (row, col) entries."""
    rng = np.random.default_rng(seed)
    key = np.unique(np.concatenate([np.array([r * n + c for r, c in pairs], np.int64),
                                    np.arange(n, dtype=np.int64) * (n + 1)]))
    r, c = key // n, key % n
    v = rng.uniform(-1.0, 1.0, key.size)
    s = np.bincount(r, weights=np.abs(v), minlength=n) + 1.0
    v[r == c] = s
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    return W.Csr(n, n, rp, c.astype(np.int32), v, name)


def _broken_chains(n=3000, seed=2):
    """Neighbour couplings dropped at random (chains of 1 to ~100 rows, others
    in L than in U) and a few distant couplings."""
    rng = np.random.default_rng(seed)
    p = [(i, i - 1) for i in range(1, n) if rng.random() > 0.04]
    p += [(i, i + 1) for i in range(n - 1) if rng.random() > 0.04]
    p += [(int(a), int(b)) for a, b in rng.integers(0, n, (n // 2, 2))]
    return _from_pairs(n, p, seed, "broken_chains")


def _circle(W_=24, K=24, L=12, seed=5):
    """Lines of L rows; line t couples to lines t - 1, t - W and t - W + 3:
    two-dimensional tiles of lines are not in order for every tile shape."""
    n = W_ * K * L
    p = []
    for i in range(n):
        t = i // L
        if i % L:
            p += [(i, i - 1), (i - 1, i)]
        for o in (1, W_, W_ - 3):
            if t >= o:
                p += [(i, i - o * L), (i - o * L, i)]
    return _from_pairs(n, p, seed, "circle")


def _wide(n=400, half=16, seed=7):
    return _from_pairs(n, [(i, j) for i in range(n) for j in range(max(0, i - half), min(n, i + half + 1))], seed, "wide")


def _random(n=900, seed=9):
    rng = np.random.default_rng(seed)
    return _from_pairs(n, [(int(a), int(b)) for a, b in rng.integers(0, n, (4 * n, 2))], seed, "short_chains")


CASES = {
    "one_row": lambda: _from_pairs(1, [], 1, "one"),
    "one_chain_beyond_lds": lambda: _from_pairs(20_000, [(i, i - 1) for i in range(1, 20_000)] +
                                                [(i - 1, i) for i in range(1, 20_000)] +
                                                [(i, i - 3) for i in range(3, 20_000, 2)], 3, "tri"),
    "lines_2d": lambda: W.convdiff_2d5(71),
    "tiles_3d7": lambda: W.convdiff_3d7(19),
    "tiles_3d27_skewed": lambda: W.stencil_3d27(18),
    "flat_grid": lambda: W.stencil_grid(40, 9, 9, *W.points_convdiff3d()),
    "broken_chains": _broken_chains,
    "tiles_out_of_order": _circle,
    "rows_wider_than_a_record": _wide,
    "short_chains": _random,
}


@pytest.mark.parametrize("name", list(CASES))
def test_exact_solves_bitwise(mxl, ctx, name):
    A = CASES[name]()
    P = mxl.ilu(matrix(mxl, ctx, A), sweeps=2)
    lu = P.info(factors=True)["lu"]
    r = W.uniform_vec(A.nrows, 5)
    want = O.ilu_apply(A, lu, r, mode=0, sweeps=0)
    z = torch.empty(A.nrows, dtype=torch.float64, device=DEV)
    for _ in range(2):  # a second application starts from the first one's work vectors
        z.fill_(7.0)
        P.apply(dev(r), z)
        assert np.array_equal(z.cpu().numpy(), want)


def test_nonfinite_right_hand_side_ends(mxl, ctx):
    """NaN and Inf pass through the substitution as in the oracle: the same
    entries are non-finite and the others equal bit for bit."""
    A = W.convdiff_3d7(13)
    P = mxl.ilu(matrix(mxl, ctx, A), sweeps=2)
    r = W.uniform_vec(A.nrows, 5)
    # the third is the pattern the kernel uses for "not solved yet"
    r[700], r[1500] = np.nan, np.inf
    r[1900] = np.array([0x7FF4A5A55A5A5A5A], np.uint64).view(np.float64)[0]
    want = O.ilu_apply(A, P.info(factors=True)["lu"], r, mode=0, sweeps=0)
    z = torch.empty(A.nrows, dtype=torch.float64, device=DEV)
    P.apply(dev(r), z)
    got = z.cpu().numpy()
    fin = np.isfinite(want)
    assert np.array_equal(fin, np.isfinite(got)) and np.array_equal(got[fin], want[fin])
