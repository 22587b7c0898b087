"""In-place inversion of uniform diagonal blocks against the oracle, bit for bit:
pivoting at every step, a short last block, mixed storage precisions found by
the look at some blocks, by the pass itself, and not at all, and blocks whose
elimination overflows (where zero entries must not pick up NaNs)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests._gpu import dev, matrix

pytestmark = pytest.mark.gpu


def _blocks(n, bs, make):
    """Block-diagonal matrix, block b filled by make(b, m)."""
    bp = O.uniform_blocks(n, bs)
    rp, val = [0], []
    for b in range(bp.size - 1):
        m = int(bp[b + 1] - bp[b])
        val.append(np.asarray(make(b, m), np.float64).reshape(-1))
        rp += [rp[-1] + m * (i + 1) for i in range(m)]
    sizes = np.diff(bp)
    col = np.concatenate([np.tile(np.arange(bp[b], bp[b + 1]), s) for b, s in enumerate(sizes)])
    return W.Csr(n, n, np.asarray(rp, np.int32), col.astype(np.int32), np.concatenate(val), f"blocks{n}_{bs}"), bp


def _check(A, bp, bs, adaptive=True):
    import paper_2006_16852_amd as mxl
    ctx = mxl.Context(0)
    inv, cond, prec = O.bj_generate(A, bp, adaptive=adaptive, accuracy=0.1)
    P = mxl.bjacobi(matrix(mxl, ctx, A), bs, adaptive=adaptive, accuracy=0.1)
    info = P.info(inverses=True)
    assert np.array_equal(info["precision"], prec)
    assert np.array_equal(info["inv"], inv, equal_nan=True)
    assert np.array_equal(info["cond"], cond, equal_nan=True)
    per = np.choose(prec, [8, 4, 2])
    assert info["storage_bytes"] == int(((bs * bs * per + 15) // 16 * 16).sum())
    if np.isfinite(inv).all():
        r = W.uniform_vec(A.nrows, 3)
        z = dev(np.zeros(A.nrows))
        P.apply(dev(r), z)
        want, absz = O.bj_apply(bp, inv, r), O.bj_apply(bp, np.abs(inv), np.abs(r))
        assert (np.abs(z.cpu().numpy() - want) <= 1e-13 * absz + 1e-300).all()
    return prec


@pytest.mark.parametrize("adaptive", [True, False])
@pytest.mark.parametrize("bs", [1, 2, 4, 8, 16, 32])
def test_pivots_at_every_step(bs, adaptive):
    rng = np.random.default_rng(bs)
    A, bp = _blocks(bs * 150 + bs // 2, bs, lambda b, m: rng.standard_normal((m, m)) * 10.0 ** rng.integers(-3, 4))
    _check(A, bp, bs, adaptive)


@pytest.mark.parametrize("case", ["look", "pass", "none"])
def test_precisions_of_a_large_storage(case):
    """8,300 blocks of 32: every eighth is looked at before the storage is made."""
    rng = np.random.default_rng(5)
    good = [np.eye(32) * 40 + rng.uniform(-1, 1, (32, 32)) for _ in range(8)]
    bad = good[0].copy()
    bad[:, 1] = bad[:, 0] + 1e-6 * bad[:, 1]

    def make(b, m):
        use_bad = (case == "look" and b % 3 == 0) or (case == "pass" and b == 8003)
        return (bad if use_bad else good[b % 8])[:m, :m]

    A, bp = _blocks(8300 * 32 - 5, 32, make)
    prec = _check(A, bp, 32)
    assert (len(set(prec.tolist())) > 1) == (case != "none")


@pytest.mark.parametrize("bs", [2, 8, 16, 32])
def test_overflowing_elimination(bs):
    def make(b, m):
        D = np.eye(m) * 3.0 + np.diag(np.ones(max(m - 1, 0)), 1) + np.diag(np.ones(max(m - 1, 0)), -1)
        if b == 2:  # 1 / pivot overflows in one row, the others have zeros there
            D[:, m - 1] = 0.0
            D[m - 1, :] = 0.0
            D[m - 1, m - 1] = 1e-310
        return D

    A, bp = _blocks(bs * 9, bs, make)
    _check(A, bp, bs)
