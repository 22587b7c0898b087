"""The batched solve by size classes with larger systems beside them: classes
and the persistent kernel run on two streams between two events, from the
caller's stream, whichever it is, and from a captured graph."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests._gpu import DEV, dev
from tests.test_gpu_batch_classes import SIZES, _band, _batch, _solve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxl():
    import paper_2006_16852_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(mxl):
    return mxl.Context(0)


def _check(B, x, it, st):
    ref = O.batch_pcg(B, reduction=1e-10)
    assert np.all(st == 1) and np.all(np.abs(it - ref["iterations"]) <= 2)
    for s in range(B.nsys):
        r0, r1 = B.sys_ptr[s], B.sys_ptr[s + 1]
        r = B.b[r0:r1] - O.spmv(B.system(s), x[r0:r1])
        assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(B.b[r0:r1]), s


@pytest.mark.parametrize("half", [1, 3, 13])
def test_classes_alone(mxl, ctx, half):
    """Few systems, none too large for a class."""
    B = _batch([_band(n, half, 10 + k) for k, n in enumerate(SIZES) if n <= 1024])
    x, it, rel, st = _solve(mxl, ctx, B)
    _check(B, x, it, st)


@pytest.mark.parametrize("half,large", [(3, 1), (13, 30)])
def test_classes_with_larger_systems_beside(mxl, ctx, half, large):
    """More systems than CUs, some of more than 1,024 rows or wider than a class."""
    n = [s for s in SIZES if s <= 1024] * 17 + [1025, 1100, 1300, 2000] * large
    B = _batch([_band(m, half if k % 40 else 14, 10 + k) for k, m in enumerate(n)])
    assert B.nsys > torch.cuda.get_device_properties(0).multi_processor_count
    x, it, rel, st = _solve(mxl, ctx, B)
    _check(B, x, it, st)


def test_another_stream_and_a_graph(mxl, ctx):
    """The larger systems' stream starts after the caller's earlier work and ends
    before its later work: right-hand sides written just before each solve on a
    stream of the caller, and replays of a captured solve between eager ones."""
    n = [60, 200, 500, 900] * 70 + [1100, 1300, 1500] * 4
    B = _batch([_band(m, 4, 10 + k) for k, m in enumerate(n)])
    op = mxl.batch(ctx, B.sys_ptr, dev(B.sys_ptr), dev(B.row_ptr), dev(B.col), dev(B.val))
    src = [dev(W.uniform_vec(B.b.size, k)) for k in range(3)]
    b, x = torch.empty_like(src[0]), torch.empty_like(src[0])
    it = torch.zeros(B.nsys, dtype=torch.int32, device=DEV)
    rel = torch.zeros(B.nsys, dtype=torch.float64, device=DEV)
    st = torch.zeros(B.nsys, dtype=torch.uint8, device=DEV)

    def go():
        op.solve_noalloc(b, x, it, rel, st, reduction=1e-10)

    want = []
    for k in range(3):
        b.copy_(src[k])
        op.solve(b, x, it, rel, st, reduction=1e-10)
        torch.cuda.synchronize()
        want.append((x.clone(), it.clone()))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = []
        for k in range(3):
            b.copy_(src[k])
            go()
            got.append((x * 1.0, it * 1))  # later work of the stream, no synchronisation
    torch.cuda.synchronize()
    for (xa, ia), (xb, ib) in zip(want, got):
        assert torch.equal(xa, xb) and torch.equal(ia, ib)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        go()
    for k in (0, 1, 2, 0, 2):
        b.copy_(src[k])
        x.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, want[k][0]) and torch.equal(it, want[k][1])
        b.copy_(src[(k + 1) % 3])  # eager work between replays
        go()
        torch.cuda.synchronize()
        assert torch.equal(x, want[(k + 1) % 3][0])
