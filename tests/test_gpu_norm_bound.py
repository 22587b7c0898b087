"""The solves inside one workgroup compare squares where tol^2 = (reduction
||b||)^2 lies in (1e-290, 1e290) and roots elsewhere.  Right-hand sides so large
and so small that tol^2 leaves the range (checked on the host) while the dots
stay finite and normal: the same iterations as the oracle, which takes roots."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests._gpu import dev, matrix
from tests.test_gpu_batch_classes import _band, _batch, _solve
from tests.test_gpu_small_solves import _matrix

pytestmark = pytest.mark.gpu

SCALES = [(1e148, 1e-3), (1e-140, 1e-10)]


def _outside(b, reduction):
    tol = reduction * np.sqrt(float((b * b).sum()))
    return not 1e-290 < tol * tol < 1e290


@pytest.mark.parametrize("scale,reduction", SCALES)
def test_batch_classes(scale, reduction):
    import paper_2006_16852_amd as mxl
    B = _batch([_band(n, 3, 5 + n) for n in (40, 100, 300, 600, 1000)])
    B.b *= scale
    assert all(_outside(B.b[B.sys_ptr[s]:B.sys_ptr[s + 1]], reduction) for s in range(B.nsys))
    ref = O.batch_pcg(B, reduction=reduction)
    x, it, rel, st = _solve(mxl, mxl.Context(0), B, reduction=reduction)
    assert np.all(st == 1) and np.all(np.abs(it - ref["iterations"]) <= 1), (it, ref["iterations"])
    for s in range(B.nsys):
        r0, r1 = B.sys_ptr[s], B.sys_ptr[s + 1]
        r = (B.b[r0:r1] - O.spmv(B.system(s), x[r0:r1])) / scale
        assert np.linalg.norm(r) <= 1.01 * reduction * np.linalg.norm(B.b[r0:r1] / scale), s


@pytest.mark.parametrize("scale,reduction", SCALES)
@pytest.mark.parametrize("kind", ["cg", "bicgstab"])
@pytest.mark.parametrize("n,width", [(100, 8), (900, 5), (4000, 5)])
def test_small_solves(n, width, kind, scale, reduction):
    import paper_2006_16852_amd as mxl
    A = _matrix(n, width, n, kind == "cg")
    b = W.uniform_vec(n, 3) * scale
    assert _outside(b, reduction)
    ref = getattr(O, "pcg" if kind == "cg" else kind)(A, b, dinv=O.jacobi_dinv(A)[0], max_iters=500, reduction=reduction)
    M = matrix(mxl, mxl.Context(0), A)
    S = mxl.solver(kind, M, mxl.jacobi(M), max_iters=500, reduction=reduction, launch_mode=2)
    x = dev(np.zeros(n))
    info = S.solve(dev(b), x)
    assert info["stop_reason"] == ref["stop_reason"] == mxl.STOP_CONVERGED
    assert abs(info["iterations"] - ref["iterations"]) <= 1, (info["iterations"], ref["iterations"])
    r = (b - O.spmv(A, x.cpu().numpy())) / scale
    assert np.linalg.norm(r) <= 1.01 * reduction * np.linalg.norm(b / scale)
