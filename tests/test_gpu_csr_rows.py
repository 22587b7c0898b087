"""The CSR operator as wrapped (runs of rows staged in LDS), as row blocks and as
COO at the edges of runs, blocks and tiles, against the FP64 oracle: rows of
exactly, just under and just over the 320 or 512 entries of a run, runs cut
inside a block of rows, equal and unequal rows, empty rows, a last block that
is not full.

Tolerance per row: 1e-12 (FP64), 1e-5 (FP32) of |alpha| sum |a||x| + |beta||y|.
"""
import numpy as np
import pytest
import torch

import workloads as W
from tests._gpu import DEV, assert_rows_close, dev, matrix, spmv_reference

pytestmark = pytest.mark.gpu


def _rows(lengths, ncols, seed):
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    row = np.repeat(np.arange(len(lengths)), lengths)
    col = ((17 * row + 3 * (np.arange(rp[-1]) - rp[row])) % ncols).astype(np.int32)
    return W.Csr(len(lengths), ncols, rp, col, rng.uniform(-1, 1, col.size))


LENGTHS = {
    "one_row": [512],
    "cap_edges": [511, 512, 513, 1, 1024, 1025, 0, 512, 512],
    "equal_runs": [27] * 3001,
    "equal_last_block": [8] * (64 * 9 + 1),
    "unequal": list(np.random.default_rng(2).integers(0, 90, 2500)),
    "one_long": [5] * 900 + [4000] + [5] * 900,
    "empty_ends": [0] * 70 + [300] * 30 + [0] * 70,
    "one_a_run": [400] * 130,
    # 64 rows a wave whatever their length (1,048,576 rows and more): several runs in a block of rows
    "two_runs_a_block": [9] * (64 * 16384 + 5),
    "two_runs_a_block_unequal": list(np.random.default_rng(4).integers(0, 20, 64 * 16384 + 70)),
    "runs_in_block_equal": [27] * (64 * 4096 + 5),
    "runs_in_block_unequal": list(np.random.default_rng(3).integers(0, 40, 64 * 4096 + 70)),
    # at most 5 entries a row: runs of 320
    "short_runs": [5] * (64 * 4096 + 3),
    "short_runs_long": ([320, 321, 319, 513] + [3, 4, 5, 6] * 40 + [0] * 300) * 6,
    "runs_in_block_long": [20] * 130000 + [700, 513, 512] + [20] * 135000,
}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("op", ["wrapped", "row_blocks", "coo"])
@pytest.mark.parametrize("name", LENGTHS)
def test_csr_rows_edges(name, op, dtype):
    import paper_2006_16852_amd as mxl
    A = _rows(LENGTHS[name], 5003, 11)
    A0 = matrix(mxl, mxl.Context(0), A, dtype)
    op = {"wrapped": lambda: A0, "row_blocks": lambda: A0.convert("csr", variant=mxl.CSR_STREAM),
          "coo": lambda: A0.convert("coo")}[op]()
    rng = np.random.default_rng(7)
    x, y0 = rng.uniform(-1, 1, A.ncols), rng.uniform(-1, 1, A.nrows)
    fp32 = dtype == torch.float32
    for alpha, beta in [(1.0, 0.0), (0.5, -2.0)]:
        y = dev(y0, dtype) if beta else torch.full((A.nrows,), float("nan"), dtype=dtype, device=DEV)
        op.apply(dev(x, dtype), y, alpha, beta)
        want, bound = spmv_reference(A, x, alpha, beta, y0, fp32)
        assert_rows_close(y.cpu().numpy(), want, bound, 1e-5 if fp32 else 1e-12, f"{name} {alpha} {beta}")
