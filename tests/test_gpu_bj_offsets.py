"""Places of block-Jacobi inverses of mixed precisions, found on the device in
one or several chunks of blocks, at the chunks' edges: precisions, inverses and
storage bytes as the oracle's, and the product through the offsets."""
import numpy as np
import pytest

from tests.test_gpu_bj_inplace import _blocks, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bs", [1, 2, 4])
@pytest.mark.parametrize("nblocks", [1, 2, 1023, 1024, 1025, 2049, 5000])
def test_offsets_of_mixed_precisions(nblocks, bs):
    rng = np.random.default_rng(nblocks + bs)
    scale = 10.0 ** rng.integers(-30, 6, nblocks)  # of the inverses: binary16, 32 and 64 by their range

    def make(b, m):
        return (np.eye(m) * 3.0 + rng.uniform(-0.3, 0.3, (m, m))) * scale[b]

    A, bp = _blocks(nblocks * bs - (bs > 2), bs, make)
    prec = _check(A, bp, bs)
    if nblocks > 1000:
        assert len(set(prec.tolist())) > 1
