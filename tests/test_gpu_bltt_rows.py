"""One operator on one to four inputs at the edges of the row kernels: columns on both sides of every
register row (256, 384, 512, 1024 and past it), rows around the 128 that leave LDS together and fewer rows
than wavefronts.  Bound: rel-L2 <= 1e-5 per input against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import log_case, to_dev
from paper_2608_21763_amd import BLTTOperator

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 20), (3, 255, 20), (127, 256, 20), (128, 257, 16), (50, 384, 20), (50, 385, 20), (129, 511, 20), (300, 513, 20), (70, 1024, 20),
          (70, 1025, 20), (20, 1920, 16), (9, 2100, 16), (1100, 40, 60), (40, 30, 256)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_bltt_rows(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nrow, ncol, nt = shape
    log_case("bltt_rows", shape=shape)
    rng = np.random.default_rng(nrow * 10000 + ncol)
    K = rng.standard_normal((nrow, ncol, nt)).astype(np.float32)
    x = rng.standard_normal((4, ncol, nt)).astype(np.float32)
    op = BLTTOperator(nrow, ncol, nt, max_batch=4)
    op.set_blocks(to_dev(K), 0)
    ref = np.stack([oracle.bltt(K.astype(np.float64), x[b].astype(np.float64)) for b in range(4)])
    xd = to_dev(x)
    for B in (1, 2, 3, 4):
        err = oracle.rel_l2_per_rupture(op.apply(xd[:B]).cpu().numpy(), ref[:B]).max()
        print(f"{shape} B={B}: {err:.2e}")
        assert err <= 1e-5
