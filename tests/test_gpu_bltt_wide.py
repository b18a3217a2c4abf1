"""One operator of more than 1,024 columns on one to four inputs: on both sides of every width of its column chunks
and of every number of them, rows that take one row chunk of 128 or leave a second one, fewer rows than
wavefronts.  Bound: rel-L2 <= 1e-5 per input against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import log_case, to_dev
from paper_2608_21763_amd import BLTTOperator

pytestmark = pytest.mark.gpu

SHAPES = [(4, 1025, 20), (3, 1280, 20), (9, 1281, 20), (5, 1536, 20), (5, 1537, 20), (30, 1792, 20), (30, 1793, 20),
          (11, 1921, 33), (11, 2048, 33), (11, 2049, 33), (7, 2688, 16), (7, 2689, 16), (1, 5400, 16),
          (4200, 1030, 2), (8300, 1100, 1), (3, 1100, 300)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_bltt_wide(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nrow, ncol, nt = shape
    log_case("bltt_wide", shape=shape)
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
