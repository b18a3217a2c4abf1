"""Float32 acoustic products of at most 32 observers (register kernel) against the tiles.

With the grid-row ranges fixed both add the same products in the same order, so the waveforms must
have the same bits: observers on both sides of 16 and 32, grid rows around the chunks of 8 and the
four chunks held, more ranges than chunks, batches at every width of 8 and past 64.
"""
import pytest
import torch

import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(2, 1, 1, 20, 1), (3, 7, 15, 20, 3), (2, 8, 16, 300, 2), (2, 33, 17, 20, 1), (4, 65, 31, 100, 2),
          (2, 200, 32, 200, 4), (2, 129, 33, 40, 2)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_few_rows_bit_identical(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt, splits = shape
    log_case("batched32_few", shape=shape)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=130, layout="batched", dt=0.5)
    s = to_dev(synth.gen_slip_batch(cfg, 0, 130))
    op.set_tuning(gemm32_splits=splits)
    for B in (1, 7, 8, 9, 24, 25, 40, 48, 56, 63, 64, 65, 72, 130):
        op.set_tuning(gemm32_cfg_k=-1)
        y = op.forward(s[:B])
        op.set_tuning(gemm32_cfg_k=4)
        assert torch.isfinite(y).all() and torch.equal(y, op.forward(s[:B])), f"B={B}"
