"""Streamed elastic product with several bursts per workgroup: its results collect in LDS, leave together, and the next
units' results take their place.  The same bits as an explicit tile, which keeps no results, with as many
units as fill the held ones (4, 2 and 1 of 64 grid rows by batch) more than twice, whole and with a rest; and
with so few slots and rows that long chains of products go to the tiles.
"""
import pytest
import torch

import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(20, 4700, 4, 200), (20, 2304, 3, 400), (40, 2400, 2, 300), (900, 64, 3, 60),
                                   (900, 65, 2, 60), (800, 256, 2, 16), (900, 10, 2, 30)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("store", [("f16", "f16", "auto"), ("bf16", "bf16", "bf16")], ids="-".join)
def test_several_bursts(shape, store):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    log_case("stream_bursts", shape=shape, store=store)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=32, g_dtype=store[0], f_dtype=store[1], products=store[2])
    s = to_dev(synth.gen_slip_batch(cfg, 0, 32))
    for B in (5, 8, 12, 20, 24, 32):
        op.set_tuning(gemm_cfg=-1)
        y = op.forward(s[:B])
        op.set_tuning(gemm_cfg=16)
        assert torch.equal(y, op.forward(s[:B])), f"B={B}"
