"""Automatic tiles of the float32 batched products against the four explicit shapes.

With the grid-row ranges fixed every tile adds the same products in the same order, so forward and
adjoint must give the same bits for batches around every tile width and for row counts on both
sides of the 64-, 128- and 256-row rules; one batch per shape is held against the oracle (1e-5).
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(5, 1, 1, 20), (60, 63, 17, 60), (130, 65, 64, 100), (300, 130, 70, 250), (18, 700, 33, 30), (450, 40, 5, 400)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_tiles_bit_identical(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    log_case("batched32_tiles", shape=shape)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=100, layout="batched", dt=0.5)
    op.set_tuning(gemm32_splits=2, adj32_splits=2)
    s = to_dev(synth.gen_slip_batch(cfg, 0, 100))
    r = to_dev(synth.normals(cfg.seed, "r", 3, (100, nobs, nt)).astype(np.float32))
    for B in (1, 8, 9, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49, 56, 57, 64, 65, 100):
        op.set_tuning(gemm32_cfg=-1, gemm32_cfg_k=-1, adj32_cfg=-1)
        y, gs = op.forward(s[:B]), op.adjoint(r[:B])
        op.set_tuning(gemm32_cfg=2, gemm32_cfg_k=4, adj32_cfg=1)
        assert torch.equal(y, op.forward(s[:B])), f"B={B}"
        assert torch.equal(gs, op.adjoint(r[:B])), f"adjoint B={B}"
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    ey = oracle.rel_l2_per_rupture(y[:3].cpu().numpy(), oracle.forward(G, F, s[:3].cpu().numpy(), dt=0.5, diff=1)).max()
    eg = oracle.rel_l2_per_rupture(gs[:3].cpu().numpy(), oracle.adjoint(G, F, r[:3].cpu().numpy(), dt=0.5, diff=1)).max()
    print(f"{shape}: forward {ey:.2e}, adjoint {eg:.2e}")
    assert ey <= 1e-5 and eg <= 1e-5
