"""Streamed products of the half-precision path (up to 32 ruptures) against the tiled ones.

Both take every output's products in the same order, so with the default tiles and with an explicit
tile (which switches the streamed kernels and the [l][g][b] workspace order off) the waveforms must be
the same bits, for grid-row counts on both sides of the 16-row blocks, the 64-row units and the
ranges of a workgroup, observer counts around the 16-row groups, every transform length and
batches around every column count; one rupture is held against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import half_limit, log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(5, 1, 1, 250), (37, 15, 3, 20), (16, 16, 16, 60), (963, 17, 17, 256), (33, 63, 64, 100), (130, 64, 70, 250),
          (60, 65, 5, 400), (300, 257, 33, 512), (48, 1100, 20, 200)]
STORES = [("bf16", "f16", "auto"), ("f16", "bf16", "auto"), ("bf16", "bf16", "bf16")]


@pytest.mark.parametrize("store", STORES, ids=["-".join(s) for s in STORES])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_streamed_products(shape, store):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    log_case("small_batches", shape=shape, store=store)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=40, dt=0.5, g_dtype=store[0], f_dtype=store[1], products=store[2])
    s = to_dev(synth.gen_slip_batch(cfg, 0, 40))
    for B in (1, 7, 8, 9, 16, 17, 24, 25, 32, 33):
        op.set_tuning(gemm_cfg=-1)
        y = op.forward(s[:B])
        yd, _ = op.forward_displacement(s[:B], [nt - 1])
        op.set_tuning(gemm_cfg=16)
        ref = op.forward(s[:B])
        assert torch.equal(y, ref), f"B={B}"
        assert torch.equal(yd, ref), f"B={B} with displacement"
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    op.set_tuning(gemm_cfg=-1)
    y = op.forward(s[:1]).cpu().numpy()
    err = oracle.rel_l2_per_rupture(y, oracle.forward(G, F, s[:1].cpu().numpy(), dt=0.5, diff=1)).max()
    print(f"{shape} {store}: {err:.2e}")
    assert err <= half_limit("bf16" if "bf16" in store[:2] else "f16", store[1])
