"""Automatic tiles of the float32 products where slots and rows are few, so that the tile is chosen by the workgroups
it gives: the same bits as explicit tiles (grid-row ranges fixed) for batches around every width, and one operator
on its own against the oracle (rel-L2 <= 1e-5) at row counts on both sides of a round of workgroups.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import log_case, make_operator, to_dev
from paper_2608_21763_amd import BLTTOperator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(70, 1000, 40, 16), (900, 300, 40, 16), (40, 2400, 33, 30), (300, 1100, 70, 60)],
                         ids=lambda s: "x".join(map(str, s)))
def test_same_bits(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    log_case("batched32_few_slots", shape=shape)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=130, layout="batched")
    op.set_tuning(gemm32_splits=2, adj32_splits=2)
    s = to_dev(synth.gen_slip_batch(cfg, 0, 130))
    r = to_dev(synth.normals(cfg.seed, "r", 3, (130, nobs, nt)).astype(np.float32))
    for B in (8, 16, 32, 53, 64, 100, 130):
        op.set_tuning(gemm32_cfg=-1, gemm32_cfg_k=-1, adj32_cfg=-1)
        y, gs = op.forward(s[:B]), op.adjoint(r[:B])
        op.set_tuning(gemm32_cfg=4, gemm32_cfg_k=2, adj32_cfg=3)
        assert torch.equal(y, op.forward(s[:B])), f"B={B}"
        assert torch.equal(gs, op.adjoint(r[:B])), f"adjoint B={B}"


@pytest.mark.parametrize("sizes", [(4096, 20, 3), (4097, 20, 3), (30, 4200, 5), (2049, 33, 20)],
                         ids=lambda s: "x".join(map(str, s)))
def test_one_operator(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nrow, ncol, nt = sizes
    log_case("bltt_few_slots", sizes=sizes)
    rng = np.random.default_rng(nrow)
    K = rng.standard_normal((nrow, ncol, nt)).astype(np.float32)
    op = BLTTOperator(nrow, ncol, nt, max_batch=64)
    op.set_blocks(to_dev(K), 0)
    x = rng.standard_normal((64, ncol, nt)).astype(np.float32)
    v = rng.standard_normal((64, nrow, nt)).astype(np.float32)
    y, a = op.apply(to_dev(x)).cpu().numpy().astype(np.float64), op.adjoint(to_dev(v)).cpu().numpy().astype(np.float64)
    for b in (0, 31, 63):
        ref = oracle.bltt(K.astype(np.float64), x[b].astype(np.float64))
        assert oracle.rel_l2(y[b], ref) <= 1e-5
        lhs, rhs = np.vdot(y[b], v[b]), np.vdot(x[b], a[b])
        assert abs(lhs - rhs) <= 1e-6 * np.linalg.norm(y[b]) * np.linalg.norm(v[b])
