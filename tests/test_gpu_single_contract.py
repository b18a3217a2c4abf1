"""Single layout where its shape rules turn.  Grid-row contraction: column counts with 16, 8 and 4 columns
per thread, with the fewest and the most row ranges, last column blocks that are not full, at every slot count
it divides differently.  Fused forward and the adjoint's row stage: one and two workgroups per CU on both sides
of 16 observers per thread, and at 512 slots.  Bound: rel-L2 <= 1e-5 (the float32 bar) against the oracle, adjoint and, for many
observers, the unfused forward.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(96, 300, 2, 130), (97, 300, 2, 130), (48, 300, 2, 130), (49, 300, 2, 130), (289, 260, 2, 130),
          (1024, 260, 1, 130), (200, 900, 2, 16), (768, 900, 1, 16), (1000, 300, 1, 40), (24, 260, 256, 260),
          (24, 260, 140, 129), (1024, 230, 1, 300),
          (3, 4100, 128, 40), (3, 4100, 129, 40), (2, 4100, 2, 258), (2, 4100, 17, 257)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_single_contract(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    log_case("single_contract", shape=shape)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=1, layout="single", dt=0.5)
    s = synth.gen_slip_batch(cfg, 0, 1)
    r = synth.normals(cfg.seed, "r", 1, (1, nobs, nt)).astype(np.float32)
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    ey = oracle.rel_l2_per_rupture(op.forward(to_dev(s)).cpu().numpy(), oracle.forward(G, F, s, dt=0.5, diff=1)).max()
    eg = oracle.rel_l2_per_rupture(op.adjoint(to_dev(r)).cpu().numpy(), oracle.adjoint(G, F, r, dt=0.5, diff=1)).max()
    print(f"{shape}: forward {ey:.2e}, adjoint {eg:.2e}")
    assert ey <= 1e-5 and eg <= 1e-5
