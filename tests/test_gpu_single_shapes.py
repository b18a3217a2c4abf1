"""Single-layout kernels at the edges of their tile choices: column counts on both sides of every rule
of the grid-row contraction (16, 8 and 4 columns per thread), row counts that leave remainders of
its unrolled rows and of the row tiles, and fewer rows than workgroups.  Bound: rel-L2 <= 1e-5 (the
float32 bar) against the oracle, forward and adjoint.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(nsub, ngrid, nobs, nt)
          for nsub, nobs, nt in [(3, 2, 200), (60, 4, 200), (450, 5, 256), (33, 7, 100), (60, 3, 20), (17, 6, 400)]
          for ngrid in (1, 5, 17, 133)] + [(20, 300, 70, 256), (9, 1030, 3, 64), (450, 2100, 2, 16)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_single_shapes(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    log_case("single_shapes", shape=shape)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=1, layout="single", dt=0.5)
    s = synth.gen_slip_batch(cfg, 0, 1)
    r = synth.normals(cfg.seed, "r", 1, (1, nobs, nt)).astype(np.float32)
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    ey = oracle.rel_l2_per_rupture(op.forward(to_dev(s)).cpu().numpy(), oracle.forward(G, F, s, dt=0.5, diff=1)).max()
    eg = oracle.rel_l2_per_rupture(op.adjoint(to_dev(r)).cpu().numpy(), oracle.adjoint(G, F, r, dt=0.5, diff=1)).max()
    print(f"{shape}: forward {ey:.2e}, adjoint {eg:.2e}")
    assert ey <= 1e-5 and eg <= 1e-5
