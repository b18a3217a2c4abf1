"""Direct layout where the sum of its partials turns from 32 threads per sum to 16, 8, 4 and 1, with more partials than
threads and fewer, forward and adjoint.  Bound: rel-L2 <= 1e-5 (the float32 bar) against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(60, 100, 3, 100), (200, 60, 3, 200), (260, 33, 2, 106), (500, 40, 2, 130), (964, 40, 2, 117), (964, 17, 2, 256),
          (3, 900, 2, 250), (1, 40, 1, 5), (2, 7, 3, 300)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_direct_sums(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    log_case("direct_sums", shape=shape)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=1, layout="direct", dt=0.5)
    s = synth.gen_slip_batch(cfg, 0, 1)
    r = synth.normals(cfg.seed, "r", 1, (1, nobs, nt)).astype(np.float32)
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    y, m = op.forward_displacement(to_dev(s))
    ey = oracle.rel_l2_per_rupture(y.cpu().numpy(), oracle.forward(G, F, s, dt=0.5, diff=1)).max()
    em = oracle.rel_l2_per_rupture(m.cpu().numpy(), oracle.bltt(G, s)).max()
    eg = oracle.rel_l2_per_rupture(op.adjoint(to_dev(r)).cpu().numpy(), oracle.adjoint(G, F, r, dt=0.5, diff=1)).max()
    print(f"{shape}: forward {ey:.2e}, displacement {em:.2e}, adjoint {eg:.2e}")
    assert max(ey, em, eg) <= 1e-5
