"""The direct layout at the edges of its row tiles: observers and subfaults on both sides of 16, 32, 64
and 128 rows, channel counts that leave some of a tile's wave groups without a channel, record lengths
around the blocks of 16 and past 256 steps, with and without the time derivative, forward, adjoint and
displacement.  Bound: rel-L2 <= 1e-5 against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

# nsub, ngrid, nobs, nt, differentiate
CASES = [(1, 1, 1, 1, 1), (3, 67, 15, 16, 1), (15, 130, 16, 17, 0), (16, 129, 17, 33, 1),
         (17, 65, 31, 100, 1), (32, 300, 32, 47, 1), (33, 2100, 33, 20, 0), (64, 1030, 4, 200, 1),
         (65, 90, 64, 257, 1), (129, 70, 65, 300, 0), (20, 40, 16, 512, 1)]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_direct_rows(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt, diff = case
    log_case("direct_rows", case=case)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=2, dt=0.5, diff=diff, layout="direct")
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    s = np.random.default_rng(nsub * 1000 + nt).standard_normal((2, nsub, nt)).astype(np.float32)
    r = np.random.default_rng(nobs * 1000 + nt).standard_normal((2, nobs, nt)).astype(np.float32)
    cols = sorted({0, nt - 1})
    y, m = op.forward_displacement(to_dev(s), cols)
    assert torch.equal(y, op.forward(to_dev(s)))
    gs = op.adjoint(to_dev(r))
    pairs = {"forward": (y, oracle.forward(G, F, s, dt=0.5, diff=diff)),
             "displacement": (m, oracle.bltt(G, s)[:, :, cols]),
             "adjoint": (gs, oracle.adjoint(G, F, r, dt=0.5, diff=diff))}
    for what, (got, ref) in pairs.items():
        err = oracle.rel_l2_per_rupture(got.cpu().numpy().astype(np.float64), ref).max()
        print(f"{case} {what}: {err:.2e}")
        assert err <= 1e-5, what
