"""Single layout: the one-launch sum and inverse transform at every transform length and on both sides of
its limit, and the fused kernel's choice of workgroups and tile rows (fewer tiles than compute units,
one and two workgroups per unit) against the oracle at the float32 bar, rel-L2 <= 1e-5; the call
without a workspace agrees bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

# nsub, ngrid, nobs, nt, tuning: two workgroups per unit start at 16 rows per unit and end past 160 subfaults
CASES = [(2, 3, 1, 7, {}), (5, 129, 3, 16, {}), (7, 1025, 5, 33, {}), (4, 700, 70, 17, {}), (3, 260, 2, 100, {}),
         (3, 1100, 2, 256, {}), (2, 4096, 1, 200, {}), (2, 4095, 1, 200, {}), (160, 4100, 2, 20, {}),
         (161, 4100, 2, 20, {}), (3, 130, 2, 300, {}), (3, 300, 2, 256, {"fused_wg_per_cu": 4}),
         (3, 300, 2, 64, {"fused_wg_per_cu": 2, "fused_rows": 4})]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c[:4])) + "".join(f"-{v}" for v in c[4].values())
                                             for c in CASES])
def test_single_sums(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt, tune = case
    log_case("single_sums", case=case)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=2, layout="single", dt=0.5)
    if tune:
        op.plan.set_tuning(**tune)
    s = synth.gen_slip_batch(cfg, 0, 2)
    r = synth.normals(cfg.seed, "r", 2, (2, nobs, nt)).astype(np.float32)
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    sd = to_dev(s)
    y, gs = op.forward(sd), op.adjoint(to_dev(r))
    if nobs <= 32:  # more observers take the unfused kernels at some lengths
        na = torch.full_like(y, float("nan"))
        op.plan.forward_noalloc(sd.data_ptr(), 2, na.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert torch.equal(na, y)
    ey = oracle.rel_l2_per_rupture(y.cpu().numpy(), oracle.forward(G, F, s, dt=0.5, diff=1)).max()
    eg = oracle.rel_l2_per_rupture(gs.cpu().numpy(), oracle.adjoint(G, F, r, dt=0.5, diff=1)).max()
    print(f"{case}: forward {ey:.2e}, adjoint {eg:.2e}")
    assert ey <= 1e-5 and eg <= 1e-5
