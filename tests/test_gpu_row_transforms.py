"""Every transform length of the library (L = 32 .. 1024) through setup, source, mid-chain and output
transforms, at the edges of each length (nt = the smallest and largest, odd ones among them), on
ragged sizes and with operator chunks whose first rows are not multiples of anything.

Bounds: float32 layouts rel-L2 <= 1e-5, float16 stores 2e-3, bfloat16 stores (whose products leave
packed activations) the ceiling of ``gpu_util`` on dense iid operators; the adjoint by the dot-product
identity <A s, r> = <s, A^T r>, whose two sides differ by the rounding of the same arithmetic.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import half_limit, log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

STORES = {
    "single": (dict(layout="single"), 1e-5, 1e-6),
    "batched": (dict(layout="batched"), 1e-5, 1e-6),
    "f16": (dict(g_dtype="f16", f_dtype="f16"), half_limit("f16", "f16"), 2e-3),
    "bf16h": (dict(g_dtype="bf16", f_dtype="bf16", products="bf16"), half_limit("bf16", "bf16"), 2e-3),
}


@pytest.mark.parametrize("store", list(STORES))
@pytest.mark.parametrize("nt", [1, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257, 511, 512])
def test_transform_lengths(nt, store):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kw, bound, dot_bound = STORES[store]
    B = 18
    log_case("row_transforms", nt=nt, store=store)
    cfg = synth.workload("small_dense").replace(nsub=19, ngrid=37, nobs=5, nt=nt)
    op = make_operator(cfg, max_batch=B, dt=0.5, chunk_rows=5, **kw)
    s = synth.gen_slip_batch(cfg, 0, B)
    r = synth.normals(cfg.seed, "r", nt, (B, cfg.nobs, nt)).astype(np.float32)
    y = op.forward(to_dev(s)).cpu().numpy().astype(np.float64)
    gs = op.adjoint(to_dev(r)).cpu().numpy().astype(np.float64)
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    errs = oracle.rel_l2_per_rupture(y, oracle.forward(G, F, s, dt=0.5, diff=1))
    print(f"nt={nt} {store}: rel-L2 max {errs.max():.2e}")
    assert errs.max() <= bound
    for b in range(B):
        a, c = np.vdot(y[b], r[b]), np.vdot(s[b].astype(np.float64), gs[b])
        assert abs(a - c) <= dot_bound * np.linalg.norm(y[b]) * np.linalg.norm(r[b])
    # one more value of the transposed map than the identity alone pins: a column against the oracle
    ga = oracle.adjoint(G, F, r[:1], dt=0.5, diff=1)
    assert oracle.rel_l2_per_rupture(gs[:1], ga).max() <= bound
