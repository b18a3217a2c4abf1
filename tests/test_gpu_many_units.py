"""Batched mid-chain and row transforms with more units than workgroups, so that every workgroup takes several: the
next unit's rows loaded under the current one, buffers and scales refilled, maxima kept from unit to unit.
Every slot count served by the general kernel and 256, with the plain mid-chain (float32), the one that keeps
maxima (float16 products, 33 ruptures), the one on [l][g][b] (8 ruptures) and the packing one (bfloat16
products), with snapshots and in the adjoint.  Bounds: rel-L2 <= 1e-5 for float32, the half stores' of
``gpu_util``, against the oracle on ruptures of the first, a middle and the last block of 16.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import half_limit, log_case, make_operator, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(3, 8300, 2, 16), (3, 9000, 2, 20), (3, 9001, 2, 60), (3, 4500, 2, 100), (3, 2500, 2, 200), (3, 2500, 2, 400)]
STORES = {"f32": (17, 1e-5, dict(layout="batched")),
          "flat": (8, half_limit("f16", "f16"), dict(g_dtype="f16", f_dtype="f16")),
          "maxima": (33, half_limit("f16", "f16"), dict(g_dtype="f16", f_dtype="f16")),
          "packed": (17, half_limit("bf16", "bf16"), dict(g_dtype="bf16", f_dtype="bf16", products="bf16"))}


@pytest.mark.parametrize("kind", list(STORES))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_many_units(shape, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = shape
    B, bound, kw = STORES[kind]
    log_case("many_units", shape=shape, kind=kind)
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, max_batch=B, dt=0.5, chunk_rows=ngrid, **kw)
    s = synth.gen_slip_batch(cfg, 0, B)
    r = synth.normals(cfg.seed, "r", nt, (B, nobs, nt)).astype(np.float32)
    sd = to_dev(s)
    y = op.forward(sd)
    times = [0, nt // 2, nt - 1]
    yd, m = op.forward_displacement(sd, times)
    gs = op.adjoint(to_dev(r))
    assert torch.equal(y, yd)
    some = sorted({0, B // 2, B - 1})
    G, F = synth.gen_G(cfg).astype(np.float64), synth.gen_F(cfg).astype(np.float64)
    errs = {
        "y": (y, oracle.forward(G, F, s[some], dt=0.5, diff=1)),
        "m": (m, oracle.bltt(G, s[some])[:, :, times]),
        "gs": (gs, oracle.adjoint(G, F, r[some], dt=0.5, diff=1)),
    }
    errs = {k: oracle.rel_l2_per_rupture(a[some].cpu().numpy(), b).max() for k, (a, b) in errs.items()}
    print(shape, kind, {k: f"{e:.2e}" for k, e in errs.items()})
    assert max(errs.values()) <= bound
