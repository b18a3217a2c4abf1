"""Tuning of the single layout: the four shape controls are automatic (-1) until set, each on its own, and what
``s2w_get_tuning`` returns keeps the automatic choices in force when it is handed back.

Two shapes of a kernel group its sums differently, so equal bits over random operators tell that the same
shapes ran; that the groupings differ at these sizes is asserted beside.
"""
import pytest
import torch

import synth
from gpu_util import log_case, make_operator, to_dev
from paper_2608_21763_amd.abi import S2WError

pytestmark = pytest.mark.gpu

FIELDS = ("fused_wg_per_cu", "fused_rows", "adj_cols", "adj_splits")
# two workgroups per CU in the forward; 8 columns per thread in the adjoint; 70 observers take the unfused forward
SIZES = [(60, 4096, 4, 64), (60, 700, 3, 200), (20, 300, 70, 256)]


def _plan(size):
    nsub, ngrid, nobs, nt = size
    cfg = synth.workload("small_dense").replace(nsub=nsub, ngrid=ngrid, nobs=nobs, nt=nt)
    op = make_operator(cfg, layout="single")
    s = to_dev(synth.gen_slip_batch(cfg, 0, 1))
    r = to_dev(synth.normals(cfg.seed, "r", 1, (1, nobs, nt)))
    return op, lambda: (op.forward(s), op.adjoint(r))


def _same(a, b):
    return torch.equal(a[0], b[0]), torch.equal(a[1], b[1])


@pytest.mark.parametrize("size", SIZES, ids=["x".join(map(str, s)) for s in SIZES])
def test_round_trip_keeps_automatic(size):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log_case("single_tuning", size=size)
    op, call = _plan(size)
    t = op.get_tuning()
    assert all(t[k] == -1 for k in FIELDS)
    auto = call()
    op.set_tuning(**t)
    assert op.get_tuning() == t
    assert _same(auto, call()) == (True, True)
    op.set_tuning(fused_wg_per_cu=1, fused_rows=8, adj_cols=16, adj_splits=16)
    assert _same(auto, call())[1] is False
    op.set_tuning(**t)
    assert _same(auto, call()) == (True, True)


def test_fields_are_set_apart():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log_case("single_tuning_fields")
    op, call = _plan(SIZES[0])
    auto = call()
    for k, v in (("fused_rows", 8), ("fused_wg_per_cu", 3), ("adj_splits", 7), ("adj_cols", 8)):
        op.set_tuning(**{k: v})
        t = op.get_tuning()
        assert t[k] == v and all(t[o] == -1 for o in FIELDS if o != k)
        call()
        op.set_tuning(**{k: -1})
        assert _same(auto, call()) == (True, True)
    # tiles of 8 rows are the automatic ones here: setting them changes nothing else
    op.set_tuning(fused_rows=8)
    assert _same(auto, call()) == (True, True)


def test_bad_values_are_refused():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    op, _ = _plan(SIZES[1])
    t = op.get_tuning()
    for kw in ({"fused_wg_per_cu": 5}, {"fused_wg_per_cu": -2}, {"fused_rows": 6}, {"fused_rows": -2}, {"adj_cols": 4},
               {"adj_cols": -2}, {"adj_splits": 65}, {"adj_splits": -2}):
        with pytest.raises(S2WError):
            op.set_tuning(**kw)
    assert op.get_tuning() == t
