"""The workspace a plan asks for is what its calls use: no more than the regions that a forward and an adjoint of
max_batch ruptures write (transformed inputs, seafloor field, split partials, scales), and nothing is written
past its end.
"""
import pytest
import torch

from gpu_util import log_case
from paper_2608_21763_amd import BLTTOperator, S2WOperator

pytestmark = pytest.mark.gpu


def _up(v, m):
    return (v + m - 1) // m * m


def _slots(nt):
    return max(32, 1 << max(2 * nt - 2, 1).bit_length()) // 2


def _guard(plan, op_store, ws_bytes, dev):
    """Binds a workspace with a tail of known bytes; returns that tail."""
    buf = torch.full((ws_bytes + 65536,), 0x5a, dtype=torch.uint8, device=dev)
    plan.bind(op_store.data_ptr(), op_store.numel(), buf.data_ptr(), ws_bytes)
    return buf, buf[ws_bytes:]


@pytest.mark.parametrize("kind", ["batched", "bf16", "f16", "bf16h"])
@pytest.mark.parametrize("sizes", [(70, 90, 20, 60, 40), (20, 300, 5, 200, 9), (9, 33, 40, 300, 65)],
                         ids=lambda s: "x".join(map(str, s)))
def test_share(sizes, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt, mb = sizes
    log_case("workspace", sizes=sizes, kind=kind)
    kw = dict(layout="batched") if kind == "batched" else dict(g_dtype=kind[:4].rstrip("h"), f_dtype=kind[:4].rstrip("h"))
    if kind == "bf16h":
        kw["products"] = "bf16"
    op = S2WOperator(nsub, ngrid, nobs, nt, max_batch=mb, **kw)
    M, bp, ws = _slots(nt), _up(mb, 8), op.plan.query_sizes()[1]
    if kind == "batched":
        nsk, nok = _up(nsub, 8), _up(nobs, 16)
        used = M * max(nsk, nok) * bp * 8 + ngrid * M * bp * 8 + max(16 * nok, 8 * nsk) * M * 2 * bp * 4
    else:
        nsq, noq = _up(nsub, 16), 16 * (1 << (_up(nobs, 16) // 16 - 1).bit_length())
        terms = 2 if kind == "bf16h" else 1
        used = (2 * min(ngrid, 4096) * M * 4 + M * nsq * bp * 8 + 4 * M * bp * 4 + M * nsq // 16 * bp // 8 * terms * 1024
                + ngrid * M * bp * 8 + max(16 * noq, nsq) * M * 2 * bp * 4)
    assert ws <= used + 16 * 256
    buf, tail = _guard(op.plan, op.op_store, ws, op.device)
    G, F = torch.randn((ngrid, nsub, nt), device=op.device), torch.randn((ngrid, nobs, nt), device=op.device)
    op.set_operators(G, F, 0)
    for B in sorted({1, min(mb, 8), min(mb, 20), mb}):
        s, r = torch.randn((B, nsub, nt), device=op.device), torch.randn((B, nobs, nt), device=op.device)
        assert torch.isfinite(op.forward(s)).all() and torch.isfinite(op.adjoint(r)).all()
    assert (tail == 0x5a).all()


@pytest.mark.parametrize("mb", [2, 4, 40])
def test_one_operator(mb):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nrow, ncol, nt = 130, 30, 60
    log_case("workspace_bltt", mb=mb)
    op = BLTTOperator(nrow, ncol, nt, max_batch=mb)
    M, bp, ws = _slots(nt), _up(mb, 8), op.plan.query_sizes()[1]
    rk, ck = _up(nrow, 8), _up(ncol, 8)
    used = M * max(rk, ck) * bp * 8 + 8 * max(rk, ck) * M * 2 * bp * 4 + min(mb, 4) * nrow * M * 8
    assert ws <= used + 4 * 256
    buf, tail = _guard(op.plan, op.op_store, ws, op.device)
    op.set_blocks(torch.randn((nrow, ncol, nt), device=op.device), 0)
    for B in sorted({1, 2, min(mb, 4), mb}):
        x, y = torch.randn((B, ncol, nt), device=op.device), torch.randn((B, nrow, nt), device=op.device)
        assert torch.isfinite(op.apply(x)).all() and torch.isfinite(op.adjoint(y)).all()
    assert (tail == 0x5a).all()
