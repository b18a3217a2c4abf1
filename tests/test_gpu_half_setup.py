"""Half-precision setup in calls of any size gives the same store, bit for bit: one row at a time, a few, all at once,
and more rows than the maxima of one pass (4,096), at every transform length and store pair; the words against
a quantization of float64 spectra: one power-of-two scale per (grid row, slot), nearest-even rounding.
"""
import numpy as np
import pytest
import torch

from gpu_util import log_case
from paper_2608_21763_amd import S2WOperator

pytestmark = pytest.mark.gpu


def _store(sizes, G, F, chunks, stores):
    nsub, ngrid, nobs, nt = sizes
    op = S2WOperator(nsub, ngrid, nobs, nt, max_batch=1, g_dtype=stores[0], f_dtype=stores[1])
    op.op_store.zero_()
    op.workspace.fill_(0xff)  # NaN patterns: nothing is read before it is written
    r0 = 0
    while r0 < ngrid:
        n = min(chunks[r0 % len(chunks)], ngrid - r0)
        op.set_operators(G[r0:r0 + n].clone(), F[r0:r0 + n].clone(), r0)
        r0 += n
    torch.cuda.synchronize()
    return op.op_store


@pytest.mark.parametrize("stores", [("bf16", "bf16"), ("f16", "f16"), ("bf16", "f16"), ("f16", "bf16")],
                         ids=lambda s: "-".join(s))
@pytest.mark.parametrize("sizes", [(17, 37, 5, 16), (3, 33, 18, 30), (33, 35, 2, 50), (70, 21, 33, 100), (20, 40, 40, 256),
                                   (18, 25, 6, 300), (2, 4200, 1, 9)], ids=lambda s: "x".join(map(str, s)))
def test_store_does_not_depend_on_the_calls(sizes, stores):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nsub, ngrid, nobs, nt = sizes
    log_case("half_setup", sizes=sizes, stores=stores)
    gen = torch.Generator(device="cuda").manual_seed(ngrid)
    # magnitudes over 12 decades from row to row, one row of zeros
    mag = 10.0 ** (12 * torch.rand((ngrid, 1, 1), generator=gen, device="cuda") - 6)
    G = torch.randn((ngrid, nsub, nt), generator=gen, device="cuda") * mag
    F = torch.randn((ngrid, nobs, nt), generator=gen, device="cuda") / mag
    G[ngrid // 2] = 0
    whole = _store(sizes, G, F, [ngrid], stores)
    for chunks in ([1], [5, 1, 16, 7]) if ngrid < 100 else ([999],):
        assert torch.equal(_store(sizes, G, F, chunks, stores), whole), chunks

    # elastic words of the first and the last row against float64 spectra
    L = max(32, 1 << (2 * nt - 2).bit_length()) if nt > 1 else 32
    M = L // 2
    nsq, ngq = (nsub + 15) // 16 * 16, (ngrid + 15) // 16 * 16
    words = whole[:ngq * M * nsq * 4].view(torch.int16).view(M, ngq // 16, nsq // 16, 16, 16, 2)
    off = (ngq * M * nsq * 4 + 255) // 256 * 256
    down = whole[off:off + ngrid * M * 4].view(torch.float32).view(ngrid, M).double()
    half = torch.bfloat16 if stores[0] == "bf16" else torch.float16
    for g in (0, ngrid // 2, ngrid - 1):
        X = torch.fft.rfft(G[g].double(), n=L)                       # [nsub][M + 1]
        re, im = X.real[:, :M].clone(), X.imag[:, :M].clone()
        im[:, 0] = X.real[:, M]                                       # packed slot 0
        w = words[:, g // 16, :, g % 16].reshape(M, nsq, 2).view(half).double()
        assert not w[:, nsub:].any()
        d = down[g][:, None]
        # half an ulp of the word at the row's maximum (2^15 scaled), and the float32 transform's own error
        step = 2.0 ** (15 - (8 if stores[0] == "bf16" else 11)) * d + 1e-6 * G[g].double().norm()
        assert ((w[:, :nsub, 0] * d - re.T).abs() <= step).all() and ((w[:, :nsub, 1] * d - im.T).abs() <= step).all()
        peak = torch.maximum(w[..., 0].abs(), w[..., 1].abs()).amax(dim=1)
        assert ((peak >= 2 ** 14 * (1 - 1e-5)) & (peak <= 2 ** 15)).all() if G[g].any() else not peak.any()
