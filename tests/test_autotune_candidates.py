"""The tuner times the library's automatic choice of every layout and puts it back in force when it wins."""
import importlib

import pytest
import torch

tuner = importlib.import_module("paper_2608_21763_amd.autotune")

FIELDS = {
    ("single", "f32"): ("fused_rows", "fused_wg_per_cu"),
    ("batched", "f32"): ("gemm32_cfg", "gemm32_cfg_k", "adj32_cfg"),
    ("batched", "bf16"): ("gemm_cfg",),
}


class Plan:
    """What the tuner sees of an operator: sizes, layout, and the tuning (zero keeps a field)."""
    nsub, ngrid, nobs, nt, max_batch, diff, f_dtype = 3, 5, 2, 4, 2, 1, "f32"
    device = torch.device("cpu")

    def __init__(self, layout, g_dtype):
        self._layout, self.g_dtype = layout, g_dtype
        self.tuning = {"fgemm_lds": 1, "hadj_tile_f": -1, "hadj_tile_g": -1}
        self.tuning.update((k, -1) for names in FIELDS.values() for k in names)

    def plan_layout(self):
        return self._layout

    def get_tuning(self):
        return dict(self.tuning)

    def set_tuning(self, **kw):
        self.tuning.update((k, v) for k, v in kw.items() if v)

    def forward(self, s, out):
        pass

    adjoint = forward


@pytest.mark.parametrize("kind", list(FIELDS), ids=["-".join(k) for k in FIELDS])
@pytest.mark.parametrize("adjoint", [False, True])
def test_automatic_is_timed_and_kept(kind, adjoint, monkeypatch):
    op = Plan(*kind)
    timed = []

    def time(o, fn, reps):
        timed.append(o.get_tuning())
        return 1.0 if all(o.tuning[k] == -1 for k in FIELDS[kind]) else 2.0

    monkeypatch.setattr(tuner, "_time", time)
    monkeypatch.setattr(tuner, "_key", lambda o, B: "key")
    start = op.get_tuning()
    res = tuner.autotune(op, 1, adjoint=adjoint)
    names = [k for k in FIELDS[kind] if adjoint or k != "adj32_cfg"]
    assert any(all(t[k] == -1 for k in names) for t in timed)
    assert all(res["best"][k] == -1 for k in names)
    assert all(op.get_tuning()[k] == start[k] for k in names)
    assert len(res["results"]) > 1
