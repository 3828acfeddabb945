"""bf16 linear heads: an element of Q or K that is no number reaches the rows that depend on it, and the carried states, and
no others, as in the gradients."""
from __future__ import annotations

import pytest

from paper_2412_19829_amd import binding as gb
from tests.gpu_util import to_device
from tests.test_gpu_parity import synth

N, AT, COL = 300, 150, 3


def forward(t, H0, **kw):
    import torch
    out = torch.full_like(t[0], 7.0)
    p = gb.make_params(n_sparse_heads=H0, **kw)
    B, H, _, d = t[0].shape
    ws = torch.empty(max(gb.gformer_attn_workspace_bytes(B, H, N, d, 16, p), 256), dtype=torch.uint8, device="cuda")
    return gb.gformer_attn_fwd(*t, out, 16, H0, workspace=ws, **kw)


# d, windowed heads, options: the read-out with and without query blocks beside it, in general chunks, over all keys
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (64, 0, {}), (64, 1, {}), (64, 0, {"segment_len": 64}), (64, 1, {"impl": gb.GF_IMPL_MFMA_CHUNK}), (64, 0, {"bidirectional": 1}),
    (128, 0, {}), (128, 1, {}), (128, 0, {"impl": gb.GF_IMPL_MFMA_CHUNK}), (128, 0, {"bidirectional": 1}),
], ids=lambda c: f"{c[0]}-{c[1]}" + "".join(f"-{k}" for k in c[2]))
def test_rows(case):
    import torch
    d, H0, kw = case
    t = [to_device(x, "bf16") for x in synth(1, 3, N, d, "bf16", 55)]
    clean = forward(t, H0, **kw)
    for which in (0, 1):
        bad = [x.clone() for x in t]
        bad[which][0, 1, AT, COL] = float("nan")
        got = forward(bad, H0, **kw)
        torch.cuda.synchronize()
        rows = torch.zeros(N, dtype=torch.bool, device="cuda")
        if which == 0: rows[AT] = True
        elif kw.get("bidirectional"): rows[:] = True
        else: rows[AT:] = True
        assert bool(got[0, 1, rows].isnan().all())
        assert torch.equal(got[0, 1, ~rows], clean[0, 1, ~rows])
        assert torch.equal(got[0, ::2], clean[0, ::2])


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
def test_carried_state(d):
    import torch
    q, k, v = (to_device(x, "bf16") for x in synth(1, 2, N, d, "bf16", 56))

    def states(k):
        out, st = torch.empty_like(q), torch.zeros(1, 2, d * d + d, device="cuda")
        gb.gformer_attn_prefill(q, k, v, out, None, None, st, 16, 0)
        torch.cuda.synchronize()
        return torch.cat([st[..., :d * d].view(1, 2, d, d), st[..., d * d:, None]], -1)   # [feature][values, Z]
    clean = states(k)
    bad = k.clone()
    bad[0, 1, AT, COL] = float("nan")
    got = states(bad)
    assert bool(got[0, 1, COL].isnan().all())
    others = torch.arange(d, device="cuda") != COL
    assert torch.equal(got[0, 1, others], clean[0, 1, others]) and torch.equal(got[0, 0], clean[0, 0])
