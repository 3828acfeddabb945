"""d = 64: the read-out kernel's launch takes the windowed heads' query blocks along.  Same bits as the
kernels launched one by one, for piece counts on and off the multiple of 8 at which the query blocks
start, ragged sequences, both forms of the layer and the prefill's read-out."""
from __future__ import annotations

import pytest

from paper_2412_19829_amd import binding as gb
from tests.gpu_util import to_device
from tests.test_gpu_parity import synth

MASKS = (gb.GF_LAUNCH_WINDOWED, gb.GF_LAUNCH_LINEAR_STATE, gb.GF_LAUNCH_LINEAR_MAIN)


# B, H, N, window, H0, options
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (1, 2, 1, 1, 1, {}), (1, 3, 100, 7, 1, {}), (2, 5, 777, 64, 2, {}), (1, 12, 2048, 128, 2, {}),
    (1, 9, 1500, 300, 8, {}), (2, 4, 1000, 2000, 1, {"segment_len": 64}), (3, 4, 577, 64, 1, {"bidirectional": 1}),
    (1, 3, 129, 33, 2, {"bidirectional": 1}), (1, 4, 640, 50, 1, {"phi": gb.GF_PHI_IDENTITY}),
    (1, 4, 640, 50, 1, {"softmax_scale": -0.5}),
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_one_launch_gives_the_bits_of_two(case):
    import torch
    B, H, N, w, H0, kw = case
    q, k, v = (to_device(x, "bf16") for x in synth(B, H, N, 64, "bf16", 81))
    if "phi" in kw:
        q, k = q.abs() + 0.125, k.abs() + 0.125
    p = gb.make_params(n_sparse_heads=H0, **kw)
    need = gb.gformer_attn_workspace_bytes(B, H, N, 64, w, p)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    got, want = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    gb.gformer_attn_fwd(q, k, v, got, w, H0, workspace=ws, **kw)
    for m in MASKS:
        gb.gformer_attn_fwd(q, k, v, want, w, H0, workspace=ws, launch_mask=m, **kw)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(want.float()).all())
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    if not kw:   # the prefill's read-out (carried states out) in the same launch
        kc, vc = (torch.zeros(B, H0, w, 64, dtype=q.dtype, device="cuda") for _ in range(2))
        st = torch.zeros(B, H - H0, 64 * 64 + 64, device="cuda")
        pre = torch.full_like(q, float("nan"))
        gb.gformer_attn_prefill(q, k, v, pre, kc, vc, st, w, H0)
        torch.cuda.synchronize()
        assert torch.equal(pre.view(torch.int16), want.view(torch.int16))
        assert bool((st[..., -64:] > 0).all())
