"""bf16 gradients with both kinds of heads: the windowed heads' passes ride in the launches of the linear heads'
segment walks (d = 64) and scans (d = 128, causal).  Same bits as the two kinds launched apart (overlap, and for
the windowed heads of a causal call at d = 64 the least workspace), for block counts on and off the multiple of 8
at which the windowed blocks start and for calls whose first launch holds no walk at all."""
from __future__ import annotations

import pytest

from paper_2412_19829_amd import binding as gb
from tests.gpu_util import to_device
from tests.test_gpu_parity import synth


# B, H, N, window, H0, options
@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", [
    (1, 2, 1, 1, 1, {}), (1, 3, 20, 7, 1, {}), (2, 5, 777, 64, 2, {}), (1, 9, 1500, 300, 8, {}),
    (1, 400, 200, 50, 1, {}),     # one segment a head: no sums in front
    (3, 4, 577, 64, 1, {"bidirectional": 1}), (1, 3, 129, 33, 2, {"bidirectional": 1}),
    (1, 4, 640, 700, 1, {"phi": gb.GF_PHI_IDENTITY}), (1, 4, 640, 50, 3, {"softmax_scale": -0.5}),
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_together_gives_the_bits_of_apart(case, d):
    import torch
    B, H, N, w, H0, kw = case
    q, k, v = (to_device(x, "bf16") for x in synth(B, H, N, d, "bf16", 91))
    dout = to_device(synth(B, H, N, d, "bf16", 92)[2], "bf16")
    if "phi" in kw:
        q, k = q.abs() + 0.125, k.abs() + 0.125
    stream = torch.cuda.current_stream().cuda_stream

    def run(nbytes, **more):
        p = gb.make_params(n_sparse_heads=H0, **kw, **more)
        need = gb.gformer_attn_bwd_workspace_bytes(B, H, N, d, w, p)
        ws = torch.full((nbytes or need,), 0xff, dtype=torch.uint8, device="cuda")
        grads = [torch.full_like(q, float("nan")) for _ in range(3)]
        assert gb.gformer_attn_bwd_raw(*(x.data_ptr() for x in (q, k, v, dout, *grads)), B, H, N, d, w, p,
                                       ws.data_ptr(), ws.numel(), stream) == gb.GF_OK
        torch.cuda.synchronize()
        return grads

    got, apart = run(0), run(0, overlap=1)
    least = got if "bidirectional" in kw or d == 128 else run((B * H * N * 8 + 255) // 256 * 256)
    for g, a, l in zip(got, apart, least):
        assert bool(torch.isfinite(g.float()).all())
        assert torch.equal(g.view(torch.int16), a.view(torch.int16))
        assert torch.equal(g[:, :H0].view(torch.int16), l[:, :H0].view(torch.int16))
