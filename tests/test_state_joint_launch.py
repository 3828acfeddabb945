"""d = 128: the state pass's launch takes the windowed heads' query blocks along.  Same bits as the kernels launched one
by one, for either order of the two kinds of block, block counts on and off the multiple of 8 at which the second kind
starts, ragged sequences, both forms of the layer; and the rings a prefill leaves, which the query blocks fill."""
from __future__ import annotations

import pytest

from paper_2412_19829_amd import binding as gb
from tests.gpu_util import to_device
from tests.test_gpu_parity import synth

D = 128


# B, H, N, window, H0, options
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (1, 2, 513, 7, 1, {}), (2, 5, 777, 64, 2, {}), (1, 10, 2048, 128, 2, {}), (1, 9, 1500, 300, 8, {}),
    (2, 4, 1000, 2000, 1, {"segment_len": 64}), (1, 3, 4100, 16, 1, {}), (1, 2, 600, 600, 1, {}),
    (3, 4, 577, 64, 1, {"bidirectional": 1}), (1, 3, 129, 33, 2, {"bidirectional": 1}),
    (1, 4, 640, 50, 1, {"phi": gb.GF_PHI_IDENTITY}), (1, 4, 640, 50, 1, {"softmax_scale": -0.5}),
    (1, 3, 2600, 200, 1, {"chunk": 128}),
    (1, 3, 8100, 16, 1, {"segment_len": 3968}), (1, 4, 8100, 3000, 3, {"segment_len": 3968}),   # chains of 31: apart, together
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_one_launch_gives_the_bits_of_two(case):
    import torch
    B, H, N, w, H0, kw = case
    q, k, v = (to_device(x, "bf16") for x in synth(B, H, N, D, "bf16", 83))
    if "phi" in kw:
        q, k = q.abs() + 0.125, k.abs() + 0.125
    p = gb.make_params(n_sparse_heads=H0, **kw)
    ws = torch.empty(max(gb.gformer_attn_workspace_bytes(B, H, N, D, w, p), 256), dtype=torch.uint8, device="cuda")
    got, want = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    gb.gformer_attn_fwd(q, k, v, got, w, H0, workspace=ws, **kw)
    for m in (gb.GF_LAUNCH_WINDOWED, gb.GF_LAUNCH_LINEAR_STATE, gb.GF_LAUNCH_LINEAR_MAIN):
        gb.gformer_attn_fwd(q, k, v, want, w, H0, workspace=ws, launch_mask=m, **kw)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(want.float()).all())
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", [
    (1, 3, 5, 16, 1, 0), (2, 4, 128, 128, 2, 0), (1, 3, 700, 130, 2, 0), (1, 2, 300, 1000, 2, 0), (2, 3, 385, 1, 1, 0),
    (1, 3, 900, 200, 2, gb.GF_IMPL_MFMA_STREAM),   # the streaming kernel leaves the rings to a launch of their own
], ids=lambda c: "x".join(map(str, c)))
def test_rings_after_prefill(case, d):
    import torch
    B, H, N, w, H0, impl = case
    q, k, v = (to_device(x, "bf16") for x in synth(B, H, N, d, "bf16", 84))
    kc, vc = (torch.full((B, H0, w, d), -7.0, dtype=q.dtype, device="cuda") for _ in range(2))
    st = torch.zeros(B, H - H0, d * d + d, device="cuda") if H0 < H else None
    gb.gformer_attn_prefill(q, k, v, torch.empty_like(q), kc, vc, st, w, H0, impl=impl)
    torch.cuda.synchronize()
    for ring, x in ((kc, k), (vc, v)):
        want = torch.full_like(ring, -7.0)     # slots of tokens that are not there stay as they are
        for t in range(max(0, N - w), N):
            want[:, :, t % w] = x[:, :H0, t]
        assert torch.equal(ring.view(torch.int16), want.view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
def test_rings_under_a_negative_scale(d):
    """The kernels of a negative scale are others, in launches of their own."""
    import torch
    B, H, N, w, H0 = 2, 3, 450, 130, 2
    q, k, v = (to_device(x, "bf16") for x in synth(B, H, N, d, "bf16", 85))
    kc, vc = (torch.full((B, H0, w, d), -7.0, dtype=q.dtype, device="cuda") for _ in range(2))
    st = torch.zeros(B, H - H0, d * d + d, device="cuda")
    gb.gformer_attn_prefill(q, k, v, torch.empty_like(q), kc, vc, st, w, H0, softmax_scale=-0.5)
    torch.cuda.synchronize()
    for ring, x in ((kc, k), (vc, v)):
        for t in range(N - w, N):
            assert torch.equal(ring[:, :, t % w].view(torch.int16), x[:, :H0, t].view(torch.int16))
