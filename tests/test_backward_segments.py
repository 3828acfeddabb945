"""bf16 gradients of the linear heads at head size 64, heads cut into segments: where chunks of 32 tokens
and segments end, few segments (a walk adds up their sums) and many (a scan ran), both forms of the
layer, and a workspace of the least size, which takes the scans instead.  Tolerance: the bf16 mode's."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from paper_2412_19829_amd import inputs as gi
from tests.gpu_util import to_device, to_host
from tests.test_backward_rounding_model import numerator_scans
from tests.test_gpu_parity import check_grad, run_bwd, synth

# B, H, N, bidirectional, segments per head (256 compute units)
CASES = [(1, 1, n, b, max(1, -(-n // 32) // 4)) for n in (1, 31, 32, 33, 64, 129, 255, 257) for b in (0, 1)] + [
    (1, 1, 400, 0, 3), (1, 1, 512, 0, 4),      # a causal walk adds up to three sums itself
    (1, 1, 1300, 0, 9), (1, 1, 1300, 1, 4),    # more: a scan ran; over all keys four at most
    (1, 1, 8190, 0, 64),                       # as many as a head is ever cut into
    (1, 200, 300, 0, 2), (2, 100, 517, 1, 3),
    (3, 300, 70, 0, 1),                        # more heads than three per compute unit
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_segments(case):
    """The counts above, from the workspace that a call asks for: two sums per segment beside the statistics."""
    B, H, N, bidir, count = case
    least = (B * H * N * 8 + 255) // 256 * 256
    need = gb.gformer_attn_bwd_workspace_bytes(B, H, N, 64, 8, gb.make_params(bidirectional=bidir))
    sums = (need - least) / (B * H * 2 * (64 * 64 + 64) * 4)
    assert sums == (4 if bidir else count if count > 1 else 0)   # over all keys room for four is always asked for


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_gradients(case):
    B, H, N, bidir, _ = case
    q, k, v = synth(B, H, N, 64, "bf16", 51)
    dout = synth(B, H, N, 64, "bf16", 52)[2]
    ref = co.attn_bwd(q, k, v, dout, 8, 0, bidirectional=bool(bidir))
    for g, r, name in zip(run_bwd(q, k, v, dout, "bf16", 8, 0, bidirectional=bidir), ref, ("dq", "dk", "dv")):
        check_grad(g, r, "bf16", f"{name} {case}", dout)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [64, 100, 235, 255, 256, 1000])
def test_no_further_from_64_bits_than_the_scans(N):
    """The scans keep more of a row's weights as pairs: no gradient of the walks may be further from the oracle's than
    theirs (by their rounding model).  Over 24 heads two such errors agree to a percent of themselves."""
    B, H = 2, 12
    q, k, v = synth(B, H, N, 64, "bf16", 57)
    dout = synth(B, H, N, 64, "bf16", 58)[2]
    ref = co.attn_bwd(q, k, v, dout, 8, 0)
    scans = [np.empty_like(r) for r in ref]
    for b in range(B):
        for h in range(H):
            one = (x[b, h].astype(np.float64) for x in (q, k, v, dout))
            for s, g in zip(scans, numerator_scans(*one, rounded=True, pairs=True)):
                s[b, h] = gi.round_to_bf16(g.astype(np.float32))
    for g, s, r, name in zip(run_bwd(q, k, v, dout, "bf16", 8, 0), scans, ref, ("dq", "dk", "dv")):
        assert np.linalg.norm(g - r) <= 1.01 * np.linalg.norm(s - r), name


def test_more_heads_over_all_keys_than_a_grid_holds_are_refused():
    # 2^22 heads; nothing is launched, so the addresses are not looked at
    p = gb.make_params(bidirectional=1)
    at = [256 * (i + 1) for i in range(8)]
    assert gb.gformer_attn_bwd_raw(*at[:7], 1 << 15, 1 << 7, 1, 64, 8, p, at[7], 1 << 50) == gb.GF_ERR_UNSUPPORTED
    assert gb.gformer_attn_bwd_raw(*at[:7], 1 << 15, 1 << 7, 1, 64, 8, p, at[7], 1 << 38) == gb.GF_ERR_WORKSPACE


@pytest.mark.gpu
@pytest.mark.parametrize("phi,eps", [(gb.GF_PHI_ELU1, 0.5), (gb.GF_PHI_IDENTITY, 0.0)], ids=["eps", "identity"])
def test_any_workspace_serves(phi, eps):
    import torch
    B, H, N, d, H0 = 1, 3, 700, 64, 1
    q, k, v = synth(B, H, N, d, "bf16", 53)
    dout = synth(B, H, N, d, "bf16", 54)[2]
    if phi == gb.GF_PHI_IDENTITY:
        q, k = (gi.round_to_bf16(abs(x) + 0.125) for x in (q, k))
    ref = co.attn_bwd(q, k, v, dout, 16, H0, phi=phi, eps=eps)
    p = gb.make_params(n_sparse_heads=H0, phi=phi, eps=eps)
    full = gb.gformer_attn_bwd_workspace_bytes(B, H, N, d, 16, p)
    least = (B * H * N * 8 + 255) // 256 * 256
    assert full > least
    dev = [to_device(x, "bf16") for x in (q, k, v, dout)]
    stream = torch.cuda.current_stream().cuda_stream
    for nbytes in (full, full - 1, least):
        ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")
        grads = [torch.full_like(dev[0], float("nan")) for _ in range(3)]
        assert gb.gformer_attn_bwd_raw(*(x.data_ptr() for x in (*dev, *grads)), B, H, N, d, 16, p, ws.data_ptr(),
                                       nbytes, stream) == gb.GF_OK
        torch.cuda.synchronize()
        for g, r, name in zip(grads, ref, ("dq", "dk", "dv")):
            check_grad(to_host(g), r, "bf16", f"{name}, {nbytes} bytes", dout)
    assert gb.gformer_attn_bwd_raw(*(x.data_ptr() for x in (*dev, *grads)), B, H, N, d, 16, p, ws.data_ptr(),
                                   least - 1, stream) == gb.GF_ERR_WORKSPACE


@pytest.mark.gpu
@pytest.mark.parametrize("bidir", [0, 1], ids=["causal", "bidirectional"])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
def test_views_of_a_fused_projection(dtype, d, bidir):
    """q, k, v as views of one [B, N, 3, H, d] buffer, dO in [B, N, H, d] storage: forward and backward give the bits
    of dense tensors."""
    import torch
    B, H, N, H0 = 2, 5, 700, 2
    dense = [to_device(x, dtype) for x in synth(B, H, N, d, dtype, 55)]
    dout = to_device(synth(B, H, N, d, dtype, 56)[2], dtype)
    buf = torch.stack([x.permute(0, 2, 1, 3) for x in dense], 2).contiguous()
    views = [buf[:, :, i].permute(0, 2, 1, 3) for i in range(3)]
    dview = dout.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    out = [torch.full_like(dout, float("nan")), torch.full_like(dview, float("nan"))]
    grads = [[torch.full_like(x, float("nan")) for x in dense]]
    gbuf = torch.full_like(buf, float("nan"))
    grads.append([gbuf[:, :, i].permute(0, 2, 1, 3) for i in range(3)])
    for (q, k, v), do, o, g in zip((dense, views), (dout, dview), out, grads):
        gb.gformer_attn_fwd(q, k, v, o, 40, H0, bidirectional=bidir)
        gb.gformer_attn_bwd(q, k, v, do, *g, 40, H0, bidirectional=bidir)
    torch.cuda.synchronize()
    ref = co.attn_bwd(*(to_host(x) for x in dense), to_host(dout), 40, H0, bidirectional=bool(bidir))
    for a, b, r in zip((out[0], *grads[0]), (out[1], *grads[1]), (None, *ref)):
        assert torch.equal(a.view(bits), b.contiguous().view(bits))
        if r is not None:
            check_grad(to_host(a), r, dtype, f"{dtype} {d}", to_host(dout))
