"""bf16 gradients of the linear heads at head size 64, heads cut into segments: where chunks of 32 tokens
and segments end, few segments (a walk adds up their sums) and many (a scan ran), both forms of the
layer, and a workspace of the least size, which takes the scans instead.  Tolerance: the bf16 mode's."""
from __future__ import annotations

import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from paper_2412_19829_amd import inputs as gi
from tests.gpu_util import to_device, to_host
from tests.test_gpu_parity import check_grad, run_bwd, synth

# B, H, N, bidirectional
CASES = [(1, 1, n, b) for n in (1, 31, 32, 33, 64, 129, 255, 257) for b in (0, 1)] + [
    (1, 1, 1300, 0), (1, 1, 1300, 1),      # ten segments with a scan; over all keys four
    (1, 200, 300, 0), (2, 100, 517, 1),    # three segments, two
    (3, 300, 70, 0),                       # more heads than three per compute unit: one segment
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_gradients(case):
    B, H, N, bidir = case
    q, k, v = synth(B, H, N, 64, "bf16", 51)
    dout = synth(B, H, N, 64, "bf16", 52)[2]
    ref = co.attn_bwd(q, k, v, dout, 8, 0, bidirectional=bool(bidir))
    for g, r, name in zip(run_bwd(q, k, v, dout, "bf16", 8, 0, bidirectional=bidir), ref, ("dq", "dk", "dv")):
        check_grad(g, r, "bf16", f"{name} {case}", dout)


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
