"""bf16 gradients of the causal linear heads by the chunk scans (d = 128, and d = 64 where a head is cut into segments, from
225 tokens on, and the workspace does not hold their sums: shorter heads of d = 64 always take the segment walks): one
tile of a chunk, both tile rows, ragged chunks, light rounds in pairs and a single one before (behind) a
segment.  Tolerance: the bf16 mode's; and no gradient further from 64 bits than the rounding model of an older form of the
scans, whose c comes from a numerator of its own."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from paper_2412_19829_amd import inputs as gi
from tests.gpu_util import to_device, to_host
from tests.test_backward_rounding_model import numerator_scans
from tests.test_gpu_parity import check_grad, synth


def _scans(q, k, v, dout, **kw):
    import torch
    B, H, N, d = q.shape
    p = gb.make_params(**kw)
    dev = [to_device(x, "bf16") for x in (q, k, v, dout)]
    grads = [torch.full_like(dev[0], float("nan")) for _ in range(3)]
    least = (B * H * N * 8 + 255) // 256 * 256
    ws = torch.full((least,), 0xff, dtype=torch.uint8, device="cuda")
    assert gb.gformer_attn_bwd_raw(*(x.data_ptr() for x in (*dev, *grads)), B, H, N, d, 8, p, ws.data_ptr(), least,
                                   torch.cuda.current_stream().cuda_stream) == gb.GF_OK
    torch.cuda.synchronize()
    return [to_host(g) for g in grads]


@pytest.mark.gpu
@pytest.mark.parametrize("d,N", [(128, n) for n in (1, 31, 32, 33, 63, 64, 65, 97, 130, 512, 515, 700, 1100)] +
                         [(64, n) for n in (225, 256, 257, 289, 512, 515, 545, 575, 607, 639, 700, 1100, 2049)])
def test_gradients(N, d):
    B, H = 1, 2
    if d == 64:   # one causal segment would need no sums, and the walks would run
        assert gb.gformer_attn_bwd_workspace_bytes(B, H, N, d, 8, gb.make_params()) > (B * H * N * 8 + 255) // 256 * 256
    q, k, v = synth(B, H, N, d, "bf16", 91)
    dout = synth(B, H, N, d, "bf16", 92)[2]
    for g, r, name in zip(_scans(q, k, v, dout), co.attn_bwd(q, k, v, dout, 8, 0), ("dq", "dk", "dv")):
        check_grad(g, r, "bf16", f"{name} {N} {d}", dout)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [64, 190, 1000])
def test_no_further_from_64_bits_than_with_a_numerator(N):
    B, H, d = 1, 12, 128
    q, k, v = synth(B, H, N, d, "bf16", 93)
    dout = synth(B, H, N, d, "bf16", 94)[2]
    ref = co.attn_bwd(q, k, v, dout, 8, 0)
    model = [np.empty_like(r) for r in ref]
    for h in range(H):
        one = (x[0, h].astype(np.float64) for x in (q, k, v, dout))
        for s, g in zip(model, numerator_scans(*one, rounded=True, pairs=True)):
            s[0, h] = gi.round_to_bf16(g.astype(np.float32))
    for g, s, r, name in zip(_scans(q, k, v, dout), model, ref, ("dq", "dk", "dv")):
        assert np.linalg.norm(g - r) <= 1.01 * np.linalg.norm(s - r), name
