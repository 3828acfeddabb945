"""Decode at the largest rings: scores that fill the LDS a launch gets without asking, and the 64 KB
the entry point accepts at most."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2412_19829_amd import binding as gb


@pytest.mark.gpu
@pytest.mark.parametrize("window", [13200, 13300, 14272])   # 59.8 KB, 60.2 KB, 64 KB of scores and row sums
def test_decode_of_the_widest_rings(window):
    import torch
    B, H, d = 1, 2, 64
    g = torch.Generator("cpu").manual_seed(window)
    q, k, v = (torch.randn(B, H, d, generator=g) for _ in range(3))
    kc, vc = (torch.randn(B, H, window, d, generator=g) for _ in range(2))
    t = window + 5
    kr, vr = kc.double(), vc.double()
    kr[:, :, t % window], vr[:, :, t % window] = k.double(), v.double()
    p = torch.softmax(0.1 * (kr * q.double()[:, :, None]).sum(-1), -1)
    want = (p[..., None] * vr).sum(2).numpy()
    dev = [x.cuda() for x in (q, k, v, kc, vc)]
    out = torch.full((B, H, d), float("nan"), device="cuda")
    gb.gformer_attn_decode(dev[0], dev[1], dev[2], out, dev[3], dev[4], None, window, H, t, softmax_scale=0.1)
    # 14,000 weights of 1/14,000 and less, summed in fp32
    assert np.abs(out.cpu().numpy() - want).max() <= 1e-5
    with pytest.raises(gb.GformerError):
        w = 14273
        big = torch.zeros(B, H, w, d, device="cuda")
        gb.gformer_attn_decode(dev[0], dev[1], dev[2], out, big, big.clone(), None, w, H, t)
