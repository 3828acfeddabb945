"""Random features on the matrix cores go by units of 32 tokens, several to a wave when there are many: ragged last
units; one and two units a wave, above 8192 units five and six (at d = 64 with two workgroups a compute unit in place of
four), at d = 128 one to six; rows of a wider buffer, in place.  Against 64 bits: the result is rounded to bf16 once (2^-9 of a
value), and the terms of an exponent add up to less than 64 in magnitude, so that their sum in single precision is off
by at most 64 * d * 2^-24, at d = 128 5e-4 and with the former below 2^-8."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,H,N,h0,in_place", [(1, 1, 1, 0, False), (1, 3, 31, 1, False), (2, 2, 33, 0, True),
                                               (1, 20, 3333, 0, True), (3, 11, 8161, 1, False), (1, 23, 8161, 1, True),
                                               (4, 20, 4001, 0, False), (3, 30, 3971, 2, True)])
def test_units(B, H, N, h0, in_place, d):
    import torch
    from paper_2412_19829_amd import binding as gb
    gen = torch.Generator("cuda").manual_seed(N + d)
    wide = torch.randn(B, N, H, d + 8, device="cuda", generator=gen).mul_(0.2).bfloat16()
    x = wide.permute(0, 2, 1, 3)[..., :d]          # rows d + 8 elements apart, heads inside a row
    w = torch.randn(d, d, device="cuda", generator=gen).bfloat16()
    kept = wide.clone()
    out = x if in_place else torch.full((B, H, N, d), 7.0, device="cuda", dtype=torch.bfloat16)
    gb.gformer_random_features(x, w, out, h0, H)
    src = kept.permute(0, 2, 1, 3)[..., :d]
    if in_place:
        assert torch.equal(wide[..., d:], kept[..., d:]) and torch.equal(out[:, :h0], src[:, :h0])
    else:
        assert torch.equal(wide, kept) and bool((out[:, :h0] == 7).all())
    for h in range(h0, H):
        xf = src[:, h].double()
        assert float((torch.matmul(xf.abs(), w.double().abs().t()) + 0.5 * xf.square().sum(-1, keepdim=True)).max()) < 64
        want = torch.exp(torch.matmul(xf, w.double().t()) - 0.5 * xf.square().sum(-1, keepdim=True)) / d ** 0.5
        assert bool(((out[:, h].double() - want).abs() <= 2.0 ** -8 * want).all())
