"""Single precision at head size 64 with both kinds of heads: the windowed heads' workgroups ride in the launches
of the linear heads' walks.  Same bits as the two kinds launched apart (forward: by launch mask; backward: with
overlap), for workgroup counts on and off the multiple of 8 at which the windowed ones start."""
from __future__ import annotations

import pytest

from paper_2412_19829_amd import binding as gb
from tests.gpu_util import to_device
from tests.test_gpu_parity import synth

# B, H, N, window, H0, bidirectional: at least 256 workgroups of 64 windowed rows, else they are launched apart
CASES = [(2, 6, 2049, 100, 4, 0), (1, 259, 40, 7, 257, 0), (4, 9, 577, 64, 7, 1), (3, 30, 200, 300, 25, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_together_gives_the_bits_of_apart(case):
    import torch
    B, H, N, w, H0, bidir = case
    q, k, v = (to_device(x, "f32") for x in synth(B, H, N, 64, "f32", 95))
    dout = to_device(synth(B, H, N, 64, "f32", 96)[2], "f32")
    kw = dict(bidirectional=bidir)
    got, want = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    gb.gformer_attn_fwd(q, k, v, got, w, H0, **kw)
    for m in (gb.GF_LAUNCH_WINDOWED, gb.GF_LAUNCH_LINEAR_STATE | gb.GF_LAUNCH_LINEAR_MAIN):
        gb.gformer_attn_fwd(q, k, v, want, w, H0, launch_mask=m, **kw)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(want).all())
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))

    stream = torch.cuda.current_stream().cuda_stream
    grads = []
    for overlap in (0, 1):
        p = gb.make_params(n_sparse_heads=H0, dtype=gb.GF_F32, overlap=overlap, **kw)
        ws = torch.full((gb.gformer_attn_bwd_workspace_bytes(B, H, N, 64, w, p),), 0xff, dtype=torch.uint8, device="cuda")
        grads.append([torch.full_like(q, float("nan")) for _ in range(3)])
        assert gb.gformer_attn_bwd_raw(*(x.data_ptr() for x in (q, k, v, dout, *grads[-1])), B, H, N, 64, w, p,
                                       ws.data_ptr(), ws.numel(), stream) == gb.GF_OK
        torch.cuda.synchronize()
    for g, a in zip(*grads):
        assert bool(torch.isfinite(g).all())
        assert torch.equal(g.view(torch.int32), a.view(torch.int32))


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES[:3], ids=lambda c: "x".join(map(str, c)))
def test_the_linear_heads_are_one_stage(case):
    """The read-out's mask runs the sums too, the sums' mask nothing; overlap gives the bits of no overlap."""
    import torch
    B, H, N, w, H0, bidir = case
    q, k, v = (to_device(x, "f32") for x in synth(B, H, N, 64, "f32", 97))
    want, main, over = (torch.full_like(q, float("nan")) for _ in range(3))
    gb.gformer_attn_fwd(q, k, v, want, w, H0, bidirectional=bidir)
    gb.gformer_attn_fwd(q, k, v, main, w, H0, bidirectional=bidir, launch_mask=gb.GF_LAUNCH_LINEAR_STATE)
    assert bool(torch.isnan(main).all())
    gb.gformer_attn_fwd(q, k, v, main, w, H0, bidirectional=bidir, launch_mask=gb.GF_LAUNCH_LINEAR_MAIN)
    gb.gformer_attn_fwd(q, k, v, over, w, H0, bidirectional=bidir, overlap=1)
    torch.cuda.synchronize()
    assert bool(torch.isnan(main[:, :H0]).all())
    assert torch.equal(main[:, H0:].view(torch.int32), want[:, H0:].view(torch.int32))
    assert torch.equal(over.view(torch.int32), want.view(torch.int32))
