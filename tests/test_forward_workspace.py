"""One workspace serves every form of a forward call: the size asked for depends on neither the kernel of the windowed
heads, nor the window, nor the options, although the cut of the state pass at d = 128 does."""
from __future__ import annotations

import pytest

from paper_2412_19829_amd import binding as gb
from tests.gpu_util import to_device, to_host
from tests.test_gpu_parity import check, oracle, synth

D = 128
# the first two are cut longer beside query blocks than where the windowed heads stream
SHAPES = [(2, 32, 15624, 1), (2, 32, 3001, 6), (1, 32, 2048, 6), (1, 8, 2048, 2), (4, 32, 8192, 6), (2, 3, 700, 3)]


def _needs(B, H, N, H0):
    for impl in (gb.GF_IMPL_AUTO, gb.GF_IMPL_MFMA, gb.GF_IMPL_MFMA_BLOCKED, gb.GF_IMPL_MFMA_STREAM):
        for w in (64, 256):
            for kw in ({}, {"overlap": 1}, {"softmax_scale": -1.0}, {"launch_mask": 6}):
                p = gb.make_params(n_sparse_heads=H0, impl=impl, **kw)
                st, pl = gb.gformer_attn_plan(B, H, N, D, w, p)
                assert st == gb.GF_OK and pl.workspace_bytes == gb.gformer_attn_workspace_bytes(B, H, N, D, w, p)
                assert pl.workspace_bytes >= pl.state_blocks * (D * D + D) * 4
                yield pl.workspace_bytes


@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_one_size(case):
    assert len(set(_needs(*case))) == 1


def test_two_cuts():
    """The same shape, cut in two ways: what the test below runs."""
    sums = {impl: gb.gformer_attn_plan(3, 19, 2500, D, 64, gb.make_params(n_sparse_heads=2, impl=impl))[1].state_blocks
            for impl in (gb.GF_IMPL_MFMA_BLOCKED, gb.GF_IMPL_MFMA_STREAM)}
    assert sums[gb.GF_IMPL_MFMA_BLOCKED] < sums[gb.GF_IMPL_MFMA_STREAM]


@pytest.mark.gpu
@pytest.mark.parametrize("sized,called", [("AUTO", "STREAM"), ("BLOCKED", "STREAM"), ("STREAM", "BLOCKED")])
def test_sized_for_one_kernel_called_with_another(sized, called):
    import torch
    B, H, N, w, H0 = 3, 19, 2500, 64, 2
    impl = {"AUTO": gb.GF_IMPL_AUTO, "BLOCKED": gb.GF_IMPL_MFMA_BLOCKED, "STREAM": gb.GF_IMPL_MFMA_STREAM}
    q, k, v = synth(B, H, N, D, "bf16", 141)
    tq, tk, tv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.full_like(tq, float("nan"))
    need = gb.gformer_attn_workspace_bytes(B, H, N, D, w, gb.make_params(n_sparse_heads=H0, impl=impl[sized]))
    ws = torch.full((need,), 0xff, dtype=torch.uint8, device="cuda")
    gb.gformer_attn_fwd(tq, tk, tv, out, w, H0, impl=impl[called], workspace=ws)
    torch.cuda.synchronize()
    check(to_host(out), oracle(q, k, v, w, H0), "bf16", f"{sized} {called}")
