"""bf16 gradients at head size 64 where the windowed heads' passes weigh more than the walks they share launches with: the
linear heads are cut into fewer segments there, and into as many as before with the passes in launches of their own
(overlap = 1).  Both against the oracle, from the workspace a call of either kind asks for."""
from __future__ import annotations

import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from tests.test_gpu_parity import check_grad, run_bwd, synth


@pytest.mark.parametrize("case", [(1, 80, 2000, 300, 16), (8, 12, 2048, 256, 4), (4, 16, 4096, 128, 3)])
def test_one_size_serves_both(case):
    B, H, N, w, H0 = case
    sizes = {gb.gformer_attn_bwd_workspace_bytes(B, H, N, 64, w, gb.make_params(n_sparse_heads=H0, overlap=o)) for o in (0, 1)}
    assert len(sizes) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("overlap", [0, 1])
def test_gradients(overlap):
    B, H, N, d, w, H0 = 1, 80, 2000, 64, 300, 16
    q, k, v = synth(B, H, N, d, "bf16", 111)
    dout = synth(B, H, N, d, "bf16", 112)[2]
    ref = co.attn_bwd(q, k, v, dout, w, H0)
    for g, r, name in zip(run_bwd(q, k, v, dout, "bf16", w, H0, overlap=overlap), ref, ("dq", "dk", "dv")):
        check_grad(g, r, "bf16", f"{name} {overlap}", dout)
