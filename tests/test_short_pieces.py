"""Small calls cut their linear heads into pieces of two to seven chunks: against the oracle at the
ends of the rule's range, and with a workspace that only holds the cut into pieces of eight."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from tests.gpu_util import run_gpu, to_device, to_host
from tests.test_gpu_parity import check, synth

# B, H, N, d, window, H0; chunks of 64 tokens per piece
CASES = [
    (1, 3, 193, 64, 20, 1, 2),      # four chunks a head, the last with one token: the rule's shortest
    (1, 3, 256, 128, 20, 1, 2),
    (1, 2, 512, 64, 30, 1, 2), (1, 3, 513, 128, 30, 1, 5), (1, 12, 1000, 64, 64, 2, 2),
    (1, 12, 1090, 64, 64, 2, 4),    # more than eight pieces of two: four
    (2, 16, 1024, 64, 64, 3, 3),    # pieces of two would crowd the chip: three
    (1, 8, 4096, 128, 64, 1, 4),    # 64 chunks, the longest heads of the rule at d = 128
    (1, 10, 2500, 64, 500, 2, 4), (1, 310, 320, 64, 16, 10, 5),   # more heads than compute units, a whole head each
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_plan(case):
    B, H, N, d, w, H0, piece = case
    st, pl = gb.gformer_attn_plan(B, H, N, d, w, gb.make_params(n_sparse_heads=H0))
    per = -(-(-(-N // 64)) // piece)
    assert st == gb.GF_OK and pl.segment_len == 64 * piece and pl.n_segments == B * (H - H0) * per


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_short_pieces_against_oracle(case):
    B, H, N, d, w, H0, _ = case
    q, k, v = synth(B, H, N, d, "bf16", 71)
    check(run_gpu(q, k, v, "bf16", w, H0), co.attn_fwd(q, k, v, w, H0), "bf16", str(case))


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(2, 16, 1024, 64, 64, 3, 52 * 2), (1, 12, 512, 128, 64, 2, 0)],
                         ids=lambda c: "x".join(map(str, c)))
def test_a_workspace_for_pieces_of_eight_still_serves(case):
    import torch
    B, H, N, d, w, H0, slots = case
    q, k, v = synth(B, H, N, d, "bf16", 72)
    p = gb.make_params(n_sparse_heads=H0)
    state = (d * d + d) * 4
    assert gb.gformer_attn_workspace_bytes(B, H, N, d, w, p) > slots * state
    tq, tk, tv = (to_device(x, "bf16") for x in (q, k, v))
    ws = torch.empty(max(slots * state, 1), dtype=torch.uint8, device="cuda")
    out = torch.full_like(tq, float("nan"))
    args = (tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), out.data_ptr(), B, H, N, d, w, p)
    stream = torch.cuda.current_stream().cuda_stream
    if slots:
        assert gb.gformer_attn_fwd_raw(*args, ws.data_ptr(), slots * state - 1, stream) == gb.GF_ERR_WORKSPACE
        assert gb.gformer_attn_fwd_raw(*args, 0, 0, stream) == gb.GF_ERR_WORKSPACE
    assert gb.gformer_attn_fwd_raw(*args, ws.data_ptr() if slots else 0, slots * state, stream) == gb.GF_OK
    torch.cuda.synchronize()
    assert np.isfinite(to_host(out)).all()
    check(to_host(out), co.attn_fwd(q, k, v, w, H0), "bf16", str(case))


@pytest.mark.gpu
def test_a_misaligned_workspace_where_pieces_of_eight_need_none():
    import torch
    B, H, N, d, w, H0 = 1, 12, 512, 64, 64, 2
    q, k, v = synth(B, H, N, d, "bf16", 73)
    p = gb.make_params(n_sparse_heads=H0)
    need = gb.gformer_attn_workspace_bytes(B, H, N, d, w, p)
    tq, tk, tv = (to_device(x, "bf16") for x in (q, k, v))
    ws = torch.zeros(need + 512, dtype=torch.uint8, device="cuda")
    out = torch.full_like(tq, float("nan"))
    at = (ws.data_ptr() + 255) // 256 * 256 + 16
    assert gb.gformer_attn_fwd_raw(tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), out.data_ptr(), B, H, N, d, w, p, at, need,
                                   torch.cuda.current_stream().cuda_stream) == gb.GF_OK
    torch.cuda.synchronize()
    check(to_host(out), co.attn_fwd(q, k, v, w, H0), "bf16", "misaligned")
    assert not ws.any()   # and nothing was written there
    # where that cut needs one too, the pointer is refused as it always was
    tq, tk, tv = (torch.zeros(1, 12, 2048, 64, dtype=torch.bfloat16, device="cuda") for _ in range(3))
    need = gb.gformer_attn_workspace_bytes(1, 12, 2048, 64, w, p)
    ws = torch.zeros(need + 512, dtype=torch.uint8, device="cuda")
    at = (ws.data_ptr() + 255) // 256 * 256 + 16
    assert gb.gformer_attn_fwd_raw(tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), torch.empty_like(tq).data_ptr(), 1, 12, 2048,
                                   64, w, p, at, need, torch.cuda.current_stream().cuda_stream) == gb.GF_ERR_INVALID_ARG
