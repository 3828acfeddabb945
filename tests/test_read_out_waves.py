"""d = 64: the read-out's two forms, the rule that chooses, and the query blocks beside the state pass.  Against the oracle where its tiles
and pieces end (chunks of 64 tokens, queries split in halves of 32), and the bits of the kernels launched one by one on both
sides of the rule that chooses it, the prefill's carried states included."""
from __future__ import annotations

import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from tests.gpu_util import run_gpu, to_device, to_host
from tests.test_gpu_parity import check, synth


# B, H, N, window, H0, identity map, threads of a read-out's workgroup
@pytest.mark.parametrize("case", [
    (1, 12, 2048, 128, 2, 0, 256), (3, 12, 2048, 128, 2, 0, 256), (8, 12, 1024, 128, 2, 0, 512), (8, 12, 4096, 256, 2, 0, 512),
    (8, 12, 4096, 256, 0, 0, 512), (4, 16, 4096, 128, 3, 1, 256), (1, 2, 10, 4, 1, 0, 256),
], ids=lambda c: "x".join(map(str, c)))
def test_plan(case):
    B, H, N, w, H0, identity, threads = case
    phi = gb.GF_PHI_IDENTITY if identity else gb.GF_PHI_ELU1
    st, pl = gb.gformer_attn_plan(B, H, N, 64, w, gb.make_params(n_sparse_heads=H0, phi=phi))
    assert st == gb.GF_OK and pl.linear_threads == threads


# more causal pieces than units: B, H, N, H0, options, pieces, threads
@pytest.mark.parametrize("case", [
    (32, 12, 400, 0, {}, 384, 256), (1, 257, 320, 0, {}, 257, 256), (16, 16, 400, 0, {}, 256, 512), (1, 12, 4096, 0, {"segment_len": 64}, 768, 256),
    (4, 12, 4096, 2, {"segment_len": 64}, 2560, 256), (1, 300, 256, 0, {"phi": gb.GF_PHI_IDENTITY}, 300, 256),
    (32, 12, 577, 0, {"bidirectional": 1}, 384, 512),
], ids=lambda c: "x".join(map(str, c[:4])) + "".join(f"-{k}" for k in c[4]))
def test_plan_of_more_pieces_than_units(case):
    B, H, N, H0, kw, pieces, threads = case
    st, pl = gb.gformer_attn_plan(B, H, N, 64, 16, gb.make_params(n_sparse_heads=H0, **kw))
    assert st == gb.GF_OK and (pl.n_segments, pl.linear_threads) == (pieces, threads)


# every head linear, or the windowed ones with the streaming kernel: B, H, N, window, H0, options, threads
@pytest.mark.parametrize("case", [
    (1, 12, 512, 16, 0, {}, 256), (1, 12, 1024, 16, 0, {}, 256), (1, 12, 2048, 16, 0, {}, 256),      # more sums than chunks
    (4, 12, 512, 16, 0, {}, 512), (1, 8, 686, 16, 0, {}, 512), (1, 12, 4096, 16, 0, {}, 512), (1, 12, 64, 16, 0, {}, 512),
    (1, 12, 512, 16, 0, {"bidirectional": 1}, 256), (1, 12, 64, 16, 0, {"bidirectional": 1}, 256),   # pieces of one chunk
    (3, 12, 1951, 16, 0, {"bidirectional": 1}, 256), (4, 12, 2857, 16, 0, {"bidirectional": 1}, 256), (2, 32, 2326, 16, 0, {"bidirectional": 1}, 512),
    (8, 12, 1000, 16, 0, {"bidirectional": 1}, 512), (1, 600, 200, 16, 0, {"bidirectional": 1}, 256),
    (8, 12, 1000, 16, 0, {"bidirectional": 1, "phi": gb.GF_PHI_IDENTITY}, 256), (4, 16, 4096, 16, 0, {"phi": gb.GF_PHI_IDENTITY}, 512),
    (1, 12, 512, 16, 0, {"phi": gb.GF_PHI_IDENTITY}, 256), (10, 16, 10491, 256, 3, {"phi": gb.GF_PHI_IDENTITY}, 512),
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_plan_without_query_blocks_beside(case):
    B, H, N, w, H0, kw, threads = case
    st, pl = gb.gformer_attn_plan(B, H, N, 64, w, gb.make_params(n_sparse_heads=H0, **kw))
    assert st == gb.GF_OK and pl.linear_threads == threads


# query blocks beside: B, H, N, window, H0, options, threads
@pytest.mark.parametrize("case", [
    (16, 12, 300, 64, 2, {}, 256),                                          # no state pass to share
    (18, 8, 364, 64, 3, {}, 256), (1, 8, 5615, 256, 1, {}, 256), (1, 16, 5484, 256, 11, {}, 512),    # three and four chunks a piece
    (8, 12, 1024, 128, 2, {}, 512), (3, 12, 2472, 38, 1, {}, 512), (1, 16, 16384, 128, 2, {}, 512),
    (6, 16, 1241, 278, 4, {}, 256), (6, 16, 1241, 128, 4, {}, 512),         # long chains of tiles
    (3, 32, 613, 256, 1, {}, 256), (1, 12, 6288, 256, 1, {}, 512), (3, 32, 613, 128, 1, {}, 512),   # ... beside few sums
    (29, 16, 188, 256, 12, {}, 256), (15, 32, 133, 256, 13, {}, 256), (17, 16, 191, 64, 13, {}, 512), (22, 32, 624, 378, 17, {}, 512),   # pieces longer than heads
    (6, 16, 1700, 28, 8, {}, 256), (11, 8, 1278, 128, 7, {}, 256), (2, 16, 2850, 256, 14, {}, 512), (25, 8, 1009, 64, 4, {}, 512),    # two rounds of sums and query blocks
    (8, 12, 1024, 128, 2, {"phi": gb.GF_PHI_IDENTITY}, 256), (9, 8, 5166, 256, 2, {"phi": gb.GF_PHI_IDENTITY}, 256),
    (8, 12, 2048, 128, 2, {"phi": gb.GF_PHI_IDENTITY}, 512), (4, 32, 16384, 64, 1, {"phi": gb.GF_PHI_IDENTITY}, 512),
    (8, 12, 1000, 64, 3, {"bidirectional": 1}, 256), (3, 12, 8811, 256, 2, {"bidirectional": 1}, 256),
    (6, 12, 2863, 64, 2, {"bidirectional": 1}, 512), (32, 12, 577, 64, 3, {"bidirectional": 1}, 512),
    (11, 16, 8014, 282, 11, {"bidirectional": 1}, 512), (13, 16, 644, 256, 13, {"bidirectional": 1}, 256),
    (45, 16, 437, 128, 1, {"bidirectional": 1}, 256), (32, 12, 577, 64, 3, {"bidirectional": 1, "phi": gb.GF_PHI_IDENTITY}, 256),
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_plan_with_query_blocks_beside(case):
    B, H, N, w, H0, kw, threads = case
    st, pl = gb.gformer_attn_plan(B, H, N, 64, w, gb.make_params(n_sparse_heads=H0, **kw))
    assert st == gb.GF_OK and pl.linear_threads == threads


# sums of whole pieces where the query blocks fit the chip beside them, and they come to three of four units: sums a piece
@pytest.mark.parametrize("case", [
    (1, 12, 18682, 128, 2, {}, 1), (2, 16, 9000, 300, 3, {}, 1), (8, 12, 4096, 256, 2, {}, 2), (11, 8, 5282, 128, 1, {}, 2),
    (1, 12, 18682, 128, 0, {}, 2), (2, 16, 11123, 256, 3, {}, 1), (1, 12, 21000, 128, 5, {}, 2),
    (1, 12, 18682, 128, 2, {"impl": gb.GF_IMPL_MFMA_STREAM}, 2), (3, 32, 3750, 508, 6, {}, 1),
    (4, 14, 4096, 64, 1, {}, 2),   # no finer than the workspace has room for
    (3, 16, 3096, 312, 7, {}, 1), (5, 16, 3936, 128, 3, {}, 1), (13, 12, 2520, 256, 2, {}, 2), (9, 32, 6795, 128, 1, {}, 2),
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_plan_of_sums(case):
    B, H, N, w, H0, kw, sub = case
    st, pl = gb.gformer_attn_plan(B, H, N, 64, w, gb.make_params(n_sparse_heads=H0, **kw))
    assert st == gb.GF_OK
    if pl.n_segments % (B * (H - H0)) == 0: assert pl.state_blocks == sub * (pl.n_segments - B * (H - H0))
    else: assert pl.state_blocks <= sub * pl.n_segments and (sub == 1 or pl.state_blocks > pl.n_segments)   # pieces across heads
    slots = pl.workspace_bytes // (4 * (64 * 64 + 64))
    assert slots % pl.n_segments == 0 and slots >= sub * pl.n_segments


# B, H, N, options; every head linear
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (1, 2, 1, {}), (1, 3, 31, {}), (1, 3, 33, {}), (2, 3, 64, {}), (1, 3, 65, {}), (3, 5, 97, {}), (1, 40, 777, {}),
    (2, 12, 300, {}), (1, 3, 700, {}),
    (7, 40, 150, {}),                     # more heads than units: pieces straddle heads
    (1, 260, 197, {}), (2, 12, 1000, {"segment_len": 64}),   # more pieces than units
    (1, 3, 1055, {"eps": 0.5}), (1, 3, 1000, {"segment_len": 64}), (2, 4, 577, {"bidirectional": 1}), (1, 1, 33, {"bidirectional": 1}),
], ids=lambda c: "x".join(map(str, c[:3])) + "".join(f"-{k}" for k in c[3]))
def test_against_oracle(case):
    B, H, N, kw = case
    q, k, v = synth(B, H, N, 64, "bf16", 91)
    args = {x: kw[x] for x in ("eps", "bidirectional") if x in kw}
    check(run_gpu(q, k, v, "bf16", 16, 0, **kw), co.attn_fwd(q, k, v, 16, 0, **args), "bf16", str(case))


# rows of the [B, N, H, d] storage: B, H, N, window, H0, options
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (2, 12, 300, 16, 0, {}), (7, 40, 150, 16, 0, {}), (1, 3, 1000, 16, 0, {"segment_len": 512}), (2, 12, 300, 16, 0, {"bidirectional": 1}),
    (8, 12, 1000, 50, 2, {}),   # query blocks beside the state pass
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_strided_rows(case):
    B, H, N, w, H0, kw = case
    q, k, v = synth(B, H, N, 64, "bf16", 93)
    dense, rows = (run_gpu(q, k, v, "bf16", w, H0, layout=x, **kw) for x in ("bhnd", "bnhd"))
    assert (dense == rows).all()
    if H0 == 0: check(rows, co.attn_fwd(q, k, v, w, H0, bidirectional=bool(kw.get("bidirectional"))), "bf16", str(case))


# features mapped beforehand, every head linear: B, H, N, options
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (1, 3, 1, {}), (1, 3, 33, {}), (1, 3, 65, {}), (3, 5, 97, {}), (1, 3, 700, {}), (7, 40, 150, {}), (1, 40, 777, {}),
    (1, 3, 1000, {"segment_len": 512}), (2, 4, 577, {"bidirectional": 1}),
], ids=lambda c: "x".join(map(str, c[:3])) + "".join(f"-{k}" for k in c[3]))
def test_mapped_features_against_oracle(case):
    import torch
    B, H, N, kw = case
    q, k, v = synth(B, H, N, 64, "bf16", 94)
    q, k = (to_host((to_device(x, "bf16").abs() + 0.125)) for x in (q, k))
    want = co.attn_fwd(q, k, v, 16, 0, phi=co.PHI_IDENTITY, bidirectional=bool(kw.get("bidirectional")))
    got = run_gpu(q, k, v, "bf16", 16, 0, phi=gb.GF_PHI_IDENTITY, **kw)
    check(got, want, "bf16", str(case))
    if kw: return
    # the prefill's read-out: same rows, and the states after the last token
    tq, tk, tv = (to_device(x, "bf16") for x in (q, k, v))
    out, st = torch.full_like(tq, float("nan")), torch.zeros(B, H, 64 * 64 + 64, device="cuda")
    gb.gformer_attn_prefill(tq, tk, tv, out, None, None, st, 16, 0, phi=gb.GF_PHI_IDENTITY)
    torch.cuda.synchronize()
    assert (to_host(out) == got).all()
    A = torch.matmul(tk.double().transpose(2, 3).contiguous(), tv.double())
    # bf16 features and values, fp32 sums of N <= 777 terms (2^-24 each)
    assert float((st[..., :4096].double().view_as(A) - A).norm() / A.norm()) < 2.0 ** -14
    assert float((st[..., 4096:].double() - tk.double().sum(2)).norm() / tk.double().sum(2).norm()) < 2.0 ** -14


# B, H, N, window, H0, options: both forms of the read-out, the query blocks in its launch and in the state pass's
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (3, 12, 2048, 128, 2, {}), (8, 12, 1000, 128, 2, {}), (4, 40, 777, 64, 20, {}), (2, 12, 4100, 300, 4, {}),
    (16, 12, 577, 64, 3, {"bidirectional": 1}), (8, 12, 1000, 50, 2, {"phi": gb.GF_PHI_IDENTITY}),
    (8, 12, 1000, 50, 2, {"softmax_scale": -0.5}), (2, 16, 1000, 50, 2, {"segment_len": 64}), (8, 12, 1000, 128, 2, {"chunk": 128}),
    (8, 12, 2011, 50, 2, {"phi": gb.GF_PHI_IDENTITY}), (23, 12, 577, 33, 1, {"bidirectional": 1}), (26, 12, 577, 64, 2, {"bidirectional": 1}),
    (1, 8, 6000, 64, 1, {"segment_len": 3008}),   # sums of 47 chunks
    (1, 12, 18682, 100, 2, {}), (2, 16, 9001, 300, 3, {}), (3, 16, 3096, 312, 7, {}),   # sums of whole pieces
], ids=lambda c: "x".join(map(str, c[:5])) + "".join(f"-{k}" for k in c[5]))
def test_one_launch_gives_the_bits_of_two(case):
    import torch
    B, H, N, w, H0, kw = case
    q, k, v = (to_device(x, "bf16") for x in synth(B, H, N, 64, "bf16", 92))
    if "phi" in kw:
        q, k = q.abs() + 0.125, k.abs() + 0.125
    p = gb.make_params(n_sparse_heads=H0, **kw)
    ws = torch.empty(max(gb.gformer_attn_workspace_bytes(B, H, N, 64, w, p), 256), dtype=torch.uint8, device="cuda")
    got, want = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    gb.gformer_attn_fwd(q, k, v, got, w, H0, workspace=ws, **kw)
    for m in (gb.GF_LAUNCH_WINDOWED, gb.GF_LAUNCH_LINEAR_STATE, gb.GF_LAUNCH_LINEAR_MAIN):
        gb.gformer_attn_fwd(q, k, v, want, w, H0, workspace=ws, launch_mask=m, **kw)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(want.float()).all())
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    if not kw:   # the prefill's read-out leaves the carried states: A and Z over all tokens
        kc, vc = (torch.zeros(B, H0, w, 64, dtype=q.dtype, device="cuda") for _ in range(2))
        st = torch.zeros(B, H - H0, 64 * 64 + 64, device="cuda")
        pre = torch.full_like(q, float("nan"))
        gb.gformer_attn_prefill(q, k, v, pre, kc, vc, st, w, H0)
        torch.cuda.synchronize()
        assert torch.equal(pre.view(torch.int16), want.view(torch.int16))
        fk = k[:, H0:].double()
        fk = torch.where(fk > 0, fk + 1, torch.exp(fk))
        A = torch.matmul(fk.transpose(2, 3).contiguous(), v[:, H0:].double())
        # phi(k) enters as bf16 (2^-9 of each of N terms, independent: far below 2^-8 of the norm)
        assert float((st[..., :4096].double().view_as(A) - A).norm() / A.norm()) < 2.0 ** -8
        assert float((st[..., 4096:].double() - fk.sum(2)).norm() / fk.sum(2).norm()) < 2.0 ** -8


# B, H, N, d, window, H0, options, launches: sums of 47 chunks and few query blocks are two at d = 64 and three at d = 128
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    (4, 32, 6000, 64, 64, 1, {"segment_len": 3008}, 2), (1, 8, 6000, 128, 64, 1, {"segment_len": 3008}, 3),
    (1, 8, 6000, 64, 64, 0, {"segment_len": 3008}, 2), (1, 8, 6000, 64, 64, 1, {"segment_len": 3008, "softmax_scale": -0.5}, 3),
    (1, 12, 2048, 64, 128, 2, {}, 2), (8, 12, 1000, 64, 128, 2, {}, 2), (8, 12, 1000, 64, 128, 2, {"chunk": 128}, 2),
], ids=lambda c: "x".join(map(str, c[:6])) + "".join(f"-{k}" for k in c[6]))
def test_launches(case):
    import ctypes

    import torch
    B, H, N, d, w, H0, kw, launches = case
    q, k, v = (torch.randn(B, H, N, d, device="cuda").to(torch.bfloat16) for _ in range(3))
    out = torch.empty_like(q)
    p = gb.make_params(n_sparse_heads=H0, **kw)
    ws = torch.empty(max(gb.gformer_attn_workspace_bytes(B, H, N, d, w, p), 256), dtype=torch.uint8, device="cuda")
    graph, side = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    gb.gformer_attn_fwd(q, k, v, out, w, H0, workspace=ws, **kw)   # loads the kernels before the capture
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        gb.gformer_attn_fwd(q, k, v, out, w, H0, workspace=ws, **kw)
    nodes = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == launches
