"""Single precision on the matrix cores: the sizes where the tiles (16 resident rows, 64 band rows,
chunks of 32 tokens) and the segments of a head end, on both workgroup shapes of the windowed
kernels, with and without the sums' workspace, against the fp64 oracle.  Tolerances: those of the
fp32 mode (max-abs 1e-5, gradients relative to the tensor's largest entry)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from tests.gpu_util import run_gpu, to_device, to_host
from tests.test_gpu_parity import check, check_grad, oracle, run_bwd, synth

# B, H, N, d, window, H0, bidirectional
EDGES = [
    (1, 2, 15, 64, 3, 1, 0), (1, 2, 16, 128, 16, 1, 0), (1, 2, 17, 64, 17, 1, 1),
    (2, 2, 31, 128, 5, 1, 1), (1, 2, 32, 64, 33, 1, 0), (1, 2, 33, 128, 64, 1, 0),
    (1, 2, 63, 64, 65, 1, 1), (1, 2, 129, 64, 15, 1, 0), (1, 2, 257, 128, 80, 1, 0),
    (1, 1, 1300, 64, 8, 0, 0),      # one head in more segments than a walk adds up itself
    (1, 1, 1300, 128, 8, 0, 1),
    (1, 2, 1291, 128, 40, 1, 0),
    (1, 33, 531, 64, 70, 32, 0),    # enough query blocks for the 64-row workgroups
    (2, 17, 523, 128, 61, 16, 1),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", EDGES, ids=lambda c: "x".join(map(str, c)))
def test_forward_and_backward_at_the_edges(case):
    B, H, N, d, w, H0, bidir = case
    q, k, v = synth(B, H, N, d, "f32", 91)
    dout = synth(B, H, N, d, "f32", 92)[2]
    got = run_gpu(q, k, v, "f32", w, H0, bidirectional=bidir)
    check(got, co.attn_fwd(q, k, v, w, H0, bidirectional=bool(bidir)), "f32", str(case))
    ref = co.attn_bwd(q, k, v, dout, w, H0, bidirectional=bool(bidir))
    for g, r, name in zip(run_bwd(q, k, v, dout, "f32", w, H0, bidirectional=bidir), ref, ("dq", "dk", "dv")):
        check_grad(g, r, "f32", f"{name} {case}", dout)


@pytest.mark.gpu
@pytest.mark.parametrize("bidir", [0, 1], ids=["causal", "bidirectional"])
def test_any_workspace_gives_the_layer(bidir):
    """The sums of a head's segments live in the workspace; a call with less of it, or none, runs
    with fewer segments."""
    import torch
    B, H, N, d, w, H0 = 1, 3, 1100, 64, 50, 1
    q, k, v = synth(B, H, N, d, "f32", 93)
    dout = synth(B, H, N, d, "f32", 94)[2]
    p = gb.make_params(dtype=gb.GF_F32, n_sparse_heads=H0, bidirectional=bidir)
    need = gb.gformer_attn_workspace_bytes(B, H, N, d, w, p)
    state = (d * d + d) * 4
    assert need > 4 * (H - H0) * state
    ref = co.attn_fwd(q, k, v, w, H0, bidirectional=bool(bidir))
    tq, tk, tv, tdo = (to_device(x, "f32") for x in (q, k, v, dout))
    stream = torch.cuda.current_stream().cuda_stream
    for nbytes in (need, need - 1, 2 * (H - H0) * state, (H - H0) * state - 1, 0):
        ws = torch.full((max(nbytes, 1),), 0xff, dtype=torch.uint8, device="cuda")
        out = torch.full_like(tq, float("nan"))
        st = gb.gformer_attn_fwd_raw(tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), out.data_ptr(), B, H, N, d, w, p,
                                     ws.data_ptr() if nbytes else 0, nbytes, stream)
        assert st == gb.GF_OK
        torch.cuda.synchronize()
        check(to_host(out), ref, "f32", f"{nbytes} bytes")
    out = torch.full_like(tq, float("nan"))
    assert gb.gformer_attn_fwd_noalloc_raw(tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), out.data_ptr(), B, H, N, d,
                                           w, p, stream) == gb.GF_OK
    torch.cuda.synchronize()
    check(to_host(out), ref, "f32", "noalloc")
    # backward: 8 bytes per token and head are the least (and, over all keys, eight sums per head)
    least = (B * H * N * 8 + 255) // 256 * 256 + (8 * (H - H0) * state if bidir else 0)
    full = gb.gformer_attn_bwd_workspace_bytes(B, H, N, d, w, p)
    assert full > least
    want = co.attn_bwd(q, k, v, dout, w, H0, bidirectional=bool(bidir))
    for nbytes in (full, least + 5 * (H - H0) * state, least):
        ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")
        grads = [torch.full_like(tq, float("nan")) for _ in range(3)]
        st = gb.gformer_attn_bwd_raw(tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), tdo.data_ptr(),
                                     *(g.data_ptr() for g in grads), B, H, N, d, w, p, ws.data_ptr(), nbytes, stream)
        assert st == gb.GF_OK
        torch.cuda.synchronize()
        for g, r, name in zip(grads, want, ("dq", "dk", "dv")):
            check_grad(to_host(g), r, "f32", f"{name}, {nbytes} bytes", dout)
    assert gb.gformer_attn_bwd_raw(tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), tdo.data_ptr(),
                                   *(g.data_ptr() for g in grads), B, H, N, d, w, p, ws.data_ptr(), least - 1,
                                   stream) == gb.GF_ERR_WORKSPACE


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H", [1, 40], ids=["16-row", "64-row"])
def test_what_a_row_does_not_see_does_not_reach_it(H, d):
    """Windowed heads, infinities and NaNs in rows outside a row's window: weight 0 times infinity
    must not appear, in either direction."""
    import torch
    B, N, w, bad = 1, 430, 20, 200
    q, k, v = synth(B, H, N, d, "f32", 95)
    dout = synth(B, H, N, d, "f32", 96)[2]
    clean = run_gpu(q, k, v, "f32", w, H)
    gclean = run_bwd(q, k, v, dout, "f32", w, H)
    q2, k2, v2, d2 = (x.copy() for x in (q, k, v, dout))
    for x, val in ((q2, np.inf), (k2, np.nan), (v2, -np.inf), (d2, np.nan)):
        x[:, :, bad, 3] = val
    got = run_gpu(q2, k2, v2, "f32", w, H)
    rows = [i for i in range(N) if not bad <= i < bad + w]          # rows that do not see token `bad`
    assert np.abs(got[:, :, rows] - clean[:, :, rows]).max() <= 1e-5
    assert not np.isfinite(got[:, :, bad]).any()
    grads = run_bwd(q2, k2, v2, d2, "f32", w, H)
    far = [i for i in range(N) if i < bad - w + 1 or i >= bad + w]   # no window holds both
    for g, c in zip(grads, gclean):
        assert np.abs(g[:, :, far] - c[:, :, far]).max() <= 1e-5 * max(1.0, np.abs(c).max())
    assert not torch.isnan(torch.from_numpy(clean)).any()


@pytest.mark.gpu
def test_prefill_hands_over_the_state_of_the_last_segment():
    import torch
    B, H, N, d, w, H0 = 1, 3, 1300, 64, 30, 1
    q, k, v = synth(B, H, N + 3, d, "f32", 97)
    tq, tk, tv = (to_device(x, "f32") for x in (q, k, v))
    kc, vc = (torch.full((B, H0, w, d), float("nan"), device="cuda") for _ in range(2))
    st = torch.full((B, H - H0, d * d + d), float("nan"), device="cuda")
    out = torch.full((B, H, N, d), float("nan"), device="cuda")
    head = [x[:, :, :N].contiguous() for x in (tq, tk, tv)]
    gb.gformer_attn_prefill(*head, out, kc, vc, st, w, H0)
    ref = oracle(q, k, v, w, H0)
    check(to_host(out), ref[:, :, :N], "f32", "prefill")
    o = torch.full((B, H, d), float("nan"), device="cuda")
    for t in range(N, N + 3):
        gb.gformer_attn_decode(*(x[:, :, t].contiguous() for x in (tq, tk, tv)), o, kc, vc, st, w, H0, t)
        check(to_host(o), ref[:, :, t], "f32", f"decode {t}")


def test_plan_cuts_heads_into_segments():
    """Host arithmetic: whole 32-token chunks, at least 128 tokens a segment, about three workgroups
    per compute unit, and never more carried sums than the library's own array holds."""
    rng = np.random.default_rng(98)
    for _ in range(200):
        d = int(rng.choice([64, 128]))
        B, H, N = int(rng.integers(1, 9)), int(rng.integers(1, 65)), int(rng.integers(1, 40000))
        H0, bidir = int(rng.integers(0, H + 1)), int(rng.integers(0, 2))
        st, pl = gb.gformer_attn_plan(B, H, N, d, 64, gb.make_params(dtype=gb.GF_F32, n_sparse_heads=H0,
                                                                     bidirectional=bidir))
        assert st == gb.GF_OK
        heads = B * (H - H0)
        if heads == 0:
            assert pl.n_segments == 0 and pl.workspace_bytes == 0
            continue
        per = pl.n_segments // heads
        assert per * heads == pl.n_segments and 1 <= per <= 64
        assert (per - 1) * pl.segment_len < N <= per * pl.segment_len
        assert per == 1 or (pl.segment_len % 32 == 0 and pl.segment_len >= 128 and pl.n_segments <= 3 * 256)
        assert pl.workspace_bytes == ((pl.n_segments * (d * d + d) * 4) if per > 1 or bidir else 0)
        assert pl.workspace_bytes <= gb.GFORMER_NOALLOC_SCRATCH_BYTES or per == 1


@pytest.mark.gpu
def test_feature_map_over_its_whole_range():
    """phi alone: after one token the carried Z is phi(k).  The argument's reduction leaves 2^-25 in the exponent, the
    power of two has one ulp: 2 ulp of a normal result, half a unit of the last place of a denormal one besides."""
    import torch
    B, H, d = 4, 64, 128
    k = -np.exp(np.random.default_rng(99).uniform(np.log(1e-8), np.log(104.5), (B, H, 1, d))).astype(np.float32)
    edges = [0.0, -0.0, -1e-45, -1e-38, -0.34657359, -0.34657362, -0.5, -1.0, -87.33654, -87.33655, -88.0, -103.27893, -103.9,
             -103.97208, -103.97209, -104.0, -150.0, -np.inf, 1e-8, 0.5, 3.0, 1e30]
    k[0, 0, 0, :len(edges)] = edges
    tk = torch.from_numpy(k).cuda()
    st = torch.full((B, H, d * d + d), float("nan"), device="cuda")
    out = torch.full_like(tk, float("nan"))
    gb.gformer_attn_prefill(tk, tk, torch.zeros_like(tk), out, None, None, st, 1, 0)
    torch.cuda.synchronize()
    got = st[..., d * d:].cpu().numpy().astype(np.float64)
    x = k[:, :, 0].astype(np.float64)
    ref = np.where(x > 0, x + 1, np.exp(np.minimum(x, 0)))
    assert (np.abs(got - ref) <= 2 * 2.0 ** -23 * ref + 2.0 ** -149).all()
    tk[..., 0] = float("nan")
    gb.gformer_attn_prefill(tk, tk, torch.zeros_like(tk), out, None, None, st, 1, 0)
    assert bool(torch.isnan(st[..., d * d]).all()) and not bool(torch.isnan(st[..., d * d + 1:]).any())


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(1, 3, 1100, 64, 1, 0), (1, 2, 700, 128, 0, 1), (20, 64, 33, 128, 0, 1)],
                         ids=lambda c: "x".join(map(str, c)))
def test_noalloc_gives_the_bits_of_a_workspace_of_its_size(case):
    """The last case asks for more than the library's array holds: not one sum per head, so plain FMAs in both."""
    import torch
    B, H, N, d, H0, bidir = case
    q, k, v = (torch.randn(B, H, N, d, device="cuda", generator=torch.Generator("cuda").manual_seed(s)) for s in (1, 2, 3))
    p = gb.make_params(dtype=gb.GF_F32, n_sparse_heads=H0, bidirectional=bidir)
    held = gb.GFORMER_NOALLOC_SCRATCH_BYTES
    assert (gb.gformer_attn_workspace_bytes(B, H, N, d, 9, p) > held) == (B == 20)
    ws = torch.full((held,), 0xff, dtype=torch.uint8, device="cuda")
    got, want = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    at = (q.data_ptr(), k.data_ptr(), v.data_ptr())
    stream = torch.cuda.current_stream().cuda_stream
    assert gb.gformer_attn_fwd_raw(*at, want.data_ptr(), B, H, N, d, 9, p, ws.data_ptr(), held, stream) == gb.GF_OK
    assert gb.gformer_attn_fwd_noalloc_raw(*at, got.data_ptr(), B, H, N, d, 9, p, stream) == gb.GF_OK
    torch.cuda.synchronize()
    assert bool(torch.isfinite(want).all()) and torch.equal(got.view(torch.int32), want.view(torch.int32))
