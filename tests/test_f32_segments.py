"""How a single-precision call cuts its linear heads: the segments per head that the rule names, and the layer with its
gradients at a cut of two workgroups per compute unit, which earlier tests do not reach."""
from __future__ import annotations

import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from tests.test_gpu_parity import check, check_grad, run_bwd, synth
from tests.gpu_util import run_gpu


# B, H, N, d, H0, bidirectional, segments per head (256 compute units)
@pytest.mark.parametrize("case", [
    (4, 16, 2048, 64, 3, 0, 8), (4, 16, 2048, 64, 0, 0, 8),    # two a unit, added up in place
    (2, 12, 1500, 64, 4, 0, 10),                               # one a unit: more of them, scanned
    (16, 12, 1024, 64, 2, 0, 4), (8, 16, 700, 64, 4, 1, 5),    # three a unit; over all keys
    (1, 1, 127, 64, 0, 0, 1), (1, 1, 256, 128, 0, 0, 2), (1, 300, 4000, 64, 0, 0, 2), (8, 100, 4000, 64, 0, 0, 1),
], ids=lambda c: "x".join(map(str, c)))
def test_count(case):
    B, H, N, d, H0, bidir, count = case
    st, pl = gb.gformer_attn_plan(B, H, N, d, 16, gb.make_params(dtype=gb.GF_F32, n_sparse_heads=H0, bidirectional=bidir))
    assert st == gb.GF_OK and pl.n_segments == B * (H - H0) * count


@pytest.mark.gpu
def test_two_workgroups_a_unit():
    B, H, N, d, w, H0 = 2, 30, 1030, 64, 8, 2
    st, pl = gb.gformer_attn_plan(B, H, N, d, w, gb.make_params(dtype=gb.GF_F32, n_sparse_heads=H0))
    assert 256 < pl.n_segments <= 512
    q, k, v = synth(B, H, N, d, "f32", 101)
    dout = synth(B, H, N, d, "f32", 102)[2]
    check(run_gpu(q, k, v, "f32", w, H0), co.attn_fwd(q, k, v, w, H0), "f32", "forward")
    for g, r, name in zip(run_bwd(q, k, v, dout, "f32", w, H0), co.attn_bwd(q, k, v, dout, w, H0), ("dq", "dk", "dv")):
        check_grad(g, r, "f32", name, dout)
