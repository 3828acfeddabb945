"""bf16 gradients at head size 64 where the windowed heads' passes share launches with the linear heads' walks: the rule that
cuts the linear heads into fewer segments for them, on the host, with the workspace that serves either cut; and both
cuts (overlap = 1 keeps the passes in launches of their own) against the oracle."""
from __future__ import annotations

import ctypes

import pytest

from oracle import cpu_oracle as co
from paper_2412_19829_amd import binding as gb
from tests.test_gpu_parity import check_grad, run_bwd, synth


class Segments(ctypes.Structure):
    _fields_ = [("len", ctypes.c_int), ("count", ctypes.c_int)]


def _cut(B, H, N, w, H0):
    """Segments of a causal call with the band in its launches, and without (the planner's own functions)."""
    L = gb.lib()
    tiles = getattr(L, "_ZN7gformer19backward_band_tilesEliii")
    tiles.restype, tiles.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    segments = getattr(L, "_ZN7gformer17backward_segmentsEliibl")
    segments.restype = Segments
    segments.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int64]
    t = tiles(B * H0, N, min(w - 1, N - 1), 0)
    return t, segments(B * (H - H0), N, 64, True, t), segments(B * (H - H0), N, 64, True, 0)


# B, H, N, window, H0; segments with the band beside the walks, and apart (256 compute units)
@pytest.mark.parametrize("case", [
    (1, 80, 2000, 300, 16, 8, 11),                                     # what test_gradients runs
    (8, 12, 2048, 256, 4, 8, 11), (8, 12, 4096, 256, 2, 6, 9),         # heavy; as good for the fullest unit
    (4, 16, 4096, 128, 3, 13, 13),                                     # light: 3 x 1152 tiles, 52 x 128 chunks
    (12, 8, 2048, 64, 2, 7, 10),                                       # 3 x 1536 tiles, 72 x 64 chunks: the lightest
    (21, 12, 3297, 32, 3, 4, 4), (12, 32, 1024, 128, 8, 2, 2),         # the fullest unit's chunks would be a third more
    (24, 16, 2500, 128, 8, 2, 4),                                      # so heavy that they may be
    (8, 32, 4096, 256, 6, 3, 3), (8, 32, 3000, 256, 6, 2, 3),          # walks of 64 chunks, of 47
], ids=lambda c: "x".join(map(str, c[:5])))
def test_the_rule(case):
    B, H, N, w, H0, joint, apart = case
    _, a, b = _cut(B, H, N, w, H0)
    assert (a.count, b.count) == (joint, apart)
    for f in (a, b):
        assert f.len % 32 == 0 and (f.count - 1) * f.len < N <= f.count * f.len
    # one size serves both: the statistics and two sums a segment of the cut that has more of them
    stats = (B * H * N * 8 + 255) // 256 * 256
    sums = B * (H - H0) * max(a.count, b.count) * 2 * (64 * 64 + 64) * 4
    for o in (0, 1):
        p = gb.make_params(n_sparse_heads=H0, overlap=o)
        assert gb.gformer_attn_bwd_workspace_bytes(B, H, N, 64, w, p) == stats + sums


def test_both_sides_of_the_line():
    """A tile for every three chunks is where the rule begins."""
    L = gb.lib()
    segments = getattr(L, "_ZN7gformer17backward_segmentsEliibl")
    segments.restype = Segments
    segments.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int64]
    count = lambda t, causal=True: segments(64, 2048, 64, causal, t).count
    assert count(1365) == count(0) == 11 and count(1366) == 8     # 64 heads x 64 chunks / 3 = 1365.3
    assert count(10 ** 6, False) == count(0, False) == 4          # over all keys: no rule


@pytest.mark.gpu
@pytest.mark.parametrize("overlap", [0, 1])
@pytest.mark.parametrize("case", [(1, 80, 2000, 300, 16), (2, 128, 520, 300, 40)], ids=["8 and 11", "2 and 4"])
def test_gradients(case, overlap):
    B, H, N, w, H0 = case
    _, a, b = _cut(*case)
    assert a.count < b.count
    q, k, v = synth(B, H, N, 64, "bf16", 111)
    dout = synth(B, H, N, 64, "bf16", 112)[2]
    ref = co.attn_bwd(q, k, v, dout, w, H0)
    for g, r, name in zip(run_bwd(q, k, v, dout, "bf16", w, H0, overlap=overlap), ref, ("dq", "dk", "dv")):
        check_grad(g, r, "bf16", f"{name} {overlap}", dout)
