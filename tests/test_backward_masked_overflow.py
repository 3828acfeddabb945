"""Causal bf16 gradients of the linear heads where dO_i . v_j of a later token j overflows a float: token i does not see
j, so the rows of dq up to j stay what they are with an ordinary v_j, bit for bit, and every gradient is finite."""
from __future__ import annotations

import numpy as np
import pytest

from tests.test_gpu_parity import run_bwd, synth


# query i, later key j of the same 32 x 32 (d = 128) or 16 x 16 (d = 64) tile and of neighbouring ones, first and second chunk
@pytest.mark.gpu
@pytest.mark.parametrize("d,i,j", [(128, 0, 1), (128, 3, 31), (128, 1, 40), (128, 33, 62), (128, 70, 95), (128, 100, 127),
                                   (64, 0, 1), (64, 2, 15), (64, 5, 20), (64, 17, 31), (64, 33, 47), (64, 50, 63)])
def test_rows_before_the_key_do_not_change(d, i, j):
    N = 130
    q, k, v = synth(1, 2, N, d, "bf16", 131)
    dout = synth(1, 2, N, d, "bf16", 132)[2]
    dout[:, :, i] *= np.float32(2.0 ** 66)
    base = run_bwd(q, k, v, dout, "bf16", 8, 0)
    v[:, :, j] = dout[:, :, i]   # dO_i . v_j = |dO_i|^2, above 2^128
    assert np.square(dout[:, :, i].astype(np.float64)).sum(-1).min() > 2.0 ** 129
    grads = run_bwd(q, k, v, dout, "bf16", 8, 0)
    for g, name in zip(grads, ("dq", "dk", "dv")):
        assert np.isfinite(g).all(), name
    assert np.array_equal(grads[0][:, :, :j], base[0][:, :, :j])
