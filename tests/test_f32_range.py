"""Linear heads in single precision where the denominators, or the gradients that come in, are near the ends of
a float's range: the result stays what the formulas give as long as it is inside that range itself."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cpu_oracle as co
from tests.gpu_util import run_gpu
from tests.test_gpu_parity import check_grad, run_bwd, synth


def small_denominators(N, d, log_den):
    """Four features of about exp(log_den / 2) / 2 each, so that a token adds exp(log_den) to a denominator; the
    other features are zero in a float."""
    rng = np.random.default_rng(60)
    q = np.full((1, 2, N, d), -110.0, np.float32)
    k = q.copy()
    for x in (q, k):
        x[..., 5:9] = log_den / 2 - np.log(2.0) + rng.uniform(-0.3, 0.3, (1, 2, N, 4))
    return q, k, synth(1, 2, N, d, "f32", 61)[2]


@pytest.mark.gpu
@pytest.mark.parametrize("bidir", [0, 1], ids=["causal", "bidirectional"])
@pytest.mark.parametrize("d", [64, 128])
def test_denominators_below_the_reciprocals_range(d, bidir):
    # 40 tokens of 4e-41: every denominator is below 2.9e-39.  A product of two features is 1e-41, in which a
    # rounding of 0.7e-45 is 7e-5; three such roundings (denominator, weight, weight times value) over a sum of at
    # least four products of either sign
    q, k, v = small_denominators(40, d, -93.0)
    got = run_gpu(q, k, v, "f32", 8, 0, bidirectional=bidir)
    ref = co.attn_fwd(q, k, v, 8, 0, bidirectional=bool(bidir))
    assert np.abs(got - ref).max() <= 2e-4 * np.abs(v).max()


@pytest.mark.gpu
@pytest.mark.parametrize("bidir", [0, 1], ids=["causal", "bidirectional"])
@pytest.mark.parametrize("d", [64, 128])
def test_gradients_under_small_denominators(d, bidir):
    # 9 tokens of 3e-40: a product of two features is 8e-41, in which a rounding of 0.7e-45 is 9e-6.  A gradient is a
    # difference of two terms with up to three such factors each, some times as large as the largest entry
    q, k, v = small_denominators(9, d, -91.0)
    dout = synth(1, 2, 9, d, "f32", 62)[2] * np.float32(1e-3)   # dO / den has to be a float
    ref = co.attn_bwd(q, k, v, dout, 8, 0, bidirectional=bool(bidir))
    for g, r, name in zip(run_bwd(q, k, v, dout, "f32", 8, 0, bidirectional=bidir), ref, ("dq", "dk", "dv")):
        assert np.abs(g - r).max() <= 2e-4 * np.abs(r).max(), name


@pytest.mark.gpu
@pytest.mark.parametrize("bidir", [0, 1], ids=["causal", "bidirectional"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("power", [118, -60])
def test_gradients_scale_with_the_gradient_that_comes_in(d, bidir, power):
    """The gradients are linear in dO: times a power of two they are the same bits, without overflow in between."""
    q, k, v = synth(1, 3, 100, d, "f32", 63)
    dout = synth(1, 3, 100, d, "f32", 64)[2]
    f = np.float32(2.0) ** np.float32(power)
    base = run_bwd(q, k, v, dout, "f32", 8, 1, bidirectional=bidir)
    ref = co.attn_bwd(q, k, v, dout, 8, 1, bidirectional=bool(bidir))
    for x, g, r, name in zip(run_bwd(q, k, v, dout * f, "f32", 8, 1, bidirectional=bidir), base, ref, ("dq", "dk", "dv")):
        check_grad(g, r, "f32", name, dout)
        assert np.array_equal(x, g * float(f)), name
