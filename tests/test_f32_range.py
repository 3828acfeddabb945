"""Linear heads in single precision where the denominators are near the lower end of a float's range: the result
stays what the formulas give."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cpu_oracle as co
from tests.gpu_util import run_gpu
from tests.test_gpu_parity import synth


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
