"""The softmax weights of fp32 attention at the ends of their range: weights
below 2^-126, fp32's smallest normal number, still count; and scores that are
small against their terms: the scale is not rounded into the products."""
import numpy as np
import pytest

from oracle import attend

from parity import check_attention
from test_gpu_attend_f32 import run

pytestmark = pytest.mark.gpu

SHAPES = [(1, 64, 4, 40), (2, 128, 33, 700), (12, 128, 129, 4500), (9, 64, 500, 2017)]  # the last two: four query waves


@pytest.mark.parametrize("H,D,q_tokens,keys", SHAPES)
@pytest.mark.parametrize("exponent", [120, 127, 135, 148])
def test_subnormal_weights(H, D, q_tokens, keys, exponent):
    """Key 5 weighs 2^-exponent of the others: an infinite value of it reaches the output (0 times infinity would be
    NaN), a large finite one adds what it is worth.  fp32 holds that weight to 2^-149."""
    q, k, v = np.zeros((q_tokens, H, D), np.float32), np.zeros((keys, H, D), np.float32), np.ones((keys, H, D), np.float32)
    q[..., 0] = np.sqrt(D)
    k[5, :, 0] = -exponent * np.log(2.0)
    v[5, :, 3], v[5, :, 4] = np.inf, 3e38
    O, _ = run(H, D, q, k, v)
    assert np.isposinf(O[..., 3]).all()
    w, n = 2.0 ** -exponent, float(keys - 1)
    # The exponent's rounding (2^-17 of 148, times ln 2), the weight's own, the sums'.
    bound = (w * 1e-5 + 2.0 ** -149) * 3e38 / n + 1e-6 * (1 + w * 3e38 / n)
    assert np.abs(O[..., 4] - (1 + w * 3e38 / n)).max() <= bound
    assert np.abs(O[..., 0] - 1.0).max() <= 1e-6


@pytest.mark.parametrize("H,D,q_tokens,keys", SHAPES)
def test_subnormal_rescale(H, D, q_tokens, keys):
    """The last key outweighs the ones before by 2^140: what they left, an infinite value among it, is kept."""
    q, k, v = np.zeros((q_tokens, H, D), np.float32), np.zeros((keys, H, D), np.float32), np.ones((keys, H, D), np.float32)
    q[..., 0] = np.sqrt(D)
    k[-1, :, 0] = 140 * np.log(2.0)
    v[5, :, 3] = np.inf
    O, _ = run(H, D, q, k, v)
    assert np.isposinf(O[..., 3]).all()
    assert np.abs(O[..., 0] - 1.0).max() <= 1e-6


@pytest.mark.parametrize("H,D,q_tokens,keys", SHAPES)
def test_scores_that_fp32_holds_are_not_rounded(H, D, q_tokens, keys):
    """Scores that are small sums of large products, all exact in fp32 (x 2^20 - x 2^20 + a whole number):
    the scale, which fp32 does not hold, must not be rounded into the products.  Rounded into q it is off by up to
    2^-24 of 0.18 x 2^20 there, differently for q = 1 and q = x, and moves weights by about 1%."""
    rng = np.random.default_rng(keys)
    q, k = np.zeros((q_tokens, H, D), np.float32), np.zeros((keys, H, D), np.float32)
    v = rng.standard_normal((keys, H, D)).astype(np.float32)
    large = rng.choice([-1.0, 0.0, 1.0], (keys, H)).astype(np.float32) * 2.0 ** 20
    k[..., 0], k[..., 4] = large, rng.integers(0, 32, (keys, H))
    q[..., 2], q[..., 4] = 1.0, 1.0
    for x in (3, 5, 7):
        q[..., 0], k[..., 2] = x, -x * large
        O, L = run(H, D, q, k, v)
        O_ref, L_ref = attend(q, [], [], k, v)
        check_attention(O, L, O_ref, L_ref, "f32", (x, H, D, q_tokens, keys))
