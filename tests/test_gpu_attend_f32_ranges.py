"""fp32 attention of few queries over many keys: the key axis is cut into as
many ranges as pay, up to a few hundred."""
import numpy as np
import pytest

from oracle import attend

from parity import check_attention
from test_gpu_attend_f32 import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,D,q_tokens,keys", [
    (1, 128, 128, 65536),  # four query waves, about 128 ranges
    (1, 64, 20, 40001),    # two, about 100
    (1, 128, 1, 4097),
    (5, 64, 64, 30000),    # ranges limited by the slots
])
def test_f32_ranges(H, D, q_tokens, keys):
    rng = np.random.default_rng(H + D + q_tokens + keys)
    q, k, v = (rng.standard_normal((n, H, D)).astype(np.float32) for n in (q_tokens, keys, keys))
    O, L = run(H, D, q, k, v)
    O_ref, L_ref = attend(q, [], [], k, v)
    check_attention(O, L, O_ref, L_ref, "f32", (H, D, q_tokens, keys))
