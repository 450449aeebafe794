"""fp32 attention at the edges of its tiles (32 queries per wave, 64 or 128
per workgroup, 32 keys per tile dealt to two or four splits): one query and
one key, splits without a tile, ranges combined by the second kernel, and the
two-query-wave and four-query-wave kernels; rows past the last key do not
reach the output, an infinite value does as it does in the definition."""
import numpy as np
import pytest

from oracle import attend

from parity import check_attention, to_np

pytestmark = pytest.mark.gpu


def run(H, D, q, k, v):
    import torch
    from paper_2606_10671_amd.fademem import Cache
    cache = Cache(budget=2, heads=H, head_dim=D, tokens_per_block=64, dtype=torch.float32)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (q, k, v)]
    lse = torch.empty((H, q.shape[0]), dtype=torch.float32, device="cuda")
    out = cache.attend(*dev, lse=lse)
    return to_np(out), to_np(lse)


@pytest.mark.parametrize("H,D,q_tokens,keys", [
    (1, 64, 1, 1), (1, 128, 1, 31), (2, 128, 32, 32), (2, 64, 33, 33), (3, 128, 65, 127), (1, 64, 64, 129),
    (2, 128, 129, 700),    # three 64-query tiles, ranges
    (5, 64, 97, 2048),     # 16 tiles per split
    (12, 128, 129, 4500),  # the four-query-wave kernel, a second 128-query tile of one query
    (9, 64, 500, 2017),    # the same at D = 64, a partial key tile
    (300, 64, 40, 200),    # more query tiles than CUs, one range each
])
def test_f32_edges(H, D, q_tokens, keys):
    rng = np.random.default_rng(H + D + q_tokens + keys)
    q, k, v = (rng.standard_normal((n, H, D)).astype(np.float32) for n in (q_tokens, keys, keys))
    O, L = run(H, D, q, k, v)
    O_ref, L_ref = attend(q, [], [], k, v)
    check_attention(O, L, O_ref, L_ref, "f32", (H, D, q_tokens, keys))


def test_infinite_value_and_tile_padding():
    """V holds an infinity in the last row: its dimension is infinite for every query (its weight is positive), and
    nothing else changes; the 31 padding rows of the tile add nothing."""
    H, D, keys = 2, 128, 33
    rng = np.random.default_rng(9)
    q, k, v = (rng.standard_normal((n, H, D)).astype(np.float32) for n in (70, keys, keys))
    O_ref, L_ref = attend(q, [], [], k, v)
    v[-1, 0, 5] = np.inf
    O, L = run(H, D, q, k, v)
    assert np.isposinf(O[:, 0, 5]).all()
    O[:, 0, 5] = O_ref[:, 0, 5]
    check_attention(O, L, O_ref, L_ref, "f32")
