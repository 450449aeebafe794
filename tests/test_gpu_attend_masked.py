"""Attention over keys whose scores are minus infinity: they weigh nothing,
wherever they lie, whole key tiles at the start of a workgroup's range and
whole ranges among them."""
import numpy as np
import pytest

from oracle import attend, round_to_bf16

from parity import check_attention, to_np

pytestmark = pytest.mark.gpu


def check(dtype, H, D, q_tokens, keys, masked):
    """masked: rows whose score is -inf for every query (one component of the key against a positive one)."""
    import torch
    from paper_2606_10671_amd.fademem import Cache
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(keys + len(masked))
    q, k, v = (round_to_bf16(rng.standard_normal((n, H, D)).astype(np.float32)) for n in (q_tokens, keys, keys))
    q[..., 0], k[..., 0] = 1.0, 0.0
    k[masked, :, 0] = -np.inf
    cache = Cache(budget=2, heads=H, head_dim=D, tokens_per_block=64, dtype=td)
    dev = [torch.from_numpy(x).to("cuda", td) for x in (q, k, v)]
    lse = torch.empty((H, q_tokens), dtype=torch.float32, device="cuda")
    out = cache.attend(*dev, lse=lse)
    O_ref, L_ref = attend(q, [], [], k, v)
    check_attention(to_np(out), to_np(lse), O_ref, L_ref, dtype, (H, D, q_tokens, keys))


def rows(tiles, size=64):
    return np.concatenate([np.arange(t * size, (t + 1) * size) for t in tiles])


@pytest.mark.parametrize("H,D,q_tokens,keys,tiles", [
    (2, 64, 40, 3 * 64, [0]), (2, 128, 40, 8 * 64, [0, 1]), (1, 128, 40, 20 * 64, [10]),
    (2, 128, 300, 60 * 64, range(0, 60, 6)),   # the first tile of every head part
    (2, 64, 40, 60 * 64 + 5, range(6, 18)),    # parts without a finite score
    (300, 64, 30, 7 * 64, [0, 5]),             # a whole round, then split tiles
    (2, 64, 40, 4 * 64, [1, 3]),               # short calls with exact row maxima
])
def test_bf16_masked_tiles(H, D, q_tokens, keys, tiles):
    check("bf16", H, D, q_tokens, keys, rows(tiles))


@pytest.mark.parametrize("H,D,q_tokens,keys,tiles", [
    (2, 64, 40, 8 * 32, [0, 1, 2, 3]),                 # every split's first tile
    (1, 128, 40, 40 * 32, range(0, 40, 2)),            # whole splits, ranges combined by the second kernel
    (12, 128, 300, 101 * 32 + 7, [0, 1, 2, 50, 51]),   # four query waves, two splits
    (2, 64, 33, 64, [0]),
])
def test_f32_masked_tiles(H, D, q_tokens, keys, tiles):
    check("f32", H, D, q_tokens, keys, rows(tiles, 32))
