"""bf16 attention where one key holds most of a row's weight and comes after
the first key tile: calls too short to be split run with the exact row max, so
that key's weight is 1 and takes no rounding."""
import numpy as np
import pytest

from oracle import attend, round_to_bf16

from parity import to_np

pytestmark = pytest.mark.gpu


def run(H, D, q, k, v):
    import torch
    from paper_2606_10671_amd.fademem import Cache
    cache = Cache(budget=2, heads=H, head_dim=D, tokens_per_block=64, dtype=torch.bfloat16)
    dev = [torch.from_numpy(x).to("cuda", torch.bfloat16) for x in (q, k, v)]
    lse = torch.empty((H, q.shape[0]), dtype=torch.float32, device="cuda")
    return to_np(cache.attend(*dev, lse=lse)), to_np(lse)


@pytest.mark.parametrize("H,D,q_tokens,keys,first", [
    (2, 64, 40, 65, 0), (2, 128, 40, 128, 0), (3, 128, 300, 192, 0), (24, 64, 33, 256, 0), (2, 64, 40, 320, 0),
    (2, 128, 257, 320, 0),
    (140, 64, 40, 7 * 64, 0),    # too few groups left for tails of two tiles
    (200, 128, 20, 12 * 64, 0),  # the same with four tails per group
    (258, 64, 20, 256, 256),     # one whole round of 256, then 2 tiles
])
def test_dominant_weight_is_not_rounded(H, D, q_tokens, keys, first):
    """Each query points at one key past the first tile, a few times heavier than all others together but less than
    2^8 times the first tile's largest.  Bound per element: the output's own rounding (half a unit in the last place)
    plus, for every other key, its weight's rounding (2^-8 of it) against its value; 1% of both for fp32 sums."""
    rng = np.random.default_rng(D + keys)
    k, v = (round_to_bf16(rng.standard_normal((keys, H, D)).astype(np.float32)) for _ in "kv")
    target = rng.integers(64, keys, q_tokens)
    norm = np.linalg.norm(k[target], axis=2, keepdims=True)
    q = round_to_bf16((k[target] / norm * 7.5).astype(np.float32))  # its score: 7.5 |k| / sqrt(D), about 7.5
    O, L = run(H, D, q, k, v)
    s = np.einsum("qhd,khd->hqk", q[:, first:].astype(np.float64), k[:, first:].astype(np.float64)) / np.sqrt(D)
    w = np.exp(s - s.max(2, keepdims=True))
    w /= w.sum(2, keepdims=True)
    O_ref, L_ref = attend(q[:, first:], [], [], k[:, first:], v[:, first:])
    others = np.where(w == w.max(2, keepdims=True), 0.0, w)
    rounded = np.einsum("hqk,khd->qhd", others, np.abs(v[:, first:]).astype(np.float64)) * 2.0 ** -8
    ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(O_ref) + rounded, 1e-30))) - 7)
    bound = 1.01 * (0.5 * ulp + rounded) + 1e-6
    over = np.abs(O[:, first:].astype(np.float64) - O_ref) / bound
    assert over.max() <= 1.0, (over.max(), float((over > 1).mean()))
    assert np.abs(L[first:] - L_ref).max() <= 1e-5 * max(1.0, np.abs(L_ref).max())
