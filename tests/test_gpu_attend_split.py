"""bf16 attention where the work split changes form: key tiles around the
smallest split, one head part and a tail, many head parts, head parts with
and without tails, a last round that is split after a whole one, waves
without queries."""
import numpy as np
import pytest

from oracle import attend
from paper_2606_10671_amd.synth import NumpyWanStream

from parity import check_attention, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,D,q_tokens,keys", [
    (2, 128, 40, 5 * 64),          # below the smallest split: one workgroup per tile
    (2, 128, 40, 5 * 64 + 1),      # 6 key tiles: one head part and a tail
    (1, 64, 256, 12 * 64),         # two head parts and a tail
    (3, 128, 33, 63 * 64 + 5),     # 10 head parts, the second wave with one query
    (3, 64, 300, 64 * 64),         # a second query tile of 44 queries
    (60, 128, 250, 24 * 64 + 7),   # 4 head parts, tails dropped (too little to take)
    (100, 64, 70, 20 * 64),        # 2 head parts, 56 groups sharing 100 tails
    (130, 64, 257, 20 * 64 - 63),  # one whole round of 256, then 4 tiles split
    (1, 128, 1, 600 * 64),         # the cap on head parts
])
def test_split_attention(H, D, q_tokens, keys):
    import torch
    from paper_2606_10671_amd.fademem import Cache
    cache = Cache(budget=2, heads=H, head_dim=D, tokens_per_block=64, dtype=torch.bfloat16)
    gen = NumpyWanStream(11, keys, H, D)
    k, v = gen.frame()
    q = gen.queries(q_tokens)
    dev = [torch.from_numpy(x).to("cuda", torch.bfloat16) for x in (q, k, v)]
    lse = torch.empty((H, q_tokens), dtype=torch.float32, device="cuda")
    out = cache.attend(*dev, lse=lse)
    O_ref, L_ref = attend(q, [], [], k, v)
    check_attention(to_np(out), to_np(lse), O_ref, L_ref, "bf16", (H, D, q_tokens, keys))
