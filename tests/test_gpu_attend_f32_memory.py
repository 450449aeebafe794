"""fp32 attention over a filled memory: key tiles of 32 rows that hold many
entries, cross from one entry to the next, or from the last entry into the
chunk, in the kernels of two and of four query waves, against the oracle."""
import numpy as np
import pytest

from oracle import attend

from parity import check_attention, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,D,N,held,q_tokens,cur", [
    (2, 64, 1, 40, 5, 1), (2, 128, 10, 7, 33, 20), (1, 64, 31, 5, 40, 31), (2, 128, 32, 4, 64, 40), (3, 64, 33, 6, 70, 65),
    (2, 128, 40, 3, 30, 0),     # no chunk: the last tile ends in the memory
    (2, 128, 1, 200, 100, 1),   # entries of one row, more of them than a wave has lanes
    # Four query waves (from 8192 tiles of 32 keys x 32 queries on), double-buffered.
    (12, 128, 390, 9, 400, 401), (12, 64, 33, 63, 400, 50), (12, 128, 10, 63, 1000, 7), (16, 64, 32, 20, 900, 129),
])
def test_f32_entries(H, D, N, held, q_tokens, cur):
    import torch
    from paper_2606_10671_amd.fademem import Cache
    rng = np.random.default_rng(N * 100 + held)
    # Entry i's rows carry an offset of their own, so a row of a neighbouring entry is not mistaken for the right one.
    mem = rng.standard_normal((2, held, N, H, D)).astype(np.float32) + np.arange(held, dtype=np.float32)[:, None, None, None] % 5
    q, k, v = (rng.standard_normal((n, H, D)).astype(np.float32) for n in (q_tokens, cur, cur))
    cache = Cache(budget=max(2, held), heads=H, head_dim=D, tokens_per_block=N, dtype=torch.float32)
    kv = [(torch.from_numpy(mem[0, i]).cuda(), torch.from_numpy(mem[1, i]).cuda()) for i in range(held)]
    cache.restore({"count": held, "first": list(range(held)), "span": [1] * held, "pos_sum": list(range(held)),
                   "newest": held - 1, "kv": [kv]})
    lse = torch.empty((H, q_tokens), dtype=torch.float32, device="cuda")
    qd, kd, vd = (torch.from_numpy(x).cuda() for x in (q, k, v))
    out = cache.attend(qd, kd, vd, lse=lse)
    O_ref, L_ref = attend(q, list(mem[0]), list(mem[1]), k, v)
    check_attention(to_np(out), to_np(lse), O_ref, L_ref, "f32", (H, D, N, held, q_tokens, cur))
