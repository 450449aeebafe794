"""The update's plan where it changes kernel: memories of up to 63 entries
(one lane per entry) and of more.  From an empty memory past its budget,
chunks of one to four frames, each call compared with the oracle's one by one
updates (metadata, decisions, stored bits) and with the host replay of the
slot table; low exponents and a budget of 2 merge an entry twice within one
call, exact ties (beta = 1 and 0.5) take the oldest pair."""
import numpy as np
import pytest

from oracle import OracleCache

from parity import check_entries, check_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,F,beta,anchor,op,staged", [
    (2, 4, 0.3, True, "sqrt_span", False), (2, 3, 0.05, False, "sqrt_span", True), (3, 4, 1.0, False, "average", False),
    (4, 2, 0.5, True, "max", True), (21, 3, 0.3, True, "sqrt_span", True), (59, 4, 0.3, True, "sqrt_span", True),
    (62, 3, 0.5, False, "select_nearest", False), (63, 4, 0.3, True, "sqrt_span", True), (63, 1, 1.0, True, "max", False),
    (64, 4, 0.3, True, "sqrt_span", True), (70, 3, 0.5, False, "sqrt_span", False),
])
def test_plan_edges(M, F, beta, anchor, op, staged):
    import torch
    from paper_2606_10671_amd.fademem import Cache
    N, H, D = 1, 1, 64
    print(f"plan M={M} F={F} beta={beta} anchor={anchor} op={op} staged={staged}", flush=True)
    cache = Cache(budget=M, heads=H, head_dim=D, tokens_per_block=N, beta=beta, anchor=anchor, dtype=torch.bfloat16,
                  merge_op=op, stage_frames=F if staged else 0)
    oc = OracleCache(budget=M, beta=beta, anchor=anchor, storage="bf16", operator=op)
    rng = np.random.default_rng(M * 10 + F)
    t = 0
    for c in range(M // F + 25):
        kv = [torch.from_numpy(rng.standard_normal((F * N, H, D)).astype(np.float32)).to(torch.bfloat16) for _ in "kv"]
        if staged:
            for f, (ks, vs) in enumerate(cache.stage(F)[0]):
                ks.copy_(kv[0][f * N:(f + 1) * N])
                vs.copy_(kv[1][f * N:(f + 1) * N])
            cache.update_staged(F, t)
        else:
            cache.update(kv[0].cuda(), kv[1].cuda(), t)
        for f in range(F):
            oc.update(kv[0][f * N:(f + 1) * N].float().numpy(), kv[1][f * N:(f + 1) * N].float().numpy(), t + f)
        t += F
        check_state(cache, oc, (c, t))
        cache.verify()
    check_entries(cache, oc)
    total, log = cache.merge_log()
    assert total == t - M and log == list(oc.merge_log)[-len(log):]
