"""Cache policies where victims leave in groups: steps that overflow the cache alone, both halves of the expert
range, repeated ids, periodic traces (equal counts and equal next requests)."""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
POLICY = {"lru": remoe.REMOE_CACHE_LRU, "fifo": remoe.REMOE_CACHE_FIFO, "lfu": remoe.REMOE_CACHE_LFU, "belady": remoe.REMOE_CACHE_BELADY}


def _trace(kind, S, T, K, N):
    g = torch.Generator().manual_seed(S * 7919 + T * 31 + K + N)
    if kind == "distinct":
        return torch.rand(S, T, N, generator=g).topk(K, dim=-1).indices.int().contiguous()
    if kind == "periodic":
        t = torch.arange(T)[None, :, None] * K + torch.arange(K)[None, None, :] + torch.arange(S)[:, None, None]
        return (t % N).int().contiguous()
    return torch.randint(0, N, (S, T, K), generator=g).int().contiguous()           # ids that repeat within a step


@pytest.mark.parametrize("policy", list(POLICY))
@pytest.mark.parametrize("S,T,K,N,C,kind", [
    (2, 150, 64, 128, 5, "distinct"), (3, 65, 40, 64, 39, "distinct"), (2, 130, 8, 128, 7, "distinct"), (2, 200, 3, 128, 70, "distinct"),
    (2, 129, 2, 65, 1, "distinct"), (3, 64, 6, 64, 64, "distinct"), (2, 160, 8, 128, 20, "periodic"), (2, 160, 5, 63, 12, "periodic"),
    (3, 100, 8, 128, 16, "any"), (3, 100, 8, 20, 4, "any"),
])
def test_policies_match_oracle(policy, S, T, K, N, C, kind):
    print(f"cache groups {policy} S={S} T={T} K={K} N={N} C={C} {kind}", flush=True)
    idx = _trace(kind, S, T, K, N)
    steps = [torch.full((S, T), 255, dtype=torch.uint8, device=DEV) for _ in range(3)]
    totals = [torch.full((S,), -1, dtype=torch.int64, device=DEV) for _ in range(3)]
    ws = torch.empty(max(256, remoe.remoe_cache_workspace_bytes(S, T, K, POLICY[policy])), dtype=torch.uint8, device=DEV)
    remoe.cache_simulate(idx.to(DEV), N, C, POLICY[policy], 3, *steps, *totals, ws)
    torch.cuda.synchronize()
    ref = oracle.cache_policy(idx, N, C, policy, 3)
    for got, name in zip(steps + totals, ("miss", "uniq", "hit_tok", "total_miss", "total_uniq", "bytes")):
        assert torch.equal(got.cpu().long(), ref[name].long()), name
