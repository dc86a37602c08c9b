"""LRU walks over tables of 1, 3 and 4 levels and halos of 128, 256 and 512 steps, one and two words of expert ids:
lru_simulate (with and without a prior state) and cache_simulate's LRU, bit for bit against the oracle."""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# C against K sets the levels (up to K or 2 K: one; up to 3 K: three; above: four) and the halo (12 K, 20 K)
@pytest.mark.parametrize("S,T,K,N,C", [
    (3, 1100, 8, 128, 3), (2, 700, 4, 128, 8), (2, 700, 4, 128, 9), (2, 1025, 4, 128, 13), (2, 1700, 4, 128, 49), (3, 1700, 2, 128, 64),
    (2, 1090, 1, 128, 127), (513, 520, 2, 128, 33), (3, 1100, 6, 64, 4), (2, 700, 6, 64, 7), (2, 1100, 5, 63, 16), (2, 1600, 1, 64, 63),
    (600, 64, 6, 64, 12), (600, 63, 2, 128, 20), (2, 1, 3, 33, 2), (2, 65, 3, 65, 200), (2, 513, 9, 64, 12)])
def test_lru_levels(S, T, K, N, C):
    print(f"lru levels S={S} T={T} K={K} N={N} C={C}", flush=True)
    g = torch.Generator().manual_seed(S * 1009 + T * 31 + K * 7 + C)
    logits = torch.randn(S, T, N, generator=g)
    for t in range(1, T):                                   # sticky, so that walks differ in length
        keep = torch.rand(S, 1, generator=g) < 0.9
        logits[:, t] = torch.where(keep, logits[:, t - 1] + 0.05 * logits[:, t], logits[:, t])
    idx = logits.topk(min(K, N), dim=-1).indices.int().contiguous()
    idx[:, ::7, -1] = idx[:, ::7, 0]                        # a repeated id
    dev = idx.to(DEV)
    steps = [torch.full((S, T), 255, dtype=torch.uint8, device=DEV) for _ in range(3)]
    totals = [torch.full((S,), -1, dtype=torch.int64, device=DEV) for _ in range(3)]
    remoe.cache_simulate(dev, N, C, remoe.REMOE_CACHE_LRU, 3, *steps, *totals, None)
    ref = oracle.cache_policy(idx, N, C, "lru", 3)
    for got, name in zip(steps + totals, ("miss", "uniq", "hit_tok", "total_miss", "total_uniq", "bytes")):
        assert torch.equal(got.cpu().long(), ref[name].long()), name
    for cut in {T, T // 3, max(0, T - 1)}:                  # the whole trace, and two pieces over a state
        state = torch.zeros(S, N, dtype=torch.int32, device=DEV)
        miss, total = [], torch.zeros(S, dtype=torch.int64)
        for a, b in ((0, cut), (cut, T)):
            if a == b:
                continue
            m = torch.full((S, b - a), 255, dtype=torch.uint8, device=DEV)
            n, by = (torch.empty(S, dtype=torch.int64, device=DEV) for _ in range(2))
            remoe.lru_simulate(dev[:, a:b].contiguous(), N, C, 3, a, state, m, n, by)
            miss.append(m.cpu())
            total += n.cpu()
        assert torch.equal(torch.cat(miss, 1).long(), ref["miss"].long()), cut
        assert torch.equal(total, ref["total_miss"].long()), cut
