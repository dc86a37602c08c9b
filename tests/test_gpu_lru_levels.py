"""LRU walks over tables of 1, 3 and 4 levels, past the staged steps and into a prior state, two and four words of expert ids:
lru_simulate (with and without a prior state) and cache_simulate's LRU, bit for bit against the oracle."""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# C against K sets the levels (up to K or 2 K: one; up to 3 K: three; above: four)
@pytest.mark.parametrize("S,T,K,N,C", [
    (3, 1100, 8, 128, 3), (2, 700, 4, 128, 8), (2, 700, 4, 128, 9), (2, 1025, 4, 128, 13), (2, 1700, 4, 128, 49), (3, 1700, 2, 128, 64),
    (2, 1090, 1, 128, 127), (513, 520, 2, 128, 33), (3, 1100, 6, 64, 4), (2, 700, 6, 64, 7), (2, 1100, 5, 63, 16), (2, 1600, 1, 64, 63),
    (600, 64, 6, 64, 12), (600, 63, 2, 128, 20), (2, 1, 3, 33, 2), (2, 65, 3, 65, 200), (2, 513, 9, 64, 12)])
def test_lru_levels(S, T, K, N, C, popularity=0.0):
    print(f"lru levels S={S} T={T} K={K} N={N} C={C} popularity={popularity}", flush=True)
    g = torch.Generator().manual_seed(S * 1009 + T * 31 + K * 7 + C)
    logits = torch.randn(S, T, N, generator=g)
    for t in range(1, T):                                   # sticky, so that walks differ in length
        keep = torch.rand(S, 1, generator=g) < 0.9
        logits[:, t] = torch.where(keep, logits[:, t - 1] + 0.05 * logits[:, t], logits[:, t])
    if popularity:
        logits += popularity * torch.randn(S, 1, N, generator=g)
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


@pytest.mark.parametrize("S,T,K,N,C", [
    (2, 2100, 8, 128, 64), (1, 5000, 8, 128, 128), (514, 1700, 4, 60, 56), (514, 2048, 2, 64, 60), (3, 1537, 1, 33, 20), (512, 1100, 3, 128, 40),
    (2, 600, 8, 128, 200), (3, 200, 6, 64, 60), (1, 4000, 6, 65, 7), (520, 1030, 7, 100, 11)])
def test_walks_past_the_staged_steps(S, T, K, N, C):
    """Some experts are rare and some never come: walks end far back, at the start of the trace or in the prior state."""
    test_lru_levels(S, T, K, N, C, popularity=2.5)


@pytest.mark.parametrize("S,N,K,C,popularity", [(768, 128, 8, 64, 1.5), (100, 64, 6, 64, 0.7)])
def test_long_walks_cost_no_more_than_a_sequential_cache(S, N, K, C, popularity):
    """The LRU cache of a trace with rare experts against the FIFO cache, which is walked step by step (a lane that looked for a rare
    expert a step at a time took 5 to 20 times as long)."""
    T = 4096
    g = torch.Generator(device=DEV).manual_seed(S)
    idx = torch.empty(S, T, K, dtype=torch.int32, device=DEV)
    for s in range(0, S, 64):
        z = torch.randn(min(64, S - s), T, N, device=DEV, generator=g) + popularity * torch.randn(min(64, S - s), 1, N, device=DEV, generator=g)
        idx[s:s + 64] = z.topk(K, -1).indices.int()
    steps = [torch.empty(S, T, dtype=torch.uint8, device=DEV) for _ in range(3)]
    totals = [torch.empty(S, dtype=torch.int64, device=DEV) for _ in range(3)]

    def best(policy):
        spans = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            remoe.cache_simulate(idx, N, C, policy, 3, *steps, *totals, None)
            b.record()
            torch.cuda.synchronize()
            spans.append(a.elapsed_time(b))
        return min(spans[2:])

    lru, fifo = best(remoe.REMOE_CACHE_LRU), best(remoe.REMOE_CACHE_FIFO)
    print(f"cache S={S} N={N} K={K} C={C}: LRU {lru * 1e3:.0f} us, FIFO {fifo * 1e3:.0f} us", flush=True)
    assert lru < 1.5 * fifo


def test_more_threads_than_one_launch_counts():
    """Traces whose threads do not fit the 32 bits that a launch counts them in: one request each but the last, which is a miss at first."""
    S, T = (1 << 25) + 3, 65                                # 128 threads each
    idx = torch.zeros(S, T, 1, dtype=torch.int32, device=DEV)
    idx[-2:, 1::2] = 1                                      # the last two take turns
    steps = [torch.full((S, T), 255, dtype=torch.uint8, device=DEV) for _ in range(3)]
    totals = [torch.full((S,), -1, dtype=torch.int64, device=DEV) for _ in range(3)]
    remoe.cache_simulate(idx, 2, 1, remoe.REMOE_CACHE_LRU, 3, *steps, *totals, None)
    miss, uniq, hit_tok = steps
    assert (miss[:-2, 0] == 1).all() and not miss[:-2, 1:].any() and (miss[-2:] == 1).all()
    assert (uniq == 1).all() and torch.equal(hit_tok, 1 - miss)
    want = torch.ones(S, dtype=torch.int64, device=DEV)
    want[-2:] = T
    assert torch.equal(totals[0], want) and (totals[1] == T).all() and torch.equal(totals[2], 3 * want)
