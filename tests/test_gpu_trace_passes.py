"""Trace statistics across the passes, halos and load widths of their kernels, bit for bit against the oracle.

LRU walks run in passes of 512 steps with 256 earlier steps staged; one workgroup takes a whole trace from 512
traces on.  Rows of a multiple of four ids are read 16 bytes at a time where the table is aligned.
"""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("S,T,K,N,C,sticky", [(3, 1537, 4, 128, 64, 60), (2, 1025, 3, 33, 30, 40), (513, 1030, 4, 64, 12, 3),
                                               (512, 511, 2, 16, 1, 1), (1, 3000, 8, 128, 127, 300), (600, 65, 5, 100, 7, 1)])
def test_trace_statistics_across_passes(S, T, K, N, C, sticky):
    print(f"trace passes S={S} T={T} K={K} N={N} C={C}", flush=True)
    g = torch.Generator().manual_seed(S * 10007 + T)
    # ids drift: every `sticky` steps a window of N / 2 experts moves, so long walks are needed when it is large
    base = torch.arange(T) // sticky * 3
    pick = torch.rand(S, T, max(K, N // 2), generator=g).topk(K, dim=-1).indices
    idx = ((pick + base[None, :, None]) % N).int()
    store = torch.empty(S * T * K + 1, dtype=torch.int32, device=DEV)
    for shift in (0, 1):                               # 16-byte aligned, and 4-byte aligned only
        tr = store[shift:shift + S * T * K].view(S, T, K)
        tr.copy_(idx)
        ov = torch.empty(S, T, dtype=torch.uint8, device=DEV)
        miss = torch.empty_like(ov)
        osum, tot, byt = (torch.empty(S, dtype=torch.int64, device=DEV) for _ in range(3))
        load, used = torch.empty(S, N, dtype=torch.int32, device=DEV), torch.empty(S, dtype=torch.int32, device=DEV)
        ent, cv = (torch.empty(S, dtype=torch.float64, device=DEV) for _ in range(2))
        remoe.trace_reuse(tr, N, ov, osum)
        remoe.lru_simulate(tr, N, C, 10, 0, None, miss, tot, byt)
        remoe.routing_balance(tr, N, load, used, ent, cv)
        n_all = torch.empty(1, S * T, dtype=torch.int16, device=DEV)
        hist, pct = torch.empty(K + 1, dtype=torch.int64, device=DEV), torch.empty(3, dtype=torch.int32, device=DEV)
        remoe.step_miss_summary(miss.view(1, 1, S * T), n_all, hist, pct)
        torch.cuda.synchronize()
        rov, rsum = oracle.trace_reuse(idx, N)
        rmiss, rtot, rbyt = oracle.lru_list(idx, N, C, 10)
        assert torch.equal(ov.cpu(), rov) and torch.equal(osum.cpu(), rsum)
        assert torch.equal(miss.cpu(), rmiss) and torch.equal(tot.cpu(), rtot) and torch.equal(byt.cpu(), rbyt)
        assert torch.equal(load.cpu(), torch.stack([torch.bincount(r.reshape(-1), minlength=N) for r in idx]).int())
        assert torch.equal(n_all.cpu().view(S, T).int(), rmiss.int())
        rh = torch.bincount(rmiss.reshape(-1).int(), minlength=K + 1)
        assert torch.equal(hist.cpu(), rh)
        cum = rh.cumsum(0)
        assert pct.cpu().tolist() == [int((100 * cum >= p * S * T).nonzero()[0]) for p in (50, 95, 99)]
