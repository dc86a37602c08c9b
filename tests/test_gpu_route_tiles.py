"""Router at the edges of its token blocks and expert tiles, against the CPU oracle.

A workgroup owns 32, 64, 128 or 256 tokens depending on the number of experts and tokens, and an expert
tile is 32 wide; the reduction runs in slices of 32.
"""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe
import workload as wl
from helpers import compare_routing

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,H,N,K", [
    (1, 32, 128, 8), (31, 64, 33, 3), (33, 96, 64, 8), (65, 160, 65, 7), (127, 32, 31, 2), (129, 64, 32, 8), (257, 96, 97, 5),
    (8193, 64, 128, 8), (16385, 64, 127, 6), (16383, 64, 64, 6), (32769, 32, 60, 4), (32769, 32, 20, 2)])
def test_route_block_edges(T, H, N, K, dtype):
    print(f"route edges T={T} H={H} N={N} K={K} {dtype}", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    x = wl.ar1_hidden_states(77, 1, T, H, 0.0, tdt, DEV)[0].contiguous()
    wr = wl.gaussian(77, "w_router", (N, H), 0.1, 0, N, torch.float32, DEV)
    desc = remoe.LayerDesc(H, N, 64, K, 1, 0, 0, 0 if dtype == "f32" else 1)
    idx = torch.full((T, K), -1, dtype=torch.int32, device=DEV)
    w = torch.full((T, K), float("nan"), device=DEV)
    margin = torch.empty(T, device=DEV)
    probs = torch.empty(T * N + 1, device=DEV)[1:].view(T, N)      # 4-byte aligned only
    remoe.moe_route(desc, x, wr, idx, w, margin, probs)
    torch.cuda.synchronize()
    orc = oracle.route(x.cpu(), wr.cpu(), K, True, want_probs=True)
    compare_routing(idx, w, orc, True)
    # fp32 softmax of logits of a few units: a few 1e-7 from the exponential and the sums (as in the other router tests)
    assert torch.allclose(probs.cpu().double(), orc["probs"], rtol=2e-5, atol=1e-7)
    assert torch.allclose(margin.cpu().double(), orc["margin"], rtol=1e-4, atol=2e-5)


@pytest.mark.parametrize("N,dtype", [(20, "f32"), (33, "bf16"), (64, "f32"), (100, "bf16"), (128, "bf16")])
def test_logits_of_minus_infinity_are_ranked_by_id(N, dtype):
    """Fewer finite logits than places: the experts whose logit is -inf follow in the order of their ids, none twice."""
    print(f"route -inf N={N} {dtype}", flush=True)
    T, H, K, finite = 5, 128, 8, (N - 3, 4)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    x = torch.full((T, H), 2.0 ** 70, dtype=tdt, device=DEV)
    wr = torch.full((N, H), -2.0 ** 70, device=DEV)                   # products of -2^140
    wr[finite[0]], wr[finite[1]] = 2.0 ** -77, 0.0                    # logits 1 and 0
    desc = remoe.LayerDesc(H, N, 64, K, 0, 0, 0, 0 if dtype == "f32" else 1)
    idx = torch.full((T, K), -1, dtype=torch.int32, device=DEV)
    w, margin, probs = (torch.full(s, 7.0, device=DEV) for s in ((T, K), (T,), (T, N)))
    remoe.moe_route(desc, x, wr, idx, w, margin, probs)
    torch.cuda.synchronize()
    want = list(finite) + [e for e in range(N) if e not in finite][:K - 2]
    assert idx.cpu().tolist() == [want] * T
    p1 = torch.sigmoid(torch.tensor(1.0))
    assert torch.allclose(w.cpu()[:, 0], p1, rtol=1e-6) and torch.allclose(w.cpu()[:, 1], 1 - p1, rtol=1e-6) and (w.cpu()[:, 2:] == 0).all()
    assert ((probs.cpu() > 0).sum(1) == 2).all()
