"""Layers whose router takes its reduction in shares: shares of unequal length, one and several expert tiles, ragged token
blocks, the token counts at which the number of shares changes; the ids and weights against the oracle."""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe
import workload as wl
from helpers import compare_routing

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,H,N,K,dtype", [
    (1, 1024, 128, 8, "bf16"), (33, 1152, 100, 8, "bf16"), (31, 1408, 64, 6, "bf16"), (129, 1152, 20, 4, "bf16"), (65, 2176, 33, 3, "bf16"),
    (17, 4096, 128, 8, "bf16"), (2049, 1024, 128, 2, "bf16"), (4096, 1024, 128, 2, "bf16"), (4097, 1024, 128, 2, "bf16"), (8193, 1024, 64, 1, "bf16"),
    (1, 1056, 128, 8, "f32"), (33, 1312, 65, 5, "f32"), (70, 1056, 60, 4, "f32"), (130, 2080, 20, 2, "f32"), (40, 992, 20, 2, "f32")])
def test_layer_router_in_shares(T, H, N, K, dtype):
    print(f"route parts T={T} H={H} N={N} K={K} {dtype}", flush=True)
    tdt, inter = (torch.float32 if dtype == "f32" else torch.bfloat16), 64
    desc = remoe.LayerDesc(H, N, inter, K, 1, 0, 0, 0 if dtype == "f32" else 1)
    x = wl.ar1_hidden_states(79, 1, T, H, 0.0, tdt, DEV)[0].contiguous()
    g = lambda name, shape, dt: wl.gaussian(79, name, shape, 0.1, 0, N, dt, DEV)
    wr = g("w_router", (N, H), torch.float32)
    y = torch.empty(T, H, dtype=tdt, device=DEV)
    idx = torch.full((T, K), -1, dtype=torch.int32, device=DEV)
    w = torch.full((T, K), float("nan"), device=DEV)
    ws = torch.full((remoe.remoe_workspace_bytes(desc, T),), 0xFF, dtype=torch.uint8, device=DEV)     # NaNs wherever nothing is written
    remoe.moe_forward(desc, x, wr, g("w_gate", (N, inter, H), tdt), g("w_up", (N, inter, H), tdt), g("w_down", (N, H, inter), tdt),
                      None, None, None, None, y, idx, w, ws)
    torch.cuda.synchronize()
    compare_routing(idx, w, oracle.route(x.cpu(), wr.cpu(), K, True, want_probs=True), True)
