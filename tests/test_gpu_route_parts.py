"""Layers of few tokens, whose router spreads over expert tiles and producer wavefronts: one and several tiles, ragged
ones and ragged token blocks, both sides of the token counts at which it gives way; the ids and weights
against the oracle, and bit for bit against moe_route."""
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


@pytest.mark.parametrize("H,N,K,dtype,counts", [
    (2048, 128, 8, "bf16", (1, 33, 2048, 2049, 8193, 16385)), (1152, 96, 2, "bf16", (2720, 2721)), (1408, 60, 4, "bf16", (129, 4096, 4097, 16385)),
    (2176, 20, 2, "bf16", (7, 8192, 8193)), (1056, 128, 8, "f32", (70, 4097, 8192, 8193)), (1312, 33, 2, "f32", (65, 13056, 13057, 16385)),
    (2080, 20, 1, "f32", (130, 18688, 18689))])
def test_routing_is_the_same_in_any_batch_and_from_either_entry_point(H, N, K, dtype, counts):
    """Bit for bit: a token's ids and weights from moe_forward and moe_route, on both sides of every change of the
    router's kernel and of its block width."""
    tdt, inter, T = (torch.float32 if dtype == "f32" else torch.bfloat16), 64, max(counts)
    desc = remoe.LayerDesc(H, N, inter, K, 0, 0, 0, 0 if dtype == "f32" else 1)
    x = wl.ar1_hidden_states(83, 1, T, H, 0.0, tdt, DEV)[0].contiguous()
    g = lambda name, shape, dt: wl.gaussian(83, name, shape, 0.1, 0, N, dt, DEV)
    wr = g("w_router", (N, H), torch.float32)
    w = [g("w_gate", (N, inter, H), tdt), g("w_up", (N, inter, H), tdt), g("w_down", (N, H, inter), tdt)]

    def out(t):
        return torch.full((t, K), -1, dtype=torch.int32, device=DEV), torch.full((t, K), float("nan"), device=DEV)

    ref_idx, ref_w = out(T)
    remoe.moe_route(desc, x, wr, ref_idx, ref_w, None, None)
    for t in counts:
        print(f"route T={t} H={H} N={N} K={K} {dtype}", flush=True)
        for entry in ("route", "forward"):
            idx, gw = out(t)
            if entry == "route":
                remoe.moe_route(desc, x[:t], wr, idx, gw, None, None)
            else:
                ws = torch.full((remoe.remoe_workspace_bytes(desc, t),), 0xFF, dtype=torch.uint8, device=DEV)
                remoe.moe_forward(desc, x[:t], wr, *w, None, None, None, None, torch.empty(t, H, dtype=tdt, device=DEV), idx, gw, ws)
            torch.cuda.synchronize()
            assert torch.equal(idx, ref_idx[:t]) and torch.equal(gw, ref_w[:t]), f"{entry} of {t} tokens"
