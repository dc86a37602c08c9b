"""fp32 layers of sizes that are no multiple of anything, at the edges of the GEMM tiles, against the CPU oracle."""
import pytest
import torch

import paper_2605_27081_amd as remoe
import workload as wl
from helpers import check_output, oracle_layer, to_oracle_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,H,N,I,K,shared", [
    (1, 32, 4, 1, 2, 0), (3, 64, 33, 33, 5, 65), (31, 96, 2, 31, 2, 0), (65, 160, 3, 64, 1, 200), (130, 32, 1, 100, 1, 32),
    (300, 288, 7, 127, 4, 0), (513, 128, 4, 257, 3, 96), (2050, 64, 2, 320, 2, 31), (4100, 96, 12, 130, 2, 0)])
def test_f32_layer_tile_edges(T, H, N, I, K, shared):
    print(f"f32 layer T={T} H={H} N={N} I={I} K={K} shared={shared}", flush=True)
    g = lambda name, shape: wl.gaussian(17, name, shape, 0.05, 0, T, torch.float32, DEV)
    w = {"w_router": g("w_router", (N, H)), "w_gate": g("w_gate", (N, I, H)), "w_up": g("w_up", (N, I, H)), "w_down": g("w_down", (N, H, I)),
         "ws_gate": None, "ws_up": None, "ws_down": None, "ws_scale": None}
    if shared:
        w.update(ws_gate=g("ws_gate", (shared, H)), ws_up=g("ws_up", (shared, H)), ws_down=g("ws_down", (H, shared)))
    x = wl.ar1_hidden_states(17, 1, T, H, 0.5, torch.float32, DEV)[0].contiguous()
    desc = remoe.LayerDesc(H, N, I, K, 0, shared, 0, 0)
    ws = torch.full((remoe.remoe_workspace_bytes(desc, T),), 0xFF, dtype=torch.uint8, device=DEV)     # NaNs wherever nothing is written
    y = torch.full((T, H), float("nan"), device=DEV)
    idx = torch.full((T, K), -1, dtype=torch.int32, device=DEV)
    gw = torch.full((T, K), float("nan"), device=DEV)
    remoe.moe_forward(desc, x, w["w_router"], w["w_gate"], w["w_up"], w["w_down"], w["ws_gate"], w["ws_up"], w["ws_down"], None, y, idx, gw, ws)
    torch.cuda.synchronize()
    _, _, y_ref = oracle_layer(x.cpu(), to_oracle_weights(w), K, 0, idx, gw)
    check_output(y, y_ref, "f32")
