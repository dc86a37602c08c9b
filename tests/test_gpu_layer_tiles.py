"""bf16 layers at the edges of the grouped GEMMs' row and column tiles, against the CPU oracle.

Row tiles are 32, 64, 128 or 256 slots high (chosen by the rows an expert sees on average), column tiles
64, 128 or 256 wide, and the shared expert's tiles run in the routed experts' launches.
"""
import pytest
import torch

import paper_2605_27081_amd as remoe
import workload as wl
from helpers import check_output, oracle_layer, to_oracle_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,H,N,I,K,shared,gate", [
    (1, 256, 16, 192, 2, 64, 1), (2, 128, 128, 64, 8, 0, 0), (31, 384, 5, 320, 5, 192, 0), (33, 256, 4, 64, 1, 704, 1),
    (64, 128, 9, 128, 4, 0, 0), (65, 256, 2, 256, 2, 128, 0), (127, 512, 60, 64, 4, 64, 0), (257, 256, 3, 448, 2, 320, 1),
    (300, 128, 7, 704, 6, 0, 0), (700, 256, 8, 192, 8, 64, 0), (1025, 128, 6, 128, 3, 192, 0), (2300, 128, 8, 192, 6, 64, 1),
    # the shared expert's row tiles in groups of 9 and 8, several column tiles in both launches: row tiles of 32, 64 and 128
    (530, 384, 100, 64, 1, 704, 0), (1060, 256, 60, 64, 1, 320, 1), (2100, 512, 100, 64, 5, 320, 0)])
def test_layer_tile_edges(T, H, N, I, K, shared, gate):
    print(f"layer tiles T={T} H={H} N={N} I={I} K={K} shared={shared}", flush=True)
    g = lambda name, shape, dt: wl.gaussian(91, name, shape, 0.05, 0, T, dt, DEV)
    bf = torch.bfloat16
    w = {"w_router": g("w_router", (N, H), torch.float32), "w_gate": g("w_gate", (N, I, H), bf), "w_up": g("w_up", (N, I, H), bf),
         "w_down": g("w_down", (N, H, I), bf), "ws_gate": None, "ws_up": None, "ws_down": None, "ws_scale": None}
    if shared:
        w.update(ws_gate=g("ws_gate", (shared, H), bf), ws_up=g("ws_up", (shared, H), bf), ws_down=g("ws_down", (H, shared), bf))
        if gate:
            w["ws_scale"] = g("ws_scale", (H,), torch.float32)
    x = wl.ar1_hidden_states(91, 1, T, H, 0.5, bf, DEV)[0].contiguous()
    desc = remoe.LayerDesc(H, N, I, K, 1, shared, gate, 1)
    ws = torch.empty(remoe.remoe_workspace_bytes(desc, T), dtype=torch.uint8, device=DEV)
    y = torch.full((T, H), float("nan"), dtype=bf, device=DEV)
    idx = torch.full((T, K), -1, dtype=torch.int32, device=DEV)
    gw = torch.full((T, K), float("nan"), device=DEV)
    remoe.moe_forward(desc, x, w["w_router"], w["w_gate"], w["w_up"], w["w_down"], w["ws_gate"], w["ws_up"], w["ws_down"],
                      w["ws_scale"], y, idx, gw, ws)
    torch.cuda.synchronize()
    _, _, y_ref = oracle_layer(x.cpu(), to_oracle_weights(w), K, 1, idx, gw)
    check_output(y, y_ref, "bf16")
