"""Token -> expert sort at the edges of its single-workgroup form: word and row ends of the token bit matrix, one and two
tokens per thread, the last size it takes and the first it does not, tiles that end exactly."""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,N,K", [(1, 1, 1), (32, 1, 1), (33, 3, 3), (64, 128, 8), (767, 128, 8), (768, 127, 8), (769, 128, 8), (1023, 16, 6),
                                   (1024, 20, 6), (1025, 60, 4), (1536, 33, 4), (1537, 33, 4), (2047, 64, 2), (2048, 5, 3), (2049, 64, 1)])
def test_layer_around_the_single_workgroup_sort(T, N, K):
    print(f"permute small T={T} N={N} K={K}", flush=True)
    H, inter = 64, 33
    desc = remoe.LayerDesc(H, N, inter, K, 0, 0, 0, 0)
    x = wl.ar1_hidden_states(91, 1, T, H, 0.5, torch.float32, DEV)[0].contiguous()
    w = {n: wl.gaussian(91, n, s, 0.1, 0, T, torch.float32, DEV) for n, s in
         (("w_router", (N, H)), ("w_gate", (N, inter, H)), ("w_up", (N, inter, H)), ("w_down", (N, H, inter)))}
    y = torch.full((T, H), float("nan"), device=DEV)
    idx = torch.full((T, K), -1, dtype=torch.int32, device=DEV)
    gw = torch.full((T, K), float("nan"), device=DEV)
    ws = torch.full((remoe.remoe_workspace_bytes(desc, T),), 0xFF, dtype=torch.uint8, device=DEV)
    remoe.moe_forward(desc, x, w["w_router"], w["w_gate"], w["w_up"], w["w_down"], None, None, None, None, y, idx, gw, ws)
    torch.cuda.synchronize()
    cpu = {k: v.cpu() for k, v in w.items()}
    ref = oracle.experts_sparse(x.cpu(), idx.cpu(), gw.cpu().double(), cpu)
    # sums of at most 64 fp32 products per value, as in the other fp32 layer tests
    assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) <= 1e-5
