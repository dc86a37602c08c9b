"""Gate gradient with bf16 hidden states at the edges of its expert, column and token tiles, against the oracle."""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,N,H", [(1, 1, 64), (15, 31, 192), (17, 33, 128), (64, 64, 320), (129, 65, 64), (1000, 97, 128),
                                   (2049, 127, 192), (4097, 32, 2048)])
@pytest.mark.parametrize("shift", [0, 1])
def test_gate_grad_tile_edges(T, N, H, shift):
    print(f"gate grad tiles T={T} N={N} H={H} shift={shift}", flush=True)
    g = torch.Generator().manual_seed(T + 7 * N)
    dz = torch.randn(T, N, generator=g) * 10.0 ** torch.randint(-6, 1, (T, 1), generator=g)
    x = torch.randn(T, H, generator=g).bfloat16()
    xd = torch.empty(T * H + 1, dtype=torch.bfloat16, device=DEV)[shift:shift + T * H].view(T, H)     # shift 1: rows 2-byte aligned
    xd.copy_(x)
    dw = torch.full((N, H), float("nan"), device=DEV)
    remoe.remoe_gate_grad(dz.to(DEV), xd, dw, torch.empty(remoe.remoe_gate_grad_workspace_bytes(T, N, H), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    bound = dz.double().abs().T @ x.double().abs()
    err = ((dw.cpu().double() - oracle.gate_grad(dz, x)).abs() / bound).max().item()
    # exact products, fp32 sums of at most a few hundred terms each: sqrt(512) 2^-24 = 1.4e-6 of the sum of |terms|
    assert err <= 2e-6, err
