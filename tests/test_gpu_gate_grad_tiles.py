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


@pytest.mark.parametrize("N", [20, 100])
def test_gate_grad_beyond_the_range_of_bf16(N):
    """dz that is infinite, or finite but rounds to infinity in bf16, gives what an fp32 product gives."""
    print(f"gate grad range N={N}", flush=True)
    T, H, big = 40, 128, torch.finfo(torch.float32).max
    dz = torch.zeros(T, N)
    dz[:, 0] = 0.25                                                   # an expert untouched by the rest
    dz[3, 1], dz[5, 2], dz[7, 3], dz[9, 4] = big, -big, float("inf"), float("-inf")
    dz[9, 5], dz[11, 5] = float("nan"), 1.0
    dz[13, 6], dz[14, 6] = float("inf"), 1.0
    x = (0.5 + torch.arange(T * H).view(T, H) % 7 / 16).bfloat16()    # 0.5 .. 0.875: big * x is finite and exact enough to compare
    dw = torch.zeros(N, H, device=DEV)
    remoe.remoe_gate_grad(dz.to(DEV), x.to(DEV), dw, torch.empty(remoe.remoe_gate_grad_workspace_bytes(T, N, H), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    got, want = dw.cpu().double(), (dz.double().T @ x.double())       # fp64: no product overflows
    assert torch.isnan(got[5]).all() and torch.isposinf(got[3]).all() and torch.isneginf(got[4]).all() and torch.isposinf(got[6]).all()
    rows = [n for n in range(N) if n not in (3, 4, 5, 6)]
    assert torch.allclose(got[rows], want[rows], rtol=2.0 ** -20, atol=0)      # fp32 sums of up to 40 terms of one sign
