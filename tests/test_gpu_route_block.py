"""The router for 33 to 64 experts and up to one block of 64 tokens per compute unit: the bits of the general kernel (which
takes the same tokens in front of a larger batch), at the edges of its blocks, steps and rings."""
import pytest
import torch

import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,H,N,K", [(1, 64, 33, 1), (63, 128, 64, 8), (64, 192, 60, 4), (65, 320, 48, 6), (300, 384, 64, 2), (129, 448, 63, 8),
                                     (1000, 512, 40, 8), (77, 1088, 64, 6), (2048, 2048, 60, 4), (16384, 576, 64, 6)])
def test_same_bits_as_in_a_larger_batch(T, H, N, K):
    print(f"route block T={T} H={H} N={N} K={K}", flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator(device=DEV).manual_seed(T + H)
    big = torch.randn(64 * cus + 64, H, device=DEV, generator=g).bfloat16()
    w = torch.randn(N, H, device=DEV, generator=g) * 0.05
    d = remoe.LayerDesc(H, N, 64, K, 1, 0, 0, remoe.binding.REMOE_BF16)

    def route(x):
        n = x.shape[0]
        out = (torch.full((n, K), -1, dtype=torch.int32, device=DEV), torch.full((n, K), float("nan"), device=DEV),
               torch.full((n,), float("nan"), device=DEV), torch.full((n, N), float("nan"), device=DEV))
        remoe.moe_route(d, x, w, *out)
        return out

    for got, ref in zip(route(big[:T].contiguous()), route(big)):
        assert torch.equal(got, ref[:T])
