"""Router regularisers and their gradient across the blocks of steps their kernels work in, against the oracle.

A block keeps the logarithms of its rows and of the partners within its halo in LDS; partners farther away, zero and
denormal probabilities, chunks shorter than a block and sequences longer than one take other paths.
"""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("S,T,N,K,window,lags", [
    (1, 700, 128, 8, 64, [1, 16, 31, 200]), (2, 65, 64, 6, 64, [3, 40]), (1, 9, 65, 3, 2, [1, 8]), (3, 4500, 16, 2, 4500, [2, 90]),
    (70, 33, 33, 5, 7, []), (1, 2, 128, 1, 1, [1]),
    (1, 4200, 64, 2, 64, [1, 16]), (2, 300, 64, 6, 16, [4, 20]), (2, 500, 128, 8, 1, [2])])
def test_losses_across_blocks(S, T, N, K, window, lags):
    print(f"loss blocks S={S} T={T} N={N} window={window} lags={lags}", flush=True)
    g = torch.Generator().manual_seed(T * 31 + N)
    P = torch.softmax(1.5 * torch.randn(S, T, N, generator=g), -1)
    Q = torch.softmax(1.5 * torch.randn(S, T, N, generator=g), -1)
    P[:, T // 2, N // 2] = P[:, max(T // 2 - 1, 0), N // 2] = 1e-41      # denormal, next to its partner
    idx = torch.rand(S, T, N, generator=g).topk(K, -1).indices.int()
    p, q, i = P.to(DEV), Q.to(DEV), idx.to(DEV)
    vals = torch.empty(S, 6, dtype=torch.float64, device=DEV)
    dz = torch.empty(S, T, N, device=DEV)
    remoe.remoe_loss_forward(p, q, i, lags, window, vals, torch.empty(remoe.remoe_loss_workspace_bytes(S), dtype=torch.uint8, device=DEV))
    coef = [1.0, 0.4, 0.7, 0.3, 0.2]
    remoe.remoe_loss_backward(p, q, i, lags, window, coef, vals, dz,
                              torch.empty(remoe.remoe_loss_backward_workspace_bytes(S, T, N, window), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    want = oracle.remoe_losses(P, Q, idx, lags, window)
    assert torch.allclose(vals.cpu(), want, rtol=1e-12, atol=1e-14)       # fp64 on both sides, other summation trees
    grad = oracle.remoe_loss_grad(P, Q, idx, lags, window, coef)
    err = ((dz.cpu().double() - grad).abs().amax() / grad.abs().amax()).item()
    assert err <= 1.5e-7, err                                             # one rounding to fp32


def test_lag_one_given_twice_is_one_smoothness_term():
    test_losses_across_blocks(2, 90, 60, 4, 8, [1, 5, 1])


def _grad(P, Q, idx, lags, window, coef, vals):
    S, T, N = P.shape
    dz = torch.zeros(S, T, N, device=DEV)
    remoe.remoe_loss_backward(P.to(DEV), Q.to(DEV), idx.to(DEV), lags, window, coef, vals, dz,
                              torch.empty(remoe.remoe_loss_backward_workspace_bytes(S, T, N, window), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    return dz.cpu()


@pytest.mark.parametrize("N", [60, 128])
def test_numbers_that_are_not_finite_stay_visible(N):
    """A NaN probability makes every step that it is a partner of NaN and no other; a diverged sequence has no
    finite gradient; ln keeps infinities and NaNs of either distribution."""
    print(f"loss not finite N={N}", flush=True)
    S, T, K, window, lags, coef = 2, 90, 4, 8, [1, 5, 70], [1.0, 0.4, 0.7, 0.3, 0.2]
    g = torch.Generator().manual_seed(N)
    P, Q = (torch.softmax(torch.randn(S, T, N, generator=g), -1) for _ in range(2))
    P[:, :, 3] = 0.0                                  # 0 gets 0, but not in a row without a finite gradient
    idx = torch.rand(S, T, N, generator=g).topk(K, -1).indices.int()
    vals = torch.empty(S, 6, dtype=torch.float64, device=DEV)
    ws = torch.empty(remoe.remoe_loss_workspace_bytes(S), dtype=torch.uint8, device=DEV)
    Q[:, :, 3] = 0.0
    remoe.remoe_loss_forward(P.to(DEV), Q.to(DEV), idx.to(DEV), lags, window, vals, ws)
    clean = _grad(P, Q, idx, lags, window, coef, vals)
    assert torch.isfinite(clean).all() and (clean[:, :, 3] == 0).all()

    t, e = 15, N - 2
    bad = P.clone()
    bad[0, t, e] = float("nan")
    hit = {t} | {t + s * d for d in lags for s in (-1, 1)} | set(range(t - t % window, t - t % window + window))
    hit = torch.tensor([u in hit for u in range(T)])
    dz = _grad(bad, Q, idx, lags, window, coef, vals)
    assert torch.isnan(dz[0, hit]).all()
    assert torch.equal(dz[0, ~hit], clean[0, ~hit]) and torch.equal(dz[1], clean[1])
    bad[1] = float("nan")
    assert torch.isnan(_grad(bad, Q, idx, lags, window, coef, vals)[1]).all()

    for value, want in ((float("inf"), float("-inf")), (float("nan"), float("nan"))):
        ref = Q.clone()
        ref[0, t, e] = value
        out = torch.empty_like(vals)
        remoe.remoe_loss_forward(P.to(DEV), ref.to(DEV), idx.to(DEV), lags, window, out, ws)
        torch.cuda.synchronize()
        trust = out[0, 2].item()
        assert trust == want or (want != want and trust != trust)
        assert torch.equal(out[1], vals[1])
        dz = _grad(P, ref, idx, lags, window, coef, vals)
        assert not torch.isfinite(dz[0, t]).any() and torch.isfinite(dz[0, t + 1]).all()
