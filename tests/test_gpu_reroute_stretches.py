"""Rerouting at the edges of its lists and stretches: trace lengths around the batch and stretch sizes, every
list length, caches whose guessed state does not settle, and rows without a list (ties, negative
scores, bonuses that overflow or underflow)."""
import pytest
import torch

import oracle
import paper_2605_27081_amd as remoe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _scores(kind, S, T, N):
    g = torch.Generator().manual_seed(S * 1000003 + T * 131 + N)
    z = torch.randn(S, T, N, generator=g)
    if kind in ("sticky", "mixed"):            # neighbouring steps alike: with a large cache guesses stay wrong for long
        for t in range(1, T):
            z[:, t] = 0.95 * z[:, t - 1] + 0.3122 * z[:, t]
    p = torch.softmax(2.0 * z, -1)
    if kind == "ties":
        p = (p * 64).round() / 64              # few distinct values, many zeros
    if kind == "signed":
        p[:, ::3] = z[:, ::3]                  # negative scores: a bonus lowers them
    if kind == "mixed":
        p[:, 5::37] = z[:, 5::37]
    if kind == "tiny":
        p = p * 1e-38                          # the plain scores are denormal or close to it
    return p.float().contiguous()


@pytest.mark.parametrize("S,T,N,K,C,factor,renorm,kind", [
    (2, 1, 128, 8, 4, 1.5, False, "plain"), (2, 15, 128, 8, 8, 1.5, True, "plain"), (2, 33, 65, 8, 9, 1.5, False, "plain"),
    (1, 511, 64, 6, 6, 4.0, False, "plain"), (1, 513, 63, 3, 130, 1.5, True, "plain"), (2, 769, 128, 1, 2, 4.0, False, "plain"),
    (1, 2, 1, 1, 1, 2.0, True, "plain"), (1, 40, 2, 2, 1, 2.0, False, "plain"),
    (2, 1500, 128, 2, 64, 4.0, False, "sticky"), (1, 1040, 100, 8, 64, 4.0, True, "sticky"), (1, 700, 128, 4, 100, 4.0, False, "sticky"),
    (2, 300, 128, 8, 16, 0.5, False, "plain"), (1, 300, 96, 40, 50, 1.5, True, "plain"), (1, 100, 128, 64, 70, 1.0, False, "plain"),
    (2, 600, 128, 6, 12, 1.5, False, "ties"), (2, 600, 60, 4, 3, 1.1, True, "ties"),
    (2, 600, 128, 6, 12, 1.5, False, "signed"), (1, 90, 128, 8, 12, 2.9e38, False, "plain"), (2, 600, 128, 8, 12, 0.75, False, "tiny"),
])
def test_reroute_edges_match_oracle(S, T, N, K, C, factor, renorm, kind):
    print(f"reroute edges S={S} T={T} N={N} K={K} C={C} factor={factor} {kind}", flush=True)
    p = _scores(kind, S, T, N)
    idx = torch.full((S, T, K), -1, dtype=torch.int32, device=DEV)
    w = torch.full((S, T, K), 7.0, dtype=torch.float32, device=DEV)
    miss = torch.full((S, T), 255, dtype=torch.uint8, device=DEV)
    tot = torch.full((S,), -1, dtype=torch.int64, device=DEV)
    remoe.reroute_lru(p.to(DEV), K, C, factor, renorm, idx, w, miss, tot)
    torch.cuda.synchronize()
    ref = oracle.reroute_lru(p, K, C, factor, renorm)
    assert torch.equal(idx.cpu(), ref["idx"]) and torch.equal(miss.cpu(), ref["miss"]) and torch.equal(tot.cpu(), ref["total_miss"])
    if kind != "tiny":                         # a sum of K fp32 values and a division: K + 1 roundings of 2^-24
        assert torch.allclose(w.cpu().double(), ref["w"], rtol=(K + 1) * 2.0 ** -24, atol=1e-12 if kind != "signed" else 1e-5)


def _reroute(p, K, C, factor):
    S, T, _ = p.shape
    idx = torch.full((S, T, K), -1, dtype=torch.int32, device=DEV)
    w = torch.full((S, T, K), 7.0, dtype=torch.float32, device=DEV)
    miss = torch.full((S, T), 255, dtype=torch.uint8, device=DEV)
    tot = torch.full((S,), -1, dtype=torch.int64, device=DEV)
    remoe.reroute_lru(p.to(DEV), K, C, factor, False, idx, w, miss, tot)
    torch.cuda.synchronize()
    return idx.cpu(), miss.cpu(), tot.cpu()


@pytest.mark.parametrize("N,K,C", [(128, 8, 100), (128, 9, 18), (90, 2, 90)])
def test_bonuses_that_overflow_are_ranked_by_id(N, K, C):
    """Scores large enough that more boosted ones than a list holds are infinite: ties go to the lower id."""
    print(f"reroute overflow N={N} K={K} C={C}", flush=True)
    T, e = 60, torch.arange(N)
    p = torch.zeros(1, T, N)
    p[0, 0::3] = (e < K) * (2.0 + e)                                  # K low ids come in,
    p[0, 1::3] = ((e >= N - 64) & (e < N - 64 + K)) * (2.0 + e)       # then K of the last 64, then those lead in the order of
    p[0, 2::3] = 200.0 - e.roll(N - 64)                              # their ids and all residents' bonuses overflow
    idx, miss, tot = _reroute(p, K, C, 2.9e38)
    ref = oracle.reroute_lru(p, K, C, 2.9e38, False)
    assert torch.equal(idx, ref["idx"]) and torch.equal(miss, ref["miss"]) and torch.equal(tot, ref["total_miss"])


@pytest.mark.parametrize("N,T", [(64, 40), (64, 900), (128, 40), (60, 40), (100, 300)])
def test_steps_of_nans_leave_the_others_alone(N, T):
    """A step whose probabilities are all NaN names one expert, 63 or the last, in every place and touches it; what follows is rerouted
    from that cache, which keeps its capacity."""
    print(f"reroute NaN N={N} T={T}", flush=True)
    K, C, factor = 4, 6, 3.0
    p = _scores("plain", 1, T, N)
    p[0, 5::11] = float("nan")
    idx, miss, tot = _reroute(p, K, C, factor)
    cache, misses = [], []                                             # least recent first
    for t in range(T):
        if torch.isnan(p[0, t]).any():
            want = [min(63, N - 1)] * K
        else:
            score = p[0, t].clone()
            score[cache] *= factor
            want = sorted(range(N), key=lambda e: (-float(score[e]), e))[:K]
        assert idx[0, t].tolist() == want, t
        misses.append(len(set(want) - set(cache)))
        cache = ([e for e in cache if e not in want] + sorted(set(want)))[-C:]
    assert miss[0].tolist() == misses and int(tot) == sum(misses)


@pytest.mark.parametrize("N,K,C", [(16, 16, 1), (63, 63, 63), (64, 64, 40), (100, 64, 90)])
def test_scores_of_minus_infinity_are_chosen_once(N, K, C):
    """Bonuses take negative scores to -inf and (nearly) all experts are asked for: none is named twice."""
    test_reroute_edges_match_oracle(2, 200, N, K, C, 2.9e38, False, "signed")


def _stretches(T, N, K, C, factor):
    """Steps of a stretch and of its warm-up where a trace is cut into up to 56 stretches; None where one workgroup walks it."""
    warm = 16 * -(-(16 + 12 * min(C, N) // K) // 16)
    if T <= 512 or T <= 16 * warm * (4 if factor > 2 and 2 * C > N else 1) or C >= N:
        return None
    stretch = 16 * -(-max(-(-T // 56), 32, warm) // 16)
    return stretch, warm


def _wrong_guesses(p, K, C, factor, ref):
    """Stretches of trace 0 in which a walk from a cold cache, warmed on the steps before, chooses otherwise than the trace."""
    T, N = p.shape[1:]
    stretch, warm = _stretches(T, N, K, C, factor)
    wrong = []
    for t0 in range(stretch, T, stretch):
        a, t1 = max(0, t0 - warm), min(T, t0 + stretch)
        guess = oracle.reroute_lru(p[:1, a:t1].contiguous(), K, C, factor, False)
        if not (torch.equal(guess["idx"][0, t0 - a:], ref["idx"][0, t0:t1]) and torch.equal(guess["miss"][0, t0 - a:], ref["miss"][0, t0:t1])):
            wrong.append(t0 // stretch)
    return wrong


@pytest.mark.parametrize("S,T,N,K,C,factor,kind,mended", [
    # trace lengths around 56 stretches of 32 and of 48 steps, and longer ones
    (2, 1791, 128, 8, 4, 1.5, "plain", 0), (2, 1792, 128, 8, 4, 1.5, "plain", 0), (2, 1793, 128, 8, 4, 1.5, "plain", 0),
    (2, 2047, 128, 8, 4, 1.5, "plain", 0), (2, 2049, 64, 6, 4, 1.5, "sticky", 0),
    (2, 2688, 128, 8, 4, 1.5, "plain", 0), (2, 2689, 64, 6, 4, 1.5, "sticky", 0), (1, 4100, 128, 8, 8, 4.0, "sticky", 0),
    # guesses that do not settle in one workgroup's 16 stretches
    (2, 2100, 128, 2, 24, 4.0, "sticky", None), (1, 3000, 128, 8, 120, 100.0, "sticky", None), (1, 2500, 60, 4, 59, 4.0, "sticky", None),
    # stretches that are mended: few and most of them, more than 16 in a row, with the last one short, caches as large as or larger than N
    (1, 4096, 64, 6, 40, 1.5, "sticky", 4), (2, 4000, 64, 2, 8, 4.0, "sticky", 4), (1, 5000, 32, 8, 24, 4.0, "sticky", 17),
    (2, 2048, 16, 8, 64, 4.0, "sticky", None), (1, 4096, 128, 8, 64, 4.0, "sticky", 17), (1, 4100, 128, 8, 100, 2.0, "sticky", 17),
    (1, 3001, 48, 16, 47, 2.0, "sticky", 17), (20, 1100, 64, 4, 12, 4.0, "sticky", 2),
    # steps without a list among them: up to 8 ids in place of the marks, 9 and 10 (the shortest row behind the marks), 11 and 16
    (2, 2000, 128, 7, 20, 3.0, "mixed", 2), (2, 2000, 128, 9, 20, 3.0, "mixed", 4), (1, 2000, 128, 10, 30, 3.0, "mixed", 4),
    (1, 2000, 100, 11, 30, 4.0, "mixed", 4), (1, 2000, 64, 16, 32, 3.0, "mixed", 4), (1, 2000, 64, 2, 8, 4.0, "mixed", 2),
    (2, 2000, 128, 9, 20, 1.5, "signed", 0), (2, 2000, 128, 10, 30, 1.5, "ties", 0), (1, 2000, 100, 11, 11, 1.5, "signed", 0),
    (1, 700, 64, 1, 1, 1.5, "signed", 0),
    (1, 400, 128, 7, 20, 1.5, "signed", None), (2, 400, 128, 9, 20, 1.5, "signed", None), (2, 400, 128, 10, 30, 1.5, "ties", None),
    (1, 400, 100, 11, 11, 1.5, "signed", None), (1, 200, 128, 64, 100, 1.5, "signed", None), (1, 200, 64, 1, 1, 1.5, "signed", None),
])
def test_reroute_checked_stretches_match_oracle(S, T, N, K, C, factor, kind, mended):
    """mended: how many stretches' guesses are wrong at least; None: the trace is one workgroup's."""
    print(f"reroute checked stretches S={S} T={T} N={N} K={K} C={C} factor={factor} {kind}", flush=True)
    p = _scores(kind, S, T, N)
    ref = oracle.reroute_lru(p, K, C, factor, False)
    assert (_stretches(T, N, K, C, factor) is None) == (mended is None)
    if mended:
        assert len(_wrong_guesses(p, K, C, factor, ref)) >= mended
    idx, miss, tot = _reroute(p, K, C, factor)
    assert torch.equal(idx, ref["idx"]) and torch.equal(miss, ref["miss"]) and torch.equal(tot, ref["total_miss"])


@pytest.mark.parametrize("N,K,C,times", [(16, 8, 64, 9), (32, 8, 32, 9), (128, 8, 32, 9)])
def test_wrong_guesses_are_mended_at_once(N, K, C, times):
    """Guesses that do not settle cost some walks in parallel, not one of the whole trace: 16 traces of 4096 steps with a bonus of
    4, against the same probabilities with a cache of top-k and no bonus (one wavefront mending a trace took 10 to 20 times as long)."""
    p = _scores("sticky", 16, 4096, N).to(DEV)
    out = (torch.empty(16, 4096, K, dtype=torch.int32, device=DEV), torch.empty(16, 4096, K, device=DEV),
           torch.empty(16, 4096, dtype=torch.uint8, device=DEV), torch.empty(16, dtype=torch.int64, device=DEV))

    def best(capacity, factor):
        spans = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            remoe.reroute_lru(p, K, capacity, factor, False, *out)
            b.record()
            torch.cuda.synchronize()
            spans.append(a.elapsed_time(b))
        return min(spans[2:])

    plain, hard = best(K, 1.0), best(C, 4.0)
    print(f"reroute N={N} K={K} C={C}: {plain * 1e3:.0f} us with guesses that settle, {hard * 1e3:.0f} us with some that do not", flush=True)
    assert hard < times * plain
