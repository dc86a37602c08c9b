"""A buffer sized for the largest batch serves every smaller one: moe_forward's workspace never shrinks when
tokens are added.  Host calls only."""
import pytest

import paper_2605_27081_amd as remoe
from paper_2605_27081_amd import build as hip_build


@pytest.mark.parametrize("hidden,experts,inter,top_k,shared,dtype", [
    (2048, 128, 768, 8, 0, 1), (2048, 64, 1408, 6, 2816, 1), (2048, 60, 1408, 4, 5632, 1), (4096, 128, 64, 8, 0, 1),
    (1024, 128, 64, 1, 0, 1), (1024, 33, 64, 1, 0, 1), (1024, 20, 64, 1, 64, 1), (1280, 100, 64, 1, 0, 1), (128, 128, 64, 1, 0, 1),
    (128, 8, 64, 1, 0, 1), (256, 16, 128, 2, 0, 0), (1056, 128, 1, 1, 0, 0), (32, 1, 1, 1, 0, 0), (1056, 40, 33, 1, 96, 0)])
def test_workspace_never_shrinks_with_more_tokens(hidden, experts, inter, top_k, shared, dtype):
    if not hip_build.is_built():
        hip_build.build()
    d = remoe.LayerDesc(hidden, experts, inter, top_k, 0, shared, 0, dtype)
    # every size past the last one at which a row tile or the router's scratch changes, and strides to the limit
    counts = list(range(0, 40000)) + list(range(40000, 1 << 22, 9973)) + [1 << 22]
    last = (0, 0)
    for t in counts:
        n = remoe.remoe_workspace_bytes(d, t)
        assert n >= last[1], f"{t} tokens need {n} bytes, {last[0]} tokens {last[1]}"
        last = (t, n)
