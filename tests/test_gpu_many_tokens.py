"""Calls of more tokens than one dimension of a launch holds workgroups for,
through the C ABI: the tiled path's prologue gives every token a workgroup of
512 threads, so from 8.3 million tokens on its launch takes two dimensions.
Every token's result is that of a call of fewer tokens, bit for bit."""
from __future__ import annotations

import pytest

from synth import make_head
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_more_than_two_to_the_23_tokens():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_02703_amd import PackedHead
    M, step = (1 << 23) + 12345, 1 << 21
    h = make_head("tiny", V=70, d=64, g=64, rc=4, rr=0)
    ph = PackedHead.from_arrays(h)
    try:
        gen = torch.Generator(device="cuda").manual_seed(1)
        x = torch.randn((M, 64), generator=gen, device="cuda", dtype=torch.float32).bfloat16()
        y = torch.randint(0, h.V, (M,), generator=gen, device="cuda")
        say(f"CE of {M} tokens")
        ce, _ = ph.logits_ce(x, y)
        torch.cuda.synchronize()
        for m in range(0, M, step):
            part, _ = ph.logits_ce(x[m:m + step], y[m:m + step])
            torch.cuda.synchronize()
            assert torch.equal(ce[m:m + step].view(torch.int32), part.view(torch.int32)), m
        assert bool(torch.isfinite(ce).all())
    finally:
        ph.close()
