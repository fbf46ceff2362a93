"""archead_logits_noalloc on the tiled path, through the C ABI: calls of many
tokens take no longer than archead_logits of the same call (their copy of x has
its place in the library's static memory), and a call whose copy is larger
than that, which only groups above 128 allow, runs in several chunks of tokens
with the same bits, from tables built once."""
from __future__ import annotations

import pytest

from synth import make_head
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _x(M, d):
    gen = torch.Generator(device="cuda").manual_seed(M)
    return torch.randn((M, d), generator=gen, device="cuda").bfloat16()


def _us(f, n=10):
    f()
    best = float("inf")
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for _ in range(5):
        e[0].record()
        for _ in range(n):
            f()
        e[1].record()
        e[1].synchronize()
        best = min(best, e[0].elapsed_time(e[1]) * 1e3 / n)
    return best


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("kw,M", [
    (dict(V=1000, d=4096, g=128, rc=64, rr=32), 1819),
    (dict(V=2000, d=8192, g=128, rc=16, rr=8), 5888),
    (dict(V=77, d=512, g=64, rc=16, rr=4), 8301),
])
def test_as_fast_as_with_a_workspace(kw, M, prepared):
    """(In chunks of an 8 MiB array the first two took 2 and 7 times as long.)"""
    from paper_2608_02703_amd import PackedHead
    ph = PackedHead.from_arrays(make_head("tiny", **kw))
    try:
        if prepared:
            ph.prepare()
        x = _x(M, kw["d"])
        a, b = ph.logits(x), ph.logits_noalloc(x)
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
        with_ws = _us(lambda: ph.logits(x, out=a))
        without = _us(lambda: ph.logits_noalloc(x, out=b))
        say(f"noalloc {kw} M={M} prepared={prepared}: {without:.1f} us, with a workspace {with_ws:.1f}")
        assert without <= 1.25 * with_ws
    finally:
        ph.close()


@pytest.mark.parametrize("prepared", [False, True])
def test_chunks_of_a_copy_beyond_the_static_memory(prepared):
    from paper_2608_02703_amd import PackedHead
    M, d = 300001, 1024
    ph = PackedHead.from_arrays(make_head("tiny", V=77, d=d, g=1024, rc=0, rr=0))
    try:
        if prepared:
            ph.prepare()
        assert ph.workspace_bytes(M) > 2 * (272 << 20)
        x = _x(M, d)
        say(f"noalloc in chunks, prepared={prepared}")
        a, b = ph.logits(x), ph.logits_noalloc(x)
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    finally:
        ph.close()
