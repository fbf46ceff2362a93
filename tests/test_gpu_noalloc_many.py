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


def _counted(ph, M, V, d, g, rc, rr):
    """The bytes the header says a call of the tiled path is counted with."""
    up = lambda n: (n + 255) // 256 * 256
    n_x = (rc + 15) // 16 + (rr + 15) // 16
    n = up(128 * M * n_x) + up(1024 * ((M + 255) // 256) * (d // g + (rc > 0) + (rr > 0)))
    n += ph.prepared_bytes() + up(2 * (rc + rr) * d)
    s, blocks = 1, ((M + 15) // 16) * ((rc + rr + 63) // 64)
    while rc + rr and blocks * s < 256 and (d // g) % (2 * s) == 0 and d // g // (2 * s) >= 8:
        s *= 2
    return n + (up(4 * s * M * (rc + rr)) if s > 1 else 0)


@pytest.mark.parametrize("kw", [
    dict(V=77, d=512, g=64, rc=16, rr=4),
    dict(V=500, d=1024, g=128, rc=0, rr=0),
    dict(V=3000, d=2048, g=64, rc=64, rr=32),    # (stage 1 split along d)
    dict(V=12000, d=512, g=64, rc=64, rr=32),    # tables close to the limit
])
def test_limit_is_the_documented_one(kw):
    from paper_2608_02703_amd import PackedHead, archead as ab
    ph = PackedHead.from_arrays(make_head("tiny", **kw))
    ph.force_path("tiled")
    try:
        count = lambda M: _counted(ph, M, **kw)
        lo, hi = 0, 1 << 20
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if count(mid) <= ab.NOALLOC_SCRATCH_BYTES else (lo, mid)
        for M in sorted({1, lo - 1, lo, lo + 1, lo + 257} & set(range(1, 1 << 20))):
            say(f"noalloc limit {kw} M={M}")
            x = torch.zeros((M, kw["d"]), dtype=torch.bfloat16, device="cuda")
            out = torch.empty((M, kw["V"]), device="cuda", dtype=torch.bfloat16)
            if count(M) <= ab.NOALLOC_SCRATCH_BYTES:
                ph.logits_noalloc(x, out=out)
            else:
                with pytest.raises(ab.ArcheadError) as e:
                    ph.logits_noalloc(x, out=out)
                assert e.value.status == ab.E_WORKSPACE
        torch.cuda.synchronize()
    finally:
        ph.close()
