"""archead_set_timing_events on calls that run in chunks of tokens, through the
C ABI: the start event belongs to the first chunk's head kernel and the stop
event to the last one's, so their time is most of the call's (that of the last
chunk alone was a fourteenth in the first case)."""
from __future__ import annotations

import pytest

from synth import make_head
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("op,kw,M", [
    ("topk", dict(V=8192, d=512), 1024),                        # 256 tokens a chunk
    ("noalloc", dict(V=77, d=1024, g=1024, rc=0, rr=0), 500000),   # a copy of x of 1 GB in 272 MiB
])
def test_events_span_the_chunks(op, kw, M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_02703_amd import PackedHead
    ph = PackedHead.from_arrays(make_head("tiny", **kw))
    try:
        x = torch.zeros((M, kw["d"]), dtype=torch.bfloat16, device="cuda")
        x[:, 0] = 1.0
        out = torch.empty((M, kw["V"]), device="cuda") if op == "noalloc" else None
        run = (lambda: ph.logits_topk(x, 5)) if op == "topk" else (lambda: ph.logits_noalloc(x, out=out))
        e = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        for v in e:
            v.record()
        run()
        torch.cuda.synchronize()
        ph.set_timing_events(e[0], e[1])
        say(f"timing events {op}")
        e[2].record()
        run()
        e[3].record()
        torch.cuda.synchronize()
        ph.set_timing_events(None, None)
        part, whole = e[0].elapsed_time(e[1]), e[2].elapsed_time(e[3])
        say(f"timing events {op}: {part * 1e3:.1f} of {whole * 1e3:.1f} us")
        assert 0.4 * whole <= part <= whole
    finally:
        ph.close()
