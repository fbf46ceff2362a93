"""GPU parity of archead_logits_topk (top-k selection; the candidate set of
top-k decoding and of the top-k agreement metric, Section 4 "Logit
Fidelity", Table 8) against the oracle's selection, through the C ABI.

The selection is an integer decision taken on the kernel's fp32 logits, so
the oracle selects over those same logits (archead_logits for the same M and
path): indices and values must match bit for bit, ties included.  Against
the oracle's fp64 logits the indices must agree wherever the order is
decided by more than the logit tolerance; where they differ, the two
entries' fp64 logits must lie within that tolerance of each other.

Cases: every kernel (forced) and the library's choice, M = 1 (the fused
single-token GEMV), small M on the decode kernels, several token tiles, and
M = 300 (two chunks of the unfused path, the second ragged); k = 1, 10, 64,
and for one token (whose lists the GEMV keeps up to k = 6) also 2, 5, 6;
8-bit scale codes, 5-bit core-left codes with ranks 10 / 6, a ragged V;
vocabulary rows duplicated so that exact ties land in the top k; and the
Qwen3-8B-shaped head at M = 1 against the full fp64 oracle logits.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

from oracle import head as ohead
from oracle import metrics
from synth import make_head, make_x
from tests.gpu_util import LOGIT_TOL, say, torch_x

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _duplicate_rows(h, src, dst):
    """The head with vocabulary rows dst replaced by copies of row src
    (bit-identical logits for every token)."""
    rep = {}
    for name in ("res_codes", "res_scales", "core_u", "core_u_scale", "corr_a",
                 "corr_a_scale", "res_row_scales"):
        a = getattr(h, name)
        if a is None or a.shape[0] != h.V:
            continue
        a = a.copy()
        a[dst] = a[src]
        rep[name] = a
    return dataclasses.replace(h, **rep)


def _check(ph, x_bits, k, ref=None, what=""):
    xt = torch_x(x_bits)
    lg = ph.logits(xt)
    vals, idx = ph.logits_topk(xt, k)
    torch.cuda.synchronize()
    lg, vals, idx = lg.cpu().numpy(), vals.cpu().numpy(), idx.cpu().numpy()
    ov, oi = metrics.topk(lg, k)
    bad = np.argwhere(idx != oi)
    assert bad.size == 0, (f"{what} k={k}: {len(bad)} indices differ, first {bad[0]}: "
                           f"{idx[tuple(bad[0])]} vs {oi[tuple(bad[0])]}")
    assert np.array_equal(vals.view(np.uint32), ov.view(np.uint32)), f"{what} k={k}: values"
    if ref is not None:
        _, ri = metrics.topk(ref, k)
        for m, j in np.argwhere(idx != ri):
            a, b = ref[m, idx[m, j]], ref[m, ri[m, j]]
            assert abs(a - b) <= 2 * LOGIT_TOL * (1 + max(abs(a), abs(b))), \
                f"{what} k={k}: token {m} slot {j}: {idx[m, j]} vs oracle {ri[m, j]} ({a} vs {b})"


HEADS = [  # (label, make_head overrides)
    ("tiny", {}),
    ("u8 scales", dict(scales="u8")),
    ("i5 rc10 rr6 g64", dict(rc=10, rr=6, core_u="i5", scales="u8")),
    ("ragged V", dict(V=1000)),
]


@pytest.mark.parametrize("label,kw", HEADS)
def test_topk_every_kernel(label, kw):
    from paper_2608_02703_amd import PackedHead
    h = make_head("tiny", **kw)
    ph = PackedHead.from_arrays(h)
    try:
        x_all = make_x("tiny", 300, d=h.d)
        ref_all = ohead.logits(h, x_all[:40])
        for path, Ms in (("auto", (1, 2, 40, 300)), ("gemv", (1, 3)), ("dec", (5,)),
                         ("mid", (21,)), ("tiled", (1, 70))):
            ph.force_path(path)
            for M in Ms:
                for k in (1, 2, 5, 6, 10, 64) if M == 1 else (1, 10, 64):
                    say(f"top-k {label}: {path} M={M} k={k}")
                    ref = ref_all[:M] if M <= 40 else None
                    _check(ph, x_all[:M], k, ref, f"{label} {path} M={M}")
    finally:
        ph.close()


def test_topk_exact_ties():
    from paper_2608_02703_amd import PackedHead
    h0 = make_head("tiny")
    x = make_x("tiny", 8)
    top = int(np.argmax(ohead.logits(h0, x[:1])[0]))
    V = h0.V
    dst = np.array(sorted({0, 1, top + 1 if top + 1 < V else top - 1, 4097, V - 1} - {top}))
    h = _duplicate_rows(h0, top, dst)
    ph = PackedHead.from_arrays(h)
    try:
        for path, M in (("gemv", 1), ("auto", 1), ("dec", 8), ("mid", 8), ("tiled", 8)):
            ph.force_path(path)
            say(f"top-k ties: {path} M={M}")
            xt = torch_x(x[:M])
            want = np.array(sorted(list(dst) + [top]))
            for k in (3, 6, 10) if M == 1 else (10,):
                vals, idx = ph.logits_topk(xt, k)
                torch.cuda.synchronize()
                idx = idx.cpu().numpy()
                # token 0: the tied copies lead, in index order
                assert np.array_equal(idx[0, :min(k, want.size)], want[:k]), (path, k, idx[0], want)
                _check(ph, x[:M], k, what=f"ties {path}")
    finally:
        ph.close()


@pytest.mark.timeout(900)
def test_topk_qwen_single_token_fused():
    from paper_2608_02703_amd import PackedHead
    h = make_head("qwen_decode")
    ph = PackedHead.from_arrays(h)
    try:
        x = make_x("qwen_decode", 1)
        say("top-k qwen M=1 (fused GEMV): oracle logits")
        ref = ohead.logits(h, x)
        for k in (1, 2, 3, 5, 6, 10, 64):   # (768 lists: the sixteen-wave merge from k = 3 on)
            say(f"top-k qwen M=1 k={k}")
            _check(ph, x, k, ref, "qwen M=1")
    finally:
        ph.close()


def test_topk_argument_checks():
    from paper_2608_02703_amd import PackedHead
    from paper_2608_02703_amd import archead as ab
    h = make_head("tiny", V=50)
    ph = PackedHead.from_arrays(h)
    try:
        xt = torch_x(make_x("tiny", 2, d=h.d))
        for k in (0, 51, 65):
            with pytest.raises(RuntimeError):
                ph.logits_topk(xt, k)
        vals, idx = ph.logits_topk(xt, 50)   # k = V: the whole row, sorted
        torch.cuda.synchronize()
        lg = ph.logits(xt).cpu().numpy()
        _, oi = metrics.topk(lg, 50)
        assert np.array_equal(idx.cpu().numpy(), oi)
        assert ab.TOPK_MAX == 64
    finally:
        ph.close()


@pytest.mark.parametrize("V", [70, 255, 1025, 5000, 65536, 65537, 270000, 1050000])
def test_topk_chunk_edges(V):
    """Rows of less than k chunks, of exactly some chunks and one more, and
    around the lengths where the chunk grows (64, 256, 1024, 2048 logits); logits
    equal in many chunks (more ties than the candidate buffer holds), signed
    zeros, infinities, NaN, and fewer than k numbers in a row."""
    from paper_2608_02703_amd import PackedHead
    # one group, no factors: logit[m, v] = scale[v] * (code row 0) . x[m]
    h = make_head("tiny", V=V, d=64, g=64, rc=0, rr=0)
    rng = np.random.default_rng(V)
    h.res_codes[:] = h.res_codes[0]
    h.res_scales[:, 0] = rng.integers(1, 40, V) / 16.0   # many ties
    h.res_scales[V // 2, 0] = np.float16(np.nan)
    h.res_scales[V - 1, 0] = np.float16(np.inf)
    x = make_x("tiny", 5, d=64)
    x[3] = 0                                             # every logit 0 (NaN where the scale is not finite)
    x[4, :] = 0x7F80                                     # NaN rows: nothing to select
    for const in (False, True):
        if const:
            h.res_scales[:] = 0.5                        # all logits of a row equal
        ph = PackedHead.from_arrays(h)
        try:
            for path in ("gemv", "mid", "tiled"):
                if path == "mid" and (V < 1024):
                    continue
                if path == "mid" and V > 60000 and const:
                    continue
                ph.force_path(path)
                for k in (1, 6, 7, 50, 64) if V < 60000 else (7, 64):
                    say(f"top-k chunk edges V={V} {path} k={k} const={const}")
                    # (one token alone may take the fused form)
                    xt = torch_x(x[:1] if k in (6, 7) else x)
                    lg = ph.logits(xt)
                    vals, idx = ph.logits_topk(xt, k)
                    torch.cuda.synchronize()
                    lg, vals, idx = lg.cpu().numpy(), vals.cpu().numpy(), idx.cpu().numpy()
                    for m in range(lg.shape[0]):
                        ok = np.nonzero(~np.isnan(lg[m]))[0]
                        order = ok[np.argsort(-lg[m, ok], kind="stable")][:k]
                        want = np.full(k, -1)
                        want[:order.size] = order
                        assert np.array_equal(idx[m], want), (V, path, k, m)
                        wv = np.full(k, -np.inf, np.float32)
                        wv[:order.size] = lg[m, order]
                        assert np.array_equal(vals[m].view(np.uint32), wv.view(np.uint32))
        finally:
            ph.close()


def test_topk_fused_grids():
    """The fused form's lists under other grids: few lists (the four-wave
    merge), many (the sixteen-wave one), and more than that holds, where one
    token takes the unfused form."""
    from paper_2608_02703_amd import PackedHead, archead as ab
    h = make_head("tiny", V=60000, d=2048, rc=256, rr=32)   # (32 rows a workgroup: up to 1875)
    x = make_x("tiny", 1, d=h.d)
    ph = PackedHead.from_arrays(h)
    ph.force_path("gemv")
    try:
        need = {}
        for grid in (7, 300, 700, 1365, 1366, 1800):
            ph.set_launch(ab.LAUNCH_GEMV_GRID, grid)
            need[grid] = ph.workspace_bytes(1, ab.OP_TOPK)
            for k in (1, 3, 6, 7):
                say(f"top-k GEMV grid {grid} k={k}")
                _check(ph, x, k, what=f"grid {grid}")
        assert need[1366] < need[1365]      # (no lists beside the logits)
    finally:
        ph.close()


@pytest.mark.parametrize("M,d", [(2100, 2048), (4100, 1024)])
def test_topk_of_chunks_selects_over_the_whole_calls_logits(M, d):
    """A call of several chunks of tokens selects over archead_logits' values
    for the same M, bit for bit, also where stage 1 of a chunk alone would be
    split along d otherwise (here 4 and 2 ways in a chunk of 256 tokens, 2 and
    1 ways in the call, which has 132 and 257 blocks of 16 tokens)."""
    from paper_2608_02703_amd import PackedHead
    h = make_head("tiny", V=256, d=d, g=64, rc=20, rr=0)
    ph = PackedHead.from_arrays(h)
    try:
        say(f"top-k chunks M={M}")
        _check(ph, make_x("tiny", M, d=d), 10, what=f"chunks M={M}")
    finally:
        ph.close()


def _row_kinds(V):
    """Heads (d = g = 64, a core and a correction of rank 1) whose logits over
    the vocabulary are of one kind, and whether x is (1, 0, ..., 0) instead of
    ones with noise."""
    v = np.arange(V)
    for kind, order in (("random", None), ("offset", None), ("ascending", v), ("descending", v[::-1]),
                        ("equal", 0 * v)):
        h = make_head("tiny", V=V, d=64, g=64, rc=1, rr=1)
        if order is None:          # +- 0.25, around 0 or around 1000
            h.res_scales[:] = 0.0017
            h.core_u[:] = h.core_v[:] = 1
            h.core_v_scale[:] = 1
            h.core_u_scale[:] = 1000 / 64 if kind == "offset" else 0
            h.corr_a[:] = 0
        else:                      # multiples of 2^-10: the whole part, then the rest
            h.res_codes[:] = 0x88
            h.res_codes[:, 0] = 0x89
            h.res_scales[:, 0] = order // 1024
            h.core_u[:] = 0
            h.corr_a[:] = 1
            h.corr_a_scale[:] = order % 1024 / 1024
            h.corr_b[:] = 0
            h.corr_b[0, 0] = 1
            h.corr_b_scale[:] = 1
        yield kind, h, order is not None


@pytest.mark.parametrize("V", [4000, 151936])
def test_topk_time_hardly_depends_on_the_values(V):
    """Rows around a large value, sorted ones and rows of equal logits (a padding
    token's) are selected from in about the time of random ones: within a
    factor of two over the whole call.  (Reading every chunk that ties at the
    floor and ranking thousands of logits one against all took 4 times as long
    for rows around 1000 and 20 to 50 times for sorted ones.)"""
    from paper_2608_02703_amd import PackedHead
    M, us = 24, {}
    for kind, h, first in _row_kinds(V):
        ph = PackedHead.from_arrays(h)
        try:
            x = torch.ones((M, 64), device="cuda")
            if first:
                x[:, 1:] = 0
            else:
                x += 0.1 * torch.randn((M, 64), generator=torch.Generator().manual_seed(1)).cuda()
            x = x.bfloat16()
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            for k in (10, 50, 64):
                say(f"top-k of {kind} rows V={V} k={k}")
                _check(ph, x.view(torch.int16).cpu().numpy().view(np.uint16), k, what=kind)
                best = float("inf")
                for _ in range(5):
                    e[0].record()
                    for _ in range(10):
                        ph.logits_topk(x, k)
                    e[1].record()
                    e[1].synchronize()
                    best = min(best, e[0].elapsed_time(e[1]) * 100)
                us[kind, k] = best
                say(f"  {best:.1f} us")
                assert best <= 2 * us["random", k]
        finally:
            ph.close()
