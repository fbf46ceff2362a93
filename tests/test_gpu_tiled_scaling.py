"""The tiled kernel's power-of-two scaling of x, through the C ABI.

Every token's x is scaled by a power of two of its own before the MFMAs and
the logits are scaled back, so a row's magnitude must not matter: rows of
magnitudes 2^-100 .. 2^90, a zero row and a subnormal row against the oracle,
a row with an infinity and one with a NaN (all logits of those rows are NaN,
their neighbours are untouched), on heads with ragged vocabulary, groups of
64, 128 and 192 (one to three stages per scale slot), with an odd number of
residual stages (the codes come for two) followed by an even and an odd number
of expansion stages and by none, both, one or no expansion part, zero scales and 8-bit scales; logits into rows that take the
16-byte stores and rows that do not, fp32 and bf16.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import head as ohead
from synth import f64_to_bf16_bits, make_head
from tests.gpu_util import bf16_bits_to_f64, say, torch_x

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# fp32 partial sums: at most d / 16 + 3 * 4 accumulations and d / g + 2
# rescales of a sum whose parts reach twice the result's scale (offset 8 codes)
ROUNDINGS = 768 / 16 + 12 + 12 + 2
REL = 2 * ROUNDINGS * 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("kw,M", [
    (dict(V=700, d=768, g=192, rc=20, rr=12), 64),
    (dict(V=515, d=768, g=64, rc=0, rr=16), 65),
    (dict(V=1000, d=512, g=128, rc=40, rr=0, scales="u8"), 130),
    (dict(V=256, d=512, g=64, rc=0, rr=0), 300),
    (dict(V=77, d=64, g=64, rc=16, rr=4), 33),      # a single stage per part
    # an odd number of residual stages, in every tile layout below
    (dict(V=300, d=192, g=64, rc=0, rr=0), 300),
    (dict(V=300, d=192, g=192, rc=16, rr=0), 64),
    (dict(V=300, d=320, g=64, rc=16, rr=4), 130),
    (dict(V=300, d=320, g=320, rc=0, rr=20, scales="u8"), 65),
    (dict(V=300, d=448, g=64, rc=20, rr=16), 1100),
])
def test_row_magnitudes(kw, M):
    from paper_2608_02703_amd import PackedHead, archead as ab
    h = make_head("tiny", **kw)
    h.res_scales[::7, 0] = 0            # zero scales inside a row
    h.res_scales[5] = 0                 # and a row of nothing else
    d, V = kw["d"], kw["V"]
    rng = np.random.default_rng(3)
    mag = np.array([0, -100, 90, -40, 40, 7, -3])[np.arange(M) % 7]
    x = f64_to_bf16_bits(rng.standard_normal((M, d)) * 2.0 ** mag[:, None])
    x[8] = 0
    x[9] = rng.integers(0, 128, d)      # bf16 subnormals
    inf_row, nan_row = 11, 20
    ref = ohead.logits(h, x)
    x[inf_row, 5] = 0x7F80
    x[nan_row, 6] = 0x7FC0
    ph = PackedHead.from_arrays(h)
    ph.force_path("tiled")
    try:
        layouts = [(0, 0)] + [(4, 64), (4, 128), (8, 0)] * (kw["d"] // 64 % 2)
        for waves, rows, pad in [(*la, pad) for la in layouts for pad in (0, 1, 4)]:
            ph.set_launch(ab.LAUNCH_TILE_WAVES, waves)
            ph.set_launch(ab.LAUNCH_TILE_ROWS, rows)
            for dtype in (torch.float32, torch.bfloat16):
                say(f"tiled scaling {kw} M={M} pad={pad} {dtype} layout {waves} {rows}")
                out = torch.full((M, V + pad + 3), 3.0, device="cuda", dtype=dtype)
                ph.logits(torch_x(x), out=out[:, :V], out_dtype=dtype)
                torch.cuda.synchronize()
                o = out.float().cpu().numpy().astype(np.float64)
                assert (o[:, V:] == 3.0).all(), "wrote past the row"
                o = o[:, :V]
                for m in range(M):
                    if m in (inf_row, nan_row):
                        assert np.isnan(o[m]).all(), f"row {m}: inf / NaN lost"
                        continue
                    # (rows at fp32's own end lose bits to its subnormals)
                    n = np.linalg.norm(ref[m])
                    err = np.linalg.norm(o[m] - ref[m])
                    rel = REL if dtype == torch.float32 else 2.0 ** -8
                    assert err <= rel * n + 2.0 ** -126 * np.sqrt(V), \
                        f"row {m} (2^{mag[m]}): {err / max(n, 1e-300):.2e}"
    finally:
        ph.close()


@pytest.mark.parametrize("low", [-40, -60, -75])
def test_small_logits_beside_a_large_element(low):
    """A token's logits keep their bits where its largest element meets only
    codes of zero and the others are 2^low of it."""
    from paper_2608_02703_amd import PackedHead
    h = make_head("tiny", V=300, d=256, g=64, rc=16, rr=4)
    codes = np.array(h.res_codes)
    codes[:, 0] = codes[:, 0] & 0xF0 | 8       # element 0: code 0
    h.res_codes[:] = codes
    h.core_v[:, 0] = 0
    h.corr_b[:, 0] = 0
    rng = np.random.default_rng(4)
    x = rng.standard_normal((33, 256)) * 2.0 ** low
    x[:, :64] = 0                              # (the large element's group holds nothing else)
    x[:, 0] = 3.0
    x = f64_to_bf16_bits(x)
    ref = ohead.logits(h, x)
    ph = PackedHead.from_arrays(h)
    ph.force_path("tiled")
    try:
        say(f"tiled small logits 2^{low}")
        o = ph.logits(torch_x(x))
        torch.cuda.synchronize()
        o = o.cpu().numpy().astype(np.float64)
        err = np.linalg.norm(o - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= REL, f"{err.max():.2e}"
    finally:
        ph.close()


def test_every_code_and_position():
    """One-hot rows read back every code value at every position of a word,
    exactly: the offset cancels, and x's extra 1 / 16 at the odd code pairs."""
    from paper_2608_02703_amd import PackedHead
    h = make_head("tiny", V=256, d=128, g=64, rc=0, rr=0)
    h.res_scales[:] = 1.0
    x = f64_to_bf16_bits(np.eye(128) * 3.0)
    ref = ohead.logits(h, x)
    assert np.unique(ref).size == 16
    ph = PackedHead.from_arrays(h)
    ph.force_path("tiled")
    try:
        say("tiled one-hot")
        o = ph.logits(torch_x(x))
        torch.cuda.synchronize()
        assert np.array_equal(o.cpu().numpy().astype(np.float64), ref)
    finally:
        ph.close()
    assert np.array_equal(bf16_bits_to_f64(x), np.eye(128) * 3.0)


def test_noalloc_in_chunks_of_tokens():
    """A call whose copy of x does not fit the static array runs in chunks,
    bit-identical to archead_logits; the limit itself leaves the copy out."""
    from paper_2608_02703_amd import PackedHead, archead as ab
    h = make_head("tiny", V=77, d=512, g=64, rc=16, rr=4)
    ph = PackedHead.from_arrays(h)
    try:
        for M in (8000, 8301):
            say(f"noalloc chunks M={M}")
            assert ph.workspace_bytes(M) > 2 * ab.NOALLOC_SCRATCH_BYTES
            x = torch.randn((M, 512), generator=torch.Generator().manual_seed(M)).bfloat16().cuda()
            a, b = ph.logits(x), ph.logits_noalloc(x)
            torch.cuda.synchronize()
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
        with pytest.raises(ab.ArcheadError) as e:
            ph.logits_noalloc(torch.zeros((16000, 512), dtype=torch.bfloat16, device="cuda"))
        assert e.value.status == ab.E_WORKSPACE
    finally:
        ph.close()
