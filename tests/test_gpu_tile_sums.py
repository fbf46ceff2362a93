"""Rounding of the tiled kernel's softmax and fidelity sums over a vocabulary
tile, through the C ABI.

One logit of 0 and all others just below the logarithm of half an ulp of 1: a
lane that adds its 32 terms one after the other, the 0 first, loses the other
31.  In groups it makes at most 7 roundings, the half-waves' sum 1, the four
waves' merge 3, and the logarithm, the tiles' merge and the result 1 each: 14
roundings of 2^-24 of a sum near 1.
"""
from __future__ import annotations

import numpy as np
import pytest

from synth import f64_to_bf16_bits, make_head
from tests.gpu_util import say, torch_x

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 14 * 2.0 ** -24
LOW = -16.65625                # exp: 0.98 * 2^-24; an fp16 scale times code -1
LOW_BF16 = -16.75              # exp: 0.89 * 2^-24


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _head(V, low):
    """logit[0] = 0, the others `low`, for x = (1, 0, ..., 0)."""
    h = make_head("tiny", V=V, d=64, g=64, rc=0, rr=0)
    h.res_codes[:] = 0x88
    h.res_codes[1:, 0] = 0x87
    h.res_scales[:] = -low
    return h


def _x(M):
    x = np.zeros((M, 64))
    x[:, 0] = 1
    return torch_x(f64_to_bf16_bits(x))


@pytest.mark.parametrize("V", [256, 1000])
@pytest.mark.parametrize("M", [33, 128, 1100])      # 64-, 128- and 256-row tiles
def test_cross_entropy(V, M):
    from paper_2608_02703_amd import PackedHead
    ph = PackedHead.from_arrays(_head(V, LOW))
    ph.force_path("tiled")
    try:
        say(f"tile sums: CE V={V} M={M}")
        ce, _ = ph.logits_ce(_x(M), torch.zeros(M, dtype=torch.int64, device="cuda"))
        torch.cuda.synchronize()
        err = np.abs(ce.cpu().numpy().astype(np.float64) - np.log1p((V - 1) * np.exp(LOW)))
        assert err.max() <= TOL, f"{err.max():.2e}"
    finally:
        ph.close()


@pytest.mark.parametrize("V", [256, 1000])
@pytest.mark.parametrize("M", [33, 130])            # 64-row and 128-row tiles
@pytest.mark.parametrize("a,b", [(LOW_BF16, -60.0), (-60.0, LOW)])
def test_divergence(V, M, a, b):
    from paper_2608_02703_amd import PackedHead
    ph = PackedHead.from_arrays(_head(V, b))
    dense = torch.zeros((V, 64), device="cuda")
    dense[1:, 0] = a
    try:
        say(f"tile sums: KL V={V} M={M} a={a} b={b}")
        kl = ph.logit_fidelity_head(_x(M), dense.bfloat16())[0]
        torch.cuda.synchronize()
        la, lb = (np.log1p((V - 1) * np.exp(v)) for v in (a, b))
        p = (V - 1) * np.exp(a - la)
        want = np.exp(-la) * (lb - la) + p * ((a - la) - (b - lb))
        err = np.abs(kl.cpu().numpy().astype(np.float64) - want)
        # (and the sum of p (a - b), fp32: 2^-20 of it)
        assert err.max() <= TOL + 2.0 ** -20 * p * abs(a - b), f"{err.max():.2e}"
    finally:
        ph.close()
