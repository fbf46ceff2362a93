"""Workloads of the packed-head forward that a serving or evaluation program
runs, for timing and for comparing outputs.

A case names a head (its shape and storage options), a public entry point of
``paper_2608_02703_amd.PackedHead`` and the number of tokens.  The heads are
this repository's own shapes (``synth.CONFIGS``: tiny, qwen, gemma,
sweep128k, and the paper's Qwen storage with 5-bit core codes, 8-bit scale
codes and ranks 10 / 6) and generic ones with an odd vocabulary.

  logits    ``logits``: fp32 or bf16 [M, V], for a program that samples
  argmax    ``logits_argmax``: greedy decoding
  topk      ``logits_topk``: top-k decoding
  ce        ``logits_ce``: perplexity of a prefill or evaluation batch
  fidelity  ``logit_fidelity_head``: the packed head against the dense one

Heads used with more than 32 tokens have their tables built with
``prepare()`` once, as a server does at load time, unless the case says a
head is used once (``prepared`` false).  Building a head happens once per
model, outside any serving path, and is not among the cases.
"""
from __future__ import annotations

import math

import torch

from paper_2608_02703_amd import PackedHead, packed_bytes
from paper_2608_02703_amd.archead import Desc, F16, I5, I8, U8

RES_SIGMA = 0.02        # group scales |N(0, 0.02)|, as in synth
FACTOR_SIGMA = 0.002    # factor scales: core and residual logits of like size
X_RMS = 0.5             # hidden states after the final norm
OUTLIERS = 4            # channels x 8, as in trained models
ROW_CHUNK = 8192

_QWEN = dict(V=151936, d=4096, g=128, rc=64, rr=32, scales="f16", core_u="i8")
_GEMMA = dict(V=262144, d=2560, g=128, rc=64, rr=32, scales="f16", core_u="i8")
_WIDE = dict(V=128256, d=8192, g=128, rc=128, rr=64, scales="f16", core_u="i8")
_TINY = dict(V=8192, d=512, g=64, rc=64, rr=32, scales="f16", core_u="i8")
_PAPER = dict(V=151936, d=4096, g=64, rc=10, rr=6, scales="u8", core_u="i5")
_RAGGED = dict(V=50257, d=1536, g=64, rc=20, rr=12, scales="f16", core_u="i8")


def listed():
    return [
        # a small head, one stream: launch and latency
        dict(name="tiny_logits_m1", op="logits", M=1, out="f32", prepared=False, **_TINY),
        # one stream that samples from the logits
        dict(name="qwen_logits_m1", op="logits", M=1, out="f32", prepared=False, **_QWEN),
        # one stream with top-k sampling
        dict(name="gemma_topk10_m1", op="topk", M=1, k=10, prepared=False, **_GEMMA),
        # eight greedy streams on the storage the paper reports
        dict(name="paper_argmax_m8", op="argmax", M=8, prepared=False, **_PAPER),
        # a decode batch whose sampler takes bf16 logits
        dict(name="qwen_logits_m16_bf16", op="logits", M=16, out="bf16", prepared=False, **_QWEN),
        # a decode batch with top-k sampling on the widest head
        dict(name="wide_topk50_m24", op="topk", M=24, k=50, prepared=False, **_WIDE),
        # a larger decode batch, a size between the powers of two
        dict(name="qwen_logits_m48", op="logits", M=48, out="f32", prepared=True, **_QWEN),
        # greedy decoding of many streams (or verification of drafts)
        dict(name="gemma_argmax_m100", op="argmax", M=100, prepared=True, **_GEMMA),
        # scoring one short document with a head loaded for it: odd vocabulary
        # and length, tables built in the call
        dict(name="ragged_ce_m333", op="ce", M=333, prepared=False, **_RAGGED),
        # logits of a prompt chunk on the widest head
        dict(name="wide_logits_m512_bf16", op="logits", M=512, out="bf16", prepared=True, **_WIDE),
        # perplexity of a prefill-sized batch
        dict(name="qwen_ce_m4096", op="ce", M=4096, prepared=True, **_QWEN),
        # quality check of the packed head against the dense one
        dict(name="qwen_fidelity_m1024", op="fidelity", M=1024, prepared=True, **_QWEN),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = {"ce": 4096 * _QWEN["V"] * _QWEN["d"], "fidelity": 1024 * _QWEN["V"] * _QWEN["d"]}
    while True:
        op = rng.choice(["logits", "logits", "argmax", "topk", "ce", "fidelity"])
        head = dict(V=_log_int(rng, 8000, 262144),
                    d=rng.choice([512, 1024, 1536, 2048, 2560, 3072, 3584, 4096, 5120, 8192]),
                    g=rng.choice([64, 128, 128]))
        head["rc"], head["rr"] = rng.choice([(64, 32), (64, 32), (128, 64), (16, 8), (10, 6)])
        head["scales"] = rng.choice(["f16", "f16", "u8"])
        head["core_u"] = "i5" if (head["rc"], head["rr"]) == (10, 6) else "i8"
        lo, hi = {"ce": (16, 4096), "fidelity": (64, 1024)}.get(op, (1, 512))
        M = _log_int(rng, lo, hi)
        if M * head["V"] * head["d"] > most.get(op, most["fidelity"]):
            continue
        case = dict(op=op, M=M, prepared=M > 32 and rng.random() < 0.75, **head)
        if op == "logits":
            case["out"] = rng.choice(["f32", "bf16"])
        if op == "topk":
            case["k"] = rng.choice([1, 5, 10, 20, 50])
        return case


def _abs_normal(shape, sigma, gen):
    return (torch.randn(shape, generator=gen, device="cuda") * sigma).abs().to(torch.float16)


def _codes8(shape, gen):
    return torch.randint(-127, 128, shape, generator=gen, device="cuda", dtype=torch.int8)


def _buffers(case, gen):
    V, d, g, rc, rr = (case[n] for n in ("V", "d", "g", "rc", "rr"))
    b = dict.fromkeys(PackedHead.BUFFERS)
    b["res_codes"] = torch.randint(0, 256, (V, d // 2), generator=gen, device="cuda", dtype=torch.uint8)
    scales = _abs_normal((V, d // g), RES_SIGMA, gen)
    if case["scales"] == "u8":
        rows = (scales.amax(1).float() / 255).to(torch.float16)
        q = torch.round(scales.float() / rows.float().clamp_min(1e-7)[:, None]).clamp_(0, 255)
        b["res_scales"], b["res_row_scales"] = q.to(torch.uint8), rows
    else:
        b["res_scales"] = scales
    if case["core_u"] == "i5":   # six 5-bit fields a word
        f = torch.randint(-15, 16, (V, (rc + 5) // 6 * 6), generator=gen, device="cuda", dtype=torch.int32)
        f[:, rc:] = 0
        shift = torch.arange(6, device="cuda", dtype=torch.int32) * 5
        b["core_u"] = ((f & 31).view(V, -1, 6) << shift).sum(-1, dtype=torch.int32)
        u_sigma = FACTOR_SIGMA * 8
    else:
        b["core_u"], u_sigma = _codes8((V, rc), gen), FACTOR_SIGMA
    b["core_u_scale"] = _abs_normal((V,), u_sigma, gen)
    b["core_v"], b["core_v_scale"] = _codes8((rc, d), gen), _abs_normal((rc, 1), FACTOR_SIGMA, gen)
    b["corr_a"], b["corr_a_scale"] = _codes8((V, rr), gen), _abs_normal((V,), FACTOR_SIGMA, gen)
    b["corr_b"], b["corr_b_scale"] = _codes8((rr, d), gen), _abs_normal((rr, 1), FACTOR_SIGMA, gen)
    return b


def _rows(case, b, v0, v1, dtype):
    """Rows [v0, v1) of the dense matrix the packed head stands for."""
    d, g, rc = case["d"], case["g"], case["rc"]
    q = b["res_codes"][v0:v1].view(torch.int32)
    shift = torch.tensor([0, 16, 4, 20, 8, 24, 12, 28], device=q.device, dtype=torch.int32)
    c = ((q[:, :, None] >> shift) & 15).view(v1 - v0, d) - 8
    s = b["res_scales"][v0:v1].to(dtype)
    if b["res_row_scales"] is not None:
        s = s * b["res_row_scales"][v0:v1, None].to(dtype)
    w = (c.to(dtype).view(v1 - v0, d // g, g) * s[:, :, None]).view(v1 - v0, d)
    u = b["core_u"][v0:v1]
    if case["core_u"] == "i5":
        left = 27 - torch.arange(6, device=u.device, dtype=torch.int32) * 5
        u = (((u[:, :, None] << left) >> 27).view(v1 - v0, -1))[:, :rc]
    for a, sa, m, sm in ((u, "core_u_scale", "core_v", "core_v_scale"),
                         (b["corr_a"][v0:v1], "corr_a_scale", "corr_b", "corr_b_scale")):
        w += (a.to(dtype) * b[sa][v0:v1, None].to(dtype)) @ (b[m].to(dtype) * b[sm].to(dtype))
    return w, s


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    b = _buffers(case, gen)
    M, d = case["M"], case["d"]
    channel = torch.exp(0.5 * torch.randn(d, generator=gen, device="cuda"))
    channel[torch.randint(0, d, (OUTLIERS,), generator=gen, device="cuda")] *= 8
    x = torch.randn((M, d), generator=gen, device="cuda") * channel
    x = (x * (X_RMS / x.square().mean(1, keepdim=True).sqrt())).to(torch.bfloat16)
    extra = None
    if case["op"] == "ce":   # token ids by frequency rank, roughly 1 / rank
        r = torch.rand(M, generator=gen, device="cuda")
        extra = torch.exp(r * math.log(case["V"])).long().clamp_(1, case["V"]) - 1
    if case["op"] == "fidelity":   # the head before its residual was rounded to 4 bits
        extra = torch.empty((case["V"], d), dtype=torch.bfloat16, device="cuda")
        for v0 in range(0, case["V"], ROW_CHUNK):
            v1 = min(v0 + ROW_CHUNK, case["V"])
            w, s = _rows(case, b, v0, v1, torch.float32)
            e = torch.rand((v1 - v0, d), generator=gen, device="cuda") - 0.5
            extra[v0:v1] = w + e * s.repeat_interleave(case["g"], 1)
    return b, x, extra


def prepare(case, seed):
    b, x, extra = _inputs(case, seed)
    head = PackedHead(case["V"], case["d"], case["g"], case["rc"], case["rr"], b)
    if case["prepared"]:
        head.prepare()
    return dict(case=case, head=head, x=x, extra=extra)


def run(state):
    case, head, x = state["case"], state["head"], state["x"]
    if case["op"] == "logits":
        return head.logits(x, out_dtype=torch.bfloat16 if case["out"] == "bf16" else torch.float32)
    if case["op"] == "argmax":
        return head.logits_argmax(x)
    if case["op"] == "topk":
        return head.logits_topk(x, case["k"])
    if case["op"] == "ce":
        return head.logits_ce(x, state["extra"])
    return head.logit_fidelity_head(x, state["extra"])


def work(case):
    V, d, M, r = case["V"], case["d"], case["M"], case["rc"] + case["rr"]
    desc = Desc.make(V, d, case["g"], case["rc"], case["rr"],
                     scale_dtype=U8 if case["scales"] == "u8" else F16,
                     core_u_dtype=I5 if case["core_u"] == "i5" else I8)
    nbytes = packed_bytes(desc) + 2 * M * d
    flops = 2 * M * V * (d + r) + 2 * M * d * r
    if case["op"] == "logits":
        nbytes += M * V * (2 if case["out"] == "bf16" else 4)
    elif case["op"] == "fidelity":
        nbytes += 2 * V * d + M * 24
        flops += 2 * M * V * d
    else:
        nbytes += M * {"argmax": 12, "ce": 12, "topk": 12 * case.get("k", 0)}[case["op"]]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Against 64 bits the fp32 logits, maxima and cross-entropies are 1e-7 to
    # 6e-7 off, the KL divergence (a small difference of large sums) 1.1e-4;
    # bf16 logits differ where two fp32 results round to either side.  Whole
    # values may differ where two logits are equal to fp32 rounding.
    if case["op"] == "logits" and case["out"] == "bf16":
        return {"rel": 2e-3}
    return {"rel": 5e-4 if case["op"] == "fidelity" else 3e-6, "differ": 0.02}


def exact(case, seed):
    b, x, extra = _inputs(case, seed)
    x = x.double()
    V, op = case["V"], case["op"]
    lg = torch.empty((case["M"], V), dtype=torch.float64, device="cuda")
    ref = torch.empty_like(lg) if op == "fidelity" else None
    for v0 in range(0, V, ROW_CHUNK):
        v1 = min(v0 + ROW_CHUNK, V)
        lg[:, v0:v1] = x @ _rows(case, b, v0, v1, torch.float64)[0].T
        if ref is not None:
            ref[:, v0:v1] = x @ extra[v0:v1].double().T
    if op == "logits":
        return lg
    if op == "argmax":
        top, idx = lg.max(1)
        return idx, top
    if op == "topk":
        return tuple(torch.topk(lg, case["k"], dim=1))
    if op == "ce":
        ce = torch.logsumexp(lg, 1) - lg.gather(1, extra[:, None])[:, 0]
        return ce, ce.mean().reshape(1)
    la, lb = torch.log_softmax(ref, 1), torch.log_softmax(lg, 1)
    kl = (la.exp() * (la - lb)).sum(1)
    sq = (ref - lg).square().sum(1)
    idx = ref.argmax(1)
    at = lg.gather(1, idx[:, None])
    return kl, sq, idx, (lg > at).sum(1)
