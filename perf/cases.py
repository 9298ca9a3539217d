"""The calls that this library's time is measured on, and exact values to hold them against.

Three paths, through the package's public functions: the gated delta-rule prefill of a prompt (dense, batched or
packed; plain, or with grouped key heads, the input transforms and state snapshots), the decode step, and the causal
attention prefill.  ``listed()`` names twelve cases, ``draw(rng)`` gives others of the same ranges:

  prefill   1 to 8 prompts of 64 to 10240 tokens, at most 18432 tokens a call; 1 to 16 heads of 64 or 128; float32
            (at most 4096 tokens a call of 16 heads) and bfloat16
  decode    1 to 512 sequences, 16 heads of 128, float32 and bfloat16
  attention 1 to 8 prompts of 64 to 10240 tokens, 16 query heads over 4, 8 or 16 key/value heads of 64 or 128

The chunk length is the functions' default.  Inputs follow the workloads' recipe (``paper_2607_14568_amd/inputs.py``),
drawn on the GPU: unit-length q and k, v ~ N(0,1), beta = sigmoid(N(0,1)), g = -softplus(N(0,1) + shift) and an initial
state of standard deviation 0.02; ``raw`` cases hand over q, k and the gates before those transforms.
"""
from __future__ import annotations

import math

import torch

import paper_2607_14568_amd as gdn

CHUNK = 64
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _prefill(name, T, H, d, io, *, B=1, Hk=None, lens="", shift=0.0, raw=False, snap=0):
    """``lens``: comma-separated lengths of packed sequences ("" for dense input); ``snap``: chunks a snapshot."""
    return dict(name=name, kind="prefill", B=B, T=T, H=H, Hk=Hk or H, d=d, io=io, lens=lens, shift=shift, raw=raw,
                snap=snap)


def _decode(name, B, io, *, H=16, Hk=None, d=128, raw=False):
    return dict(name=name, kind="decode", B=B, H=H, Hk=Hk or H, d=d, io=io, raw=raw)


def _attention(name, T, *, B=1, H=16, Hkv=8, d=128, lens=""):
    return dict(name=name, kind="attention", B=B, T=T, H=H, Hkv=Hkv, d=d, lens=lens)


def listed():
    packed = "903,3412,1777,4096,512,2650,1231,2900"
    return [
        # one user's next token, the model's own inputs (grouped heads, transforms in the kernel): latency
        _decode("decode_b1_bf16", 1, "bf16", Hk=8, raw=True),
        # the next token of a serving batch, plain inputs
        _decode("decode_b64_f32", 64, "f32"),
        # a large serving batch: more state than the last-level cache holds
        _decode("decode_b512_f32", 512, "f32"),
        # the smallest prompt, two small heads: launches and their latency
        _prefill("prefill_tiny_f32", 256, 2, 64, "f32"),
        # a 2k prompt in float32, all heads
        _prefill("prefill_2k_f32", 2048, 16, 128, "f32"),
        # four prompts of equal, odd length in float32, long memory
        _prefill("prefill_batch_f32", 999, 16, 128, "f32", B=4, shift=-3.0),
        # the long prompt in bfloat16, all heads: the library's main workload
        _prefill("prefill_10k_bf16", 10240, 16, 128, "bf16", shift=2.0),
        # the same prompt as one of eight devices sees it when the heads are split
        _prefill("prefill_10k_h2_bf16", 10240, 2, 128, "bf16", shift=-2.0),
        # eight packed prompts of a serving batch
        _prefill("prefill_packed_bf16", 17481, 16, 128, "bf16", lens=packed),
        # a model's layer that fills a prefix cache: grouped heads, transforms in the kernel, a state every 512 tokens
        _prefill("prefill_snap_bf16", 3001, 16, 128, "bf16", Hk=8, shift=-1.0, raw=True, snap=8),
        # the long prompt through an attention layer
        _attention("attention_10k_bf16", 10240),
        # the serving batch's packed prompts through an attention layer
        _attention("attention_packed_bf16", 17481, lens=packed),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lengths(rng, n, lo, hi, total):
    """n lengths in [lo, hi], spread over their logarithm, shrunk to at most ``total`` together."""
    ls = [_log_int(rng, lo, hi) for _ in range(n)]
    while sum(ls) > total:
        ls = [max(lo, x * 3 // 4) for x in ls]
    return ls


def draw(rng):
    kind = rng.choice(["prefill"] * 5 + ["decode"] * 2 + ["attention"] * 2)
    if kind == "decode":
        H_k = rng.choice([4, 8, 16])
        c = _decode("", _log_int(rng, 1, 512), rng.choice(["f32", "bf16"]), Hk=H_k, raw=rng.random() < 0.5)
    elif kind == "attention":
        lens, B = "", 1
        T = _log_int(rng, 64, 10240)
        if rng.random() < 0.5:
            ls = _lengths(rng, rng.randint(2, 8), 64, 4096, 17481)
            lens, T = ",".join(map(str, ls)), sum(ls)
        elif T <= 2048:
            B = rng.randint(1, 4)
        c = _attention("", T, B=B, Hkv=rng.choice([4, 8, 16]), d=rng.choice([64, 128, 128]), lens=lens)
    else:
        io = rng.choice(["f32", "bf16", "bf16"])
        H, d = rng.choice([1, 2, 4, 8, 16, 16, 16]), rng.choice([64, 128, 128, 128])
        limit = min(10240, 4096 * 16 // H) if io == "f32" else 10240
        T, B, lens, snap = _log_int(rng, 64, limit), 1, "", 0
        form = rng.choice(["one", "one", "batch", "packed", "snap"])
        if form == "batch":
            B = rng.randint(2, 8)
            T = min(T, limit // B)
        elif form == "packed":
            ls = _lengths(rng, rng.randint(2, 8), 64, 4096, limit if io == "f32" else 17481)
            lens, T = ",".join(map(str, ls)), sum(ls)
        elif form == "snap":
            snap = rng.choice([4, 8, 16])
        raw = rng.random() < 0.4
        c = _prefill("", T, H, d, io, B=B, Hk=max(1, H // rng.choice([1, 2])) if raw else H, lens=lens,
                     shift=rng.choice([2.0, 0.0, -2.0, -4.0]), raw=raw, snap=snap)
    del c["name"]
    return c


def _seq_lengths(case):
    return [int(x) for x in case["lens"].split(",")] if case["lens"] else [case["T"]] * case["B"]


def _cu(case, device):
    if not case["lens"]:
        return None
    return torch.tensor([0] + _seq_lengths(case), dtype=torch.int32).cumsum(0, dtype=torch.int32).to(device)


def _inputs(case, seed):
    """The call's inputs on the GPU, from the seed alone."""
    dev = torch.device("cuda", torch.cuda.current_device())
    rng = torch.Generator(device=dev)
    rng.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=rng, device=dev, dtype=torch.float32)

    if case["kind"] == "attention":
        B, T, H, Hkv, d = (case[x] for x in ("B", "T", "H", "Hkv", "d"))
        return dict(q=normal(B, T, H, d).bfloat16(), k=normal(B, T, Hkv, d).bfloat16(),
                    v=normal(B, T, Hkv, d).bfloat16(), cu=_cu(case, dev))
    H, Hk, d, io = case["H"], case["Hk"], case["d"], DTYPES[case["io"]]
    rows = (case["B"],) if case["kind"] == "decode" else (case["B"], case["T"])
    n = case["B"] if case["kind"] == "decode" else len(_seq_lengths(case))
    q, k, v = normal(*rows, Hk, d), normal(*rows, Hk, d), normal(*rows, H, d)
    b, a = normal(*rows, H), normal(*rows, H) + case.get("shift", 0.0)
    if not case["raw"]:
        q, k = q / q.norm(dim=-1, keepdim=True), k / k.norm(dim=-1, keepdim=True)
        b, a = torch.sigmoid(b), -torch.nn.functional.softplus(a)
    return dict(q=q.to(io), k=k.to(io), v=v.to(io), g=a, beta=b, S0=0.02 * normal(n, H, d, d),
                cu=None if case["kind"] == "decode" else _cu(case, dev))


def prepare(case, seed):
    """Inputs, and the output buffers and workspace that a serving program keeps."""
    x = _inputs(case, seed)
    if case["kind"] == "attention":
        return dict(x, case=case, o=torch.empty_like(x["q"]))
    state = dict(x, case=case, o=torch.empty_like(x["v"]),
                 flags=gdn.GDN_QK_L2NORM | gdn.GDN_GATE_LOGITS if case["raw"] else 0)
    if case["kind"] == "decode":
        return state
    lens = _seq_lengths(case)
    H, d = case["H"], case["d"]
    io = gdn.GDN_BF16 if case["io"] == "bf16" else gdn.GDN_F32
    need = gdn.gdn_chunk_prefill_workspace_bytes_ex(case["B"], case["T"], H, d, d, CHUNK,
                                                    len(lens) if case["lens"] else 0, io, state["flags"], 0)
    state["workspace"] = torch.empty(need, dtype=torch.uint8, device=x["q"].device)
    state["S_T"] = torch.empty_like(x["S0"])
    if case["snap"]:
        n_snap = (case["T"] - 1) // (case["snap"] * CHUNK)
        state["snaps"] = torch.zeros(len(lens), n_snap, H, d, d, device=x["q"].device)
    return state


def run(state):
    case, s = state["case"], state
    if case["kind"] == "attention":
        return gdn.gdn_attention_prefill(s["q"], s["k"], s["v"], cu_seqlens=s["cu"], o=s["o"])
    if case["kind"] == "decode":
        if case["raw"] or case["Hk"] != case["H"]:
            o = gdn.gdn_decode_step_ex(s["q"], s["k"], s["v"], s["g"], s["beta"], s["S0"], flags=s["flags"], o=s["o"])
        else:
            o = gdn.gdn_decode_step(s["q"], s["k"], s["v"], s["g"], s["beta"], s["S0"], o=s["o"])
        return o, s["S0"]
    keep = dict(cu_seqlens=s["cu"], o=s["o"], S_T=s["S_T"], workspace=s["workspace"])
    if case["snap"]:
        return gdn.gdn_chunk_prefill_snapshots_ex(s["q"], s["k"], s["v"], s["g"], s["beta"], s["S0"],
                                                  snap_every=case["snap"], flags=s["flags"], snaps=s["snaps"], **keep)
    if case["raw"] or case["Hk"] != case["H"]:
        return gdn.gdn_chunk_prefill_ex(s["q"], s["k"], s["v"], s["g"], s["beta"], s["S0"], flags=s["flags"], **keep)
    return gdn.gdn_chunk_prefill(s["q"], s["k"], s["v"], s["g"], s["beta"], s["S0"], **keep)


def work(case):
    """Every input read once, every output written once; the recurrence's three products with the state per token."""
    if case["kind"] == "attention":
        B, T, H, Hkv, d = (case[x] for x in ("B", "T", "H", "Hkv", "d"))
        return dict(bytes=B * T * (2 * H + 2 * Hkv) * d * 2, flops=sum(2 * d * H * n * (n + 1) for n in _seq_lengths(case)))
    H, Hk, d, size = case["H"], case["Hk"], case["d"], 2 if case["io"] == "bf16" else 4
    lens = [1] * case["B"] if case["kind"] == "decode" else _seq_lengths(case)
    tokens, states = sum(lens), 2 * len(lens)
    if case.get("snap"):
        states += sum((n - 1) // (case["snap"] * CHUNK) for n in lens)
    return dict(bytes=tokens * ((2 * Hk + 2 * H) * d * size + 8 * H) + states * H * d * d * 4,
                flops=tokens * H * 6 * d * d)


def tolerance(case):
    """About four times the largest error against float64 that was measured over these ranges: 2.1e-3 for attention,
    1.7e-3 and 1.4e-7 for the decode step, 3.6e-3 and 7e-6 for the prefill (whose float32 products are split bfloat16)."""
    if case["kind"] == "attention":
        return {"rel": 8e-3}
    if case["kind"] == "decode":
        return {"rel": 7e-3 if case["io"] == "bf16" else 6e-7}
    return {"rel": 1.4e-2 if case["io"] == "bf16" else 3e-5}


def _recurrence(q, k, v, g, beta, S, snap):
    """One token after the other in float64: q, k, v [n,T,H,d], g, beta [n,T,H], S [n,H,d,d]."""
    o, snaps, T = torch.empty_like(v), [], q.shape[1]
    alpha = torch.exp(g)[..., None, None]
    for t in range(T):
        S = S * alpha[:, t]
        kt = k[:, t, :, None, :]
        u = beta[:, t, :, None] * (v[:, t] - (S * kt).sum(-1))
        S = S + u[..., None] * kt
        o[:, t] = (S * q[:, t, :, None, :]).sum(-1)
        if snap and (t + 1) % (snap * CHUNK) == 0 and t + 1 < T:
            snaps.append(S)
    return o, S, snaps


def _exact_attention(case, x):
    q, k, v = x["q"].double(), x["k"].double(), x["v"].double()
    B, H, Hkv, d = case["B"], case["H"], case["Hkv"], case["d"]
    o = torch.empty_like(q)
    spans, at = [], 0
    if case["lens"]:
        for n in _seq_lengths(case):
            spans.append((0, at, at + n))
            at += n
    else:
        spans = [(b, 0, case["T"]) for b in range(B)]
    for b, lo, hi in spans:
        for h in range(H):
            kh, vh = k[b, lo:hi, h // (H // Hkv)].contiguous(), v[b, lo:hi, h // (H // Hkv)].contiguous()
            for i in range(lo, hi, 2048):
                j = min(hi, i + 2048)
                s = (q[b, i:j, h].contiguous() @ kh[:j - lo].t().contiguous()) / d ** 0.5
                mask = torch.arange(i, j, device=s.device)[:, None] < torch.arange(lo, j, device=s.device)
                o[b, i:j, h] = torch.softmax(s.masked_fill(mask, -math.inf), dim=1) @ vh[:j - lo]
    return o


def exact(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "attention":
        return _exact_attention(case, x)
    q, k, v, g, beta = (x[n].double() for n in ("q", "k", "v", "g", "beta"))
    if case["raw"]:
        q, k = (t / torch.sqrt((t * t).sum(-1, keepdim=True) + 1e-6) for t in (q, k))
        g, beta = -torch.nn.functional.softplus(g), torch.sigmoid(beta)
    group = case["H"] // case["Hk"]
    q, k = (t.repeat_interleave(group, dim=-2) for t in (q, k))
    S0 = x["S0"].double()
    if case["kind"] == "decode":
        o, S, _ = _recurrence(*(t[:, None] for t in (q, k, v, g, beta)), S0, 0)
        return o[:, 0], S
    if not case["lens"]:
        o, S, snaps = _recurrence(q, k, v, g, beta, S0, case["snap"])
        return (o, S, torch.stack(snaps, 1) if snaps else S0.new_zeros(S0.shape[0], 0, *S0.shape[1:])) \
            if case["snap"] else (o, S)
    o, S, at = torch.empty_like(v), [], 0
    for i, n in enumerate(_seq_lengths(case)):
        part = slice(at, at + n)
        o[:, part], Si, _ = _recurrence(q[:, part], k[:, part], v[:, part], g[:, part], beta[:, part], S0[i:i + 1], 0)
        S.append(Si)
        at += n
    return o, torch.cat(S)
