"""Performance cases of the engine: what a program that decodes with it spends its time on.

Three kinds of call, through the Python binding of the C ABI (the sizes are those of the workload shapes in
`asd_inputs.SHAPES`, cut to one or two layers where a layer says as much as the whole model):

  rows      `Engine.forward_noalloc`: one decoding pass of 1..16 rows over a filled cache.  One row is a plain or a
            draft step (with `skip`, a step of the layer-skipping draft model), several are a verification pass.
  prefill   `Engine.prefill`: the prompt pass (more than 16 tokens: the matrix-core path in blocks).
  generate  `Engine.generate`: prompt pass, Algorithm 1 or a fixed mask, the draft / verify / accept loop; greedy, or
            sampled at a temperature; then `Engine.forward` on the last token, so that logits come back as well.

Weights are random: normal with standard deviation 0.02, the output projections of the sublayers smaller (0.02 / 8), so
that a sublayer changes the residual stream by a part of its length as it does in a trained model; norm gains 1 + 0.1 z;
token ids uniform.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import asd_inputs as si
import paper_2410_01028_amd as asd

DEVICE = "cuda:0"
PAGE = {"tiny": 64, "7b": 256, "13b": 256, "70b": 256}
# longest context of a `rows` case: the scratch of forward_noalloc holds the attention partials of so many positions
MOST_CTX = {"tiny": 4000, "7b": 7600, "13b": 5800, "70b": 3500}


def listed():
    return [
        # the smallest call: one token of the small fp32 model, launch latency and nothing else
        {"name": "row-tiny", "kind": "rows", "shape": "tiny", "layers": 4, "rows": 1, "ctx": 45, "skip": ""},
        # plain decoding, one token of the 7B shape behind a 512-token prompt and a few tokens more: streams every weight once
        {"name": "row-7b", "kind": "rows", "shape": "7b", "layers": 2, "rows": 1, "ctx": 515, "skip": ""},
        # verification of six drafts on the 13B shape at its workload's context
        {"name": "verify-13b", "kind": "rows", "shape": "13b", "layers": 2, "rows": 7, "ctx": 1031, "skip": ""},
        # verification of eight drafts on the grouped-query 70B shape
        {"name": "verify-70b", "kind": "rows", "shape": "70b", "layers": 1, "rows": 9, "ctx": 2053, "skip": ""},
        # verification at a long context: the attention over the cache weighs as much as the weights
        {"name": "verify-7b-long", "kind": "rows", "shape": "7b", "layers": 2, "rows": 7, "ctx": 7411, "skip": ""},
        # the whole program on the small fp32 model: prompt 32, 32 tokens, four drafts a cycle, Algorithm 1's mask
        {"name": "generate-tiny", "kind": "generate", "shape": "tiny", "layers": 4, "prompt": 32, "new": 32, "draft": 4, "temp": 0.0, "skip": ""},
        # sampled speculative decoding (T = 0.6) at 7B width, the draft model without the first attention sublayer
        {"name": "generate-7b-sampled", "kind": "generate", "shape": "7b", "layers": 2, "prompt": 300, "new": 24, "draft": 4, "temp": 0.6, "skip": "1000"},
        # a short instruction as prompt: 45 tokens, where the weights are read for few rows
        {"name": "prefill-7b-short", "kind": "prefill", "shape": "7b", "layers": 2, "rows": 45},
        # the prompt pass of the 7B workload, whole model
        {"name": "prefill-7b", "kind": "prefill", "shape": "7b", "layers": 32, "rows": 512},
        # a news article on the 13B shape: about 1000 tokens, a ragged last block
        {"name": "prefill-13b", "kind": "prefill", "shape": "13b", "layers": 2, "rows": 1003},
        # the long-context workload's prompt: attention over 8192 tokens beside the contractions
        {"name": "prefill-7b-long", "kind": "prefill", "shape": "7b", "layers": 2, "rows": 8192},
        # the 70B workload's prompt: wide layers, eight query heads to a KV head
        {"name": "prefill-70b", "kind": "prefill", "shape": "70b", "layers": 1, "rows": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rows", "rows", "prefill", "prefill", "prefill", "generate"])
    if kind == "generate":
        shape = rng.choice(["tiny", "7b"])
        layers = 4 if shape == "tiny" else rng.randint(1, 2)
        temp = rng.choice([0.0, 0.6])
        skip = "".join(rng.choice("01") for _ in range(2 * layers)) if shape == "7b" or rng.random() < 0.5 else ""
        return {"kind": kind, "shape": shape, "layers": layers, "prompt": _log_int(rng, 8, 600), "new": rng.randint(8, 32),
                "draft": rng.randint(0, 8), "temp": temp, "skip": skip}
    shape = rng.choice(["tiny", "7b", "13b", "70b"])
    layers = {"tiny": rng.randint(1, 4), "7b": rng.randint(1, 2), "13b": 1, "70b": 1}[shape]
    if kind == "rows":
        rows = rng.randint(1, 16)
        skip = "".join(rng.choice("0001") for _ in range(2 * layers)) if rows == 1 and layers > 1 else ""
        return {"kind": kind, "shape": shape, "layers": layers, "rows": rows, "ctx": _log_int(rng, 16, MOST_CTX[shape] - 16), "skip": skip}
    most = {"tiny": 2048, "7b": 8192, "13b": 6000, "70b": 2048}[shape]
    return {"kind": kind, "shape": shape, "layers": layers, "rows": _log_int(rng, 17, most)}


# ------------------------------------------------------------------------------------------------ inputs
def _shape(case):
    return si.SHAPES[case["shape"]].with_(n_layers=case["layers"])


def _weight(s, seed, tensor, layer):
    """One tensor on the GPU in its storage type (fp32 gains)."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed((seed * 1000003 + layer * 101 + tensor) % (1 << 62))
    size = si.tensor_shape(s, tensor)
    z = torch.randn(size, generator=g, device=DEVICE, dtype=torch.float32)
    if tensor in si.NORM_TENSORS:
        return 1.0 + 0.1 * z
    z *= 0.02 / 8 if tensor in (si.T_WO, si.T_WD) else 0.02
    return z.bfloat16() if s.dtype == si.DT_BF16 else z


def _tokens(s, seed, n):
    return np.random.default_rng(seed).integers(0, s.vocab, n, dtype=np.int32)


def _skip(case):
    """The skip mask of a case's text, one digit for each sublayer, 1 = left out; None where nothing is."""
    return np.array([int(c) for c in case["skip"]], np.uint8) if "1" in case.get("skip", "") else None


def _engine(case, seed, max_seq):
    s = _shape(case)
    eng = asd.Engine(asd.make_config(s, max_seq, page_tokens=PAGE[case["shape"]]), DEVICE)
    todo = [(t, 0) for t in si.GLOBAL_TENSORS] + [(t, l) for l in range(s.n_layers) for t in si.LAYER_TENSORS]
    for t, l in todo:
        w = _weight(s, seed, t, l)
        torch.cuda.synchronize()              # the engine copies on a stream of its own
        eng._ck(asd.lib().asd_set_weight(eng._h, t, l, w.data_ptr(), w.numel() * w.element_size(), 1))
    return s, eng


def prepare(case, seed):
    st = {"case": case}
    if case["kind"] == "rows":
        n, ctx = case["rows"], case["ctx"]
        s, eng = _engine(case, seed, ctx + n)
        toks = _tokens(s, seed, ctx + n)
        eng.prefill(toks[:ctx])
        st.update(tokens=torch.from_numpy(toks[ctx:].copy()).to(DEVICE), skip=_skip(case),
                  logits=torch.empty((n, s.vocab), dtype=torch.float32, device=DEVICE),
                  cos=torch.empty(2 * s.n_layers, dtype=torch.float32, device=DEVICE),
                  argmax=torch.empty(n, dtype=torch.int32, device=DEVICE))
    elif case["kind"] == "prefill":
        s, eng = _engine(case, seed, case["rows"] + 64)
        st["prompt"] = _tokens(s, seed, case["rows"])
    else:
        s, eng = _engine(case, seed, case["prompt"] + case["new"] + case["draft"] + 1)
        st["prompt"] = _tokens(s, seed, case["prompt"])
        st["options"] = dict(alpha=0.985, m=2, n=1) if _skip(case) is None else dict(fixed_mask=_skip(case))
        if case["temp"] > 0:
            st["options"].update(temperature=case["temp"], seed=seed)
    st["engine"] = eng
    torch.cuda.synchronize()
    return st


def run(st):
    case, eng = st["case"], st["engine"]
    if case["kind"] == "rows":
        # The scratch of forward_noalloc is one array per GPU: the program orders its calls, on whichever engine, behind
        # one another through its own stream.
        mine = torch.cuda.current_stream()
        eng.stream.wait_stream(mine)
        eng.forward_noalloc(st["tokens"], case["ctx"], st["skip"], False, st["logits"], st["cos"], st["argmax"])
        mine.wait_stream(eng.stream)
        return {"logits": st["logits"], "cos": st["cos"], "argmax": st["argmax"]}
    if case["kind"] == "prefill":
        first, cos, logits = eng.prefill(st["prompt"], want_logits=True)
        return {"first": first, "cos": cos, "logits": logits}
    tokens, stats, mask = eng.generate(st["prompt"], case["new"], case["draft"], **st["options"])
    last = eng.forward(tokens[-1:], eng.kv_len, commit=False)
    return {"tokens": tokens, "mask": mask, "accepted": stats["accepted"], "logits": last["logits"], "cos": last["cos"]}


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _params(s, skip=None):
    """Weights of the kept sublayers."""
    att = s.d_model * (2 * s.q_dim + 2 * s.kv_dim)
    mlp = 3 * s.d_model * s.d_ffn
    kept = skip if skip is not None else np.zeros(2 * s.n_layers, np.uint8)
    return int((1 - kept[0::2]).sum()) * att + int((1 - kept[1::2]).sum()) * mlp


def _pass_work(s, rows, ctx, skip=None, logit_rows=None):
    """Bytes and multiply-adds x 2 of a pass of `rows` rows over `ctx` cached positions."""
    es = 2 if s.dtype == si.DT_BF16 else 4
    lr = rows if logit_rows is None else logit_rows
    att = s.n_layers if skip is None else int((1 - skip[0::2]).sum())
    head = s.vocab * s.d_model
    by = es * (_params(s, skip) + head + rows * s.d_model) + es * att * 2 * s.kv_dim * (ctx + rows) + 4 * lr * s.vocab
    fl = 2.0 * rows * _params(s, skip) + 2.0 * lr * head + 4.0 * att * s.q_dim * rows * (ctx + 0.5 * (rows + 1))
    return np.array([by, fl], np.float64)


def work(case):
    s = _shape(case)
    if case["kind"] == "rows":
        w = _pass_work(s, case["rows"], case["ctx"], _skip(case))
    elif case["kind"] == "prefill":
        w = _pass_work(s, case["rows"], 0, None, 1)
    else:
        # the prompt pass, then the fewest cycles: every draft kept (Algorithm 1's mask is known for its fixed rule only)
        p, n, k = case["prompt"], case["new"], case["draft"]
        skip = _skip(case)
        if skip is None:
            skip = asd.admg(np.zeros(s.n_layers, np.float32), 0.985, 2, 1)
        w, done = _pass_work(s, p, 0, None, 1), 1
        while done < n:
            kk = min(k, n - done - 1)
            for j in range(kk):
                w = w + _pass_work(s, 1, p + done - 1 + j, skip)
            w = w + _pass_work(s, kk + 1, p + done - 1)
            done += kk + 1
        w = w + _pass_work(s, 1, p + n - 1)
    return {"bytes": float(w[0]), "flops": float(w[1])}


def tolerance(case):
    # Sums are fp32 on both storage types and bf16 models take activations as two bf16 values (16 mantissa bits); what
    # two correct implementations differ by is mostly K and V values that fall on the other side of a bf16 rounding
    # boundary, and, over the layers of a whole model, what those cause.  Measured against `exact`: 2e-7 (fp32), 1e-4 .. 5e-4
    # (one or two bf16 layers), 2e-3 (32 layers); about four times that, and 1e-5 for 32-bit sums in another order.
    if case["shape"] == "tiny":
        return {"rel": 1e-5}
    return {"rel": 1e-2 if case["layers"] > 2 else 2e-3}


# ------------------------------------------------------------------------------------------------ in 64 bits
def _rope(x, pos, theta):
    """x [n, heads, h], dims (i, i + h/2) rotated by pos * theta^(-2i/h)."""
    h = x.shape[-1]
    i = torch.arange(h // 2, device=x.device, dtype=torch.float64)
    ang = pos.double()[:, None] * (theta ** (-2.0 * i / h))[None, :]
    c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., : h // 2], x[..., h // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attention(q, k, v, pos):
    """Causal attention of rows at positions `pos` over keys 0, 1, ...: q [n, heads, h], k and v [m, kv heads, h]."""
    n, heads, h = q.shape
    out = torch.empty_like(q)
    group = heads // k.shape[1]
    keys = torch.arange(k.shape[0], device=q.device)
    for i in range(heads):
        ki, vi = k[:, i // group], v[:, i // group]
        for r0 in range(0, n, 2048):
            sc = q[r0:r0 + 2048, i] @ ki.T / math.sqrt(h)
            sc.masked_fill_(keys[None, :] > pos[r0:r0 + 2048, None], -math.inf)
            out[r0:r0 + 2048, i] = torch.softmax(sc, -1) @ vi
    return out


def exact(case, seed):
    """The decoder in 64 bits; K and V are rounded to the storage type as they enter the cache (the cache's type belongs to
    the model).  None for the generating loop, whose tokens are decisions."""
    if case["kind"] == "generate":
        return None
    s = _shape(case)
    rows = case["rows"]
    ctx = case.get("ctx", 0)
    toks = torch.from_numpy(_tokens(s, seed, ctx + rows)).to(DEVICE).long()
    stored = torch.bfloat16 if s.dtype == si.DT_BF16 else torch.float32
    W = lambda t, l=0: _weight(s, seed, t, l).double()                                       # noqa: E731
    norm = lambda x, g: x * torch.rsqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * g      # noqa: E731
    keep = lambda x: x.float().to(stored).double()                                           # noqa: E731

    def cosine(x, y):
        return ((x * y).sum(-1) * torch.rsqrt((x * x).sum(-1).clamp_min(1e-16) * (y * y).sum(-1).clamp_min(1e-16))).clamp(-1, 1)

    skip = _skip(case)
    # the cached positions went through the full model, the rows of the pass through the masked one
    pos_all = torch.arange(ctx + rows, device=DEVICE)
    x = W(si.T_EMBED)[toks]
    cos = np.ones(2 * s.n_layers)
    for l in range(s.n_layers):
        for half in (0, 1):
            left = skip is not None and skip[2 * l + half] == 1
            if left and not ctx:
                continue
            if half == 0:
                nx = norm(x, W(si.T_ATTN_NORM, l))
                q = _rope((nx @ W(si.T_WQ, l).T).view(-1, s.n_heads, s.head_dim), pos_all, s.rope_theta)
                k = keep(_rope((nx @ W(si.T_WK, l).T).view(-1, s.n_kv_heads, s.head_dim), pos_all, s.rope_theta))
                v = keep((nx @ W(si.T_WV, l).T).view(-1, s.n_kv_heads, s.head_dim))
                d = _attention(q, k, v, pos_all).reshape(-1, s.q_dim) @ W(si.T_WO, l).T
            else:
                nx = norm(x, W(si.T_MLP_NORM, l))
                d = (torch.nn.functional.silu(nx @ W(si.T_WG, l).T) * (nx @ W(si.T_WU, l).T)) @ W(si.T_WD, l).T
            if left:
                d[ctx:] = 0.0
            y = x + d
            if not left:
                cos[2 * l + half] = cosine(x[ctx:], y[ctx:]).mean().item()
            x = y
    last = x[ctx:] if case["kind"] == "rows" else x[-1:]
    logits = norm(last, W(si.T_FINAL_NORM)) @ W(si.T_LM_HEAD).T
    if case["kind"] == "rows":
        return {"logits": logits, "cos": torch.from_numpy(cos), "argmax": None}
    return {"first": None, "cos": cos, "logits": logits[0]}
