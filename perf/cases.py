"""Workloads of the SwiftKV prefill library, as its callers run them.

Most cases are a shortened stack: the first layers of a decoder of full width
(every matrix, head and ffn size as in the whole model, only fewer layers and a
vocabulary shortened in the same proportion), called once through
`Context.prefill` with the batches a serving engine forms: decode steps, single
prompts, chunks of a prompt over its cached prefix (alone or next to decode
tokens), packed prompts.  One case is a whole small model.  The fused K/V
projection and the prefill attention are also called by themselves.

A case is a dict of plain values:
  kind    "stack" (Context.prefill), "kv" (Context.kv_from_hidden) or
          "attention" (op_attention_prefill)
  width   key of WIDTHS
  layers, full, group   decoder layers, layers every token runs, AcrossKV group
  batch   "[count x]new[@cached]" items; cached "a-b" spreads the count over a..b
  cache   "bf16", "fp8" (one scale per head, computed by the call), "fp8_given"
          (one scale per head, kept) or "fp8_token" (one scale per token)
"""
import math

import torch

from paper_2410_03960_amd import binding as B
from workloads import ModelShape

BLOCK = 16
# hidden, query heads, KV heads, head dim, ffn, vocabulary of a stack
WIDTHS = {
    "8b": (4096, 32, 8, 128, 14336, 8192),
    "70b": (8192, 64, 8, 128, 28672, 8192),
    "small": (2048, 32, 8, 64, 8192, 32000),
}


def listed():
    return [
        # the smallest call: one sequence, one new token (interactive decoding; latency and launches)
        {"name": "decode_1", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 1, "batch": "1@777", "cache": "bf16"},
        # a small decode batch of the large model, contexts of mixed length
        {"name": "decode_24_70b", "kind": "stack", "width": "70b", "layers": 2, "full": 1, "group": 1, "batch": "24x1@200-4100", "cache": "bf16"},
        # the decode step of the benchmark's own decode workload: 64 sequences over 2048 cached tokens
        {"name": "decode_64", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 1, "batch": "64x1@2048", "cache": "bf16"},
        # a loaded server's decode step: 160 sequences of mixed length over an FP8 cache with fixed scales
        {"name": "decode_160_fp8", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 2, "batch": "160x1@300-1500", "cache": "fp8_given"},
        # one short chat prompt, of no round length
        {"name": "prompt_333", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 1, "batch": "333", "cache": "bf16"},
        # a continuous-batching step with a budget of 512 tokens: a chunk of one prompt next to 38 decode tokens
        {"name": "mixed_512_fp8", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 1, "batch": "474@1536 38x1@100-2000",
         "cache": "fp8_token"},
        # the last 2048-token chunk of one 8192-token prompt
        {"name": "chunk_2048", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 1, "batch": "2048@6144", "cache": "bf16"},
        # packed prompts of mixed length, FP8 cache, two layers sharing each later cache layer
        {"name": "varlen_fp8", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 2, "batch": "3017 1801 1204 935 711 640 523",
         "cache": "fp8"},
        # the benchmark's batch: 8 prompts of 2048 tokens
        {"name": "prefill_8x2048", "kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": 1, "batch": "8x2048", "cache": "bf16"},
        # a whole small model (16 layers, 64-wide heads) over a few prompts
        {"name": "small_model", "kind": "stack", "width": "small", "layers": 16, "full": 8, "group": 1, "batch": "211 160 127 99", "cache": "bf16"},
        # the fused K/V projection of 16 later layers by itself, from a given layer output
        {"name": "later_kv_1500", "kind": "kv", "width": "8b", "layers": 17, "full": 1, "group": 1, "batch": "1021 479", "cache": "bf16"},
        # causal grouped-query attention by itself over ragged prompts
        {"name": "attention_ragged", "kind": "attention", "width": "8b", "layers": 1, "full": 1, "group": 1, "batch": "3001 1537 800 257 64 7",
         "cache": "bf16"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more call of the ranges above: 1..16384 new tokens, up to 8192 cached ones per sequence."""
    what = rng.choice(["decode", "decode", "chunk", "chunk", "prompts", "prompts", "kv", "attention"])
    case = {"kind": "stack", "width": "8b", "layers": 4, "full": 2, "group": rng.choice([1, 1, 2]), "batch": "", "cache": "bf16"}
    if what == "decode":
        n = _log(rng, 1, 256)
        case["width"] = rng.choice(["8b", "8b", "8b", "small", "70b" if n <= 64 else "8b"])
        lo = _log(rng, 32, 1000)
        hi = min(lo + _log(rng, 64, 6000), 400000 // n)
        case["batch"] = "%dx1@%d-%d" % (n, min(lo, hi), hi)
        case["cache"] = rng.choice(["bf16", "bf16", "fp8_given", "fp8_token"])
    elif what == "chunk":   # a chunk of a prompt, perhaps with decode tokens of other sequences beside it
        items = ["%d@%d" % (_log(rng, 60, 4096), _log(rng, 100, 6144))]
        n = rng.choice([0, _log(rng, 1, 96)])
        if n:
            items.append("%dx1@%d-%d" % (n, 50, _log(rng, 200, 3000)))
        case["batch"] = " ".join(items)
        case["width"] = rng.choice(["8b", "8b", "8b", "small"])
        case["cache"] = rng.choice(["bf16", "bf16", "fp8_given", "fp8_token"])
    elif what == "prompts":
        left, items = 14000, []
        for _ in range(_log(rng, 1, 16)):
            n = min(left, _log(rng, 16, 4096))
            if n < 16:
                break
            items.append(str(n))
            left -= n
        case["batch"] = " ".join(items)
        case["width"] = rng.choice(["8b", "8b", "8b", "small"])
        case["cache"] = rng.choice(["bf16", "bf16", "fp8", "fp8_token"])
    elif what == "kv":
        case.update(kind="kv", layers=17, full=1, group=rng.choice([1, 2]), batch=" ".join(str(_log(rng, 40, 4096)) for _ in range(rng.choice([1, 2, 3]))),
                    cache=rng.choice(["bf16", "bf16", "fp8"]))
    else:
        case.update(kind="attention", layers=1, full=1, group=1, width=rng.choice(["8b", "8b", "70b", "small"]),
                    batch=" ".join(str(_log(rng, 16, 4096)) for _ in range(rng.choice([1, 2, 4, 6]))))
    if case["width"] == "small" and case["kind"] == "stack":
        case.update(layers=16, full=8, group=rng.choice([1, 2]))
    if case["width"] == "70b" and case["kind"] == "stack":
        case.update(layers=2, full=1, group=1)
    return case


# ------------------------------------------------------------------ inputs ----
def _batch(case):
    """(new tokens, cached tokens) of every sequence."""
    new, ctx = [], []
    for item in case["batch"].split():
        item, _, cached = item.partition("@")
        count, _, n = item.rpartition("x")
        count, n = int(count or 1), int(n)
        lo, _, hi = (cached or "0").partition("-")
        lo, hi = int(lo), int(hi or lo)
        for i in range(count):
            new.append(n)
            ctx.append(lo + int((hi - lo) * ((i * 0.6180339887) % 1.0)))
    return new, ctx


def _shape(case):
    d, hq, hkv, hd, f, v = WIDTHS[case["width"]]
    return ModelShape(case["layers"], d, hq, hkv, hd, f, v, 5e5, 1e-5)


def _normal(gen, shape, std, mean=0.0):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(mean, std, generator=gen)


def _model(case, gen):
    """Random bf16 weights; the projections back into the residual stream are scaled by 1/sqrt(2 layers), as initialised for training."""
    sh = _shape(case)
    d, q, k, f = sh.hidden, sh.q_dim, sh.kv_dim, sh.ffn
    out = 0.02 / math.sqrt(2 * sh.n_layers)
    w = {"embed": _normal(gen, (sh.vocab, d), 1.0), "final_norm": _normal(gen, (d,), 0.02, 1.0), "lm_head": _normal(gen, (sh.vocab, d), 0.02)}
    for j in range(sh.n_layers):
        w["norm1.%d" % j] = _normal(gen, (d,), 0.02, 1.0)
        w["wk.%d" % j], w["wv.%d" % j] = _normal(gen, (k, d), 0.02), _normal(gen, (k, d), 0.02)
        if case["kind"] == "kv" and j > 0:   # the fused projection reads nothing else of these layers
            for n in ("norm2", "wq", "wo", "wgate", "wup", "wdown"):
                w["%s.%d" % (n, j)] = w[n + ".0"]
            continue
        w["norm2.%d" % j] = _normal(gen, (d,), 0.02, 1.0)
        w["wq.%d" % j], w["wo.%d" % j] = _normal(gen, (q, d), 0.02), _normal(gen, (d, q), out)
        w["wgate.%d" % j], w["wup.%d" % j], w["wdown.%d" % j] = _normal(gen, (f, d), 0.02), _normal(gen, (f, d), 0.02), _normal(gen, (d, f), out)
    return sh, w


def _pool(case, sh, new, ctx, gen, seed):
    """Shuffled block tables and the paged cache as earlier calls left it."""
    need = [(c + n + BLOCK - 1) // BLOCK for c, n in zip(ctx, new)]
    n_blocks = sum(need) + (sum(need) + 9) // 10
    order = torch.randperm(n_blocks, generator=torch.Generator().manual_seed(seed)).to(torch.int32)
    tables = torch.zeros((len(new), max(need)), dtype=torch.int32)
    at = 0
    for b, n in enumerate(need):
        tables[b, :n] = order[at:at + n]
        at += n
    layers = sh.n_layers if case["kind"] == "attention" else case["full"] + (case["layers"] - case["full"]) // case["group"]
    mode = {"bf16": 0, "fp8": B.SWIFTKV_SCALE_COMPUTE_ABSMAX, "fp8_given": B.SWIFTKV_SCALE_USE_GIVEN, "fp8_token": B.SWIFTKV_SCALE_PER_TOKEN}[case["cache"]]
    kv = B.KVCache(layers, n_blocks, sh.n_kv_heads, sh.head_dim, tables, ctx, fp8=case["cache"] != "bf16", scale_mode=mode)
    if any(ctx) or case["cache"] == "fp8_given":
        rows = 0.02 * math.sqrt(sh.hidden)   # the size K and V rows have on these weights
        for c in range(layers):
            for t in range(2):
                x = _normal(gen, kv.data.shape[2:], rows)
                if case["cache"] == "fp8_token":
                    kv.scales[c, t] = x.float().abs().amax(dim=(1, 2)) / 448.0
                    kv.data[c, t] = (x.float() / kv.scales[c, t][:, None, None]).to(torch.float8_e4m3fn).view(torch.uint8)
                elif case["cache"] == "fp8_given":
                    kv.scales[c, t].uniform_(4.5 * rows / 448, 6.0 * rows / 448, generator=gen)
                    kv.data[c, t] = (x.float() / kv.scales[c, t][None, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
                else:
                    kv.data[c, t] = x
    return tables, kv


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    new, ctx = _batch(case)
    T, s = sum(new), {"case": case, "new": new, "ctx": ctx}
    if case["kind"] == "attention":
        sh = s["shape"] = _shape(case)
        s["q"], s["k"], s["v"] = (_normal(gen, (T, n), 1.3) for n in (sh.q_dim, sh.kv_dim, sh.kv_dim))
        return s
    sh, s["w"] = _model(case, gen)
    s["shape"] = sh
    s["tables"], s["kv"] = _pool(case, sh, new, ctx, gen, seed)
    if case["kind"] == "kv":
        s["hidden"] = _normal(gen, (T, sh.hidden), 1.0)
    else:
        s["ids"] = torch.randint(0, sh.vocab, (T,), generator=gen, device="cuda", dtype=torch.int32)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "attention":
        return s
    sh, new, ctx = s["shape"], s["new"], s["ctx"]
    s["ctx_handle"] = h = B.Context(sh, s["w"], case["full"], case["group"])
    prefix = sum(c for c, n in zip(ctx, new) if n > 1)
    dtype = B.SWIFTKV_KV_BF16 if case["cache"] == "bf16" else B.SWIFTKV_KV_FP8_E4M3
    s["ws"] = torch.empty(h.workspace_bytes(sum(new), len(new), dtype, prefix), dtype=torch.uint8, device="cuda")
    s["logits"] = torch.empty((len(new), sh.vocab), dtype=torch.float32, device="cuda")
    return s


def run(s):
    sh, kind = s["shape"], s["case"]["kind"]
    if kind == "attention":
        return {"out": B.op_attention_prefill(s["q"], s["k"], s["v"], s["new"], sh.n_q_heads, sh.n_kv_heads, sh.head_dim)}
    kv = s["kv"]
    out = {"cache": kv.data}
    if kind == "kv":
        s["ctx_handle"].kv_from_hidden(s["hidden"], s["new"], kv, s["ws"])
        if kv.fp8:   # (this call fills the later layers' part)
            out["scales"] = kv.scales
    else:
        s["ctx_handle"].prefill(s["ids"], s["new"], kv, s["logits"], s["ws"])
        out["logits"] = s["logits"]
        if kv.fp8:
            out["scales"] = kv.scales
    if kv.fp8:
        out["cache"] = kv.data.view(torch.float8_e4m3fn)
    return out


# ----------------------------------------------------- what a pass has to do ----
def work(case):
    sh = _shape(case)
    new, ctx = _batch(case)
    T, n_seq = sum(new), len(new)
    d, q, k, f, v = sh.hidden, sh.q_dim, sh.kv_dim, sh.ffn, sh.vocab
    l, later = case["full"], case["layers"] - case["full"]
    P = later // case["group"]
    pairs = sum(n * c + n * (n + 1) // 2 for n, c in zip(new, ctx))
    if case["kind"] == "attention":
        return {"bytes": 2.0 * T * (2 * q + 2 * k), "flops": 4.0 * q * pairs}
    e = 2 if case["cache"] == "bf16" else 1
    if case["kind"] == "kv":
        return {"bytes": 2.0 * P * 2 * k * d + 2.0 * T * d + e * 2.0 * P * T * k, "flops": 2.0 * T * d * P * 2 * k}
    tail = 2.0 * d * q + 3.0 * d * f                     # weights of a later layer that its rows read
    params = l * (tail + 2.0 * d * k) + P * 2.0 * d * k + later * tail + d * v + min(T, v) * d
    keys = sum(n + c for n, c in zip(new, ctx))
    cached = sum(ctx)
    kv_bytes = e * 2.0 * k * (l * cached + later * keys + (l + P) * T)   # full layers read the cached rows, later ones all, each new row is written
    flops = T * (l * (2.0 * tail + 4.0 * d * k) + P * 4.0 * d * k) + n_seq * (later * 2.0 * tail + 2.0 * d * v)
    flops += 4.0 * q * (l * pairs + later * keys)
    return {"bytes": 2.0 * params + kv_bytes + 4.0 * n_seq * v, "flops": flops}


def tolerance(case):
    # measured as the distance of the outputs from 64 bits, about four times that (bf16 operands of every product;
    # an e4m3 code moves by up to 1/8 of its value where its input crosses a rounding boundary)
    if case["kind"] == "attention":
        return {"rel": 0.01}
    if case["kind"] == "kv":
        return {"rel": 0.01 if case["cache"] == "bf16" else 0.03, "max": 0.4}
    if case["width"] == "small":
        return {"rel": 0.015 if case["cache"] == "bf16" else 0.03, "max": 0.6}
    return {"rel": 0.02 if case["cache"] == "bf16" else 0.03, "max": 0.6}


# ------------------------------------------------------------- 64-bit result ----
def _rms(x, gain):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5) * gain


def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * theta ** (-torch.arange(half, dtype=torch.float64, device=x.device) * 2.0 / x.shape[-1])
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(q, q_pos, k, v):
    """q [n, Hq, hd] at positions q_pos over k, v [keys, Hkv, hd]."""
    n, hq, hd = q.shape
    r = hq // k.shape[1]
    out = torch.empty_like(q)
    hidden = torch.arange(k.shape[0], device=q.device)[None, :] > q_pos[:, None]
    for h in range(hq):
        s = q[:, h] @ k[:, h // r].T.contiguous() / math.sqrt(hd)
        out[:, h] = torch.softmax(s.masked_fill_(hidden, -math.inf), -1) @ v[:, h // r].contiguous()
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    sh, new, ctx = s["shape"], s["new"], s["ctx"]
    hq, hkv, hd, theta = sh.n_q_heads, sh.n_kv_heads, sh.head_dim, float(torch.tensor(sh.rope_theta, dtype=torch.float32))
    starts = [sum(new[:b]) for b in range(len(new))]
    T = sum(new)
    pos = torch.cat([torch.arange(c, c + n) for n, c in zip(new, ctx)]).cuda()
    if case["kind"] == "attention":
        q, k, v = (s[n].double().view(T, -1, hd) for n in "qkv")
        return {"out": torch.cat([_attend(q[a:a + n], pos[a:a + n], k[a:a + n], v[a:a + n]) for a, n in zip(starts, new)]).view(T, -1)}
    w, kv, fp8 = s["w"], s["kv"], case["cache"]
    all_slots = [(s["tables"][b].long()[:, None] * BLOCK + torch.arange(BLOCK)).view(-1)[:n + c].cuda() for b, (n, c) in enumerate(zip(new, ctx))]
    slots = torch.cat([a[c:] for a, c in zip(all_slots, ctx)])
    W = lambda name, j: w["%s.%d" % (name, j)].double()  # noqa: E731
    data = kv.data.double() if fp8 == "bf16" else kv.data.view(torch.float8_e4m3fn).double()
    scales = None if fp8 == "bf16" else kv.scales.clone()

    def factor(c, t):   # of the stored values, shaped to multiply [slots, heads, dims]
        return scales[c, t].double()[:, None, None] if fp8 == "fp8_token" else scales[c, t].double()[None, :, None]

    def store(c, j, h):
        a = _rms(h, W("norm1", j))
        for t, x in enumerate((_rope((a @ W("wk", j).T).view(T, hkv, hd), pos, theta), (a @ W("wv", j).T).view(T, hkv, hd))):
            if fp8 == "bf16":
                data[c, t, slots] = x
                continue
            x = x.float()
            if fp8 == "fp8":
                scales[c, t] = x.abs().amax(dim=(0, 2)) / 448.0
            elif fp8 == "fp8_token":
                scales[c, t, slots] = x.abs().amax(dim=(1, 2)) / 448.0
            sc = scales[c, t, slots][:, None, None] if fp8 == "fp8_token" else scales[c, t][None, :, None]
            data[c, t, slots] = (x / sc).clamp(-448, 448).to(torch.float8_e4m3fn).double()

    def layer(c, j, h, rows):
        """The rest of layer j for the rows (per sequence) over cache layer c."""
        a = _rms(h, W("norm1", j))
        p = torch.cat([pos[starts[b]:][r] for b, r in enumerate(rows)])
        q = _rope((a @ W("wq", j).T).view(-1, hq, hd), p, theta)
        o, at = torch.empty_like(q), 0
        for b, r in enumerate(rows):
            n = len(range(*r.indices(new[b])))
            k, v = data[c, 0, all_slots[b]], data[c, 1, all_slots[b]]
            if fp8 != "bf16":
                fk, fv = factor(c, 0), factor(c, 1)
                k, v = (k * fk[all_slots[b]], v * fv[all_slots[b]]) if fp8 == "fp8_token" else (k * fk, v * fv)
            o[at:at + n] = _attend(q[at:at + n], p[at:at + n], k, v)
            at += n
        h = h + o.view(-1, hq * hd) @ W("wo", j).T
        m = _rms(h, W("norm2", j))
        gate = m @ W("wgate", j).T
        return h + (gate * torch.sigmoid(gate) * (m @ W("wup", j).T)) @ W("wdown", j).T

    if case["kind"] == "kv":
        h = s["hidden"].double()
    else:
        h = w["embed"].double()[s["ids"].long()]
        for j in range(case["full"]):
            store(j, j, h)
            h = layer(j, j, h, [slice(0, n) for n in new])
    for p in range((case["layers"] - case["full"]) // case["group"]):
        store(case["full"] + p, case["full"] + p * case["group"], h)
    out = {"cache": data}
    if scales is not None:
        out["scales"] = scales.double()
    if case["kind"] == "stack":
        last = torch.tensor([a + n - 1 for a, n in zip(starts, new)], device="cuda")
        h = h[last]
        for j in range(case["full"], case["layers"]):
            h = layer(case["full"] + (j - case["full"]) // case["group"], j, h, [slice(n - 1, n) for n in new])
        out["logits"] = _rms(h, w["final_norm"].double()) @ w["lm_head"].double().T
    return out
