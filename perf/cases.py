"""Performance cases of the pipeline stage, through its public entry points.

Each case is one call (or the short sequence of calls) that a program serving a
model makes once per token, per prompt chunk or per cache hand-over: decode
steps with and without the head, prefill chunks, prompt scoring and cache
restore.  Stages hold one or two layers of a named shape: a stage's step is the
same launches per layer however many layers it holds.

A case is a dict of plain values; ``kind`` says which call it times:
  decode   one step for ``batch`` users at contexts ``ctx`` (comma-separated), hidden rows in and out, or
           with ``head`` token ids in and logits out (the output rows stay in the stage for the head)
  prefill  a chunk of ``n`` tokens at position ``pos0``
  logits   the unembedding of ``rows`` hidden rows
  cache    ``n`` saved positions written into a user's cache and read back
"""
import math

import torch

import synth
from paper_2609_34045_amd import stage as kf

SHAPES = {
    "tiny": synth.SHAPE_TINY,
    "qwen3_tiny": synth.SHAPE_QWEN3_TINY,
    "8b": synth.SHAPE_8B,
    "qwen3_8b": synth.SHAPE_QWEN3_8B,
    "32b": synth.SHAPE_32B,
    "qwen3_32b": synth.SHAPE_QWEN3_32B,
    "70b": synth.SHAPE_70B,
}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
MAX_CTX = 32768


def _decode(name, shape, ctx, layers=1, io="f32", paged=False, ordered=False, head=False):
    return {"name": name, "kind": "decode", "shape": shape, "layers": layers, "ctx": ctx, "io": io, "paged": paged,
            "ordered": ordered, "head": head}


def _prefill(name, shape, n, pos0, layers=1, io="f32", paged=False):
    return {"name": name, "kind": "prefill", "shape": shape, "layers": layers, "n": n, "pos0": pos0, "io": io,
            "paged": paged}


def listed():
    return [
        # a whole small model on one member, one user: the latency of a token, launches and little else
        _decode("decode_tiny_head_b1", "tiny", "128", layers=2, head=True),
        # a middle member of an 8B ring, one user: the token rate of the paper's single-request runs
        _decode("decode_8b_b1", "8b", "2048", layers=2),
        # the head member of an 8B ring with four users of different lengths, embedding to logits
        _decode("decode_8b_head_b4", "8b", "256,1024,2048,4096", head=True),
        # a middle member of a 32B ring serving four users together
        _decode("decode_32b_b4", "32b", "4096,4096,4096,4096", io="bf16"),
        # one user deep into a long conversation, paged cache, reproducible sums, per-head q/k norms
        _decode("decode_qwen3_32b_b1_long", "qwen3_32b", "30001", paged=True, ordered=True),
        # a short chat prompt: time to first token of an ordinary request
        _prefill("prefill_qwen3_8b_37", "qwen3_8b", 37, 0, layers=2, io="bf16"),
        # a follow-up message into a conversation: the last, ragged chunk of a prompt
        _prefill("prefill_8b_200_at_1000", "8b", 200, 1000),
        # a short follow-up deep into a long conversation: attention over the cache outweighs the chunk
        _prefill("prefill_8b_64_at_30000", "8b", 64, 30000, paged=True),
        # the chunk size a large model's prompt is cut into, near the end of a 4096-token context
        _prefill("prefill_70b_512_at_3584", "70b", 512, 3584),
        # a long document in one chunk
        _prefill("prefill_32b_2048", "32b", 2048, 0),
        # scoring a prompt: logits of every position of a 256-token chunk
        {"name": "logits_8b_256", "kind": "logits", "shape": "8b", "rows": 256, "io": "f32"},
        # restoring a saved prefix of 4096 positions into a user's cache, and saving it back
        {"name": "cache_8b_4096", "kind": "cache", "shape": "8b", "n": 4096, "pos0": 0, "io": "f16", "paged": True},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def _seconds(case):
    """A rough time of a case's work, to keep drawn cases below the largest listed one."""
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / 0.8e15


def draw(rng):
    most = max(_seconds(c) for c in listed())
    while True:
        c = _draw(rng)
        if _seconds(c) <= most:
            return c


def _draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "logits", "cache"])
    flag = lambda: rng.random() < 0.5  # noqa: E731
    if kind == "decode":
        head = rng.random() < 0.3
        shape = rng.choice(["tiny", "qwen3_tiny", "8b"]) if head else rng.choice(sorted(SHAPES))
        ctx = ",".join(str(_log_int(rng, 1, MAX_CTX - 64)) for _ in range(rng.randint(1, 4)))
        c = _decode("", shape, ctx, rng.randint(1, 2), rng.choice(["f32", "bf16"]), flag(), flag(), head)
    elif kind == "prefill":
        n = _log_int(rng, 1, 2048)
        pos0 = 0 if rng.random() < 0.3 else _log_int(rng, 1, MAX_CTX - 64 - n)
        c = _prefill("", rng.choice(sorted(SHAPES)), n, pos0, 1, rng.choice(["f32", "bf16"]), flag())
    elif kind == "logits":
        c = {"kind": kind, "shape": rng.choice(["tiny", "qwen3_tiny", "8b"]), "rows": _log_int(rng, 1, 512),
             "io": rng.choice(["f32", "bf16"])}
    else:
        n = _log_int(rng, 1, 16384)
        c = {"kind": kind, "shape": rng.choice(["tiny", "8b", "qwen3_32b"]), "n": n, "pos0": rng.randint(0, 1000),
             "io": rng.choice(["f32", "bf16", "f16"]), "paged": flag()}
    c.pop("name", None)
    return c


# ---------------------------------------------------------------- inputs


def _contexts(case):
    return [int(v) for v in case["ctx"].split(",")]


def _inputs(case, seed):
    """Every input of a case, on the GPU, from the seed alone: N(0, 0.02^2) projections, gains around 1,
    unit-variance hidden rows, keys and values at the scale such projections give them."""
    s = SHAPES[case["shape"]]
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(shape, mean=0.0, std=1.0, dtype=torch.bfloat16):
        v = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(mean, std, generator=g)
        return v.to(dtype)

    kind = case["kind"]
    layers = case.get("layers", 1)
    d = {"layers": [], "head": None, "kv": {}}
    if kind == "logits":
        layers = 1
        weights = dict(s.__dict__, ffn=64, n_q_heads=s.n_kv_heads)  # the layer beside the head is not used
        s = synth.ModelShape(**weights)
    d["shape"] = s
    for _ in range(layers):
        d["layers"].append({k: normal(s.tensor_shape(k), 1.0 if k in synth.GAIN_KINDS else 0.0, 0.02)
                            for k in s.layer_kinds()})
    if kind == "logits" or case.get("head"):
        d["head"] = {k: normal(s.tensor_shape(k), 1.0 if k in synth.GAIN_KINDS else 0.0, 0.02)
                     for k in synth.HEAD_KINDS}
    std = 0.02 * math.sqrt(s.hidden)
    if kind == "decode":
        d["ctx"] = _contexts(case)
        if case["head"]:
            d["tokens"] = torch.randint(0, s.vocab, (len(d["ctx"]),), generator=g, device="cuda").to(torch.int32)
        else:
            d["hidden"] = normal((len(d["ctx"]), s.hidden), dtype=DTYPES[case["io"]])
    elif kind == "prefill":
        d["ctx"] = [case["pos0"]]
        d["hidden"] = normal((case["n"], s.hidden), dtype=DTYPES[case["io"]])
    elif kind == "logits":
        d["ctx"] = []
        d["hidden"] = normal((case["rows"], s.hidden), dtype=DTYPES[case["io"]])
    else:
        d["ctx"] = []
        d["saved"] = [normal((case["n"], s.n_kv_heads, s.head_dim), 0.0, std, DTYPES[case["io"]]) for _ in range(2)]
    for l in range(layers):
        for u, n in enumerate(d["ctx"]):
            if n:
                d["kv"][l, u] = [normal((n, s.n_kv_heads, s.head_dim), 0.0, std) for _ in range(2)]
    return d


def _bits(tensors):
    return {k: v.view(torch.int16).cpu().numpy().view("uint16") for k, v in tensors.items()}


class _Held:
    """What a serving program holds: a stage, its cache and a call's input; closed when dropped."""

    def __init__(self, case, seed):
        d = _inputs(case, seed)
        s = d["shape"]
        layers = [_bits(w) for w in d["layers"]]
        self.case = case
        self.kv = None
        self.stage = kf.Stage(s, 0, len(layers), lambda l: layers[l], _bits(d["head"]) if d["head"] else None)
        if case.get("ordered"):
            self.stage.set_flags(kf.KF_STAGE_ORDERED)
        self.users = list(range(max(1, len(d["ctx"]))))
        self.ctx = d["ctx"]
        extra = {"decode": 1, "prefill": case.get("n", 0), "cache": case.get("n", 0) + case.get("pos0", 0)}
        if case["kind"] != "logits":
            max_ctx = max([n + extra[case["kind"]] for n in self.ctx] or [extra["cache"]])
            pages = None
            if case["paged"]:
                pages = len(self.users) * ((max_ctx + 63) // 64)
            self.kv = self.stage.kv(len(self.users), max_ctx, pages)
        for (l, u), (k, v) in d["kv"].items():
            self.kv.write(l, u, 0, k, v)
        for u, n in enumerate(self.ctx):
            self.kv.set_len(u, n)
        self.hidden, self.tokens, self.saved = d.get("hidden"), d.get("tokens"), d.get("saved")
        self.stage.sync()

    def __del__(self):
        if getattr(self, "kv", None) is not None:
            self.kv.close()
        if getattr(self, "stage", None) is not None:
            self.stage.close()


def prepare(case, seed):
    return _Held(case, seed)


def run(state):
    case, stage, kv = state.case, state.stage, state.kv
    kind = case["kind"]
    if kind == "logits":
        return stage.head_logits(state.hidden)
    if kind == "cache":
        kv.write(0, 0, case["pos0"], state.saved[0], state.saved[1])
        return kv.read(0, 0, case["pos0"], case["n"])
    for u, n in zip(state.users, state.ctx):  # the step or chunk is at this length again
        kv.set_len(u, n)
    if kind == "prefill":
        return stage.prefill(kv, 0, case["pos0"], hidden=state.hidden)
    if case["head"]:
        stage.decode(kv, state.users, state.ctx, tokens=state.tokens, keep=True)
        return stage.head_logits(None, rows=len(state.users))
    return stage.decode(kv, state.users, state.ctx, hidden=state.hidden)


# ---------------------------------------------------------------- what a pass cannot do without


def work(case):
    """Weights, cache and rows read once, results written once; a multiply and an add per product."""
    s = SHAPES[case["shape"]]
    io = 2 if case["io"] == "bf16" else 4
    kind = case["kind"]
    kv_row = 2 * s.n_kv_heads * s.head_dim  # values per position, keys and values
    head = 2 * s.vocab * s.hidden
    if kind == "logits":
        return {"bytes": head + case["rows"] * (s.hidden * io + s.vocab * 4), "flops": 2.0 * case["rows"] * s.vocab * s.hidden}
    if kind == "cache":
        return {"bytes": case["n"] * kv_row * ({"f32": 4, "bf16": 2, "f16": 2}[case["io"]] + 2 + 2 + 4), "flops": 0}
    layers = case["layers"]
    qw = s.n_q_heads * s.head_dim
    mats = (2 * qw + kv_row) * s.hidden + 3 * s.ffn * s.hidden
    if kind == "decode":
        ctx = _contexts(case)
        keys, rows = sum(n + 1 for n in ctx), len(ctx)
        read = keys * kv_row * 2
    else:
        rows = case["n"]
        keys = sum(range(case["pos0"] + 1, case["pos0"] + rows + 1))
        read = (case["pos0"] + rows) * kv_row * 2
    w = {"bytes": layers * (s.block_bytes() + read + rows * kv_row * 2),
         "flops": layers * (2.0 * rows * mats + 4.0 * qw * keys)}
    if case.get("head"):
        w["bytes"] += head + rows * (s.hidden * 2 + s.vocab * 4)
        w["flops"] += 2.0 * rows * s.vocab * s.hidden
    else:
        w["bytes"] += 2 * rows * s.hidden * io
    return w


def tolerance(case):
    """About four times the largest error against exact() over the listed and some forty drawn cases: weights rounded
    to fp16 with their norm's gain (2e-4 on logits), fp16 matrix operands (up to 1e-3 on hidden rows and on the logits
    of a step), bf16 rows out (1.8e-3)."""
    if case["kind"] == "cache":
        return "exact"
    if case["kind"] == "logits":
        return {"rel": 1e-3}
    return {"rel": 8e-3 if case["io"] == "bf16" and not case.get("head") else 4e-3}


# ---------------------------------------------------------------- the same in 64 bits


def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, theta):
    """Rotate-half over the last axis of [n, heads, hd] at positions [n]."""
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    a = (pos.double()[:, None] * inv)[:, None, :]
    c, sn = torch.cos(a), torch.sin(a)
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * sn, hi * c + lo * sn], -1)


def _attend(q, k, v, pos):
    """q [n, nq, hd] at positions pos [n]; k, v [L, nkv, hd] of positions 0 .. L - 1."""
    n, nq, hd = q.shape
    group = nq // k.shape[1]
    out = torch.empty_like(q)
    at = torch.arange(k.shape[0], device=q.device)
    for h in range(nq):
        kh, vh = k[:, h // group].contiguous(), v[:, h // group].contiguous()
        for r in range(0, n, 512):
            sc = q[r:r + 512, h] @ kh.t().contiguous() / math.sqrt(hd)
            sc.masked_fill_(at[None, :] > pos[r:r + 512, None], -math.inf)
            out[r:r + 512, h] = torch.softmax(sc, -1) @ vh
    return out


def _linear(x, w):
    return x @ w.double().t().contiguous()


def _block(s, w, x, segments):
    """One layer over rows x; segments: (row slice, cached keys and values or None, first position)."""
    n = x.shape[0]
    xn = _norm(x, w["attn_norm"], s.rms_eps)
    q = _linear(xn, w["wq"]).view(n, s.n_q_heads, s.head_dim)
    k = _linear(xn, w["wk"]).view(n, s.n_kv_heads, s.head_dim)
    v = _linear(xn, w["wv"]).view(n, s.n_kv_heads, s.head_dim)
    if s.qk_norm:
        q, k = _norm(q, w["q_norm"], s.rms_eps), _norm(k, w["k_norm"], s.rms_eps)
    o = torch.empty_like(q)
    for rows, cached, pos0 in segments:
        m = rows.stop - rows.start
        pos = torch.arange(pos0, pos0 + m, device=x.device)
        kk, vv = _rope(k[rows], pos, s.rope_theta), v[rows]
        if cached:
            kk, vv = torch.cat([cached[0].double(), kk]), torch.cat([cached[1].double(), vv])
        o[rows] = _attend(_rope(q[rows], pos, s.rope_theta), kk, vv, pos)
    x = x + _linear(o.reshape(n, -1), w["wo"])
    xn = _norm(x, w["mlp_norm"], s.rms_eps)
    return x + _linear(torch.nn.functional.silu(_linear(xn, w["wg"])) * _linear(xn, w["wu"]), w["wd"])


def exact(case, seed):
    d = _inputs(case, seed)
    s, kind = d["shape"], case["kind"]
    if kind == "cache":
        return tuple(t.double() for t in d["saved"])
    if kind == "logits":
        return _linear(_norm(d["hidden"].double(), d["head"]["final_norm"], s.rms_eps), d["head"]["lm_head"])
    x = d["hidden"].double() if "hidden" in d else d["head"]["embed"][d["tokens"].long()].double()
    if kind == "prefill":
        spans = [(slice(0, case["n"]), 0, case["pos0"])]
    else:
        spans = [(slice(b, b + 1), b, n) for b, n in enumerate(d["ctx"])]
    for l, w in enumerate(d["layers"]):
        x = _block(s, w, x, [(rows, d["kv"].get((l, u)), pos0) for rows, u, pos0 in spans])
    if case.get("head"):
        x = _linear(_norm(x, d["head"]["final_norm"], s.rms_eps), d["head"]["lm_head"])
    return x
