"""Measured cases of the decode step: what a program that decodes with this framework has it do.

Every case is one or more batch-1 decode steps through ``amk.Decoder``, the framework's entry point,
over seeded random weights made on the GPU.  A case is a dict of plain values:

    hidden, layers, heads, kv_heads, head_dim, intermediate, vocab, tied, theta   the model
    fmt         weight format: "bf16", "w8a16" or "w4a16"
    group       input columns per int4 scale ("w4a16" only, else 0)
    pos, steps  the first position decoded, and how many steps follow each other
    read_token  whether the program reads the greedy token back after the step (generation), or feeds
                tokens it already has (a prompt, or scoring a text)

The model shapes are those of ``synth/configs.py`` (whole, or the first layers of one, as a draft model
or a slice of a deeper model has them) and generic ragged ones.
"""
from __future__ import annotations

import math

import torch

from paper_2606_09682_amd import amk

EPS = 1e-5

_SHAPES = {
    # name: hidden, layers, heads, kv_heads, head_dim, intermediate, vocab, tied, theta
    "tiny": (256, 4, 4, 2, 64, 688, 4096, False, 1e4),
    "smollm2_135m": (576, 30, 9, 3, 64, 1536, 49152, True, 1e4),
    "tinyllama_1b": (2048, 22, 32, 4, 64, 5632, 32000, False, 1e4),
    "llama32_1b": (2048, 16, 32, 8, 64, 8192, 128256, True, 5e5),
    "llama3_8b": (4096, 32, 32, 8, 128, 14336, 128256, False, 5e5),
}
_FIELDS = ("hidden", "layers", "heads", "kv_heads", "head_dim", "intermediate", "vocab", "tied", "theta")


def _case(shape, fmt, pos, steps=1, read_token=False, group=0, **over):
    c = dict(zip(_FIELDS, _SHAPES[shape] if isinstance(shape, str) else shape))
    c.update(over)
    c.update(fmt=fmt, group=group, pos=pos, steps=steps, read_token=read_token)
    return c


def listed():
    cases = [
        # the smallest call: a toy decoder's first token, all launch and hand-over latency
        ("tiny_bf16_first", _case("tiny", "bf16", 0)),
        # a short prompt fed token by token to a small model: steps follow each other without a readback
        ("135m_w8a16_prompt", _case("smollm2_135m", "w8a16", 0, steps=32)),
        # a small model in the middle of an answer: one step and its token
        ("135m_bf16_generate", _case("smollm2_135m", "bf16", 200, read_token=True)),
        # a 1B model in int4 past a page of context
        ("1b_w4a16_1024", _case("tinyllama_1b", "w4a16", 1024, group=128, read_token=True)),
        # a 1B model with a tied head and long context
        ("1b_tied_w8a16_4096", _case("llama32_1b", "w8a16", 4096, read_token=True)),
        # nothing divides anything: odd head count, ragged rows, odd vocabulary, odd position
        ("ragged_bf16_577", _case((1040, 7, 15, 5, 64, 2768, 32003, False, 1e4), "bf16", 577)),
        # a draft model for speculative decoding: one large layer under a full vocabulary
        ("draft_bf16_300", _case("llama3_8b", "bf16", 300, layers=1)),
        # a slice of a large model in int4 at long context
        ("slice_w4a16_8000", _case("llama3_8b", "w4a16", 8000, group=128, layers=6, vocab=32000)),
        # the headline: an 8B model's first token in bf16
        ("8b_bf16_first", _case("llama3_8b", "bf16", 0)),
        # an 8B model in bf16 at long context
        ("8b_bf16_8192", _case("llama3_8b", "bf16", 8192, read_token=True)),
        # the 8B model in int8, a short conversation
        ("8b_w8a16_100", _case("llama3_8b", "w8a16", 100, read_token=True)),
        # the 8B model in int4, a longer conversation
        ("8b_w4a16_2000", _case("llama3_8b", "w4a16", 2000, group=128, read_token=True)),
    ]
    return [dict(c, name=n) for n, c in cases]


def draw(rng):
    """One more case: a named shape with fewer layers and another vocabulary, or a ragged shape."""
    fmt = rng.choice(["bf16", "w8a16", "w4a16"])
    if rng.random() < 0.5:
        name = rng.choice(["smollm2_135m", "tinyllama_1b", "llama32_1b", "llama3_8b", "llama3_8b"])
        base = dict(zip(_FIELDS, _SHAPES[name]))
        base["layers"] = rng.randint(1, base["layers"])
        base["vocab"] = rng.randint(base["vocab"] // 8, base["vocab"])
    else:
        head_dim = rng.choice([64, 128])
        kv = rng.randint(1, 8)
        q = rng.choice([1, 2, 3, 4, 5, 7, 8])
        while kv * q * head_dim > 4096:
            kv -= 1
        unit = 64 if fmt == "w4a16" else 16
        hidden = int(math.exp(rng.uniform(math.log(256), math.log(4096)))) // unit * unit
        inter = int(hidden * rng.uniform(2.0, 3.5)) // unit * unit
        base = dict(hidden=hidden, layers=rng.randint(1, 24), heads=kv * q, kv_heads=kv, head_dim=head_dim,
                    intermediate=inter, vocab=int(math.exp(rng.uniform(math.log(2000), math.log(128256)))),
                    tied=rng.random() < 0.5, theta=rng.choice([1e4, 5e5]))
    group = 0
    if fmt == "w4a16":
        widths = (base["hidden"], base["intermediate"], base["heads"] * base["head_dim"])
        group = rng.choice([g for g in (32, 64, 128) if all(w % g == 0 for w in widths)])
    pos = int(math.exp(rng.uniform(0.0, math.log(8193)))) - 1
    steps = 1 if rng.random() < 0.7 else rng.randint(2, 6)
    c = dict(base, fmt=fmt, group=group, pos=pos, steps=steps, read_token=steps == 1 and rng.random() < 0.5)
    while work(c)["bytes"] > 16e9:  # no more than the largest listed case
        if c["steps"] > 1:
            c["steps"] -= 1
        else:
            c["layers"] = max(1, c["layers"] * 2 // 3)
    return c


# ------------------------------------------------------------------ inputs
def _capacity(c):
    return (c["pos"] + c["steps"] + 255) // 256 * 256


def _linears(c):
    H, I, qd, kd = c["hidden"], c["intermediate"], c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
    return [("wq", qd, H), ("wk", kd, H), ("wv", kd, H), ("wo", H, qd), ("wg", I, H), ("wu", I, H), ("wd", H, I)]


def _normal(gen, shape, std, mean=0.0):
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    flat = out.view(-1)
    step = 1 << 27
    for a in range(0, flat.numel(), step):
        n = min(step, flat.numel() - a)
        flat[a:a + n] = torch.randn(n, generator=gen, device="cuda").mul_(std).add_(mean)
    return out


def _int8(w):
    """Symmetric int8 with one fp32 scale per output row."""
    w = w.float()
    s = w.abs().amax(dim=1) / 127.0
    q = torch.round(w / torch.where(s > 0, s, torch.ones_like(s))[:, None]).clamp_(-127, 127).to(torch.int8)
    return q, s


def _int4(w, group):
    """Symmetric int4 with one fp16 scale per row and `group` columns, in the decoder's nibble layout."""
    out, k = w.shape
    w = w.float().view(out, k // group, group)
    s = (w.abs().amax(dim=2) / 7.0).half()
    f = s.float()
    q = torch.round(w / torch.where(f > 0, f, torch.ones_like(f))[:, :, None]).clamp_(-8, 7)
    u = (q.view(out, k // 8, 2, 4) + 8).to(torch.uint8)
    return (u[:, :, 0] | (u[:, :, 1] << 4)).reshape(out, k // 2).contiguous(), s


def _quantised(c, w):
    if c["fmt"] == "w8a16":
        parts = [_int8(p) for p in w.split(1 << 14)]
    else:
        parts = [_int4(p, c["group"]) for p in w.split(1 << 14)]
    return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])


def _tensors(c, seed):
    """Name -> device tensor, as ``amk.Decoder`` takes them."""
    gen = torch.Generator(device="cuda").manual_seed(1000 + seed)
    H, V = c["hidden"], c["vocab"]
    t = {"embed": _normal(gen, (V, H), 0.02), "final_norm": _normal(gen, (H,), 0.01, 1.0)}

    def linear(name, out, inp):
        w = _normal(gen, (out, inp), 0.02)
        if c["fmt"] == "bf16":
            t[name] = w
        else:
            t[name], t[name + ".scale"] = _quantised(c, w)

    for l in range(c["layers"]):
        p = "layers.%d." % l
        t[p + "attn_norm"] = _normal(gen, (H,), 0.01, 1.0)
        t[p + "mlp_norm"] = _normal(gen, (H,), 0.01, 1.0)
        for name, out, inp in _linears(c):
            linear(p + name, out, inp)
    if not c["tied"]:
        linear("lm_head", V, H)
    return t


def _context(c, seed):
    """KV cache with the positions before `pos` filled, and the tokens to feed."""
    gen = torch.Generator(device="cuda").manual_seed(5000 + seed)
    kv = torch.zeros(c["layers"], 2, c["kv_heads"], _capacity(c), c["head_dim"], dtype=torch.bfloat16, device="cuda")
    for l in range(c["layers"]):
        kv[l, :, :, :c["pos"]] = torch.randn(2, c["kv_heads"], c["pos"], c["head_dim"], generator=gen, device="cuda")
    tokens = torch.randint(0, c["vocab"], (c["steps"],), generator=gen, device="cuda").tolist()
    return kv, tokens


class _State:
    pass


def prepare(case, seed):
    s = _State()
    c = s.case = case
    s.tensors = _tensors(c, seed)
    s.kv, s.tokens = _context(c, seed)
    s.logits = torch.empty(c["steps"], (c["vocab"] + 3) // 4 * 4, dtype=torch.float32, device="cuda")
    cfg = amk.make_config(c["hidden"], c["layers"], c["heads"], c["kv_heads"], c["head_dim"], c["intermediate"],
                          c["vocab"], _capacity(c), c["theta"], EPS, c["tied"], c["fmt"], group_size=c["group"])
    s.decoder = amk.Decoder(cfg, s.tensors)
    return s


def run(s):
    c = s.case
    token = None
    for i, t in enumerate(s.tokens):
        s.decoder.step(t, c["pos"] + i, s.kv, s.logits[i])
        if c["read_token"]:
            token = s.decoder.next_token()
    out = {"logits": s.logits[:, :c["vocab"]], "rows": s.kv[:, :, :, c["pos"]:c["pos"] + c["steps"]], "kv": s.kv}
    if token is not None:
        out["token"] = token
    return out


# ------------------------------------------------------------------ the same in 64 bits
def _dequantised(c, t, name):
    w = t[name]
    if name + ".scale" not in t:
        return w.double()
    s = t[name + ".scale"].double()
    if c["fmt"] == "w8a16":
        return w.double() * s[:, None]
    out, half = w.shape
    words = w.view(out, half // 4, 4)
    q = torch.stack([words & 15, words >> 4], dim=2).reshape(out, 2 * half).double() - 8.0
    return (q.view(out, -1, c["group"]) * s[:, :, None]).view(out, 2 * half)


def _matvec(c, t, name, x):
    rows = t[name].shape[0]
    step = 1 << 14
    if rows <= step:
        return torch.mv(_dequantised(c, t, name), x)
    parts = []
    for a in range(0, rows, step):
        part = {k: t[k][a:a + step] for k in (name, name + ".scale") if k in t}
        parts.append(torch.mv(_dequantised(c, part, name), x))
    return torch.cat(parts)


def _rms(x, g):
    return x / torch.sqrt(torch.mean(x * x) + EPS) * g.double()


def _rope(x, pos, theta):
    d = x.shape[-1]
    inv = float(torch.tensor(theta, dtype=torch.float32)) ** (-2.0 * torch.arange(d // 2, device="cuda").double() / d)
    cos, sin = torch.cos(pos * inv), torch.sin(pos * inv)
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)


def exact(case, seed):
    c = case
    # every dequantised matrix is made anew for each step: keep that within the time allowed
    if c["steps"] * (c["layers"] * sum(o * i for _, o, i in _linears(c)) + c["vocab"] * c["hidden"]) > 3e10:
        return None
    t = _tensors(c, seed)
    kv, tokens = _context(c, seed)
    nq, nkv, d = c["heads"], c["kv_heads"], c["head_dim"]
    rows = torch.zeros(c["layers"], 2, nkv, c["steps"], d, dtype=torch.float64, device="cuda")
    logits = []
    for i, tok in enumerate(tokens):
        pos = c["pos"] + i
        x = t["embed"][tok].double()
        for l in range(c["layers"]):
            p = "layers.%d." % l
            h = _rms(x, t[p + "attn_norm"])
            q = _rope(_matvec(c, t, p + "wq", h).view(nq, d), pos, c["theta"])
            rows[l, 0, :, i] = _rope(_matvec(c, t, p + "wk", h).view(nkv, d), pos, c["theta"])
            rows[l, 1, :, i] = _matvec(c, t, p + "wv", h).view(nkv, d)
            kv[l, :, :, pos] = rows[l, :, :, i].to(torch.bfloat16)  # the cache is bf16 by definition
            k, v = kv[l, 0, :, :pos + 1].double(), kv[l, 1, :, :pos + 1].double()
            s = (k[:, None] * q.view(nkv, nq // nkv, 1, d)).sum(-1) / math.sqrt(d)
            w = torch.softmax(s, dim=-1)
            o = (w[..., None] * v[:, None]).sum(2).reshape(-1)
            x = x + _matvec(c, t, p + "wo", o)
            h = _rms(x, t[p + "mlp_norm"])
            g = _matvec(c, t, p + "wg", h)
            x = x + _matvec(c, t, p + "wd", g * torch.sigmoid(g) * _matvec(c, t, p + "wu", h))
        logits.append(_matvec(c, t, "embed" if c["tied"] else "lm_head", _rms(x, t["final_norm"])))
    # Rows as computed, before their rounding to bf16.  Where many layers each average few positions, the logits say
    # which elements that rounding flipped and not how exactly they were summed (two seeds of one case differ
    # fivefold), so they have no value here.
    logits = torch.stack(logits) if c["pos"] >= 64 * c["layers"] else None
    out = {"logits": logits, "rows": rows, "kv": None}
    if c["read_token"]:
        out["token"] = None
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    H, L, V, I = c["hidden"], c["layers"], c["vocab"], c["intermediate"]
    lin = sum(o * i for _, o, i in _linears(c)) * L
    rows = sum(o for _, o, _ in _linears(c)) * L
    head = V * H
    if c["fmt"] == "bf16":
        weights = 2 * lin + 2 * head
    elif c["fmt"] == "w8a16":
        weights = lin + 4 * rows + (2 * head if c["tied"] else head + 4 * V)
    else:
        weights = lin // 2 + 2 * lin // c["group"] + (2 * head if c["tied"] else head // 2 + 2 * head // c["group"])
    per_step = weights + (2 * L + 1) * H * 2 + H * 2 + 4 * V
    row = c["kv_heads"] * c["head_dim"] * 2
    nbytes = flops = 0
    for i in range(c["steps"]):
        n = c["pos"] + i + 1
        nbytes += per_step + L * 2 * row * n
        flops += 2 * (lin + head) + 4 * L * c["heads"] * c["head_dim"] * n
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Activations and sums are 32 bits on the way; what moves a result is the rounding of an appended K or V
    element to bf16, which another order of summation can flip (one bf16 step, 0.4% of that element).  Such a flip
    travels through the layers that follow, most at the first positions, where the new row is most of what the
    attention averages.  Measured against 64 bits: up to 1.5e-3 from position 0 through 30 layers, up to 2.2e-4
    (the rows) and 1.4e-5 (the logits) from position 64 on."""
    if case["pos"] < 64:
        return {"rel": 6e-3, "max": 0.1}
    return {"rel": 1e-3, "max": 0.04}
