"""The work that a program using this library has it do, as cases that can be timed and compared.

A case names one call through the public Python entry points with its sizes: a mat-vec, decode attention, the output
layer, a window of decoder layers advanced by one token, by several (speculative verification), by one token for each
of a batch of sequences, or by a whole prompt.  Layer shapes are those of workloads/configs.py (8B, 14B, 32B and 70B
models); windows are cut to a few layers, which costs per layer what a long window does.

Inputs: weights of mean about zero and standard deviation 0.02 whatever the format, every quant uniform over its range,
activations, KV cache rows and x ~ N(0, 1), norm gains 1 + N(0, 0.1), so that hidden states, attention logits and
softmaxes have the magnitudes that trained models have.
"""
import math
import random

import torch

import paper_2504_08791_amd as prima
from workloads.configs import ModelDims

DIMS = {
    "8b": ModelDims(4096, 32, 8, 128, 14336, 5e5),
    "14b": ModelDims(5120, 40, 8, 128, 13824, 1e6),
    "32b": ModelDims(5120, 40, 8, 128, 27648, 1e6),
    "70b": ModelDims(8192, 64, 8, 128, 28672, 5e5),
}
VOCAB = 128256
WEIGHTS = ("wq", "wk", "wv", "wo", "wgate", "wup", "wdown")
BYTES_PER_WEIGHT = {"q4_k": 144 / 256, "q5_k": 176 / 256, "q6_k": 210 / 256, "q8_0": 272 / 256, "f16": 2.0}
STD = 0.02


# ---- the cases -------------------------------------------------------------------------------------------------------

def listed():
    return [
        # the smallest projection of an 8B layer (K or V) on its own: launch latency
        dict(name="gemv_1024x4096_t1", op="gemv", rows=1024, cols=4096, T=1),
        # one decode step of attention behind a long conversation
        dict(name="attn_14b_ctx30001_t1", op="attn", model="14b", n_past=30001, T=1),
        # output layer of a "Q4K" checkpoint, which keeps that matrix in Q6_K: plain decode
        dict(name="head_70b_q6k_t1", op="head", model="70b", fmt="q6_k", vocab=VOCAB, T=1),
        # ... and 8 draft tokens verified jointly
        dict(name="head_70b_q6k_t8", op="head", model="70b", fmt="q6_k", vocab=VOCAB, T=8),
        # the smallest window: one layer of an 8B model, short context
        dict(name="window_8b_t1", op="window", model="8b", mix="q4k", layers=1, n_past=512, T=1),
        # plain decode on a slice of the 70B window, the benchmark's headline shape
        dict(name="window_70b_t1", op="window", model="70b", mix="q4k", layers=3, n_past=4096, T=1),
        # speculative verification, 4 and 8 draft tokens
        dict(name="window_32b_t4", op="window", model="32b", mix="q4k", layers=4, n_past=4096, T=4),
        dict(name="window_70b_t8", op="window", model="70b", mix="q4k", layers=2, n_past=8192, T=8),
        # a checkpoint with V and down projections in Q6_K in every other layer, a few draft tokens
        dict(name="mixed_14b_t3", op="window", model="14b", mix="q6k_half", layers=4, n_past=2047, T=3),
        # continuous batching: 16 sequences of different lengths, one token each
        dict(name="batch_14b_b16", op="batch", model="14b", mix="q4k", layers=3, n_past=2048, T=16),
        # time to the first token: a prompt of 1024 tokens
        dict(name="prefill_70b_1024", op="prefill", model="70b", mix="q4k", layers=1, n_past=0, T=1024),
        # the next turn of a conversation on a checkpoint with some tensors in Q6_K
        dict(name="prefill_mixed_8b_333", op="prefill", model="8b", mix="q6k_half", layers=2, n_past=777, T=333),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["gemv", "attn", "head", "window", "window", "window", "batch", "prefill", "prefill"])
    model = rng.choice(sorted(DIMS))
    mix = rng.choice(["q4k", "q4k", "q6k_half", "q5k_q6k", "q8_down"])
    if op == "gemv":
        return dict(op=op, rows=_log_int(rng, 500, 60000), cols=256 * _log_int(rng, 4, 112), T=rng.choice([1, 1, 2, 4, 5, 8, 16]))
    if op == "attn":
        return dict(op=op, model=model, n_past=_log_int(rng, 16, 33000), T=rng.choice([1, 1, 1, 2, 4, 7, 8, 16]))
    if op == "head":
        fmt = rng.choice(["q4_k", "q6_k", "q6_k", "q8_0", "q5_k", "f16"])
        vocab = _log_int(rng, 32000, 152001)
        if fmt == "f16":
            vocab = min(vocab, 64001)
        return dict(op=op, model=model, fmt=fmt, vocab=vocab, T=rng.choice([1, 1, 2, 4, 6, 8, 11, 16]))
    if op == "window":
        layers = rng.randint(1, 2 if model == "70b" else 3)
        return dict(op=op, model=model, mix=mix, layers=layers, n_past=_log_int(rng, 1, 8192), T=rng.choice([1, 1, 2, 3, 4, 5, 8, 13, 16]))
    if op == "batch":
        return dict(op=op, model=model, mix=mix, layers=rng.randint(1, 2), n_past=_log_int(rng, 16, 4096), T=rng.randint(2, 16))
    # prompts: at most the work of 1024 tokens through one 70B layer
    cap = {"8b": 4000, "14b": 3000, "32b": 1700, "70b": 1000}[model]
    T = _log_int(rng, 17, cap)
    return dict(op=op, model=model, mix=mix, layers=1, n_past=rng.choice([0, 0, rng.randint(1, 4096)]), T=T)


# ---- inputs ----------------------------------------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed % (1 << 62))


def _bytes(g, n):
    return torch.randint(-(1 << 31), 1 << 31, ((n + 3) // 4,), dtype=torch.int32, device="cuda", generator=g).view(torch.uint8)[:n]


def _half(g, n, mean):
    """n binary16 scales, uniform in [0.5, 1.5] x mean."""
    return (mean * (0.5 + torch.rand(n, device="cuda", generator=g))).to(torch.float16)


def _fields(g, n, d, centre):
    """16-byte headers of n super-blocks of Q4_K / Q5_K: d, dmin and sixteen 6-bit fields, with sub-mins that put the
    middle of the quants' range (`centre`) near zero."""
    sc = torch.randint(16, 64, (n, 8), dtype=torch.int32, device="cuda", generator=g)
    m = (sc + torch.randint(-3, 4, (n, 8), dtype=torch.int32, device="cuda", generator=g)).clamp_(0, 63)
    f = torch.cat([sc, m], 1).view(n, 4, 4)
    v = f[..., 0] | f[..., 1] << 6 | f[..., 2] << 12 | f[..., 3] << 18
    h = torch.empty((n, 16), dtype=torch.uint8, device="cuda")
    h[:, 0:4] = torch.stack([d, (d.float() * centre).to(torch.float16)], 1).view(torch.uint8).view(n, 4)
    h[:, 4:] = torch.stack([v & 255, (v >> 8) & 255, v >> 16], 2).to(torch.uint8).view(n, 12)
    return h


def _tensor(g, fmt, rows, cols):
    """A rows x cols matrix in `fmt`: uint8 [rows, cols/256, 144] for q4_k, flat uint8 otherwise."""
    n = rows * cols // 256
    if fmt == "q4_k":
        w = _bytes(g, n * 144).view(n, 144)
        w[:, :16] = _fields(g, n, _half(g, n, STD / (4.61 * 40)), 7.5)
        return w.view(rows, cols // 256, 144)
    if fmt == "q5_k":
        return torch.cat([_fields(g, n, _half(g, n, STD / (9.23 * 40)), 15.5).view(-1), _bytes(g, n * 160)])
    if fmt == "q6_k":
        return torch.cat([_bytes(g, n * 208), _half(g, n, STD / (18.5 * 74)).view(torch.uint8)])
    if fmt == "q8_0":
        return torch.cat([_bytes(g, n * 256), _half(g, n * 8, STD / 74).view(torch.uint8)])
    return (STD * torch.randn(rows * cols, device="cuda", generator=g)).to(torch.float16).view(torch.uint8)


def _formats(mix, layers):
    """Formats of the matrices that are not Q4_K, layer by layer (None: every matrix of the window is Q4_K)."""
    odd = {"q6k_half": {"wv": "q6_k", "wdown": "q6_k"}, "q5k_q6k": {"wv": "q6_k", "wk": "q5_k", "wo": "q5_k", "wdown": "q6_k"},
           "q8_down": {"wdown": "q8_0"}}
    return None if mix == "q4k" else [odd[mix] if l % 2 == 0 else {} for l in range(layers)]


def _shapes(d):
    return {"wq": (d.qd, d.e), "wk": (d.kvd, d.e), "wv": (d.kvd, d.e), "wo": (d.e, d.qd), "wgate": (d.ffn, d.e), "wup": (d.ffn, d.e),
            "wdown": (d.e, d.ffn)}


def _normal(g, *shape, dtype=torch.float32):
    return torch.randn(shape, device="cuda", dtype=dtype, generator=g)


def _gain(g, n):
    return 1.0 + 0.1 * _normal(g, n)


def _lengths(case):
    """Cached rows of the sequences of a batch: spread from n_past / 8 to n_past, the longest among them."""
    B, n = case["T"], case["n_past"]
    r = random.Random(n * 31 + B)
    return [n] + [max(1, int(n * r.uniform(0.125, 1.0))) for _ in range(B - 1)]


def prepare(case, seed):
    g = _generator(seed)
    op, T = case["op"], case["T"]
    if op == "gemv":
        W = _tensor(g, "q4_k", case["rows"], case["cols"])
        ws = torch.empty(prima.gemv_workspace_bytes(case["rows"], case["cols"], T), dtype=torch.uint8, device="cuda")
        return dict(case=case, W=W, x=_normal(g, T, case["cols"]), y=torch.empty((T, case["rows"]), device="cuda"), ws=ws)
    d = DIMS[case["model"]]
    if op == "attn":
        cap = case["n_past"] + T
        k, v = (_normal(g, d.n_kv_heads, cap, d.head_dim, dtype=torch.float16) for _ in range(2))
        ws = torch.empty(max(256, prima.attn_workspace_bytes(d, cap, T)), dtype=torch.uint8, device="cuda")
        q = _normal(g, T, d.n_q_heads, d.head_dim)
        return dict(case=case, dims=prima.make_dims(d), q=q, k=k, v=v, o=torch.empty_like(q), ws=ws)
    if op == "head":
        s = dict(case=case, dims=prima.make_dims(d), gain=_gain(g, d.e), W=_tensor(g, case["fmt"], case["vocab"], d.e), x=_normal(g, T, d.e),
                 y=torch.empty((T, case["vocab"]), device="cuda"))
        if case["fmt"] == "q4_k":
            s["ws"] = torch.empty(max(256, prima.lm_head_workspace_bytes(d, case["vocab"], T)), dtype=torch.uint8, device="cuda")
        return s
    fm = _formats(case["mix"], case["layers"])
    cap = case["n_past"] + (1 if op == "batch" else T)
    layers, caches = [], []
    for l in range(case["layers"]):
        t = {k: _tensor(g, (fm[l] if fm else {}).get(k, "q4_k"), *_shapes(d)[k]) for k in WEIGHTS}
        t["g_attn"], t["g_ffn"] = _gain(g, d.e), _gain(g, d.e)
        if op == "batch":  # the sequences' caches of a layer, side by side; the window's own are not used
            kv = tuple(_normal(g, T, d.n_kv_heads, cap, d.head_dim, dtype=torch.float16) for _ in range(2))
            t["k_cache"], t["v_cache"] = kv[0][0], kv[1][0]
        else:
            kv = tuple(_normal(g, d.n_kv_heads, cap, d.head_dim, dtype=torch.float16) for _ in range(2))
            t["k_cache"], t["v_cache"] = kv
        layers.append(t)
        caches.append(kv)
    x = _normal(g, T, d.e)
    win = prima.Window(d, layers, cap, T_max=min(T, 16), formats=fm)
    s = dict(case=case, win=win, x=x, y=torch.empty_like(x), caches=caches)
    if op == "batch":
        s["n_past"] = _lengths(case)
        s["seq_caches"] = [[(k[b], v[b]) for b in range(T)] for k, v in caches]
    return s


# ---- one pass ----------------------------------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    op = case["op"]
    if op == "gemv":
        return prima.q4k_gemv(s["W"], s["x"], s["y"], s["ws"])
    if op == "attn":
        return prima.attn_decode(s["dims"], s["q"], s["k"], s["v"], case["n_past"], s["o"], s["ws"])
    if op == "head":
        if case["fmt"] == "q4_k":
            return prima.lm_head(s["dims"], s["gain"], s["W"], s["x"], s["y"], s["ws"])
        return prima.lm_head_fmt(s["dims"], case["fmt"], s["gain"], s["W"], case["vocab"], s["x"], s["y"])
    if op == "window":
        s["win"].decode(s["x"], case["n_past"], s["y"])
    elif op == "batch":
        s["win"].decode_batch(s["x"], s["n_past"], s["seq_caches"], s["y"])
    else:
        s["win"].prefill(s["x"], case["n_past"], s["y"])
    return dict(y=s["y"], caches=s["caches"])


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------

def work(case):
    op, T = case["op"], case["T"]
    if op == "gemv":
        n = case["rows"] * case["cols"]
        return dict(bytes=n * 0.5625 + 4 * T * (case["rows"] + case["cols"]), flops=2 * n * T)
    d = DIMS[case["model"]]
    if op == "batch":
        rows, keys = sum(_lengths(case)) + T, sum(_lengths(case)) + T
    else:
        n = case.get("n_past", 0)
        rows, keys = n + T, T * n + T * (T + 1) // 2  # cache rows read or written; (token, key) pairs
    attn_bytes, attn_flops = 4 * d.kvd * rows, 4 * d.qd * keys
    if op == "attn":
        return dict(bytes=attn_bytes + 8 * T * d.qd, flops=attn_flops)
    if op == "head":
        n = case["vocab"] * d.e
        return dict(bytes=n * BYTES_PER_WEIGHT[case["fmt"]] + 4 * (T + 1) * d.e + 4 * T * case["vocab"], flops=2 * n * T)
    fm = _formats(case["mix"], case["layers"])
    nbytes, flops = 8 * T * d.e, 0
    for l in range(case["layers"]):
        for k, (r, c) in _shapes(d).items():
            nbytes += r * c * BYTES_PER_WEIGHT[(fm[l] if fm else {}).get(k, "q4_k")]
            flops += 2 * r * c * T
        nbytes += attn_bytes + 8 * d.e
        flops += attn_flops
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    # fp32 sums over up to 28672 columns of activations held in 22 to 30 bits: 1.6e-7 to 3.5e-7 against 64 bits.
    if case["op"] in ("gemv", "attn", "head"):
        return dict(rel=1.5e-6, max=4e-5)
    # A window appends K and V rows rounded to binary16: a value near the middle of two of them goes one way or the other
    # (2^-11 of that value), which every later layer carries on and which shows most where few keys are attended to.
    # Against 64 bits: windows 3e-7 to 2.4e-5 (the last behind a few cached rows), a prompt 1.2e-5 to 4.3e-5.
    return dict(rel=2e-4 if case["op"] == "prefill" else 1e-4, max=2e-2)


# ---- 64 bits ----------------------------------------------------------------------------------------------------------

def _fields64(h):
    """Headers uint8 [n, 16] -> d, dmin [n, 1] and the sixteen fields [n, 16] in float64."""
    n = h.shape[0]
    dd = h[:, :4].contiguous().view(torch.float16).to(torch.float64)
    b = h[:, 4:].to(torch.int32).view(n, 4, 3)
    v = b[..., 0] | b[..., 1] << 8 | b[..., 2] << 16
    f = torch.stack([(v >> (6 * i)) & 63 for i in range(4)], 2).view(n, 16).to(torch.float64)
    return dd[:, 0:1], dd[:, 1:2], f


def _words64(low, high, bits):
    """Quants of Q5_K / Q6_K super-blocks: low [n, 128] bytes, high [n, 32 * bits] bytes -> int32 [n, 256]."""
    n = low.shape[0]
    t = torch.arange(256, device=low.device)
    lo = (low.to(torch.int32)[:, 4 * (t // 8) + t % 4] >> (4 * ((t % 8) // 4))) & 15
    per = 8 // bits * 4  # weights per word of the high plane
    hi = (high.to(torch.int32)[:, 4 * (t // per) + t % 4] >> (bits * ((t % per) // 4))) & ((1 << bits) - 1)
    return (lo | hi << 4).view(n, 256)


def _rows64(fmt, W, rows, cols, r0, r1):
    """Rows [r0, r1) of a matrix as float64."""
    nb, n = cols // 256, rows * cols // 256
    a, b = r0 * nb, r1 * nb

    def plane(offset, size):
        return W[offset + a * size:offset + b * size].view(b - a, size)

    if fmt == "q4_k":
        w = W.view(n, 144)[a:b]
        d, dmin, f = _fields64(w[:, :16])
        q = torch.stack([w[:, 16:] & 15, w[:, 16:] >> 4], 2).view(b - a, 8, 32).to(torch.float64)
        out = (d * f[:, :8])[:, :, None] * q - (dmin * f[:, 8:])[:, :, None]
    elif fmt == "q5_k":
        d, dmin, f = _fields64(plane(0, 16))
        q = _words64(plane(16 * n, 128), plane(144 * n, 32), 1).view(b - a, 8, 32).to(torch.float64)
        out = (d * f[:, :8])[:, :, None] * q - (dmin * f[:, 8:])[:, :, None]
    elif fmt == "q6_k":
        q = _words64(plane(0, 128), plane(128 * n, 64), 2).view(b - a, 16, 16).to(torch.float64)
        sc = plane(192 * n, 16).view(torch.int8).to(torch.float64)
        d = plane(208 * n, 2).contiguous().view(torch.float16).to(torch.float64)
        out = (d * sc)[:, :, None] * (q - 32)
    elif fmt == "q8_0":
        q = plane(0, 256).view(torch.int8).view(b - a, 8, 32).to(torch.float64)
        d = plane(256 * n, 16).contiguous().view(torch.float16).to(torch.float64)
        out = d[:, :, None] * q
    else:
        out = W.view(torch.float16).view(rows, cols)[r0:r1].to(torch.float64)
    return out.reshape(r1 - r0, cols)


def _product64(fmt, W, rows, cols, x):
    step = max(1, (1 << 27) // cols)
    return torch.cat([x @ _rows64(fmt, W, rows, cols, r, min(rows, r + step)).T for r in range(0, rows, step)], 1)


def _norm64(x, gain, eps=float(torch.tensor(1e-5, dtype=torch.float32))):
    return x * gain.double() / torch.sqrt((x * x).mean(1, keepdim=True) + eps)


def _rope64(d, x, pos):
    """x [T, heads, D], pairs (i, i + D/2), angle pos * theta^(-2 i / D)."""
    D = d.head_dim
    i = torch.arange(D // 2, device=x.device, dtype=torch.float64)
    ang = pos.to(torch.float64)[:, None] * float(d.rope_theta) ** (-2.0 * i / D)
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :D // 2], x[..., D // 2:]
    return torch.cat([a * c - b * s, a * s + b * c], 2)


def _attention64(d, q, k, v, n_past):
    """q [T, Hq, D] float64, k and v float16 [Hkv, rows, D]: token t sees the rows up to n_past + t."""
    T, G = q.shape[0], d.n_q_heads // d.n_kv_heads
    n = n_past + T
    seen = torch.arange(n, device=q.device)[None] <= n_past + torch.arange(T, device=q.device)[:, None]
    out = torch.empty_like(q)
    for h in range(d.n_q_heads):
        s = (q[:, h] @ k[h // G, :n].double().T) / math.sqrt(d.head_dim)
        out[:, h] = torch.softmax(s.masked_fill(~seen, -math.inf), 1) @ v[h // G, :n].double()
    return out


def _layer64(d, t, fm, x, kv, n_past):
    """One layer; kv: [(k, v, tokens)] per sequence, k and v float16 and written to; n_past per sequence."""
    shapes = _shapes(d)

    def mul(name, a):
        return _product64(fm.get(name, "q4_k"), t[name], *shapes[name], a)

    a = _norm64(x, t["g_attn"])
    q, k, v = (mul(n, a).view(x.shape[0], -1, d.head_dim) for n in ("wq", "wk", "wv"))
    o = torch.empty_like(q)
    for (kc, vc, tok), n in zip(kv, n_past):
        T = tok.stop - tok.start
        pos = torch.arange(n, n + T, device=x.device)
        kc[:, n:n + T] = _rope64(d, k[tok], pos).float().to(torch.float16).transpose(0, 1)
        vc[:, n:n + T] = v[tok].float().to(torch.float16).transpose(0, 1)
        o[tok] = _attention64(d, _rope64(d, q[tok], pos), kc, vc, n)
    h = x + mul("wo", o.reshape(x.shape[0], -1))
    a = _norm64(h, t["g_ffn"])
    gate = mul("wgate", a)
    return h + mul("wdown", gate / (1 + torch.exp(-gate)) * mul("wup", a))


def exact(case, seed):
    s = prepare(case, seed)
    op, T = case["op"], case["T"]
    if op == "gemv":
        return _product64("q4_k", s["W"], case["rows"], case["cols"], s["x"].double())
    d = DIMS[case["model"]]
    if op == "attn":
        return _attention64(d, s["q"].double(), s["k"], s["v"], case["n_past"])
    if op == "head":
        return _product64(case["fmt"], s["W"], case["vocab"], d.e, _norm64(s["x"].double(), s["gain"]))
    x = s["x"].double()
    fm = _formats(case["mix"], case["layers"])
    for l, t in enumerate(s["win"].layers):
        k, v = s["caches"][l]
        if op == "batch":
            kv, n = [(k[b], v[b], slice(b, b + 1)) for b in range(T)], s["n_past"]
        else:
            kv, n = [(k, v, slice(0, T))], [case["n_past"]]
        x = _layer64(d, t, fm[l] if fm else {}, x, kv, n)
    # a cache row is a rounded number: its exact value is not that of the row
    return dict(y=x, caches=None)
