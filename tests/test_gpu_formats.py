"""GPU parity of the other weight formats (Q5_K, Q6_K, Q8_0, FP16, FP32) against the CPU oracle, through
the C ABI: dequantisation bit for bit, mat-vec and output layer within the mat-vec tolerance."""
import numpy as np
import pytest
import torch

import oracle
from metrics import rel_err
from tolerance import EPS_FP32, check_hidden
from test_gpu_prefill import _centred, _shapes
from workloads import synth
from workloads.configs import CONFIGS, TINY

pytestmark = pytest.mark.gpu

FORMATS = ["q5_k", "q6_k", "q8_0", "f16", "f32"]
GEMV_TOL = 1e-4      # fp32 sums of up to 28672 terms against fp64 (the Q4_K mat-vec tests use the same bound)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rand_tensor(rng, fmt, rows, cols):
    """every field uniform over its range, scales any finite binary16 of moderate size (either sign)"""
    n = rows * cols // 256
    nbytes = int(n * 256 * synth.FORMAT_BITS[fmt] / 8)
    if fmt == "f32":
        return rng.standard_normal((rows, cols)).astype(np.float32).view(np.uint8).reshape(-1)
    if fmt == "f16":
        return rng.standard_normal((rows, cols)).astype(np.float16).view(np.uint8).reshape(-1)
    raw = rng.integers(0, 256, nbytes, dtype=np.uint8)

    def halves(count):
        return ((rng.integers(0, 2, count) << 15) | (rng.integers(8, 18, count) << 10) | rng.integers(0, 1024, count)).astype("<u2").view(np.uint8)

    if fmt == "q5_k":
        raw[:16 * n].reshape(n, 16)[:, 0:4] = halves(2 * n).reshape(n, 4)
    elif fmt == "q6_k":
        raw[208 * n:] = halves(n)
    else:
        raw[rows * cols:] = halves(8 * n)
    return raw


@pytest.mark.parametrize("fmt", FORMATS + ["q4_k"])
def test_dequant_bit_exact(gpu_lib, fmt):
    rng = np.random.default_rng(3)
    for rows, cols in [(1, 256), (5, 768), (67, 2048), (3, 28672)]:
        W = synth.fmt_tensor(0, 1, "wq", fmt, rows, cols) if fmt == "q4_k" else _rand_tensor(rng, fmt, rows, cols)
        ref = oracle.fmt_dequant(fmt, W, rows, cols)
        got = gpu_lib.fmt_dequant(fmt, _dev(W), rows, cols).cpu().numpy()
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (fmt, rows, cols)


@pytest.mark.parametrize("fmt", FORMATS)
def test_gemv_shapes_and_token_counts(gpu_lib, fmt):
    """Rows ragged against the 4-, 2- and 1-row groups (few and many rows: both choices of rows per wave), K from one
    super-block to 40960 (whole and partial pieces of 1024 weights, one and several chunks of K in LDS), every token
    count (passes of up to 8), activations with a different scale per token: each against the oracle, and twice with
    identical bits."""
    rng = np.random.default_rng(77)
    cases = [(1, 256, 1), (2, 256, 16), (3, 512, 2), (5, 768, 3), (37, 1024, 4), (130, 1280, 5), (64, 4096, 6), (63, 4352, 7),
             (257, 8192, 8), (33, 8192, 9), (7, 28672, 1), (18, 28672, 12), (1000, 3584, 1), (4096, 2048, 1),
             # K beyond what LDS holds for one and two tokens (chunks of 32768 and 16384 weights), 16 tokens in two passes
             (9, 40960, 1), (6, 33024, 2), (5, 12288, 16), (40000, 256, 1), (33000, 512, 3)]
    for rows, cols, T in cases:
        W = _rand_tensor(rng, fmt, rows, cols)
        x = (rng.standard_normal((T, cols)) * np.exp(2 * rng.standard_normal((T, 1)))).astype(np.float32)
        ref = oracle.fmt_gemv(fmt, W, rows, cols, x.astype(np.float64))
        Wd, xd = _dev(W), _dev(x)
        got = gpu_lib.fmt_gemv(fmt, Wd, rows, cols, xd).cpu().numpy()
        again = gpu_lib.fmt_gemv(fmt, Wd, rows, cols, xd).cpu().numpy()
        assert rel_err(got, ref) < GEMV_TOL, (fmt, rows, cols, T, rel_err(got, ref))
        assert np.array_equal(got.view(np.uint32), again.view(np.uint32)), (fmt, rows, cols, T)


def test_gemv_strided_activations_and_outputs(gpu_lib):
    rng = np.random.default_rng(8)
    rows, cols, T = 50, 1024, 3
    W = _rand_tensor(rng, "q6_k", rows, cols)
    xbig = torch.full((T, cols + 64), float("nan"), device="cuda")
    x = rng.standard_normal((T, cols)).astype(np.float32)
    xbig[:, :cols] = _dev(x)
    ybig = torch.full((T, rows + 7), -7.0, device="cuda")
    gpu_lib.fmt_gemv("q6_k", _dev(W), rows, cols, xbig[:, :cols], y=ybig[:, :rows])
    ref = oracle.fmt_gemv("q6_k", W, rows, cols, x.astype(np.float64))
    assert rel_err(ybig[:, :rows].cpu().numpy(), ref) < GEMV_TOL
    assert (ybig[:, rows:] == -7.0).all()


def test_gemv_argument_errors(gpu_lib):
    W = torch.zeros(gpu_lib.fmt_tensor_bytes("q8_0", 4, 256), dtype=torch.uint8, device="cuda")
    x = torch.zeros((1, 256), device="cuda")
    with pytest.raises(gpu_lib.PrimaError):
        gpu_lib.fmt_gemv("q8_0", W, 4, 256, torch.zeros((17, 256), device="cuda"))       # too many tokens
    with pytest.raises(gpu_lib.PrimaError):
        gpu_lib.fmt_gemv("q4_k", torch.zeros(4 * 144, dtype=torch.uint8, device="cuda"), 4, 256, x)   # has its own entry point
    with pytest.raises(ValueError):
        gpu_lib.fmt_gemv("q8_0", W[:-2], 4, 256, x)
    assert gpu_lib.fmt_tensor_bytes("q6_k", 4, 100) == 0


@pytest.mark.parametrize("fmt,T", [("q6_k", 1), ("q6_k", 8), ("q8_0", 3), ("f16", 1)])
def test_lm_head_in_another_format(gpu_lib, fmt, T):
    """Output layer: final RMSNorm fused in front of the mat-vec; vocabulary ragged against the row groups."""
    cfg = CONFIGS["c1"]
    d = cfg.dims
    vocab = 3001
    W = synth.fmt_tensor(cfg.config_id, 0, "w_lm", fmt, vocab, d.e)
    g = synth.gain_f32(cfg.config_id, 0, "g_final", d.e)
    x = (synth.normal_f32(cfg.config_id, 0, "x_in", (T, d.e)).astype(np.float64) * 1e3).astype(np.float32)
    ref = oracle.lm_head_fmt(d, fmt, g, W, vocab, x.astype(np.float64))
    got = gpu_lib.lm_head_fmt(d, fmt, _dev(g), _dev(W), vocab, _dev(x)).cpu().numpy()
    assert rel_err(got, ref) < 2e-3          # the hidden-state tolerance
    assert rel_err(got, ref) < 1e-4, rel_err(got, ref)


def test_lm_head_q6k_full_vocab_sampled(gpu_lib):
    """Config 4's output layer (128256 x 8192) in Q6_K, one token: logits sampled across the vocabulary and its
    ragged end recomputed one by one by a brute-force fp64 product on the dequantised rows."""
    cfg = CONFIGS["c4k1"]
    d = cfg.dims
    vocab = cfg.vocab
    W = synth.fmt_tensor(cfg.config_id, 0, "w_lm", "q6_k", vocab, d.e)
    g = synth.gain_f32(cfg.config_id, 0, "g_final", d.e)
    x = synth.normal_f32(cfg.config_id, 0, "x_in", (1, d.e))
    got = gpu_lib.lm_head_fmt(d, "q6_k", _dev(g), _dev(W), vocab, _dev(x)).cpu().numpy()[0]
    assert np.isfinite(got).all()
    rows = [0, 1, 2, 3, 4, 1023, 65535, 65536, 100000, vocab - 5, vocab - 4, vocab - 1]
    n = x[0].astype(np.float64)
    n = n / np.sqrt((n ** 2).mean() + float(np.float32(d.rms_eps))) * g.astype(np.float64)
    # rows one by one: a one-row tensor cut out of the planes
    nblk = d.e // 256
    N = vocab * nblk
    ref = []
    for r in rows:
        one = np.concatenate([W[r * nblk * 128:(r + 1) * nblk * 128], W[128 * N + r * nblk * 64:128 * N + (r + 1) * nblk * 64],
                              W[192 * N + r * nblk * 16:192 * N + (r + 1) * nblk * 16], W[208 * N + r * nblk * 2:208 * N + (r + 1) * nblk * 2]])
        ref.append(float(oracle.fmt_dequant("q6_k", one, 1, d.e)[0].astype(np.float64) @ n))
    ref = np.array(ref)
    scale = np.sqrt((ref ** 2).mean())
    assert np.abs(got[rows] - ref).max() / scale < 1e-4


MIXES = {
    # the usual mix of a "Q4K" model: V and down projections in Q6_K
    "q4_k_m": [{"wv": "q6_k", "wdown": "q6_k"}, {}, {"wv": "q6_k", "wdown": "q6_k"}],
    # every matrix in some other format, gate / up not both Q4_K (SwiGLU as its own launch), one Q4_K matrix alone in its group
    "all_kinds": [{"wq": "q8_0", "wk": "q5_k", "wv": "f16", "wo": "q6_k", "wgate": "q5_k", "wup": "q8_0", "wdown": "f32"},
                  {"wq": "q6_k", "wgate": "q6_k"},
                  {"wk": "q8_0", "wv": "q8_0", "wup": "f16", "wo": "f16", "wdown": "q5_k"}],
}


@pytest.mark.parametrize("mix", sorted(MIXES))
@pytest.mark.parametrize("name,T", [("t1", 1), ("t2", 5), ("c1", 4), ("c0", 11)])
def test_window_with_mixed_formats(gpu_lib, mix, name, T):
    """Three layers with matrices in several formats, one and several tokens (passes of 8 in the format mat-vec):
    hidden state against the oracle within the hidden-state tolerance; the appended K/V rows too."""
    n_layers = 3
    formats = MIXES[mix][-n_layers:]
    cfg = {**CONFIGS, **TINY}[name].with_(n_layers=n_layers, T=T)
    d = cfg.dims
    cap = cfg.n_past + T
    x = synth.window_input(cfg)
    host = [synth.layer_tensors(cfg, l, kv_cap=cap, formats=formats[l]) for l in range(n_layers)]
    dev_layers = [{k: _dev(v) for k, v in t.items()} for t in host]
    ref = oracle.window(d, host, x.astype(np.float64), cfg.n_past, formats=formats)     # appends to the host caches
    win = gpu_lib.Window(d, dev_layers, cap, T_max=T, formats=formats)
    win.workspace.fill_(0xFF)
    y = win.decode(_dev(x), cfg.n_past).cpu().numpy()
    err = rel_err(y, ref)
    print("mixed formats", mix, name, T, "hidden-state max rel err", err, flush=True)
    check_hidden(f"mixed {mix} {name} T={T}", err, d, host, x.astype(np.float64), cfg.n_past, formats=formats, eps=EPS_FP32)
    # the first layer's appended rows (deeper layers' rows inherit the hidden state's error)
    for c in ("k_cache", "v_cache"):
        new_ref = host[0][c][:, cfg.n_past:cfg.n_past + T].astype(np.float64).reshape(1, -1)
        new_got = dev_layers[0][c][:, cfg.n_past:cfg.n_past + T].float().cpu().numpy().reshape(1, -1)
        assert rel_err(new_got, new_ref) < 2e-3


def test_mixed_window_of_q4k_only_equals_the_q4k_window(gpu_lib):
    """With every format Q4_K the mixed entry point runs the same launches: identical bits."""
    cfg = CONFIGS["c1"].with_(n_layers=2)
    d = cfg.dims
    cap = cfg.n_past + cfg.T
    xd = _dev(synth.window_input(cfg))
    dev_layers = [{k: _dev(v) for k, v in synth.layer_tensors(cfg, l, kv_cap=cap).items()} for l in range(2)]
    a = gpu_lib.Window(d, dev_layers, cap, T_max=cfg.T).decode(xd, cfg.n_past).clone()
    b = gpu_lib.Window(d, dev_layers, cap, T_max=cfg.T, formats=[{}, {}]).decode(xd, cfg.n_past)
    assert torch.equal(a, b)


def test_mixed_window_full_shape(gpu_lib):
    """Config 3's layer shape, 4 layers, V and down projections in Q6_K (the usual mix), one token."""
    formats = [{"wv": "q6_k", "wdown": "q6_k"}] * 4
    cfg = CONFIGS["c3"].with_(n_layers=4)
    d = cfg.dims
    cap = cfg.n_past + cfg.T
    x = synth.window_input(cfg)
    dev_layers, h = [], x.astype(np.float64)
    for l in range(4):
        t = synth.layer_tensors(cfg, l, kv_cap=cap, formats=formats[l])
        dev_layers.append({k: _dev(v) for k, v in t.items()})
        h = oracle.layer(d, t, h, cfg.n_past, formats=formats[l])
        del t
    win = gpu_lib.Window(d, dev_layers, cap, T_max=cfg.T, formats=formats)
    win.workspace.fill_(0xFF)
    y = win.decode(_dev(x), cfg.n_past).cpu().numpy()
    check_hidden("config 3's shape, V and down in Q6_K", rel_err(y, h), d,
                 lambda: [synth.layer_tensors(cfg, l, kv_cap=cap, formats=formats[l]) for l in range(4)], x.astype(np.float64), cfg.n_past,
                 formats=formats, eps=EPS_FP32)


@pytest.mark.parametrize("name,more,mix", [("t0", 0, "all_kinds"), ("t1", 0, "all_kinds"), ("t2", 0, "all_kinds"), ("t1", 4, "all_kinds"),
                                           ("t0", 6, "q4_k_m"), ("t2", 11, "q4_k_m")])
def test_batch_of_sequences_with_mixed_formats(gpu_lib, name, more, mix):
    """One token for each of several sequences of different lengths (one empty, one full) through two layers whose
    matrices are in several formats: hidden states against the oracle (each sequence alone), appended rows."""
    formats = MIXES[mix][:2]
    cfg = TINY[name].with_(n_layers=2)
    d = cfg.dims
    lens = [0, 5, cfg.n_past, 17, 5] + [3 * i + 1 for i in range(more)]
    B = len(lens)
    cap = cfg.n_past + 1
    host = [synth.layer_tensors(cfg.with_(n_past=0), l, kv_cap=1, formats=formats[l]) for l in range(2)]
    dev_layers = [{k: _dev(v) for k, v in t.items()} for t in host]
    for dl in dev_layers:      # the window's own caches are not used by a batch
        dl["k_cache"] = torch.zeros((d.n_kv_heads, cap, d.head_dim), dtype=torch.float16, device="cuda")
        dl["v_cache"] = dl["k_cache"]
    caches = synth.batch_caches(cfg, 2, lens, cap)
    dev_caches = [[(_dev(k), _dev(v)) for k, v in per_layer] for per_layer in caches]
    xb = synth.batch_input(cfg, B)
    ref = oracle.window_batch(d, host, caches, xb.astype(np.float64), lens, formats=formats)     # appends to the host caches
    win = gpu_lib.Window(d, dev_layers, cap, T_max=B, formats=formats)
    win.workspace.fill_(0xFF)
    y = win.decode_batch(_dev(xb), lens, dev_caches).cpu().numpy()
    assert rel_err(y, ref) < 2e-3, rel_err(y, ref)
    for l in range(2):
        for b in range(B):
            for i in range(2):
                got = dev_caches[l][b][i][:, lens[b]].float().cpu().numpy().reshape(1, -1)
                want = caches[l][b][i][:, lens[b]].astype(np.float64).reshape(1, -1)
                assert rel_err(got, want) < 2e-3


@pytest.mark.parametrize("fmt", ["q5_k", "q6_k", "q8_0", "f16"])
@pytest.mark.parametrize("rows,cols,tokens", [(98289, 256, (2, 3)),   # a tile of one row at the end, rows of one super-block
                                              (32775, 1280, (4, 6)),  # an odd number of super-blocks, 7 rows over
                                              (17, 9 * 256, (7, 8)),  # two tiles: parts of a unit
                                              (5, 20 * 256, (7, 8)),  # one tile, not full
                                              (16513, 768, (4, 6)),   # just above a round of the mat-vec
                                              (1001, 4352, (9, 10)),  # 8 tokens there and the others through the fp32 mat-vec
                                              (131105, 256, (9, 16))])  # more rounds than sums fit LDS
def test_matrix_core_matvec_edges(gpu_lib, fmt, rows, cols, tokens):
    """The several-token kernel at the edges of its tiles, parts, chunks and rounds, rows sampled from both ends and between."""
    rng = np.random.default_rng(11)
    W = _rand_tensor(rng, fmt, rows, cols)
    Wd = _dev(W)
    pick = np.unique(np.concatenate([np.arange(min(rows, 40)), np.arange(max(0, rows - 40), rows), rng.integers(0, rows, 40)]))
    w = gpu_lib.fmt_dequant(fmt, Wd, rows, cols)[torch.from_numpy(pick).cuda()].cpu().numpy().astype(np.float64)
    for T in tokens:
        x = rng.standard_normal((T, cols)).astype(np.float32) * np.logspace(-3, 3, T, dtype=np.float32)[:, None]
        got = gpu_lib.fmt_gemv(fmt, Wd, rows, cols, _dev(x)).cpu().numpy()
        again = gpu_lib.fmt_gemv(fmt, Wd, rows, cols, _dev(x)).cpu().numpy()
        assert np.array_equal(got, again)
        one = gpu_lib.fmt_gemv(fmt, Wd, rows, cols, _dev(x[:1])).cpu().numpy()
        assert not np.array_equal(got[:1], one)      # (the fp32 mat-vec's sums: not the same bits)
        ref = x.astype(np.float64) @ w.T
        assert rel_err(got[:, pick], ref) <= GEMV_TOL, (fmt, rows, T)


@pytest.mark.parametrize("dist", ["normal", "spread"])
@pytest.mark.parametrize("fmt", ["q4_k", "q5_k", "q6_k", "q8_0", "f16"])
def test_several_tokens_are_no_less_exact_than_one(gpu_lib, fmt, dist):
    """2-norm error against 64 bits of the several-token mat-vecs beside that of the same tokens one (Q4_K: eight) at a time, which
    the fp32 mat-vec (the integer one) multiplies: no larger for activations of one magnitude.  With magnitudes over six
    decades within a row the two binary16 parts of an activation (22 bits or more of it) show: a tenth at most.  The largest
    error of an output stays below 1e-6 of the outputs' rms either way."""
    rng = np.random.default_rng(17)
    for rows, cols in ((20000, 4096), (5120, 13824)) if fmt != "q4_k" else ((28673, 4096),):
        W = _dev(_centred(rng, fmt, rows, cols))
        if fmt == "q4_k":
            W = W.view(rows, cols // 256, 144)
        x = rng.standard_normal((16, cols)) * (1 if dist == "normal" else 10 ** rng.uniform(-3, 3, (16, cols)))
        x = _dev(x.astype(np.float32))
        w = (gpu_lib.q4k_dequant(W) if fmt == "q4_k" else gpu_lib.fmt_dequant(fmt, W, rows, cols)).double()   # (within 2^-24 of the exact weights)
        ref = x.double() @ w.T
        mul = (lambda v: gpu_lib.q4k_gemv(W, v)) if fmt == "q4_k" else (lambda v: gpu_lib.fmt_gemv(fmt, W, rows, cols, v))
        apart = torch.cat([mul(x[i:i + (8 if fmt == "q4_k" else 1)].contiguous()) for i in range(0, 16, 8 if fmt == "q4_k" else 1)])
        for T in (4, 7, 8, 16) if fmt != "q4_k" else (11, 16):
            got = mul(x[:T].contiguous())
            e, e1 = ((v[:T] - ref[:T]).norm() / ref[:T].norm() for v in (got.double(), apart.double()))
            big = ((got - ref[:T]).abs() / torch.maximum(ref[:T].abs(), ref[:T].pow(2).mean(1, keepdim=True).sqrt())).max()
            print(fmt, dist, rows, cols, T, f"{e:.3e} {e1:.3e} {big:.2e}", flush=True)
            assert e <= (1.0 if dist == "normal" else 1.1) * e1 and big < 1e-6, (fmt, rows, cols, T, float(e), float(e1), float(big))


@pytest.mark.parametrize("rows,nb,T", [(28672, 1, 11), (28687, 3, 16), (65537, 2, 9)])
def test_tall_q4k_matvec_of_many_tokens(gpu_lib, rows, nb, T):
    """Many tokens of a tall Q4_K matrix (one pass on the matrix cores): ragged last tile, one super-block, an odd number of
    them; with and without scratch the same bits."""
    rng = np.random.default_rng(rows + T)
    W = _dev(synth.fmt_tensor(0, 1, "wq", "q4_k", rows, nb * 256)).view(rows, nb, 144)
    x = rng.standard_normal((T, nb * 256)).astype(np.float32) * np.logspace(-3, 3, T, dtype=np.float32)[:, None]
    w = gpu_lib.q4k_dequant(W).cpu().numpy().astype(np.float64)
    ref = x.astype(np.float64) @ w.T
    got = gpu_lib.q4k_gemv(W, _dev(x))
    assert rel_err(got.cpu().numpy(), ref) <= GEMV_TOL
    other = torch.empty_like(got)
    gpu_lib.q4k_gemv_noalloc(W, _dev(x), other)
    assert torch.equal(got, other)


@pytest.mark.parametrize("mix", sorted(MIXES))
@pytest.mark.parametrize("name,T", [("t1", 8), ("t1", 9), ("t1", 16), ("c1", 13)])
def test_window_of_many_tokens(gpu_lib, mix, name, T):
    """8 to 16 tokens (streams over laid-out activations: the narrow layers from 9 on, at 8 their matrices in other formats): rows of 3 and 5 super-blocks and of a model's size, slabs and
    parts of one stage, layers with and without an FP32 matrix behind one another."""
    test_window_with_mixed_formats(gpu_lib, mix, name, T)


def test_scratch_of_a_wide_model_serves_every_token_count(gpu_lib):
    """Rows of more than 131072 columns, no scratch region for the weight streams: a window made for 16 tokens takes steps of
    any number, and short prompts whose last piece has 4 to 8 tokens leave their scratch alone."""
    from workloads.configs import ModelDims, WindowConfig
    d = ModelDims(256, 2, 1, 128, 131328, 1e4)
    fm = [{"wv": "q6_k", "wgate": "q5_k", "wup": "q6_k", "wdown": "q6_k"}]     # (Q4_K rows of this width take four tokens at most)
    rng = np.random.default_rng(5)
    for n_past, counts in ((64, (5, 8, 9, 16)), (3, (7,))):
        host = synth.layer_tensors(WindowConfig("wide", 77, d, 1, 16, n_past), 0, kv_cap=n_past + 20, formats=fm[0])
        x = rng.standard_normal((20, d.e)).astype(np.float32)
        ref = oracle.layer(d, {k: np.array(v) for k, v in host.items()}, x.astype(np.float64), n_past, formats=fm[0])
        dev = {k: _dev(v) for k, v in host.items()}
        win = gpu_lib.Window(d, [dev], n_past + 20, T_max=16, formats=fm)
        win.workspace.fill_(0xFF)
        for T in counts:
            y = win.decode(_dev(x[:T]), n_past).cpu().numpy()
            check_hidden(f"wide, {n_past} cached rows, T={T}", rel_err(y, ref[:T]), d, [host], x[:T].astype(np.float64), n_past, formats=fm, eps=EPS_FP32)
        gpu_lib.set_prefill_small_tokens(32)
        try:
            y = win.prefill(_dev(x), n_past).cpu().numpy()
        finally:
            gpu_lib.set_prefill_small_tokens(gpu_lib.PREFILL_SMALL_TOKENS)
        check_hidden(f"wide, {n_past} cached rows, prompt", rel_err(y, ref), d, [host], x.astype(np.float64), n_past, formats=fm, eps=EPS_FP32)


@pytest.mark.parametrize("fmt", ["q5_k", "q6_k", "q8_0", "f16"])
@pytest.mark.parametrize("T", [8, 16])
def test_activations_that_are_not_finite_and_tiny_ones(gpu_lib, fmt, T):
    """Infinities and NaN in some tokens of a several-token mat-vec: Q8_0 and FP16 (a weight times an activation, nothing taken
    off again) give what one token at a time gives, infinity for infinity and NaN for NaN; no other token notices.  Activations
    of 1e-35 keep their precision."""
    rng = np.random.default_rng(23)
    rows, cols = 300, 1024
    W = _dev(_centred(rng, fmt, rows, cols))
    x = _dev(rng.standard_normal((T, cols)).astype(np.float32))
    x[1] *= 1e-35
    clean = gpu_lib.fmt_gemv(fmt, W, rows, cols, x)
    w = gpu_lib.fmt_dequant(fmt, W, rows, cols).double()
    ref = x.double() @ w.T
    err = (clean.double() - ref).norm(dim=1) / ref.norm(dim=1)
    assert float(err.max()) < 1e-6, err
    bad = x.clone()
    bad[2, 5], bad[3, 700], bad[4, 3], bad[4, 900], bad[5, 17] = float("inf"), float("-inf"), float("inf"), float("-inf"), float("nan")
    bad[3, 10:40] = 3e4                     # beside an infinity of the same super-block and of another
    bad[3, 690:699] = -3e4
    got = gpu_lib.fmt_gemv(fmt, W, rows, cols, bad)
    others = [t for t in range(T) if t not in (2, 3, 4, 5)]
    assert torch.equal(got[others], clean[others])
    assert not torch.isfinite(got[2:6]).any()
    if fmt in ("q8_0", "f16"):
        apart = torch.cat([gpu_lib.fmt_gemv(fmt, W, rows, cols, bad[t:t + 1].contiguous()) for t in range(2, 6)])
        assert torch.equal(torch.nan_to_num(got[2:6], 7.0, 8.0, -8.0), torch.nan_to_num(apart, 7.0, 8.0, -8.0))


@pytest.mark.parametrize("T,n_past", [(3, 2500), (5, 700), (9, 300), (16, 70)])
def test_streams_between_launches(gpu_lib, T, n_past):
    """The launches that add the streams' shares: rows of more than 64 super-blocks (their sums of squares take a wave twice), 16 and more
    shares of a short matrix, vectors of 64 rows (a wave's 256 end inside), shares of two formats for gate and up; attention merged there:
    18, 5, 2 and one key range, four heads of 64 columns in a wave."""
    from workloads.configs import ModelDims, WindowConfig
    d = ModelDims(16640, 4, 1, 64, 768, 1e4)
    fm = [{"wq": "q8_0", "wk": "q5_k", "wv": "q5_k", "wo": "q6_k", "wgate": "q5_k", "wup": "q6_k", "wdown": "q6_k"}, {}]
    host = [synth.layer_tensors(WindowConfig("rows", 78, d, 2, T, n_past), l, kv_cap=n_past + T, formats=fm[l]) for l in range(2)]
    x = np.random.default_rng(T).standard_normal((T, d.e)).astype(np.float32)
    dev = [{k: _dev(v) for k, v in t.items()} for t in host]
    ref = oracle.window(d, host, x.astype(np.float64), n_past, formats=fm)
    win = gpu_lib.Window(d, dev, n_past + T, T_max=T, formats=fm)
    win.workspace.fill_(0xFF)
    y = win.decode(_dev(x), n_past).cpu().numpy()
    check_hidden(f"launches between streams, T={T}", rel_err(y, ref), d, host, x.astype(np.float64), n_past, formats=fm, eps=EPS_FP32)



@pytest.mark.parametrize("e,ffn,T", [(512, 65536, 16), (512, 65536, 9), (256, 131072, 16), (2048, 28672, 16)])
def test_many_shares_of_a_product_add_up_no_less_exactly_than_few(gpu_lib, e, ffn, T):
    """A down projection cut into many shares of K, against 64 bits from the activations that the step itself made.  A product's own error
    is 1.3 to 1.45e-7 (activations of 22 bits, fp32 sums along a share); n shares added pairwise put sqrt(log2 n) roundings of 2.4e-8 beside it
    (0.5e-7 for 32: 1.4 to 1.55e-7), one after the other sqrt(n / 2) of them (1e-7: 1.65e-7 and more)."""
    from workloads.configs import ModelDims
    d = ModelDims(e, 4, 1, 64, ffn, 1e4)
    n_past = 70
    rng = np.random.default_rng(e + T)
    dev = {k: _dev(_centred(rng, "q4_k", r, c).reshape(r, c // 256, 144)) for k, (r, c) in _shapes(d).items()}
    for k in ("k_cache", "v_cache"):
        dev[k] = _dev(rng.standard_normal((1, n_past + T, 64)).astype(np.float16))
    for k in ("g_attn", "g_ffn"):
        dev[k] = _dev((1 + 0.1 * rng.standard_normal(e)).astype(np.float32))
    win = gpu_lib.Window(d, [dev], n_past + T, T_max=T)
    x = _dev((1e-3 * rng.standard_normal((T, e))).astype(np.float32))   # (a small residual beside the product)
    y, taps = win.decode_layer_taps(0, x, n_past)
    product = taps["a"].double() @ gpu_lib.q4k_dequant(dev["wdown"]).double().T
    err = float((y.double() - taps["h"].double() - product).norm() / product.norm())
    print("shares", e, ffn, T, err, flush=True)
    assert err < 1.6e-7, err


Q4, Q8, Q6 = {}, {"wdown": "q8_0"}, {"wdown": "q6_k"}
ALL_Q8 = {k: "q8_0" for k in ("wq", "wk", "wo", "wgate", "wup", "wdown", "wv")}


@pytest.mark.parametrize("e,fm,T,n_past,streams", [
    (4352, Q4, 3, 300, False), (4352, Q4, 4, 507, False), (4352, Q4, 4, 508, True), (4096, Q4, 4, 900, False), (4096, Q4, 5, 64, True),
    (2048, Q4, 5, 64, True), (1792, Q4, 8, 600, False), (1792, Q4, 9, 64, True),
    (4352, Q8, 3, 300, False), (4352, Q8, 3, 600, True), (4096, Q8, 3, 600, False), (4096, ALL_Q8, 3, 64, True), (2048, ALL_Q8, 3, 64, False),
    (3072, Q6, 3, 64, True), (2048, Q6, 3, 600, False), (1024, Q6, 5, 100, False)])
def test_from_how_many_tokens_a_layer_takes_the_streams(gpu_lib, e, fm, T, n_past, streams):
    """Which way a layer goes, on both sides of every line of the rule.  V is zero (cache and matrix), so that the attention adds nothing
    and the result depends on the way alone: behind 63 rows the mat-vecs, whose bits the step behind n_past rows has or has not."""
    from workloads.configs import ModelDims, WindowConfig
    d = ModelDims(e, 4, 1, 64, 512, 1e4)
    cap = n_past + T
    t = synth.layer_tensors(WindowConfig("way", 80, d, 1, T, n_past), 0, kv_cap=cap, formats=fm)
    t["wv"] = np.zeros_like(t["wv"])
    t["v_cache"] = np.zeros_like(t["v_cache"])
    win = gpu_lib.Window(d, [{k: _dev(v) for k, v in t.items()}], cap, T_max=T, formats=[fm])
    x = _dev(np.random.default_rng(e + T).standard_normal((T, e)).astype(np.float32))
    vecs, here = win.decode(x, 63).clone(), win.decode(x, n_past)
    assert torch.equal(vecs, here) != streams
    assert rel_err(here.cpu().numpy(), vecs.cpu().numpy().astype(np.float64)) < GEMV_TOL
