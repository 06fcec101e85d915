"""GPU parity of prompt processing (all layers of a window for T consecutive tokens in one call) against the CPU
oracle, through the C ABI.

The oracle advances at most 64 tokens a call; a prompt goes through it in such pieces, each through all layers
(the layers' caches carry what the earlier pieces appended), which is the same causal computation.
Bar: hidden states max relative error <= 2e-3 (tests/metrics.rel_err), appended cache rows within one fp16 step.
"""
import copy
import ctypes

import numpy as np
import pytest
import torch

import oracle
from metrics import rel_err
from tolerance import EPS_FP32, EPS_GEMM, EPS_Q4K, check_hidden
from workloads import synth
from workloads.configs import CONFIGS, TINY, ModelDims, WindowConfig

pytestmark = pytest.mark.gpu

HID_TOL = 2e-3
# the accuracy class of the prompt call's matrix product, asserted on the products themselves in tests/test_gpu_gemm.py
PREFILL_EPS = EPS_GEMM


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _oracle_prompt(dims, host, x, n_past, formats=None):
    out = []
    for t0 in range(0, x.shape[0], 64):
        out.append(oracle.window(dims, host, x[t0:t0 + 64].astype(np.float64), n_past + t0, formats=formats))
    return np.concatenate(out, axis=0)


DECODE_ROUTE = 64   # a threshold that sends these tests' short prompts through the decode kernels (the default is 16)


@pytest.fixture(params=["matrix product", "decode kernels"])
def route(request, gpu_lib):
    """The prompt call's two routes: always the matrix product (threshold 0), or prompts of up to 64 tokens advanced by
    the decode kernels, 16 tokens a call (the library's default does that up to 16 tokens)."""
    gpu_lib.set_prefill_small_tokens(0 if request.param == "matrix product" else DECODE_ROUTE)
    yield request.param
    gpu_lib.set_prefill_small_tokens(gpu_lib.PREFILL_SMALL_TOKENS)


@pytest.fixture
def matrix_product_route(gpu_lib):
    gpu_lib.set_prefill_small_tokens(0)
    yield
    gpu_lib.set_prefill_small_tokens(gpu_lib.PREFILL_SMALL_TOKENS)


def _window(gpu_lib, cfg, cap, host):
    dev_layers = [{k: _dev(v) for k, v in t.items()} for t in host]
    return gpu_lib.Window(cfg.dims, dev_layers, cap, T_max=16), dev_layers


@pytest.mark.parametrize("name,T,n_past", [("t0", 50, 37), ("t1", 70, 0), ("t2", 33, 63), ("t0", 1, 5), ("t1", 16, 130), ("t0", 150, 37),
                                           ("t2", 129, 63)])
def test_prefill_vs_oracle(gpu_lib, route, name, T, n_past):
    cfg = TINY[name].with_(T=T, n_past=n_past)
    cap = n_past + T + 3
    host = [synth.layer_tensors(cfg, l, kv_cap=cap) for l in range(cfg.n_layers)]
    win, dev_layers = _window(gpu_lib, cfg, cap, host)
    x = synth.window_input(cfg)
    print("case", name, T, n_past, flush=True)
    y = win.prefill(_dev(x), n_past).cpu().numpy()
    ref = _oracle_prompt(cfg.dims, host, x, n_past)       # appends to the host caches
    check_hidden(f"prefill {name} T={T} n_past={n_past} ({route})", rel_err(y, ref), cfg.dims, host, x.astype(np.float64), n_past,
                 eps=PREFILL_EPS)
    for l in range(cfg.n_layers):
        for key in ("k_cache", "v_cache"):
            g = dev_layers[l][key].cpu().numpy().astype(np.float64)
            r = host[l][key].astype(np.float64)
            assert np.array_equal(g[:, :n_past], r[:, :n_past])
            assert np.array_equal(g[:, n_past + T:], r[:, n_past + T:])
            if l == 0:   # deeper layers' rows inherit the hidden states' error
                assert rel_err(g[:, n_past:n_past + T].reshape(1, -1), r[:, n_past:n_past + T].reshape(1, -1)) < 1e-3


@pytest.mark.parametrize("name,T,n_past", [("t0", 7, 700), ("t1", 15, 1500), ("t2", 1, 505), ("t2", 12, 4000), ("t2", 1, 9000)])
def test_short_prompts_merge_several_key_ranges_inside_the_launch(gpu_lib, matrix_product_route, name, T, n_past):
    """Fewer than 16 tokens on the matrix-product route: the workgroup of the first key range merges the others' records (2, 5, 1, 15 and 34
    ranges, the last more than one request brings; queries for fewer and for more waves than a workgroup has) and marks them
    for the next layer's launch.  Twice with the same bits: the second call finds the scratch as the first left it."""
    cfg = TINY[name].with_(T=T, n_past=n_past)
    cap = n_past + T
    host = [synth.layer_tensors(cfg, l, kv_cap=cap) for l in range(cfg.n_layers)]
    win, _ = _window(gpu_lib, cfg, cap, host)
    x = synth.window_input(cfg)
    print("case", name, T, n_past, flush=True)
    first = win.prefill(_dev(x), n_past).clone()
    again = win.prefill(_dev(x), n_past)
    assert torch.equal(first, again)
    ref = _oracle_prompt(cfg.dims, host, x, n_past)
    check_hidden(f"short prompt {name} T={T} n_past={n_past}", rel_err(first.cpu().numpy(), ref), cfg.dims, host, x.astype(np.float64), n_past,
                 eps=PREFILL_EPS)


def test_prefill_fills_the_cache_to_its_last_row(gpu_lib, route):
    """n_past + T == kv_cap: the last piece ends on the cache's last row; a token count with full pieces only and one
    with a rest."""
    for T, n_past in [(32, 5), (45, 0)]:
        cfg = TINY["t0"].with_(T=T, n_past=n_past)
        cap = n_past + T
        host = [synth.layer_tensors(cfg, l, kv_cap=cap) for l in range(cfg.n_layers)]
        win, dev_layers = _window(gpu_lib, cfg, cap, host)
        x = synth.window_input(cfg)
        print("case", T, n_past, flush=True)
        y = win.prefill(_dev(x), n_past).cpu().numpy()
        ref = _oracle_prompt(cfg.dims, host, x, n_past)
        assert rel_err(y, ref) < HID_TOL, rel_err(y, ref)
        g = dev_layers[0]["k_cache"].cpu().numpy().astype(np.float64)
        assert rel_err(g[:, n_past:].reshape(1, -1), host[0]["k_cache"][:, n_past:].astype(np.float64).reshape(1, -1)) < 1e-3


MIXES = {
    # the usual mix of a "Q4K" model: V and down projections in Q6_K
    "q4_k_m": [{"wv": "q6_k", "wdown": "q6_k"}, {}, {"wv": "q6_k", "wdown": "q6_k"}],
    # every matrix in some other format, gate / up not both Q4_K (SwiGLU as its own launch), Q4_K matrices alone in their groups
    "all_kinds": [{"wq": "q8_0", "wk": "q5_k", "wv": "f16", "wo": "q6_k", "wgate": "q5_k", "wup": "q8_0", "wdown": "f32"},
                  {"wq": "q6_k", "wgate": "q6_k"},
                  {"wk": "q8_0", "wv": "q8_0", "wup": "f16", "wo": "f16", "wdown": "q5_k"}],
}


@pytest.mark.parametrize("mix", sorted(MIXES))
@pytest.mark.parametrize("name,T,n_past", [("t1", 37, 130), ("t2", 16, 63), ("t0", 70, 37), ("t1", 37, 9), ("t2", 100, 0), ("t0", 32, 5)])
def test_prefill_with_mixed_formats(gpu_lib, route, mix, name, T, n_past):
    """Layers whose matrices are in several formats (Q4_K ones through the matrix product, the others 16 tokens a launch
    through the format mat-vec): hidden state and appended rows against the oracle.  (With 37 tokens behind 9 rows the
    first of these mixes has top-2 logit gaps of 0.03 to 0.1 in every layer: a case for the computed bound.)"""
    base = TINY[name]
    formats = MIXES[mix][-base.n_layers:]
    cfg = base.with_(T=T, n_past=n_past)
    cap = n_past + T + 1
    host = [synth.layer_tensors(cfg, l, kv_cap=cap, formats=formats[l]) for l in range(cfg.n_layers)]
    dev_layers = [{k: _dev(v) for k, v in t.items()} for t in host]
    win = gpu_lib.Window(cfg.dims, dev_layers, cap, T_max=16, formats=formats)
    x = synth.window_input(cfg)
    print("case", mix, name, T, n_past, flush=True)
    y = win.prefill(_dev(x), n_past).cpu().numpy()
    ref = _oracle_prompt(cfg.dims, host, x, n_past, formats)
    check_hidden(f"prefill mixed {mix} {name} T={T} n_past={n_past} ({route})", rel_err(y, ref), cfg.dims, host, x.astype(np.float64), n_past,
                 formats=formats, eps=EPS_FP32)
    g = dev_layers[0]["v_cache"].cpu().numpy().astype(np.float64)
    r = host[0]["v_cache"].astype(np.float64)
    assert rel_err(g[:, n_past:n_past + T].reshape(1, -1), r[:, n_past:n_past + T].reshape(1, -1)) < 1e-3


def _centred(rng, fmt, rows, cols):
    """A matrix of mean about zero and standard deviation about 0.02: every quant uniform, Q4_K / Q5_K sub-mins that put the
    middle of the quants' range at zero on average."""
    W = synth.fmt_tensor(7, 0, int(rng.integers(1 << 20)), fmt, rows, cols)
    n = rows * cols // 256
    if fmt == "f16":
        return (0.02 * rng.standard_normal(rows * cols)).astype(np.float16).view(np.uint8)
    size, mean = {"q4_k": (n, 4e-5), "q5_k": (n, 2e-5), "q6_k": (n, 1.5e-5), "q8_0": (8 * n, 2.7e-4)}[fmt]
    d = (mean * (0.5 + rng.random(size))).astype(np.float16)
    if fmt in ("q4_k", "q5_k"):
        head = W.reshape(n, 144) if fmt == "q4_k" else W[:16 * n].reshape(n, 16)
        head[:, 0:2] = d.view(np.uint8).reshape(n, 2)
        head[:, 2:4] = (d.astype(np.float32) * (7.5 if fmt == "q4_k" else 15.5)).astype(np.float16).view(np.uint8).reshape(n, 2)
    else:
        W[-2 * size:] = d.view(np.uint8)
    return W


def _layer64(gpu_lib, d, fmt, t, x, n_past):
    """A layer in 64 bits from dequantised weights, with the cache rows as the library left them (their rounding to binary16,
    which no product is to blame for, is then the same on both sides)."""
    w = {k: gpu_lib.fmt_dequant(fmt, t[k], *s).double() for k, s in _shapes(d).items()}
    norm = lambda v, g: v * g.double() / torch.sqrt((v * v).mean(1, keepdim=True) + float(np.float32(d.rms_eps)))
    T, D, G = x.shape[0], d.head_dim, d.n_q_heads // d.n_kv_heads
    x = x.double()
    q = (norm(x, t["g_attn"]) @ w["wq"].T).view(T, d.n_q_heads, D)
    ang = torch.arange(n_past, n_past + T, device="cuda").double()[:, None] * float(d.rope_theta) ** (-2.0 * torch.arange(D // 2, device="cuda").double() / D)
    c, s, p, r = torch.cos(ang)[:, None], torch.sin(ang)[:, None], q[..., :D // 2], q[..., D // 2:]
    q = torch.cat([p * c - r * s, p * s + r * c], 2)
    n = n_past + T
    seen = torch.arange(n, device="cuda")[None] <= torch.arange(n_past, n, device="cuda")[:, None]
    o = torch.empty_like(q)
    for h in range(d.n_q_heads):
        k, v = (t[c][h // G, :n].double() for c in ("k_cache", "v_cache"))
        o[:, h] = torch.softmax((q[:, h] @ k.T / D ** 0.5).masked_fill(~seen, -float("inf")), 1) @ v
    h = x + o.view(T, -1) @ w["wo"].T
    a = norm(h, t["g_ffn"])
    g = a @ w["wgate"].T
    return h + (g / (1 + torch.exp(-g)) * (a @ w["wup"].T)) @ w["wdown"].T


def _shapes(d):
    return {"wq": (d.qd, d.e), "wk": (d.kvd, d.e), "wv": (d.kvd, d.e), "wo": (d.e, d.qd), "wgate": (d.ffn, d.e), "wup": (d.ffn, d.e),
            "wdown": (d.e, d.ffn)}


@pytest.mark.parametrize("dist", ["normal", "spread"])
@pytest.mark.parametrize("T", [17, 64, 65, 129, 490])
@pytest.mark.parametrize("fmt", ["q5_k", "q6_k", "q8_0", "f16"])
def test_products_of_the_other_formats_are_no_less_exact_than_the_mat_vec(gpu_lib, fmt, T, dist):
    """One layer with all seven matrices in one format, as one prompt call (matrix product: 64- and 128-token workgroups, ragged
    last ones, rows ragged against 128, K divided and whole) and as decode calls of 3 tokens (the fp32 mat-vec), each against
    64 bits: the prompt's error no larger, both below 1e-6 of what the layer adds.  spread: magnitudes over six decades within a
    token, whose activations share a power of two in a super-block; what is added is then small beside the token and its rounding
    (2^-24 of the token's largest values) is most of the error."""
    d = ModelDims(2560, 20, 5, 128, 8448, 1e5)
    # the tall matrices go through 128-token workgroups from 449 tokens on, all others through 64-token ones; 17, 65 and 129 tokens leave workgroups without tiles
    plan = {n: gpu_lib.fmt_gemm_plan(fmt, T, r, c)[::2] for n, (r, c) in _shapes(d).items()}
    full = T in (64, 490)
    assert plan == {n: (128 if T == 490 and n in ("wgate", "wup") else 64, full) for n in plan}, plan
    _no_less_exact_than_the_mat_vec(gpu_lib, fmt, T, dist, d)


def _no_less_exact_than_the_mat_vec(gpu_lib, fmt, T, dist, d):
    rng = np.random.default_rng(T)
    t = {k: _dev(_centred(rng, fmt, *s)) for k, s in _shapes(d).items()}
    n_past, cap = 64, 64 + T
    t["g_attn"], t["g_ffn"] = (_dev((1 + 0.1 * rng.standard_normal(d.e)).astype(np.float32)) for _ in range(2))
    kv = [_dev(rng.standard_normal((d.n_kv_heads, cap, d.head_dim)).astype(np.float16)) for _ in range(2)]
    x = rng.standard_normal((T, d.e)) * (1 if dist == "normal" else 10 ** rng.uniform(-3, 3, (T, d.e)))
    x = _dev(x.astype(np.float32))
    fm = [{k: fmt for k in _shapes(d)}]
    layers = [dict(t, k_cache=kv[0].clone(), v_cache=kv[1].clone()) for _ in range(2)]
    wins = [gpu_lib.Window(d, [l], cap, formats=fm) for l in layers]
    print("case", fmt, T, dist, flush=True)
    got = wins[0].prefill(x, n_past)
    assert torch.equal(got, wins[0].prefill(x, n_past))
    apart = torch.cat([wins[1].decode(x[i:i + 3].contiguous(), n_past + i).clone() for i in range(0, T, 3)])
    err = []
    for y, l in ((got, layers[0]), (apart, layers[1])):
        ref = _layer64(gpu_lib, d, fmt, l, x, n_past)
        err.append(float((y.double() - ref).norm() / (ref - x.double()).norm()))
    print(f"{err[0]:.3e} {err[1]:.3e}", flush=True)
    assert err[0] <= 1.02 * err[1] and (dist == "spread" or err[1] < 1e-6), err


@pytest.mark.parametrize("T,ffn,blocks", [(333, 11264, 3), (208, 16640, 2)])
@pytest.mark.parametrize("fmt", ["q5_k", "q6_k", "q8_0", "f16"])
def test_workgroups_of_128_tokens_that_lack_some(gpu_lib, fmt, T, ffn, blocks):
    """21 and 13 token tiles of a tall matrix: workgroups of 128 tokens with seven tiles each, or seven and six, the absent ones skipped (waves with
    four tiles beside waves with three, or two groups of three)."""
    d = ModelDims(1024, 8, 2, 128, ffn, 1e5)
    assert gpu_lib.fmt_gemm_plan(fmt, T, ffn, 1024) == (128, blocks, False)
    _no_less_exact_than_the_mat_vec(gpu_lib, fmt, T, "normal", d)


def test_prefill_then_decode_continues(gpu_lib, route):
    """A prompt through the prefill call, the next token through the decode call: against the oracle doing the same."""
    cfg = TINY["t1"].with_(T=40, n_past=0)
    cap = 48
    host = [synth.layer_tensors(cfg, l, kv_cap=cap) for l in range(cfg.n_layers)]
    win, _ = _window(gpu_lib, cfg, cap, host)
    x = synth.window_input(cfg)
    nxt = synth.batch_input(cfg, 1)
    win.prefill(_dev(x), 0)
    y = win.decode(_dev(nxt), 40).cpu().numpy()
    _oracle_prompt(cfg.dims, host, x, 0)
    ref = oracle.window(cfg.dims, host, nxt.astype(np.float64), 40)
    assert rel_err(y, ref) < HID_TOL, rel_err(y, ref)


def test_prefill_agrees_with_decode_calls(gpu_lib, matrix_product_route):
    """The same prompt through decode calls of 16 tokens (integer-digit mat-vec) and through one prefill call
    (binary16 matrix product): far inside the bar of each other, and prefill gives the same bits twice, in place too.
    With the threshold above its length the prompt is advanced by the decode kernels: the same bits as the decode calls."""
    cfg = TINY["t2"].with_(T=48, n_past=10)
    cap = 64
    x = synth.window_input(cfg)
    host = [synth.layer_tensors(cfg, l, kv_cap=cap) for l in range(cfg.n_layers)]
    wa, _ = _window(gpu_lib, cfg, cap, copy.deepcopy(host))
    wb, _ = _window(gpu_lib, cfg, cap, copy.deepcopy(host))
    wc, _ = _window(gpu_lib, cfg, cap, copy.deepcopy(host))
    xd = _dev(x)
    ya = torch.cat([wa.decode(xd[t:t + 16].contiguous(), 10 + t) for t in range(0, 48, 16)]).cpu().numpy()
    yb = wb.prefill(xd, 10)
    assert rel_err(yb.cpu().numpy(), ya.astype(np.float64)) < HID_TOL / 4
    xc = xd.clone()
    yc = wc.prefill(xc, 10, x_out=xc)
    assert torch.equal(yb, yc)
    gpu_lib.set_prefill_small_tokens(DECODE_ROUTE)
    wd, _ = _window(gpu_lib, cfg, cap, copy.deepcopy(host))
    assert np.array_equal(wd.prefill(xd, 10).cpu().numpy(), ya)
    gpu_lib.set_prefill_small_tokens(gpu_lib.PREFILL_SMALL_TOKENS)


@pytest.mark.parametrize("T", [80, 40])
def test_prefill_model_shape_one_layer(gpu_lib, matrix_product_route, T):
    """One 70B-shaped layer (config 3's dimensions), 80 or 40 prompt tokens behind 4000 cached rows.  At these token counts
    the Q/K/V, output and down products divide K among workgroups (6 or 8 shares), at 40 tokens the gate / up product does
    too (2 shares, SwiGLU behind the addition)."""
    cfg = CONFIGS["c3"].with_(T=T, n_past=4000, n_layers=1)
    cap = 4096
    host = [synth.layer_tensors(cfg, 0, kv_cap=cap)]
    win, _ = _window(gpu_lib, cfg, cap, host)
    x = synth.window_input(cfg)
    print(f"case c3 one layer, {T} tokens", flush=True)
    y = win.prefill(_dev(x), 4000).cpu().numpy()
    ref = _oracle_prompt(cfg.dims, host, x, 4000)
    assert rel_err(y, ref) < HID_TOL, rel_err(y, ref)


@pytest.mark.parametrize("mode,T,n_past", [(0, 17, 0), (1, 20, 33), (1, 260, 5)])
def test_the_launches_between_the_products(gpu_lib, matrix_product_route, mode, T, n_past):
    """Three layers of several formats whose products divide K (but for 260 tokens' gate and up): shares added into the rotation, the residual and SwiGLU, and
    laid out for the next layer or not (its Q, K and V in FP32); few and many waves a launch; 20 super-blocks, more than the 16 lanes that add a token's
    sums of squares."""
    d = ModelDims(5120, 10, 5, 128, 2560, 1e4, rope_mode=mode) if mode else ModelDims(5120, 10, 5, 128, 2560, 1e4)
    cfg = WindowConfig("between", 81, d, 3, T, n_past)
    formats = [{"wv": "q6_k", "wk": "q8_0"}, {"wq": "f32", "wk": "f32", "wv": "f32", "wo": "q5_k"}, {"wdown": "f32"}]
    cap = n_past + T
    host = [synth.layer_tensors(cfg, l, kv_cap=cap, formats=formats[l]) for l in range(3)]
    win = gpu_lib.Window(d, [{k: _dev(v) for k, v in t.items()} for t in host], cap, T_max=16, formats=formats)
    x = synth.window_input(cfg)
    print("case", mode, T, n_past, flush=True)
    y = win.prefill(_dev(x), n_past)
    assert torch.equal(y, win.prefill(_dev(x), n_past))
    ref = _oracle_prompt(d, host, x, n_past, formats)
    check_hidden(f"launches between mode={mode} T={T}", rel_err(y.cpu().numpy(), ref), d, host, x.astype(np.float64), n_past, formats=formats, eps=EPS_FP32)


@pytest.mark.parametrize("e,formats", [(8448, {}), (33024, {}), (33024, {"wgate": "q6_k"})])
def test_prompt_of_a_very_wide_model(gpu_lib, matrix_product_route, e, formats):
    """33 and 129 super-blocks a token: more than the 32 and 128 whose sums of squares the launches behind divided products request at first (SwiGLU: 16 lanes a
    token; RoPE, and the sum of a product on its own: a wave)."""
    d = ModelDims(e, 2, 1, 128, 512, 1e4)
    cfg = WindowConfig("wide", 83, d, 1, 17, 5)
    host = [synth.layer_tensors(cfg, 0, kv_cap=22, formats=formats)]
    win = gpu_lib.Window(d, [{k: _dev(v) for k, v in t.items()} for t in host], 22, T_max=16, formats=[formats])
    x = synth.window_input(cfg)
    x[:, -256:] *= 30   # the last super-block's share of the sum of squares is most of it
    print("case", e, formats, flush=True)
    y = win.prefill(_dev(x), 5).cpu().numpy()
    ref = _oracle_prompt(d, host, x, 5, [formats])
    check_hidden(f"wide e={e}", rel_err(y, ref), d, host, x.astype(np.float64), 5, formats=[formats], eps=EPS_GEMM)


@pytest.mark.parametrize("T", [17, 130])
def test_shares_of_k_leave_what_is_still_needed(gpu_lib, matrix_product_route, T):
    """The shares of a product lie in what the layer does not use at that time: three layers (either vector between layers is input and output once), Q, K, V and gate, up
    launched one by one, a gate and up pair whose activations are stored beside the shares (down in FP32) or laid out (down in Q6_K)."""
    d = ModelDims(1024, 8, 2, 128, 2048, 1e4)
    cfg = WindowConfig("shares", 82, d, 3, T, 9)
    formats = [{"wq": "q5_k", "wk": "q8_0", "wv": "q6_k", "wo": "f16", "wgate": "q6_k", "wup": "q8_0", "wdown": "q5_k"}, {"wup": "q5_k", "wdown": "f32"},
               {"wdown": "f32"}]
    for fm in (formats, [{"wdown": "q6_k"}, formats[0], {}]):
        cap = 9 + T
        host = [synth.layer_tensors(cfg, l, kv_cap=cap, formats=fm[l]) for l in range(3)]
        win = gpu_lib.Window(d, [{k: _dev(v) for k, v in t.items()} for t in host], cap, T_max=16, formats=fm)
        x = synth.window_input(cfg)
        print("case", T, fm, flush=True)
        y = win.prefill(_dev(x), 9)
        ref = _oracle_prompt(d, host, x, 9, fm)
        check_hidden(f"shares T={T}", rel_err(y.cpu().numpy(), ref), d, host, x.astype(np.float64), 9, formats=fm, eps=EPS_FP32)
        # a scratch made for a longer prompt gives the same bits
        need = gpu_lib._ffi.lib().prima_prefill_workspace_bytes
        longer = max(need(ctypes.byref(win.dims), win.kv_cap, t) for t in (T, 600))
        win._prefill_ws = torch.empty(longer, dtype=torch.uint8, device="cuda")
        assert torch.equal(y, win.prefill(_dev(x), 9))


def test_prefill_at_the_largest_token_count(gpu_lib):
    """8192 prompt tokens (the call's limit) through one 8B-shaped layer, filling the cache to its last row.  The oracle
    would take hours; checked instead: the first 8176 tokens' outputs are, bit for bit, those of a call with only them
    (no result depends on how many tokens a call has), the last 16 agree with a decode call behind that shorter prompt,
    and the last appended cache rows are the same."""
    cfg = CONFIGS["c0"].with_(T=8192, n_past=0, n_layers=1)
    cap = 8192
    host = [synth.layer_tensors(cfg, 0, kv_cap=cap)]
    x = _dev(synth.window_input(cfg))
    wa, la = _window(gpu_lib, cfg, cap, host)
    wb, lb = _window(gpu_lib, cfg, cap, host)
    print("case c0 one layer, 8192 tokens", flush=True)
    ya = wa.prefill(x, 0)
    yb = wb.prefill(x[:8176].contiguous(), 0)
    yc = wb.decode(x[8176:].contiguous(), 8176)
    assert torch.isfinite(ya).all()
    assert torch.equal(ya[:8176], yb)
    # (a K or V element that rounds to the other fp16 neighbour in one of the two paths moves that token by up to ~1e-3;
    # the others agree to 1e-6)
    per_token = [rel_err(ya[8176 + t].cpu().numpy(), yc[t].cpu().numpy().astype(np.float64)) for t in range(16)]
    assert max(per_token) < HID_TOL and float(np.median(per_token)) < 1e-5, per_token
    for key in ("k_cache", "v_cache"):
        a = la[0][key][:, 8176:].float().cpu().numpy().reshape(1, -1)
        b = lb[0][key][:, 8176:].float().cpu().numpy().astype(np.float64).reshape(1, -1)
        assert rel_err(a, b) < 1e-3
        assert torch.equal(la[0][key][:, :8176], lb[0][key][:, :8176])


@pytest.mark.parametrize("T", [8177, 8185])
def test_prompt_whose_last_piece_does_not_fit_one_grid(gpu_lib, T):
    """128 query heads on one KV head: 511 pieces of 16 tokens are 65408 query groups, one piece more is past the 65535 of a launch's
    grid, so the last, short piece takes a launch of its own.  The full pieces' outputs are those of a call without it, bit for bit;
    the rest agrees with a decode call behind them.  8192 tokens, 512 full pieces, are refused."""
    from paper_2504_08791_amd import _ffi
    d = ModelDims(256, 128, 1, 64, 256, 1e4)
    cfg = WindowConfig("heads", 79, d, 1, 8192, 0)
    cap = 8192
    host = [synth.layer_tensors(cfg, 0, kv_cap=cap)]
    x = _dev(synth.window_input(cfg))
    wa, la = _window(gpu_lib, cfg, cap, host)
    wb, lb = _window(gpu_lib, cfg, cap, host)
    print("case 128 heads,", T, "tokens", flush=True)
    ya = wa.prefill(x[:T].contiguous(), 0)
    yb = wb.prefill(x[:8176].contiguous(), 0)
    yc = wb.decode(x[8176:T].contiguous(), 8176)
    assert torch.equal(ya[:8176], yb)
    per_token = [rel_err(ya[8176 + t].cpu().numpy(), yc[t].cpu().numpy().astype(np.float64)) for t in range(T - 8176)]
    assert max(per_token) < HID_TOL, per_token
    assert torch.equal(la[0]["v_cache"][:, :8176], lb[0]["v_cache"][:, :8176])
    with pytest.raises(_ffi.PrimaError):
        wa.prefill(x, 0)


def test_prefill_argument_errors(gpu_lib):
    from paper_2504_08791_amd import _ffi
    import ctypes as C
    cfg = TINY["t0"]
    cap = 64
    host = [synth.layer_tensors(cfg, l, kv_cap=cap) for l in range(cfg.n_layers)]
    win, _ = _window(gpu_lib, cfg, cap, host)
    L = _ffi.lib()
    x = torch.zeros((8, cfg.dims.e), dtype=torch.float32, device="cuda")
    need = L.prima_prefill_workspace_bytes(C.byref(win.dims), cap, 8)
    assert need > 0 and L.prima_prefill_workspace_bytes(C.byref(win.dims), cap, 0) == 0
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    call = lambda **k: L.prima_layer_window_prefill(C.byref(win.dims), win._arr, k.get("L", 2), cap, k.get("n_past", 0), k.get("T", 8),
                                                    k.get("x", x.data_ptr()), x.data_ptr(), ws.data_ptr(), k.get("wsb", need), None)
    assert _ffi.STATUS[call(x=None)] == "PRIMA_E_NULL"
    assert _ffi.STATUS[call(T=0)] == "PRIMA_E_RANGE"
    assert _ffi.STATUS[call(n_past=60)] == "PRIMA_E_RANGE"
    assert _ffi.STATUS[call(L=0)] == "PRIMA_E_RANGE"
    assert _ffi.STATUS[call(wsb=need - 256)] == "PRIMA_E_WORKSPACE"
    assert _ffi.STATUS[call(x=x.data_ptr() + 4)] == "PRIMA_E_ALIGN"
    assert call() == 0
    torch.cuda.synchronize()
