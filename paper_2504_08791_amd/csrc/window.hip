// C-ABI entry points: argument validation on the host, workspace carving and the per-layer
// launch sequence of a layer window (arXiv 2504.08791, Sec. 3.1: a device advances its window
// of consecutive layers and hands e FP32 values per token to its successor).
#include <algorithm>
#include <initializer_list>
#include <mutex>

#include "attn_common.h"
#include "tok_stream.h"

using namespace prima;

namespace {

struct WindowWs {
    size_t q, k, v, o, h, a, u, xb0, xb1, rope, attn, gemv, gemv_bytes, arrivals_bytes, total;
    // 4 and more tokens: activations laid out for Q4_K and for the other formats, their sums of squares, the shares of K
    size_t tok_rec[2], tok_ss, tok_part, tok_part_floats;
};

bool dims_ok(const prima_dims *d)
{
    return d->e > 0 && d->e % QK == 0 && d->ffn > 0 && d->ffn % QK == 0 && d->n_kv_heads > 0 &&
           d->n_q_heads > 0 && d->n_q_heads % d->n_kv_heads == 0 && (d->head_dim == 64 || d->head_dim == 128) &&
           (static_cast<int64_t>(d->n_q_heads) * d->head_dim) % QK == 0 && (d->rope_mode == 0 || d->rope_mode == 1);
}

// Layers of several tokens go through tok_stream.hip, its launches between the streams included, from so many tokens on; it has four launches a layer
// more than run_layer() (five behind fewer than 512 rows, where that has no merge of key ranges), which narrow models and few tokens feel.
// Windows, us, run_layer() / there:
// 5 to 8 tokens, a hidden size of 2048 and more: 4 to 16 % whatever the formats and the rows.  Four layers of 2048 behind 64 rows 5: 224 / 214, 8: 244 / 222, behind
// 2000 5: 241 / 226; 8B, three layers, 64 5: 261 / 233, 2000 8: 281 / 244; 70B, two, 64 5: 332 / 290, 2000 8: 343 / 302; down in Q8_0 in every other layer, 2048, 64 5:
// 237 / 223, 14B, two, 64 5: 198 / 174; 8 sequences through two 14B layers 214 / 188.  Narrower, six layers of 1024 behind 64 rows: V and down in
// Q6_K in every other one 5: 260 / 263, 6: 269 / 267, 7: 253 / 267, 8: 273 / 270, down in Q8_0 5: 234 / 248, 8: 241 / 255, four matrices in Q5_K and Q6_K 6: 301 / 282, 7: 272 / 284.
// 3 and 4 tokens, Q4_K: 8B as fast either way (2000 3: 236 / 236).  14B, two layers, 64 3: 169 / 169, 500: 178 / 170, 2000: 178 / 174, 8000: 180 / 177; 32B, two, 64
// 3: 213 / 219, 4: 215 / 221, 300 3: 217 / 221, 500: 223 / 221, 2000: 223 / 221, 8000: 224 / 227; 70B, two, 130 3: 288 / 296, 4: 297 / 298, 300 3: 292 / 296, 1000: 297 / 295, 4:
// 304 / 302, 4096 4: 305 / 299: from 512 rows on, within 2 % (32B) or faster, and more exact (below).  Down in Q8_0 as with Q4_K alone: 8B, three, 64 3: 241 / 245, 4:
// 240 / 249; 3072, four, 64 3: 230 / 240; 14B, two, 64 4: 177 / 179, 500 3: 186 / 173.  Every matrix in Q8_0: 14B 64 3: 270 / 218, 3072, four 349 / 305.
// Other formats, 3 tokens, 64 rows: V and down in Q6_K in every other layer 3072 254 / 251, 8B 272 / 257, 14B 190 / 180, 70B 340 / 312; down in FP16 3072 281 / 249,
// 8B 309 / 265 (4 tokens 262 / 268); 2048, eight layers, 1000 rows, Q6_K as above 441 / 467.
// Error against 64 bits (2-norm of the result, the reference attending to the step's own cache rows, so that no rounding of a cache element that goes the other
// way is counted; median of 8 inputs, 1e-7): Q4_K, 8B, two layers, 5 tokens behind 70 rows 5.6 / 4.3, 2047 5.0 / 3.7; 14B, two, 3: 70 6.7 / 4.8, 2047 5.6 / 3.8, 8000 5.4 / 3.7;
// 32B, one, 4: 70 5.3 / 3.9, 2047 4.4 / 2.9, 8000 4.1 / 2.8; 70B, one, 3: 70 6.3 / 5.1, 2047 5.7 / 4.4; 14B with Q6_K as above 3: 2047 5.8 / 3.9, with Q8_0 5.3 / 3.8; no case of 3 to 8 tokens
// was less exact there.  (Weights far from mean zero, which no case has: 0.7 to 1.0 / 1.0 to 1.2 a product, see tok_common.h.)
// K long enough to need hundreds of slabs and layers with an FP32 matrix go through run_layer().
constexpr int TOK_LEAST = 3; // (the scratch has a region for the streams from here on)
// others: a matrix in another format than Q4_K and Q8_0, or none in Q4_K; rows: of the longest sequence behind the step
int tok_from(const prima_dims &d, bool others, int rows)
{
    if (others ? d.e >= 3072 : d.e > 4096 && rows >= 512) return TOK_LEAST;
    return d.e >= 2048 ? 5 : 9;
}
// In run_layer(), tokens from which the matrices in other formats go through streams of their own.  Two layers, V
// and down in Q6_K in one of them, us, there / through a mat-vec for each: 14B shape 4 tokens 213 / 221, 5: 230 / 248, 8: 236 / 290.
constexpr int TOK_OTHERS = 4;
// A group of these matrices takes a launch in front of its streams (one per format) and one behind, the mat-vecs one per matrix.  Up to
// 7 tokens a launch more pays from about this many weights on.  Two layers, us, mat-vecs / streams, 4 tokens: hidden size 512, V
// and down in Q6_K 86 / 99, V in Q5_K too 103 / 119; 2048, V in FP16 128 / 129; 4096, V in FP16 192 / 187, all in Q8_0 295 / 251.
constexpr int64_t TOK_LAUNCH_WEIGHTS = int64_t{1} << 21;
// One sequence behind fewer cached rows than this keeps the mat-vecs, so that its results stay what they were, bit for bit; it is neither
// the faster nor the more exact way.  Three 8B-shaped layers, mat-vecs / streams: 16 tokens behind 9 rows 486 / 299 us, median error
// of 40 inputs against 64 bits 4.1e-5 / 3.5e-5; 13 behind 1 row 482 / 293 us, 5.9e-5 / 5.5e-5; 13 behind 40 rows 483 / 297 us, 2.0e-5 /
// 1.8e-5.  Where a token sees few keys, one rounding of an appended K or V element to binary16 that goes the other way is felt in
// every later layer: the two ways' deeper cache rows differ by up to 1.5e-4 behind 1 to 9 rows and 6e-5 behind 40, and a caller who
// holds a step to an earlier one at 1e-4 would see them change.  (A batch appends one row per sequence; its steps differ by less.)
constexpr int TOK_MIN_ROWS = 64;
bool tok_context(int n_past, const AttnSeqs *seq) { return seq || n_past >= TOK_MIN_ROWS; }
// Whether these dimensions have a region for the streams in their scratch: a rule on the widths alone, so that scratch sized for
// more tokens holds what fewer need (with the token slots in it, K beyond 131072 had a region for 4 to 8 tokens and none for 9 to 16).
bool tok_dims(const prima_dims &d)
{
    const int64_t qd = static_cast<int64_t>(d.n_q_heads) * d.head_dim, widest = std::max<int64_t>({d.e, qd, d.ffn});
    return widest / QK <= 1024 && tok_max_parts(static_cast<int>(widest / QK), tok_slots(PRIMA_MAX_TOK), 1) <= 256 &&
           (2 * static_cast<int64_t>(d.ffn) + qd + 2 * static_cast<int64_t>(d.n_kv_heads) * d.head_dim) < (int64_t{1} << 30);
}
// ... and whether a step of T tokens on this scratch uses it
bool tok_takes(const WindowWs &w, int T, int from) { return T >= from && w.tok_part_floats != 0; }

WindowWs carve(const prima_dims &d, int kv_cap, int T)
{
    WindowWs w{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += round_up(bytes, 256); return o; };
    const size_t qd = static_cast<size_t>(d.n_q_heads) * d.head_dim, kvd = static_cast<size_t>(d.n_kv_heads) * d.head_dim;
    const size_t f = sizeof(float);
    w.q = take(T * qd * f);
    w.k = take(T * kvd * f);
    w.v = take(T * kvd * f);
    w.o = take(T * qd * f);
    w.h = take(T * static_cast<size_t>(d.e) * f);
    w.a = take(T * static_cast<size_t>(d.ffn) * f);
    w.u = take(T * static_cast<size_t>(d.ffn) * f); // up projection, when gate / up are not both Q4_K
    w.xb0 = take(T * static_cast<size_t>(d.e) * f);
    w.xb1 = take(T * static_cast<size_t>(d.e) * f);
    w.rope = take(T * static_cast<size_t>(d.head_dim) * f);
    w.attn = take(attn_ws_bytes(d, kv_cap, T));
    // mat-vec scratch: sized for the largest of the layer's (and the output layer's) launches
    const int64_t rows_max = std::max<int64_t>({2 * static_cast<int64_t>(d.ffn), static_cast<int64_t>(qd + 2 * kvd), static_cast<int64_t>(d.e)});
    // (the last five: subsets of a group, launched when its other matrices are in other formats)
    const int64_t shapes[9][2] = {{static_cast<int64_t>(qd + 2 * kvd), d.e}, {d.e, static_cast<int64_t>(qd)}, {2 * static_cast<int64_t>(d.ffn), d.e}, {d.e, d.ffn},
                                  {static_cast<int64_t>(qd), d.e}, {static_cast<int64_t>(kvd), d.e}, {static_cast<int64_t>(qd + kvd), d.e},
                                  {static_cast<int64_t>(2 * kvd), d.e}, {d.ffn, d.e}};
    w.gemv_bytes = 0;
    w.arrivals_bytes = gemv_arrivals_bytes(rows_max);
    for (const auto &sh : shapes) w.gemv_bytes = std::max(w.gemv_bytes, gemv_ws_bytes(sh[0], sh[1], T)); // counters + partial sums
    w.gemv_bytes += w.arrivals_bytes; // the counter region is sized for the tallest matrix
    // The shares of the streams lie where the mat-vec keeps its partial sums, behind its counters (which a step needs cleared): a launch of
    // one kind has used up its own before one of the other kind starts.
    size_t region = w.gemv_bytes;
    const bool tok = T >= TOK_LEAST && tok_dims(d);
    if (tok) {
        auto floats = [&](size_t rows, int64_t cols) { return tok_part_floats(static_cast<int64_t>(rows), cols, T); };
        w.tok_part_floats = std::max({floats(qd, d.e) + 2 * floats(kvd, d.e), floats(d.e, static_cast<int64_t>(qd)), 2 * floats(d.ffn, d.e), floats(d.e, d.ffn)});
        region = std::max(region, round_up(w.arrivals_bytes, 256) + w.tok_part_floats * sizeof(float));
    }
    w.gemv = take(region);
    w.tok_part = w.gemv + round_up(w.arrivals_bytes, 256);
    if (tok) {
        const int64_t widest = std::max<int64_t>({d.e, static_cast<int64_t>(qd), d.ffn});
        for (size_t &r : w.tok_rec) r = take(tok_rec_bytes(widest, T));
        w.tok_ss = take(tok_ss_bytes(d.e, T));
    }
    w.total = off;
    return w;
}

template <class P> P *at(void *ws, size_t off) { return reinterpret_cast<P *>(static_cast<char *>(ws) + off); }

GemvSeg seg(const void *W, float *y, int64_t rows, int64_t ldy, const float *resid = nullptr, int64_t ldr = 0)
{
    return GemvSeg{static_cast<const uint8_t *>(W), y, resid, rows, ldy, ldr};
}

prima_status check_layer(const prima_layer &l, bool with_caches = true)
{
    const void *ptrs[] = {l.wq, l.wk, l.wv, l.wo, l.wgate, l.wup, l.wdown, l.g_attn, l.g_ffn,
                          with_caches ? l.k_cache : l.wq, with_caches ? l.v_cache : l.wq};
    for (const void *p : ptrs) {
        if (!p) return PRIMA_E_NULL;
        if (!aligned(p, 16)) return PRIMA_E_ALIGN;
    }
    return PRIMA_OK;
}

GemvArgs gemv_args(int nseg, int64_t n_cols, const float *x, int64_t ldx, int T, int xmode = X_PLAIN,
                   const float *gain = nullptr, float eps = 0.f, int epi = EPI_ROWS)
{
    GemvArgs ga{};
    ga.nseg = nseg; ga.n_cols = n_cols; ga.x = x; ga.ldx = ldx; ga.T = T;
    ga.xmode = xmode; ga.epi = epi; ga.gain = gain; ga.eps = eps;
    return ga;
}

// the four projections of a layer as mat-vec arguments, in launch order (Q/K/V, output, gate/up, down)
void layer_gemv_args(const prima_dims &d, const prima_layer &L, int T, const float *x, float *y, void *ws, const WindowWs &w, GemvArgs ga[4])
{
    const int64_t e = d.e, qd = static_cast<int64_t>(d.n_q_heads) * d.head_dim, kvd = static_cast<int64_t>(d.n_kv_heads) * d.head_dim, F = d.ffn;
    float *q = at<float>(ws, w.q), *k = at<float>(ws, w.k), *v = at<float>(ws, w.v);
    float *o = at<float>(ws, w.o), *h = at<float>(ws, w.h), *act = at<float>(ws, w.a);
    ga[0] = gemv_args(3, e, x, e, T, X_RMSNORM, L.g_attn, d.rms_eps);
    ga[0].seg[0] = seg(L.wq, q, qd, qd);
    ga[0].seg[1] = seg(L.wk, k, kvd, kvd);
    ga[0].seg[2] = seg(L.wv, v, kvd, kvd);
    ga[1] = gemv_args(1, qd, o, qd, T);
    ga[1].seg[0] = seg(L.wo, h, e, e, x, e);
    ga[2] = gemv_args(2, e, h, e, T, X_RMSNORM, L.g_ffn, d.rms_eps, EPI_SWIGLU);
    ga[2].seg[0] = seg(L.wgate, act, F, F); // silu(gate) * up lands here
    ga[2].seg[1] = seg(L.wup, nullptr, F, F);
    ga[3] = gemv_args(1, F, act, F, T);
    ga[3].seg[0] = seg(L.wdown, y, e, e, h, e);
}

// prompts of up to this many tokens go through the decode kernels, PRIMA_MAX_TOK tokens a call (measured on config 3's shape,
// ms per layer, matrix-product route / decode route: 8 tokens 0.39 / 0.19, 16: 0.38 / 0.37, 24: 0.40 / 0.56, 32: 0.40 / 0.73,
// 64: 0.43 / 1.46, 128: 0.60 / 2.93, 256: 1.04 / 5.87).  A process-wide setting, read when a prompt call is enqueued.
int g_prefill_small_tokens = 16;

// The matrices of a group with their activations already laid out in the scratch: one stream per format; out[i]: where the
// shares of matrix i lie.
prima_status tok_streams(const TokMat *m, const int *fmt, int count, int64_t cols, int T, void *ws, const WindowWs &w, TokPart *out, hipStream_t st)
{
    float *const part = at<float>(ws, w.tok_part);
    size_t used = 0;
    for (int i = 0; i < count; ++i) {
        bool first = true;
        for (int j = 0; j < i; ++j) first = first && fmt[j] != fmt[i];
        if (!first) continue;
        TokMat same[3];
        TokPart parts[3];
        int at_i[3], c = 0;
        for (int j = i; j < count; ++j)
            if (fmt[j] == fmt[i]) { same[c] = m[j]; at_i[c++] = j; }
        const uint8_t *rec = at<uint8_t>(ws, w.tok_rec[fmt[i] == PRIMA_FMT_Q4_K ? 0 : 1]);
        const prima_status s = launch_tok_stream(fmt[i], same, c, cols, rec, T, part + used, w.tok_part_floats - used, parts, st);
        if (s != PRIMA_OK) return s;
        for (int j = 0; j < c; ++j) out[at_i[j]] = parts[j];
        used += static_cast<size_t>(parts[0].n_parts) * T * static_cast<size_t>(parts[0].rows);
    }
    return PRIMA_OK;
}

// one decoder layer; x -> y (fp32 [T][e]); taps may be null.  Six launches: Q/K/V projections
// (RMSNorm fused), attention (RoPE + KV append fused), the merge of its key ranges (none with one range), output projection
// (+ residual), gate/up projections (RMSNorm fused in front, SwiGLU behind), down projection (+ residual).
prima_status run_layer(const prima_dims &d, const prima_layer &L, int kv_cap, int n_past, int T,
                       const float *x, float *y, void *ws, const WindowWs &w, hipStream_t st,
                       float *tap_q, float *tap_o, float *tap_h, float *tap_a, int only = -1, const AttnSeqs *seq = nullptr,
                       const prima_layer_formats *fm = nullptr)
{
    // fm: formats of the seven matrices (null: all Q4_K).  Q4_K matrices go through the MFMA mat-vec (those of one
    // group in one launch), the others through the format mat-vec, one launch each, with the same fused RMSNorm /
    // residual; SwiGLU is a launch of its own unless gate and up are both Q4_K.
    const int f_q = fm ? fm->wq : 0, f_k = fm ? fm->wk : 0, f_v = fm ? fm->wv : 0, f_o = fm ? fm->wo : 0;
    const int f_g = fm ? fm->wgate : 0, f_u = fm ? fm->wup : 0, f_d = fm ? fm->wdown : 0;
    auto other = [&](int fmt, const void *W, int64_t rows, int64_t cols, const float *xin, const float *gain,
                     const float *resid, float *out) {
        return launch_fmt_gemv(fmt, static_cast<const uint8_t *>(W), rows, cols, xin, cols, T, gain, d.rms_eps, resid, rows, out, rows, st,
                               tok_context(n_past, seq));
    };
    // The matrices of a group in other formats than Q4_K, n of them.  From TOK_OTHERS tokens on all but FP32 through the weight
    // streams of tok_stream.hip (activations laid out, streamed, shares added), else a format mat-vec each.
    struct Other { int fmt; const void *W; int64_t rows; float *out; };
    auto others = [&](const Other *m, int n, int64_t cols, const float *xin, const float *gain, const float *resid) -> prima_status {
        TokMat mats[3];
        int n_tok = 0, fmts[3];
        TokSum sum{};
        bool tok = tok_takes(w, T, TOK_OTHERS) && tok_context(n_past, seq);
        if (T < 8) { // the streams' launches more than the mat-vecs', against what they save on the weights
            int64_t weights = 0;
            int n_fmt = 0, n_mats = 0;
            for (int i = 0; i < n; ++i) {
                if (m[i].fmt == PRIMA_FMT_F32) continue;
                bool seen = false;
                for (int j = 0; j < i; ++j) seen = seen || m[j].fmt == m[i].fmt;
                n_fmt += !seen;
                ++n_mats;
                weights += m[i].rows * cols;
            }
            tok = tok && weights >= TOK_LAUNCH_WEIGHTS * (2 + n_fmt - n_mats);
        }
        for (int i = 0; i < n; ++i) {
            if (!tok || m[i].fmt == PRIMA_FMT_F32) {
                const prima_status ps = other(m[i].fmt, m[i].W, m[i].rows, cols, xin, gain, resid, m[i].out);
                if (ps != PRIMA_OK) return ps;
                continue;
            }
            mats[n_tok] = TokMat{static_cast<const uint8_t *>(m[i].W), m[i].rows};
            sum.rows[n_tok] = m[i].rows;
            sum.y[n_tok] = m[i].out;
            fmts[n_tok++] = m[i].fmt;
        }
        if (n_tok == 0) return PRIMA_OK;
        TokPrepare a{};
        a.mode = TOK_PLAIN; a.T = T; a.nb = static_cast<int>(cols / QK); a.x = xin; a.gain = gain; a.ss = at<float>(ws, w.tok_ss);
        a.rec[1] = at<uint8_t>(ws, w.tok_rec[1]);
        prima_status ps = launch_tok_prepare(a, StepInit{}, st);
        if (ps != PRIMA_OK) return ps;
        ps = tok_streams(mats, fmts, n_tok, cols, T, ws, w, sum.p, st);
        if (ps != PRIMA_OK) return ps;
        sum.n = n_tok; sum.T = T; sum.nt = tok_slots(T); sum.resid = resid;
        if (gain) sum.norm = TokNorm{a.ss, a.nb, d.rms_eps};
        return launch_tok_sum(sum, st);
    };
    const int64_t e = d.e, qd = static_cast<int64_t>(d.n_q_heads) * d.head_dim, kvd = static_cast<int64_t>(d.n_kv_heads) * d.head_dim, F = d.ffn;
    float *q = at<float>(ws, w.q), *k = at<float>(ws, w.k), *v = at<float>(ws, w.v);
    float *o = at<float>(ws, w.o), *h = at<float>(ws, w.h), *act = at<float>(ws, w.a);
    prima_status s;
#define PRIMA_TRY(call) do { s = (call); if (s != PRIMA_OK) return s; } while (0)
#define PRIMA_WANT(k) (only < 0 || only == (k))
    if (PRIMA_WANT(PRIMA_K_QKV)) {
        GemvArgs ga = gemv_args(0, e, x, e, T, X_RMSNORM, L.g_attn, d.rms_eps);
        if (f_q == PRIMA_FMT_Q4_K) ga.seg[ga.nseg++] = seg(L.wq, q, qd, qd);
        if (f_k == PRIMA_FMT_Q4_K) ga.seg[ga.nseg++] = seg(L.wk, k, kvd, kvd);
        if (f_v == PRIMA_FMT_Q4_K) ga.seg[ga.nseg++] = seg(L.wv, v, kvd, kvd);
        if (ga.nseg) PRIMA_TRY(launch_gemv_mfma(ga, at<char>(ws, w.gemv), w.gemv_bytes, w.arrivals_bytes, st));
        Other m[3];
        int n = 0;
        if (f_q != PRIMA_FMT_Q4_K) m[n++] = Other{f_q, L.wq, qd, q};
        if (f_k != PRIMA_FMT_Q4_K) m[n++] = Other{f_k, L.wk, kvd, k};
        if (f_v != PRIMA_FMT_Q4_K) m[n++] = Other{f_v, L.wv, kvd, v};
        PRIMA_TRY(others(m, n, e, x, L.g_attn, nullptr));
    }
    if (PRIMA_WANT(PRIMA_K_ATTN))
        PRIMA_TRY(launch_attn(d, q, tap_q, k, v, at<float>(ws, w.rope), static_cast<__half *>(L.k_cache),
                              static_cast<__half *>(L.v_cache), kv_cap, n_past, T, o, at<char>(ws, w.attn), st, seq,
                              ATTN_MERGE_APART));
    if (tap_o && hipMemcpyAsync(tap_o, o, T * qd * sizeof(float), hipMemcpyDeviceToDevice, st) != hipSuccess) return PRIMA_E_DEVICE;
    if (PRIMA_WANT(PRIMA_K_WO)) {
        if (f_o == PRIMA_FMT_Q4_K) {
            GemvArgs ga = gemv_args(1, qd, o, qd, T);
            ga.seg[0] = seg(L.wo, h, e, e, x, e);
            PRIMA_TRY(launch_gemv_mfma(ga, at<char>(ws, w.gemv), w.gemv_bytes, w.arrivals_bytes, st));
        } else {
            const Other m{f_o, L.wo, e, h};
            PRIMA_TRY(others(&m, 1, qd, o, nullptr, x));
        }
    }
    if (tap_h && hipMemcpyAsync(tap_h, h, T * e * sizeof(float), hipMemcpyDeviceToDevice, st) != hipSuccess) return PRIMA_E_DEVICE;
    if (PRIMA_WANT(PRIMA_K_GATE_UP)) {
        if (f_g == PRIMA_FMT_Q4_K && f_u == PRIMA_FMT_Q4_K) {
            GemvArgs ga = gemv_args(2, e, h, e, T, X_RMSNORM, L.g_ffn, d.rms_eps, EPI_SWIGLU);
            ga.seg[0] = seg(L.wgate, act, F, F); // silu(gate) * up lands here
            ga.seg[1] = seg(L.wup, nullptr, F, F);
            PRIMA_TRY(launch_gemv_mfma(ga, at<char>(ws, w.gemv), w.gemv_bytes, w.arrivals_bytes, st));
        } else {
            float *up = at<float>(ws, w.u);
            const void *Wm[2] = {L.wgate, L.wup};
            float *out[2] = {act, up};
            const int fmt2[2] = {f_g, f_u};
            Other m[2];
            int n = 0;
            for (int i = 0; i < 2; ++i) {
                if (fmt2[i] == PRIMA_FMT_Q4_K) {
                    GemvArgs ga = gemv_args(1, e, h, e, T, X_RMSNORM, L.g_ffn, d.rms_eps);
                    ga.seg[0] = seg(Wm[i], out[i], F, F);
                    PRIMA_TRY(launch_gemv_mfma(ga, at<char>(ws, w.gemv), w.gemv_bytes, w.arrivals_bytes, st));
                } else {
                    m[n++] = Other{fmt2[i], Wm[i], F, out[i]};
                }
            }
            PRIMA_TRY(others(m, n, e, h, L.g_ffn, nullptr));
            PRIMA_TRY(launch_swiglu(act, up, static_cast<int64_t>(T) * F, st));
        }
    }
    if (tap_a && hipMemcpyAsync(tap_a, act, T * F * sizeof(float), hipMemcpyDeviceToDevice, st) != hipSuccess) return PRIMA_E_DEVICE;
    if (PRIMA_WANT(PRIMA_K_DOWN)) {
        if (f_d == PRIMA_FMT_Q4_K) {
            GemvArgs ga = gemv_args(1, F, act, F, T);
            ga.seg[0] = seg(L.wdown, y, e, e, h, e);
            PRIMA_TRY(launch_gemv_mfma(ga, at<char>(ws, w.gemv), w.gemv_bytes, w.arrivals_bytes, st));
        } else {
            const Other m{f_d, L.wdown, e, y};
            PRIMA_TRY(others(&m, 1, F, act, nullptr, h));
        }
    }
#undef PRIMA_WANT
#undef PRIMA_TRY
    return PRIMA_OK;
}

// One decoder layer for several tokens (tok_stream.hip), x -> y.  Launches: the weight streams (one per format in a group), and
// between them one that adds their shares, finishes the vector and lays it out for the next stream.  prepared: the layer
// before this one has laid out x for the Q/K/V streams; next: the layer after it, whose Q/K/V activations the last launch
// lays out (null: none); init: done by the first launch (tab null: done before; not with prepared).  Every matrix in a format that the streams take.
prima_status run_layer_tok(const prima_dims &d, const prima_layer &L, int kv_cap, int n_past, int T,
                           const float *x, float *y, void *ws, const WindowWs &w, hipStream_t st,
                           float *tap_q, float *tap_o, float *tap_h, float *tap_a, int only, const AttnSeqs *seq,
                           const prima_layer_formats *fm, bool prepared, const prima_layer *next, const prima_layer_formats *next_fm,
                           const StepInit &init = StepInit{})
{
    static constexpr prima_layer_formats ALL_Q4_K = {0, 0, 0, 0, 0, 0, 0};
    const prima_layer_formats &f = fm ? *fm : ALL_Q4_K, &nf = next_fm ? *next_fm : ALL_Q4_K;
    const int64_t e = d.e, qd = static_cast<int64_t>(d.n_q_heads) * d.head_dim, kvd = static_cast<int64_t>(d.n_kv_heads) * d.head_dim, F = d.ffn;
    float *q = at<float>(ws, w.q), *k = at<float>(ws, w.k), *v = at<float>(ws, w.v), *o = at<float>(ws, w.o), *h = at<float>(ws, w.h);
    float *const ss = at<float>(ws, w.tok_ss);
    prima_status s;
#define PRIMA_TRY(call) do { s = (call); if (s != PRIMA_OK) return s; } while (0)
#define PRIMA_WANT(k) (only < 0 || only == (k))
    auto streams = [&](const TokMat *m, const int *fmt, int count, int64_t cols, TokPart *out) { return tok_streams(m, fmt, count, cols, T, ws, w, out, st); };
    auto prepare = [&](int mode, int64_t cols, const float *gain, std::initializer_list<int> fmts) {
        TokPrepare a{};
        a.mode = mode; a.T = T; a.nb = static_cast<int>(cols / QK); a.gain = gain; a.ss = ss;
        for (int ff : fmts) a.rec[ff == PRIMA_FMT_Q4_K ? 0 : 1] = at<uint8_t>(ws, w.tok_rec[ff == PRIMA_FMT_Q4_K ? 0 : 1]);
        return a;
    };
    const TokNorm norm{ss, static_cast<int>(e / QK), d.rms_eps};
    auto W = [](const void *p) { return static_cast<const uint8_t *>(p); };

    if (PRIMA_WANT(PRIMA_K_QKV)) {
        if (!prepared) {
            TokPrepare a = prepare(TOK_PLAIN, e, L.g_attn, {f.wq, f.wk, f.wv});
            a.x = x;
            PRIMA_TRY(launch_tok_prepare(a, init, st));
        }
        const TokMat m[3] = {{W(L.wq), qd}, {W(L.wk), kvd}, {W(L.wv), kvd}};
        const int fmts[3] = {f.wq, f.wk, f.wv};
        TokSum a{3, T, tok_slots(T), {}, {qd, kvd, kvd}, {q, k, v}, norm, nullptr};
        PRIMA_TRY(streams(m, fmts, 3, e, a.p));
        PRIMA_TRY(launch_tok_sum(a, st));
    }
    if (PRIMA_WANT(PRIMA_K_ATTN))
        PRIMA_TRY(launch_attn(d, q, tap_q, k, v, at<float>(ws, w.rope), static_cast<__half *>(L.k_cache),
                              static_cast<__half *>(L.v_cache), kv_cap, n_past, T, o, at<char>(ws, w.attn), st, seq, ATTN_MERGE_LATER));
    if (PRIMA_WANT(PRIMA_K_WO)) {
        const AttnRecords rec = attn_records(d, n_past, T, at<char>(ws, w.attn), seq);
        TokPrepare a = prepare(rec.nsplit == 1 ? TOK_PLAIN : TOK_ATTENTION, qd, nullptr, {f.wo});
        a.x = o;
        a.att = rec;
        a.D = d.head_dim;
        a.out = tap_o && rec.nsplit != 1 ? o : nullptr;
        PRIMA_TRY(launch_tok_prepare(a, StepInit{}, st));
        if (tap_o && hipMemcpyAsync(tap_o, o, T * qd * sizeof(float), hipMemcpyDeviceToDevice, st) != hipSuccess) return PRIMA_E_DEVICE;
        const TokMat m{W(L.wo), e};
        a = prepare(TOK_RESIDUAL, e, L.g_ffn, {f.wgate, f.wup});
        PRIMA_TRY(streams(&m, &f.wo, 1, qd, a.p));
        a.x = x;
        a.out = h;
        PRIMA_TRY(launch_tok_prepare(a, StepInit{}, st));
    }
    if (tap_h && hipMemcpyAsync(tap_h, h, T * e * sizeof(float), hipMemcpyDeviceToDevice, st) != hipSuccess) return PRIMA_E_DEVICE;
    if (PRIMA_WANT(PRIMA_K_GATE_UP)) {
        const TokMat m[2] = {{W(L.wgate), F}, {W(L.wup), F}};
        const int fmts[2] = {f.wgate, f.wup};
        TokPrepare a = prepare(TOK_SWIGLU, F, nullptr, {f.wdown});
        PRIMA_TRY(streams(m, fmts, 2, e, a.p));
        a.norm = norm;
        a.out = tap_a ? at<float>(ws, w.a) : nullptr;
        PRIMA_TRY(launch_tok_prepare(a, StepInit{}, st));
    }
    if (tap_a && hipMemcpyAsync(tap_a, at<char>(ws, w.a), T * F * sizeof(float), hipMemcpyDeviceToDevice, st) != hipSuccess) return PRIMA_E_DEVICE;
    if (PRIMA_WANT(PRIMA_K_DOWN)) {
        const TokMat m{W(L.wdown), e};
        if (next) {
            TokPrepare a = prepare(TOK_RESIDUAL, e, next->g_attn, {nf.wq, nf.wk, nf.wv});
            PRIMA_TRY(streams(&m, &f.wdown, 1, F, a.p));
            a.x = h;
            a.out = y;
            PRIMA_TRY(launch_tok_prepare(a, StepInit{}, st));
        } else {
            TokSum a{1, T, tok_slots(T), {}, {e, 0, 0}, {y, nullptr, nullptr}, TokNorm{nullptr, 0, 0.f}, h};
            PRIMA_TRY(streams(&m, &f.wdown, 1, F, a.p));
            PRIMA_TRY(launch_tok_sum(a, st));
        }
    }
#undef PRIMA_WANT
#undef PRIMA_TRY
    return PRIMA_OK;
}

// whether a layer with these formats goes through run_layer_tok()
bool layer_is_tok(const prima_dims &d, const WindowWs &w, int T, int n_past, const AttnSeqs *seq, const prima_layer_formats *f)
{
    bool others = false, q4k = !f;
    int rows = n_past + T;
    if (f) {
        for (int32_t v : {f->wq, f->wk, f->wv, f->wo, f->wgate, f->wup, f->wdown}) {
            if (v == PRIMA_FMT_F32) return false;
            q4k = q4k || v == PRIMA_FMT_Q4_K;
            others = others || (v != PRIMA_FMT_Q4_K && v != PRIMA_FMT_Q8_0);
        }
    }
    if (seq)
        for (int b = 0; b < T; ++b) rows = std::max(rows, seq->n_past[b] + 1);
    return tok_takes(w, T, tok_from(d, others || !q4k, rows)) && tok_context(n_past, seq);
}

// all layers of a step; caches(i, seq): a batch's caches of layer i
template <class Caches>
prima_status run_layers(const prima_dims &d, const prima_layer *layers, const prima_layer_formats *formats, int L, int kv_cap, int n_past, int T,
                        const float *x_in, float *x_out, void *ws, const WindowWs &w, hipStream_t st, Caches caches, const int *positions = nullptr)
{
    const float *cur = x_in;
    bool prepared = false;
    // before the first layer: RoPE table, the counters of the mat-vec zeroed; in the first layer's first launch where that is a small one
    StepInit init = step_init_args(at<float>(ws, w.rope), T, d.head_dim, n_past, d.rope_theta, positions, at<char>(ws, w.gemv), w.arrivals_bytes);
    if (!layer_is_tok(d, w, T, n_past, caches(0), formats)) {
        const prima_status s = launch_step_init(init, st);
        if (s != PRIMA_OK) return s;
        init = StepInit{};
    }
    for (int i = 0; i < L; ++i) {
        float *dst = (i == L - 1) ? x_out : at<float>(ws, (i & 1) ? w.xb1 : w.xb0);
        const prima_layer_formats *f = formats ? &formats[i] : nullptr, *nf = formats && i + 1 < L ? &formats[i + 1] : nullptr;
        const AttnSeqs *seq = caches(i);
        prima_status s;
        if (layer_is_tok(d, w, T, n_past, seq, f)) {
            const bool chain = i + 1 < L && layer_is_tok(d, w, T, n_past, seq, nf);
            s = run_layer_tok(d, layers[i], kv_cap, n_past, T, cur, dst, ws, w, st, nullptr, nullptr, nullptr, nullptr, -1, seq, f, prepared,
                              chain ? &layers[i + 1] : nullptr, nf, init);
            init = StepInit{};
            prepared = chain;
        } else {
            s = run_layer(d, layers[i], kv_cap, n_past, T, cur, dst, ws, w, st, nullptr, nullptr, nullptr, nullptr, -1, seq, f);
            prepared = false;
        }
        if (s != PRIMA_OK) return s;
        cur = dst;
    }
    return PRIMA_OK;
}

prima_status check_window_args(const prima_dims *d, int32_t kv_cap, int32_t n_past, int32_t T,
                               const float *x_in, float *x_out, void *ws, size_t ws_bytes)
{
    if (!d || !x_in || !x_out || !ws) return PRIMA_E_NULL;
    if (!dims_ok(d)) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK || n_past < 0 || kv_cap < 1 || static_cast<int64_t>(n_past) + T > kv_cap) return PRIMA_E_RANGE;
    if (!aligned(x_in, 16) || !aligned(x_out, 16) || !aligned(ws, 256)) return PRIMA_E_ALIGN;
    if (ws_bytes < carve(*d, kv_cap, T).total) return PRIMA_E_WORKSPACE;
    return PRIMA_OK;
}

struct Span {
    size_t at, bytes;
};
struct PrefillWs {
    size_t q, k, v, o, h, a, u, xb0, xb1, rope, attn, ss, acts, total;
    // where the shares of K of a product lie: Q/K/V; output projection and down; gate and up sharing a launch (`pair_act`: the launch behind it
    // stores the activations); gate and up one by one
    Span s_qkv, s_out, s_pair, s_pair_act, s_gate, s_up;
    WindowWs dec; // short prompts: the scratch of a decode call of PRIMA_MAX_TOK tokens, in place of all this
};

// Scratch of a prompt-processing call: the layer's intermediate activations for all T tokens, the RoPE table, the
// matrix product's scratch (sized for the widest matrix), and the attention scratch of one 16-token call.  Every part grows with T, so that
// scratch for more tokens holds what fewer need.
// The shares of K lie in what the layer does not use at that time, around a region of their own:
//   a, u, the region, o, q, k, v, xb0, xb1
// Q/K/V leave them in a .. o (RoPE writes q, k and v while others still read shares), output projection and down in a .. v (the layer's input or
// output may be in xb0 or xb1), gate and up in all but what they write (the layer's input has been added by then).  The region holds what the most
// shares need beyond that (for prompts of a few tokens up to LEAST, their plans follow no such rule), and no more than MOST: from some T on what lies around is
// nearly enough.  A region that held the shares of just this T alone rose and fell with T.
// MB with 8192 cache rows, that / this (a decode call's scratch in the same place instead of behind): 8B 17 tokens 68 / 54, 276 255 / 226, 333 187 / 240, 1024 394 / 424;
// 70B 151 / 79, 381 / 315, 436 / 344, 729 / 705.
PrefillWs carve_prefill(const prima_dims &d, int kv_cap, int T)
{
    constexpr size_t LEAST = size_t{32} << 20, MOST = size_t{128} << 20;
    PrefillWs w{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += round_up(bytes, 256); return o; };
    const size_t qd = static_cast<size_t>(d.n_q_heads) * d.head_dim, kvd = static_cast<size_t>(d.n_kv_heads) * d.head_dim;
    const size_t f = sizeof(float), t = static_cast<size_t>(T);
    w.a = take(t * static_cast<size_t>(d.ffn) * f);
    w.u = take(t * static_cast<size_t>(d.ffn) * f); // up projection, when gate / up are not both Q4_K
    size_t part;
    {
        const int64_t e = d.e, F = d.ffn, Q = static_cast<int64_t>(qd), KV = static_cast<int64_t>(kvd), rows[3] = {Q, KV, KV};
        auto most = [](int64_t n_rows, int64_t n_cols) { return std::max(gemm_most_shares(&n_rows, 1, n_cols), fmt_gemm_most_shares(n_rows, n_cols)); };
        const int64_t beyond = std::max<int64_t>({
            gemm_most_shares(rows, 3, e) - (2 * F + Q),
            most(Q, e) + 2 * most(KV, e) - (2 * F + Q), // one by one when the formats differ, all there until the launch behind them
            most(e, Q) - 2 * (F + Q + KV), most(e, F) - 2 * (F + Q + KV),
            gemm_most_shares(&F, 1, e, true) - (F + 2 * (Q + KV + e)), most(F, e) - 2 * (Q + KV + e), 0});
        const size_t widest = static_cast<size_t>(std::max<int64_t>({Q + 2 * KV, e, 2 * F}));
        part = take(std::min(MOST, std::max(t * static_cast<size_t>(beyond) * f, std::min(LEAST, 16 * t * widest * f))));
    }
    w.o = take(t * qd * f);
    w.q = take(t * qd * f);
    w.k = take(t * kvd * f);
    w.v = take(t * kvd * f);
    w.xb0 = take(t * static_cast<size_t>(d.e) * f);
    w.xb1 = take(t * static_cast<size_t>(d.e) * f);
    w.h = take(t * static_cast<size_t>(d.e) * f);
    auto span = [](size_t from, size_t to) { return Span{from, to - from}; };
    w.s_qkv = span(w.a, w.q);
    w.s_out = span(w.a, w.xb0);
    w.s_pair = span(w.a, w.h);
    w.s_pair_act = w.s_gate = span(w.u, w.h);
    w.s_up = span(part, w.h);
    w.rope = take(t * static_cast<size_t>(d.head_dim) * f);
    w.attn = take(attn_ws_bytes(d, kv_cap, PRIMA_MAX_TOK));
    w.ss = take(gemm_ss_bytes(T, d.e));
    w.acts = take(gemm_acts_bytes(T, std::max<int64_t>({d.e, static_cast<int64_t>(qd), d.ffn})));
    w.dec = carve(d, kv_cap, PRIMA_MAX_TOK);
    w.total = std::max(off, w.dec.total);
    return w;
}

// One decoder layer for T prompt tokens: the projections as matrix products over all tokens, attention for pieces of PRIMA_MAX_TOK tokens (each sees
// the rows cached before it and, causally, its own), all pieces in one launch; between them the launches of gemm_prepare.hip.  prepared: the layer
// before this one has laid out x for this one's Q/K/V; next: the layer after it, whose Q/K/V activations the last launch may lay out (null: none), and
// then sets next_prepared; table: the RoPE table to be filled in by the layer's first launch or one in front (tab null: done before).
// fm: formats of the seven matrices (null: all Q4_K).  Each goes through the matrix product of its format; FP32 (whose
// weights are not exact in the product's binary16 operands) through the format mat-vec, PRIMA_MAX_TOK tokens a launch
prima_status run_layer_prefill(const prima_dims &d, const prima_layer &L, int kv_cap, int n_past, int T, const float *x, float *y, void *ws,
                               const PrefillWs &w, hipStream_t st, const prima_layer_formats *fm, bool prepared, const prima_layer *next,
                               const prima_layer_formats *next_fm, bool *next_prepared, const RopeTable &table)
{
    static constexpr prima_layer_formats ALL_Q4_K = {0, 0, 0, 0, 0, 0, 0};
    const prima_layer_formats &f = fm ? *fm : ALL_Q4_K, &nf = next_fm ? *next_fm : ALL_Q4_K;
    const int64_t e = d.e, qd = static_cast<int64_t>(d.n_q_heads) * d.head_dim, kvd = static_cast<int64_t>(d.n_kv_heads) * d.head_dim, F = d.ffn;
    float *q = at<float>(ws, w.q), *k = at<float>(ws, w.k), *v = at<float>(ws, w.v);
    float *o = at<float>(ws, w.o), *h = at<float>(ws, w.h), *act = at<float>(ws, w.a), *ss = at<float>(ws, w.ss);
    uint8_t *const acts = at<uint8_t>(ws, w.acts);
    auto part = [&](const Span &p) { return at<char>(ws, p.at); };
    prima_status s;
#define PRIMA_TRY(call) do { s = (call); if (s != PRIMA_OK) return s; } while (0)
    const GemmActs plain{acts, GemmNorm{}};
    const GemmActs normed{acts, GemmNorm{ss, static_cast<int>(e / QK), (T + 15) / 16 * 16, d.rms_eps}};
    auto mat = [](const void *W, float *out, int64_t rows) { return GemmMat{static_cast<const uint8_t *>(W), out, rows, rows}; };
    // Whether a matrix goes through a matrix product.  A small one alone in its group and few tokens: two mat-vecs are fewer launches than the
    // split, the product and its shares' sum (two layers of hidden size 512, down in Q8_0, us, product / mat-vecs: 17 tokens 255 / 212, 33 tokens 288 / 278).
    auto takes = [](int fmt) { return fmt == PRIMA_FMT_Q4_K || fmt_gemm_takes(fmt); };
    auto takes_alone = [&](int fmt, int64_t rows, int64_t cols) {
        return fmt == PRIMA_FMT_Q4_K || (fmt_gemm_takes(fmt) && !(T <= 2 * PRIMA_MAX_TOK && rows * cols < (int64_t{1} << 20)));
    };
    // one matrix: out = W a (+ resid); its shares of K left to the next launch, or added
    auto product = [&](int fmt, const GemmMat &m, int64_t cols, const GemmActs &a, const float *resid, const Span &to, GemmShares *later) {
        return fmt == PRIMA_FMT_Q4_K ? launch_q4k_gemm(&m, 1, false, cols, a, T, resid, m.n_rows, part(to), to.bytes, later, st)
                                     : launch_fmt_gemm(fmt, m, cols, a, T, resid, m.n_rows, part(to), to.bytes, later, st);
    };
    auto mat_vecs = [&](int fmt, const GemmMat &m, int64_t cols, const float *xin, const float *gain, const float *resid) -> prima_status {
        for (int t0 = 0; t0 < T; t0 += PRIMA_MAX_TOK) {
            const prima_status ps = launch_fmt_gemv(fmt, m.W, m.n_rows, cols, xin + t0 * cols, cols, std::min<int>(PRIMA_MAX_TOK, T - t0), gain, d.rms_eps,
                                                    resid ? resid + t0 * m.n_rows : nullptr, m.n_rows, m.y + t0 * m.n_rows, m.n_rows, st);
            if (ps != PRIMA_OK) return ps;
        }
        return PRIMA_OK;
    };
    // v (x, or the shares + x, or SwiGLU of the shares), stored to out and laid out as activations (lay), its gain applied
    auto prepare = [&](int mode, int64_t cols, const float *xin, const GemmShares &p, float *out, const float *gain, bool lay,
                       const RopeTable &tab = RopeTable{}) -> prima_status {
        if (!lay && !out) return PRIMA_OK;
        GemmPrepare a{};
        a.mode = mode; a.T = T; a.nb = static_cast<int>(cols / QK); a.x = xin; a.ldx = cols; a.p = p; a.norm = normed.norm;
        a.out = out; a.ldo = cols; a.gain = gain; a.ss = ss; a.A = lay ? acts : nullptr;
        return launch_gemm_prepare(a, tab, st);
    };
    const float *g_attn = static_cast<const float *>(L.g_attn), *g_ffn = static_cast<const float *>(L.g_ffn);

    { // Q, K, V: those in Q4_K in one launch, each of the others in one of its own
        const int fmts[3] = {f.wq, f.wk, f.wv};
        const GemmMat m[3] = {mat(L.wq, q, qd), mat(L.wk, k, kvd), mat(L.wv, v, kvd)};
        RopeAppend r{};
        if (takes(f.wq) || takes(f.wk) || takes(f.wv)) {
            if (!prepared) PRIMA_TRY(prepare(GEMM_PLAIN, e, x, GemmShares{}, nullptr, g_attn, true, table));
            r.norm = normed.norm;
        } else if (table.tab) {
            PRIMA_TRY(launch_rope_table(table, st));
        }
        Span to = w.s_qkv;
        auto used_by = [&](const GemmShares &p) {
            const size_t n = std::min(to.bytes, round_up(static_cast<size_t>(p.n) * static_cast<size_t>(p.stride) * sizeof(float), 256));
            to = Span{to.at + n, to.bytes - n};
        };
        GemmMat q4[3];
        int at_q4[3], n_q4 = 0;
        for (int i = 0; i < 3; ++i)
            if (fmts[i] == PRIMA_FMT_Q4_K) { at_q4[n_q4] = i; q4[n_q4++] = m[i]; }
        if (n_q4) {
            GemmShares p;
            PRIMA_TRY(launch_q4k_gemm(q4, n_q4, false, e, normed, T, nullptr, 0, part(to), to.bytes, &p, st));
            used_by(p);
            for (int i = 0; i < n_q4; ++i) {
                r.p[at_q4[i]] = p;
                r.p[at_q4[i]].col[0] = p.col[i];
            }
        }
        for (int i = 0; i < 3; ++i) {
            if (fmts[i] == PRIMA_FMT_Q4_K) continue;
            if (!takes(fmts[i])) {
                PRIMA_TRY(mat_vecs(fmts[i], m[i], e, x, g_attn, nullptr));
                continue;
            }
            PRIMA_TRY(product(fmts[i], m[i], e, normed, nullptr, to, &r.p[i]));
            used_by(r.p[i]);
        }
        for (int i = 0; i < 3; ++i)
            if (r.p[i].n == 0) r.p[i] = GemmShares{m[i].y, 0, 0, m[i].n_rows, {0, 0, 0}};
        // RoPE and the cache rows of all T tokens first; then the pieces of PRIMA_MAX_TOK tokens in one launch, or fewer tokens
        // than that in a launch of the decode kind (caches complete, queries rotated)
        r.tab = at<float>(ws, w.rope); r.q = q; r.kv_cap = kv_cap; r.n_past = n_past;
        r.K = static_cast<__half *>(L.k_cache); r.V = static_cast<__half *>(L.v_cache);
        PRIMA_TRY(launch_rope_append(r, d, T, st));
        if (T >= PRIMA_MAX_TOK) PRIMA_TRY(launch_attn_prompt(d, q, r.K, r.V, kv_cap, n_past, T, o, st));
        else PRIMA_TRY(launch_attn(d, q, nullptr, nullptr, nullptr, nullptr, r.K, r.V, kv_cap, n_past, T, o, at<char>(ws, w.attn), st, nullptr,
                                   ATTN_MERGE_INSIDE));
    }
    { // output projection, h = x + ..
        GemmShares p{};
        const bool lay = takes(f.wgate) || takes(f.wup);
        if (takes_alone(f.wo, e, qd)) {
            PRIMA_TRY(prepare(GEMM_PLAIN, qd, o, GemmShares{}, nullptr, nullptr, true));
            PRIMA_TRY(product(f.wo, mat(L.wo, h, e), qd, plain, x, w.s_out, &p));
        } else {
            PRIMA_TRY(mat_vecs(f.wo, mat(L.wo, h, e), qd, o, nullptr, x));
        }
        if (p.n) PRIMA_TRY(prepare(GEMM_RESIDUAL, e, x, p, h, g_ffn, lay));
        else PRIMA_TRY(prepare(GEMM_PLAIN, e, h, p, nullptr, g_ffn, lay));
    }
    const bool down = takes_alone(f.wdown, e, F);
    if (f.wgate == PRIMA_FMT_Q4_K && f.wup == PRIMA_FMT_Q4_K) {
        const GemmMat gate_up[2] = {mat(L.wgate, act, F), mat(L.wup, nullptr, F)};
        GemmShares p;
        const Span &to = down ? w.s_pair : w.s_pair_act;
        PRIMA_TRY(launch_q4k_gemm(gate_up, 2, true, e, normed, T, nullptr, 0, part(to), to.bytes, &p, st));
        if (p.n) PRIMA_TRY(prepare(GEMM_SWIGLU, F, nullptr, p, down ? nullptr : act, nullptr, down));
        else PRIMA_TRY(prepare(GEMM_PLAIN, F, act, p, nullptr, nullptr, down));
    } else {
        float *up = at<float>(ws, w.u);
        const GemmMat m[2] = {mat(L.wgate, act, F), mat(L.wup, up, F)};
        const int fmts[2] = {f.wgate, f.wup};
        for (int i = 0; i < 2; ++i) {
            if (takes(fmts[i])) PRIMA_TRY(product(fmts[i], m[i], e, normed, nullptr, i == 0 ? w.s_gate : w.s_up, nullptr));
            else PRIMA_TRY(mat_vecs(fmts[i], m[i], e, h, g_ffn, nullptr));
        }
        PRIMA_TRY(launch_swiglu(act, up, static_cast<int64_t>(T) * F, st));
        PRIMA_TRY(prepare(GEMM_PLAIN, F, act, GemmShares{}, nullptr, nullptr, down));
    }
    *next_prepared = false;
    if (!down) {
        PRIMA_TRY(mat_vecs(f.wdown, mat(L.wdown, y, e), F, act, nullptr, h));
    } else {
        GemmShares p;
        PRIMA_TRY(product(f.wdown, mat(L.wdown, y, e), F, plain, h, w.s_out, &p));
        if (p.n && next && (takes(nf.wq) || takes(nf.wk) || takes(nf.wv))) {
            PRIMA_TRY(prepare(GEMM_RESIDUAL, e, h, p, y, static_cast<const float *>(next->g_attn), true));
            *next_prepared = true;
        } else if (p.n) {
            PRIMA_TRY(launch_gemm_sum(p, GemmNorm{}, h, e, y, e, e, T, st));
        }
    }
#undef PRIMA_TRY
    return PRIMA_OK;
}

} // namespace

extern "C" {

int prima_abi_version(void) { return PRIMA_ABI_VERSION; }

const char *prima_status_str(prima_status s)
{
    switch (s) {
    case PRIMA_OK: return "ok";
    case PRIMA_E_NULL: return "null pointer";
    case PRIMA_E_SHAPE: return "unsupported shape";
    case PRIMA_E_ALIGN: return "misaligned pointer or leading dimension";
    case PRIMA_E_RANGE: return "T, n_past or kv_cap out of range";
    case PRIMA_E_WORKSPACE: return "workspace too small";
    case PRIMA_E_DEVICE: return "kernel launch failed";
    }
    return "unknown status";
}

prima_status prima_q4k_dequant(const void *W, int64_t n_rows, int64_t n_cols, float *out, void *hip_stream)
{
    if (n_rows < 0 || n_cols < 0 || n_cols % QK) return PRIMA_E_SHAPE;
    if (n_rows == 0 || n_cols == 0) return PRIMA_OK; // nothing to do; pointers may be null
    if (!W || !out) return PRIMA_E_NULL;
    if (!aligned(W, 16) || !aligned(out, 16)) return PRIMA_E_ALIGN;
    return launch_dequant(static_cast<const uint8_t *>(W), n_rows, n_cols, out, static_cast<hipStream_t>(hip_stream));
}

prima_status prima_stream_read_probe(const void *src, size_t bytes, void *sink, void *hip_stream)
{
    if (!src || !sink) return PRIMA_E_NULL;
    if (!aligned(src, 16) || !aligned(sink, 4)) return PRIMA_E_ALIGN;
    if (bytes < 16) return PRIMA_OK;
    return launch_stream_read(src, bytes, sink, static_cast<hipStream_t>(hip_stream), false);
}

prima_status prima_stream_read_probe_nt(const void *src, size_t bytes, void *sink, void *hip_stream)
{
    if (!src || !sink) return PRIMA_E_NULL;
    if (!aligned(src, 16) || !aligned(sink, 4)) return PRIMA_E_ALIGN;
    if (bytes < 16) return PRIMA_OK;
    return launch_stream_read(src, bytes, sink, static_cast<hipStream_t>(hip_stream), true);
}

size_t prima_gemv_workspace_bytes(int64_t n_rows, int64_t n_cols, int32_t T)
{
    if (n_rows < 0 || n_cols < 0 || T < 1) return 0;
    const size_t b = gemv_ws_bytes(n_rows, n_cols, T);
    return b < 256 ? 256 : b;
}

prima_status prima_q4k_gemv(const void *W, int64_t n_rows, int64_t n_cols, const float *x, int64_t ldx, int32_t T,
                            float *y, int64_t ldy, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!W || !x || !y || !workspace) return PRIMA_E_NULL;
    if (n_rows < 0 || n_cols <= 0 || n_cols % QK || ldx < n_cols || ldy < n_rows) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK) return PRIMA_E_RANGE;
    if (!aligned(W, 16) || !aligned(x, 16) || !aligned(y, 4) || ldx % 4 || !aligned(workspace, 256)) return PRIMA_E_ALIGN;
    if (workspace_bytes < std::max<size_t>(256, gemv_ws_bytes(n_rows, n_cols, T))) return PRIMA_E_WORKSPACE;
    if (n_rows == 0) return PRIMA_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (tok_gemv_takes(PRIMA_FMT_Q4_K, n_rows, n_cols, T))
        return launch_tok_gemv(PRIMA_FMT_Q4_K, static_cast<const uint8_t *>(W), n_rows, n_cols, x, ldx, T, nullptr, 0.f, nullptr, 0, y, ldy, st);
    GemvArgs ga = gemv_args(1, n_cols, x, ldx, T);
    ga.seg[0] = seg(W, y, n_rows, ldy);
    // The arrival counters are cleared only where a pass counts arrivals: a launch less for K that fits one slab, which
    // in a small mat-vec (1024 x 4096, one token) was half of the call
    return launch_gemv_mfma(ga, workspace, workspace_bytes, gemv_arrivals_bytes(n_rows), st, true);
}

} // extern "C"

// Scratch of prima_q4k_gemv_noalloc: part of the device image, one copy per GPU.  In host code the array's name is
// only a handle for hipGetSymbolAddress; kernels and fills get the device address looked up below.
static __device__ __align__(256) unsigned char scratch[PRIMA_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[NOALLOC_MAX_DEVICES]; // device address of `scratch` on each GPU, null until looked up

// the current device's copy of the array (looked up once per device, with that device current)
prima_status noalloc_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= NOALLOC_MAX_DEVICES) return PRIMA_E_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PRIMA_E_DEVICE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return PRIMA_OK;
}
} // namespace

extern "C" {

prima_status prima_q4k_gemv_noalloc(const void *W, int64_t n_rows, int64_t n_cols, const float *x, int64_t ldx, int32_t T,
                                    float *y, int64_t ldy, void *hip_stream)
{
    if (!W || !x || !y) return PRIMA_E_NULL;
    if (n_rows < 0 || n_cols <= 0 || n_cols % QK || ldx < n_cols || ldy < n_rows) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK) return PRIMA_E_RANGE;
    if (!aligned(W, 16) || !aligned(x, 16) || !aligned(y, 4) || ldx % 4) return PRIMA_E_ALIGN;
    const size_t need = std::max<size_t>(256, gemv_ws_bytes(n_rows, n_cols, T));
    if (need > PRIMA_NOALLOC_SCRATCH_BYTES) return PRIMA_E_WORKSPACE; // beyond the fixed array: use prima_q4k_gemv
    if (n_rows == 0) return PRIMA_OK;
    if (tok_gemv_takes(PRIMA_FMT_Q4_K, n_rows, n_cols, T))
        return launch_tok_gemv(PRIMA_FMT_Q4_K, static_cast<const uint8_t *>(W), n_rows, n_cols, x, ldx, T, nullptr, 0.f, nullptr, 0, y, ldy,
                               static_cast<hipStream_t>(hip_stream));
    void *ws = nullptr;
    prima_status s = noalloc_scratch(&ws);
    if (s != PRIMA_OK) return s;
    GemvArgs ga = gemv_args(1, n_cols, x, ldx, T);
    ga.seg[0] = seg(W, y, n_rows, ldy);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    // the array keeps what the last call left: where a pass looks at the counters they are cleared by a fill kernel (not a memset node)
    return launch_gemv_mfma(ga, ws, PRIMA_NOALLOC_SCRATCH_BYTES, gemv_arrivals_bytes(n_rows), st, true);
}

// scratch of a product on its own: the sums of squares, the activations laid out, then the shares of K
static size_t gemm_ws_bytes(int T, int64_t n_cols) { return gemm_ss_bytes(T, n_cols) + gemm_acts_bytes(T, n_cols); }

size_t prima_gemm_workspace_bytes(int32_t T, int64_t n_cols) { return (T < 1 || n_cols <= 0 || n_cols % QK) ? 0 : gemm_ws_bytes(T, n_cols); }

int32_t prima_gemm_ksplit(int32_t T, int64_t n_rows, int64_t n_cols)
{
    return (T < 1 || n_rows < 0 || n_cols <= 0 || n_cols % QK) ? 0 : gemm_ksplit(T, n_rows, n_cols);
}

size_t prima_gemm_workspace_bytes_ksplit(int32_t T, int64_t n_rows, int64_t n_cols)
{
    if (T < 1 || n_rows < 0 || n_cols <= 0 || n_cols % QK) return 0;
    return round_up(gemm_ws_bytes(T, n_cols), 256) + gemm_part_bytes(T, n_rows, n_cols);
}

prima_status prima_fmt_gemm_plan(int32_t fmt, int32_t T, int64_t n_rows, int64_t n_cols, int32_t *tokens, int32_t *blocks, int32_t *full)
{
    if (!tokens || !blocks || !full) return PRIMA_E_NULL;
    if (!fmt_gemm_takes(fmt) || n_rows < 1 || n_cols <= 0 || n_cols % QK) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_PREFILL_MAX_TOK) return PRIMA_E_RANGE;
    const FmtGemmBlocks p = fmt_gemm_blocks(T, n_rows, n_cols);
    *tokens = p.tokens; *blocks = p.blocks; *full = p.full ? 1 : 0;
    return PRIMA_OK;
}

prima_status prima_q4k_gemm(const void *W, int64_t n_rows, int64_t n_cols, const float *x, int64_t ldx, int32_t T,
                            const float *gain, float eps, const float *resid, int64_t ldr, float *y, int64_t ldy,
                            void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!W || !x || !y || !workspace) return PRIMA_E_NULL;
    if (n_rows < 0 || n_cols <= 0 || n_cols % QK || ldx < n_cols || ldy < n_rows || (resid && ldr < n_rows)) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_GEMM_MAX_TOK) return PRIMA_E_RANGE;
    if (!aligned(W, 16) || !aligned(x, 16) || !aligned(y, 4) || ldx % 4 || (gain && !aligned(gain, 16)) || (resid && !aligned(resid, 4)) ||
        !aligned(workspace, 256))
        return PRIMA_E_ALIGN;
    if (workspace_bytes < gemm_ws_bytes(T, n_cols)) return PRIMA_E_WORKSPACE;
    // what lies behind the minimum holds the shares of K, if it holds them all
    const size_t part_off = round_up(gemm_ws_bytes(T, n_cols), 256);
    void *part = workspace_bytes > part_off ? static_cast<char *>(workspace) + part_off : nullptr;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (n_rows == 0) return PRIMA_OK;
    GemmPrepare a{};
    a.mode = GEMM_PLAIN; a.T = T; a.nb = static_cast<int>(n_cols / QK); a.x = x; a.ldx = ldx; a.gain = gain;
    a.ss = static_cast<float *>(workspace);
    a.A = static_cast<uint8_t *>(workspace) + gemm_ss_bytes(T, n_cols);
    if (n_cols / QK >= (int64_t{1} << 31)) return PRIMA_E_SHAPE;
    const prima_status s = launch_gemm_prepare(a, RopeTable{}, st);
    if (s != PRIMA_OK) return s;
    GemmActs acts{a.A, GemmNorm{}};
    if (gain) acts.norm = GemmNorm{a.ss, a.nb, (T + 15) / 16 * 16, eps};
    const GemmMat m{static_cast<const uint8_t *>(W), y, n_rows, ldy};
    return launch_q4k_gemm(&m, 1, false, n_cols, acts, T, resid, ldr, part, part ? workspace_bytes - part_off : 0, nullptr, st);
}

size_t prima_attn_workspace_bytes(const prima_dims *d, int32_t kv_cap, int32_t T)
{
    if (!d || !dims_ok(d) || T < 1) return 0;
    return attn_ws_bytes(*d, kv_cap, T);
}

prima_status prima_attn_decode(const prima_dims *d, const float *q, const void *k_cache, const void *v_cache,
                               int32_t kv_cap, int32_t n_past, int32_t T, float *o,
                               void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!d || !q || !k_cache || !v_cache || !o || !workspace) return PRIMA_E_NULL;
    if (!dims_ok(d)) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK || n_past < 0 || kv_cap < 1 || static_cast<int64_t>(n_past) + T > kv_cap) return PRIMA_E_RANGE;
    if (!aligned(q, 16) || !aligned(o, 16) || !aligned(k_cache, 16) || !aligned(v_cache, 16) || !aligned(workspace, 256)) return PRIMA_E_ALIGN;
    if (workspace_bytes < attn_ws_bytes(*d, kv_cap, T)) return PRIMA_E_WORKSPACE;
    return launch_attn(*d, q, nullptr, nullptr, nullptr, nullptr,
                       static_cast<__half *>(const_cast<void *>(k_cache)), static_cast<__half *>(const_cast<void *>(v_cache)),
                       kv_cap, n_past, T, o, workspace, static_cast<hipStream_t>(hip_stream), nullptr, ATTN_MERGE_APART);
}

size_t prima_fmt_tensor_bytes(int32_t fmt, int64_t n_rows, int64_t n_cols) { return fmt_tensor_bytes(fmt, n_rows, n_cols); }

prima_status prima_fmt_dequant(int32_t fmt, const void *W, int64_t n_rows, int64_t n_cols, float *out, void *hip_stream)
{
    if (fmt == PRIMA_FMT_Q4_K) return prima_q4k_dequant(W, n_rows, n_cols, out, hip_stream);
    if (fmt < PRIMA_FMT_Q4_K || fmt > PRIMA_FMT_F32 || n_rows < 0 || n_cols < 0 || n_cols % QK) return PRIMA_E_SHAPE;
    if (n_rows == 0 || n_cols == 0) return PRIMA_OK;
    if (!W || !out) return PRIMA_E_NULL;
    if (!aligned(W, 16) || !aligned(out, 16)) return PRIMA_E_ALIGN;
    return launch_fmt_dequant(fmt, static_cast<const uint8_t *>(W), n_rows, n_cols, out, static_cast<hipStream_t>(hip_stream));
}

prima_status prima_fmt_gemv(int32_t fmt, const void *W, int64_t n_rows, int64_t n_cols,
                            const float *x, int64_t ldx, int32_t T, float *y, int64_t ldy, void *hip_stream)
{
    if (!W || !x || !y) return PRIMA_E_NULL;
    if (fmt <= PRIMA_FMT_Q4_K || fmt > PRIMA_FMT_F32) return PRIMA_E_SHAPE;
    if (n_rows < 0 || n_cols <= 0 || n_cols % QK || ldx < n_cols || ldy < n_rows) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK) return PRIMA_E_RANGE;
    if (!aligned(W, 16) || !aligned(x, 16) || !aligned(y, 4) || ldx % 4) return PRIMA_E_ALIGN;
    return launch_fmt_gemv(fmt, static_cast<const uint8_t *>(W), n_rows, n_cols, x, ldx, T, nullptr, 0.f, nullptr, 0, y, ldy,
                           static_cast<hipStream_t>(hip_stream));
}

prima_status prima_lm_head_fmt(const prima_dims *d, int32_t fmt, const float *g_final, const void *w_lm, int64_t vocab,
                               const float *x, int32_t T, float *logits, void *hip_stream)
{
    if (!d || !g_final || !w_lm || !x || !logits) return PRIMA_E_NULL;
    if (!dims_ok(d) || vocab < 1 || fmt <= PRIMA_FMT_Q4_K || fmt > PRIMA_FMT_F32) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK) return PRIMA_E_RANGE;
    if (!aligned(w_lm, 16) || !aligned(x, 16) || !aligned(g_final, 16) || !aligned(logits, 4)) return PRIMA_E_ALIGN;
    return launch_fmt_gemv(fmt, static_cast<const uint8_t *>(w_lm), vocab, d->e, x, d->e, T, g_final, d->rms_eps, nullptr, 0,
                           logits, vocab, static_cast<hipStream_t>(hip_stream));
}

prima_status prima_gemv_plan_status(int64_t n_rows, int64_t n_cols, int32_t T)
{
    if (n_rows < 0 || n_cols <= 0 || n_cols % QK) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK) return PRIMA_E_RANGE;
    if (n_rows == 0) return PRIMA_OK;
    if (tok_gemv_takes(PRIMA_FMT_Q4_K, n_rows, n_cols, T)) return tok_gemv_plan_status(PRIMA_FMT_Q4_K, n_rows, n_cols, T);
    static float dummy[4]; // addresses only: nothing is read or written
    GemvArgs ga = gemv_args(1, n_cols, dummy, n_cols, T);
    ga.seg[0] = seg(dummy, dummy, n_rows, n_rows);
    return gemv_plan_status(ga, dummy, std::max<size_t>(256, gemv_ws_bytes(n_rows, n_cols, T)), gemv_arrivals_bytes(n_rows));
}

prima_status prima_window_plan_status(const prima_dims *d, int32_t kv_cap, int32_t T)
{
    if (!d) return PRIMA_E_NULL;
    if (!dims_ok(d)) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK || kv_cap < T) return PRIMA_E_RANGE;
    const WindowWs w = carve(*d, kv_cap, T);
    const int64_t e = d->e, qd = static_cast<int64_t>(d->n_q_heads) * d->head_dim, kvd = static_cast<int64_t>(d->n_kv_heads) * d->head_dim, F = d->ffn;
    static float dummy[4];                       // addresses only: nothing is read or written
    char *const ws = reinterpret_cast<char *>(dummy);
    struct Launch { int nseg; int64_t rows[3]; int64_t cols; int xmode, epi; };
    // the launches of a layer, and those of its groups when some of their matrices are in other formats
    const Launch launches[] = {{3, {qd, kvd, kvd}, e, X_RMSNORM, EPI_ROWS}, {2, {qd, kvd, 0}, e, X_RMSNORM, EPI_ROWS},
                               {2, {kvd, kvd, 0}, e, X_RMSNORM, EPI_ROWS}, {1, {qd, 0, 0}, e, X_RMSNORM, EPI_ROWS},
                               {1, {kvd, 0, 0}, e, X_RMSNORM, EPI_ROWS}, {1, {e, 0, 0}, qd, X_PLAIN, EPI_ROWS},
                               {2, {F, F, 0}, e, X_RMSNORM, EPI_SWIGLU}, {1, {F, 0, 0}, e, X_RMSNORM, EPI_ROWS},
                               {1, {e, 0, 0}, F, X_PLAIN, EPI_ROWS}};
    for (const Launch &l : launches) {
        GemvArgs ga = gemv_args(l.nseg, l.cols, dummy, l.cols, T, l.xmode, dummy, d->rms_eps, l.epi);
        for (int i = 0; i < l.nseg; ++i) ga.seg[i] = seg(ws, dummy, l.rows[i], l.rows[i]);
        const prima_status s = gemv_plan_status(ga, ws, w.gemv_bytes, w.arrivals_bytes);
        if (s != PRIMA_OK) return s;
    }
    // the same groups, and their matrices alone, in every format through the weight streams and the format mat-vec
    for (const Launch &l : launches) {
        int64_t rows = 0;
        size_t floats = 0;
        for (int i = 0; i < l.nseg; ++i) {
            rows += l.rows[i];
            if (w.tok_part_floats != 0) floats += tok_part_floats(l.rows[i], l.cols, T);
        }
        for (int fmt = PRIMA_FMT_Q4_K; fmt <= PRIMA_FMT_F16; ++fmt) {
            prima_status s = PRIMA_OK;
            if (tok_takes(w, T, TOK_LEAST)) s = tok_stream_plan_status(fmt, rows, l.cols, T, std::min(floats, w.tok_part_floats));
            const int first = tok_gemv_first(fmt, rows, l.cols, T);
            if (s == PRIMA_OK && l.nseg == 1 && fmt != PRIMA_FMT_Q4_K && tok_gemv_takes(fmt, rows, l.cols, T)) s = tok_gemv_plan_status(fmt, rows, l.cols, first);
            if (s != PRIMA_OK) return s;
        }
    }
    return PRIMA_OK;
}

size_t prima_workspace_bytes(const prima_dims *d, int32_t kv_cap, int32_t T)
{
    if (!d || !dims_ok(d) || T < 1 || T > PRIMA_MAX_TOK || kv_cap < 0) return 0;
    return carve(*d, kv_cap, T).total;
}

prima_status prima_layer_window_decode(const prima_dims *d, const prima_layer *layers, int32_t L,
                                       int32_t kv_cap, int32_t n_past, int32_t T,
                                       const float *x_in, float *x_out,
                                       void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!layers) return PRIMA_E_NULL;
    prima_status s = check_window_args(d, kv_cap, n_past, T, x_in, x_out, workspace, workspace_bytes);
    if (s != PRIMA_OK) return s;
    if (L < 1) return PRIMA_E_RANGE;
    for (int i = 0; i < L; ++i)
        if ((s = check_layer(layers[i])) != PRIMA_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const WindowWs w = carve(*d, kv_cap, T);
    return run_layers(*d, layers, nullptr, L, kv_cap, n_past, T, x_in, x_out, workspace, w, st, [](int) { return static_cast<const AttnSeqs *>(nullptr); });
}

prima_status prima_layer_window_decode_mixed(const prima_dims *d, const prima_layer *layers, const prima_layer_formats *formats,
                                             int32_t L, int32_t kv_cap, int32_t n_past, int32_t T,
                                             const float *x_in, float *x_out,
                                             void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!layers || !formats) return PRIMA_E_NULL;
    prima_status s = check_window_args(d, kv_cap, n_past, T, x_in, x_out, workspace, workspace_bytes);
    if (s != PRIMA_OK) return s;
    if (L < 1) return PRIMA_E_RANGE;
    for (int i = 0; i < L; ++i) {
        if ((s = check_layer(layers[i])) != PRIMA_OK) return s;
        const int32_t f[7] = {formats[i].wq, formats[i].wk, formats[i].wv, formats[i].wo, formats[i].wgate, formats[i].wup, formats[i].wdown};
        for (int32_t v : f)
            if (v < PRIMA_FMT_Q4_K || v > PRIMA_FMT_F32) return PRIMA_E_SHAPE;
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const WindowWs w = carve(*d, kv_cap, T);
    return run_layers(*d, layers, formats, L, kv_cap, n_past, T, x_in, x_out, workspace, w, st, [](int) { return static_cast<const AttnSeqs *>(nullptr); });
}

prima_status prima_layer_window_decode_batch(const prima_dims *d, const prima_layer *layers, int32_t L,
                                             int32_t kv_cap, int32_t B, const int32_t *n_past,
                                             void *const *k_caches, void *const *v_caches,
                                             const float *x_in, float *x_out,
                                             void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return prima_layer_window_decode_batch_mixed(d, layers, nullptr, L, kv_cap, B, n_past, k_caches, v_caches, x_in, x_out,
                                                 workspace, workspace_bytes, hip_stream);
}

prima_status prima_layer_window_decode_batch_mixed(const prima_dims *d, const prima_layer *layers, const prima_layer_formats *formats,
                                                   int32_t L, int32_t kv_cap, int32_t B, const int32_t *n_past,
                                                   void *const *k_caches, void *const *v_caches,
                                                   const float *x_in, float *x_out,
                                                   void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!layers || !n_past || !k_caches || !v_caches) return PRIMA_E_NULL;
    prima_status s = check_window_args(d, kv_cap, 0, B, x_in, x_out, workspace, workspace_bytes);
    if (s != PRIMA_OK) return s;
    if (L < 1) return PRIMA_E_RANGE;
    for (int b = 0; b < B; ++b)
        if (n_past[b] < 0 || static_cast<int64_t>(n_past[b]) + 1 > kv_cap) return PRIMA_E_RANGE;
    for (int i = 0; i < L; ++i) {
        if ((s = check_layer(layers[i], false)) != PRIMA_OK) return s;
        if (formats) {
            const int32_t f[7] = {formats[i].wq, formats[i].wk, formats[i].wv, formats[i].wo, formats[i].wgate, formats[i].wup, formats[i].wdown};
            for (int32_t v : f)
                if (v < PRIMA_FMT_Q4_K || v > PRIMA_FMT_F32) return PRIMA_E_SHAPE;
        }
        for (int b = 0; b < B; ++b) {
            const void *kc = k_caches[static_cast<size_t>(i) * B + b], *vc = v_caches[static_cast<size_t>(i) * B + b];
            if (!kc || !vc) return PRIMA_E_NULL;
            if (!aligned(kc, 16) || !aligned(vc, 16)) return PRIMA_E_ALIGN;
        }
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const WindowWs w = carve(*d, kv_cap, B);
    __half *kc[PRIMA_MAX_TOK], *vc[PRIMA_MAX_TOK];
    const AttnSeqs seq{n_past, kc, vc};
    return run_layers(*d, layers, formats, L, kv_cap, 0, B, x_in, x_out, workspace, w, st, [&](int i) {
        for (int b = 0; b < B; ++b) {
            kc[b] = static_cast<__half *>(k_caches[static_cast<size_t>(i) * B + b]);
            vc[b] = static_cast<__half *>(v_caches[static_cast<size_t>(i) * B + b]);
        }
        return &seq;
    }, n_past);
}

void prima_set_prefill_small_tokens(int32_t n) { g_prefill_small_tokens = n < 0 ? 0 : n; }

size_t prima_prefill_workspace_bytes(const prima_dims *d, int32_t kv_cap, int32_t T)
{
    if (!d || !dims_ok(d) || T < 1 || T > PRIMA_PREFILL_MAX_TOK || kv_cap < 1) return 0;
    return carve_prefill(*d, kv_cap, T).total;
}

prima_status prima_layer_window_prefill(const prima_dims *d, const prima_layer *layers, int32_t L,
                                        int32_t kv_cap, int32_t n_past, int32_t T,
                                        const float *x_in, float *x_out, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return prima_layer_window_prefill_mixed(d, layers, nullptr, L, kv_cap, n_past, T, x_in, x_out, workspace, workspace_bytes, hip_stream);
}

prima_status prima_layer_window_prefill_mixed(const prima_dims *d, const prima_layer *layers, const prima_layer_formats *formats, int32_t L,
                                              int32_t kv_cap, int32_t n_past, int32_t T,
                                              const float *x_in, float *x_out, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!d || !x_in || !x_out || !workspace || !layers) return PRIMA_E_NULL;
    if (!dims_ok(d)) return PRIMA_E_SHAPE;
    if (L < 1 || T < 1 || T > PRIMA_PREFILL_MAX_TOK || n_past < 0 || kv_cap < 1 || static_cast<int64_t>(n_past) + T > kv_cap) return PRIMA_E_RANGE;
    if (!aligned(x_in, 16) || !aligned(x_out, 16) || !aligned(workspace, 256)) return PRIMA_E_ALIGN;
    const PrefillWs w = carve_prefill(*d, kv_cap, T);
    if (workspace_bytes < w.total) return PRIMA_E_WORKSPACE;
    for (int i = 0; i < L; ++i) {
        const prima_status c = check_layer(layers[i]);
        if (c != PRIMA_OK) return c;
        if (formats) {
            const int32_t f[7] = {formats[i].wq, formats[i].wk, formats[i].wv, formats[i].wo, formats[i].wgate, formats[i].wup, formats[i].wdown};
            for (int32_t v : f)
                if (v < PRIMA_FMT_Q4_K || v > PRIMA_FMT_F32) return PRIMA_E_SHAPE;
        }
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (T <= g_prefill_small_tokens) {
        // a short prompt: a matrix-product workgroup does the work of 64 tokens whatever their number; up to one decode call's
        // worth of tokens the decode kernels are faster
        for (int t0 = 0; t0 < T; t0 += PRIMA_MAX_TOK) {
            const int Tc = std::min<int>(PRIMA_MAX_TOK, T - t0);
            const prima_status cs = run_layers(*d, layers, formats, L, kv_cap, n_past + t0, Tc, x_in + static_cast<int64_t>(t0) * d->e, x_out + static_cast<int64_t>(t0) * d->e,
                            workspace, w.dec, st, [](int) { return static_cast<const AttnSeqs *>(nullptr); });
            if (cs != PRIMA_OK) return cs;
        }
        return PRIMA_OK;
    }
    prima_status s = PRIMA_OK;
    if (T < PRIMA_MAX_TOK) { // the attention launch then merges its key ranges inside: its records marked "not written"
        char *const attn = at<char>(workspace, w.attn);
        const size_t head_bytes = attn_counter_bytes(*d, T); // the records start behind it
        s = launch_fill_words(attn, head_bytes, 0u, attn + head_bytes, attn_records_bytes(*d, n_past + T, T), ATTN_REC_EMPTY, st);
        if (s != PRIMA_OK) return s;
    }
    const float *cur = x_in;
    bool prepared = false;
    for (int i = 0; i < L; ++i) {
        float *dst = (i == L - 1) ? x_out : at<float>(workspace, (i & 1) ? w.xb1 : w.xb0);
        const bool more = i + 1 < L;
        s = run_layer_prefill(*d, layers[i], kv_cap, n_past, T, cur, dst, workspace, w, st, formats ? &formats[i] : nullptr, prepared,
                              more ? &layers[i + 1] : nullptr, formats && more ? &formats[i + 1] : nullptr, &prepared,
                              i == 0 ? rope_table(at<float>(workspace, w.rope), T, d->head_dim, n_past, d->rope_theta) : RopeTable{});
        if (s != PRIMA_OK) return s;
        cur = dst;
    }
    return PRIMA_OK;
}

prima_status prima_window_check(const prima_dims *d, int32_t kv_cap, int32_t T, const void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!d || !workspace) return PRIMA_E_NULL;
    if (!dims_ok(d) || T < 1 || T > PRIMA_MAX_TOK || kv_cap < 1) return PRIMA_E_SHAPE;
    const WindowWs w = carve(*d, kv_cap, T);
    if (workspace_bytes < w.total) return PRIMA_E_WORKSPACE;
    return hipStreamSynchronize(static_cast<hipStream_t>(hip_stream)) == hipSuccess ? PRIMA_OK : PRIMA_E_DEVICE;
}

prima_status prima_layer_window_decode_profiled(const prima_dims *d, const prima_layer *layers, int32_t L,
                                                int32_t kv_cap, int32_t n_past, int32_t T,
                                                const float *x_in, float *x_out,
                                                void *workspace, size_t workspace_bytes, void *hip_stream,
                                                float *ms_by_kind, int32_t *launches_by_kind)
{
    if (!layers || !ms_by_kind || !launches_by_kind) return PRIMA_E_NULL;
    prima_status s = check_window_args(d, kv_cap, n_past, T, x_in, x_out, workspace, workspace_bytes);
    if (s != PRIMA_OK) return s;
    if (L < 1) return PRIMA_E_RANGE;
    for (int i = 0; i < L; ++i)
        if ((s = check_layer(layers[i])) != PRIMA_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const WindowWs w = carve(*d, kv_cap, T);
    // one ordinary step first: every intermediate buffer then holds this step's values
    auto ordinary_step = [&]() {
        return run_layers(*d, layers, nullptr, L, kv_cap, n_past, T, x_in, x_out, workspace, w, st, [](int) { return static_cast<const AttnSeqs *>(nullptr); });
    };
    s = ordinary_step();
    // then each kind of launch on its own, once per layer (L different weight sets, so nothing is
    // served from a cache that the real step would not have), between two events
    hipEvent_t ev[PRIMA_N_KINDS + 1];
    int n_ev = 0;
    const int kinds[] = {PRIMA_K_QKV, PRIMA_K_ATTN, PRIMA_K_WO, PRIMA_K_GATE_UP, PRIMA_K_DOWN};
    const int n_kinds = static_cast<int>(sizeof(kinds) / sizeof(kinds[0]));
    for (int k = 0; k < PRIMA_N_KINDS; ++k) { ms_by_kind[k] = 0.f; launches_by_kind[k] = 0; }
    auto mark = [&]() {
        if (hipEventCreate(&ev[n_ev]) != hipSuccess) return false;
        ++n_ev;
        return hipEventRecord(ev[n_ev - 1], st) == hipSuccess;
    };
    if (s == PRIMA_OK && !mark()) s = PRIMA_E_DEVICE;
    float *scratch_out = at<float>(workspace, w.xb0); // the isolated down projections write here, not to x_out
    for (int ki = 0; ki < n_kinds && s == PRIMA_OK; ++ki) {
        for (int i = 0; i < L && s == PRIMA_OK; ++i)
            s = layer_is_tok(*d, w, T, n_past, nullptr, nullptr)
                    ? run_layer_tok(*d, layers[i], kv_cap, n_past, T, x_in, scratch_out, workspace, w, st, nullptr, nullptr, nullptr, nullptr, kinds[ki], nullptr,
                                    nullptr, false, nullptr, nullptr)
                    : run_layer(*d, layers[i], kv_cap, n_past, T, x_in, scratch_out, workspace, w, st, nullptr, nullptr, nullptr, nullptr, kinds[ki]);
        if (s == PRIMA_OK && !mark()) s = PRIMA_E_DEVICE;
    }
    // The replayed attention launches appended rows n_past .. n_past+T-1 of every layer's caches from whatever the
    // replayed projections left in the scratch (each layer's projections of x_in, not of that layer's own input).
    // The ordinary step once more writes the right rows again (and x_out): the same bits as a plain decode call.
    if (s == PRIMA_OK) s = ordinary_step();
    if (s == PRIMA_OK && hipStreamSynchronize(st) != hipSuccess) s = PRIMA_E_DEVICE;
    for (int ki = 0; ki < n_kinds && s == PRIMA_OK; ++ki) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, ev[ki], ev[ki + 1]) != hipSuccess) { s = PRIMA_E_DEVICE; break; }
        ms_by_kind[kinds[ki]] = ms;
        launches_by_kind[kinds[ki]] = L;
    }
    for (int i = 0; i < n_ev; ++i) (void)hipEventDestroy(ev[i]);
    return s;
}

prima_status prima_layer_decode_taps(const prima_dims *d, const prima_layer *layer,
                                     int32_t kv_cap, int32_t n_past, int32_t T,
                                     const float *x_in, float *x_out,
                                     float *tap_q, float *tap_o, float *tap_h, float *tap_a,
                                     void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!layer) return PRIMA_E_NULL;
    prima_status s = check_window_args(d, kv_cap, n_past, T, x_in, x_out, workspace, workspace_bytes);
    if (s != PRIMA_OK) return s;
    if ((s = check_layer(*layer)) != PRIMA_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const WindowWs w = carve(*d, kv_cap, T);
    s = launch_step_init(step_init_args(at<float>(workspace, w.rope), T, d->head_dim, n_past, d->rope_theta, nullptr, at<char>(workspace, w.gemv), w.arrivals_bytes), st);
    if (s != PRIMA_OK) return s;
    if (layer_is_tok(*d, w, T, n_past, nullptr, nullptr))
        return run_layer_tok(*d, *layer, kv_cap, n_past, T, x_in, x_out, workspace, w, st, tap_q, tap_o, tap_h, tap_a, -1, nullptr, nullptr, false, nullptr, nullptr);
    return run_layer(*d, *layer, kv_cap, n_past, T, x_in, x_out, workspace, w, st, tap_q, tap_o, tap_h, tap_a);
}

size_t prima_lm_head_workspace_bytes(const prima_dims *d, int64_t vocab, int32_t T)
{
    if (!d || !dims_ok(d) || vocab < 1 || T < 1 || T > PRIMA_MAX_TOK) return 0;
    return std::max<size_t>(256, gemv_ws_bytes(vocab, d->e, T));
}

prima_status prima_lm_head(const prima_dims *d, const float *g_final, const void *w_lm, int64_t vocab,
                           const float *x, int32_t T, float *logits,
                           void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!d || !g_final || !w_lm || !x || !logits || !workspace) return PRIMA_E_NULL;
    if (!dims_ok(d) || vocab < 1) return PRIMA_E_SHAPE;
    if (T < 1 || T > PRIMA_MAX_TOK) return PRIMA_E_RANGE;
    if (!aligned(g_final, 16) || !aligned(w_lm, 16) || !aligned(x, 16) || !aligned(logits, 4) || !aligned(workspace, 256)) return PRIMA_E_ALIGN;
    if (workspace_bytes < prima_lm_head_workspace_bytes(d, vocab, T)) return PRIMA_E_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (tok_gemv_takes(PRIMA_FMT_Q4_K, vocab, d->e, T))
        return launch_tok_gemv(PRIMA_FMT_Q4_K, static_cast<const uint8_t *>(w_lm), vocab, d->e, x, d->e, T, g_final, d->rms_eps, nullptr, 0, logits, vocab, st);
    GemvArgs ga = gemv_args(1, d->e, x, d->e, T, X_RMSNORM, g_final, d->rms_eps);
    ga.seg[0] = seg(w_lm, logits, vocab, vocab);
    return launch_gemv_mfma(ga, workspace, workspace_bytes, gemv_arrivals_bytes(vocab), st, true);
}

} // extern "C"
