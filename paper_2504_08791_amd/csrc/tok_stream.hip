// The projections of a layer window for several tokens (speculative verification, batches of sequences; from how many on: tok_from() in
// window.hip), and of narrow windows of 4 to 8 tokens those in other formats than Q4_K: mat-vecs on the matrix
// cores over activations that are prepared once per projection, with the sums finished by the kernel that prepares the next
// one.  Arithmetic and layouts: tok_common.h.
//
//   tok_stream_kernel   the weight stream: every format but FP32.  K is cut into slabs whose activations fit in LDS beside the
//                       waves' stage buffers; a workgroup copies its slab's records (one pass over L2, no arithmetic) and
//                       its waves stream (tile, part of the slab) units.  A unit's sums go to global memory, nothing meets
//                       inside the launch: no barrier behind the first, no arrival counts, no waiting.
//   tok_prepare_kernel  adds the shares of K in a fixed order, finishes them (residual, or 1/rms and SwiGLU; attention's key ranges are
//                       merged there too), stores the vector where it is needed and lays it out as the next projection's activations (gain applied; its sums of
//                       squares beside it: 1/rms multiplies the finished sums of the next projection).
//   tok_sum_kernel      adds the shares where plain vectors are wanted (Q, K, V; the window's output).
//
// The Q4_K mat-vec of one to eight tokens (q4k_gemv_mfma.hip) takes 16 tokens in two passes over the weights; here one pass
// serves them.  A 14B-shaped layer, 16 sequences, us with the tracer: Q/K/V 38 -> 19, output 31 -> 21, gate and up 65 -> 38,
// down 44 -> 25 (adding and preparing included); the batch step of three layers 586 -> 380.  What bounds the stream at 16
// tokens: 27648 x 5120 (80 MB, 12 us at the rate of a linear read) takes 30 us, 21 without its products, 31 without its
// loads: the LDS reads of the operands (17 KB a super-block and wave) and the unpacking under two waves a SIMD.
// At 3 to 8 tokens the stream alone, products left out, takes 52 of the 59 us of 57344 x 8192 at 8 tokens (5.0 TB/s; 34 of 37 of 55296 x 5120 at 4):
// it stands at what ordinary loads of short runs reach, with about 5 us of fixed parts a launch.  Twelve waves (three a SIMD) for
// Q4_K and Q5_K: 2 to 5 % slower; non-temporal loads of Q4_K: 6 % slower (a row's run of a stage is 288 bytes, and the
// lines that straddle two stages are fetched twice); the waves' walks along K begun at different stages: no change.
#include <algorithm>
#include <atomic>

#include "tok_common.h"
#include "tok_stream.h"

namespace prima {
namespace {

struct StreamSeg {
    const uint8_t *W;
    int64_t n_rows;
    int tile0; // first tile (INT_MAX: unused)
};

struct StreamArgs {
    StreamSeg seg[3];
    const uint8_t *rec; // activations: nb records
    float *part;        // sums: [slab][part][token][row], rows = 16 n_tiles
    int nb, T, n_tiles;
    int n_slabs, slab; // slabs of K, super-blocks of one (a multiple of the stage's; the last may be shorter)
    int ks_shift;      // a unit is one of 2^ks_shift parts of a (tile, slab)
    int rounds, per_round; // as in tok_gemv.hip, among the workgroups of a slab
    // a slab has wg_slab workgroups, the first wg_more one more; workgroup / n_slabs by a multiplication (n_slabs 1: not needed)
    int wg_slab, wg_more;
    unsigned slab_magic;
};

template <int FMT, int NT>
__global__ void __launch_bounds__(TkFmt<FMT>::WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) tok_stream_kernel(StreamArgs a)
{
    request_args<sizeof(a)>();
    extern __shared__ __align__(16) uint8_t smem[];
    constexpr int SBS = TkFmt<FMT>::SBS, WAVES = TkFmt<FMT>::WAVES;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    uint8_t *const l_stage = smem + wave * tk_stage_bytes<FMT>;
    uint8_t *const l_a = smem + WAVES * tk_stage_bytes<FMT>;

    // The matrices' fields as one and what the next has more: picked by a number they are fetched through a picked address, each a wait in front
    // of the first weights.
    const uint8_t *const W0 = a.seg[0].W;
    const int64_t W1 = a.seg[1].W - a.seg[0].W, W2 = a.seg[2].W - a.seg[1].W;
    const int64_t rows0 = a.seg[0].n_rows, rows1 = a.seg[1].n_rows - rows0, rows2 = a.seg[2].n_rows - rows1 - rows0;
    const int first1 = a.seg[1].tile0, first2 = a.seg[2].tile0;
    const int rank = a.n_slabs == 1 ? blockIdx.x : static_cast<int>(__umulhi(blockIdx.x, a.slab_magic)), slab = static_cast<int>(blockIdx.x) - rank * a.n_slabs;
    const int ranks = a.wg_slab + (slab < a.wg_more ? 1 : 0); // workgroups of this slab
    const int nb = a.nb, ks_shift = a.ks_shift, ks = 1 << ks_shift;
    const int sb0 = slab * a.slab, nsb = min(a.slab, nb - sb0);
    const int my_l = wave >> ks_shift, part = wave & (ks - 1);
    const int stages = (nsb + SBS - 1) / SBS, s0 = (stages * part) >> ks_shift, s1 = (stages * (part + 1)) >> ks_shift; // this wave's stages (not none: host)
    const int my_tile = rank + my_l * ranks; // counted from the round's first
    // the first round from k on in which this wave has a tile (rounds: none), and the tile
    auto next_round = [&](int k, int &tile) __attribute__((always_inline)) {
        tile = k * a.per_round + my_tile;
        if (my_tile >= a.per_round || tile >= a.n_tiles) return a.rounds;
        return min(k, a.rounds);
    };
    // (all rounds but the last are full)
    const int n_active = my_tile >= a.per_round ? 0 : a.rounds - 1 + (my_tile < a.n_tiles - (a.rounds - 1) * a.per_round ? 1 : 0);
    const int total = (s1 - s0) * n_active;

    // requests, two stages ahead (past the end the last stage again: the loads in flight are then the same on every path)
    TkSrc<FMT> src;
    TkRegs<FMT> r0, r1;
    int ld_k = -1, ld_b = 0, ld_left = 0, ld_step = SBS;
    auto ld_next = [&]() __attribute__((always_inline)) {
        int tile;
        const int k = next_round(ld_k + 1, tile);
        if (k < a.rounds) {
            ld_k = k;
            ld_b = sb0 + s0 * SBS;
            ld_left = s1 - s0;
            const bool one = tile >= first1, two = tile >= first2;
            const uint8_t *W = W0 + ((one ? W1 : 0) + (two ? W2 : 0));
            const int64_t n_rows = rows0 + (one ? rows1 : 0) + (two ? rows2 : 0);
            const int first = two ? first2 : (one ? first1 : 0);
            tk_tile<FMT>(src, W, n_rows, nb, static_cast<int64_t>(tile - first) * 16, lane);
        } else {
            ld_b -= ld_step;
            ld_step = 0;
            ld_left = 0x7fffffff;
        }
    };
    auto request = [&](TkRegs<FMT> &r) __attribute__((always_inline)) {
        tk_load<FMT>(r, src, max(min(ld_b, nb - SBS), 0)); // (the last stage of an odd number of super-blocks: its second one)
        ld_b += ld_step;
        if (--ld_left == 0) ld_next();
    };
    if (total != 0) {
        ld_next();
        request(r0);
        request(r1);
    }
    // the slab's records
    {
        const uint8_t *from = a.rec + static_cast<int64_t>(sb0) * tk_rec(NT);
        const int bytes = nsb * tk_rec(NT);
        const uint32_t to = __builtin_amdgcn_readfirstlane(lds_address(l_a));
        for (int o = wave * 1024; o < bytes; o += WAVES * 1024)
            if (o + lane * 16 < bytes) dma16(from + o + lane * 16, to + o);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // (the compiler does not know these loads)
        __syncthreads();
    }

    int tile, k = next_round(0, tile), s = s0;
    float y[4] = {0.f, 0.f, 0.f, 0.f};
    const int64_t rows = static_cast<int64_t>(a.n_tiles) * 16;
    float *const out = a.part + static_cast<int64_t>((slab << ks_shift) + part) * a.T * rows + n;
    auto consume = [&](TkRegs<FMT> &r, bool real, auto second) __attribute__((always_inline)) {
        tk_put<FMT>(r, l_stage, lane);
        request(r);
        if (real) {
            auto mul = [&](int slot, int b, auto odd) __attribute__((always_inline)) {
                tk_mul<FMT, NT, decltype(odd)::value>(l_stage, slot, l_a + b * tk_rec(NT), lane, y);
            };
            if constexpr (SBS == 1) {
                mul(0, s, second);
            } else if (2 * s + 1 < nsb) {
                tk_mul2<FMT, NT>(l_stage, l_a + 2 * s * tk_rec(NT), l_a + (2 * s + 1) * tk_rec(NT), lane, y);
            } else {
                mul(nb == 1 ? 0 : 1, 2 * s, std::false_type{});
            }
            if (++s == s1) { // the unit's sums (lanes past the token slots repeat others)
                constexpr int NY = NT <= 8 ? 2 : 4;
                const int gt = NT <= 8 ? (g & (NT / 2 - 1)) : g;
                if (NT >= 8 || g < NT / 2) {
#pragma unroll
                    for (int i = 0; i < NY; ++i)
                        if (NY * gt + i < a.T) out[(NY * gt + i) * rows + static_cast<int64_t>(tile) * 16] = y[i];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i] = 0.f;
                s = s0;
                k = next_round(k + 1, tile);
            }
        }
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    };
    for (int i = 0; i < total; i += 2) {
        consume(r0, true, std::false_type{});
        consume(r1, i + 1 < total, std::true_type{});
    }
}

// What the launches between the streams have to do is little; they are chains of trips through memory (the shares come from other
// XCDs).  So a wave takes 256 numbers of one token, four a lane, and everything that it will read is requested in front of the first use:
// one trip.  (Four waves that took every fourth share and met in LDS, wave 0 going on to read the residual, the gains and the
// sums of squares one after the other: 4.6 to 5.3 us a launch, 6.8 in front of the down projection; now 3 to 4.8.  16 sequences through
// three 14B-shaped layers 365 -> 335 us.)
constexpr int ADD_WAVES = 4;
typedef float tk_f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ tk_f4 load_f4(const float *p) { return *reinterpret_cast<const tk_f4 *>(p); }

// v, u: the sums over the shares of p, q (TWO) of this lane's four rows of token t.  N: shares requested at a time, and added pairwise: one
// after the other a product's error grew with its shares (512 x 65536, 16 tokens, 32 shares: 1.90e-7 of the product, now 1.39e-7; 2048 x 28672 1.66 / 1.43e-7;
// whole layers 1 to 2 %).
template <int N, bool TWO>
__device__ __forceinline__ void add_shares_n(const TokPart &p, const TokPart &q, int T, int t, int64_t row, tk_f4 &v, tk_f4 &u)
{
    const float *const sp = p.part + t * p.rows + p.row0 + row, *const sq = TWO ? q.part + t * q.rows + q.row0 + row : nullptr;
    const int64_t dp = static_cast<int64_t>(T) * p.rows, dq = static_cast<int64_t>(T) * q.rows;
    const int parts = TWO ? max(p.n_parts, q.n_parts) : p.n_parts;
    for (int i = 0; i < parts; i += N) {
        tk_f4 a[N], b[TWO ? N : 1];
#pragma unroll
        for (int j = 0; j < N; ++j) { // (past the last share: the last again, not added)
            a[j] = load_f4(sp + min(i + j, p.n_parts - 1) * dp);
            if constexpr (TWO) b[j] = load_f4(sq + min(i + j, q.n_parts - 1) * dq);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const tk_f4 none = {0.f, 0.f, 0.f, 0.f};
            if (i + j >= p.n_parts) a[j] = none;
            if constexpr (TWO) {
                if (i + j >= q.n_parts) b[j] = none;
            }
        }
#pragma unroll
        for (int s = N / 2; s > 0; s /= 2) {
#pragma unroll
            for (int j = 0; j < s; ++j) {
                a[j] += a[j + s];
                if constexpr (TWO) b[j] += b[j + s];
            }
        }
        v += a[0];
        if constexpr (TWO) u += b[0];
    }
}
template <bool TWO>
__device__ __forceinline__ void add_shares(const TokPart &p, const TokPart &q, int T, int t, int64_t row, tk_f4 &v, tk_f4 &u)
{
    const int parts = TWO ? max(p.n_parts, q.n_parts) : p.n_parts;
    if (parts <= 4) add_shares_n<4, TWO>(p, q, T, t, row, v, u);
    else if (parts <= 8) add_shares_n<8, TWO>(p, q, T, t, row, v, u);
    else add_shares_n<16, TWO>(p, q, T, t, row, v, u);
}

// this lane's part of the sums of squares of token t; then 1/rms from those of the wave
__device__ __forceinline__ float squares_of(const TokNorm &nm, int nt, int t, int lane)
{
    float s = lane < nm.nb ? nm.ss[lane * nt + t] : 0.f;
    if (nm.nb > 64)
        for (int b = lane + 64; b < nm.nb; b += 64) s += nm.ss[b * nt + t];
    return s;
}
__device__ __forceinline__ float inv_rms(const TokNorm &nm, float squares)
{
    return 1.0f / sqrtf(wave_sum(squares) / (static_cast<float>(nm.nb) * 256.f) + nm.eps);
}

// Attention's key ranges merged, this lane's four columns of its head (heads: 64 or 128 columns, so several in a wave):
// o = sum_i o_i exp(m_i - M) / sum_i l_i exp(m_i - M); a range without a visible key has (max, sum) = (-inf, 0).  N ranges at a time
template <int N>
__device__ __forceinline__ tk_f4 merge_records(const float *rec, int nsplit, int64_t stride, int c)
{
    float M = -INFINITY, L = 0.f;
    tk_f4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nsplit; s0 += N) {
        tk_f4 o[N];
        float2 ml[N];
#pragma unroll
        for (int i = 0; i < N; ++i) { // (past the last range: the last again, with weight 0)
            const float *r = rec + min(s0 + i, nsplit - 1) * stride;
            ml[i] = *reinterpret_cast<const float2 *>(r);
            o[i] = load_f4(r + ATTN_REC_HDR + c);
        }
        float m = M;
#pragma unroll
        for (int i = 0; i < N; ++i) m = fmaxf(m, ml[i].x);
        const float keep = M == -INFINITY ? 0.f : __expf(M - m);
        acc *= keep;
        L *= keep;
        M = m;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float w = s0 + i >= nsplit || ml[i].x == -INFINITY ? 0.f : __expf(ml[i].x - m);
            L = fmaf(ml[i].y, w, L);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = fmaf(o[i][k], w, acc[k]);
        }
    }
    return acc * (1.0f / L);
}

// A (token, super-block) pair a wave.  Token slots past T: zeros.
template <int NT>
__device__ __forceinline__ void prepare_pair(const TokPrepare &a)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pi = blockIdx.x * ADD_WAVES + wave, t = pi & (NT - 1), b = pi / NT; // (pairs: a multiple of four)
    const int64_t col = static_cast<int64_t>(b) * 256 + lane * 4, K = static_cast<int64_t>(a.nb) * 256;
    tk_f4 v = {0.f, 0.f, 0.f, 0.f};
    if (t < a.T) {
        const tk_f4 one = {1.f, 1.f, 1.f, 1.f};
        const tk_f4 gain = a.gain ? load_f4(a.gain + col) : one;
        if (a.mode == TOK_SWIGLU) {
            const float squares = squares_of(a.norm, NT, t, lane);
            tk_f4 u = v;
            add_shares<true>(a.p[0], a.p[1], a.T, t, col, v, u);
            const float ir = inv_rms(a.norm, squares);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float gt = v[k] * ir;
                v[k] = gt / (1.0f + expf(-gt)) * (u[k] * ir);
            }
        } else if (a.mode == TOK_ATTENTION) {
            const int head = static_cast<int>(col) / a.D, c = static_cast<int>(col) - head * a.D;
            const int64_t stride = ATTN_REC_HDR + a.D;
            const float *rec = a.att.part + (t * (K / a.D) + head) * a.att.nsplit * stride;
            if (a.att.nsplit <= 4) v = merge_records<4>(rec, a.att.nsplit, stride, c);
            else if (a.att.nsplit <= 8) v = merge_records<8>(rec, a.att.nsplit, stride, c);
            else v = merge_records<16>(rec, a.att.nsplit, stride, c);
        } else { // the vector itself, or the residual of the sums
            const tk_f4 x = load_f4(a.x + t * K + col);
            if (a.mode != TOK_PLAIN) add_shares<false>(a.p[0], a.p[0], a.T, t, col, v, v);
            v += x;
        }
        if (a.out) *reinterpret_cast<tk_f4 *>(a.out + t * K + col) = v;
        if (a.gain) {
            const float ss = wave_sum(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]);
            if (lane == 0) a.ss[b * NT + t] = ss;
            v *= gain;
        }
    }
    const float o[4] = {v[0], v[1], v[2], v[3]};
    if (a.rec[0]) tk_split_wave<NT, 0, false>(o, lane, t, a.rec[0] + static_cast<int64_t>(b) * tk_rec(NT));
    if (a.rec[1]) tk_split_wave<NT, 1, true>(o, lane, t, a.rec[1] + static_cast<int64_t>(b) * tk_rec(NT));
}

template <int NT>
__global__ void __launch_bounds__(64 * ADD_WAVES) tok_prepare_kernel(TokPrepare a)
{
    request_args<sizeof(a)>();
    prepare_pair<NT>(a);
}

// A step's first launch: the first layer's activations, and behind them the RoPE table and the counters (3 to 4 us as a launch in front)
template <int NT>
__global__ void __launch_bounds__(64 * ADD_WAVES) tok_first_kernel(TokPrepare a, StepInit s)
{
    const int blocks = a.nb * NT / ADD_WAVES;
    if (static_cast<int>(blockIdx.x) < blocks) prepare_pair<NT>(a);
    else step_init_entry(s, (blockIdx.x - blocks) * (64 * ADD_WAVES) + threadIdx.x);
}

// y[t][row] = 1/rms * sum of the shares (+ residual) of up to three vectors of their own lengths, 256 rows a wave
__global__ void __launch_bounds__(64 * ADD_WAVES) tok_sum_kernel(TokSum a)
{
    request_args<sizeof(a)>();
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = blockIdx.y;
    int64_t first = (static_cast<int64_t>(blockIdx.x) * ADD_WAVES + wave) * 256;
    // which vector: fields as those of the one before and what it has more (picked by a number they are fetched through a picked address)
    const int64_t r0 = (a.rows[0] + 255) / 256 * 256, r1 = r0 + (a.rows[1] + 255) / 256 * 256, r2 = r1 + (a.rows[2] + 255) / 256 * 256;
    const bool one = first >= r0, two = first >= r1;
    if (first >= (a.n == 3 ? r2 : (a.n == 2 ? r1 : r0))) return;
    first -= two ? r1 : (one ? r0 : 0);
    auto pick = [&](auto x, auto y, auto z) { return x + ((one ? y - x : 0) + (two ? z - y : 0)); };
    const TokPart p{pick(a.p[0].part, a.p[1].part, a.p[2].part), pick(a.p[0].n_parts, a.p[1].n_parts, a.p[2].n_parts),
                    pick(a.p[0].rows, a.p[1].rows, a.p[2].rows), pick(a.p[0].row0, a.p[1].row0, a.p[2].row0)};
    const int64_t rows = pick(a.rows[0], a.rows[1], a.rows[2]);
    float *const y = pick(a.y[0], a.y[1], a.y[2]);
    const bool mine = first + lane * 4 < rows; // (rows are a multiple of 16)
    const int64_t row = mine ? first + lane * 4 : 0; // (else a valid address, not stored)
    tk_f4 v = {0.f, 0.f, 0.f, 0.f}, r = v;
    float squares = 0.f;
    if (a.norm.ss) squares = squares_of(a.norm, a.nt, t, lane);
    if (a.resid) r = load_f4(a.resid + t * rows + row);
    add_shares<false>(p, p, a.T, t, row, v, v);
    const float ir = a.norm.ss ? inv_rms(a.norm, squares) : 1.f;
    if (mine) *reinterpret_cast<tk_f4 *>(y + t * rows + row) = v * ir + r;
}

struct StreamPlan {
    int n_slabs, slab, ks_shift, rounds;
    size_t lds;
};

template <int FMT> size_t stage_lds() { return static_cast<size_t>(TkFmt<FMT>::WAVES) * tk_stage_bytes<FMT>; }

// the fewest slabs that any format needs (the one with the largest stage buffers)
int most_slabs(int nb, int nt)
{
    const int cap = static_cast<int>((TK_LDS - stage_lds<PRIMA_FMT_Q8_0>()) / tk_rec(nt)) / 2 * 2;
    return (nb + cap - 1) / cap;
}

// Slabs of K and parts of a slab: by the longest wave's stages, what a workgroup copies and the shares' traffic.
// Times in units of a stage of a wave (about 2.2 us with two waves a SIMD).
template <int FMT>
StreamPlan plan_stream(int n_tiles, int nb, int nt)
{
    constexpr int SBS = TkFmt<FMT>::SBS, WAVES = TkFmt<FMT>::WAVES;
    const int cap = static_cast<int>((TK_LDS - stage_lds<FMT>()) / tk_rec(nt)) / SBS * SBS;
    const int min_slabs = (nb + cap - 1) / cap, max_parts = tok_max_parts(nb, nt, static_cast<int64_t>(n_tiles) * 16);
    StreamPlan best{};
    double best_t = 0.;
    for (int ns = min_slabs; ns <= std::min(max_parts, 2 * min_slabs + 6) && ns <= TK_CUS; ++ns) {
        const int slab = ((nb + ns - 1) / ns + SBS - 1) / SBS * SBS;
        if ((nb + slab - 1) / slab != ns) continue; // rounding to whole stages merged two slabs
        const int last = (nb - (ns - 1) * slab + SBS - 1) / SBS; // stages of the last slab
        const int ranks = TK_CUS / ns;
        for (int sh = 0; (1 << sh) <= WAVES && (1 << sh) <= last && (ns << sh) <= max_parts; ++sh) {
            const int per_round = ranks * (WAVES >> sh), rounds = (n_tiles + per_round - 1) / per_round;
            const int part = (slab / SBS + (1 << sh) - 1) >> sh;
            const double t = static_cast<double>(rounds) * part * (SBS == 2 ? 1.0 : 0.6) + 0.04 * slab * nt / 8 +
                             static_cast<double>(ns << sh) * n_tiles * 16 * nt * 8 / 8e6; // (written and read, about 4 TB/s)
            if (best_t == 0. || t < best_t * 0.999) {
                best_t = t;
                best = StreamPlan{ns, slab, sh, rounds, stage_lds<FMT>() + static_cast<size_t>(slab) * tk_rec(nt)};
            }
        }
    }
    return best;
}

template <int FMT, int NT>
prima_status launch_nt(StreamArgs &a, const StreamPlan &p, hipStream_t st)
{
    static std::atomic<bool> attr_set{false}; // set twice by two threads at worst: the attribute call is idempotent
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(tok_stream_kernel<FMT, NT>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(TK_LDS)) != hipSuccess)
            return PRIMA_E_DEVICE;
        attr_set = true;
    }
    const int grid = std::min<int64_t>(TK_CUS, static_cast<int64_t>(a.n_tiles) * a.n_slabs);
    a.wg_slab = grid / a.n_slabs; a.wg_more = grid % a.n_slabs;
    a.slab_magic = static_cast<unsigned>((uint64_t{1} << 32) / a.n_slabs + 1); // exact: a workgroup's number times n_slabs is far below 2^32
    hipLaunchKernelGGL((tok_stream_kernel<FMT, NT>), dim3(grid), dim3(TkFmt<FMT>::WAVES * 64), p.lds, st, a);
    return last_launch_status();
}

// launches, or plans only
template <int FMT>
prima_status launch_fmt(StreamArgs &a, size_t part_floats, int &n_parts, bool plan_only, hipStream_t st)
{
    const int nt = tok_slots(a.T);
    const StreamPlan p = plan_stream<FMT>(a.n_tiles, a.nb, nt);
    if (p.n_slabs == 0) return PRIMA_E_SHAPE;
    a.n_slabs = p.n_slabs; a.slab = p.slab; a.ks_shift = p.ks_shift; a.rounds = p.rounds;
    a.per_round = (a.n_tiles + p.rounds - 1) / p.rounds;
    n_parts = p.n_slabs << p.ks_shift;
    if (static_cast<size_t>(n_parts) * a.T * a.n_tiles * 16 > part_floats) return PRIMA_E_WORKSPACE;
    if (plan_only) return p.lds > TK_LDS ? PRIMA_E_SHAPE : PRIMA_OK;
    if (nt == 16) return launch_nt<FMT, 16>(a, p, st);
    return nt == 8 ? launch_nt<FMT, 8>(a, p, st) : launch_nt<FMT, 4>(a, p, st);
}

prima_status launch_any(int fmt, StreamArgs &a, size_t part_floats, int &n_parts, bool plan_only, hipStream_t st)
{
    switch (fmt) {
    case PRIMA_FMT_Q4_K: return launch_fmt<PRIMA_FMT_Q4_K>(a, part_floats, n_parts, plan_only, st);
    case PRIMA_FMT_Q5_K: return launch_fmt<PRIMA_FMT_Q5_K>(a, part_floats, n_parts, plan_only, st);
    case PRIMA_FMT_Q6_K: return launch_fmt<PRIMA_FMT_Q6_K>(a, part_floats, n_parts, plan_only, st);
    case PRIMA_FMT_Q8_0: return launch_fmt<PRIMA_FMT_Q8_0>(a, part_floats, n_parts, plan_only, st);
    case PRIMA_FMT_F16: return launch_fmt<PRIMA_FMT_F16>(a, part_floats, n_parts, plan_only, st);
    default: return PRIMA_E_SHAPE;
    }
}

} // namespace

// Tall launches fill the device without many shares (57344 x 8192 takes 8 at 16 tokens, 4 at 8), and theirs are the largest of the scratch.
int tok_max_parts(int nb, int nt, int64_t n_rows)
{
    const int least = most_slabs(nb, nt);
    return n_rows > 12288 ? std::max(8, least) : std::max(16, 2 * least);
}
size_t tok_rec_bytes(int64_t n_cols, int T) { return static_cast<size_t>(n_cols / QK) * tk_rec(tok_slots(T)); }
size_t tok_part_floats(int64_t n_rows, int64_t n_cols, int T)
{
    return static_cast<size_t>(tok_max_parts(static_cast<int>(n_cols / QK), tok_slots(T), n_rows)) * T * static_cast<size_t>(n_rows);
}
size_t tok_ss_bytes(int64_t n_cols, int T) { return static_cast<size_t>(n_cols / QK) * tok_slots(T) * sizeof(float); }
int tok_slots(int T) { return std::max(4, tk_slots(T)); }

prima_status tok_stream_plan_status(int fmt, int64_t n_rows, int64_t n_cols, int T, size_t part_floats)
{
    StreamArgs a{};
    a.nb = static_cast<int>(n_cols / QK); a.T = T; a.n_tiles = static_cast<int>(n_rows / 16);
    int n_parts = 0;
    return launch_any(fmt, a, part_floats, n_parts, true, nullptr);
}

prima_status launch_tok_stream(int fmt, const TokMat *mats, int n_mats, int64_t n_cols, const uint8_t *rec, int T, float *part, size_t part_floats,
                               TokPart *out, hipStream_t st)
{
    StreamArgs a{};
    int64_t tiles = 0;
    for (int i = 0; i < 3; ++i) {
        a.seg[i].tile0 = 0x7fffffff;
        if (i >= n_mats) continue;
        a.seg[i] = StreamSeg{mats[i].W, mats[i].n_rows, static_cast<int>(tiles)};
        tiles += mats[i].n_rows / 16;
    }
    if (tiles >= (int64_t{1} << 27) || n_cols / QK >= (1 << 18)) return PRIMA_E_SHAPE;
    a.rec = rec; a.part = part; a.nb = static_cast<int>(n_cols / QK); a.T = T; a.n_tiles = static_cast<int>(tiles);
    int n_parts = 0;
    const prima_status s = launch_any(fmt, a, part_floats, n_parts, false, st);
    for (int i = 0; i < n_mats; ++i) out[i] = TokPart{part, n_parts, tiles * 16, static_cast<int64_t>(a.seg[i].tile0) * 16};
    return s;
}

prima_status launch_tok_prepare(const TokPrepare &a, const StepInit &init, hipStream_t st)
{
    const int nt = tok_slots(a.T), grid = a.nb * nt / ADD_WAVES;
    static_assert(ADD_WAVES == 4, "step_init_blocks() counts blocks of 256 threads");
    if (init.tab) {
        const dim3 more(grid + step_init_blocks(init));
        switch (nt) {
        case 4: hipLaunchKernelGGL((tok_first_kernel<4>), more, dim3(64 * ADD_WAVES), 0, st, a, init); break;
        case 8: hipLaunchKernelGGL((tok_first_kernel<8>), more, dim3(64 * ADD_WAVES), 0, st, a, init); break;
        case 16: hipLaunchKernelGGL((tok_first_kernel<16>), more, dim3(64 * ADD_WAVES), 0, st, a, init); break;
        default: return PRIMA_E_SHAPE;
        }
        return last_launch_status();
    }
    switch (nt) {
    case 4: hipLaunchKernelGGL((tok_prepare_kernel<4>), dim3(grid), dim3(64 * ADD_WAVES), 0, st, a); break;
    case 8: hipLaunchKernelGGL((tok_prepare_kernel<8>), dim3(grid), dim3(64 * ADD_WAVES), 0, st, a); break;
    case 16: hipLaunchKernelGGL((tok_prepare_kernel<16>), dim3(grid), dim3(64 * ADD_WAVES), 0, st, a); break;
    default: return PRIMA_E_SHAPE;
    }
    return last_launch_status();
}

prima_status launch_tok_sum(const TokSum &a, hipStream_t st)
{
    int64_t groups = 0;
    for (int i = 0; i < a.n; ++i) groups += (a.rows[i] + 255) / 256;
    hipLaunchKernelGGL(tok_sum_kernel, dim3(static_cast<unsigned>((groups + 3) / 4), a.T), dim3(64 * ADD_WAVES), 0, st, a);
    return last_launch_status();
}

} // namespace prima
