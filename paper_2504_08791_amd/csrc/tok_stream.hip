// The projections of a layer window for 9 to 16 tokens (speculative verification, batches of sequences), and for 4 to 8 those in other
// formats than Q4_K: mat-vecs on the matrix
// cores over activations that are prepared once per projection, with the sums finished by the kernel that prepares the next
// one.  Arithmetic and layouts: tok_common.h.
//
//   tok_stream_kernel   the weight stream: every format but FP32.  K is cut into slabs whose activations fit in LDS beside the
//                       waves' stage buffers; a workgroup copies its slab's records (one pass over L2, no arithmetic) and
//                       its waves stream (tile, part of the slab) units.  A unit's sums go to global memory, nothing meets
//                       inside the launch: no barrier behind the first, no arrival counts, no waiting.
//   tok_prepare_kernel  adds the shares of K in a fixed order, finishes them (residual, or 1/rms and SwiGLU), stores the vector
//                       where it is needed and lays it out as the next projection's activations (gain applied; its sums of
//                       squares beside it: 1/rms multiplies the finished sums of the next projection).
//   tok_sum_kernel      adds the shares where plain vectors are wanted (Q, K, V; the window's output).
//
// The Q4_K mat-vec of one to eight tokens (q4k_gemv_mfma.hip) takes 16 tokens in two passes over the weights; here one pass
// serves them.  A 14B-shaped layer, 16 sequences, us with the tracer: Q/K/V 38 -> 19, output 31 -> 21, gate and up 65 -> 38,
// down 44 -> 25 (adding and preparing included); the batch step of three layers 586 -> 380.  What bounds the stream at 16
// tokens: 27648 x 5120 (80 MB, 12 us at the rate of a linear read) takes 30 us, 21 without its products, 31 without its
// loads: the LDS reads of the operands (17 KB a super-block and wave) and the unpacking under two waves a SIMD.
// From four tokens on the other formats' matrices of a window come here too (prepared, streamed and added each group for itself).
// Up to eight tokens the Q4_K kernel stays the better one (start / this, us: four layers of a 32B shape at 4 tokens 457 / 523, two of a 70B
// shape at 8 364 / 379): the launches between the streams cost 4 to 5 us each and the streams gain less than that.
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
};

template <int FMT, int NT>
__global__ void __launch_bounds__(TkFmt<FMT>::WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) tok_stream_kernel(StreamArgs a)
{
    extern __shared__ __align__(16) uint8_t smem[];
    constexpr int SBS = TkFmt<FMT>::SBS, WAVES = TkFmt<FMT>::WAVES;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    uint8_t *const l_stage = smem + wave * tk_stage_bytes<FMT>;
    uint8_t *const l_a = smem + WAVES * tk_stage_bytes<FMT>;

    const int rank = static_cast<int>(blockIdx.x) / a.n_slabs, slab = static_cast<int>(blockIdx.x) - rank * a.n_slabs;
    const int ranks = (static_cast<int>(gridDim.x) - slab + a.n_slabs - 1) / a.n_slabs; // workgroups of this slab
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
    int n_active = 0;
    {
        int tile;
        for (int k = next_round(0, tile); k < a.rounds; k = next_round(k + 1, tile)) ++n_active;
    }
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
            const int sg = tile >= a.seg[2].tile0 ? 2 : (tile >= a.seg[1].tile0 ? 1 : 0);
            const uint8_t *W = sg == 0 ? a.seg[0].W : (sg == 1 ? a.seg[1].W : a.seg[2].W);
            const int64_t n_rows = sg == 0 ? a.seg[0].n_rows : (sg == 1 ? a.seg[1].n_rows : a.seg[2].n_rows);
            const int first = sg == 0 ? a.seg[0].tile0 : (sg == 1 ? a.seg[1].tile0 : a.seg[2].tile0);
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

// Sum over the shares of 16 consecutive rows (this lane's) of a token.  The shares come from other XCDs, a trip through memory
// each: the four waves of a workgroup take every fourth share, up to four of them at a time, and wave 0 adds the waves' sums
// in order (one wave adding two shares at a time took 5 to 8 us a launch).
constexpr int ADD_WAVES = 4;
__device__ __forceinline__ void add_shares(const TokPart &p, int T, int t, int64_t row, int wave, float (&v)[16])
{
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = 0.f;
    const float *s = p.part + t * p.rows + p.row0 + row;
    const int64_t stride = static_cast<int64_t>(T) * p.rows;
    for (int i = wave; i < p.n_parts; i += 4 * ADD_WAVES) {
        float4 a[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float *sj = s + min(i + j * ADD_WAVES, p.n_parts - 1) * stride; // (past the last: the last again, not added)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[j][k] = *reinterpret_cast<const float4 *>(sj + 4 * k);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i + j * ADD_WAVES < p.n_parts) {
#pragma unroll
                for (int k = 0; k < 4; ++k) { v[4 * k] += a[j][k].x; v[4 * k + 1] += a[j][k].y; v[4 * k + 2] += a[j][k].z; v[4 * k + 3] += a[j][k].w; }
            }
        }
    }
}
// wave 0's v becomes the sum over the waves' (all threads; `buf`: 12 KiB of LDS)
__device__ __forceinline__ void add_waves(float (&v)[16], int wave, int lane, float4 (*buf)[4][64])
{
    if (wave != 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) buf[wave - 1][k][lane] = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 0; w < ADD_WAVES - 1; ++w)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 q = buf[w][k][lane];
                v[4 * k] += q.x; v[4 * k + 1] += q.y; v[4 * k + 2] += q.z; v[4 * k + 3] += q.w;
            }
    }
}

// 1/rms of token t from the sums of squares of its super-blocks; sixteen lanes together (i: lane in the group)
__device__ __forceinline__ float inv_rms(const TokNorm &nm, int nt, int t, int i)
{
    float s = 0.f;
    for (int b = i; b < nm.nb; b += 16) s += nm.ss[b * nt + t];
    return 1.0f / sqrtf(row_sum16(s) / (static_cast<float>(nm.nb) * 256.f) + nm.eps);
}

// Four (token, super-block) pairs a workgroup, one per 16 lanes.  Token slots past T: zeros.
template <int NT>
__global__ void __launch_bounds__(64 * ADD_WAVES) tok_prepare_kernel(TokPrepare a)
{
    __shared__ float4 buf[2][ADD_WAVES - 1][4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15;
    const int pi = blockIdx.x * 4 + (lane >> 4), t = pi & (NT - 1), b = pi / NT; // (pairs: a multiple of four)
    const int64_t col = static_cast<int64_t>(b) * 256 + n * 16, K = static_cast<int64_t>(a.nb) * 256;
    const int ts = min(t, a.T - 1); // (a slot past the last token reads the last)
    float v[16], u[16];
    if (a.mode != TOK_PLAIN) {
        add_shares(a.p[0], a.T, ts, col, wave, v);
        if (a.mode == TOK_SWIGLU) {
            add_shares(a.p[1], a.T, ts, col, wave, u);
            add_waves(u, wave, lane, buf[1]);
        }
        add_waves(v, wave, lane, buf[0]);
    }
    if (wave != 0) return;
    if (a.mode == TOK_SWIGLU) {
        const float ir = inv_rms(a.norm, NT, ts, n);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float gt = v[k] * ir;
            v[k] = gt / (1.0f + expf(-gt)) * (u[k] * ir);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) { // the vector itself, or the residual of the sums
            const float4 q = *reinterpret_cast<const float4 *>(a.x + ts * K + col + 4 * k);
            const float r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * k + e] = a.mode == TOK_PLAIN ? r[e] : v[4 * k + e] + r[e];
        }
    }
    if (t >= a.T) {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = 0.f;
    } else if (a.out) {
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<float4 *>(a.out + t * K + col + 4 * k) = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    }
    if (a.gain) {
        float ss = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) ss += v[k] * v[k];
        ss = row_sum16(ss);
        if (n == 0) a.ss[b * NT + t] = ss;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 q = *reinterpret_cast<const float4 *>(a.gain + col + 4 * k);
            v[4 * k] *= q.x; v[4 * k + 1] *= q.y; v[4 * k + 2] *= q.z; v[4 * k + 3] *= q.w;
        }
    }
    if (a.rec[0]) tk_split<NT, 0, false, true>(v, n, t, a.rec[0] + static_cast<int64_t>(b) * tk_rec(NT));
    if (a.rec[1]) tk_split<NT, 1, true, true>(v, n, t, a.rec[1] + static_cast<int64_t>(b) * tk_rec(NT));
}

// y[t][row] = 1/rms * sum of the shares (+ residual) of up to three vectors of their own lengths, 256 rows per 16 lanes
__global__ void __launch_bounds__(64 * ADD_WAVES) tok_sum_kernel(TokSum a)
{
    __shared__ float4 buf[ADD_WAVES - 1][4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15;
    const int t = blockIdx.y;
    int64_t row = (static_cast<int64_t>(blockIdx.x) * 4 + (lane >> 4)) * 256 + n * 16;
    int i = 0;
    while (i < a.n && row >= (a.rows[i] + 255) / 256 * 256) { row -= (a.rows[i] + 255) / 256 * 256; ++i; }
    const bool mine = i < a.n && row < a.rows[i < 3 ? i : 2]; // (rows are a multiple of 16)
    const int j = mine ? i : 0;
    const TokPart p = j == 0 ? a.p[0] : (j == 1 ? a.p[1] : a.p[2]);
    const int64_t rows = j == 0 ? a.rows[0] : (j == 1 ? a.rows[1] : a.rows[2]);
    float *const y = j == 0 ? a.y[0] : (j == 1 ? a.y[1] : a.y[2]);
    if (!mine) row = 0; // (a valid address, not stored)
    float v[16];
    add_shares(p, a.T, t, row, wave, v);
    add_waves(v, wave, lane, buf);
    if (wave != 0) return;
    const float ir = a.norm.ss ? inv_rms(a.norm, a.nt, t, n) : 1.f;
    if (!mine) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float4 o = make_float4(v[4 * k] * ir, v[4 * k + 1] * ir, v[4 * k + 2] * ir, v[4 * k + 3] * ir);
        if (a.resid) {
            const float4 q = *reinterpret_cast<const float4 *>(a.resid + t * rows + row + 4 * k);
            o.x += q.x; o.y += q.y; o.z += q.z; o.w += q.w;
        }
        *reinterpret_cast<float4 *>(y + t * rows + row + 4 * k) = o;
    }
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
    hipLaunchKernelGGL((tok_stream_kernel<FMT, NT>), dim3(grid), dim3(TkFmt<FMT>::WAVES * 64), p.lds, st, a);
    return last_launch_status();
}

// launches, or plans only
template <int FMT>
prima_status launch_fmt(StreamArgs &a, size_t part_floats, int &n_parts, bool plan_only, hipStream_t st)
{
    const int nt = tk_slots(a.T);
    const StreamPlan p = plan_stream<FMT>(a.n_tiles, a.nb, nt);
    if (p.n_slabs == 0 || nt < (FMT == PRIMA_FMT_Q4_K ? 16 : 4)) return PRIMA_E_SHAPE;
    a.n_slabs = p.n_slabs; a.slab = p.slab; a.ks_shift = p.ks_shift; a.rounds = p.rounds;
    a.per_round = (a.n_tiles + p.rounds - 1) / p.rounds;
    n_parts = p.n_slabs << p.ks_shift;
    if (static_cast<size_t>(n_parts) * a.T * a.n_tiles * 16 > part_floats) return PRIMA_E_WORKSPACE;
    if (plan_only) return p.lds > TK_LDS ? PRIMA_E_SHAPE : PRIMA_OK;
    if (nt == 16) return launch_nt<FMT, 16>(a, p, st);
    if constexpr (FMT != PRIMA_FMT_Q4_K) { // (Q4_K: windows of 9 to 16 tokens only, see window.hip)
        if (nt == 4) return launch_nt<FMT, 4>(a, p, st);
        if (nt == 8) return launch_nt<FMT, 8>(a, p, st);
    }
    return PRIMA_E_SHAPE;
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
size_t tok_rec_bytes(int64_t n_cols, int T) { return static_cast<size_t>(n_cols / QK) * tk_rec(tk_slots(T)); }
size_t tok_part_floats(int64_t n_rows, int64_t n_cols, int T)
{
    return static_cast<size_t>(tok_max_parts(static_cast<int>(n_cols / QK), tk_slots(T), n_rows)) * T * static_cast<size_t>(n_rows);
}
size_t tok_ss_bytes(int64_t n_cols, int T) { return static_cast<size_t>(n_cols / QK) * tk_slots(T) * sizeof(float); }
int tok_slots(int T) { return tk_slots(T); }

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

prima_status launch_tok_prepare(const TokPrepare &a, hipStream_t st)
{
    const int nt = tk_slots(a.T), grid = a.nb * nt / 4;
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
