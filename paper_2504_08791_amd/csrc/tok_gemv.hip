// Mat-vec of 2 to 16 tokens for weights in the other formats (Q5_K, Q6_K, Q8_0, FP16), and of 9 to 16 (11 to 16) for tall Q4_K matrices,
// without scratch: the kernel behind prima_fmt_gemv and prima_lm_head_fmt for several tokens (one token: fmt_gemv.hip), and
// behind prima_q4k_gemv and prima_lm_head where tok_gemv_takes() says so.  Arithmetic and layouts: tok_common.h.
//
// One workgroup of 8 waves per compute unit.  It owns a share of the 16-row tiles and walks all of K in chunks: the
// activations of a chunk (all tokens) are normalised, split and laid out in LDS by the workgroup, then the waves stream
// their units (a tile, or with few tiles a part of the chunk of one) against them; a unit's sums stay in LDS from chunk to
// chunk.  The weight stream runs ahead by two stages in registers and does not stop between chunks.  1 / rms multiplies the
// finished sums, so that no pass over the activations is needed in front.
//
// What bounds it: the output layer 128256 x 8192 in Q6_K at 8 tokens takes 203 us (4.2 TB/s of weights; the fp32 mat-vec took
// 514 to 578): its stream alone, products left out, 156 us; its products alone, requests left out, 178 us (200 vector
// instructions a super-block and tile, and the latencies of its LDS reads and matrix instructions under two waves a SIMD).
// FP16 and Q8_0, with little to unpack, run at 6.1 and 5.9 TB/s.  Sixteen waves of half the stage were slower (253 us: fields
// of 2 to 64 bytes a row and stage are then fetched twice as often).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "tok_common.h"

namespace prima {
namespace {

struct TokArgs {
    const uint8_t *W;
    int64_t n_rows;
    int nb; // super-blocks of a row
    const float *x;
    int64_t ldx;
    const float *gain; // null: plain activations
    float eps;
    const float *resid; // null: none
    int64_t ldr;
    float *y;
    int64_t ldy;
    int T;
    int n_tiles;  // 16-row tiles
    int chunk;    // super-blocks per chunk of K (a multiple of the stage's)
    int ks_shift; // a unit is one of 2^ks_shift parts of a (tile, chunk)
    // Rounds: in each every wave has one unit at most.  Round k covers tiles k per_round .. (k + 1) per_round - 1 (the last: what is left, maybe
    // none), dealt to the workgroups one by one (a run of neighbouring tiles for each was measured 3 to 10 % slower: the requests of the
    // device then crowd on fewer memory channels).  (Rounds of n_tiles k / rounds tiles took some 600 scalar instructions of division per
    // unit and wave, a fifth of its time at 8 tokens.)
    int rounds, per_round, blk_rounds; // blk_rounds: whose sums are in LDS at a time
};

// LDS: the waves' stage buffers | activations [chunk] | sums of squares [chunk][NT] | 1/rms [NT] |
// units' sums [blk_rounds][waves][NT][16]
template <int FMT, int NT>
__global__ void __launch_bounds__(TkFmt<FMT>::WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) tok_gemv_kernel(TokArgs a)
{
    extern __shared__ __align__(16) uint8_t smem[];
    constexpr int SBS = TkFmt<FMT>::SBS, WAVES = TkFmt<FMT>::WAVES, THREADS = WAVES * 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    uint8_t *const l_stage = smem + wave * tk_stage_bytes<FMT>;
    uint8_t *const l_a = smem + WAVES * tk_stage_bytes<FMT>;
    float *const l_ss = reinterpret_cast<float *>(l_a + a.chunk * tk_rec(NT));
    float *const l_rms = l_ss + a.chunk * NT;
    float *const l_acc = l_rms + NT;

    const int ks_shift = a.ks_shift, ks = 1 << ks_shift, nb = a.nb, chunk = a.chunk;
    const int my_l = wave >> ks_shift, part = wave & (ks - 1); // this wave's tile of a round's and its part
    const int my_tile = static_cast<int>(blockIdx.x) + my_l * static_cast<int>(gridDim.x); // counted from the round's first
    // the first round from k on in which this wave has a tile (k_end: none), and the tile
    auto next_round = [&](int k, int k_end, int &tile) __attribute__((always_inline)) {
        tile = k * a.per_round + my_tile;
        if (my_tile >= a.per_round || tile >= a.n_tiles) return k_end;
        return min(k, k_end);
    };
    // stages [s0, s1) of the chunk of `len` super-blocks are this wave's part (never empty: the host keeps ks <= a chunk's stages)
    auto part_of = [&](int len, int &s0, int &s1) __attribute__((always_inline)) {
        const int stages = (len + SBS - 1) / SBS;
        s0 = (stages * part) >> ks_shift;
        s1 = (stages * (part + 1)) >> ks_shift;
    };

    for (int k0 = 0; k0 < a.rounds; k0 += a.blk_rounds) {
        const int k_end = min(k0 + a.blk_rounds, a.rounds);
        int n_active = 0; // rounds in which this wave has a tile
        {
            int tile;
            for (int k = next_round(k0, k_end, tile); k < k_end; k = next_round(k + 1, k_end, tile)) ++n_active;
        }
        // The requesting side of the wave's stream of stages: chunk by chunk, round by round, stage by stage.  A wave's stages of
        // a chunk come in pairs, one for each of its two sets of registers (so that the loads in flight behind a set are the
        // same on every path and the compiler's wait in front of its use leaves them out): an odd number is padded with a
        // stage that is requested again and not used; so is whatever is requested past the end.
        TkSrc<FMT> src;
        int ld_sb0 = 0, ld_len = min(chunk, nb), ld_k = k0 - 1, ld_b = 0, ld_left = 0, ld_step = SBS;
        bool ld_padded = false;
        auto ld_next = [&]() __attribute__((always_inline)) { // a unit has been requested to its end
            for (;;) {
                int s0, s1;
                part_of(ld_len, s0, s1);
                if (!ld_padded) {
                    int tile;
                    const int k = next_round(ld_k + 1, k_end, tile);
                    if (k < k_end) {
                        ld_k = k;
                        ld_b = ld_sb0 + s0 * SBS;
                        ld_left = s1 - s0;
                        tk_tile<FMT>(src, a.W, a.n_rows, nb, static_cast<int64_t>(tile) * 16, lane);
                        return;
                    }
                    if (((s1 - s0) * n_active) & 1) { ld_padded = true; ld_b -= ld_step; ld_left = 1; return; }
                }
                if (ld_sb0 + ld_len >= nb) { ld_b -= ld_step; ld_step = 0; ld_left = 0x7fffffff; return; }
                ld_sb0 += ld_len;
                ld_len = min(chunk, nb - ld_sb0);
                ld_k = k0 - 1;
                ld_padded = false;
            }
        };
        TkRegs<FMT> r0, r1;
        auto request = [&](TkRegs<FMT> &r) __attribute__((always_inline)) {
            tk_load<FMT>(r, src, max(min(ld_b, nb - SBS), 0)); // (the last stage of an odd number of super-blocks: its second one)
            ld_b += ld_step;
            if (--ld_left == 0) ld_next();
        };

        float ss_run = 0.f; // sum of squares of token threadIdx.x
        for (int i = threadIdx.x; i < (k_end - k0) * WAVES * NT * 16; i += THREADS) l_acc[i] = 0.f;
        if (n_active != 0) { // (else this wave has nothing to request in any chunk)
            ld_next();
            request(r0);
            request(r1);
        }

        for (int sb0 = 0; sb0 < nb; sb0 += chunk) {
            const int nsb = min(chunk, nb - sb0);
            __syncthreads(); // the previous chunk's operands have been used (and the sums' region is clear)
            for (int p0 = 0; p0 < nsb * NT; p0 += WAVES * 4) {
                const int pi = p0 + wave * 4 + g;
                const int t = pi & (NT - 1), b = pi / NT;
                if (b < nsb) {
                    float v[16], ss = 0.f;
                    const bool real = t < a.T;
                    const int64_t col = static_cast<int64_t>(sb0 + b) * 256 + n * 16;
                    const float *xp = a.x + (real ? t : 0) * a.ldx + col;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float4 q = *reinterpret_cast<const float4 *>(xp + 4 * k);
                        v[4 * k] = q.x; v[4 * k + 1] = q.y; v[4 * k + 2] = q.z; v[4 * k + 3] = q.w;
                    }
                    if (!real) {
#pragma unroll
                        for (int k = 0; k < 16; ++k) v[k] = 0.f;
                    }
                    if (a.gain) {
#pragma unroll
                        for (int k = 0; k < 16; ++k) ss += v[k] * v[k];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float4 q = *reinterpret_cast<const float4 *>(a.gain + col + 4 * k);
                            v[4 * k] *= q.x; v[4 * k + 1] *= q.y; v[4 * k + 2] *= q.z; v[4 * k + 3] *= q.w;
                        }
                        ss = row_sum16(ss);
                        if (n == 0) l_ss[b * NT + t] = ss;
                    }
                    tk_split<NT, TkFmt<FMT>::ORD, FMT == PRIMA_FMT_Q8_0 || FMT == PRIMA_FMT_F16, FMT == PRIMA_FMT_Q4_K || FMT == PRIMA_FMT_Q5_K>(v, n, t, l_a + b * tk_rec(NT));
                }
            }
            __syncthreads();
            if (a.gain && threadIdx.x < NT) {
                for (int b = 0; b < nsb; ++b) ss_run += l_ss[b * NT + threadIdx.x];
                if (sb0 + nsb == nb) l_rms[threadIdx.x] = 1.0f / sqrtf(ss_run / (static_cast<float>(nb) * 256.f) + a.eps);
            }
            // ---- this wave's stages of the chunk ----
            int s0, s1;
            part_of(nsb, s0, s1);
            const int total = (s1 - s0) * n_active;
            int tile, k = next_round(k0, k_end, tile), s = s0;
            float y[4] = {0.f, 0.f, 0.f, 0.f};
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
                    if (++s == s1) { // the unit ends: its sums of this chunk (lanes past the token slots repeat others)
                        float *dst = l_acc + ((k - k0) * WAVES + wave) * (NT * 16) + n;
                        constexpr int NY = NT <= 8 ? 2 : 4;
                        if (NT >= 8 || g < NT / 2) {
#pragma unroll
                            for (int i = 0; i < NY; ++i) dst[(NY * g + i) * 16] += y[i];
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) y[i] = 0.f;
                        s = s0;
                        k = next_round(k + 1, k_end, tile);
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
        __syncthreads();
        // ---- a unit's parts in order, 1/rms, the residual ----
        for (int k = k0; k < k_end; ++k) {
            // this workgroup's tiles of the round: first + i * gridDim.x, i < count
            const int first = k * a.per_round + static_cast<int>(blockIdx.x);
            const int left = min(a.per_round, a.n_tiles - k * a.per_round) - static_cast<int>(blockIdx.x);
            const int count = left > 0 ? static_cast<int>((static_cast<unsigned>(left) + gridDim.x - 1) / gridDim.x) : 0;
            const int n_out = count * 16 * a.T;
            for (int idx = threadIdx.x; idx < n_out; idx += THREADS) {
                const int l = idx / (16 * a.T), rem = idx - l * (16 * a.T), t = rem >> 4, j = rem & 15;
                const int64_t row = (first + static_cast<int64_t>(l) * gridDim.x) * 16 + j;
                if (row >= a.n_rows) continue;
                const float *u = l_acc + ((k - k0) * WAVES + (l << ks_shift)) * (NT * 16) + t * 16 + j;
                float v = u[0];
                for (int p = 1; p < ks; ++p) v += u[p * (NT * 16)];
                if (a.gain) v *= l_rms[t];
                if (a.resid) v += a.resid[t * a.ldr + row];
                a.y[t * a.ldy + row] = v;
            }
        }
        __syncthreads(); // the sums' region and 1/rms are used again
    }
}

int grid_of(const TokArgs &a) { return std::min(a.n_tiles, TK_CUS); }

// chunks of K, parts of a unit and rounds (into a); the LDS they take
template <int FMT, int NT>
prima_status plan_nt(TokArgs &a, size_t &lds)
{
    constexpr int SBS = TkFmt<FMT>::SBS, WAVES = TkFmt<FMT>::WAVES;
    constexpr size_t per_sb = tk_rec(NT) + 4 * NT, fixed = WAVES * tk_stage_bytes<FMT> + NT * 4;
    const int grid = grid_of(a);
    // Parts of a unit: with few tiles the waves share them (what the longest wave has to do counts); the sums of a workgroup's
    // units take at most 32 KiB, more rounds than that are worked off in blocks, each with a walk over K of its own.
    constexpr int ROUND_BYTES = WAVES * NT * 64, MAX_BLK = 32 * 1024 / ROUND_BYTES;
    double best = 0.;
    for (int sh = 0; (1 << sh) <= WAVES; ++sh) {
        const int64_t per_round = static_cast<int64_t>(grid) * (WAVES >> sh);
        const int rounds = static_cast<int>((a.n_tiles + per_round - 1) / per_round), blk = std::min(rounds, MAX_BLK);
        int chunk = static_cast<int>((TK_LDS - fixed - static_cast<size_t>(blk) * ROUND_BYTES) / per_sb) / SBS * SBS;
        const int n_chunks = (a.nb + chunk - 1) / chunk;
        chunk = ((a.nb + n_chunks - 1) / n_chunks + SBS - 1) / SBS * SBS;
        const int last = a.nb - (a.nb - 1) / chunk * chunk; // super-blocks of the last chunk
        if (sh > 0 && (1 << sh) > (last + SBS - 1) / SBS) continue; // every part of every chunk has a stage
        // A chunk costs its operands (about two stages' time) and, round by round, the longest part and half a stage for the unit (its
        // addresses and sums; without that tall matrices went in eighths: Q6_K 100000 x 4096, 2 tokens, 109 us, now 80).  A wave requests its stages of
        // a chunk in pairs; where the stream bounds the launch the odd one counts (us, not counted / counted, 8 tokens: FP16
        // 8192 x 1024 11.6 / 8.8, 4096 x 8192 34 / 30, Q8_0 8192 x 4096 26 / 19; in Q6_K and Q5_K, which unpack longer
        // than they load, 4096 x 2048 would go from 9.4 to 10.2).
        const int part = (chunk / SBS + (1 << sh) - 1) >> sh, blocks = (rounds + blk - 1) / blk, last_blk = rounds - (blocks - 1) * blk;
        const bool padding = FMT == PRIMA_FMT_F16 || (FMT == PRIMA_FMT_Q8_0 && NT <= 8 && a.n_tiles > grid);
        auto requested = [&](int stages) { return padding ? (stages + 1) / 2 * 2 : stages; };
        const double t = static_cast<double>(n_chunks) * (2.0 * blocks + 0.5 * rounds + (blocks - 1) * requested(blk * part) + requested(last_blk * part));
        if (sh == 0 || t < best * 0.999) {
            best = t;
            a.ks_shift = sh;
            a.rounds = rounds;
            a.per_round = (a.n_tiles + rounds - 1) / rounds;
            a.blk_rounds = blk;
            a.chunk = chunk;
        }
    }
    lds = fixed + static_cast<size_t>(a.chunk) * per_sb + static_cast<size_t>(a.blk_rounds) * ROUND_BYTES;
    return lds > TK_LDS || a.chunk < SBS ? PRIMA_E_SHAPE : PRIMA_OK; // (the smallest chunk fits beside the largest sums)
}

// launches, or plans only
template <int FMT, int NT>
prima_status launch_nt(TokArgs a, bool plan_only, hipStream_t st)
{
    size_t lds = 0;
    const prima_status s = plan_nt<FMT, NT>(a, lds);
    if (s != PRIMA_OK || plan_only) return s;
    static std::atomic<bool> attr_set{false}; // set twice by two threads at worst: the attribute call is idempotent
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(tok_gemv_kernel<FMT, NT>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(TK_LDS)) != hipSuccess)
            return PRIMA_E_DEVICE;
        attr_set = true;
    }
    hipLaunchKernelGGL((tok_gemv_kernel<FMT, NT>), dim3(grid_of(a)), dim3(TkFmt<FMT>::WAVES * 64), lds, st, a);
    return last_launch_status();
}

template <int FMT>
prima_status launch_fmt(const TokArgs &a, bool plan_only, hipStream_t st)
{
    if (a.T <= 2) return launch_nt<FMT, 2>(a, plan_only, st);
    if (a.T <= 4) return launch_nt<FMT, 4>(a, plan_only, st);
    if (a.T <= 8) return launch_nt<FMT, 8>(a, plan_only, st);
    return launch_nt<FMT, 16>(a, plan_only, st);
}

prima_status launch_any(int fmt, const TokArgs &a, bool plan_only, hipStream_t st)
{
    switch (fmt) {
    case PRIMA_FMT_Q4_K: return a.T > 8 ? launch_nt<PRIMA_FMT_Q4_K, 16>(a, plan_only, st) : PRIMA_E_SHAPE;
    case PRIMA_FMT_Q5_K: return launch_fmt<PRIMA_FMT_Q5_K>(a, plan_only, st);
    case PRIMA_FMT_Q6_K: return launch_fmt<PRIMA_FMT_Q6_K>(a, plan_only, st);
    case PRIMA_FMT_Q8_0: return launch_fmt<PRIMA_FMT_Q8_0>(a, plan_only, st);
    case PRIMA_FMT_F16: return launch_fmt<PRIMA_FMT_F16>(a, plan_only, st);
    default: return PRIMA_E_SHAPE;
    }
}

} // namespace

// Where the lines lie, us, this kernel / the fp32 mat-vec (replayed from a graph, weights cold; 256 shapes of 16 to 128256 rows and
// 512 to 28672 columns in each format):
//   7, 8 tokens     Q6_K 1024 x 8192   8 tokens  24 / 37   Q8_0 8192 x 4096  8: 19 / 20   FP16 8192 x 1024  7: 9.7 / 9.8, 4096 x 8192  8: 26 / 39
//                   one tile of rows: Q6_K 16 x 4096  7: 14 / 11 (every activation laid out for 16 rows), 16 x 14336  7: 33 / 45; 16 x 28672  8: FP16 69 / 91, Q8_0 103 / 84,
//                   12: Q5_K 127 / 146, Q6_K 138 / 143
//   9, 10 tokens    as 16 slots: Q6_K 1024 x 8192  9: 48 / 45, 16 x 8192  47 / 31; FP16 1024 x 8192  39 / 49
//   4 to 6 tokens   16384 rows fill a round of the mat-vec: Q8_0 16384 x 2048  5: 16.8 / 15.7, 6: 16.7 / 17.9, 16384 x 4096  5: 27.6 / 25.0,
//                   17408 x 4096  5: 27 / 33, 16384 x 12288  4: 47 / 57; FP16 16384 x 1024  5: 14.1 / 12.2, 17408 x 1024  5: 12.4 / 15.6
//   2 tokens        Q6_K 128256 x 8192  162 / 167, 100000 x 4096  80 / 80, 65536 x 4096  48 / 54; Q8_0 128256 x 8192  184 / 175, 65536 x 4096  56 / 50, 65536 x 512  15.9 / 17.9
// Below the lines several tokens stay with the mat-vec; 9 and 10 tokens of few rows go as 8 here and the rest there.
// Q4_K, against two passes of the integer mat-vec (q4k_gemv_mfma.hip), which has scratch to divide K among workgroups:
//   128256 x 8192        9 tokens 190 / 256, 16: 192 / 326    60000 x 2048   9: 32 / 46, 16: 33 / 59
//   28672 x 8192        11 tokens  66 / 77,  16: 66 / 86      8192 x 28672   9: 130 / 73, 16: 131 / 91
//   33000 x 8192        11 tokens  86 / 81 (a second round of tiles for 15 rows in a thousand), 33000 x 5120  11: 61 / 66
namespace {
// share of the waves' places in the rounds of a launch that have a tile (one round: the tiles are divided among the waves)
double places_filled(int64_t n_rows)
{
    const int64_t tiles = (n_rows + 15) / 16, per_round = static_cast<int64_t>(TK_CUS) * 8, rounds = (tiles + per_round - 1) / per_round;
    return rounds <= 1 ? 1. : static_cast<double>(tiles) / static_cast<double>(rounds * per_round);
}
bool in_limits(int64_t n_rows, int64_t n_cols) { return n_cols / QK < (1 << 18) && n_rows < (int64_t{1} << 34); } // (32-bit offsets in a tile's 16 rows, 32-bit tile numbers)
} // namespace

bool tok_gemv_takes(int fmt, int64_t n_rows, int64_t n_cols, int T)
{
    if (T > PRIMA_MAX_TOK || !in_limits(n_rows, n_cols)) return false;
    if (fmt == PRIMA_FMT_Q4_K) return (T >= 9 && n_rows >= 65536) || (T >= 11 && n_rows >= 28672 && (n_cols <= 6144 || places_filled(n_rows) >= 0.6));
    const bool q8 = fmt == PRIMA_FMT_Q8_0, k_quant = fmt == PRIMA_FMT_Q5_K || fmt == PRIMA_FMT_Q6_K;
    if (!q8 && !k_quant && fmt != PRIMA_FMT_F16) return false;
    if (n_rows <= 16) return T >= (n_cols > 16384 ? 12 : 13) || (T >= 9 && n_cols <= 1024) || ((T == 7 || T == 8) && n_cols >= 5120 && !(q8 && n_cols > 16384));
    if (T >= 7) return !(q8 && T == 7 && n_cols > 16384 && n_rows <= 8192);
    if (T >= 4) return n_rows > (T == 4 ? 16512 : 16384) || (n_rows == 16384 && T == 6) || (n_rows >= 16384 && (k_quant || n_cols <= 512 || n_cols >= (q8 ? 8192 : 2048)));
    return T >= 2 && n_rows >= 65536 && (T == 3 || !q8 || n_cols <= 512);
}

// tokens of T that go to launch_tok_gemv() in a call of few rows; the others after them to the fp32 mat-vec
int tok_gemv_first(int fmt, int64_t n_rows, int64_t n_cols, int T)
{
    const bool few = n_cols >= 4096 && n_rows <= (fmt == PRIMA_FMT_Q8_0 ? 2048 : 4096);
    return (T == 9 || T == 10) && few && fmt != PRIMA_FMT_Q4_K && fmt != PRIMA_FMT_F16 && tok_gemv_takes(fmt, n_rows, n_cols, 8) ? 8 : T;
}

prima_status launch_tok_gemv(int fmt, const uint8_t *W, int64_t n_rows, int64_t n_cols, const float *x, int64_t ldx, int T,
                             const float *gain, float eps, const float *resid, int64_t ldr, float *y, int64_t ldy, hipStream_t st)
{
    TokArgs a{};
    a.W = W; a.n_rows = n_rows; a.nb = static_cast<int>(n_cols / QK); a.x = x; a.ldx = ldx; a.gain = gain; a.eps = eps;
    a.resid = resid; a.ldr = ldr; a.y = y; a.ldy = ldy; a.T = T; a.n_tiles = static_cast<int>((n_rows + 15) / 16);
    return launch_any(fmt, a, false, st);
}

prima_status tok_gemv_plan_status(int fmt, int64_t n_rows, int64_t n_cols, int T)
{
    TokArgs a{};
    a.nb = static_cast<int>(n_cols / QK); a.T = T; a.n_tiles = static_cast<int>((n_rows + 15) / 16);
    return launch_any(fmt, a, true, nullptr);
}

} // namespace prima
