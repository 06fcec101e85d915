// Matrix product for many tokens with weights in the other formats (Q5_K, Q6_K, Q8_0, FP16): what q4k_gemm.hip is for Q4_K.
//
//     y[t][r] = sum_c W[r][c] * a[t][c],   a = x (or RMSNorm(x; gain)),   + resid[t][r] (optional)
//
// The activations are those of the Q4_K product (gemm_common.h: two binary16 parts, split once per activation tensor and
// shared with the group's Q4_K matrices).  The B operand is, per sub-block of 32 weights, as binary16 numbers:
//   Q5_K  sc_s (q - 16), exact.  The 16 sc_s come back, and the min term is formed, as one MFMA step each on the sub-block
//         sums of the activations (uncentred, the two sums that nearly cancel are twice as large: error 3.4e-7 against 1.9e-7);
//   Q6_K  sc_s (q - 32), up to 4096 in magnitude: 13 bits.  Rounded to 11 bits, and the remainder (-1, 0 or 1) as a second
//         operand that meets the hi parts of the activations alone (its product with the lo parts is 2^-23 of the largest
//         term and is left out): three MFMAs per step, d per super-block;
//   Q8_0  q: exact; the sum of a sub-block is multiplied by its d and added;
//   FP16  the weight itself.
// Roundings.  A sub-block's MFMAs start from zero, small terms first, and their sum is added to the super-block's: 8 roundings
// per super-block at its magnitude where one accumulator through all of them would have 16 or 24.  The matrix cores round
// their fp32 sums towards minus infinity, which over 28672 columns adds up to -2e-7 of the outputs' rms in every output: odd
// sub-blocks are multiplied as their negatives and subtracted, and it cancels.  The chain of super-blocks is compensated (Kahan;
// the compensation as bfloat16, two to a register) in all but Q6_K, whose registers are full.
// Error against 64 bits (2-norm, 256 to 28672 columns, 17 to 1024 tokens) beside that of the fp32 mat-vec: Q5_K 1.4-1.6e-7
// (2.1-2.3e-7), Q6_K 1.1-2.2e-7 (2.2-2.3e-7), Q8_0 1.0-1.3e-7 (1.1-1.4e-7), FP16 1.0-1.3e-7 (1.1-1.4e-7).
// What bounds it: at many tokens the matrix cores and the LDS reads that feed them, as in the Q4_K product; at few the weight
// stream and the length of the position chain.  Before, the prompt call streamed these matrices once per 8 tokens through the
// fp32 multiply-adds of the mat-vec.  us, this kernel / that: 4096 x 14336 at 17 tokens 52-56 / 148-182, at 64 60 / 570-650, at
// 333 220-250 / 2800-3250; 8192 x 28672 at 1024 tokens 1360-1570 (307-355 TFLOP/s) / 17700-20500.
//
// A workgroup of 4 waves owns 128 rows x 32 WT tokens, a wave 64 rows x 16 WT tokens.  Per position (sub-block) a thread
// decodes 16 weights of one row for the next position into LDS, where both row halves of the workgroup's waves read them
// as operands: a weight is decoded once per workgroup, not once per wave.  Activations come by 16-byte global->LDS loads.  Both
// are double-buffered with one barrier per position; 37 to 73 KiB of LDS by format and tokens, so that two workgroups share a compute unit and one's
// waits run under the other's matrix instructions.  At 64 tokens three share one in Q5_K, Q8_0 and FP16 (41 KiB and 168 registers at the most; Q5_K, 14B 700 tokens, every matrix,
// 178 registers 1638 us, 164 1527); Q6_K has 53 KiB.
#include <algorithm>
#include <atomic>

#include "gemm_common.h"

namespace prima {
namespace {

constexpr int FM_THREADS = 256;
constexpr int FM_ROWS = 128;
constexpr int FM_RT = 4; // 16-row tiles per wave

struct FmtGemmArgs {
    const uint8_t *W;
    int64_t n_rows, n_cols;
    const uint8_t *A;   // split activations
    GemmNorm norm;
    const float *resid;
    int64_t ldr;
    float *y;
    int64_t ldy;
    int T, n_tiles, n_rb, n_tb, band;
    int share_q, share_r, tile_q, tile_r; // as in q4k_gemm.hip
    int ksplit; // as in q4k_gemm.hip: shares of K, each share's sums in part[share][token][ldp]
    float *part;
    int64_t ldp;
};

// value of the neighbouring lane (lane ^ 1)
__device__ __forceinline__ unsigned swap1(unsigned v) { return __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0xB1, 0xf, 0xf, true); }

// bytes of the 4-byte words u (weights 0..3) and v (weights 4..7) -> four binary16 pairs (0,4) (1,5) (2,6) (3,7) of 1024 + byte
__device__ __forceinline__ void bytes_to_pairs(unsigned u, unsigned v, half2v *p)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned sel = 0x0c040c00u + 0x00010001u * i; // {0, byte i of v, 0, byte i of u}
        p[i] = __builtin_bit_cast(half2v, __builtin_amdgcn_perm(v, u, sel) | 0x64006400u);
    }
}

// what a thread holds of its row's weights: a pair of sub-blocks (2 i, 2 i + 1), of which thread h of the row's two
// threads loads sub-block 2 i + h (Q5_K, Q6_K: the neighbours exchange halves), or its 16 weights of one sub-block
template <int FMT> struct Quants;
template <> struct Quants<PRIMA_FMT_Q5_K> { uint4 lo; unsigned hi; };
template <> struct Quants<PRIMA_FMT_Q6_K> { uint4 lo; uint2 hi; };
template <> struct Quants<PRIMA_FMT_Q8_0> { uint4 q; };
template <> struct Quants<PRIMA_FMT_F16> { uint4 a, b; };
template <int FMT> constexpr bool fm_pairwise = FMT == PRIMA_FMT_Q5_K || FMT == PRIMA_FMT_Q6_K;

template <int FMT, int WT>
struct FmLds {
    static constexpr int A_SLOT = 2 * WT * 2048;            // 2 WT token tiles x (hi, lo) of a sub-block
    static constexpr int B_PARTS = FMT == PRIMA_FMT_Q6_K ? 2 : 1;
    static constexpr int B_SLOT = B_PARTS * FM_ROWS * 64;   // [part][16-row tile][lane][16 bytes]
    static constexpr int B0 = 2 * A_SLOT;
    static constexpr int D0 = B0 + 2 * B_SLOT;              // d: [2][128] floats (Q8_0: per position; Q5_K: d, dmin)
    static constexpr int M0 = D0 + 2 * FM_ROWS * 4;         // sums slabs of the tokens; Q5_K: then the m_s and the 16 sc_s of every row
    static constexpr int TOTAL = M0 + 2 * WT * 1024 + (FMT == PRIMA_FMT_Q5_K ? 2 * FM_ROWS * 16 : 0);
    static_assert(TOTAL <= 81920, "two workgroups per compute unit");
};

// FULL: every workgroup does 2 WT token tiles (past the last: the last again, not stored); else the tiles are shared out evenly over the
// workgroups, which skip those they do not have.  (The branches, and the unpacking in front of the products, cost 3 to 7 %; both in one kernel spill.)
template <int FMT, int WT, bool FULL>
__global__ void __launch_bounds__(FM_THREADS, 2) fmt_gemm_kernel(FmtGemmArgs a)
{
    request_args<sizeof(a)>();
    extern __shared__ __align__(16) uint8_t smem[];
    typedef FmLds<FMT, WT> L;
    // Q5_K has no registers left for its unpacking between the products (all seven matrices, 8B 1024 tokens: 1739 us in front, 1785 woven; Q8_0 1697 / 1648, Q6_K
    // 1867 / 1783), and workgroups that lack tiles have branches there.
    constexpr bool WOVEN = FULL && FMT != PRIMA_FMT_Q5_K;
    constexpr bool Q5 = FMT == PRIMA_FMT_Q5_K, Q6 = FMT == PRIMA_FMT_Q6_K, Q8 = FMT == PRIMA_FMT_Q8_0, H = FMT == PRIMA_FMT_F16;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    int rb, tb, share;
    if (!gemm_unit(blockIdx.x, a.n_rb, a.n_tb, a.ksplit, a.band, rb, tb, share)) return; // the whole workgroup, before any barrier
    const int tile0 = FULL ? tb * 2 * WT : tb * a.tile_q + min(tb, a.tile_r);
    const int tiles = FULL ? 2 * WT : a.tile_q + (tb < a.tile_r ? 1 : 0);
    const int nb = static_cast<int>(a.n_cols >> 8);
    const int b_lo = share * a.share_q + min(share, a.share_r), b_hi = b_lo + a.share_q + (share < a.share_r ? 1 : 0); // (not empty: the host keeps ksplit <= nb)
    // this wave's half of the rows and of the tiles (every other one)
    const int wr = wave & 1, wt = wave >> 1, my_tiles = FULL ? WT : (tiles - wt + 1) / 2;

    // ---- this thread's row of the workgroup's weights and its half h (16 weights) of every sub-block ----
    const int drow = threadIdx.x >> 1, h = threadIdx.x & 1;
    const int64_t grow = min<int64_t>(static_cast<int64_t>(rb) * FM_ROWS + drow, a.n_rows - 1); // past the end: a valid row, not stored
    const int64_t blk0 = grow * nb, nblk = a.n_rows * nb;
    // where its decoded weights go: operand lane (row % 16, g = 2 h and 2 h + 1) of the row's tile
    uint8_t *const bdst = smem + L::B0 + (drow >> 4) * 1024 + (2 * h * 16 + (drow & 15)) * 16;
    float *const l_d = reinterpret_cast<float *>(smem + L::D0);
    uint8_t *const l_xs = smem + L::M0, *const l_m = l_xs + 2 * WT * 1024;

    auto load_quants = [&](Quants<FMT> &q, int b, int s) __attribute__((always_inline)) { // s even where a pair is loaded
        const int64_t blk = blk0 + b;
        if constexpr (Q6) {
            q.lo = *reinterpret_cast<const uint4 *>(a.W + blk * 128 + (s + h) * 16);
            q.hi = *reinterpret_cast<const uint2 *>(a.W + nblk * 128 + blk * 64 + (s + h) * 8);
        } else if constexpr (Q5) {
            q.lo = *reinterpret_cast<const uint4 *>(a.W + nblk * 16 + blk * 128 + (s + h) * 16);
            q.hi = *reinterpret_cast<const unsigned *>(a.W + nblk * 144 + blk * 32 + (s + h) * 4);
        } else if constexpr (Q8) {
            q.q = *reinterpret_cast<const uint4 *>(a.W + blk * 256 + s * 32 + h * 16);
        } else {
            q.a = *reinterpret_cast<const uint4 *>(a.W + blk * 512 + s * 64 + h * 32);
            q.b = *reinterpret_cast<const uint4 *>(a.W + blk * 512 + s * 64 + h * 32 + 16);
        }
    };
    // scales of a super-block: Q5_K its header, Q6_K sixteen sub-scales (and d beside them), Q8_0 eight d
    auto load_header = [&](uint4 &hd, unsigned &hx, int b) __attribute__((always_inline)) {
        const int64_t blk = blk0 + b;
        if constexpr (Q5) hd = *reinterpret_cast<const uint4 *>(a.W + blk * 16);
        if constexpr (Q6) {
            hd = *reinterpret_cast<const uint4 *>(a.W + nblk * 192 + blk * 16);
            hx = *reinterpret_cast<const unsigned short *>(a.W + nblk * 208 + blk * 2);
        }
        if constexpr (Q8) hd = *reinterpret_cast<const uint4 *>(a.W + nblk * 256 + blk * 16);
    };
    auto h2f = [](unsigned v) { return __half2float(__ushort_as_half(static_cast<unsigned short>(v & 0xffffu))); };
    auto word = [](const uint4 &v, int i) __attribute__((always_inline)) { return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w)); };

    // Half c (8) of this thread's 16 weights of sub-block s as operand bytes in buffer `buf`; of an odd sub-block their negatives, whose sums
    // are subtracted (see the top of the file)
    auto decode = [&](const Quants<FMT> &q, const uint4 &hd, unsigned hx, int s, int buf, int c) __attribute__((always_inline)) {
        half2v hi[4], lo[4];
        if constexpr (Q5 || Q6) {
            // thread s & 1 of the row holds the sub-block; its neighbour takes its own half from there
            const bool own = (s & 1) == h;
            unsigned w;
            if ((s & 1) == 0) {
                const unsigned t = swap1(c ? q.lo.w : q.lo.z);
                w = own ? (c ? q.lo.y : q.lo.x) : t;
            } else {
                const unsigned t = swap1(c ? q.lo.y : q.lo.x);
                w = own ? (c ? q.lo.w : q.lo.z) : t;
            }
            unsigned u, v;
            if constexpr (Q6) {
                unsigned hb;
                if ((s & 1) == 0) { const unsigned t = swap1(q.hi.y); hb = own ? q.hi.x : t; }
                else { const unsigned t = swap1(q.hi.x); hb = own ? q.hi.y : t; }
                u = (w & 0x0F0F0F0Fu) | ((c ? hb : hb << 4) & 0x30303030u);
                v = ((w >> 4) & 0x0F0F0F0Fu) | ((c ? hb >> 2 : hb << 2) & 0x30303030u);
            } else {
                const unsigned t = swap1(q.hi);
                const unsigned hb = (own ? q.hi : t) >> (4 * h); // bits 4 h .. 4 h + 3 of every byte: this half's groups of four
                u = (w & 0x0F0F0F0Fu) | ((c ? hb << 2 : hb << 4) & 0x10101010u);
                v = ((w >> 4) & 0x0F0F0F0Fu) | ((c ? hb << 1 : hb << 3) & 0x10101010u);
            }
            bytes_to_pairs(u, v, hi);
            if constexpr (Q6) {
                const unsigned sw = word(hd, s >> 1);
                const int sc = static_cast<int>(sw << (24 - 16 * (s & 1) - 8 * h)) >> 24; // byte 2 s + h, signed
                const _Float16 f = static_cast<_Float16>(static_cast<float>(s & 1 ? -sc : sc));
                const half2v sc2 = {f, f}, off = {static_cast<_Float16>(-1056.f), static_cast<_Float16>(-1056.f)};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const half2v x = hi[i] + off; // q - 32, exact
                    hi[i] = x * sc2;              // rounded to 11 bits
                    lo[i] = __builtin_elementwise_fma(x, sc2, -hi[i]); // the remainder, exact
                }
            } else {
                const float fs = static_cast<float>(hdr_field(hd, s));
                const _Float16 f = static_cast<_Float16>(s & 1 ? -fs : fs);
                const half2v sc2 = {f, f}, off = {static_cast<_Float16>(-1040.f), static_cast<_Float16>(-1040.f)};
#pragma unroll
                for (int i = 0; i < 4; ++i) hi[i] = (hi[i] + off) * sc2; // (q - 16) sc: both steps exact
            }
        } else if constexpr (Q8) {
            bytes_to_pairs((c ? q.q.z : q.q.x) ^ 0x80808080u, (c ? q.q.w : q.q.y) ^ 0x80808080u, hi);
            const half2v off = {static_cast<_Float16>(-1152.f), static_cast<_Float16>(-1152.f)};
#pragma unroll
            for (int i = 0; i < 4; ++i) hi[i] = s & 1 ? -off - hi[i] : hi[i] + off;
        } else {
            // numbers 0..7 as pairs (0,4) (1,5) (2,6) (3,7)
            const unsigned neg = s & 1 ? 0x80008000u : 0u;
            const uint4 &x = c ? q.b : q.a;
            const unsigned v[4] = {x.x ^ neg, x.y ^ neg, x.z ^ neg, x.w ^ neg};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                hi[i] = __builtin_bit_cast(half2v, __builtin_amdgcn_perm(v[2 + (i >> 1)], v[i >> 1], (i & 1) ? 0x07060302u : 0x05040100u));
        }
        uint8_t *dst = bdst + buf * L::B_SLOT + c * 256;
        auto store = [&](uint8_t *to, const half2v *p) __attribute__((always_inline)) {
            *reinterpret_cast<uint4 *>(to) = make_uint4(__builtin_bit_cast(unsigned, p[0]), __builtin_bit_cast(unsigned, p[1]),
                                                        __builtin_bit_cast(unsigned, p[2]), __builtin_bit_cast(unsigned, p[3]));
        };
        store(dst, hi);
        if constexpr (Q6) store(dst + FM_ROWS * 64, lo);
        if constexpr (Q8) {
            const unsigned w = word(hd, s >> 1);
            if (c == 0 && h == 0) l_d[buf * FM_ROWS + drow] = h2f(s & 1 ? w >> 16 : w);
        }
    };
    // what the fold of a super-block needs of its rows: d (Q6_K), d, dmin and the m_s (Q5_K)
    auto put_scales = [&](const uint4 &hd, unsigned hx) __attribute__((always_inline)) {
        if constexpr (Q6) {
            if (h == 0) l_d[drow] = h2f(hx);
        }
        if constexpr (Q5) {
            if (h == 0) {
                l_d[drow] = hdr_d(hd);
                l_d[FM_ROWS + drow] = hdr_dmin(hd);
                half8 m, c;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    m[i] = static_cast<_Float16>(static_cast<float>(hdr_field(hd, 8 + i)));
                    c[i] = static_cast<_Float16>(static_cast<float>(16 * hdr_field(hd, i)));
                }
                *reinterpret_cast<half8 *>(l_m + drow * 16) = m;
                *reinterpret_cast<half8 *>(l_m + (FM_ROWS + drow) * 16) = c;
            }
        }
    };

    // ---- activation requests: 4 WT slabs of 1 KiB per position, WT per wave; a sums slab per token tile and super-block ----
    const uint32_t lds0 = lds_address(smem), lane16 = lane * 16;
    // A base per tile, not per slab: scalar registers short of the 128-token kernels were kept in lanes of vector registers.  (One layer,
    // every matrix in Q5_K, 70B 1024 tokens 5559 -> 5395 us, 8B 1685 -> 1650, Q6_K 14B 700 1777 -> 1750; FP16, which has them free: 8B 128 tokens a base per tile 327, per slab 320, before 325.)
    constexpr int PER_BASE = H ? 1 : 2;
    const uint8_t *abase[WT / PER_BASE];
#pragma unroll
    for (int j = 0; j < WT / PER_BASE; ++j) {
        const int slab = wave * WT + j * PER_BASE;
        abase[j] = a.A + (static_cast<int64_t>(min(tile0 + (slab >> 1), a.n_tiles - 1)) * nb * GM_SLABS + (slab & 1)) * 1024;
    }
    auto issue = [&](int b, int s, int buf) __attribute__((always_inline)) {
        const int64_t off = (static_cast<int64_t>(b) * GM_SLABS + 2 * s) * 1024;
#pragma unroll
        for (int j = 0; j < WT; ++j)
            if (FULL || wave * WT + j < 2 * tiles) dma16_base(abase[j / PER_BASE] + off + j % PER_BASE * 1024, lane16, lds0 + buf * L::A_SLOT + (wave * WT + j) * 1024);
    };
    auto issue_sums = [&](int b) __attribute__((always_inline)) {
        {
#pragma unroll
            for (int j = wave; j < 2 * WT; j += 4)
                if (FULL || j < tiles) dma16_base(a.A + ((static_cast<int64_t>(min(tile0 + j, a.n_tiles - 1)) * nb + b) * GM_SLABS + 16) * 1024, lane16, lds0 + L::M0 + j * 1024);
        }
    };

    gm_v4f acc[WT][FM_RT], ysum[WT][FM_RT];
    const gm_v4f zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tt = 0; tt < WT; ++tt)
#pragma unroll
        for (int rt = 0; rt < FM_RT; ++rt) acc[tt][rt] = ysum[tt][rt] = zero;
    unsigned comp[Q6 ? 1 : WT][FM_RT][2] = {}; // Kahan's compensation of ysum, bfloat16 pairs

    // prologue: position 0's activations and decoded weights, the quants after it, the header
    uint4 hd, hd_next;
    unsigned hx = 0, hx_next = 0;
    Quants<FMT> qc, qn;
    issue(b_lo, 0, 0);
    load_header(hd, hx, b_lo);
    load_quants(qc, b_lo, 0);
    if constexpr (fm_pairwise<FMT>) load_quants(qn, b_lo, 2);
    else load_quants(qn, b_lo, 1);
    decode(qc, hd, hx, 0, 0, 0);
    decode(qc, hd, hx, 0, 0, 1);
    hd_next = hd; hx_next = hx;

    for (int b = b_lo; b < b_hi; ++b) {
        const bool more = b + 1 < b_hi;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int buf = s & 1;
            // everything requested at the position before has landed; everyone has written its operands of this position
            // and is done with the buffers of the one before
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            gm_barrier();
            if (s < 7 || more) issue(s < 7 ? b : b + 1, (s + 1) & 7, buf ^ 1);
            if (s == 6) issue_sums(b);
            if (s == 0) put_scales(hd, hx);
            // quants of the next position (requested a pair, or a position, ahead), and the request after them
            if constexpr (fm_pairwise<FMT>) {
                if (s & 1) {
                    qc = qn;
                    const int s2 = (s + 3) & 7; // the pair behind the one that is decoded next
                    if (s + 3 < 8 || more) load_quants(qn, s + 3 < 8 ? b : b + 1, s2);
                }
            } else {
                qc = qn;
                if (s + 2 < 8 || more) load_quants(qn, s + 2 < 8 ? b : b + 1, (s + 2) & 7);
            }
            if (s == 5 && more) load_header(hd_next, hx_next, b + 1);
            // The operands of the next position.  WOVEN: unpacked between the matrix instructions of the first two tiles, a half each; else in
            // front.  (Past the last position those of the last super-block again, unused.)
            auto decode_next = [&](int c) __attribute__((always_inline)) {
                if constexpr (Q8) { // (chosen by reference they are an array in scratch memory: 128 tokens a workgroup, 70B 1024 tokens 5667 -> 4882 us; the others 1 to 3 % slower like this)
                    if (s < 7) decode(qc, hd, hx, s + 1, buf ^ 1, c);
                    else decode(qc, hd_next, hx_next, 0, buf ^ 1, c);
                } else {
                    decode(qc, s < 7 ? hd : hd_next, s < 7 ? hx : hx_next, (s + 1) & 7, buf ^ 1, c);
                }
            };
            if constexpr (!WOVEN) {
                decode_next(0);
                decode_next(1);
            }

            const uint8_t *ab = smem + buf * L::A_SLOT + wt * 2048 + lane * 16;
            const uint8_t *bb = smem + L::B0 + buf * L::B_SLOT + wr * 4096 + lane * 16;
            half8 B[FM_RT], Bl[FM_RT];
#pragma unroll
            for (int rt = 0; rt < FM_RT; ++rt) {
                B[rt] = *reinterpret_cast<const half8 *>(bb + rt * 1024);
                if constexpr (Q6) Bl[rt] = *reinterpret_cast<const half8 *>(bb + FM_ROWS * 64 + rt * 1024);
            }
            float ds[FM_RT];
            if constexpr (Q8) {
#pragma unroll
                for (int rt = 0; rt < FM_RT; ++rt) ds[rt] = l_d[buf * FM_ROWS + wr * 64 + rt * 16 + n];
            }
#pragma unroll
            for (int tt = 0; tt < WT; ++tt) {
                if (!FULL && tt >= my_tiles) break;
                const half8 ah = *reinterpret_cast<const half8 *>(ab + tt * 4096);
                const half8 al = *reinterpret_cast<const half8 *>(ab + tt * 4096 + 1024);
#pragma unroll
                for (int rt = 0; rt < FM_RT; ++rt) {
                    gm_v4f c = zero;
                    if constexpr (Q6) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, Bl[rt], c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, B[rt], c, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, B[rt], c, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float ci = s & 1 ? -c[i] : c[i];
                        if constexpr (Q8) acc[tt][rt][i] = s == 0 ? ds[rt] * ci : fmaf(ds[rt], ci, acc[tt][rt][i]);
                        else acc[tt][rt][i] = s == 0 ? ci : acc[tt][rt][i] + ci;
                    }
                }
                if constexpr (WOVEN) {
                    if (tt == 0) decode_next(0);
                    if (tt == (WT > 1 ? 1 : 0)) decode_next(1);
                    __builtin_amdgcn_sched_group_barrier(0x100, 12, 0);
#pragma unroll
                    for (int k = 0; k < (Q6 ? 3 : 2) * FM_RT; ++k) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                    }
                }
                // the sums are made here (the compiler would move products and additions into the next position's block, where
                // they are used, and spill their operands), tile by tile
#pragma unroll
                for (int rt = 0; rt < FM_RT; ++rt) asm volatile("" : "+v"(acc[tt][rt]));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (s == 7) { // the super-block's term is formed at its own magnitude and added in one step
                // The sums slabs were requested a position ago by all waves and have landed before this position's barrier.  What the fold needs of them is
                // read in front of it where the registers hold it (read where it is used, each read waited for: Q6_K, 64 tokens a workgroup, 4 % slower).
                constexpr bool FRONT = !Q5 || WT == 2;
                gm_v4f scale[FRONT ? WT : 1]; // of this lane's tokens: powers of two
                half8 ax[Q5 && FRONT ? WT : 1];
                auto read_sums = [&](int tt, int to) __attribute__((always_inline)) {
                    const uint8_t *const sums = l_xs + (2 * tt + wt) * 1024;
                    const int l = lane_anew(); // (kept, it spills)
                    scale[to] = *reinterpret_cast<const gm_v4f *>(sums + GM_SCALES + (l >> 4) * 16);
                    if constexpr (Q5) ax[to] = gemm_sums_operand(*reinterpret_cast<const half8 *>(sums + l * 16), g);
                };
                if constexpr (FRONT) {
#pragma unroll
                    for (int tt = 0; tt < WT; ++tt) read_sums(tt, tt);
                }
#pragma unroll
                for (int rt = 0; rt < FM_RT; ++rt) {
                    const int r = wr * 64 + rt * 16 + (Q5 ? lane_anew() & 15 : n); // (Q5_K: kept, the addresses spill eight registers; 64 tokens: 178 registers, now 164, three workgroups a compute unit)
                    float d = 1.f, dm = 0.f;
                    half8 m = {}, sc16 = {};
                    if constexpr (Q5 || Q6) d = l_d[r];
                    if constexpr (Q5) {
                        dm = l_d[FM_ROWS + r];
                        m = *reinterpret_cast<const half8 *>(l_m + r * 16);
                        sc16 = *reinterpret_cast<const half8 *>(l_m + (FM_ROWS + r) * 16);
                    }
#pragma unroll
                    for (int tt = 0; tt < WT; ++tt) {
                        if constexpr (!FRONT) read_sums(tt, 0);
                        const int at = FRONT ? tt : 0;
                        gm_v4f am = zero, t = acc[tt][rt];
                        if constexpr (Q5) {
                            am = __builtin_amdgcn_mfma_f32_16x16x32_f16(ax[at], m, zero, 0, 0, 0);
                            t = __builtin_amdgcn_mfma_f32_16x16x32_f16(ax[at], sc16, t, 0, 0, 0);
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if constexpr (Q6) {
                                ysum[tt][rt][i] = fmaf(d * scale[at][i], t[i], ysum[tt][rt][i]);
                            } else {
                                const float term = (Q5 ? fmaf(d, t[i], -(dm * am[i])) : t[i]) * scale[at][i];
                                unsigned &cw = comp[tt][rt][i >> 1];
                                const float c0 = __builtin_bit_cast(float, i & 1 ? cw & 0xffff0000u : cw << 16);
                                const float v = term - c0, yn = ysum[tt][rt][i] + v;
                                const unsigned cn = __builtin_bit_cast(unsigned, (yn - ysum[tt][rt][i]) - v); // (cut off: its error is 2^-8 of it)
                                cw = i & 1 ? (cw & 0xffffu) | (cn & 0xffff0000u) : (cw & 0xffff0000u) | cn >> 16;
                                ysum[tt][rt][i] = yn;
                            }
                        }
                    }
                }
            }
        }
        hd = hd_next;
        hx = hx_next;
    }

    const float *inv = nullptr; // 1/rms of the workgroup's tokens
    if (a.norm.ss && a.ksplit == 1) {
        float *const red = reinterpret_cast<float *>(smem);
        gm_barrier(); // (the last operands have been read)
        gemm_inv_rms_tokens<32 * WT>(a.norm, tile0 * 16, red, red + 256);
        inv = red + 256;
    }
#pragma unroll
    for (int rt = 0; rt < FM_RT; ++rt) {
        const int64_t row = static_cast<int64_t>(rb) * FM_ROWS + wr * 64 + rt * 16 + n;
        if (row >= a.n_rows) continue;
        float add[WT][4] = {}; // the residual, requested at once (as in q4k_gemm.hip)
        if (a.resid && a.ksplit == 1) {
#pragma unroll
            for (int tt = 0; tt < WT; ++tt)
#pragma unroll
                for (int i = 0; i < 4; ++i) add[tt][i] = a.resid[min((tile0 + 2 * tt + wt) * 16 + 4 * g + i, a.T - 1) * a.ldr + row];
        }
#pragma unroll
        for (int tt = 0; tt < WT; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = (tile0 + 2 * tt + wt) * 16 + 4 * g + i;
                if ((FULL || tt < my_tiles) && t < a.T) {
                    const float v = ysum[tt][rt][i];
                    if (a.ksplit > 1) a.part[(static_cast<int64_t>(share) * a.T + t) * a.ldp + row] = v;
                    else a.y[t * a.ldy + row] = v * (inv ? inv[16 * (2 * tt + wt) + 4 * g + i] : 1.f) + add[tt][i];
                }
            }
    }
}

template <int FMT, int WT, bool FULL>
prima_status launch_wt(const FmtGemmArgs &a, unsigned grid, hipStream_t st)
{
    static std::atomic<bool> attr_set{false}; // set twice by two threads at worst: the attribute call is idempotent
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(fmt_gemm_kernel<FMT, WT, FULL>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                FmLds<FMT, WT>::TOTAL) != hipSuccess)
            return PRIMA_E_DEVICE;
        attr_set = true;
    }
    hipLaunchKernelGGL((fmt_gemm_kernel<FMT, WT, FULL>), dim3(grid), dim3(FM_THREADS), (FmLds<FMT, WT>::TOTAL), st, a);
    return last_launch_status();
}

// Token blocks and shares of K
struct FmPlan {
    bool narrow, full;
    int n_tb, ksplit;
};
// own_sum: a launch of their own adds the shares (else the caller's next one, which there is anyway)
FmPlan plan_fm(int T, int64_t n_rows, int64_t n_cols, int64_t part_bytes, bool own_sum)
{
    const int64_t n_rb = (n_rows + FM_ROWS - 1) / FM_ROWS, nb = n_cols / QK;
    const int n_tiles = (T + 15) / 16;
    FmPlan p{};
    // 128 tokens per workgroup, 64 where that leaves fewer tokens of padding or twice the workgroups on an idle device
    p.narrow = (n_tiles + 3) / 4 * 4 < (n_tiles + 7) / 8 * 8 || n_rb * ((n_tiles + 7) / 8) * 2 <= 2 * GM_CUS;
    p.n_tb = p.narrow ? (n_tiles + 3) / 4 : (n_tiles + 7) / 8;
    // Full workgroups where that leaves less than a seventh of padding.  (A twentieth before: one layer, every matrix in one format, us, before / now: 70B 450 tokens (29
    // tiles) Q5_K 3117 / 2983, Q6_K 3152 / 3089, Q8_0 2862 / 2651, FP16 2861 / 2683, 14B 720 (45) Q6_K 1772 / 1736, Q8_0 1606 / 1524, 8B 900 (57) Q5_K 1646 / 1574; 96 of 8B to
    // 70B and 200 to 1170 tokens 0.926 to 1.005 of before.  At a seventh, 21 tiles, 70B 333 in Q8_0 full 2101, not full 2018.)
    p.full = (p.n_tb * (p.narrow ? 4 : 8) - n_tiles) * 7 < n_tiles;
    const int64_t wgs = n_rb * p.n_tb, slots = 2 * GM_CUS;
    // Shares of K (as far as the scratch holds them; with four super-blocks of each at the least, two 8B layers with V and down in Q6_K took 293 us at 17 tokens, 248 without): rounds of workgroups times a share's super-blocks, about
    // 7 us each at 64 tokens and 14 at 128, against the shares' way to memory and back (4 TB/s).  (As many as fit the device at once
    // left a quarter of it idle where they do not come out even: 4096 x 14336 in Q6_K, 333 tokens, two shares 227 us and 6 for their sum, five 200 and 7.)
    // The two figures serve every format: one layer of 8B, 14B and 70B shapes, 40 to 900 tokens, us, that rule / this one where they differ: down in Q5_K 8B 333
    // tokens (two shares / five) 576 / 553, Q8_0 576 / 561, FP16 604 / 587; 14B 400 (one / three) Q5_K 934 / 837, Q6_K 958 / 855, Q8_0 920 / 834, FP16 949 / 848; 70B
    // 180 (two / five) Q5_K 1034 / 971, FP16 1057 / 1018; every matrix, 14B, 180 tokens Q5_K 623 / 581, Q8_0 652 / 602, 512 tokens 1364 / 1197, 1357 / 1202.
    p.ksplit = 1;
    if (part_bytes > 0 && T <= 65535) {
        const int64_t share_bytes = static_cast<int64_t>(T) * n_rows * static_cast<int64_t>(sizeof(float));
        const int64_t most = std::min<int64_t>({nb, 16, part_bytes / share_bytes});
        // Where a launch of its own adds them (a gate and an up matrix one by one), a last round that leaves half of the slots empty counts four fifths (a
        // workgroup alone on its compute unit is faster), and more shares have to save 2 %.  One layer, every matrix in one format, us, without these two / with: 14B 700 tokens
        // (two shares / one) Q8_0 1497 / 1433, FP16 1523 / 1448, 70B 450 FP16 2922 / 2861, Q8_0 2968 / 2911.  Over 28 shapes of 8B to 70B widths and 100 to
        // 1400 tokens 0.8 % above the best of one to six shares on average.
        const double alone = own_sum ? 0.8 : 1., least_gain = own_sum ? 0.98 : 1.;
        double best = 0.;
        for (int64_t ks = 1; ks <= std::max<int64_t>(1, most); ++ks) {
            const int64_t full = wgs * ks / slots, rest = wgs * ks % slots;
            const double rounds = static_cast<double>(full) + (rest == 0 ? 0. : (rest <= GM_CUS ? alone : 1.));
            const double us = rounds * static_cast<double>((nb + ks - 1) / ks) * (p.narrow ? 7. : 14.) +
                              (ks > 1 ? 4. + static_cast<double>(ks * share_bytes) * 2. / 4e6 : 0.);
            if (ks == 1 || us < best * least_gain) {
                best = us;
                p.ksplit = static_cast<int>(ks);
            }
        }
    }
    return p;
}

template <int FMT>
prima_status launch_fm(FmtGemmArgs a, const FmPlan &p, hipStream_t st)
{
    const int64_t wgs = static_cast<int64_t>(a.n_rb) * p.n_tb, nb = a.n_cols / QK;
    if (wgs * p.ksplit >= (int64_t{1} << 31) - GM_XCDS) return PRIMA_E_SHAPE;
    a.n_tb = p.n_tb;
    a.ksplit = p.ksplit;
    a.band = gemm_band(a.n_tb);
    a.share_q = static_cast<int>(nb / a.ksplit); a.share_r = static_cast<int>(nb % a.ksplit);
    a.tile_q = a.n_tiles / a.n_tb; a.tile_r = a.n_tiles % a.n_tb;
    const unsigned grid = gemm_grid(wgs * a.ksplit);
    if (p.narrow) return p.full ? launch_wt<FMT, 2, true>(a, grid, st) : launch_wt<FMT, 2, false>(a, grid, st);
    return p.full ? launch_wt<FMT, 4, true>(a, grid, st) : launch_wt<FMT, 4, false>(a, grid, st);
}

} // namespace

bool fmt_gemm_takes(int fmt) { return fmt == PRIMA_FMT_Q5_K || fmt == PRIMA_FMT_Q6_K || fmt == PRIMA_FMT_Q8_0 || fmt == PRIMA_FMT_F16; }

FmtGemmBlocks fmt_gemm_blocks(int T, int64_t n_rows, int64_t n_cols)
{
    const FmPlan p = plan_fm(T, n_rows, n_cols, 0, false);
    return FmtGemmBlocks{p.narrow ? 64 : 128, p.n_tb, p.full};
}

int64_t fmt_gemm_most_shares(int64_t n_rows, int64_t n_cols)
{
    const int64_t n_rb = (n_rows + FM_ROWS - 1) / FM_ROWS;
    return std::max<int64_t>(1, std::min<int64_t>({16, n_cols / QK, 2 * GM_CUS / n_rb})) * n_rows;
}

prima_status launch_fmt_gemm(int fmt, const GemmMat &m, int64_t n_cols, const GemmActs &x, int T, const float *resid, int64_t ldr, void *part,
                             size_t part_bytes, GemmShares *later, hipStream_t st)
{
    if (later) *later = GemmShares{};
    if (T == 0 || m.n_rows == 0) return PRIMA_OK;
    const int64_t n_rb = (m.n_rows + FM_ROWS - 1) / FM_ROWS;
    const int n_tiles = (T + 15) / 16;
    if (n_rb >= (int64_t{1} << 30) || n_tiles > 65535 || n_cols / QK >= (int64_t{1} << 31)) return PRIMA_E_SHAPE;
    const FmPlan p = plan_fm(T, m.n_rows, n_cols, part ? static_cast<int64_t>(part_bytes) : 0, !later);
    FmtGemmArgs a{};
    a.W = m.W; a.n_rows = m.n_rows; a.n_cols = n_cols; a.A = x.A; a.norm = x.norm;
    a.resid = resid; a.ldr = ldr; a.y = m.y; a.ldy = m.ldy; a.T = T; a.n_tiles = n_tiles; a.n_rb = static_cast<int>(n_rb);
    a.part = static_cast<float *>(part);
    a.ldp = m.n_rows;
    prima_status s;
    switch (fmt) {
    case PRIMA_FMT_Q5_K: s = launch_fm<PRIMA_FMT_Q5_K>(a, p, st); break;
    case PRIMA_FMT_Q6_K: s = launch_fm<PRIMA_FMT_Q6_K>(a, p, st); break;
    case PRIMA_FMT_Q8_0: s = launch_fm<PRIMA_FMT_Q8_0>(a, p, st); break;
    case PRIMA_FMT_F16: s = launch_fm<PRIMA_FMT_F16>(a, p, st); break;
    default: return PRIMA_E_SHAPE;
    }
    if (s != PRIMA_OK || p.ksplit == 1) return s;
    const GemmShares sh{a.part, p.ksplit, static_cast<int64_t>(T) * a.ldp, a.ldp, {0, 0, 0}};
    if (!later) return launch_gemm_sum(sh, x.norm, resid, ldr, m.y, m.ldy, m.n_rows, T, st);
    *later = sh;
    return PRIMA_OK;
}

} // namespace prima
