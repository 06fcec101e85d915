// Mat-vecs of 2 to 16 tokens on the matrix cores: what their kernels share (tok_gemv.hip, tok_stream.hip).  The activations as binary16
// operands in LDS, the weight stream of a wave, and the products of one super-block of 16 rows with all tokens.
//
// Arithmetic.  A weight becomes a binary16 number in a register (sub-scale times quant, exact; Q6_K, 13 bits: two numbers, the
// sub-scale's high and low bits times the quant) and is the B operand of v_mfma_f32_16x16x32_f16 for all tokens at once; d (and dmin) scale the sums of a
// super-block.  The activations are the A operand: per token and super-block a power of two brings them below 2^10, and each
// is the sum of two binary16 numbers hi + lo (22 bits, relative to the activation, down to 2^-11 of the super-block's largest; every
// smaller one to 2^-35 of that).  The integer mat-vec holds Q4_K's activations to 2^-30 of the slab's largest and adds exactly, the fp32
// mat-vec the other formats' as they are; the sums here have fewer roundings.  2-norm error of a product against 64 bits, N(0, 1)
// activations and weights of mean zero, 2048 to 13824 columns, at 16 tokens / of those mat-vecs: Q4_K 1.30 to 1.42e-7 / 1.86 to 2.14e-7,
// Q5_K 1.35 to 1.45 / 2.10 to 2.20, Q6_K 1.01 to 1.22 / 2.15 to 2.21, Q8_0 0.92 to 1.15 / 1.04 to 1.15, FP16 0.93 to 1.12 / 1.03 to 1.15.  Q4_K
// whose minima do not balance its quants (a mean of half the largest weight): 0.96 to 1.16e-7 / 0.73 to 1.01e-7.  Magnitudes over six
// decades within a row: Q4_K 1.37 to 1.52 / 1.80 to 2.05, Q8_0 1.00 to 1.21 / 1.04 to 1.15, FP16 1.02 to 1.18 / 1.02 to 1.15.  Up to 8 tokens: the 16 rows of the A
// operand are (token, part) pairs, so that one instruction does both parts; up to 16 tokens: rows are tokens, hi and lo are
// instructions of their own.  Fewer than 8 tokens: the operand is stored for 2 or 4 tokens and the other rows repeat them
// (LDS bytes and bandwidth fall with the tokens; the instructions do not).
// Which 8 weights a lane contributes to an instruction is free as long as both operands agree, so lane (row n, g) takes
// whole sub-blocks: step (h, j) contracts the 8-weight slice j of sub-blocks 4h .. 4h+3, lane group g holding sub-block
// 4h+g.  A lane needs two sub-scales per super-block then instead of eight, and one 16-byte read brings the quants of four
// steps.  (Q8_0, whose scales multiply finished sums: step s contracts sub-block s, lane group g its slice g.)
// Quants are centred before the product (q - 8, 16, 32), the sub-block sums of the activations bring the centre back in one
// more step together with the minima: uncentred, two sums of twice the result's size would cancel.
// The matrix cores round their sums towards minus infinity; every other super-block (Q8_0: sub-block, FP16: step) is multiplied as
// its negative and subtracted, so that this cancels.
// An FP16 weight's 11 bits fill the products: a chain of four steps inside the matrix cores rounded them more than the fp32 mat-vec
// does (20000 x 4096, 4 to 16 tokens, 2-norm against 64 bits 1.12 to 1.14e-7; the mat-vec 1.08e-7).  Each step starts from
// zero there and is added in the vector units: 0.98 to 1.04e-7 at the same time (64001 x 8192, 8 tokens: 176 us before and now).
#pragma once
#include <hip/hip_fp16.h>

#include <type_traits>

#include "common.h"

namespace prima {

typedef _Float16 tk_half8 __attribute__((ext_vector_type(8)));
typedef _Float16 tk_half2 __attribute__((ext_vector_type(2)));
typedef float tk_v4f __attribute__((ext_vector_type(4)));
typedef unsigned tk_v4u __attribute__((ext_vector_type(4)));

constexpr int TK_CUS = 256;
constexpr size_t TK_LDS = 160 * 1024;

// The activations of one super-block for NT token slots, a record: operands | sub-block sums | 2^-p per token
constexpr int tk_sums_at(int nt) { return nt * 1024; }
constexpr int tk_inv_at(int nt) { return nt * 1056; }
constexpr int tk_rec(int nt) { return nt * 1056 + (nt < 4 ? 16 : nt * 4); }
constexpr int tk_slots(int T) { return T <= 2 ? 2 : (T <= 4 ? 4 : (T <= 8 ? 8 : 16)); }

// ---- activations -> operands ----------------------------------------------------------------------------------------
// Sixteen lanes hold one token's super-block, lane i columns 16 i .. 16 i + 15 in v (RMSNorm gain applied); into the record.  ORD: the order of
// a slice's 8 columns in the operand: 0: 0 4 1 5 2 6 3 7 (Q4_K's nibbles), 1: 0 2 1 3 4 6 5 7 (bytes).
// INF: for formats whose products are not corrected afterwards (Q8_0, FP16), infinities pass as such; Q5_K and Q6_K give NaN for them,
// as their one-token mat-vec does.  SUMS: the sub-block sums too (what Q4_K and Q5_K take the centre and the minima from; without them
// Q6_K 16 x 14336, 8 tokens, 36.8 -> 32.8 us: every workgroup lays out all of the activations).
// A 16-byte piece (8 columns of one row) c = 4 S + j, S the sub-block, j the slice, lies at a[c][row ^ f(c)], f(c) = (c >> 1) & 15:
// the sixteen lanes write pieces whose rows would otherwise share their banks.
template <int NT, int ORD, bool INF, bool SUMS>
__device__ __forceinline__ void tk_split(const float (&v)[16], int i, int t, uint8_t *rec)
{
    uint8_t *const a = rec, *const sums = rec + tk_sums_at(NT);
    constexpr int MR = NT <= 8 ? 2 * NT : 16; // rows (of one part with 16 tokens)
    float amax = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) amax = fmaxf(amax, fabsf(v[k]));
    amax = row_max16(amax);
    int ex = 0;
    if (amax > 0.f) frexpf(amax, &ex); // amax < 2^ex
    int p = 10 - ex;
    p = p > 126 ? 126 : (p < -120 ? -120 : p); // (2^p and 2^-p are normal numbers)
    // INF, an infinite activation: its hi part is infinite and its lo part finite (below), so that a product with a weight that is not zero
    // stays infinite; the others, which no longer matter, must not become infinite beside it.
    if constexpr (INF) p = amax > 3.40282347e38f ? -113 : p;
    const float S = ldexpf(1.0f, p);
    _Float16 hh[16], ll[16];
    // The sum of what the products will see: hi parts (whose sum is exact or nearly so) and lo parts on their own
    float sum = 0.f, suml = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        float sv = v[k] * S;
        asm volatile("" : "+v"(sv)); // one rounded number for hi and lo (else the compiler folds the product into what uses it)
        hh[k] = static_cast<_Float16>(sv);
        float r = sv - static_cast<float>(hh[k]);
        if constexpr (INF) r = fmaxf(r, -1024.f); // (in a NaN's place: inf - inf; any other is smaller)
        ll[k] = static_cast<_Float16>(r);
        if constexpr (SUMS) {
            sum += static_cast<float>(hh[k]);
            suml += static_cast<float>(ll[k]);
        }
    }
#pragma unroll
    for (int gi = 0; gi < 2; ++gi) {
        const int c = 2 * i + gi;
        tk_half8 h, l;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int col = 8 * gi + (ORD == 0 ? (k & 1) * 4 + (k >> 1) : (k & 4) + (k & 1) * 2 + ((k >> 1) & 1));
            h[k] = hh[col];
            l[k] = ll[col];
        }
        const int f = (c >> 1) & 15;
        if constexpr (NT <= 8) {
            *reinterpret_cast<tk_half8 *>(a + (c * MR + (((2 * t) ^ f) & (MR - 1))) * 16) = h;
            *reinterpret_cast<tk_half8 *>(a + (c * MR + (((2 * t + 1) ^ f) & (MR - 1))) * 16) = l;
        } else {
            *reinterpret_cast<tk_half8 *>(a + (c * 32 + ((t ^ f) & 15)) * 16) = h;
            *reinterpret_cast<tk_half8 *>(a + (c * 32 + 16 + ((t ^ f) & 15)) * 16) = l;
        }
    }
    // the sub-block's sum (this lane and its neighbour), as hi + lo; [part (16 tokens)][S & 3][row][S >> 2]
    if constexpr (SUMS) {
        sum += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sum), 0xB1, 0xf, 0xf, true));
        suml += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, suml), 0xB1, 0xf, 0xf, true));
    }
    if (SUMS && (i & 1) == 0) {
        const int S8 = i >> 1;
        const _Float16 sh = static_cast<_Float16>(sum + suml), sl = static_cast<_Float16>((sum - static_cast<float>(sh)) + suml);
        _Float16 *q = reinterpret_cast<_Float16 *>(sums);
        if constexpr (NT <= 8) {
            q[((S8 & 3) * MR + 2 * t) * 2 + (S8 >> 2)] = sh;
            q[((S8 & 3) * MR + 2 * t + 1) * 2 + (S8 >> 2)] = sl;
        } else {
            q[((S8 & 3) * 16 + t) * 2 + (S8 >> 2)] = sh;
            q[((4 + (S8 & 3)) * 16 + t) * 2 + (S8 >> 2)] = sl;
        }
    }
    if (i == 0) reinterpret_cast<float *>(rec + tk_inv_at(NT))[t] = ldexpf(1.0f, -p);
}

// The same record by a whole wave, lane i columns 4 i .. 4 i + 3 in v, with the sub-block sums.  Two neighbouring lanes hold a piece's eight columns; they
// exchange halves, so that the even lane stores the hi part's piece and the odd lane the lo part's.
template <int CTRL>
__device__ __forceinline__ unsigned tk_dpp(unsigned v) { return static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, true)); }
template <int CTRL>
__device__ __forceinline__ float tk_dppf(float v) { return __builtin_bit_cast(float, tk_dpp<CTRL>(__builtin_bit_cast(unsigned, v))); }
__device__ __forceinline__ float tk_sum8(float v) // over the eight lanes of a sub-block
{
    v += tk_dppf<0xB1>(v);         // its neighbour's
    v += tk_dppf<0x4E>(v);         // the other pair's of the four
    return v + tk_dppf<0x141>(v);  // the other four's
}
template <int NT, int ORD, bool INF>
__device__ __forceinline__ void tk_split_wave(const float (&v)[4], int i, int t, uint8_t *rec)
{
    uint8_t *const a = rec, *const sums = rec + tk_sums_at(NT);
    constexpr int MR = NT <= 8 ? 2 * NT : 16;
    const float amax = wave_max(fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
    int ex = 0;
    if (amax > 0.f) frexpf(amax, &ex); // amax < 2^ex
    int p = 10 - ex;
    p = p > 126 ? 126 : (p < -120 ? -120 : p);
    if constexpr (INF) p = amax > 3.40282347e38f ? -113 : p; // (see tk_split)
    const float S = ldexpf(1.0f, p);
    tk_half2 hh[2], ll[2];
    float sum = 0.f, suml = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float sv = v[k] * S;
        asm volatile("" : "+v"(sv));
        const _Float16 h = static_cast<_Float16>(sv);
        float r = sv - static_cast<float>(h);
        if constexpr (INF) r = fmaxf(r, -1024.f);
        const _Float16 l = static_cast<_Float16>(r);
        hh[k >> 1][k & 1] = h;
        ll[k >> 1][k & 1] = l;
        sum += static_cast<float>(h);
        suml += static_cast<float>(l);
    }
    const bool odd = i & 1;
    unsigned w0[2], w1[2]; // columns 0..3 and 4..7 of the piece this lane stores
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const unsigned h = __builtin_bit_cast(unsigned, hh[k]), l = __builtin_bit_cast(unsigned, ll[k]);
        const unsigned own = odd ? l : h, got = tk_dpp<0xB1>(odd ? h : l);
        w0[k] = odd ? got : own;
        w1[k] = odd ? own : got;
    }
    tk_v4u o;
    if constexpr (ORD == 0) { // 0 4 1 5 2 6 3 7
        o[0] = __builtin_amdgcn_perm(w1[0], w0[0], 0x05040100u);
        o[1] = __builtin_amdgcn_perm(w1[0], w0[0], 0x07060302u);
        o[2] = __builtin_amdgcn_perm(w1[1], w0[1], 0x05040100u);
        o[3] = __builtin_amdgcn_perm(w1[1], w0[1], 0x07060302u);
    } else { // 0 2 1 3 4 6 5 7
        o[0] = __builtin_amdgcn_perm(w0[1], w0[0], 0x05040100u);
        o[1] = __builtin_amdgcn_perm(w0[1], w0[0], 0x07060302u);
        o[2] = __builtin_amdgcn_perm(w1[1], w1[0], 0x05040100u);
        o[3] = __builtin_amdgcn_perm(w1[1], w1[0], 0x07060302u);
    }
    const int c = i >> 1, f = (c >> 1) & 15, part = i & 1;
    if constexpr (NT <= 8) *reinterpret_cast<tk_v4u *>(a + (c * MR + (((2 * t + part) ^ f) & (MR - 1))) * 16) = o;
    else *reinterpret_cast<tk_v4u *>(a + (c * 32 + part * 16 + ((t ^ f) & 15)) * 16) = o;
    sum = tk_sum8(sum);
    suml = tk_sum8(suml);
    if ((i & 7) == 0) {
        const int S8 = i >> 3;
        const _Float16 sh = static_cast<_Float16>(sum + suml), sl = static_cast<_Float16>((sum - static_cast<float>(sh)) + suml);
        _Float16 *q = reinterpret_cast<_Float16 *>(sums);
        if constexpr (NT <= 8) {
            q[((S8 & 3) * MR + 2 * t) * 2 + (S8 >> 2)] = sh;
            q[((S8 & 3) * MR + 2 * t + 1) * 2 + (S8 >> 2)] = sl;
        } else {
            q[((S8 & 3) * 16 + t) * 2 + (S8 >> 2)] = sh;
            q[((4 + (S8 & 3)) * 16 + t) * 2 + (S8 >> 2)] = sl;
        }
    }
    if (i == 0) reinterpret_cast<float *>(rec + tk_inv_at(NT))[t] = ldexpf(1.0f, -p);
}

// ---- the weight stream of a wave --------------------------------------------------------------------------------------
// A stage is 16 rows x SBS super-blocks: requested in runs along the rows into registers, written to the wave's LDS buffer (a
// row's fields side by side, rows an odd number of 16-byte pieces apart) and read from there in operand order.
// PL: planes of a format, in 16-byte pieces a super-block and row (Q4_K: one plane of 9); d of Q6_K comes in halves.
template <int FMT> struct TkFmt;
template <> struct TkFmt<PRIMA_FMT_Q4_K> { static constexpr int SBS = 2, WAVES = 8, ORD = 0, NREG = 5, RS = 19; };
template <> struct TkFmt<PRIMA_FMT_Q5_K> { static constexpr int SBS = 2, WAVES = 8, ORD = 1, NREG = 6, RS = 23; };  // low 16 | hi 4 | header 2
template <> struct TkFmt<PRIMA_FMT_Q6_K> { static constexpr int SBS = 2, WAVES = 8, ORD = 1, NREG = 7, RS = 27; };  // low 16 | hi 8 | sub-scales 2 | d 1
template <> struct TkFmt<PRIMA_FMT_Q8_0> { static constexpr int SBS = 2, WAVES = 8, ORD = 1, NREG = 9, RS = 35; };  // quants 32 | d 2
template <> struct TkFmt<PRIMA_FMT_F16> { static constexpr int SBS = 1, WAVES = 8, ORD = 1, NREG = 8, RS = 33; };
template <int FMT> constexpr int tk_stage_bytes = 16 * TkFmt<FMT>::RS * 16;

template <int FMT> struct TkRegs {
    tk_v4u v[TkFmt<FMT>::NREG];
    unsigned short d; // Q6_K
};

template <bool NT>
__device__ __forceinline__ tk_v4u tk_load16(const uint8_t *base, uint32_t off)
{
    const tk_v4u *p = reinterpret_cast<const tk_v4u *>(base + off);
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// Piece (row, c) of this lane in request i of a plane with PR pieces a row: runs along the rows.  With fewer than four pieces a
// row four neighbouring lanes share the row and repeat its pieces (four lanes that name four rows take the address unit
// four times as long).
template <int PR>
__device__ __forceinline__ void tk_slot(int i, int lane, int &row, int &c)
{
    if constexpr (PR >= 4) {
        row = (i * 64 + lane) / PR;
        c = (i * 64 + lane) % PR;
    } else {
        row = lane >> 2;
        c = PR == 2 ? (lane & 3) >> 1 : 0;
    }
}
template <int PR>
__device__ __forceinline__ bool tk_owner(int lane) { return PR >= 4 || (PR == 2 ? (lane & 1) == 0 : (lane & 3) == 0); }

// Where a wave's requests of a tile start: a pointer per plane, an offset per request and lane (set once per tile)
template <int FMT> struct TkSrc {
    const uint8_t *p[4];
    uint32_t off[TkFmt<FMT>::NREG], off_d;
};
// bytes of a super-block in plane i (in the order of TkSrc::p)
template <int FMT> constexpr int tk_plane_bytes(int i)
{
    constexpr int b[5][4] = {{144, 0, 0, 0}, {128, 32, 16, 0}, {128, 64, 16, 2}, {256, 16, 0, 0}, {512, 0, 0, 0}};
    return b[FMT][i];
}
template <int FMT> constexpr int tk_planes = FMT == PRIMA_FMT_Q6_K ? 4 : (FMT == PRIMA_FMT_Q5_K ? 3 : (FMT == PRIMA_FMT_Q8_0 ? 2 : 1));

// rows row0 .. row0 + 15 of a matrix (past the end: the last row again, not stored)
template <int FMT>
__device__ __forceinline__ void tk_tile(TkSrc<FMT> &src, const uint8_t *__restrict__ W, int64_t n_rows, int nb, int64_t row0, int lane)
{
    constexpr int SBS = TkFmt<FMT>::SBS;
    const int last = static_cast<int>(n_rows - row0 < 16 ? n_rows - row0 : 16) - 1;
    const int64_t n = n_rows * nb, blk = row0 * nb;
    auto offset = [&](int row, int c, int pb) __attribute__((always_inline)) {
        const int cc = SBS == 2 && c >= pb && nb == 1 ? c - pb : c; // (a row of one super-block has no second one)
        return static_cast<uint32_t>(min(row, last)) * static_cast<uint32_t>(nb * pb * 16) + static_cast<uint32_t>(cc * 16);
    };
    auto plane = [&](int i, const uint8_t *base, auto pbc, int first) __attribute__((always_inline)) {
        constexpr int PB = decltype(pbc)::value, PR = PB * SBS, N = (16 * PR + 63) / 64;
        src.p[i] = base + blk * (PB * 16);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            int row, c;
            tk_slot<PR>(k, lane, row, c);
            src.off[first + k] = offset(row, c, PB);
        }
    };
    if constexpr (FMT == PRIMA_FMT_Q4_K) {
        src.p[0] = W + blk * 144;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int slot = i * 64 + lane, row = min(slot / 18, 15);
            src.off[i] = offset(row, min(slot - row * 18, 17), 9);
        }
    } else if constexpr (FMT == PRIMA_FMT_Q5_K) {
        plane(0, W + n * 16, std::integral_constant<int, 8>{}, 0);
        plane(1, W + n * 144, std::integral_constant<int, 2>{}, 4);
        plane(2, W, std::integral_constant<int, 1>{}, 5);
    } else if constexpr (FMT == PRIMA_FMT_Q6_K) {
        plane(0, W, std::integral_constant<int, 8>{}, 0);
        plane(1, W + n * 128, std::integral_constant<int, 4>{}, 4);
        plane(2, W + n * 192, std::integral_constant<int, 1>{}, 6);
        src.p[3] = W + n * 208 + blk * 2;
        src.off_d = (static_cast<uint32_t>(min(lane >> 2, last)) * static_cast<uint32_t>(nb) + (nb == 1 ? 0 : (lane & 3) >> 1)) * 2;
    } else if constexpr (FMT == PRIMA_FMT_Q8_0) {
        plane(0, W, std::integral_constant<int, 16>{}, 0);
        plane(1, W + n * 256, std::integral_constant<int, 1>{}, 8);
    } else {
        plane(0, W, std::integral_constant<int, 32>{}, 0);
    }
}

// super-blocks b .. b + SBS - 1 of the tile (all of them in the row, or nb == 1)
template <int FMT>
__device__ __forceinline__ void tk_load(TkRegs<FMT> &r, const TkSrc<FMT> &src, int b)
{
    // Whole lines read once in a launch carry the non-temporal bit; fields whose lines the next stages come back to do not
    // (with the bit on all of them, or on none, the output layer of 128256 x 8192 in Q8_0 takes 205 us instead of 180).
    auto some = [&](auto nt, int i, int first, int count) __attribute__((always_inline)) {
        const uint8_t *base = src.p[i] + static_cast<uint32_t>(b) * static_cast<uint32_t>(tk_plane_bytes<FMT>(i));
#pragma unroll
        for (int k = 0; k < count; ++k) r.v[first + k] = tk_load16<decltype(nt)::value>(base, src.off[first + k]);
    };
    typedef std::integral_constant<bool, true> Once;
    typedef std::integral_constant<bool, false> Again;
    if constexpr (FMT == PRIMA_FMT_Q4_K) {
        some(Again{}, 0, 0, 5);
    } else if constexpr (FMT == PRIMA_FMT_Q5_K) {
        some(Once{}, 0, 0, 4);
        some(Again{}, 1, 4, 1);
        some(Again{}, 2, 5, 1);
    } else if constexpr (FMT == PRIMA_FMT_Q6_K) {
        some(Once{}, 0, 0, 4);
        some(Once{}, 1, 4, 2);
        some(Again{}, 2, 6, 1);
        r.d = *reinterpret_cast<const unsigned short *>(src.p[3] + static_cast<uint32_t>(b) * 2u + src.off_d);
    } else if constexpr (FMT == PRIMA_FMT_Q8_0) {
        some(Once{}, 0, 0, 8);
        some(Again{}, 1, 8, 1);
    } else {
        some(Once{}, 0, 0, 8);
    }
}

template <int FMT>
__device__ __forceinline__ void tk_put(const TkRegs<FMT> &r, uint8_t *buf, int lane)
{
    constexpr int RS = TkFmt<FMT>::RS, SBS = TkFmt<FMT>::SBS;
    auto put = [&](int row, int c, const tk_v4u &v) __attribute__((always_inline)) { *reinterpret_cast<tk_v4u *>(buf + (row * RS + c) * 16) = v; };
    auto plane = [&](auto pbc, int at, int first) __attribute__((always_inline)) {
        constexpr int PR = decltype(pbc)::value * SBS, N = (16 * PR + 63) / 64;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            int row, c;
            tk_slot<PR>(i, lane, row, c);
            if (tk_owner<PR>(lane)) put(row, at + c, r.v[first + i]);
        }
    };
    if constexpr (FMT == PRIMA_FMT_Q4_K) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int slot = i * 64 + lane, row = slot / 18;
            if (i < 4 || lane < 32) put(row, slot - row * 18, r.v[i]);
        }
    } else if constexpr (FMT == PRIMA_FMT_Q5_K) {
        plane(std::integral_constant<int, 8>{}, 0, 0);
        plane(std::integral_constant<int, 2>{}, 8 * SBS, 4);
        plane(std::integral_constant<int, 1>{}, 10 * SBS, 5);
    } else if constexpr (FMT == PRIMA_FMT_Q6_K) {
        plane(std::integral_constant<int, 8>{}, 0, 0);
        plane(std::integral_constant<int, 4>{}, 8 * SBS, 4);
        plane(std::integral_constant<int, 1>{}, 12 * SBS, 6);
        if ((lane & 1) == 0) *reinterpret_cast<unsigned short *>(buf + ((lane >> 2) * RS + 13 * SBS) * 16 + ((lane & 3) >> 1) * 2) = r.d;
    } else if constexpr (FMT == PRIMA_FMT_Q8_0) {
        plane(std::integral_constant<int, 16>{}, 0, 0);
        plane(std::integral_constant<int, 1>{}, 16 * SBS, 8);
    } else {
        plane(std::integral_constant<int, 32>{}, 0, 0);
    }
    // other lanes of the wave read these bytes next: the LDS serves a wave in order, the compiler must not reorder
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// ---- one super-block: 16 rows (lane (n, g): row n) x all tokens ---------------------------------------------------------
// a constant in a vector register: an and-or takes one scalar operand, which the mask is
__device__ __forceinline__ unsigned tk_vconst(unsigned v)
{
    asm("" : "+v"(v));
    return v;
}
// four bytes -> binary16 pairs (0, 2), (1, 3) of 1024 + (byte & mask); e: 0x64006400 in a vector register
__device__ __forceinline__ void tk_pairs(unsigned u, unsigned mask, unsigned e, tk_half2 *p)
{
    p[0] = __builtin_bit_cast(tk_half2, (u & mask) | e);
    p[1] = __builtin_bit_cast(tk_half2, ((u >> 8) & mask) | e);
}
__device__ __forceinline__ tk_half8 tk_join(const tk_half2 *p)
{
    tk_v4u v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __builtin_bit_cast(unsigned, p[i]);
    return __builtin_bit_cast(tk_half8, v);
}
__device__ __forceinline__ tk_half2 tk_both(_Float16 v) { return tk_half2{v, v}; }
__device__ __forceinline__ _Float16 tk_small(unsigned v) { return static_cast<_Float16>(static_cast<unsigned short>(v)); }
__device__ __forceinline__ float tk_h2f(unsigned v) { return __half2float(__ushort_as_half(static_cast<unsigned short>(v & 0xffffu))); }
// bits of m from a, the others from b
__device__ __forceinline__ unsigned tk_sel(unsigned m, unsigned a, unsigned b) { return (a & m) | (b & ~m); }

// One super-block of 16 rows: its share of y[i], tokens 2 g' + i (NT <= 8, g' = g modulo the token pairs) or 4 g + i of row n.  ODD: multiplied
// as its negative (the K-quants).  In steps, so that two super-blocks can be worked on at a time (tk_mul2)
template <int FMT, int NT, bool ODD> struct TkSb {
    static constexpr int RS = TkFmt<FMT>::RS, SBS = TkFmt<FMT>::SBS;
    static constexpr int MR = NT <= 8 ? 2 * NT : 16, PS = NT <= 8 ? MR : 32; // rows of a part, rows between pieces
    static constexpr int NY = NT <= 8 ? 2 : 4;
    static constexpr bool Q4 = FMT == PRIMA_FMT_Q4_K, Q5 = FMT == PRIMA_FMT_Q5_K, Q6 = FMT == PRIMA_FMT_Q6_K, H = FMT == PRIMA_FMT_F16;

    const uint8_t *row, *a; // this lane's row in the wave's stage buffer; the activations' record
    int b, n, g;            // super-block of the stage; lane coordinates
    unsigned e1024, e64;    // exponents of 1024 and 64 in both halves
    float d = 1.f, dmin = 0.f;
    unsigned sc[2] = {}, mn[2] = {};
    tk_v4u quants[H ? 1 : 2]; // as stored, of a half of the super-block each
    uint2 high[2];            // Q5_K, Q6_K: their high bits
    tk_half8 Bc = {}, Bm = {}; // sums: centre times sub-scale, sub-min (slots 0 and 1: sub-blocks g and 4 + g)
    tk_v4f acc[2] = {}, rem = {}, lo = {}, ac = {}, am = {}; // a chain per half of the super-block; Q6_K's R; 16 tokens: the lo parts; centres, minima
    tk_half8 B[2][4], R[2][Q6 ? 4 : 1]; // Q6_K: R with the sub-scale's low 4 bits, B with the others (and a 16th of their value)
    tk_half8 A[2][4], Al[2][NT > 8 ? 4 : 1]; // the activations of a half

    __device__ __forceinline__ TkSb(const uint8_t *stage, int b_, const uint8_t *a_, int lane) : row(stage + (lane & 15) * RS * 16), a(a_), b(b_), n(lane & 15), g(lane >> 4)
    {
        e1024 = tk_vconst(0x64006400u);
        e64 = tk_vconst(0x54005400u);
    }
    __device__ __forceinline__ tk_half8 a_at(int c_static, int c_lane, int f_static, int f_lane, int part) const
    {
        const int m = ((n ^ f_lane) ^ f_static) & (MR - 1);
        return *reinterpret_cast<const tk_half8 *>(a + (c_lane * PS + m) * 16 + (c_static * PS + part * 16) * 16);
    }
    // the fields of the super-block (FP16: read where they are unpacked)
    __device__ __forceinline__ void fetch()
    {
        if constexpr (Q4 || Q5) {
            const uint4 hdr = *reinterpret_cast<const uint4 *>(row + (Q4 ? b * 9 : 10 * SBS + b) * 16);
            const int fsh = 6 * g;
            sc[0] = __builtin_amdgcn_ubfe(hdr.y, fsh, 6);
            sc[1] = __builtin_amdgcn_ubfe(__builtin_amdgcn_alignbit(hdr.z, hdr.y, 24), fsh, 6);
            mn[0] = __builtin_amdgcn_ubfe(__builtin_amdgcn_alignbit(hdr.w, hdr.z, 16), fsh, 6);
            mn[1] = __builtin_amdgcn_ubfe(hdr.w, 8 + fsh, 6);
            d = hdr_d(hdr);
            dmin = hdr_dmin(hdr);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (Q4) quants[h] = *reinterpret_cast<const tk_v4u *>(row + (b * 9 + 1 + 4 * h + g) * 16);
            if constexpr (Q5 || Q6) quants[h] = *reinterpret_cast<const tk_v4u *>(row + (8 * b + 4 * h + g) * 16);
            if constexpr (Q5) high[h].x = *reinterpret_cast<const unsigned *>(row + (8 * SBS + 2 * b) * 16 + (4 * h + g) * 4);
            if constexpr (Q6) {
                high[h] = *reinterpret_cast<const uint2 *>(row + (8 * SBS + 4 * b) * 16 + (4 * h + g) * 8);
                sc[h] = *reinterpret_cast<const unsigned short *>(row + (12 * SBS + b) * 16 + (4 * h + g) * 2);
            }
        }
        if constexpr (Q6) d = tk_h2f(*reinterpret_cast<const unsigned short *>(row + 13 * SBS * 16 + b * 2));
    }
    // half h (sub-blocks 4h .. 4h+3): its activations, its weights, their products
    template <int h> __device__ __forceinline__ void operands()
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            A[h][j] = a_at(16 * h + j, 4 * g, 8 * h | (j >> 1), 2 * g, 0);
            if constexpr (NT > 8) Al[h][j] = a_at(16 * h + j, 4 * g, 8 * h | (j >> 1), 2 * g, 1);
        }
    }
    template <int h> __device__ __forceinline__ void unpack()
    {
        if constexpr (Q4 || Q5) {
            const _Float16 s = ODD ? -tk_small(sc[h]) : tk_small(sc[h]), m = ODD ? -tk_small(mn[h]) : tk_small(mn[h]);
            Bc[h] = static_cast<_Float16>(Q4 ? 8.f : 16.f) * s;
            Bm[h] = m;
            const tk_half2 s2 = tk_both(s);
            if constexpr (Q4) {
                // A nibble in bits 0..3 of a half is the binary16 number q 2^-24, in bits 4..7 q 2^-20: times the sub-scale's 2^10 and 2^6, less
                // 8 of them, every pair becomes (q - 8) s 2^-14 (exact, and a normal number) with one instruction and one mask
                const tk_half2 s10 = s2 * tk_both(static_cast<_Float16>(1024.f)), s6 = s2 * tk_both(static_cast<_Float16>(64.f));
                const tk_half2 off = s2 * tk_both(static_cast<_Float16>(-0.00048828125f)); // -8 s 2^-14
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned w = quants[h][j], w8 = w >> 8;
                    tk_half2 p[4];
                    p[0] = __builtin_elementwise_fma(__builtin_bit_cast(tk_half2, w & 0x000f000fu), s10, off);
                    p[1] = __builtin_elementwise_fma(__builtin_bit_cast(tk_half2, w & 0x00f000f0u), s6, off);
                    p[2] = __builtin_elementwise_fma(__builtin_bit_cast(tk_half2, w8 & 0x000f000fu), s10, off);
                    p[3] = __builtin_elementwise_fma(__builtin_bit_cast(tk_half2, w8 & 0x00f000f0u), s6, off);
                    B[h][j] = tk_join(p);
                }
            } else {
                const unsigned hb = high[h].x;
                const tk_half2 off = s2 * tk_both(static_cast<_Float16>(-80.f)); // exact
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // bit 4 of the four weights 8 j + 4 x .. : bit 2 j + x of every byte
                    const unsigned w = quants[h][j];
                    const unsigned h0 = 2 * j <= 4 ? hb << (4 - 2 * j) : hb >> (2 * j - 4), h1 = 2 * j + 1 <= 4 ? hb << (3 - 2 * j) : hb >> (2 * j - 3);
                    const unsigned u0 = tk_sel(0x0f0f0f0fu, w, h0), u1 = tk_sel(0x0f0f0f0fu, w >> 4, h1);
                    // a byte's 5 bits in bits 4..8 of a half, under the exponent of 64: 64 + q
                    const unsigned u[4] = {u0 << 4, u0 >> 4, u1 << 4, u1 >> 4};
                    tk_half2 p[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        p[i] = __builtin_elementwise_fma(__builtin_bit_cast(tk_half2, (u[i] & 0x01f001f0u) | e64), s2, off);
                    B[h][j] = tk_join(p);
                }
            }
        } else if constexpr (Q6) {
            const uint2 hw = high[h];
            const unsigned scw = sc[h];
            // sub-scale = 16 s1 + s2, 0 <= s2 < 16: both parts' products with q - 32, and with 1056, are exact in 11 bits.  The two
            // sub-scales of the sub-block as bytes s + 128 in the halves of a word, their parts under the exponent of 1024
            const unsigned sb = __builtin_amdgcn_perm(0u, scw, 0x0c010c00u) ^ 0x00800080u;
            const tk_half2 c1 = tk_both(static_cast<_Float16>(1032.f)), c2 = tk_both(static_cast<_Float16>(1024.f)), off = tk_both(static_cast<_Float16>(-1056.f));
            const tk_half2 v1 = __builtin_bit_cast(tk_half2, ((sb >> 4) & 0x000f000fu) | e1024), v2 = __builtin_bit_cast(tk_half2, (sb & 0x000f000fu) | e1024);
            const tk_half2 s1 = ODD ? c1 - v1 : v1 - c1, s2 = ODD ? c2 - v2 : v2 - c2;
            const tk_half2 o1 = s1 * off, o2 = s2 * off;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const unsigned x = jj == 0 ? hw.x : hw.y;
#pragma unroll
                for (int j2 = 0; j2 < 2; ++j2) {
                    const unsigned w = quants[h][2 * jj + j2];
                    const unsigned u0 = tk_sel(0x0f0f0f0fu, w, j2 ? x : x << 4), u1 = tk_sel(0x0f0f0f0fu, w >> 4, j2 ? x >> 2 : x << 2);
                    tk_half2 v[4], p[4], e[4];
                    tk_pairs(u0, 0x003f003fu, e1024, v);
                    tk_pairs(u1, 0x003f003fu, e1024, v + 2);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        p[i] = __builtin_elementwise_fma(v[i], tk_both(s1[jj]), tk_both(o1[jj]));
                        e[i] = __builtin_elementwise_fma(v[i], tk_both(s2[jj]), tk_both(o2[jj]));
                    }
                    B[h][2 * jj + j2] = tk_join(p);
                    R[h][2 * jj + j2] = tk_join(e);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned neg = j & 1 ? 0x80008000u : 0u;
                const tk_v4u q = *reinterpret_cast<const tk_v4u *>(row + ((4 * h + g) * 4 + j) * 16);
                tk_v4u o; // numbers 0..7 as pairs (0, 2) (1, 3) (4, 6) (5, 7)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_perm(q[(i & 2) + 1], q[i & 2], (i & 1) ? 0x07060302u : 0x05040100u) ^ neg;
                B[h][j] = __builtin_bit_cast(tk_half8, o);
            }
        }
    }
    template <int h> __device__ __forceinline__ void products()
    {
        const tk_v4f zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (H) {
                tk_v4f c = zero;
                if constexpr (NT > 8) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(Al[h][j], B[h][j], c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[h][j], B[h][j], c, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[h][i] = j & 1 ? acc[h][i] - c[i] : (j == 0 ? c[i] : acc[h][i] + c[i]);
                continue;
            }
            if constexpr (Q6) rem = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[h][j], R[h][j], rem, 0, 0, 0);
            acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[h][j], B[h][j], acc[h], 0, 0, 0);
            if constexpr (NT > 8) {
                lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(Al[h][j], B[h][j], lo, 0, 0, 0);
                if constexpr (Q6) rem = __builtin_amdgcn_mfma_f32_16x16x32_f16(Al[h][j], R[h][j], rem, 0, 0, 0);
            }
        }
    }
    // the sub-block sums times centres and minima
    __device__ __forceinline__ void centre()
    {
        if constexpr (Q4 || Q5) {
            const uint8_t *const sums = a + tk_sums_at(NT);
            tk_v4u xs = {0u, 0u, 0u, 0u};
            if constexpr (NT > 8) {
                xs[0] = *reinterpret_cast<const unsigned *>(sums + ((4 + g) * MR + n) * 4);
                ac = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(tk_half8, xs), Bc, ac, 0, 0, 0);
                am = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(tk_half8, xs), Bm, am, 0, 0, 0);
            }
            xs[0] = *reinterpret_cast<const unsigned *>(sums + (g * MR + (n & (MR - 1))) * 4);
            ac = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(tk_half8, xs), Bc, ac, 0, 0, 0);
            am = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(tk_half8, xs), Bm, am, 0, 0, 0);
        }
    }
    // d s + (d ac - dmin am): the two in brackets are larger than their difference, the second's rounding is taken back
    __device__ __forceinline__ float scaled(float v, float vc, float vm) const
    {
        const float p = __fmul_rn(dmin, vm), e = __fmaf_rn(dmin, vm, -p);
        return fmaf(Q4 ? d * 16384.f : d, v, __fmaf_rn(d, vc, -p) - e); // (Q4_K's products are 2^-14 of the sums: exact)
    }
    __device__ __forceinline__ void finish(float *y) const
    {
        const float *const inv = reinterpret_cast<const float *>(a + tk_inv_at(NT));
        float iv[NY];
        if constexpr (NT <= 8) {
            const float2 t = *reinterpret_cast<const float2 *>(inv + 2 * (g & (NT / 2 - 1)));
            iv[0] = t.x; iv[1] = t.y;
        } else {
            const float4 t = *reinterpret_cast<const float4 *>(inv + 4 * g);
            iv[0] = t.x; iv[1] = t.y; iv[2] = t.z; iv[3] = t.w;
        }
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            float s;
            if constexpr (NT <= 8) {
                const float s0 = acc[0][2 * i] + acc[1][2 * i], s1 = acc[0][2 * i + 1] + acc[1][2 * i + 1];
                s = s0 + s1;
                if constexpr (Q6) s = fmaf(16.f, s, rem[2 * i] + rem[2 * i + 1]);
                if constexpr (Q4 || Q5) s = scaled(s, ac[2 * i] + ac[2 * i + 1], am[2 * i] + am[2 * i + 1]);
            } else {
                s = (acc[0][i] + acc[1][i]) + lo[i];
                if constexpr (Q6) s = fmaf(16.f, s, rem[i]);
                if constexpr (Q4 || Q5) s = scaled(s, ac[i], am[i]);
            }
            if constexpr (Q6) s *= d;
            y[i] = fmaf(s, ODD && !H ? -iv[i] : iv[i], y[i]);
        }
    }
};

// Q8_0, whose scales multiply finished sums
template <int NT>
__device__ __forceinline__ void tk_mul_q8(const uint8_t *stage, int b, const uint8_t *a, int lane, float *y)
{
    constexpr int RS = TkFmt<PRIMA_FMT_Q8_0>::RS, SBS = TkFmt<PRIMA_FMT_Q8_0>::SBS;
    constexpr int MR = NT <= 8 ? 2 * NT : 16, PS = NT <= 8 ? MR : 32, NY = NT <= 8 ? 2 : 4;
    const int n = lane & 15, g = lane >> 4;
    const uint8_t *row = stage + n * RS * 16;
    const tk_v4f zero = {0.f, 0.f, 0.f, 0.f};
    const unsigned e1024 = tk_vconst(0x64006400u);
    auto a_at = [&](int c_static, int c_lane, int f_static, int f_lane, int part) __attribute__((always_inline)) {
        const int m = ((n ^ f_lane) ^ f_static) & (MR - 1);
        return *reinterpret_cast<const tk_half8 *>(a + (c_lane * PS + m) * 16 + (c_static * PS + part * 16) * 16);
    };
    const float *const inv = reinterpret_cast<const float *>(a + tk_inv_at(NT));
    float iv[NY];
    if constexpr (NT <= 8) {
        const float2 t = *reinterpret_cast<const float2 *>(inv + 2 * (g & (NT / 2 - 1)));
        iv[0] = t.x; iv[1] = t.y;
    } else {
        const float4 t = *reinterpret_cast<const float4 *>(inv + 4 * g);
        iv[0] = t.x; iv[1] = t.y; iv[2] = t.z; iv[3] = t.w;
    }
    const tk_v4u dv = *reinterpret_cast<const tk_v4u *>(row + (16 * SBS + b) * 16);
    float t[NY];
#pragma unroll
    for (int i = 0; i < NY; ++i) t[i] = 0.f;
    const tk_half2 off = tk_both(static_cast<_Float16>(-1152.f));
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const uint2 w = *reinterpret_cast<const uint2 *>(row + b * 256 + s * 32 + g * 8);
        tk_half2 p[4];
        tk_pairs(w.x ^ 0x80808080u, 0x00ff00ffu, e1024, p);
        tk_pairs(w.y ^ 0x80808080u, 0x00ff00ffu, e1024, p + 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = s & 1 ? -off - p[i] : p[i] + off;
        const tk_half8 B = tk_join(p);
        const float d = tk_h2f(s & 1 ? dv[s >> 1] >> 16 : dv[s >> 1]);
        if constexpr (NT <= 8) {
            const tk_v4f c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_at(4 * s, g, 2 * s, g >> 1, 0), B, zero, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 2; ++i) t[i] = fmaf(s & 1 ? -d : d, c[2 * i] + c[2 * i + 1], t[i]);
        } else {
            tk_v4f c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_at(4 * s, g, 2 * s, g >> 1, 1), B, zero, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_at(4 * s, g, 2 * s, g >> 1, 0), B, c, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = fmaf(s & 1 ? -d : d, c[i], t[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < NY; ++i) y[i] = fmaf(t[i], iv[i], y[i]);
}

// y[i] += the share of super-block b of the stage
template <int FMT, int NT, bool ODD>
__device__ __forceinline__ void tk_mul(const uint8_t *stage, int b, const uint8_t *a, int lane, float *y)
{
    if constexpr (FMT == PRIMA_FMT_Q8_0) {
        tk_mul_q8<NT>(stage, b, a, lane, y);
    } else {
        TkSb<FMT, NT, ODD> s(stage, b, a, lane);
        s.fetch();
        s.template operands<0>();
        s.template unpack<0>();
        s.template operands<1>();
        s.template products<0>();
        s.template unpack<1>();
        s.template products<1>();
        s.centre();
        s.finish(y);
    }
}

// a matrix instruction, then some of the vector instructions that stand beside it, N times
template <int N, int V>
__device__ __forceinline__ void tk_interleave()
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// ... and of both super-blocks of a stage (a0, a1: their records), the second as its negative
template <int FMT, int NT>
__device__ __forceinline__ void tk_mul2(const uint8_t *stage, const uint8_t *a0, const uint8_t *a1, int lane, float *y)
{
    if constexpr (FMT == PRIMA_FMT_Q8_0) {
        tk_mul_q8<NT>(stage, 0, a0, lane, y);
        tk_mul_q8<NT>(stage, 1, a1, lane, y);
    } else {
        constexpr int M = (NT > 8 ? 8 : 4) * (FMT == PRIMA_FMT_Q6_K ? 2 : 1); // matrix instructions of a half
        constexpr int V = (FMT == PRIMA_FMT_Q6_K ? 100 : (FMT == PRIMA_FMT_Q5_K ? 72 : 52)) / M;
        TkSb<FMT, NT, false> s(stage, 0, a0, lane);
        TkSb<FMT, NT, true> t(stage, 1, a1, lane);
        s.fetch();
        s.template operands<0>();
        t.fetch();
        s.template unpack<0>();
        __builtin_amdgcn_sched_barrier(0);
        s.template operands<1>();
        s.template products<0>();
        s.template unpack<1>();
        tk_interleave<M, V>();
        t.template operands<0>();
        s.template products<1>();
        t.template unpack<0>();
        tk_interleave<M, V>();
        s.centre();
        t.template operands<1>();
        t.template products<0>();
        t.template unpack<1>();
        tk_interleave<M, V>();
        t.template products<1>();
        s.finish(y);
        t.centre();
        t.finish(y);
    }
}

} // namespace prima
