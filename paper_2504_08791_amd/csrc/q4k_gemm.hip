// Q4_K matrix product for many tokens (prompt processing: the paper reports the time to the first token next to
// the time per output token, Sec. 4.1 / Table 2; the same projections as in decode, App. A.3, for T tokens at once).
//
//     y[t][r] = sum_c W[r][c] * a[t][c],   a = x (or RMSNorm(x; gain)),   + resid[t][r] (optional)
//
// With tens to thousands of tokens the product is a real contraction and belongs on the matrix cores; the decode
// kernel (tokens as int8 digits, sub-scales applied to every MFMA result) spends four multiply-adds per MFMA and
// token group and stops scaling at 8 tokens.  Here:
//   * the B operand is the weight tile itself: per sub-block of 32 weights the integers sc_s * q (at most 945:
//     exact in binary16), built in registers once per super-block and used for every token of the workgroup;
//   * the A operand is the activations as two binary16 numbers hi + lo (22 bits), scaled per token and super-block by a
//     power of two so that |a| < 1024; products of two binary16 numbers are exact in fp32, the MFMA adds in fp32;
//   * one accumulator per super-block (256 weights, 8 MFMA steps x 2); the min term sum_s m_s * xs_s (xs_s: the
//     sub-block sums of the scaled activations, again as hi + lo) is one more MFMA step with the m_s as B operand;
//     then  y += d * acc - dmin * acc_m  in fp32.
// gemm_prepare.hip splits the activations and lays them out in A-operand order per (16-token tile, super-block): 17 slabs of 1 KiB
// (8 sub-blocks x (hi, lo), and the sums), so that the product kernel moves them into LDS with 16-byte global->LDS loads and no
// arithmetic; the split is done once, not once per row block.  The product: a workgroup of 4 waves owns 256 rows x up to 64 tokens,
// a wave 64 rows (four B tiles in registers: every A tile read from LDS feeds four MFMAs per part); two workgroups
// share a compute unit, so that one's VALU and LDS phases run under the other's MFMAs.  The super-block is walked
// sub-block by sub-block; global->LDS loads fill a ring of activation slots two positions ahead and, per wave,
// two buffers with half a super-block of its rows' quants each (the comment at the kernel has the details).  Every XCD takes an equal run of
// (row block, token block, share of K) units in which neighbours share operands in its L2 (gemm_unit).  Up to three
// matrices with the same columns share a launch (Q / K / V), and so do a gate and an up matrix, with SwiGLU behind.
// The weights stay exact: dequantised to binary16 (one accumulator for all of K) they would be off by ~1e-3 per
// product, measured in the metric of the tests.
#include <hip/hip_fp16.h>

#include <atomic>
#include <type_traits>

#include "gemm_common.h"

namespace prima {
namespace {

typedef gm_v4f v4f;

constexpr int GM_THREADS = 256;
constexpr int GM_WAVES = GM_THREADS / 64;       // one wave per SIMD and workgroup
constexpr int GM_RT = 4;                        // 16-row tiles per wave
constexpr int GM_TT = 4;                        // 16-token tiles per workgroup
constexpr int GM_ROWS = 16 * GM_RT * GM_WAVES;  // rows per workgroup
constexpr int GM_TM = 16 * GM_TT;               // tokens per workgroup
constexpr int GM_NS = 3;                        // ring slots: positions whose activations are in LDS or on their way (a divisor
                                                // of the 9 positions of a super-block: the slot of a position is a constant; 4
                                                // and 5 slots measured the same)
constexpr int GM_SLOT = GM_TT * 2048;                                     // 8 KiB of activations
constexpr int GM_WQ = 2 * 4096;                                           // per wave: the quants of half a super-block, twice
// per wave: a super-block's headers as they come, and what its 64 rows need of them: the sub-scales as binary16 pairs [sub-block][row], the m_s [row], d and dmin
// [row] twice, of super-blocks in turn
constexpr int GM_HDR = 1024, GM_SC = 8 * 256, GM_M = 1024, GM_D = 512, GM_DEC = GM_SC + GM_M + 2 * GM_D;
constexpr int GM_LDS_BYTES = GM_NS * GM_SLOT + GM_WAVES * (GM_WQ + GM_HDR + GM_DEC); // 76 KiB: two workgroups per compute unit
static_assert(2 * GM_LDS_BYTES <= 160 * 1024, "two workgroups per compute unit");
struct GemmSegDev {
    const uint8_t *W;
    float *y;
    int64_t n_rows, ldy;
    int rb0; // first row block of this matrix (INT_MAX: unused)
};

// Up to three matrices with the same columns against the same activations in one launch (Q / K / V): their row blocks
// are numbered one matrix after the other.  pair: two matrices of equal shape (gate, up); a wave's two row tiles are
// then the same 16 rows of the one and of the other, a row block is 128 rows, and silu(gate) * up is stored to seg[0].y.
struct GemmArgs {
    GemmSegDev seg[3];
    int pair;
    int64_t n_cols;
    const uint8_t *A; // split activations: [token tile][super-block][17][64 lanes] x 16 bytes
    GemmNorm norm;
    const float *resid; // null: none (added to every stored row; launches with a residual have one matrix)
    int64_t ldr;
    int T, n_rb, n_tb; // row blocks, token blocks
    int band;                   // gemm_band()
    // K divided among ksplit workgroups per (row block, token block): each walks its share of the
    // super-blocks and stores its sums to part[split][token][ldp] (column: row block * GM_ROWS + row in the block); a
    // launch of gemm_prepare.hip adds them.  ksplit == 1: the sums go straight to y.
    int ksplit;
    int share_q, share_r, tile_q, tile_r; // super-blocks of a share and tiles of a token block: quotients, and how many have one more
    float *part;
    int64_t ldp;
};

// dma16_base with a per-lane pointer plus a constant byte offset (0 .. 4095) in the instruction instead.  The instruction adds
// its offset to the LDS address as well as to the global one, so M0 gets the LDS address less the offset.
template <int OFF>
__device__ __forceinline__ void dma16_off(const void *gptr, uint32_t lds_addr)
{
    static_assert(OFF >= 0 && OFF < 4096, "instruction offset");
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off offset:%2" : : "v"(gptr), "s"(lds_addr - OFF), "n"(OFF) : "memory");
}

// Requests a wave makes at the positions p - GM_AHEAD + 1 .. p - 1 behind position p = (b, s) of the product kernel's schedule
// (activations GM_AHEAD positions ahead: dm, or 1 where the target is the sums position; at s == 3, 4, 7 of a super-block with
// a successor 4, 1, 4 weight requests).  successor: whether super-block b has one; the one before b always had.
constexpr int GM_AHEAD = GM_NS - 1; // positions between an activation request and its use
constexpr int requests_at(int sk, bool successor, int dm) // sk < 0: a position of the super-block before (or the prologue)
{
    const int sp = sk < 0 ? sk + 9 : sk;
    return ((sp + GM_AHEAD) % 9 < 8 ? dm : 1) + ((sk < 0 || successor) ? (sp == 3 ? 4 : (sp == 4 ? 1 : (sp == 7 ? 4 : 0))) : 0);
}
constexpr int requests_behind(int s, bool successor, int dm)
{
    int n = 0;
    for (int k = 1; k < GM_AHEAD; ++k) n += requests_at(s - k, successor, dm);
    return n;
}
static_assert(GM_AHEAD >= 2 && GM_AHEAD <= 4, "the weight requests at s == 3, 4, 7 must be older than the activation requests a wait lets pass");

// One workgroup: 4 waves, one per SIMD; a wave owns 64 rows (four B tiles) x 64 tokens, i.e. 16 accumulator tiles for the
// super-block in hand and as many running sums; two workgroups share a compute unit (up to 256 registers per wave, 76 KiB of
// LDS per workgroup) and run out of step with each other.  The super-block is walked sub-block by sub-block ("positions"
// 0..7, then position 8: the sums slab and the min term).  Everything comes through LDS by 16-byte global->LDS loads:
//   activations: a ring of NS slots of 8 KiB, [4 token tiles][hi 1 KiB | lo 1 KiB] of a sub-block, shared by the four
//     waves, requested NS - 1 positions ahead (position 8 uses the slot's first 4 KiB for the sums slabs);
//   quants: per wave two buffers of 4 KiB, sub-blocks 0-3 and 4-7 of its 64 rows, each filled by four requests of 64
//     bytes x 16 rows as soon as the B tiles of the half super-block before have been built from it;
//   headers: 64 rows x 16 bytes per wave and super-block, decoded into LDS of the wave.
// Per position: wait until everything this wave requested two positions ago or earlier has landed (requests complete
// in order; the wait names the number of requests made since, which the schedule fixes), barrier (everyone's share of
// the activations is there, and everyone has finished reading the slot of the position before, which is the slot
// requested next), the position's requests, and then, token tile by token tile, the MFMAs of this position with,
// between them, the VALU work that builds the B tiles of the next position.  No global load is left for the compiler
// to wait on.  Measured with parts of the work switched off (8192 x 28672 weights, 1024 tokens): the LDS reads of the
// activations cost 30 % of the time, the requests 12 %, the B tiles 10 %, the barrier 3 %: a wave reads every
// activation of its 64 tokens once per position, whatever the tiling, so LDS bandwidth is met before the MFMA rate.
// TT: the token tiles of this workgroup.  The tiles are shared out evenly, so that 21 tiles (333 tokens) in six blocks are three workgroups
// of four and three of three; a tile past the last one was multiplied and thrown away.
template <int TT>
__device__ __forceinline__ void q4k_gemm_block(const GemmArgs &a, uint8_t *smem, int rb, int share, int tile0)
{
    constexpr int SLOT = GM_SLOT;
    constexpr int WQ_BASE = GM_NS * SLOT;            // per wave two buffers of 4 KiB: quants of sub-blocks 0-3, of 4-7
    constexpr int HDR = WQ_BASE + GM_WAVES * GM_WQ, DEC = HDR + GM_WAVES * GM_HDR;
    constexpr int DM = (TT + 1) / 2;                 // activation requests per wave at a sub-block position (one at the sums position)
    static_assert(TT >= 1 && TT <= GM_WAVES && GM_WAVES == 4, "requests per wave and position are counted for up to 4 tiles and 4 waves");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int nb = static_cast<int>(a.n_cols >> 8);
    const int sg = a.pair ? 0 : (rb >= a.seg[2].rb0 ? 2 : (rb >= a.seg[1].rb0 ? 1 : 0));
    const GemmSegDev &my = a.seg[sg];
    // first row of this wave: 64 rows of one matrix, or (pair) the same 32 rows of the gate and of the up matrix
    const int64_t row0 = a.pair ? static_cast<int64_t>(rb) * (GM_ROWS / 2) + wave * 32
                                : static_cast<int64_t>(rb - my.rb0) * GM_ROWS + wave * 64;
    // Weight requests of this lane.  Headers: 16 bytes of local row `lane`.  Quants: request k of a half super-block
    // brings 64 bytes (four sub-blocks) of each of the local rows 16k .. 16k+15, this lane the 16 bytes of sub-block
    // (lane & 3) of row 16k + (lane >> 2): 16 runs of 64 bytes per request (16 bytes of each of 64 rows per request cost
    // about 12 % at 1024 tokens and more).  Local row r: row0 + r of the matrix, or (pair) row0 + (r & 31) of the gate
    // (r < 32) or the up matrix; past the end: a valid row, not stored.
    const uint32_t stride = static_cast<uint32_t>(nb) * 144; // of a row (the host refuses more)
    const int64_t row_c = min<int64_t>(row0, my.n_rows - 1);
    const int left = static_cast<int>(min<int64_t>(my.n_rows - 1 - row_c, 63)); // rows of this wave behind its first
    // The four 16-byte pieces of a row's half lie in LDS in an order of their own for every fourth row, which the requests bring about: read in
    // the file's order, rows n and n + 4 share the banks (a row is 64 bytes), four lanes to each.
    const uint32_t lds0 = lds_address(smem);
    // this workgroup's share of K: super-blocks [b_lo, b_lo + nbl) (all of them unless K is divided; never empty: the
    // host keeps ksplit <= nb); below, `b` counts from b_lo
    const int b_lo = share * a.share_q + min(share, a.share_r);
    const int nbl = a.share_q + (share < a.share_r ? 1 : 0);
    const int64_t w_off = row_c * stride + static_cast<int64_t>(b_lo) * 144;
    const uint8_t *const w0 = my.W + w_off, *const w1 = (a.pair ? a.seg[1].W : my.W) + w_off; // local rows 0 .. 31, 32 .. 63
    const int total = 9 * nbl; // positions (n_cols < 2^32: no overflow)

    // Wave-uniform bases of this wave's activation requests: request jj of a sub-block position is slab (part, tile)
    // with part = wave & 1, tile = 2 jj + (wave >> 1); that of a sums position is tile `wave`.  Past the workgroup's
    // last tile: that one again, the same bytes to the same place.
    const uint8_t *abase[DM];
    auto tile_of = [&](int jj) __attribute__((always_inline)) { return TT % 2 == 0 ? 2 * jj + (wave >> 1) : min(2 * jj + (wave >> 1), TT - 1); };
#pragma unroll
    for (int jj = 0; jj < DM; ++jj) abase[jj] = a.A + ((static_cast<int64_t>(tile0 + tile_of(jj)) * nb + b_lo) * GM_SLABS + (wave & 1)) * 1024;
    const int xtile = TT == GM_WAVES ? wave : min(wave, TT - 1);
    const uint8_t *const xbase = a.A + ((static_cast<int64_t>(tile0 + xtile) * nb + b_lo) * GM_SLABS + 16) * 1024;
    const uint32_t lane16 = lane * 16;

    // the quants of half `half` (sub-blocks 4 half .. 4 half + 3) of super-block b: four requests; its headers: one
    auto issue_quants = [&](int b, int half) __attribute__((always_inline)) {
        const uint32_t dst = lds0 + WQ_BASE + wave * GM_WQ + half * 4096;
        const int64_t off = static_cast<int64_t>(b) * 144;
        const int l = lane_anew(), r = l >> 2;
        const uint32_t c = 16 + ((l & 3) ^ (l >> 4)) * 16;
        auto from = [&](int k) __attribute__((always_inline)) {
            const uint32_t rk = min((a.pair ? 16 * (k & 1) : 16 * k) + r, left);
            return (k < 2 ? w0 : w1) + off + (static_cast<uint64_t>(rk) * stride + c);
        };
        if (half == 0) {
            dma16_off<0>(from(0), dst);
            dma16_off<0>(from(1), dst + 1024);
            dma16_off<0>(from(2), dst + 2048);
            dma16_off<0>(from(3), dst + 3072);
        } else {
            dma16_off<64>(from(0), dst);
            dma16_off<64>(from(1), dst + 1024);
            dma16_off<64>(from(2), dst + 2048);
            dma16_off<64>(from(3), dst + 3072);
        }
    };
    auto issue_headers = [&](int b) __attribute__((always_inline)) {
        const int r = lane_anew();
        const uint32_t rr = min(a.pair ? r & 31 : r, left);
        dma16_off<0>((r < 32 ? w0 : w1) + static_cast<int64_t>(b) * 144 + static_cast<uint64_t>(rr) * stride, lds0 + HDR + wave * GM_HDR);
    };
    // the activation requests of position (b, s), into ring slot `slot` (s is a constant wherever this is called)
    auto issue = [&](int b, int s, int slot) __attribute__((always_inline)) {
        const uint32_t base = lds0 + slot * SLOT;
        const int64_t boff = static_cast<int64_t>(b) * (GM_SLABS * 1024);
        if (s < 8) {
#pragma unroll
            for (int jj = 0; jj < DM; ++jj)
                dma16_base(abase[jj] + boff + 2048 * s, lane16, base + tile_of(jj) * 2048 + (wave & 1) * 1024);
        } else {
            dma16_base(xbase + boff, lane16, base + xtile * 1024);
        }
    };

    v4f yacc[TT][GM_RT], acch[TT][GM_RT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int rt = 0; rt < GM_RT; ++rt) yacc[tt][rt] = acch[tt][rt] = {0.f, 0.f, 0.f, 0.f};

    // Requests complete in the order in which a wave made them, and every wait below names how many of the newest may
    // still be out.  Per position (b, s), behind the barrier: the activations of position p + NS - 1; at s == 3 the first
    // half of super-block b + 1's quants (their buffer was last read for position (b, 3), built during (b, 2)), at
    // s == 4 its headers, at s == 7 the second half (last read during (b, 6)).  The prologue makes its requests in the
    // order a super-block before this one would have: headers, first half, then the activations of the first NS - 1
    // positions with the second half where position (b - 1, 7) would have requested it.
    issue_headers(0);
    issue_quants(0, 0);
#pragma unroll
    for (int q = 0; q < GM_AHEAD; ++q) {
        issue(0, q, q);
        if (q == GM_AHEAD - 2) issue_quants(0, 1); // as position (b - 1, 7) would have
    }

    // A super-block's headers are decoded once, a lane a row, into LDS of the wave's own, at the last sub-block position of the super-block before
    // (the sub-scales there have been read then, and its m_s are read first).  (Decoded where they are used, by the four lanes
    // that share a row, for every tile, they were 18 of the 52 vector instructions of a position and 80 of those in front of the sums.)
    uint8_t *const dec = smem + DEC + wave * GM_DEC;
    auto decode_scales = [&](const uint4 &hd, int l, int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) {
            if (s8 < from || s8 >= to) continue;
            const _Float16 sc = static_cast<_Float16>(static_cast<unsigned short>(hdr_field(hd, s8)));
            *reinterpret_cast<half2v *>(dec + s8 * 256 + l * 4) = half2v{sc, sc} * half2v{static_cast<_Float16>(1024.f), static_cast<_Float16>(64.f)};
        }
    };
    auto decode_m = [&](const uint4 &hd, int l) __attribute__((always_inline)) {
        half8 m;
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) m[s8] = static_cast<_Float16>(static_cast<unsigned short>(hdr_field(hd, 8 + s8)));
        *reinterpret_cast<half8 *>(dec + GM_SC + l * 16) = m;
    };
    auto decode_d = [&](const uint4 &hd, int l, int bb) __attribute__((always_inline)) {
        *reinterpret_cast<float2 *>(dec + GM_SC + GM_M + (bb & 1) * GM_D + l * 8) = make_float2(hdr_d(hd) * 16384.f, hdr_dmin(hd)); // (the B tiles are 2^-14 of sc q)
    };
    auto header = [&](int l) __attribute__((always_inline)) { return *reinterpret_cast<const uint4 *>(smem + HDR + wave * GM_HDR + l * 16); };
    auto scale_of = [&](int rt, int s) __attribute__((always_inline)) { return *reinterpret_cast<const half2v *>(dec + s * 256 + (16 * rt + n) * 4); };
    // B tile `rt` of sub-block s from this wave's quants and sub-scales: 2^-14 sc_s q as binary16 (exact: 10 bits, 2^-14 at the
    // least).  A dword holds the eight weights of lane (n, g).  Masked in pairs (0,4) (1,5) (2,6) (3,7) they are subnormal binary16 numbers as
    // they stand, 2^-24 q and, the odd pairs (bits 4..7 of a half), 2^-20 q: one multiplication by 2^10 sc or 2^6 sc each.  (With an exponent
    // put in, 1024 + q, a fused multiply-add that took 1024 sc off again: four vector instructions more per tile pair; 70B 1024 tokens 3920 -> 3860 us, 8B
    // 333 489 -> 483.)
    // The quants are read a tile ahead of their use, with two VALU instructions a matrix instruction while they are unpacked.  This, the order of the
    // pieces above and the tiles pinned where they are built, one layer, us: 14B 333 tokens 700.6 -> 689.4, 64: 223.8 -> 218.9, 8B 333 490.4 -> 483.3; 70B
    // 256: 1030 -> 1020, 1024: 3648 -> 3620, 8B 2000 2098 -> 2087 (the last two within twice the spread of the runs)
    const int lane_q = n * 64 + ((n >> 2) << 4) + 4 * g;
    auto quants_of = [&](int rt, int s) __attribute__((always_inline)) {
        // request rt of the half brought rows 16 rt .. 16 rt + 15: [row][sub-block of the half][16 bytes]
        return *reinterpret_cast<const uint32_t *>(smem + WQ_BASE + wave * GM_WQ + (s >> 2) * 4096 + rt * 1024 + (lane_q ^ ((s & 3) << 4)));
    };
    auto build_b = [&](half8 &B, uint32_t w, half2v sc2) __attribute__((always_inline)) {
        const half2v sca = {sc2[0], sc2[0]}, scb = {sc2[1], sc2[1]};
#pragma unroll
        for (int pr = 0; pr < 4; ++pr) {
            const uint32_t v = pr < 2 ? w : w >> 8;
            const half2v r = __builtin_bit_cast(half2v, v & (pr & 1 ? 0x00f000f0u : 0x000f000fu)) * (pr & 1 ? scb : sca);
            B[2 * pr] = r[0];
            B[2 * pr + 1] = r[1];
        }
    };
    // the m_s, B operand of the sums position, and d and dmin
    auto m_of = [&](int l, int rt) __attribute__((always_inline)) { return *reinterpret_cast<const half8 *>(dec + GM_SC + (16 * rt + (l & 15)) * 16); };
    auto d_of = [&](int l, int rt, int bb) __attribute__((always_inline)) {
        return *reinterpret_cast<const float2 *>(dec + GM_SC + GM_M + (bb & 1) * GM_D + (16 * rt + (l & 15)) * 8);
    };

    // A wave issues in order: an MFMA occupies the matrix pipe for 16 cycles, during which
    // the same wave can issue three or four other instructions for free, and only then.  So the B tiles of position
    // p + 1 are built (VALU) between the MFMAs of position p, in the order the scheduling groups below prescribe;
    // built in front of their own MFMAs they would cost their full issue time with the matrix pipe idle.  The quants
    // and headers that position p + 1 needs are this wave's own requests; the wait below covers them.
    half8 Bc[GM_RT];     // B tiles of the current position (at the sums position: the m_s)
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(GM_AHEAD * DM + 4) : "memory"); // headers and first half of super-block 0 have landed
    {
        const uint4 hd = header(lane);
        decode_scales(hd, lane, 0, 8);
        decode_m(hd, lane);
        decode_d(hd, lane, 0);
#pragma unroll
        for (int rt = 0; rt < GM_RT; ++rt) build_b(Bc[rt], quants_of(rt, 0), scale_of(rt, 0));
    }

    for (int b = 0; b < nbl; ++b) {
        // one position; s as a constant of the type system (a loop over s with "#pragma unroll" is refused by the
        // optimizer once its body, which holds every case of s until it is unrolled, passes a size limit)
        auto position = [&](auto s_const) __attribute__((always_inline)) {
            constexpr int s = decltype(s_const)::value;
            constexpr int slot = s % GM_NS; // ring slot of this position
            static_assert(9 % GM_NS == 0, "a position's slot must not depend on the super-block");
            const int p = 9 * b + s;
            // Everything requested at position p - GM_AHEAD or before has landed (this wave's share of position p's
            // activations; the quants and headers that the B tiles built during this position need are no younger) once at
            // most the requests of the positions behind it are out (requests_behind: activations, DM or, where the target is a sums position,
            // one, and, where they fall on s == 3, 4, 7 of a super-block that has a successor, 4, 1, 4 weight requests).
            // The last position waits for everything.
            if (p + GM_AHEAD - 1 >= total) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else if (b + 1 < nbl) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(requests_behind(s, true, DM)) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" : : "n"(requests_behind(s, false, DM)) : "memory"); // the last super-block requests no weights
            gm_barrier();
            {
                // position p + NS - 1 goes into the slot that position p - 1 has just left
                const int s_t = (s + GM_NS - 1) % 9;
                const int b_t = b + (s + GM_NS - 1) / 9;
                constexpr int slot_t = (slot + GM_NS - 1) % GM_NS;
                if (b_t < nbl) issue(b_t, s_t, slot_t);
                if (b + 1 < nbl) {
                    if (s == 3) issue_quants(b + 1, 0);
                    if (s == 4) issue_headers(b + 1);
                    if (s == 7) issue_quants(b + 1, 1);
                }
            }
            const uint8_t *base = smem + slot * SLOT + lane * 16;
            const v4f zero = {0.f, 0.f, 0.f, 0.f};
            half8 Bn[GM_RT];
            // Token tile by token tile, each a scheduling region of its own (the scheduler, left alone, hoists all of
            // a position's LDS reads and runs out of registers): the tile's MFMAs, the LDS reads of the next tile, and
            // during the first four tiles one B tile of the next position each.
            if (s < 8) {
                // The hi and the lo parts alternate in one accumulator: 16 fp32 roundings per super-block at the
                // accumulator's magnitude.  Accumulators of their own for the lo parts (whose sums are 2^-11 of the hi
                // sums, so that only 8 roundings count) lower the product's rms error from 2.2e-7 to 1.8e-7 of the
                // output's rms, but need 64 registers more than a wave has with two workgroups on a compute unit.
                // LDS reads run two tiles ahead of their MFMAs (one tile, 8 MFMAs, is shorter than the LDS latency
                // while four waves and the incoming requests share the LDS)
                half8 ah[3], al[3];
                uint32_t wn[GM_RT];
                half2v sn[GM_RT];
                uint4 hd;
#pragma unroll
                for (int rt = 0; rt < GM_RT; ++rt)
                    if (s < 7 && rt * TT < GM_RT) { wn[rt] = quants_of(rt, s + 1); sn[rt] = scale_of(rt, s + 1); }
#pragma unroll
                for (int tt = 0; tt < (TT < 2 ? TT : 2); ++tt) {
                    ah[tt] = *reinterpret_cast<const half8 *>(base + tt * 2048);
                    al[tt] = *reinterpret_cast<const half8 *>(base + tt * 2048 + 1024);
                }
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    const half8 ch = ah[tt % 3], cl = al[tt % 3];
                    if (tt + 2 < TT) {
                        ah[(tt + 2) % 3] = *reinterpret_cast<const half8 *>(base + (tt + 2) * 2048);
                        al[(tt + 2) % 3] = *reinterpret_cast<const half8 *>(base + (tt + 2) * 2048 + 1024);
                    }
#pragma unroll
                    for (int rt = 0; rt < GM_RT; ++rt) {
                        acch[tt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ch, Bc[rt], s == 0 ? zero : acch[tt][rt], 0, 0, 0);
                        acch[tt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(cl, Bc[rt], acch[tt][rt], 0, 0, 0);
                    }
                    // the B tiles of the next position are shared out over the token tiles
#pragma unroll
                    for (int rt = 0; rt < GM_RT; ++rt) {
                        if (s < 7 && rt * TT / GM_RT == tt + 1) { wn[rt] = quants_of(rt, s + 1); sn[rt] = scale_of(rt, s + 1); }
                        if (s < 7 && rt * TT / GM_RT == tt) build_b(Bn[rt], wn[rt], sn[rt]);
                        if (s == 7 && rt * TT / GM_RT == tt) Bn[rt] = m_of(lane_anew(), rt);
                    }
                    if (s == 7) { // the headers of the next super-block (past the last: the last ones again)
                        const int l = lane_anew();
                        if (tt == 0) hd = header(l);
                        if (tt == (TT > 1 ? 1 : 0)) decode_scales(hd, l, 0, TT > 2 ? 4 : 8);
                        if (TT > 2 && tt == 2) decode_scales(hd, l, 4, 8);
                        if (tt == TT - 1) {
                            decode_m(hd, l);
                            decode_d(hd, l, b + 1);
                        }
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, TT == 4 ? 4 : 2 + 2 * GM_RT, 0);
#pragma unroll
                    for (int k = 0; k < 2 * GM_RT; ++k) { // one MFMA, then up to so many VALU instructions of the builds
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, (s < 7 ? 2 : 5) * ((GM_RT + TT - 1) / TT), 0);
                    }
                    // built here, not where it is used: the compiler moved the unpacking into the next position, in front of its
                    // first matrix instruction
#pragma unroll
                    for (int rt = 0; rt < GM_RT; ++rt)
                        if (rt * TT / GM_RT == tt) asm volatile("" : "+v"(Bn[rt]));
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // the min term: sum_s m_s * xs_s, one MFMA step with the m_s as B operand; then the super-block's term
                // is formed at its own magnitude, scaled back (a power of two) and added in one step (one rounding per super-block
                // at the magnitude of the running sum)
                const uint8_t *const scales = smem + slot * SLOT + GM_SCALES + (lane_anew() >> 4) * 16;
                float2 dd[GM_RT];
                const int l = lane_anew();
#pragma unroll
                for (int rt = 0; rt < GM_RT; ++rt) dd[rt] = d_of(l, rt, b);
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    const half8 cx = gemm_sums_operand(*reinterpret_cast<const half8 *>(base + tt * 1024), g);
                    const v4f cs = *reinterpret_cast<const v4f *>(scales + tt * 1024);
#pragma unroll
                    for (int rt = 0; rt < GM_RT; ++rt) {
                        const v4f am = __builtin_amdgcn_mfma_f32_16x16x32_f16(cx, Bc[rt], zero, 0, 0, 0);
                        // this lane: row n of row tile rt, tokens 4g .. 4g+3 of the tile
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            yacc[tt][rt][i] = fmaf(fmaf(dd[rt].x, acch[tt][rt][i], -(dd[rt].y * am[i])), cs[i], yacc[tt][rt][i]);
                    }
#pragma unroll
                    for (int rt = 0; rt < GM_RT; ++rt) {
                        if (rt * TT / GM_RT != tt) continue;
                        if (b + 1 < nbl) build_b(Bn[rt], quants_of(rt, 0), scale_of(rt, 0));
                        else Bn[rt] = Bc[rt];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int rt = 0; rt < GM_RT; ++rt) Bc[rt] = Bn[rt];
        };
        position(std::integral_constant<int, 0>{});
        position(std::integral_constant<int, 1>{});
        position(std::integral_constant<int, 2>{});
        position(std::integral_constant<int, 3>{});
        position(std::integral_constant<int, 4>{});
        position(std::integral_constant<int, 5>{});
        position(std::integral_constant<int, 6>{});
        position(std::integral_constant<int, 7>{});
        position(std::integral_constant<int, 8>{});
    }

    if (a.ksplit > 1) { // this share's sums
#pragma unroll
        for (int rt = 0; rt < GM_RT; ++rt) {
            const int64_t out_row = row0 + (a.pair ? 16 * (rt & 1) : 16 * rt) + n;
            if (out_row >= my.n_rows) continue;
            float *dst = a.part + static_cast<int64_t>(rb) * GM_ROWS + wave * 64 + 16 * rt + n;
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = (tile0 + tt) * 16 + 4 * g + i;
                    if (t < a.T) dst[(static_cast<int64_t>(share) * a.T + t) * a.ldp] = yacc[tt][rt][i];
                }
        }
        return;
    }
    const float *inv = nullptr; // 1/rms of the workgroup's tokens
    if (a.norm.ss) {
        float *const red = reinterpret_cast<float *>(smem);
        gm_barrier(); // (the ring's last slots have been read)
        gemm_inv_rms_tokens<GM_TM>(a.norm, tile0 * 16, red, red + 256);
        inv = red + 256;
    }
    auto of = [&](int tt, int i) __attribute__((always_inline)) { return inv ? inv[16 * tt + 4 * g + i] : 1.f; };
    if (a.pair) { // row tiles 0, 1: rows of the gate matrix; 2, 3: the same rows of the up matrix
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            const int64_t out_row = row0 + 16 * rt + n;
            if (out_row >= my.n_rows) continue;
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = (tile0 + tt) * 16 + 4 * g + i;
                    if (t < a.T) {
                        const float sc = of(tt, i);
                        const float gt = yacc[tt][rt][i] * sc, up = yacc[tt][rt + 2][i] * sc;
                        my.y[t * my.ldy + out_row] = gt / (1.0f + expf(-gt)) * up;
                    }
                }
        }
        return;
    }
    // The residual is requested at once: number by number, each between the stores of the ones before, a trip through memory each (4096 x 4096,
    // 1024 tokens, K undivided, 110 us, now 99).
    float add[GM_RT][TT][4];
    if (a.resid) {
#pragma unroll
        for (int rt = 0; rt < GM_RT; ++rt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    add[rt][tt][i] = a.resid[min((tile0 + tt) * 16 + 4 * g + i, a.T - 1) * a.ldr + min<int64_t>(row0 + 16 * rt + n, my.n_rows - 1)];
    } else {
#pragma unroll
        for (int rt = 0; rt < GM_RT; ++rt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int i = 0; i < 4; ++i) add[rt][tt][i] = 0.f;
    }
#pragma unroll
    for (int rt = 0; rt < GM_RT; ++rt) {
        const int64_t out_row = row0 + 16 * rt + n;
        if (out_row >= my.n_rows) continue;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = (tile0 + tt) * 16 + 4 * g + i;
                if (t < a.T) my.y[t * my.ldy + out_row] = yacc[tt][rt][i] * of(tt, i) + add[rt][tt][i];
            }
    }
}

__global__ void __launch_bounds__(GM_THREADS, 2) q4k_gemm_kernel(GemmArgs a)
{
    request_args<sizeof(a)>();
    extern __shared__ __align__(16) uint8_t smem[];
    int rb, tb, share;
    if (!gemm_unit(blockIdx.x, a.n_rb, a.n_tb, a.ksplit, a.band, rb, tb, share)) return; // the whole workgroup, before any barrier
    const int tile0 = tb * a.tile_q + min(tb, a.tile_r);
    switch (a.tile_q + (tb < a.tile_r ? 1 : 0)) {
    case 1: q4k_gemm_block<1>(a, smem, rb, share, tile0); break;
    case 2: q4k_gemm_block<2>(a, smem, rb, share, tile0); break;
    case 3: q4k_gemm_block<3>(a, smem, rb, share, tile0); break;
    default: q4k_gemm_block<4>(a, smem, rb, share, tile0); break;
    }
}

// Into how many shares K is cut: none while the row and token blocks alone give every compute unit a workgroup; else as
// many as fill the workgroup slots of the device (two per compute unit), each share at least GM_MIN_SHARE super-blocks
constexpr int GM_MIN_SHARE = 4, GM_MAX_KSPLIT = 16;
int ksplit_for(int64_t n_rb, int64_t n_tb, int64_t nb)
{
    const int64_t wgs = n_rb * n_tb, slots = 2 * GM_CUS;
    if (wgs <= 0 || wgs * 2 > slots) return 1;
    const int64_t s = std::min<int64_t>({slots / wgs, nb / GM_MIN_SHARE, GM_MAX_KSPLIT});
    return s < 2 ? 1 : static_cast<int>(s);
}
// Token blocks and shares of K, `least` to `most` of these, by the time of the rounds of workgroups.  A super-block of t token tiles takes a workgroup that
// has its compute unit to itself 2.0 + 0.75 t us, two that share one 2.7 + 1.35 t (tiles of unequal blocks count mostly by their mean: the
// blocks of one compute unit even out); an undivided product has 4 us at its end that shares leave to the launch behind, shares go to memory and back.
// So the tokens are cut into more blocks than they need where the last round is better filled by it: 21 tiles (333 tokens) into seven blocks of three instead of
// six, the output projection of 8B 50.7 -> 45 us with its shares.  A block more costs what the unpacking of the weights once more costs: 5 % of
// its part, in long launches, which run at the card's power limit, 30 % (70B, 400 tokens, gate and up in eight blocks or nine 40 us slower than in seven, two shares).
// Where the step between the two lies does not matter from 150 to 700 us: with blocks and shares of each of 32 products (8 prompts of 8B to 70B) forced in turn, the choices
// are the same; without a step, 30 % or 5 % for all, they cost 0.1 % of a call on average and up to 46 us (70B, 400 tokens).
// Fitted to single launches (16 prompts of 17 to 1500 tokens, 8B to 70B, up to 4 more blocks and 14 shares) and to whole calls back to back.
// Whole calls, one layer, us, the fewest blocks and the shares by rounds times tiles / this: 8B 180 tokens 264 / 258, 800 831 / 816, 14B 333 520 / 498, 1500 1962 / 1926, 70B 1024
// 3601 / 3561; 28 others (8B to 70B, 17 to 1500 tokens) between 0.98 and 1.004 of what they were.
struct GemmPlan {
    int n_tb, shares;
};
GemmPlan plan_gemm(int64_t n_rb, int n_tiles, int64_t nb, int T, int64_t least, int64_t most)
{
    constexpr int64_t slots = 2 * GM_CUS;
    constexpr int MORE = 4; // blocks beyond the fewest
    const int fewest = (n_tiles + GM_TT - 1) / GM_TT;
    most = std::max(least, std::min<int64_t>({most, GM_MAX_KSPLIT, nb}));
    GemmPlan best{fewest, static_cast<int>(least)};
    double best_us = 0.;
    for (int n_tb = fewest; n_tb <= std::min(n_tiles, fewest + MORE); ++n_tb) {
        const double t = 0.2 * ((n_tiles + n_tb - 1) / n_tb) + 0.8 * n_tiles / n_tb, alone = 2. + 0.75 * t, both = 2.7 + 1.35 * t;
        for (int64_t ks = least; ks <= most; ++ks) {
            const int64_t units = n_rb * n_tb * ks, rest = units % slots;
            if (n_tb > fewest && units >= (int64_t{1} << 31) - GM_XCDS) break;
            const double rounds = static_cast<double>(units / slots) * both + (rest == 0 ? 0. : (rest <= GM_CUS ? alone : both));
            double us = rounds * static_cast<double>((nb + ks - 1) / ks) +
                        (ks == 1 ? 4. : 1. + static_cast<double>(ks) * T * static_cast<double>(n_rb) * GM_ROWS * 1.2e-6);
            us *= 1. + (us > 300. ? 0.3 : 0.05) * (n_tb - fewest) / fewest;
            if (best_us == 0. || us < best_us) {
                best_us = us;
                best = GemmPlan{n_tb, static_cast<int>(ks)};
            }
        }
    }
    return best;
}
// row blocks of one matrix; of a (gate, up) pair of n_rows each: 128 rows of both per block
int64_t row_blocks(int64_t n_rows, bool pair = false) { return pair ? (n_rows + GM_ROWS / 2 - 1) / (GM_ROWS / 2) : (n_rows + GM_ROWS - 1) / GM_ROWS; }
int token_blocks(int T) { return ((T + 15) / 16 + GM_TT - 1) / GM_TT; }

} // namespace

int gemm_ksplit(int T, int64_t n_rows, int64_t n_cols) { return ksplit_for(row_blocks(n_rows), token_blocks(T), n_cols / QK); }

size_t gemm_part_bytes(int T, int64_t n_rows, int64_t n_cols)
{
    const int s = gemm_ksplit(T, n_rows, n_cols);
    return s == 1 ? 0 : static_cast<size_t>(s) * static_cast<size_t>(T) * static_cast<size_t>(row_blocks(n_rows)) * GM_ROWS * sizeof(float);
}

// plan_gemm() takes no more shares than the first of them that fills the device with one token block, or four (its plans for 10 shapes of 1B to 70B widths, 20 to
// 8192 tokens)
int64_t gemm_most_shares(const int64_t *n_rows, int n_mats, int64_t n_cols, bool pair)
{
    int64_t n_rb = 0;
    for (int i = 0; i < (pair ? 1 : n_mats); ++i) n_rb += row_blocks(n_rows[i], pair);
    return std::min<int64_t>({GM_MAX_KSPLIT, n_cols / QK, std::max<int64_t>(4, (2 * GM_CUS + n_rb - 1) / n_rb)}) * n_rb * GM_ROWS;
}

size_t gemm_acts_bytes(int T, int64_t n_cols) { return (static_cast<size_t>(T) + 15) / 16 * static_cast<size_t>(n_cols / QK) * GM_TILE_BYTES; }
size_t gemm_ss_bytes(int T, int64_t n_cols) { return round_up((static_cast<size_t>(T) + 15) / 16 * 16 * static_cast<size_t>(n_cols / QK) * sizeof(float), 1024); }

prima_status launch_q4k_gemm(const GemmMat *mats, int n_mats, bool pair, int64_t n_cols, const GemmActs &x, int T, const float *resid, int64_t ldr,
                             void *part, size_t part_bytes, GemmShares *later, hipStream_t st)
{
    if (later) *later = GemmShares{};
    if (n_mats < 1 || n_mats > 3 || (pair && (n_mats != 2 || mats[0].n_rows != mats[1].n_rows || resid)) || (n_mats > 1 && !later))
        return PRIMA_E_SHAPE;
    if (T == 0) return PRIMA_OK;
    GemmArgs a{};
    int64_t n_rb = 0;
    for (int i = 0; i < 3; ++i) {
        a.seg[i].rb0 = 0x7fffffff;
        if (i >= n_mats || mats[i].n_rows == 0 || (pair && i == 1)) {
            if (i < n_mats) a.seg[i] = GemmSegDev{mats[i].W, mats[i].y, mats[i].n_rows, mats[i].ldy, 0x7fffffff};
            continue;
        }
        a.seg[i] = GemmSegDev{mats[i].W, mats[i].y, mats[i].n_rows, mats[i].ldy, static_cast<int>(n_rb)};
        n_rb += pair ? (mats[i].n_rows + GM_ROWS / 2 - 1) / (GM_ROWS / 2) : (mats[i].n_rows + GM_ROWS - 1) / GM_ROWS;
        if (n_rb >= (int64_t{1} << 30)) return PRIMA_E_SHAPE;
    }
    if (n_rb == 0) return PRIMA_OK;
    const int64_t nb = n_cols / QK;
    const int n_tiles = (T + 15) / 16;
    if (nb >= (int64_t{1} << 32) / 144) return PRIMA_E_SHAPE; // (a row of 4 GiB: its activations laid out would be 500)
    if (n_rb * token_blocks(T) >= (int64_t{1} << 31) - GM_XCDS || n_tiles > 65535 || nb >= (int64_t{1} << 31)) return PRIMA_E_SHAPE;
    static std::atomic<bool> attr_set{false}; // set twice by two threads at worst: the attribute call is idempotent
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(q4k_gemm_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, GM_LDS_BYTES) != hipSuccess)
            return PRIMA_E_DEVICE;
        attr_set = true;
    }
    a.pair = pair ? 1 : 0;
    a.n_cols = n_cols; a.A = x.A; a.norm = x.norm; a.resid = resid; a.ldr = ldr;
    a.T = T; a.n_rb = static_cast<int>(n_rb);
    a.ldp = n_rb * GM_ROWS;
    // K is divided when that fills the device and the caller's scratch holds the shares (T: a grid dimension of the launch that adds them)
    const int64_t share_bytes = static_cast<int64_t>(T) * a.ldp * static_cast<int64_t>(sizeof(float));
    const int64_t held = part && T <= 65535 ? static_cast<int64_t>(part_bytes / static_cast<size_t>(share_bytes)) : 0;
    GemmPlan p{};
    if (later) {
        p = plan_gemm(n_rb, n_tiles, nb, T, 1, std::max<int64_t>(1, held));
    } else {
        const int ks = ksplit_for(n_rb, token_blocks(T), nb), divided = held >= ks ? ks : 1;
        p = plan_gemm(n_rb, n_tiles, nb, T, divided, divided);
    }
    a.n_tb = p.n_tb; a.ksplit = p.shares; a.band = gemm_band(a.n_tb);
    a.share_q = static_cast<int>(nb / a.ksplit); a.share_r = static_cast<int>(nb % a.ksplit);
    a.tile_q = n_tiles / a.n_tb; a.tile_r = n_tiles % a.n_tb;
    a.part = a.ksplit > 1 ? static_cast<float *>(part) : nullptr;
    hipLaunchKernelGGL(q4k_gemm_kernel, dim3(gemm_grid(n_rb * a.n_tb * a.ksplit)), dim3(GM_THREADS), GM_LDS_BYTES, st, a);
    const prima_status ps = last_launch_status();
    if (ps != PRIMA_OK || a.ksplit == 1) return ps;
    GemmShares sh{a.part, a.ksplit, static_cast<int64_t>(T) * a.ldp, a.ldp, {0, 0, 0}};
    for (int i = 0; i < 3; ++i)
        if (a.seg[i].rb0 != 0x7fffffff) sh.col[i] = static_cast<int64_t>(a.seg[i].rb0) * GM_ROWS;
    if (!later) return launch_gemm_sum(sh, x.norm, resid, ldr, mats[0].y, mats[0].ldy, mats[0].n_rows, T, st);
    *later = sh;
    return PRIMA_OK;
}

} // namespace prima
