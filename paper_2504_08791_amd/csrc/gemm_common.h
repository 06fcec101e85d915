// What the matrix products for many tokens share (q4k_gemm.hip, fmt_gemm.hip): the layout of the split activations and
// the loads and barriers of their pipelines.
#pragma once
#include "common.h"

namespace prima {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float gm_v4f __attribute__((ext_vector_type(4)));

// Split activations: [token tile of 16][super-block][17 slabs][64 lanes] x 16 bytes; slabs 2 s and 2 s + 1 are the hi and lo
// parts of sub-block s (lane (m, g): token m, columns 8g .. 8g+7 of the sub-block in the order 0 4 1 5 2 6 3 7: that in which a dword of
// eight 4-bit weights unpacks into pairs), scaled by a power of two per token and super-block to less than 1024.  Slab 16: the sub-block sums, lane (m, 0)
// their hi parts, lane (m, 1) their lo parts; behind them, at GM_SCALES, the 16 tokens' scales as floats, 2^-p, and then nothing that was written: the
// lanes (m, 2) and (m, 3) of that operand have to be zeros (gemm_sums_operand()).
constexpr int GM_SLABS = 17;
constexpr int GM_TILE_BYTES = GM_SLABS * 1024;
constexpr int GM_SCALES = 512;
constexpr int GM_XCDS = 8;
constexpr int GM_CUS = 256;

// Which (row block, token block, share of K) workgroup `wg` takes.  Consecutive workgroup numbers go to consecutive XCDs; each XCD
// takes an equal run of the units in an order in which neighbours share weights and activations in its L2: shares outermost, then bands
// of `band` row blocks, a band's row blocks of one token block one after the other.
// False: none left.  (An XCD that took the row blocks xcd, xcd + 8, .. had three of 20 where others had two, 72 workgroups for 64 slots: 5120 rows, 512
// tokens, three shares 241 us.)
__device__ __forceinline__ bool gemm_unit(unsigned wg, int n_rb, int n_tb, int n_shares, int band, int &rb, int &tb, int &share)
{
    const int xcd = wg % GM_XCDS, seq = wg / GM_XCDS, plane = n_rb * n_tb;
    const int64_t units = static_cast<int64_t>(plane) * n_shares;
    const int first = static_cast<int>(units * xcd / GM_XCDS), u = first + seq;
    if (u >= static_cast<int>(units * (xcd + 1) / GM_XCDS)) return false;
    share = u / plane;
    const int v = u - share * plane, r0 = v / (band * n_tb) * band, h = min(band, n_rb - r0), w = v - r0 * n_tb;
    tb = w / h;
    rb = r0 + w - tb * h;
    return true;
}
inline unsigned gemm_grid(int64_t units) { return static_cast<unsigned>((units + GM_XCDS - 1) / GM_XCDS * GM_XCDS); }
// Up to eight token blocks: a row block's all together, its weights fetched once; beyond, eight row blocks by token block, whose activations they share: the 64
// workgroups that an XCD runs at a time are then eight by eight either way.  (Bands of 1, 4 and 8 measured the same to 1 %.)
inline int gemm_band(int n_tb) { return n_tb <= 8 ? 1 : 8; }

__device__ __forceinline__ half8 gemm_sums_operand(half8 v, int g)
{
    const half8 none = {};
    return g < 2 ? v : none;
}

// 1/rms of token t from its sums of squares over super-blocks, added by a wave or by 16 lanes (requested and added apart, so that
// other requests share the trip through memory), or by a workgroup of 256 threads for the NT
// tokens from t0 on (into inv[NT]; red[256]: scratch; both in LDS, a barrier in between and behind)
__device__ __forceinline__ float gemm_inv_rms(const GemmNorm &n, float squares) { return 1.0f / sqrtf(squares / (static_cast<float>(n.nb) * 256.f) + n.eps); }
struct GemmSquares {
    float s, u;
};
template <int LANES> // 16 or 64: requests the first 2 LANES super-blocks'
__device__ __forceinline__ GemmSquares gemm_squares(const GemmNorm &n, int t, int lane)
{
    return {n.ss[static_cast<int64_t>(min(lane, n.nb - 1)) * n.ld + t], n.ss[static_cast<int64_t>(min(lane + LANES, n.nb - 1)) * n.ld + t]};
}
template <int LANES>
__device__ __forceinline__ float gemm_inv_rms_of(const GemmNorm &n, int t, int lane, const GemmSquares &q)
{
    float s = (lane < n.nb ? q.s : 0.f) + (lane + LANES < n.nb ? q.u : 0.f);
    for (int b = lane + 2 * LANES; b < n.nb; b += LANES) s += n.ss[static_cast<int64_t>(b) * n.ld + t];
    return gemm_inv_rms(n, LANES == 16 ? row_sum16(s) : wave_sum(s));
}
template <int NT>
__device__ __forceinline__ void gemm_inv_rms_tokens(const GemmNorm &n, int t0, float *red, float *inv)
{
    constexpr int P = 256 / NT;
    constexpr int AT = 8; // requested at a time
    const int k = threadIdx.x % NT, t = min(t0 + k, n.ld - 1);
    float s = 0.f;
    for (int b = threadIdx.x / NT; b < n.nb; b += AT * P) {
        float v[AT];
#pragma unroll
        for (int j = 0; j < AT; ++j) v[j] = n.ss[static_cast<int64_t>(min(b + j * P, n.nb - 1)) * n.ld + t];
#pragma unroll
        for (int j = 0; j < AT; ++j) s += b + j * P < n.nb ? v[j] : 0.f;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < NT) {
#pragma unroll
        for (int i = 1; i < P; ++i) s += red[i * NT + k];
        inv[k] = gemm_inv_rms(n, s);
    }
    __syncthreads();
}

// The lane's number, made anew: what is addressed with it is formed where it is used (kept over a kernel's loop it spills).
__device__ __forceinline__ int lane_anew()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// 16 bytes per lane from global memory straight into LDS (as dma16), with the address as a wave-uniform base plus a
// 32-bit lane offset: the bases live in scalar registers and cost no vector register per request in flight
__device__ __forceinline__ void dma16_base(const void *sbase, uint32_t lane_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off), "s"(sbase), "s"(lds_addr) : "memory");
}

// workgroup barrier that orders LDS traffic only (__syncthreads() would also wait for every global load in flight,
// that is, for the whole ring of requests)
__device__ __forceinline__ void gm_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The shares of K of one number, `stride` numbers apart, eight added pairwise and the eights in order.  Eight are requested at a time (one by one, a trip through memory
// each: 333 tokens of 4096 rows, four or five shares, 8.5 to 9.6 us, now 8 to 8.5).
__device__ __forceinline__ float gemm_add_shares(const float *p, int64_t stride, int n)
{
    constexpr int AT = 8;
    float v = 0.f;
    for (int i = 0; i < n; i += AT) {
        float a[AT];
#pragma unroll
        for (int j = 0; j < AT; ++j) a[j] = p[min(i + j, n - 1) * stride]; // (past the last: the last again, not added)
#pragma unroll
        for (int j = 1; j < AT; ++j)
            if (i + j >= n) a[j] = 0.f;
        const float s = ((a[0] + a[4]) + (a[2] + a[6])) + ((a[1] + a[5]) + (a[3] + a[7]));
        v = i == 0 ? s : v + s;
    }
    return v;
}

} // namespace prima
