// What the matrix products for many tokens share (q4k_gemm.hip, fmt_gemm.hip): the layout of the split activations and
// the loads and barriers of their pipelines.
#pragma once
#include "common.h"

namespace prima {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float gm_v4f __attribute__((ext_vector_type(4)));

// Split activations: [token tile of 16][super-block][17 slabs][64 lanes] x 16 bytes; slabs 2 s and 2 s + 1 are the hi and lo
// parts of sub-block s (lane (m, g): token m, columns 8g .. 8g+7 of the sub-block in the order 0 4 1 5 2 6 3 7), slab 16
// the sub-block sums (lane (m, 0) their hi parts, lane (m, 1) their lo parts).
constexpr int GM_SLABS = 17;
constexpr int GM_TILE_BYTES = GM_SLABS * 1024;
constexpr size_t GM_STAT_ALIGN = 1024;
constexpr int GM_XCDS = 8;
constexpr int GM_CUS = 256;

// Which (row block, token block, share of K) workgroup `wg` takes.  Consecutive workgroup numbers go to consecutive XCDs; each XCD
// takes an equal run of the units in an order in which neighbours share weights and activations in its L2: shares outermost, then bands
// of `band` row blocks, a band's row blocks of one token block one after the other (32 units at a time: 4 row blocks x 8 token blocks).
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
inline int gemm_band(int n_tb) { return 32 / (n_tb < 8 ? n_tb : 8); }

// the split activations and the per-token (2^p [* 1/rms], 2^-p) inside the scratch of gemm_ws_bytes(T, n_cols)
inline float2 *gemm_stat(void *ws) { return static_cast<float2 *>(ws); }
inline uint8_t *gemm_split(void *ws, int T)
{
    return static_cast<uint8_t *>(ws) + round_up(static_cast<size_t>(T) * sizeof(float2), GM_STAT_ALIGN);
}
// fills both (two launches)
prima_status launch_gemm_split(int64_t n_cols, const float *x, int64_t ldx, int T, const float *gain, float eps, void *ws, hipStream_t st);

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

// The shares of K of one number, `stride` numbers apart, added in order.  Eight are requested at a time (one by one, a trip through memory
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
        for (int j = 0; j < AT; ++j) v = i + j == 0 ? a[j] : (i + j < n ? v + a[j] : v);
    }
    return v;
}

} // namespace prima
