// The launches between the matrix products of a prompt (q4k_gemm.hip, fmt_gemm.hip): they add the shares of K that a product left,
// finish the vector (residual; 1/rms and SwiGLU; rotation and cache append) and lay it out as the next product's activations.
//
//   gemm_prepare_kernel  a vector, shares + residual, or SwiGLU of shares -> split activations (gemm_common.h), the vector itself where
//                        it is needed, and its sums of squares: RMSNorm's gain is applied here, 1/rms to the finished sums of the product.
//   rope_append_kernel   Q, K, V (or their shares) -> rotated queries and cache rows.
//   gemm_sum_kernel      shares (+ residual) -> a plain vector (the window's output, a product on its own).
//
// They do little and are launches of 5 us mostly for their trips through memory.  With a launch for the tokens' scales, one for the split, one for the
// shares' sum and one for rope, a layer of a prompt had seventeen launches; now ten.  The scale is therefore a power of two per token and super-block,
// which needs no pass over the row.
#include <algorithm>

#include "gemm_common.h"

namespace prima {
namespace {

typedef float gp_f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ gp_f4 ld4(const float *p) { return *reinterpret_cast<const gp_f4 *>(p); }
__device__ __forceinline__ unsigned gp_u(half2v v) { return __builtin_bit_cast(unsigned, v); }
template <int CTRL> __device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ unsigned dpp(unsigned v) { return __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, true); }

// N vectors of four numbers of each share of K, at off[] from p.  AT shares are requested at a time, and added pairwise (one layer in FP16, 17 tokens, error
// against 64 bits 2.40e-7 with 2 to 4 shares a product one after the other, 2.53 with 4 to 16, pairwise 2.34).
template <int N, int AT>
__device__ __forceinline__ void add_shares(const float *p, const int *off, int64_t stride, int n, gp_f4 *v)
{
    for (int s0 = 0; s0 < n; s0 += AT) {
        gp_f4 a[AT][N];
#pragma unroll
        for (int j = 0; j < AT; ++j) { // (past the last: the last again, not added)
            const float *const q = p + min(s0 + j, n - 1) * stride;
#pragma unroll
            for (int i = 0; i < N; ++i) a[j][i] = ld4(q + off[i]);
        }
#pragma unroll
        for (int j = 1; j < AT; ++j)
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (s0 + j >= n) a[j][i] = gp_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int h = AT / 2; h > 0; h /= 2)
#pragma unroll
            for (int j = 0; j < h; ++j)
#pragma unroll
                for (int i = 0; i < N; ++i) a[j][i] += a[j + h][i];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = s0 == 0 ? a[0][i] : v[i] + a[0][i];
    }
}

// A wave takes four tokens of a super-block: lane (m, j) the columns 64 i + 4 j .. + 3 of token m, a row of 16 lanes per token, so that the
// sums over a super-block stay in the row and nothing goes through LDS.  Everything is requested in front of the first use.
template <int MODE>
__device__ __forceinline__ void prepare_unit(const GemmPrepare &a)
{
    const int lane = threadIdx.x & 63, m = lane >> 4, j = lane & 15;
    // every argument that the launch will look at, requested at once
    if (MODE == GEMM_PLAIN) asm volatile("" ::"s"(a.T), "s"(a.nb), "s"(a.n_tiles), "s"(a.x), "s"(a.ldx), "s"(a.out), "s"(a.gain), "s"(a.A), "s"(a.waves));
    else asm volatile("" ::"s"(a.T), "s"(a.nb), "s"(a.n_tiles), "s"(a.x), "s"(a.ldx), "s"(a.out), "s"(a.gain), "s"(a.A), "s"(a.waves), "s"(a.p.part), "s"(a.p.n), "s"(a.p.stride),
                      "s"(a.p.ld), "s"(a.p.col[0]), "s"(a.norm.ss), "s"(a.norm.nb), "s"(a.norm.ld));
    const unsigned unit = blockIdx.x * a.waves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t4 = unit / static_cast<unsigned>(a.nb), b = unit - t4 * a.nb;
    if (t4 >= 4 * a.n_tiles) return;
    const int t = 4 * t4 + m, ts = min(t, a.T - 1);
    const int c0 = b * 256 + 4 * j;
    gp_f4 v[4], g[4];
    if (a.gain) {
#pragma unroll
        for (int i = 0; i < 4; ++i) g[i] = ld4(a.gain + c0 + 64 * i);
    }
    if (MODE == GEMM_PLAIN) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = ld4(a.x + ts * a.ldx + c0 + 64 * i);
    } else if (MODE == GEMM_RESIDUAL) {
        gp_f4 r[4];
        int off[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r[i] = ld4(a.x + ts * a.ldx + c0 + 64 * i);
            off[i] = 64 * i;
        }
        add_shares<4, 4>(a.p.part + ts * a.p.ld + a.p.col[0] + c0, off, a.p.stride, a.p.n, v);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] += r[i];
    } else { // column c of silu(gate) * up: see GemmShares
        const GemmSquares squares = gemm_squares<16>(a.norm, ts, j);
        int off[8];
        const int gc = c0 / 128 * 256 + c0 % 128 / 32 * 64 + c0 % 32;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = c0 + 64 * i;
            off[2 * i] = c / 128 * 256 + c % 128 / 32 * 64 + c % 32 - gc;
            off[2 * i + 1] = off[2 * i] + 32;
        }
        gp_f4 gu[8];
        add_shares<8, 2>(a.p.part + ts * a.p.ld + gc, off, a.p.stride, a.p.n, gu);
        const float ir = gemm_inv_rms_of<16>(a.norm, ts, j, squares);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float gt = gu[2 * i][k] * ir;
                v[i][k] = gt / (1.0f + expf(-gt)) * (gu[2 * i + 1][k] * ir);
            }
    }
    if (a.out && t < a.T) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<gp_f4 *>(a.out + t * a.ldo + c0 + 64 * i) = v[i];
    }
    if (!a.A) return;
    const gp_f4 none = {0.f, 0.f, 0.f, 0.f};
    if (t >= a.T) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = none;
    }
    if (a.gain) {
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ss += v[i][0] * v[i][0] + v[i][1] * v[i][1] + v[i][2] * v[i][2] + v[i][3] * v[i][3];
            v[i] *= g[i];
        }
        ss = row_sum16(ss);
        if (j == 3) a.ss[static_cast<int64_t>(b) * a.n_tiles * 16 + t] = ss;
    }
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) amax = fmaxf(amax, fabsf(v[i][k]));
    amax = row_max16(amax);
    int ex = 0;
    if (amax > 0.f) frexpf(amax, &ex); // amax < 2^ex
    const int p = min(100, max(-100, 10 - ex));
    const float scale = ldexpf(1.0f, p);
    uint8_t *const dst = a.A + (static_cast<int64_t>(t4 >> 2) * a.nb + b) * GM_TILE_BYTES;
    const int m16 = t & 15;
    const bool odd = j & 1;
    float sums[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        half2v h[2], l[2];
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float sv = v[i][k] * scale;
            // an opaque fp32 number: left visible, the compiler may form the stored hi from the rounded product with the gain and the hi that lo is
            // taken against from the exact one (fused multiply-convert); the two differ now and then by one binary16 step
            asm volatile("" : "+v"(sv));
            const _Float16 hi = static_cast<_Float16>(sv);
            const _Float16 lo = static_cast<_Float16>(sv - static_cast<float>(hi));
            h[k >> 1][k & 1] = hi;
            l[k >> 1][k & 1] = lo;
            sum += static_cast<float>(hi) + static_cast<float>(lo); // what the matrix cores will see
        }
        // columns 0..3 and 4..7 of a group of eight lie in neighbouring lanes; the even one stores the group's hi parts, the odd one the lo parts
        const unsigned s0 = dpp<0xB1>(odd ? gp_u(h[0]) : gp_u(l[0])), s1 = dpp<0xB1>(odd ? gp_u(h[1]) : gp_u(l[1]));
        const unsigned a0 = odd ? s0 : gp_u(h[0]), a1 = odd ? s1 : gp_u(h[1]), b0 = odd ? gp_u(l[0]) : s0, b1 = odd ? gp_u(l[1]) : s1;
        const uint4 o = make_uint4(__builtin_amdgcn_perm(b0, a0, 0x05040100u), __builtin_amdgcn_perm(b0, a0, 0x07060302u),
                                   __builtin_amdgcn_perm(b1, a1, 0x05040100u), __builtin_amdgcn_perm(b1, a1, 0x07060302u));
        *reinterpret_cast<uint4 *>(dst + (2 * (2 * i + (j >> 3)) + (odd ? 1 : 0)) * 1024 + (m16 + 16 * ((j & 7) >> 1)) * 16) = o;
        sum += dpp<0xB1>(sum);  // over the eight lanes of a sub-block: the neighbour, the pair beside, the other four
        sum += dpp<0x4E>(sum);
        sums[i] = sum + dpp<0x141>(sum);
    }
    // the sums slab: lane 0 of the token its hi parts, lane 1 its lo parts, lane 2 the scale
    half8 sh, sl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float other = row_ror<8>(sums[i]);
        const float e = j < 8 ? sums[i] : other, o = j < 8 ? other : sums[i];
        sh[2 * i] = static_cast<_Float16>(e);
        sh[2 * i + 1] = static_cast<_Float16>(o);
        sl[2 * i] = static_cast<_Float16>(e - static_cast<float>(sh[2 * i]));
        sl[2 * i + 1] = static_cast<_Float16>(o - static_cast<float>(sh[2 * i + 1]));
    }
    if (j == 0) *reinterpret_cast<half8 *>(dst + 16 * 1024 + m16 * 16) = sh;
    if (j == 1) *reinterpret_cast<half8 *>(dst + 16 * 1024 + 256 + m16 * 16) = sl;
    if (j == 2) *reinterpret_cast<float *>(dst + 16 * 1024 + GM_SCALES + m16 * 4) = ldexpf(1.0f, -p);
}

template <int MODE>
__global__ void __launch_bounds__(256) gemm_prepare_kernel(GemmPrepare a) { prepare_unit<MODE>(a); }

// A prompt's first launch: the first layer's activations, and behind them its RoPE table (a launch of 4.7 us by itself).
__global__ void __launch_bounds__(256) gemm_first_kernel(GemmPrepare a, RopeTable r, unsigned blocks)
{
    if (blockIdx.x < blocks) prepare_unit<GEMM_PLAIN>(a);
    else rope_table_entry(r, static_cast<int64_t>(blockIdx.x - blocks) * blockDim.x + threadIdx.x);
}

// y[t][row] = 1/rms * the shares of K of a number (+ residual)
__global__ void __launch_bounds__(256) gemm_sum_kernel(GemmShares p, GemmNorm norm, const float *resid, int64_t ldr, float *y, int64_t ldy, int64_t n_rows)
{
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int t = blockIdx.y;
    GemmSquares squares{};
    if (norm.ss) squares = gemm_squares<64>(norm, t, threadIdx.x & 63);
    const float r = resid && row < n_rows ? resid[t * ldr + row] : 0.f;
    float v = gemm_add_shares(p.part + t * p.ld + p.col[0] + min(row, n_rows - 1), p.stride, p.n);
    if (norm.ss) v *= gemm_inv_rms_of<64>(norm, t, threadIdx.x & 63, squares);
    if (row < n_rows) y[t * ldy + row] = resid ? v + r : v;
}

// One thread per four rotation pairs of a head of q, k or v of token blockIdx.y.  Pair i is (i, i + D/2) (mode 0) or (2i, 2i + 1): the
// two runs of four numbers that a thread reads are apart or side by side.
__global__ void __launch_bounds__(256) rope_append_kernel(RopeAppend a)
{
    asm volatile("" ::"s"(a.p[0].part), "s"(a.p[1].part), "s"(a.p[2].part), "s"(a.p[0].n), "s"(a.p[1].n), "s"(a.p[2].n), "s"(a.p[0].stride), "s"(a.p[0].ld),
                 "s"(a.norm.ss), "s"(a.norm.nb), "s"(a.norm.ld), "s"(a.tab), "s"(a.q), "s"(a.K), "s"(a.V), "s"(a.Hq), "s"(a.block)); // (requested at once)
    const int t = blockIdx.y, D = a.D, per = D / 8, heads = a.Hq + 2 * a.Hkv;
    const int u = blockIdx.x * a.block + threadIdx.x, h = min(u / per, heads - 1), i4 = (u % per) * 4;
    const int which = h < a.Hq ? 0 : (h < a.Hq + a.Hkv ? 1 : 2), hh = which == 0 ? h : (which == 1 ? h - a.Hq : h - a.Hq - a.Hkv);
    auto pick = [&](auto q, auto k, auto v) { return which == 0 ? q : (which == 1 ? k : v); };
    const GemmShares p = {pick(a.p[0].part, a.p[1].part, a.p[2].part), pick(a.p[0].n, a.p[1].n, a.p[2].n), pick(a.p[0].stride, a.p[1].stride, a.p[2].stride),
                          pick(a.p[0].ld, a.p[1].ld, a.p[2].ld), {pick(a.p[0].col[0], a.p[1].col[0], a.p[2].col[0]), 0, 0}};
    GemmSquares squares{};
    if (a.norm.ss) squares = gemm_squares<64>(a.norm, t, threadIdx.x & 63);
    const int ia = a.mode ? 2 * i4 : i4, ib = a.mode ? 2 * i4 + 4 : i4 + D / 2;
    const float *tab = a.tab + (static_cast<int64_t>(t) * (D / 2) + i4) * 2; // (cos, sin) of four pairs
    const gp_f4 cs0 = ld4(tab), cs1 = ld4(tab + 4);
    const int off[2] = {0, ib - ia};
    gp_f4 v[2];
    add_shares<2, 8>(p.part + t * p.ld + p.col[0] + hh * D + ia, off, p.stride, max(p.n, 1), v);
    if (a.norm.ss) {
        const float ir = gemm_inv_rms_of<64>(a.norm, t, threadIdx.x & 63, squares); // (all lanes of the wave)
        if (p.n > 0) { v[0] *= ir; v[1] *= ir; } // (0: complete)
    }
    if (u >= heads * per) return;
    if (which != 2) {
        const float c[4] = {cs0[0], cs0[2], cs1[0], cs1[2]}, s[4] = {cs0[1], cs0[3], cs1[1], cs1[3]};
        const gp_f4 x = v[0], y = v[1];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float p0 = a.mode ? (k < 2 ? x[2 * k] : y[2 * k - 4]) : x[k], p1 = a.mode ? (k < 2 ? x[2 * k + 1] : y[2 * k - 3]) : y[k];
            const float r0 = p0 * c[k] - p1 * s[k], r1 = p0 * s[k] + p1 * c[k];
            if (a.mode) {
                v[k >> 1][2 * (k & 1)] = r0;
                v[k >> 1][2 * (k & 1) + 1] = r1;
            } else {
                v[0][k] = r0;
                v[1][k] = r1;
            }
        }
    }
    if (which == 0) {
        float *const q = a.q + (static_cast<int64_t>(t) * a.Hq + hh) * D;
        *reinterpret_cast<gp_f4 *>(q + ia) = v[0];
        *reinterpret_cast<gp_f4 *>(q + ib) = v[1];
        return;
    }
    __half *const row = (which == 1 ? a.K : a.V) + (static_cast<int64_t>(hh) * a.kv_cap + a.n_past + t) * D;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        __half2 o[2] = {__floats2half2_rn(v[i][0], v[i][1]), __floats2half2_rn(v[i][2], v[i][3])};
        *reinterpret_cast<uint2 *>(row + (i ? ib : ia)) = *reinterpret_cast<const uint2 *>(o);
    }
}

} // namespace

prima_status launch_gemm_prepare(GemmPrepare a, const RopeTable &table, hipStream_t st)
{
    a.n_tiles = (a.T + 15) / 16;
    const int64_t units = static_cast<int64_t>(a.n_tiles) * 4 * a.nb;
    if (a.T < 1 || a.n_tiles > 65535 || units >= (int64_t{1} << 31)) return PRIMA_E_SHAPE;
    // a wave a workgroup while that spreads them over more compute units
    a.waves = units <= 8 * GM_CUS ? 1 : 4;
    const dim3 grid(static_cast<unsigned>((units + a.waves - 1) / a.waves)), block(64 * a.waves);
    if (table.tab) {
        const int64_t more = (table.n + block.x - 1) / block.x;
        if (a.mode != GEMM_PLAIN || grid.x + more >= (int64_t{1} << 31)) return PRIMA_E_SHAPE;
        hipLaunchKernelGGL(gemm_first_kernel, dim3(grid.x + static_cast<unsigned>(more)), block, 0, st, a, table, grid.x);
    } else if (a.mode == GEMM_PLAIN) hipLaunchKernelGGL(gemm_prepare_kernel<GEMM_PLAIN>, grid, block, 0, st, a);
    else if (a.mode == GEMM_RESIDUAL) hipLaunchKernelGGL(gemm_prepare_kernel<GEMM_RESIDUAL>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(gemm_prepare_kernel<GEMM_SWIGLU>, grid, block, 0, st, a);
    return last_launch_status();
}

prima_status launch_gemm_sum(const GemmShares &p, const GemmNorm &norm, const float *resid, int64_t ldr, float *y, int64_t ldy, int64_t n_rows, int T,
                             hipStream_t st)
{
    hipLaunchKernelGGL(gemm_sum_kernel, dim3(static_cast<unsigned>((n_rows + 255) / 256), T), dim3(256), 0, st, p, norm, resid, ldr, y, ldy, n_rows);
    return last_launch_status();
}

prima_status launch_rope_append(RopeAppend a, const prima_dims &d, int T, hipStream_t st)
{
    if (T <= 0) return PRIMA_OK;
    if (T > 65535 || static_cast<int64_t>(a.n_past) + T > a.kv_cap) return PRIMA_E_SHAPE;
    a.Hq = d.n_q_heads; a.Hkv = d.n_kv_heads; a.D = d.head_dim; a.mode = d.rope_mode;
    const int64_t n = static_cast<int64_t>(a.Hq + 2 * a.Hkv) * (a.D / 8);
    if (n >= (int64_t{1} << 30)) return PRIMA_E_SHAPE;
    a.block = n * T <= 64 * 8 * GM_CUS ? 64 : 256;
    hipLaunchKernelGGL(rope_append_kernel, dim3(static_cast<unsigned>((n + a.block - 1) / a.block), T), dim3(a.block), 0, st, a);
    return last_launch_status();
}

} // namespace prima
