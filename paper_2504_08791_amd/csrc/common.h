// Shared declarations of the HIP decode path (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stddef.h>
#include <stdint.h>

#include "prima.h"

namespace prima {

constexpr int QK = 256;          // weights per Q4_K super-block
constexpr int BLOCK_BYTES = 144; // bytes per super-block
constexpr int WAVE = 64;

inline prima_status last_launch_status()
{
    return hipGetLastError() == hipSuccess ? PRIMA_OK : PRIMA_E_DEVICE;
}

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- Q4_K header decoding (layout version 1, see prima.h) ----
// hdr = the first 16 bytes of a super-block as four little-endian dwords:
// hdr.x = d | dmin << 16, hdr.y/z/w = bits 0-31 / 32-63 / 64-95 of the field stream.
__device__ __forceinline__ float hdr_d(const uint4 &hdr)
{
    return __half2float(__ushort_as_half(static_cast<unsigned short>(hdr.x & 0xffffu)));
}
__device__ __forceinline__ float hdr_dmin(const uint4 &hdr)
{
    return __half2float(__ushort_as_half(static_cast<unsigned short>(hdr.x >> 16)));
}
// 6-bit field i (0..15): i < 8 sub-scale sc_i, otherwise sub-min m_{i-8}
__device__ __forceinline__ uint32_t hdr_field(const uint4 &hdr, int i)
{
    const int bit = 6 * i, w = bit >> 5, sh = bit & 31;
    const uint32_t lo = w == 0 ? hdr.y : (w == 1 ? hdr.z : hdr.w);
    const uint32_t hi = w == 0 ? hdr.z : (w == 1 ? hdr.w : 0u);
    const uint64_t two = static_cast<uint64_t>(lo) | (static_cast<uint64_t>(hi) << 32);
    return static_cast<uint32_t>(two >> sh) & 63u;
}

// ---- launchers implemented in the .hip files (host side, all asynchronous on `st`) ----

struct GemvSeg {
    const uint8_t *W;   // Q4_K matrix of this segment
    float *y;           // fp32 output [T][ldy]
    const float *resid; // optional fp32 [T][ldr] added to the product (may alias y)
    int64_t n_rows, ldy, ldr;
};

// how the mat-vec obtains its activation vector
enum XMode {
    X_PLAIN = 0,  // x as given
    X_RMSNORM = 1 // x * gain / sqrt(mean(x^2) + eps)
};

// what a launch stores
enum Epilogue {
    EPI_ROWS = 0,  // every segment's rows (+ residual) to its own y
    EPI_SWIGLU = 1 // two segments of equal shape (gate, up): silu(gate_r) * up_r to seg[0].y, nothing else
};

// up to three matrices with the same n_cols multiplied with the same activations in one launch
struct GemvArgs {
    GemvSeg seg[3];
    int nseg;
    int64_t n_cols;
    const float *x; // fp32 [T][ldx]
    int64_t ldx;
    int T;
    int xmode;         // XMode
    int epi;           // Epilogue
    const float *gain; // X_RMSNORM: fp32 [n_cols]
    float eps;         // X_RMSNORM
};

// the other weight formats (fmt_gemv.hip)
size_t fmt_tensor_bytes(int fmt, int64_t n_rows, int64_t n_cols);
prima_status launch_fmt_dequant(int fmt, const uint8_t *W, int64_t n_rows, int64_t n_cols, float *out, hipStream_t st);
// matrix_cores: several tokens may go to launch_tok_gemv()
prima_status launch_fmt_gemv(int fmt, const uint8_t *W, int64_t n_rows, int64_t n_cols, const float *x, int64_t ldx, int T,
                             const float *gain, float eps, const float *resid, int64_t ldr, float *y, int64_t ldy, hipStream_t st,
                             bool matrix_cores = true);

// 2 to 16 tokens in the formats whose weights are exact in binary16 operands (tok_gemv.hip); launch_fmt_gemv goes there
bool tok_gemv_takes(int fmt, int64_t n_rows, int64_t n_cols, int T);
int tok_gemv_first(int fmt, int64_t n_rows, int64_t n_cols, int T);
prima_status tok_gemv_plan_status(int fmt, int64_t n_rows, int64_t n_cols, int T); // host only: whether launch_tok_gemv() finds a plan
prima_status launch_tok_gemv(int fmt, const uint8_t *W, int64_t n_rows, int64_t n_cols, const float *x, int64_t ldx, int T,
                             const float *gain, float eps, const float *resid, int64_t ldr, float *y, int64_t ldy, hipStream_t st);

prima_status launch_dequant(const uint8_t *W, int64_t n_rows, int64_t n_cols, float *out, hipStream_t st);
// ws: scratch; its first arrivals_region bytes (>= gemv_arrivals_bytes(rows)) are counters that must be
// zero before the first launch (launch_zero_arrivals) and are left zero by every launch; the partial
// sums follow (gemv_ws_bytes() covers both for a region of gemv_arrivals_bytes(rows))
// zero_arrivals: the counters may hold anything; they are cleared by a launch of its own where a pass looks at them.
prima_status launch_gemv_mfma(const GemvArgs &a, void *ws, size_t ws_bytes, size_t arrivals_region, hipStream_t st, bool zero_arrivals = false);
size_t gemv_ws_bytes(int64_t n_rows_total, int64_t n_cols, int T);
size_t gemv_arrivals_bytes(int64_t n_rows_total);
prima_status launch_zero_arrivals(void *ws, size_t bytes, hipStream_t st);
// host only: whether every pass of this launch finds a plan and fits the scratch (nothing is launched)
prima_status gemv_plan_status(const GemvArgs &a, void *ws, size_t ws_bytes, size_t arrivals_region);

// RoPE table [T][D/2] of (cos, sin) for the positions n_past .. n_past + T - 1 (any T)
struct RopeTable {
    float2 *tab; // null: none
    int64_t n;   // T * half
    int half, n_past;
    double theta;
};
inline RopeTable rope_table(float *tab, int T, int D, int n_past, float theta)
{
    return RopeTable{reinterpret_cast<float2 *>(tab), static_cast<int64_t>(T) * (D / 2), D / 2, n_past, static_cast<double>(theta)};
}
// What a window step needs before its first layer: the RoPE table of up to PRIMA_MAX_TOK positions, counters zeroed
struct RopePositions {
    int pos[PRIMA_MAX_TOK];
};
struct StepInit {
    float2 *tab;
    int T, half;
    RopePositions p;
    double theta;
    unsigned *zero;
    unsigned n_zero;
};

// ---- many tokens (gemm_prepare.hip, q4k_gemm.hip, fmt_gemm.hip) ----
// The activations of a product: split and laid out for the matrix cores (gemm_common.h) by launch_gemm_prepare(), without 1/rms: that multiplies the
// finished sums, from the sums of squares ss[super-block][ld] of the tokens (ss null: no norm).
struct GemmNorm {
    const float *ss;
    int nb, ld; // ld: tokens rounded up to 16
    float eps;
};
struct GemmActs {
    const uint8_t *A;
    GemmNorm norm;
};
// K divided among workgroups leaves shares of the sums, without 1/rms: share s of token t, row r of matrix i at part[s * stride + t * ld + col[i] + r].
// (gate, up) pair: row r of the gate at r / 128 * 256 + r % 128 / 32 * 64 + r % 32 instead, of the up matrix 32 further.  n 0: there are none, the product is complete.
struct GemmShares {
    const float *part;
    int n;
    int64_t stride, ld, col[3];
};
enum { GEMM_PLAIN = 0, GEMM_RESIDUAL = 1, GEMM_SWIGLU = 2 };
struct GemmPrepare {
    int mode, T, n_tiles, nb; // v: [T][256 nb]
    const float *x;           // GEMM_PLAIN: v; GEMM_RESIDUAL: added to the shares p
    int64_t ldx;
    GemmShares p;             // GEMM_SWIGLU: of a pair
    GemmNorm norm;            // GEMM_SWIGLU: of the pair's activations
    float *out;               // v stored (null: not); may be x
    int64_t ldo;
    const float *gain; // null: none; else ss gets the sums of squares of v, and v * gain is laid out
    float *ss;
    uint8_t *A; // null: not laid out
    int waves;  // of a workgroup (filled in by the launch)
};
// table: beside GEMM_PLAIN, the prompt's RoPE table too (tab null: not)
prima_status launch_gemm_prepare(GemmPrepare a, const RopeTable &table, hipStream_t st);
size_t gemm_acts_bytes(int T, int64_t n_cols); // A
size_t gemm_ss_bytes(int T, int64_t n_cols);   // ss
// y = 1/rms * the shares of one matrix (+ resid)
prima_status launch_gemm_sum(const GemmShares &p, const GemmNorm &norm, const float *resid, int64_t ldr, float *y, int64_t ldy, int64_t n_rows, int T,
                             hipStream_t st);
// K divided among workgroups (a launch whose rows and tokens alone would leave most of the device idle) where the product itself has its shares added:
// the number of shares for T tokens and one matrix (1: none), and the bytes of `part` that hold their sums (0: none).  A launch divides K only if it
// is given that much.
int gemm_ksplit(int T, int64_t n_rows, int64_t n_cols);
size_t gemm_part_bytes(int T, int64_t n_rows, int64_t n_cols);
// Where the shares are left to the caller's next launch: room for the most numbers a token that they take, whatever T (prompts of a few tokens of
// very tall matrices excepted)
int64_t gemm_most_shares(const int64_t *n_rows, int n_mats, int64_t n_cols, bool pair = false);
// up to three matrices with the same columns against the same activations (Q / K / V), or, with pair set, two of equal
// shape (gate, up) with silu(gate) * up stored to mats[0].y; the residual only with one matrix.  later: the shares of K, if there are any, are left to
// the caller's next launch (resid and y then unused); null: one matrix, they are added here.
struct GemmMat {
    const uint8_t *W;
    float *y;
    int64_t n_rows, ldy;
};
prima_status launch_q4k_gemm(const GemmMat *mats, int n_mats, bool pair, int64_t n_cols, const GemmActs &x, int T, const float *resid, int64_t ldr,
                             void *part, size_t part_bytes, GemmShares *later, hipStream_t st);
// the same for one matrix in another format (fmt_gemm.hip), where fmt_gemm_takes(fmt) (all of them but FP32, whose weights
// are not exact in binary16)
bool fmt_gemm_takes(int fmt);
int64_t fmt_gemm_most_shares(int64_t n_rows, int64_t n_cols); // as gemm_most_shares()
struct FmtGemmBlocks {
    int tokens, blocks; // of a workgroup, and of these in a row block
    bool full;          // every workgroup does all of its tokens; else the blocks share the 16-token tiles out evenly
};
FmtGemmBlocks fmt_gemm_blocks(int T, int64_t n_rows, int64_t n_cols);
prima_status launch_fmt_gemm(int fmt, const GemmMat &m, int64_t n_cols, const GemmActs &x, int T, const float *resid, int64_t ldr, void *part,
                             size_t part_bytes, GemmShares *later, hipStream_t st);
// RoPE on q and k, k and v appended to the caches as rows n_past .. n_past + T - 1; p: shares of q, k, v (n 0: complete, at part); q: where the rotated
// queries go; tab from launch_rope_table
struct RopeAppend {
    GemmShares p[3];
    GemmNorm norm;
    const float *tab;
    float *q;
    __half *K, *V;
    int kv_cap, n_past;
    int Hq, Hkv, D, mode, block; // (filled in by the launch)
};
prima_status launch_rope_append(RopeAppend a, const prima_dims &d, int T, hipStream_t st);
prima_status launch_rope_table(const RopeTable &r, hipStream_t st);

prima_status launch_stream_read(const void *src, size_t bytes, void *sink, hipStream_t st, bool nt);
prima_status launch_swiglu(float *a, const float *u, int64_t n, hipStream_t st);
// the RoPE table [T][D/2] of (cos, sin), and `zero` cleared, in one launch (or at the end of a window's first, tok_stream.h).
// positions: null (token t sits at n_past + t) or T positions, one per token (a batch of sequences)
StepInit step_init_args(float *tab, int T, int D, int n_past, float theta, const int *positions, void *zero, size_t zero_bytes);
prima_status launch_step_init(const StepInit &s, hipStream_t st);
prima_status launch_fill_words(void *a, size_t a_bytes, unsigned a_word, void *b, size_t b_bytes, unsigned b_word, hipStream_t st);
size_t attn_ws_bytes(const prima_dims &d, int kv_cap, int T);
// The attention scratch: attn_counter_bytes() whose first word is the flag a bounded wait raises when it gives up
// (zero before a launch), then the key ranges' records.  Where a launch merges them itself, a record that has not been written holds
// ATTN_REC_EMPTY in every word: before the first such launch the records a launch will use (attn_records_bytes) must be filled with it
// (launch_fill_words); every launch leaves them so.
size_t attn_counter_bytes(const prima_dims &d, int T);
constexpr unsigned ATTN_REC_EMPTY = 0x7fa5c3e1u; // a NaN pattern that no arithmetic produces
// bytes of records (from the start of the record area) that such a launch for T tokens over n_total rows uses
size_t attn_records_bytes(const prima_dims &d, int n_total, int T);
// q: [T][Hq][D].  With rope_tab set, q and k_new are un-rotated and the kernel rotates them and
// appends k_new / v_new to the caches; otherwise q is used as is and the caches are complete.
// seq: null, or (a batch of T sequences, one token each) per token its sequence's caches and length; K, V and
// n_past are then not used.
// merge: by the workgroup of the first key range inside the launch (the records must be "not written" before); by a launch of its own; or
// by the caller's next one (tok_prepare_kernel), which finds them with attn_records() (nsplit 1: none, o is complete).
struct AttnSeqs;
enum AttnMerge { ATTN_MERGE_INSIDE = 0, ATTN_MERGE_APART = 1, ATTN_MERGE_LATER = 2 };
void attn_ranges(const prima_dims &d, int n_total, int T, bool batch, AttnMerge merge, int &keys_per_split, int &nsplit);
constexpr int ATTN_REC_HDR = 4; // a record: (max, sum, -, -), o[D]
struct AttnRecords {
    const float *part; // [T][Hq][nsplit][ATTN_REC_HDR + D]
    int nsplit;
};
prima_status launch_attn(const prima_dims &d, const float *q, float *q_rot_out, const float *k_new, const float *v_new,
                         const float *rope_tab, __half *K, __half *V, int kv_cap, int n_past, int T, float *o,
                         void *ws, hipStream_t st, const AttnSeqs *seq, AttnMerge merge);
// where that launch's records lie
AttnRecords attn_records(const prima_dims &d, int n_past, int T, void *ws, const AttnSeqs *seq);

// a prompt: rotated K / V rows already in the caches, q rotated; pieces of PRIMA_MAX_TOK tokens in one launch
prima_status launch_attn_prompt(const prima_dims &d, const float *q, __half *K, __half *V, int kv_cap, int n_past, int T,
                                float *o, hipStream_t st);
// (cos, sin) of pos * theta^(-2i/D), in fp64: at positions of several thousand an fp32 angle would already be off by ~1e-4 rad
__device__ __forceinline__ float2 rope_angle(int64_t pos, int i, int half, double theta)
{
    const double ang = static_cast<double>(pos) * pow(theta, -static_cast<double>(i) / static_cast<double>(half));
    return make_float2(static_cast<float>(cos(ang)), static_cast<float>(sin(ang)));
}
__device__ __forceinline__ void rope_table_entry(const RopeTable &r, int64_t idx)
{
    if (idx >= r.n) return;
    const int t = static_cast<int>(idx / r.half), i = static_cast<int>(idx - static_cast<int64_t>(t) * r.half);
    r.tab[idx] = rope_angle(static_cast<int64_t>(r.n_past) + t, i, r.half, r.theta);
}
__device__ __forceinline__ void step_init_entry(const StepInit &s, unsigned idx)
{
    if (idx < s.n_zero) s.zero[idx] = 0u;
    if (idx >= static_cast<unsigned>(s.T * s.half)) return;
    const int t = idx / s.half, i = idx - t * s.half;
    int pos = 0;
#pragma unroll
    for (int k = 0; k < PRIMA_MAX_TOK; ++k) pos = (k == t) ? s.p.pos[k] : pos; // no run-time index into the arguments
    s.tab[idx] = rope_angle(pos, i, s.half, s.theta);
}
inline unsigned step_init_blocks(const StepInit &s) // of 256 threads
{
    const unsigned n = static_cast<unsigned>(s.T * s.half) > s.n_zero ? static_cast<unsigned>(s.T * s.half) : s.n_zero;
    return (n + 255) / 256;
}

// Requests every line of a kernel's `bytes` of arguments at once, as its first thing.  A launch starts with cold scalar caches, and the
// compiler fetches an argument where it is first needed: two to five trips through memory one after the other (half a microsecond and more
// each) before the first load of data went out.  With this and the streams' matrices picked without fetches of their own, us, before / now: four 32B layers,
// 4 tokens 443 / 429, 14B with Q6_K 3 tokens 369 / 354, 16 sequences through three 14B layers 340 / 331, 14B 2 tokens 254 / 250, 8B prompt of 24 227 / 220.
// (One token's mat-vec requests most of them by itself: 147.7 / 147.3.  Not in the output layer's kernels: no change.)
template <int BYTES>
__device__ __forceinline__ void request_args()
{
    typedef const __attribute__((address_space(4))) uint32_t Word;
    Word *const p = (Word *)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t x = p[BYTES / 4 - 1];
#pragma unroll
    for (int i = 0; i < BYTES; i += 64) x ^= p[i / 4];
    asm volatile("" ::"s"(x));
}

// 16 bytes per lane from global memory straight into LDS: lane l writes bytes [16 l, 16 l + 16) of the
// 1 KiB at LDS byte address lds_addr (wave-uniform, goes through M0).  Written as inline assembly on
// purpose: the compiler then does not know these loads write LDS and leaves the ordering against the
// later LDS reads to the explicit s_waitcnt vmcnt(N) below, which lets newer stages stay in flight
// (with the builtin it waits for *all* outstanding loads before any LDS read).  Loads complete in
// order, so loads the compiler does not know about can only make its own waits stricter.
// NT: the load carries the non-temporal bit: the line is marked to leave the caches first.  For bytes that are read
// once in a launch (the weight stream of a one-token mat-vec, the cache rows of attention) that was measured 7 % faster
// on a 264 MB launch; not for the several-token mat-vec, whose row runs are short and whose lines that straddle two
// stages or two slabs are then fetched from memory twice.
template <bool NT = false>
__device__ __forceinline__ void dma16(const void *gptr, uint32_t lds_addr)
{
    // one wait state is required between the SALU write of M0 and the load that reads it; M0 is a reserved
    // register that nothing else in this file uses
    if (NT) asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" : : "v"(gptr), "s"(lds_addr) : "memory");
    else asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gptr), "s"(lds_addr) : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p)); // low half of a flat LDS pointer is the LDS byte address
}

// value of lane (i + n) % 16 of the same 16-lane row
template <int N>
__device__ __forceinline__ float row_ror(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_max16(float v)
{
    v = fmaxf(v, row_ror<8>(v));
    v = fmaxf(v, row_ror<4>(v));
    v = fmaxf(v, row_ror<2>(v));
    return fmaxf(v, row_ror<1>(v));
}
__device__ __forceinline__ float row_sum16(float v)
{
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    return v + row_ror<1>(v);
}

// Combining a value across the four 16-lane rows of a wave without LDS permutes: v_permlane16_swap_b32 a, b
// (gfx950) exchanges the odd rows of a with the even rows of b, v_permlane32_swap_b32 the upper half of a with the
// lower half of b.  With the value in both registers the results are (rows r0 r0 r2 r2, rows r1 r1 r3 r3) and
// (lower half twice, upper half twice); combining the two leaves, in every lane, the combination of its own
// value with the one 16 (32) lanes away.  (ds_bpermute, which __shfl_xor uses for these distances, costs an
// LDS round trip each.)  Written as inline assembly, with the wait states the instruction needs after a VALU
// write of its operands and before a VALU read of its results: the compiler's builtin for it was seen to take
// the two results for the same register (x + y compiled to x + x).
__device__ __forceinline__ void swap16_rows(unsigned &a, unsigned &b)
{
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32_halves(unsigned &a, unsigned &b)
{
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float add_across_16(float v)
{
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    swap16_rows(a, b);
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float add_across_32(float v)
{
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    swap32_halves(a, b);
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float max_across_16(float v)
{
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    swap16_rows(a, b);
    return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float max_across_32(float v)
{
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    swap32_halves(a, b);
    return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
// over all 64 lanes, the result in every lane: rotations inside the rows, then across them
__device__ __forceinline__ float wave_sum(float v) { return add_across_32(add_across_16(row_sum16(v))); }
__device__ __forceinline__ float wave_max(float v) { return max_across_32(max_across_16(row_max16(v))); }

} // namespace prima
