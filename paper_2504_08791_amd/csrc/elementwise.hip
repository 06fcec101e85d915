// RoPE angle table of a window step.  (RMSNorm and SwiGLU are fused into the mat-vec that consumes
// them; the rotation itself and the fp16 KV append are fused into the attention kernel.)
#include <algorithm>

#include "common.h"

namespace prima {

// Everything a window step needs before its first layer, in one launch: the mat-vec's counters zeroed and the RoPE table,
// tab[t][i] = (cos, sin) of pos_t * theta^(-2i/D) with pos_t = n_past + t (or the token's own position in a batch of sequences)
__global__ void __launch_bounds__(256) step_init_kernel(StepInit s) { step_init_entry(s, blockIdx.x * 256 + threadIdx.x); }

StepInit step_init_args(float *tab, int T, int D, int n_past, float theta, const int *positions, void *zero, size_t zero_bytes)
{
    StepInit s{reinterpret_cast<float2 *>(tab), T, D / 2, {}, static_cast<double>(theta), static_cast<unsigned *>(zero),
               static_cast<unsigned>(zero_bytes / sizeof(unsigned))};
    for (int t = 0; t < T && t < PRIMA_MAX_TOK; ++t) s.p.pos[t] = positions ? positions[t] : n_past + t;
    return s;
}

prima_status launch_step_init(const StepInit &s, hipStream_t st)
{
    hipLaunchKernelGGL(step_init_kernel, dim3(step_init_blocks(s)), dim3(256), 0, st, s);
    return last_launch_status();
}

// two regions filled with a word each (null: none), in one launch
__global__ void __launch_bounds__(256) fill_words_kernel(unsigned *a, unsigned na, unsigned va, unsigned *b, unsigned nb, unsigned vb)
{
    const unsigned idx = blockIdx.x * 256 + threadIdx.x;
    if (idx < na) a[idx] = va;
    if (idx < nb) b[idx] = vb;
}

prima_status launch_fill_words(void *a, size_t a_bytes, unsigned a_word, void *b, size_t b_bytes, unsigned b_word, hipStream_t st)
{
    const unsigned na = a ? static_cast<unsigned>(a_bytes / 4) : 0u, nb = b ? static_cast<unsigned>(b_bytes / 4) : 0u;
    const unsigned n = na > nb ? na : nb;
    if (n == 0) return PRIMA_OK;
    hipLaunchKernelGGL(fill_words_kernel, dim3((n + 255) / 256), dim3(256), 0, st, static_cast<unsigned *>(a), na, a_word,
                       static_cast<unsigned *>(b), nb, b_word);
    return last_launch_status();
}

// the same table for any number of consecutive positions (prompt processing; usually beside the first layer's activations, gemm_prepare.hip)
__global__ void __launch_bounds__(256) rope_table_kernel(RopeTable r) { rope_table_entry(r, static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x); }

prima_status launch_rope_table(const RopeTable &r, hipStream_t st)
{
    if (r.n <= 0) return PRIMA_OK;
    hipLaunchKernelGGL(rope_table_kernel, dim3(static_cast<unsigned>((r.n + 255) / 256)), dim3(256), 0, st, r);
    return last_launch_status();
}

// Read-only streaming probe: every thread reads 16 bytes per step with a grid-wide stride and folds them
// into one word, so that the loads cannot be dropped.  States what this device delivers for a plain
// linear read, next to the nominal HBM peak.
// NT: the loads carry the non-temporal bit (bytes read once: lines marked to leave the caches first), as the weight
// stream of the one-token mat-vec does.
template <bool NT>
__global__ void __launch_bounds__(256) stream_read_kernel(const uint4 *__restrict__ src, size_t n16, uint32_t *sink)
{
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    const v4u *p = reinterpret_cast<const v4u *>(src);
    uint32_t acc = 0;
    const size_t stride = static_cast<size_t>(gridDim.x) * 256;
    for (size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x; i < n16; i += stride) {
        const v4u v = NT ? __builtin_nontemporal_load(p + i) : p[i];
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == 0x9e3779b9u) sink[0] = acc; // practically never: keeps the loop alive without a store per thread
}

// a[i] = silu(a[i]) * u[i]: SwiGLU as a launch of its own, for gate / up projections that are not both Q4_K
// (for Q4_K the epilogue of their shared launch does it)
__global__ void __launch_bounds__(256) swiglu_kernel(float *__restrict__ a, const float *__restrict__ u, int64_t n)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) {
        const float g = a[i];
        a[i] = g / (1.0f + expf(-g)) * u[i];
    }
}

prima_status launch_swiglu(float *a, const float *u, int64_t n, hipStream_t st)
{
    if (n <= 0) return PRIMA_OK;
    hipLaunchKernelGGL(swiglu_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, a, u, n);
    return last_launch_status();
}

prima_status launch_stream_read(const void *src, size_t bytes, void *sink, hipStream_t st, bool nt)
{
    int dev = 0, cus = 256;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0) cus = prop.multiProcessorCount;
    if (nt) hipLaunchKernelGGL(stream_read_kernel<true>, dim3(cus * 8), dim3(256), 0, st, static_cast<const uint4 *>(src), bytes / 16,
                               static_cast<uint32_t *>(sink));
    else hipLaunchKernelGGL(stream_read_kernel<false>, dim3(cus * 8), dim3(256), 0, st, static_cast<const uint4 *>(src), bytes / 16,
                            static_cast<uint32_t *>(sink));
    return last_launch_status();
}

} // namespace prima
