// 16-bit glue around the expert kernels: weighted average of the selected experts' outputs
// (paper §1) with the residual add of the chained configuration (§3: non-expert parts are
// always 16-bit).  The RMSNorm of that configuration lives in the gating kernel.
#include "common.hpp"
#include "kernels.hpp"

namespace moemix {

// v += y[p] for p = 1 .. splits - 1, in order, up to seven of them asked for per trip to memory (added one load at a
// time, the 14 partial results of 5 tokens in the Mixtral shape took 10.2 us; 5.7 us here).
__device__ __forceinline__ void add_splits(const float* __restrict__ y, int splits, size_t split_stride, float4_t& v) {
    for (int p0 = 1; p0 < splits; p0 += 7) {
        float4_t part[7];
#pragma unroll
        for (int p = 0; p < 7; ++p) {
            const int at = p0 + p < splits ? p0 + p : splits - 1;
            part[p] = *(const float4_t*)(y + at * split_stride);
        }
#pragma unroll
        for (int p = 0; p < 7; ++p)
            if (p0 + p < splits) v += part[p];
    }
}

// out[t, c] = fp16( residual[t, c] + sum_s gate[t, s] * sum_p y[p][inv[t*k+s], c] ), slots and partials added in order.
// INLINE: the grouped row of a pair is the number of pairs of lower experts and of earlier pairs of its own, counted
// by ballots over all of them.
template <bool INLINE>
__global__ __launch_bounds__(256) void combine_kernel(const float* __restrict__ y, int splits, size_t split_stride,
                                                       const float* __restrict__ gate, const int32_t* __restrict__ inv,
                                                       const int32_t* __restrict__ idx, int P, int d, int k,
                                                       const half_t* __restrict__ residual, half_t* __restrict__ out) {
    const int t = blockIdx.y;
    int pairs[INLINE ? kInlinePairs / 64 : 1];
    if (INLINE) load_pairs(idx, P, threadIdx.x & 63, pairs);
    const int c = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (!INLINE && c >= d) return;                     // (the ballots want every lane)
    float4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < k; ++s) {
        int r;
        if (INLINE) {
            const int me = t * k + s, e = idx[me], lane = threadIdx.x & 63;
            r = 0;
#pragma unroll
            for (int q = 0; q < kInlinePairs / 64; ++q)
                r += __popcll(__ballot(pairs[q] >= 0 && (pairs[q] < e || (pairs[q] == e && 64 * q + lane < me))));
        } else {
            r = inv[t * k + s];
            if (r < 0) continue;
        }
        if (INLINE && c >= d) continue;
        const float g = gate[t * k + s];
        const float* const row = y + (size_t)r * d + c;
        float4_t v = *(const float4_t*)row;
        add_splits(row, splits, split_stride, v);
        acc += g * v;
    }
    if (INLINE && c >= d) return;
    if (residual) {
        const half4_t rv = *(const half4_t*)(residual + (size_t)t * d + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += (float)rv[j];
    }
    half4_t o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (half_t)acc[j];
    *(half4_t*)(out + (size_t)t * d + c) = o;
}

void launch_combine(const float* y, int splits, size_t split_stride, const float* gate, const int32_t* inv, int T, int d,
                    int k, const half_t* residual, half_t* out, hipStream_t st, const int32_t* idx) {
    TraceScope trace(kKernelCombine, st);
    // few tokens: one wavefront per workgroup, or there are no more workgroups than a quarter of the compute units
    // (block, 64 and 256 threads: 2 tokens of the Mixtral shape, 4-bit, 95.7, 97.0 us; 5 tokens, three precisions, 229.4,
    // 230.5; 5 tokens, 1024 x 2816, 29.1, 29.6; no difference at 16 to 500 tokens, so the line may lie anywhere there)
    const int threads = (size_t)T * d <= 64 * 4096 ? 64 : 256;
    dim3 grid((d / 4 + threads - 1) / threads, T);
    if (inv) combine_kernel<false><<<grid, threads, 0, st>>>(y, splits, split_stride, gate, inv, nullptr, 0, d, k, residual, out);
    else combine_kernel<true><<<grid, threads, 0, st>>>(y, splits, split_stride, gate, nullptr, idx, T * k, d, k, residual, out);
}

// out[c] = fp16( sum_s gate[s] * slot_sums[s, c] ) over the slots whose expert ran, in slot order.
__global__ __launch_bounds__(256) void average_slots_kernel(const float* __restrict__ slot_sums, const int32_t* __restrict__ idx,
                                                             const float* __restrict__ gate, uint32_t ran, int d, int k,
                                                             half_t* __restrict__ out) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= d) return;
    float acc = 0.0f;
    for (int s = 0; s < k; ++s)
        if ((ran >> idx[s]) & 1u) acc = fmaf(gate[s], slot_sums[(size_t)s * d + c], acc);
    out[c] = (half_t)(0.0f + acc);
}

void launch_average_slots(const float* slot_sums, const int32_t* idx, const float* gate, uint32_t ran, int d, int k, half_t* out,
                          hipStream_t st) {
    TraceScope trace(kKernelCombine, st);
    average_slots_kernel<<<(d + 255) / 256, 256, 0, st>>>(slot_sums, idx, gate, ran, d, k, out);
}

// dst[i] = sum_p y[p][i], partials added in order
__global__ __launch_bounds__(256) void reduce_splits_kernel(const float* __restrict__ y, int splits, size_t split_stride,
                                                             size_t n4, float* __restrict__ dst) {
    for (size_t i = blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
        float4_t v = ((const float4_t*)y)[i];
        add_splits(y + i * 4, splits, split_stride, v);
        ((float4_t*)dst)[i] = v;
    }
}

void launch_reduce_splits(const float* y, int splits, size_t split_stride, size_t n, float* dst, hipStream_t st) {
    if (n == 0) return;
    const size_t n4 = n / 4;
    const int blocks = (int)((n4 + 255) / 256 < 2048 ? (n4 + 255) / 256 : 2048);
    reduce_splits_kernel<<<blocks, 256, 0, st>>>(y, splits, split_stride, n4, dst);
}

typedef uint4_t __attribute__((aligned(2))) uint4_half_aligned_t;
__global__ __launch_bounds__(256) void copy_halves_kernel(const half_t* __restrict__ src, size_t n8, half_t* __restrict__ dst) {
    for (size_t i = blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256)
        ((uint4_t*)dst)[i] = ((const uint4_half_aligned_t*)src)[i];
}

void launch_copy_halves(const half_t* src, size_t n, half_t* dst, hipStream_t st) {
    const size_t n8 = n / 8;
    copy_halves_kernel<<<(int)((n8 + 255) / 256 < 2048 ? (n8 + 255) / 256 : 2048), 256, 0, st>>>(src, n8, dst);
}

// Fill kernel used instead of a memset node so that every launch sequence stays graph-capturable.
__global__ void zero_words_kernel(int32_t* p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

void launch_zero_words(int32_t* p, int n, hipStream_t st) {
    if (n > 0) zero_words_kernel<<<(n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024, 256, 0, st>>>(p, n);
}

}  // namespace moemix
