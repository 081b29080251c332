// Gating network with top-k selection (paper §1, §2.1) and the grouping of (token, slot)
// pairs by expert.
#include <type_traits>

#include "common.hpp"
#include "gating.hpp"
#include "kernels.hpp"

namespace moemix {

// One workgroup of four wavefronts per token.  Every wavefront holds the whole token row (lane L the 8-column
// chunks L, L + 64, ...), normalises it when the block input is RMSNorm(x) * gain, and evaluates the experts
// w, w + 4, ... of the gate matrix, each as one wavefront-wide dot product (gating.hpp), kAtOnce of them per trip to
// memory; the first wavefront then selects the top_k and computes the softmax over the selected logits.
// COPY: the token row goes to xn as it is.  (A kernel of its own: with the same line taken by all calls the one for 4096 columns
// had 213 registers instead of 117, 1792 tokens, 32 experts of 2560 x 640, top-1, 104 -> 113 us a block.)
template <int NCHUNK, bool COPY>
__global__ __launch_bounds__(256) void route_kernel(const half_t* __restrict__ x, const half_t* __restrict__ wg,
                                                     const float* __restrict__ bias, int d, int E, int k,
                                                     int32_t* __restrict__ idx, float* __restrict__ gate,
                                                     int32_t* __restrict__ idx2, float* __restrict__ gate2,
                                                     int32_t* __restrict__ status, const half_t* __restrict__ rms_gain,
                                                     float eps, half_t* __restrict__ xn) {
    __shared__ float logit[MOE_MAX_EXPERTS];
    const int t = blockIdx.x;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (t == 0 && tid == 0 && status) *status = 0;   // status word describes the call that starts here
    uint4_t xv[NCHUNK];
    gate_load_row<NCHUNK>(x + (size_t)t * d, d, lane, xv);
    const auto write_row = [&] {
        if (wave == 0) {
#pragma unroll
            for (int j = 0; j < NCHUNK; ++j) {
                const int c = (lane + 64 * j) * 8;
                if (c < d) *(uint4_t*)(xn + (size_t)t * d + c) = xv[j];
            }
        }
    };
    if (COPY) {
        write_row();
    } else if (rms_gain) {
        // chained configuration: the block input is RMSNorm(x) * gain, rounded to fp16; it is written to xn for the
        // expert kernels and used for the logits in the same pass
        gate_rmsnorm<NCHUNK>(xv, rms_gain, d, eps, lane);
        write_row();
    }
    constexpr int kAtOnce = NCHUNK <= 4 ? 4 : NCHUNK <= 8 ? 2 : 1;   // 64 registers of gate matrix rows
    for (int e = wave; e < E; e += 4 * kAtOnce) {
        float l[kAtOnce];
        gate_logits<kAtOnce, NCHUNK>(xv, wg, e, 4, E, d, lane, l);
        if (lane == 0) {
#pragma unroll
            for (int n = 0; n < kAtOnce; ++n)
                if (e + 4 * n < E) logit[e + 4 * n] = l[n] + (bias ? bias[e + 4 * n] : 0.0f);
        }
    }
    __syncthreads();
    if (wave == 0) {
        int sel[MOE_MAX_TOPK];
        float lsel[MOE_MAX_TOPK], g[MOE_MAX_TOPK];
        gate_select(logit, E, k, lane, sel, lsel);
        gate_weights(lsel, k, g);
#pragma unroll
        for (int s = 0; s < MOE_MAX_TOPK; ++s) {
            if (s < k && lane == s) {
                idx[(size_t)t * k + s] = sel[s];
                gate[(size_t)t * k + s] = g[s];
                if (idx2) idx2[(size_t)t * k + s] = sel[s];
                if (gate2) gate2[(size_t)t * k + s] = g[s];
            }
        }
    }
}

void launch_route(const half_t* x, const half_t* wg, const float* bias, int T, int d, int E, int k, int32_t* idx,
                  float* gate, int32_t* idx2, float* gate2, int32_t* status, hipStream_t st, const half_t* rms_gain,
                  float eps, half_t* xn) {
    TraceScope trace(kKernelRoute, st);
    const auto launch = [&](auto copy) {
        constexpr bool COPY = decltype(copy)::value;
        if (d <= 2048)
            route_kernel<4, COPY><<<T, 256, 0, st>>>(x, wg, bias, d, E, k, idx, gate, idx2, gate2, status, rms_gain, eps, xn);
        else if (d <= 4096)
            route_kernel<8, COPY><<<T, 256, 0, st>>>(x, wg, bias, d, E, k, idx, gate, idx2, gate2, status, rms_gain, eps, xn);
        else
            route_kernel<kGateMaxChunks, COPY><<<T, 256, 0, st>>>(x, wg, bias, d, E, k, idx, gate, idx2, gate2, status,
                                                                   rms_gain, eps, xn);
    };
    if (xn && !rms_gain) launch(std::true_type{});
    else launch(std::false_type{});
}

// One workgroup of 16 wavefronts; wavefront w owns the w-th of 16 contiguous runs of pairs and walks it 64 at a time.
// Five ballots (one per bit of the expert index) tell every lane which lanes of its 64 go to the same expert, so one
// walk counts the run's pairs per expert and a second one, from the prefix sums of those counts over (expert, run),
// gives every pair its place: the unique stable grouping.  What bounds it is the trips to memory and LDS per 64
// pairs: a wavefront per expert that walked all the pairs took 54.7 us for 4000 pairs over 32 experts, 16.1 us for
// 2000 over 8 and 9.8 us for 1024 over 8; this takes 7.2, 5.1 and 5.1 us.
constexpr int kPermuteWaves = 16;

__global__ __launch_bounds__(64 * kPermuteWaves) void permute_kernel(const int32_t* __restrict__ idx, int P, int E,
                                                                     int32_t* __restrict__ counts,
                                                                     int32_t* __restrict__ offsets,
                                                                     int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                                     int32_t* __restrict__ status) {
    __shared__ int32_t place[kPermuteWaves][MOE_MAX_EXPERTS];   // pairs of the run per expert, then the next free place
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int chunks = (P + 63) >> 6, per_wave = (chunks + kPermuteWaves - 1) / kPermuteWaves;
    const int c0 = wave * per_wave, c1 = c0 + per_wave < chunks ? c0 + per_wave : chunks;
    const unsigned long long before = (1ull << lane) - 1ull;
    if (lane < MOE_MAX_EXPERTS) place[wave][lane] = 0;
    auto load = [&](int c) {
        const int i = c * 64 + lane;
        return c < c1 && i < P ? idx[i] : -1;
    };
    // the lanes whose pair goes to the same expert as this lane's (none for an index outside [0, E))
    auto same_expert = [&](int v) {
        const bool valid = (unsigned)v < (unsigned)E;
        unsigned long long m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 5; ++b) {
            const bool bit = (v >> b) & 1;
            const unsigned long long set = __ballot(bit);
            m &= bit ? set : ~set;
        }
        return valid ? m : 0ull;
    };
    static_assert(MOE_MAX_EXPERTS == 32, "five bits");
    wave_lds_handover();
    int next = load(c0);
    for (int c = c0; c < c1; ++c) {
        const int v = next;
        next = load(c + 1);
        const unsigned long long m = same_expert(v);
        if (m && !(m & before)) place[wave][v] += __popcll(m);
        wave_lds_handover();
        const int i = c * 64 + lane;
        if (!m && i < P) {                       // belongs to no expert: flag it
            inv[i] = -1;
            atomicOr(status, kStatusBadIndex);
        }
    }
    __syncthreads();
    if (wave == 0) {
        int total = 0;
        if (lane < E)
            for (int w = 0; w < kPermuteWaves; ++w) total += place[w][lane];
        int end = total;                         // inclusive prefix sum over the experts
#pragma unroll
        for (int m = 1; m < MOE_MAX_EXPERTS; m <<= 1) {
            const int below = __shfl_up(end, m, kWave);
            if (lane >= m) end += below;
        }
        if (lane < E) {
            counts[lane] = total;
            offsets[lane] = end - total;
            if (lane == E - 1) offsets[E] = end;
            int run = end - total;
            for (int w = 0; w < kPermuteWaves; ++w) {
                const int n = place[w][lane];
                place[w][lane] = run;
                run += n;
            }
        }
    }
    __syncthreads();
    next = load(c0);
    for (int c = c0; c < c1; ++c) {
        const int v = next;
        next = load(c + 1);
        const unsigned long long m = same_expert(v);
        if (m) {
            const int i = c * 64 + lane, r = place[wave][v] + __popcll(m & before);
            perm[r] = i;
            inv[i] = r;
        }
        wave_lds_handover();
        if (m && !(m & before)) place[wave][v] += __popcll(m);
        wave_lds_handover();
    }
}

void launch_permute(const int32_t* idx, int P, int E, int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv,
                    int32_t* status, hipStream_t st) {
    TraceScope trace(kKernelPermute, st);
    permute_kernel<<<1, 64 * kPermuteWaves, 0, st>>>(idx, P, E, counts, offsets, perm, inv, status);
}

}  // namespace moemix
