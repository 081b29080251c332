// The 4-bit weight format on the device: dequantizer (check hook, 4-bit -> 16-bit switch),
// quantizer (16-bit -> 4-bit switch when the expert table is re-planned, paper §3), and the seeded
// synthetic-tensor fill.
#include "common.hpp"
#include "kernels.hpp"

namespace moemix {

// One thread per 8 weights (one 32-bit word of codes).
__global__ __launch_bounds__(256) void dequant_int4_kernel(DevMat m, size_t n_words, int in, half_t* __restrict__ w) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_words) return;
    const size_t col0 = (i * 8) % (size_t)in, row = (i * 8) / (size_t)in;
    const size_t g = row * (size_t)(in >> 6) + (col0 >> 6);
    const float s = (float)m.scale[g], z = (float)m.zero[g];
    const uint32_t word = ((const uint32_t*)m.data)[i];
    half8_t o;
#pragma unroll
    for (int n = 0; n < 8; ++n) o[n] = dequant_one((word >> (4 * n)) & 0xFu, s, z);
    *(half8_t*)(w + i * 8) = o;
}

void launch_dequant_int4(const DevMat& m, int out, int in, half_t* w, hipStream_t st) {
    const size_t n_words = (size_t)out * in / 8;
    if (n_words == 0) return;
    dequant_int4_kernel<<<(unsigned)((n_words + 255) / 256), 256, 0, st>>>(m, n_words, in, w);
}

// One wavefront per group of 64 weights: lane = column.  Min and max by shuffles, every fp32 step
// rounded on its own (division is the correctly rounded one), codes packed by lane pairs.  For arrays that are not
// aligned for the vector accesses of quantize_kernel below; one code per byte (BITS 8) or two (BITS 4).
template <int BITS>
__global__ __launch_bounds__(256) void quantize_unaligned_kernel(const half_t* __restrict__ w, size_t n_groups,
                                                                  uint8_t* __restrict__ codes, half_t* __restrict__ scale,
                                                                  half_t* __restrict__ zero) {
    constexpr float kTop = (float)((1 << BITS) - 1);
    const size_t g = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= n_groups) return;
    const int lane = threadIdx.x & 63;
    const float v = (float)w[g * 64 + lane];
    float mn = v, mx = v;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, m, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, m, kWave));
    }
    const float range = __fsub_rn(mx, mn);
    const half_t s16 = f32_to_f16_rne(__fdiv_rn(range, kTop));
    const float s = (float)s16;
    uint32_t q = 0;
    if (s != 0.0f) {
        float r = rintf(__fdiv_rn(__fsub_rn(v, mn), s));
        r = fminf(fmaxf(r, 0.0f), kTop);
        q = (uint32_t)r;
    }
    if (BITS == 4) {
        const uint32_t hi = __shfl_down(q, 1, kWave);
        if ((lane & 1) == 0) codes[g * 32 + (lane >> 1)] = (uint8_t)(q | (hi << 4));
    } else {
        codes[g * 64 + lane] = (uint8_t)q;
    }
    if (lane == 0) {
        scale[g] = s16;
        zero[g] = (half_t)mn;
    }
}

// The same quantizer at the rate of device memory.  A lane holds 8 consecutive weights (one 128-bit load), a group of
// 64 is 8 lanes: min and max take 7 + 7 steps inside the lane and three on the DPP network, where the kernel above
// spends six shuffles each per 64 weights and loads and stores 2 and 1 bytes per lane.  Every lane asks for
// kQuantItems pieces before it uses the first.
// The definition's code is rint(RN((v - min) / s)).  The correctly rounded division costs a dozen instructions per
// weight, so a product with the approximate reciprocal of s stands in for it where it cannot matter: that product is
// off by at most 383 * 2^-21.6 = 1.2e-4 (1 ulp of the reciprocal, half an ulp each of the product and of the
// quotient; quotients reach 255 * 1.5 where a subnormal s was rounded down), so its nearest integer is the quotient's
// unless it lies within 2e-4 of half way between two integers, and there the division is done.
// 14336 x 4096 to 4 bits: 169 us -> 30 us (117 MB read, 34 MB written: 5.0 TB/s, the rate of a large copy).
constexpr int kQuantItems = 4;

template <int BITS>
__global__ __launch_bounds__(256) void quantize_kernel(const half_t* __restrict__ w, size_t n, uint8_t* __restrict__ codes,
                                                        half_t* __restrict__ scale, half_t* __restrict__ zero) {
    constexpr float kTop = (float)((1 << BITS) - 1);
    const size_t first = (size_t)blockIdx.x * (256 * 8 * kQuantItems) + (size_t)threadIdx.x * 8;
    half8_t in[kQuantItems];
#pragma unroll
    for (int i = 0; i < kQuantItems; ++i) {
        const size_t at = first + (size_t)i * (256 * 8);
        if (at < n) in[i] = __builtin_bit_cast(half8_t, __builtin_nontemporal_load((const uint4_t*)(w + at)));
    }
#pragma unroll
    for (int i = 0; i < kQuantItems; ++i) {
        const size_t at = first + (size_t)i * (256 * 8);
        if (at >= n) return;                            // (n is a multiple of 64: the 8 lanes of a group agree)
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (float)in[i][j];
        float mn = fminf(fminf(fminf(v[0], v[1]), fminf(v[2], v[3])), fminf(fminf(v[4], v[5]), fminf(v[6], v[7])));
        float mx = fmaxf(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7])));
        mn = fminf(mn, dpp_move<0xB1>(mn));             // lanes 1 apart,
        mx = fmaxf(mx, dpp_move<0xB1>(mx));
        mn = fminf(mn, dpp_move<0x4E>(mn));             // 2 apart,
        mx = fmaxf(mx, dpp_move<0x4E>(mx));
        mn = fminf(mn, dpp_move<0x141>(mn));            // and the other four of the eight
        mx = fmaxf(mx, dpp_move<0x141>(mx));
        const half_t s16 = f32_to_f16_rne(__fdiv_rn(__fsub_rn(mx, mn), kTop));
        const float s = (float)s16, inv = __builtin_amdgcn_rcpf(s);
        uint32_t q[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float a = __fsub_rn(v[j], mn);
            const float t = a * inv;
            float r = rintf(t);
            if (fabsf(t - r) > 0.4998f) r = rintf(__fdiv_rn(a, s));
            r = fminf(fmaxf(r, 0.0f), kTop);
            q[j] = s != 0.0f ? (uint32_t)r : 0u;
        }
        if (BITS == 4) {
            uint32_t word = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) word |= q[j] << (4 * j);
            __builtin_nontemporal_store(word, (uint32_t*)(codes + at / 2));
        } else {
            const uint2_t words = {q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24),
                                   q[4] | (q[5] << 8) | (q[6] << 16) | (q[7] << 24)};
            __builtin_nontemporal_store(words, (uint2_t*)(codes + at));
        }
        if ((threadIdx.x & 7) == 0) {
            scale[at / 64] = s16;
            zero[at / 64] = (half_t)mn;
        }
    }
}

template <int BITS>
static void launch_quantize(const half_t* w, int out, int in, uint8_t* codes, half_t* scale, half_t* zero, hipStream_t st) {
    const size_t n = (size_t)out * in;
    if (n == 0) return;
    if ((uintptr_t)w % 16 || (uintptr_t)codes % BITS) {     // (BITS bytes of codes per lane and store)
        quantize_unaligned_kernel<BITS><<<(unsigned)((n / 64 + 3) / 4), 256, 0, st>>>(w, n / 64, codes, scale, zero);
        return;
    }
    constexpr size_t per_block = 256 * 8 * kQuantItems;
    quantize_kernel<BITS><<<(unsigned)((n + per_block - 1) / per_block), 256, 0, st>>>(w, n, codes, scale, zero);
}

void launch_quantize_int4(const half_t* w, int out, int in, uint8_t* packed, half_t* scale, half_t* zero,
                          hipStream_t st) {
    launch_quantize<4>(w, out, in, packed, scale, zero, st);
}

void launch_quantize_int8(const half_t* w, int out, int in, uint8_t* codes, half_t* scale, half_t* zero, hipStream_t st) {
    launch_quantize<8>(w, out, in, codes, scale, zero, st);
}

// 8-bit form: one thread per 4 weights (one 32-bit word of codes).
__global__ __launch_bounds__(256) void dequant_int8_kernel(DevMat m, size_t n_words, int in, half_t* __restrict__ w) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_words) return;
    const size_t col0 = (i * 4) % (size_t)in, row = (i * 4) / (size_t)in;
    const size_t g = row * (size_t)(in >> 6) + (col0 >> 6);
    const float s = (float)m.scale[g], z = (float)m.zero[g];
    const uint32_t word = ((const uint32_t*)m.data)[i];
    half4_t o;
#pragma unroll
    for (int n = 0; n < 4; ++n) o[n] = dequant_one((word >> (8 * n)) & 0xFFu, s, z);
    *(half4_t*)(w + i * 4) = o;
}

void launch_dequant_int8(const DevMat& m, int out, int in, half_t* w, hipStream_t st) {
    const size_t n_words = (size_t)out * in / 4;
    if (n_words == 0) return;
    dequant_int8_kernel<<<(unsigned)((n_words + 255) / 256), 256, 0, st>>>(m, n_words, in, w);
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Element i = pure function of (key, first + i); see the generator module for the recipe.
__global__ __launch_bounds__(256) void synth_fill_kernel(half_t* __restrict__ dst, size_t n, size_t first, uint64_t key,
                                                          float scale, int kind) {
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t j = (size_t)blockIdx.x * 256 + threadIdx.x; j < n; j += stride) {
        const uint64_t i = (uint64_t)first + j;
        const uint64_t h0 = mix64(key + 2 * i);
        int32_t c;
        if (kind == 0) {
            const uint64_t h1 = mix64(key + 2 * i + 1);
            uint32_t s = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                s += (uint32_t)((h0 >> (16 * b)) & 0xFFFFu);
                s += (uint32_t)((h1 >> (16 * b)) & 0xFFFFu);
            }
            c = 2 * (int32_t)s - 8 * 65535;
        } else {
            c = 2 * (int32_t)(h0 >> 40) - ((1 << 24) - 1);
        }
        dst[j] = f32_to_f16_rne(__fmul_rn((float)c, scale));
    }
}

void launch_synth_fill(half_t* dst, size_t n, size_t first, uint64_t seed, uint64_t stream_id, float scale, int kind,
                       hipStream_t st) {
    if (n == 0) return;
    // host-side key derivation (same two mixing steps as on the device)
    auto hmix = [](uint64_t z) {
        z += 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    const uint64_t key = hmix(hmix(seed) + stream_id);
    const size_t blocks = (n + 255) / 256;
    synth_fill_kernel<<<(unsigned)(blocks < 65536 ? blocks : 65536), 256, 0, st>>>(dst, n, first, key, scale, kind);
}

}  // namespace moemix
