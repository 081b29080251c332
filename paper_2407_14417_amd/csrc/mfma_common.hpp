// What the kernels of grouped matrix products on the matrix cores share (ffn_mfma.hip, ffn_prefill.hip): arguments,
// what a workgroup works on, addressing, products, and the expansion of 4-bit and 8-bit codes.
#pragma once

#include <atomic>

#include "common.hpp"

namespace moemix {

constexpr int kKTile = 128;                 // contraction elements per LDS tile
constexpr int kChunkRows = 256;             // most activation rows of a chunk in ffn_prefill.hip
constexpr unsigned kComputeUnits = 256;     // of the MI355X

struct MfmaArgs {
    DevExperts ex;
    const int32_t* offsets;   // [E+1] grouped rows per expert, or null in direct mode
    const int32_t* perm;      // up, grouped: grouped row -> flat pair (token = pair / top_k); null: rows in order
    const int32_t* idx;       // [P] the routing result, if the grouping is worked out from it (offsets, perm unused)
    int P;
    int top_k;
    int direct_expert, direct_n;
    const half_t* in;         // up: x [T, K]; down: h [rows, K]
    void* out;                // up: h [rows, N] fp16; down: y [splits][rows_total, N] fp32
    int K, N, E;
    int k_per_split;          // contraction elements per split (multiple of 128)
    int tiles;                // tiles of weight rows (grid.x = tiles * splits)
    size_t split_stride;      // elements of y between two splits
    int unit_bytes;           // LDS bytes per A operand for weight staging: 4096 if any expert is 16-bit, else 2048
    uint32_t prec16, prec8;   // the experts held in 16 and in 8 bits, one bit each
    int waves;                // ffn_prefill.hip: wavefronts per workgroup (prefill_waves); else 0
    int quant_rows;           // its 8-wavefront form: most rows of a chunk of a 4-bit or 8-bit expert (quant_chunk_rows)
    int32_t* status;
};

// Pointers into device (global) memory, typed as such, and a pin that keeps a uniform pointer in scalar
// registers so that "uniform base + 32-bit lane offset" compiles to the scalar-base addressing form.
#define MOEMIX_GLOBAL __attribute__((address_space(1)))
typedef const char MOEMIX_GLOBAL* gptr_t;
__device__ __forceinline__ gptr_t scalar_ptr(const void* p) {
    gptr_t g = (gptr_t)p;
    asm volatile("" : "+s"(g));
    return g;
}

__device__ __forceinline__ float4_t mfma16(half8_t a, half8_t b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// Nothing moves across this point when the compiler schedules instructions.
__device__ __forceinline__ void pin_schedule() { __builtin_amdgcn_sched_barrier(0); }

// Two neighbouring scales or zeros: rows of an odd number of them start on 2-byte boundaries.
typedef uint32_t __attribute__((aligned(2))) uint32_half_aligned_t;

// (a & mask) | bits in one instruction: the mask travels in a scalar register, the OR-ed bits in a vector one
// (the instruction may read a single scalar operand, which is why the compiler does not form it by itself).
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t mask, uint32_t bits) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(mask), "v"(bits));
    return r;
}

// A 32-bit lane offset as a value the compiler has not seen before: its widening to 64 bits then stays next to the
// load that uses it (scalar base + 32-bit lane offset in one instruction) instead of being hoisted out of the loop
// as a register pair per offset.
__device__ __forceinline__ uint32_t fresh_offset(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}
// A constant (fp16 pairs such as 1024, 1024) held in a vector register (not volatile: identical copies are merged).
__device__ __forceinline__ uint32_t vreg_const(uint32_t v) {
    uint32_t m;
    asm("v_mov_b32 %0, %1" : "=v"(m) : "s"(v));
    return m;
}

// Eight 4-bit codes of one word -> their dequantized fp16 values, in the order (0,4,1,5,2,6,3,7).
__device__ __forceinline__ half8_t expand_word(uint32_t w, half2_t s2, half2_t z2, uint32_t m1024, uint32_t m64) {
    const uint32_t w8 = w >> 8;
    // low nibbles land in the mantissa of 1024 (ulp 1), high nibbles in the mantissa of 64 (ulp 1/16, code << 4)
    const half2_t q04 = as_half2(and_or(w, 0x000F000Fu, m1024)) - as_half2(m1024);
    const half2_t q15 = as_half2(and_or(w, 0x00F000F0u, m64)) - as_half2(m64);
    const half2_t q26 = as_half2(and_or(w8, 0x000F000Fu, m1024)) - as_half2(m1024);
    const half2_t q37 = as_half2(and_or(w8, 0x00F000F0u, m64)) - as_half2(m64);
    const half2_t a = __builtin_elementwise_fma(q04, s2, z2), b = __builtin_elementwise_fma(q15, s2, z2);
    const half2_t c = __builtin_elementwise_fma(q26, s2, z2), d = __builtin_elementwise_fma(q37, s2, z2);
    return half8_t{a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}

// Eight 8-bit codes (two words) -> their dequantized fp16 values, in column order.
__device__ __forceinline__ half8_t expand_bytes(uint32_t w0, uint32_t w1, half2_t s2, half2_t z2, uint32_t m1024,
                                                uint32_t m64x4) {
    // a byte permute puts each code into the low byte of an fp16 whose high byte is 0x64: 1024 + code, exactly
    const half2_t q01 = as_half2(__builtin_amdgcn_perm(m64x4, w0, 0x04010400u)) - as_half2(m1024);
    const half2_t q23 = as_half2(__builtin_amdgcn_perm(m64x4, w0, 0x04030402u)) - as_half2(m1024);
    const half2_t q45 = as_half2(__builtin_amdgcn_perm(m64x4, w1, 0x04010400u)) - as_half2(m1024);
    const half2_t q67 = as_half2(__builtin_amdgcn_perm(m64x4, w1, 0x04030402u)) - as_half2(m1024);
    const half2_t a = __builtin_elementwise_fma(q01, s2, z2), b = __builtin_elementwise_fma(q23, s2, z2);
    const half2_t c = __builtin_elementwise_fma(q45, s2, z2), d = __builtin_elementwise_fma(q67, s2, z2);
    return half8_t{a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}

// What one workgroup works on, set up once by the kernel and handed to the precision-specific body.
struct TileCtx {
    const half_t* in;        // activations
    const int32_t* perm;     // up, grouped: grouped row -> flat pair; else null
    const uint16_t* tokens;  // up, grouping worked out by the workgroup: the chunk's rows -> tokens (LDS); else null
    int top_k;
    int K, N;
    int begin, m0, rows;     // grouped rows [begin + m0, begin + m0 + rows)
    int n0;                  // first weight row of the workgroup
    int k_begin, n_steps;    // contraction range [k_begin, k_begin + 128 n_steps), up to the end of the rows
    bool tail;               // the last step holds 64 columns: the range ends with rows of an odd multiple of 64
    int rot;                 // the workgroup walks the range from step rot on, wrapping around (a multiple of 4; see below)
    int mc;                  // rows per LDS buffer (16 * ct of the launch)
    int unit_bytes;          // LDS bytes per A operand of the weight staging regions (2048: 4-bit only, 4096)
    uint8_t* lds;
    uint32_t lds_base;       // the same as an LDS byte address
    int team, team_bytes, barriers;   // grouped_mfma_kernel with several teams: which one, LDS of each, barriers of the longest part
};

// Grid: x = tile of weight rows + tiles * contraction split, y = chunk: workgroups are handed out chunk by chunk.
// Workgroups go to the 8 XCDs (each with an L2 of its own) in turn, in launch order: with 2, 4 or 8 contraction
// splits those of one chunk and split, which read the same slice of the activations, get the indices that
// land on the same 4, 2 or 1 XCDs.
__device__ __forceinline__ void place_workgroup(int tiles, int& tile_x, int& split_z) {
    const int sp = gridDim.x / tiles, i = blockIdx.x, xcd = i & 7, slot = i >> 3;
    if (sp > 1 && (tiles * sp) % 8 == 0 && 8 % sp == 0) {
        const int q = 8 / sp;                              // XCDs per split
        split_z = xcd / q; tile_x = slot * q + xcd % q;
    } else {
        tile_x = i % tiles; split_z = i / tiles;
    }
}

// The workgroup's expert cannot run: its rows contribute nothing, and the status word says so.
template <bool UP>
__device__ __forceinline__ void leave_out(const TileCtx& c, void* out_base, int32_t* status, int tile_x, int n_rows, int threads) {
    if (threadIdx.x == 0 && tile_x == 0) atomicOr(status, kStatusNotResident);
    if (!UP) {
        float* y = (float*)out_base;
        for (int i = threadIdx.x; i < c.rows * n_rows; i += threads) {
            const int rr = i / n_rows, cc = c.n0 + i % n_rows;
            if (cc < c.N) y[(size_t)(c.begin + c.m0 + rr) * c.N + cc] = 0.0f;
        }
    }
}

// Lets a kernel be launched with up to `bytes` of LDS.  The attribute belongs to (kernel, device): it is set once per device of
// the process (bit d of `configured`, one per kernel; devices past the 64th set it on every launch).
inline void allow_lds(const void* kernel, size_t bytes, std::atomic<unsigned long long>& configured) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const unsigned long long bit = dev < 64 ? 1ull << dev : 0ull;
    if (!(configured.load(std::memory_order_relaxed) & bit) || !bit) {
        (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        configured.fetch_or(bit, std::memory_order_relaxed);
    }
}

// Launches with a.waves != 0 (ffn_prefill.hip).
template <bool UP>
void launch_prefill(const MfmaArgs& a, dim3 grid, hipStream_t st);

}  // namespace moemix
