// Expert feed-forward layers on many rows (prefill; prefill_waves in ffn_mfma.hip says which launches): the grouped products
// of ffn_mfma.hip with device memory brought straight into LDS.
//
// One workgroup = 8 wavefronts = one (expert, tile of 128 rows of w1 and w3 or 256 of w2, chunk of up to 256 activation rows,
// contraction split), one workgroup per compute unit; or 4 wavefronts, half the weight rows, half of LDS, chunks of up to 128
// rows, two per compute unit.  Two wavefronts per SIMD either way.  A wavefront multiplies 32 weight rows (two A operands of
// v_mfma_f32_16x16x32_f16) with all rows of the chunk.  The contraction goes in stages of 64 columns = one quantization group =
// two sub-steps of 32.  What a stage needs lies in LDS rings filled by global-to-LDS transfers, several stages ahead and
// without registers: activations [rows][128 bytes], brought by all wavefronts together; weights as they are stored, scales and
// zeros, brought by each wavefront for itself.  One meeting of the wavefronts per stage, before its last unit of products.
//
// Why this shape.  One wavefront per SIMD with weights in registers, which this replaces, added up what it did: products, the
// expansion of the codes and waiting.  Measured here: a product occupies the SIMD's issue for 8 of its 16 cycles, so two
// vector instructions per product are free and every further one costs 4 cycles, whichever wavefront it comes from; LDS
// delivers 256 bytes per cycle to conflict-free 16-byte reads, so reading each B operand for two products only is no burden,
// while the expansion is done once per weight.  What bounds the launches now: the clock, which falls to 1.8 - 2.0 GHz of 2.4 in
// those of many rows (the same launches with weights of zero keep 2.3 - 2.4 and take 0.76 - 0.89 of the time, few and short
// ones 0.95 - 1), and instructions and waiting beside the products: matrix cores busy 0.41 (512 tokens, Mixtral shape, skewed,
// up-projection) and 0.49 (1000 tokens, 8-bit) of the cycles, wavefronts at a wait 0.32 and 0.41 of theirs, LDS busy 0.28.
// Blocks, before and after (both libraries in turn): 1000 tokens, 8 experts of 4096 x 14336, all 8-bit 842 -> 797 us; 500
// tokens, 32 experts of 2048 x 1408, half 16-bit 192 -> 160; 80 tokens on every expert, 16-bit 638 -> 568; 600 tokens,
// 2816 x 2816, 16-bit 173 -> 131; 256 tokens on every expert, 4-bit 741 -> 670.
#include <algorithm>
#include <atomic>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.hpp"
#include "mfma_common.hpp"

namespace moemix {

namespace {

constexpr int kLdsBytes = 163840;                          // of a compute unit

// ---- device memory straight into LDS

// 16 bytes per lane from p + v + OFFSET, lane l's to LDS byte lds + OFFSET + 16 l (the instruction's offset counts on both
// sides; kBack makes up for it).  M0 is an operand of its own, so that the compiler knows what it holds; the wait state is the one
// that a write of M0 asks for.  (A base from a lane read would ask for five: 1 % of a launch as s_nop 4; there is none, which a test
// of the built code checks.)
template <int OFFSET>
__device__ __forceinline__ void bring(uint32_t lds, gptr_t p, uint32_t v) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"{m0}"(lds), "v"(v), "s"(p), "n"(OFFSET) : "memory");
}
constexpr int kBack = 4096;   // base pointers point this far back, lane offsets are that much larger less OFFSET
// 4 bytes per lane, lane l's to LDS byte lds + 4 l
__device__ __forceinline__ void bring_words(uint32_t lds, gptr_t p, uint32_t v) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %1, %2" ::"{m0}"(lds), "v"(v), "s"(p) : "memory");
}
// At most COUNT of the wavefront's own transfers are under way, its LDS accesses are done; then all wavefronts meet.
template <int COUNT>
__device__ __forceinline__ void wait_and_meet() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(COUNT) : "memory");
}

// slot of 16-byte piece p of row r in rows of 128 and of 64 bytes is p ^ swizzle(r)
__device__ __forceinline__ int swizzle128(int r) {
    const int h = (r >> 1) & 7;
    return (h & 4) | ((h & 1) << 1) | (((h >> 1) ^ (h >> 2)) & 1);
}
__device__ __forceinline__ int swizzle64(int r) {
    const int q = (r >> 2) & 3;
    return (((q >> 1) ^ q) & 1) << 1 | (q >> 1);
}

// f(0), f(1), .. with the index as a type
template <class F, int... I>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f) {
    (f(std::integral_constant<int, I>{}), ...);
}

constexpr int min_of(int a, int b) { return a < b ? a : b; }

// LDS rings of a chunk of N tiles: stages of activations, slabs of weights (4-bit: of two stages), in KB
template <int WAVES, int PREC, int N>
struct Rings {
    static constexpr int kScales = PREC == MOE_PREC_FP16 ? 0 : 2 * WAVES, kRoom = kLdsBytes / 1024 * WAVES / 8 - kScales;
    static constexpr int kX = 2 * N, kSlab = PREC == MOE_PREC_FP16 ? 4 * WAVES : 2 * WAVES;
    static constexpr int slabs(int d) { return PREC == MOE_PREC_INT4G64 ? (d + 4) / 2 : d; }
    static constexpr bool fits(int d) { return d * kX + slabs(d) * kSlab <= kRoom; }
    // As deep as LDS allows up to six stages; 4-bit four, whose stages need fewer bytes than the rings take to fill (80 tokens
    // on every expert, Mixtral shape, 4-bit with up to six, four and three 357, 351, 369 us; 8-bit 416, 425, 426).
    static constexpr int kMost = PREC == MOE_PREC_INT4G64 ? 4 : 6;
    static constexpr int kDepth = kMost == 6 && fits(6) ? 6 : kMost == 6 && fits(5) ? 5 : fits(4) ? 4 : 3;
    static constexpr int kStages = fits(kDepth) ? kDepth : 2;         // (16-bit, more than 10 tiles: two stages, three slabs)
    static constexpr int kSlabs = slabs(kDepth);
    static_assert(kStages * kX + kSlabs * kSlab <= kRoom, "LDS");
};

// One workgroup's chunk of N tiles of 16 rows.  Rings: stage i's activations in slot i mod XR, weights of slab u in slot
// u mod R (a slab is a stage's weights, for 4-bit ones two stages').  What stage i asks for overwrites what stage i - 1 read
// last (its reads are done when the wavefronts have met in stage i - 1) and is there when they meet XR - 2 stages later.
template <int WAVES, bool UP, int PREC, int N>
__device__ __forceinline__ void chunk_body(const TileCtx& c, const DevExpert& ee, void* out_base) {
    constexpr bool INT4 = PREC == MOE_PREC_INT4G64, INT8 = PREC == MOE_PREC_INT8G64, QUANT = INT4 || INT8;
    typedef Rings<WAVES, PREC, N> L;
    constexpr int XR = L::kStages, R = L::kSlabs, XSTAGE = L::kX * 1024, SLAB = L::kSlab * 1024, WSLAB = SLAB / WAVES;
    constexpr int kSlabs = XR * XSTAGE, kScales = kSlabs + R * SLAB;
    constexpr int NX = (2 * N + WAVES - 1) / WAVES, XREM = 2 * N % WAVES;  // 1 KB runs of a stage's activations per wavefront; the first
                                                           // XREM wavefronts (0: all) have the last one
    constexpr int SPW = QUANT ? 2 : 4;                     // ... of a slab's weights
    constexpr int NS = INT4 ? 1 : SPW;                     // ... per stage
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, c4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = c.K, Nw = c.N, n_steps = c.n_steps, nb = 2 * n_steps;
    const bool more_x = !XREM || wave < XREM;
    const uint32_t lds0 = c.lds_base;

    // ---- the tokens of the rows it brings.  (Asked for and turned into offsets before anything else is on its way: transfers end
    // in order, so tokens that are asked for behind weights come when those have come, 2 to 3 us later.)
    const int run0 = XREM ? wave * (NX - 1) + (wave < XREM ? wave : XREM) : wave * NX;
    uint32_t xv[NX];
    {
        const uint32_t rcp = UP && c.perm && c.top_k > 1 ? 0xFFFFFFFFu / (uint32_t)c.top_k + 1 : 0;   // (pairs: less than 2^24)
        uint32_t pair[NX];
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int row = (run0 + k) * 8 + (lane >> 3);
            const int g = c.begin + c.m0 + (row < c.rows ? row : c.rows - 1);
            pair[k] = UP && c.perm ? (uint32_t)c.perm[g] : (uint32_t)g;
        }
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const uint32_t src = rcp ? __umulhi(pair[k], rcp) : pair[k];
            xv[k] = src * (uint32_t)K * 2 + (((lane & 7) ^ swizzle128(((run0 + k) * 8 + (lane >> 3)) & 15)) * 16) + (kBack - 1024 * k);
        }
        pin_schedule();
    }

    // ---- weights, scales and zeros: every wavefront brings its own
    const int row0 = c.n0 + wave * (UP ? 16 : 32);
    gptr_t wb[2], sb[2], zb[2];
    uint32_t wv[SPW], sv[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const DevMat& m = UP ? (t ? ee.w3 : ee.w1) : ee.w2;
        wb[t] = scalar_ptr(m.data + (INT4 ? c.k_begin >> 1 : INT8 ? c.k_begin : c.k_begin * 2) - kBack);
        sb[t] = QUANT ? scalar_ptr(m.scale + (c.k_begin >> 6)) : nullptr;
        zb[t] = QUANT ? scalar_ptr(m.zero + (c.k_begin >> 6)) : nullptr;
        int row = row0 + (UP ? 0 : 16 * t) + r16;
        row = row < Nw ? row : Nw - 1;                     // rows past the end repeat the last row, never stored
        sv[t] = (uint32_t)row * (uint32_t)(K >> 6) * 2;
    }
#pragma unroll
    for (int k = 0; k < SPW; ++k) {
        const int t = QUANT ? k : k >> 1, r = QUANT ? lane >> 2 : 8 * (k & 1) + (lane >> 3);
        int row = row0 + (UP ? 0 : 16 * t) + r;
        row = row < Nw ? row : Nw - 1;
        wv[k] = (uint32_t)row * (uint32_t)(INT4 ? K >> 1 : INT8 ? K : 2 * K) +
                (QUANT ? ((lane & 3) ^ swizzle64(r)) * 16 : ((lane & 7) ^ swizzle128(r)) * 16) + (kBack - 1024 * k);
    }
    constexpr int kUnit = INT4 || INT8 ? 64 : 128;         // bytes of a row per slab
    const uint32_t w_end = n_steps * (INT4 ? 64 : INT8 ? 128 : 256);
    uint32_t w_at = c.rot * (INT4 ? 64 : INT8 ? 128 : 256), w_dst = lds0 + kSlabs + wave * WSLAB;
    auto bring_w = [&](auto kc) {                          // run k of the next slab
        constexpr int k = decltype(kc)::value;
        bring<1024 * k>(w_dst, wb[QUANT ? k : k >> 1] + w_at, wv[k]);
        if (k == SPW - 1) {
            w_at += kUnit;
            if (w_at == w_end) w_at = 0;
            w_dst += SLAB;
            if (w_dst == lds0 + kSlabs + R * SLAB + wave * WSLAB) w_dst -= R * SLAB;
        }
    };
    // scales and zeros of four steps: [operand][scale, zero][step][16 rows]
    auto bring_scales = [&](int q) {
        int s = 4 * q + c4;
        s = s < n_steps ? s : n_steps - 1;
        s = s + c.rot < n_steps ? s + c.rot : s + c.rot - n_steps;
        const uint32_t d = lds0 + kScales + (q & 1) * (1024 * WAVES) + wave * 1024;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            bring_words(d + t * 512, sb[t], sv[t] + s * 4);
            bring_words(d + t * 512 + 256, zb[t], sv[t] + s * 4);
        }
    };

    // ---- activations: an equal share each
    const gptr_t xb0 = scalar_ptr(c.in + c.k_begin - kBack / 2);
    const uint32_t x_end = n_steps * 256;
    uint32_t x_at = c.rot * 256, x_dst = lds0 + run0 * 1024;
    auto bring_x = [&](auto kc) {                          // run k of the next stage
        constexpr int k = decltype(kc)::value;
        if (k < NX - 1 || more_x) bring<1024 * k>(x_dst, xb0 + x_at, xv[k]);
        if (k == NX - 1) {
            x_at += 128;
            if (x_at == x_end) x_at = 0;
            x_dst += XSTAGE;
            if (x_dst == lds0 + XR * XSTAGE + run0 * 1024) x_dst -= XR * XSTAGE;
        }
    };
    // what stage i (a time before the first one too) asks for: activations of stage i + XR - 1, then weights of stage
    // i + R (4-bit: operand i & 1 of slab i / 2 + R - 1)
    auto asks_x = [&](int i) { return i + XR - 1 < nb; };
    auto asks_w = [&](int i) { return INT4 ? (i >> 1) + R - 1 < n_steps : i + R < nb; };
    auto ask = [&](auto oc, bool x, bool w, auto par_c) {
        constexpr int o = decltype(oc)::value, par = decltype(par_c)::value;
        if constexpr (o < NX) {
            if (x) bring_x(std::integral_constant<int, o>{});
        } else {
            if (w) bring_w(std::integral_constant<int, INT4 ? par : o - NX>{});
        }
    };
    // transfers that may be under way when the next stage's activations and the weights of the one after it have to be there
    constexpr int kSlabLead = INT4 ? 2 * R - 5 : R - 2;
    constexpr int kOpen = min_of((XR - 2) * (NX + NS) + NS, kSlabLead * (NX + NS));
    constexpr int kOpenLess = min_of((XR - 2) * (NX - 1 + NS) + NS, kSlabLead * (NX - 1 + NS));
    auto wait_stage = [&](bool steady) {
        if (!steady) wait_and_meet<0>();
        else if (more_x) wait_and_meet<kOpen>();
        else wait_and_meet<kOpenLess>();
    };

    // ---- what it reads
    uint32_t b_off[2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) b_off[sub] = r16 * 128 + (((2 * c4 + sub) ^ swizzle128(r16)) * 16);
    constexpr int W = INT4 ? 2 : INT8 ? 4 : 8;             // words of an operand per stage
    uint32_t a_off[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        a_off[q] = kSlabs + wave * WSLAB;
        if (INT4) a_off[q] += r16 * 64 + (((2 * q + (c4 >> 1)) ^ swizzle64(r16)) * 16) + (c4 & 1) * 8;
        else if (INT8) a_off[q] += r16 * 64 + ((c4 ^ swizzle64(r16)) * 16);
        else a_off[q] += b_off[q];
    }
    const uint32_t s_off = kScales + wave * 1024 + r16 * 4;
    auto read_raw = [&](uint32_t (&raw)[2][W], uint32_t slot, int par) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (INT4) {
                const uint2_t v = *(const uint2_t*)(c.lds + a_off[par] + slot + t * 1024);
                raw[t][0] = v[0]; raw[t][1] = v[1];
            } else if (INT8) {
                const uint4_t v = *(const uint4_t*)(c.lds + a_off[0] + slot + t * 1024);
#pragma unroll
                for (int i = 0; i < 4; ++i) raw[t][i] = v[i];
            } else {
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) {
                    const uint4_t v = *(const uint4_t*)(c.lds + a_off[sub] + slot + t * 2048);
#pragma unroll
                    for (int i = 0; i < 4; ++i) raw[t][4 * sub + i] = v[i];
                }
            }
        }
    };
    auto read_sz = [&](uint32_t (&sz)[2][2], int step) {   // the two groups of a step: scales, zeros
        const uint32_t at = s_off + ((step >> 2) & 1) * (1024 * WAVES) + (step & 3) * 64;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int a = 0; a < 2; ++a) sz[t][a] = *(const uint32_t*)(c.lds + at + t * 512 + a * 256);
    };
    // 8-bit: 1024 with the code in the mantissa, both halves; 4-bit: 1024 with an even column's code (ulp 1), 64 with an odd
    // one's, which comes four bits up (ulp 1/16)
    const uint32_t magic = vreg_const(INT4 ? 0x54006400u : 0x64006400u), m64x4 = vreg_const(0x64646464u);
    // The expansion of a sub-step's two operands as NOPS single instructions, stage by stage over its eight pairs of columns
    constexpr int NOPS = INT4 ? 32 : INT8 ? 24 : 8;
    auto expand_op = [&](int k, uint32_t (&dst)[2][4], const uint32_t (&raw)[2][W], const uint32_t (&sz)[2][2], int sub, int par) {
        const int t = (k >> 2) & 1, q = k & 3, op = k >> 3;
        uint32_t& d = dst[t][q];
        if (!QUANT) { d = raw[t][(4 * sub + q) % W]; return; }
        if (op == 0) {
            if (INT4) d = __builtin_amdgcn_perm(0u, raw[t][sub % W], 0x0C000C00u + 0x00010001u * q);   // byte q in both halves
            else d = __builtin_amdgcn_perm(m64x4, raw[t][(2 * sub + (q >> 1)) % W], (q & 1) ? 0x04030402u : 0x04010400u);
        } else if (INT4 && op == 1) {
            d = and_or(d, 0x00F0000Fu, magic);
        } else if (op == (INT4 ? 2 : 1)) {
            d = __builtin_bit_cast(uint32_t, as_half2(d) - as_half2(magic));
        } else {
            const half2_t sw = as_half2(sz[t][0]), zw = as_half2(sz[t][1]);
            d = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(as_half2(d), half2_t{sw[par], sw[par]}, half2_t{zw[par], zw[par]}));
        }
    };

    float4_t acc[2][N];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < N; ++j) acc[t][j] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- first transfers, in the order of the stages that would have asked for them
    constexpr int kAhead = INT4 ? 2 * R - 2 : R;           // stages before the first one that ask for something
    if (QUANT) bring_scales(0);
    unrolled(std::make_integer_sequence<int, kAhead>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value - kAhead;    // stage
        const bool x = i >= -(XR - 1) && asks_x(i), w = asks_w(i);
        unrolled(std::make_integer_sequence<int, NX + NS>{}, [&](auto oc) { ask(oc, x, w, std::integral_constant<int, (i & 1)>{}); });
    });
    const int steady_end = INT4 ? min(nb - XR + 1, 2 * (n_steps - R + 1)) : min(nb - XR + 1, nb - R);   // stages that ask for both
    wait_stage(steady_end > 0);
    uint32_t raw[2][2][W], af[2][2][4], sz[2][2], szn[2][2];
    read_raw(raw[0], 0, 0);
    if (QUANT) read_sz(sz, 0);
#pragma unroll
    for (int k = 0; k < NOPS; ++k) expand_op(k, af[0], raw[0], sz, 0, 0);
    constexpr int UPS = (N + 3) / 4, NU = 2 * UPS, UB = (N + UPS - 1) / UPS;   // units per sub-step and stage; tiles per unit at most
    auto first_tile = [](int u) { return u * N / UPS; };
    half8_t bq[2][UB];
#pragma unroll
    for (int j = 0; j < UB; ++j)
        if (j < first_tile(1)) bq[0][j] = *(const half8_t*)(c.lds + b_off[0] + j * 2048);
    pin_schedule();

    uint32_t xslot = 0;                                    // of this stage
    uint32_t rslot = INT4 ? 0 : SLAB;                      // 8-bit, 16-bit: of the next stage's slab; 4-bit: of this step's
    auto stage = [&](auto par_c, int s) {
        constexpr int par = decltype(par_c)::value;
        const int i = 2 * s + par;
        uint32_t xnext = xslot + XSTAGE, rnext = rslot + SLAB;
        if (xnext == XR * XSTAGE) xnext = 0;
        if (rnext == R * SLAB) rnext = 0;
        // (past the end: whatever lies there, never used)
        read_raw(raw[par ^ 1], INT4 && par ? rnext : rslot, par ^ 1);
        if (QUANT && par) read_sz(szn, s + 1);
        const uint8_t* const xb = c.lds + xslot;
        const uint8_t* const xn = c.lds + xnext;
        const bool steady = i < steady_end;
        const bool x = steady || asks_x(i), w = steady || asks_w(i);
        unrolled(std::make_integer_sequence<int, NU>{}, [&](auto kc) {
            constexpr int k = decltype(kc)::value;
            constexpr int sub = k / UPS, u = k % UPS;
            if constexpr (k == NU - 1) {
                wait_stage(steady);
                pin_schedule();
            }
            // Of the two wavefronts of a SIMD the one further behind goes first: left to themselves the older one does, waits
            // for the younger at every meeting, and each alone cannot keep the matrix cores busy.
            if constexpr (WAVES == 8 && (k == 0 || 4 * k / NU != 4 * (k - 1) / NU)) __builtin_amdgcn_s_setprio(3 - 4 * k / NU);
            // next unit's operands
            constexpr int nk = (k + 1) % NU, nsub = nk / UPS, nu = nk % UPS;
            const uint8_t* const nbase = (k + 1 < NU ? xb : xn) + b_off[nsub] + first_tile(nu) * 2048;
#pragma unroll
            for (int j = 0; j < UB; ++j)
                if (first_tile(nu) + j < first_tile(nu + 1)) bq[(k + 1) & 1][j] = *(const half8_t*)(nbase + j * 2048);
            pin_schedule();
#pragma unroll
            for (int j = 0; j < UB; ++j) {
                const int tile = first_tile(u) + j;
                if (tile < first_tile(u + 1)) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[t][tile] = mfma16(__builtin_bit_cast(half8_t, uint4_t{af[sub][t][0], af[sub][t][1], af[sub][t][2], af[sub][t][3]}),
                                              bq[k & 1][j], acc[t][tile]);
                    // the other sub-step's operands, spread over the tiles
#pragma unroll
                    for (int o = (tile * NOPS + N - 1) / N; o < ((tile + 1) * NOPS + N - 1) / N; ++o) {
                        if (sub == 0) expand_op(o, af[1], raw[par], sz, 1, par);
                        else expand_op(o, af[0], raw[par ^ 1], par ? szn : sz, 0, par ^ 1);
                    }
                    pin_schedule();
                }
            }
            // transfers, spread over the units before the last
            if constexpr (k < NU - 1) {
                constexpr int OPS = NX + NS, lo = k * OPS / (NU - 1), hi_ = (k + 1) * OPS / (NU - 1);
                unrolled(std::make_integer_sequence<int, hi_ - lo>{}, [&](auto oc) {
                    ask(std::integral_constant<int, lo + decltype(oc)::value>{}, x, w, par_c);
                });
                if constexpr (QUANT && !par && k == NU - 2)
                    if ((s & 3) == 0 && s + 4 < n_steps) bring_scales((s >> 2) + 1);
                pin_schedule();
            }
        });
        if (QUANT && par) {
#pragma unroll
            for (int t = 0; t < 2; ++t) { sz[t][0] = szn[t][0]; sz[t][1] = szn[t][1]; }
        }
        xslot = xnext;
        if (!INT4 || par) rslot = rnext;
    };
    for (int s = 0; s < n_steps; ++s) {
        stage(std::integral_constant<int, 0>{}, s);
        stage(std::integral_constant<int, 1>{}, s);
    }

    // ---- results: lane (r16, c4) holds, for activation row 16 j + r16, weight rows 4 c4 + (0..3) of each operand
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int rr = 16 * j + r16;
        if (rr < c.rows) {
            const size_t g = (size_t)(c.begin + c.m0 + rr);
            if (UP) {
                const int col = row0 + c4 * 4;
                if (col < Nw) {
                    half4_t o;
#pragma unroll
                    for (int v = 0; v < 4; ++v) o[v] = (half_t)silu_mul(acc[0][j][v], acc[1][j][v]);
                    *(half4_t*)((half_t*)out_base + g * Nw + col) = o;
                }
            } else {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int col = row0 + t * 16 + c4 * 4;
                    if (col < Nw) *(float4_t*)((float*)out_base + g * Nw + col) = acc[t][j];
                }
            }
        }
    }
}

template <int WAVES, bool UP, int PREC>
__device__ __forceinline__ void run_chunk(const TileCtx& c, const DevExpert& ee, void* out_base) {
    const int nct = (c.rows + 15) >> 4;
#define MOEMIX_CASE(n) case n: chunk_body<WAVES, UP, PREC, (n) <= WAVES * 2 ? (n) : WAVES * 2>(c, ee, out_base); break;
    switch (nct) {
        MOEMIX_CASE(1) MOEMIX_CASE(2) MOEMIX_CASE(3) MOEMIX_CASE(4) MOEMIX_CASE(5) MOEMIX_CASE(6) MOEMIX_CASE(7) MOEMIX_CASE(8)
        MOEMIX_CASE(9) MOEMIX_CASE(10) MOEMIX_CASE(11) MOEMIX_CASE(12) MOEMIX_CASE(13) MOEMIX_CASE(14) MOEMIX_CASE(15) MOEMIX_CASE(16)
    }
#undef MOEMIX_CASE
}

// WIDE: the block holds 8-bit experts as well.
template <int WAVES, bool UP, bool WIDE>
__global__ __launch_bounds__(64 * WAVES, 2) void prefill_kernel(const MfmaArgs a) {
    constexpr int kThreads = 64 * WAVES, NT = (UP ? 16 : 32) * WAVES;   // weight rows per workgroup
    extern __shared__ __align__(16) uint8_t lds[];
    const int tid = threadIdx.x;
    int tile_x, split_z;
    place_workgroup(a.tiles, tile_x, split_z);
    const int k_begin = split_z * a.k_per_split;
    const int n_steps = a.k_per_split / kKTile;
    // ---- which expert, which rows.  (The precisions as two words: read lane by lane out of the expert table they would be
    // vector loads from the kernel's arguments.)
    auto prec_of = [&](int expert) {
        return (a.prec16 >> expert) & 1u ? MOE_PREC_FP16 : (a.prec8 >> expert) & 1u ? MOE_PREC_INT8G64 : MOE_PREC_INT4G64;
    };
    // chunks of an expert with n rows, split evenly in whole tiles; rows per chunk
    auto split = [&](int expert, int n, int& per) {
        const int prec = prec_of(expert);
        per = 128;
        const int cap = WAVES == 4 || n <= 128 ? 128 : prec == MOE_PREC_FP16 ? 256 : a.quant_rows;
        if (cap <= 128 && (cap == 0 || n <= 128 || WAVES == 4)) return (n + 127) >> 7;
        // (cap: 128, 192 or 256)
        const int nch = cap == 192 ? (int)(__umulhi((uint32_t)n + 191, 0xAAAAAAABu) >> 7) : (n + cap - 1) >> (cap == 256 ? 8 : 7);
        per = (((n + nch - 1) / nch) + 15) & ~15;
        return nch;
    };
    int e, begin, cnt, per, chunk = blockIdx.y;
    TileCtx c;
    c.tokens = nullptr;
    if (a.direct_expert >= 0) {
        e = a.direct_expert; begin = 0; cnt = a.direct_n;
        split(e, cnt, per);
    } else {
        // Chunks are handed out expert by expert, those whose workgroups run longest first: a launch ends when its last
        // workgroup does, so the long ones must not start last.  Microseconds of a workgroup with 4096 columns: 4-bit 56 and
        // 113 (5 and 16 tiles), 8-bit 65 and 130, 16-bit 91 - 125 (bound by its weight stream up to 8 tiles).  16-bit experts
        // go by their rows, so that those with two chunks come first: the chunks run side by side then and the second finds
        // its weights in L2.  Lane i of every wavefront looks after expert i.
        const int lane = tid & 63;
        const bool mine = lane < a.E;
        int n = 0, b = 0;
        if (mine) {
            b = a.offsets[lane];
            n = a.offsets[lane + 1] - b;
        }
        int pr;
        const int nch = split(lane & 31, n, pr);           // (the last one may be empty)
        const int tiles = (min(n, pr) + 15) >> 4, prec = prec_of(lane & 31);
        const int cost = prec == MOE_PREC_FP16 ? 1000 + n : (prec == MOE_PREC_INT8G64 ? 45 : 35) + 7 * tiles;
        // chunks handed out before this expert's.  (Lane numbers as constants: a loop over them took 265 cycles a round, 4 of
        // the 9 us that a workgroup of a launch with 32 experts spent before its first product.)
        const int key = mine ? cost * 64 + 63 - lane : -1;
        int first = 0;
#pragma unroll
        for (int g = 0; g < MOE_MAX_EXPERTS; g += 8)
            if (g < a.E) {
#pragma unroll
                for (int i = g; i < g + 8; ++i) {
                    const int ki = __builtin_amdgcn_readlane(key, i), ni = __builtin_amdgcn_readlane(nch, i);
                    first += ki > key ? ni : 0;
                }
            }
        const unsigned long long owner = __ballot(mine && chunk >= first && chunk < first + nch);
        if (!owner) return;
        e = __builtin_ctzll(owner);
        begin = __builtin_amdgcn_readlane(b, e);
        cnt = __builtin_amdgcn_readlane(n, e);
        per = __builtin_amdgcn_readlane(pr, e);
        chunk -= __builtin_amdgcn_readlane(first, e);
    }
    c.m0 = chunk * per;
    if (c.m0 >= cnt) return;
    c.in = a.in; c.perm = a.perm; c.top_k = a.top_k; c.K = a.K; c.N = a.N;
    c.begin = begin;
    c.rows = min(per, cnt - c.m0);
    c.n0 = tile_x * NT;
    c.k_begin = k_begin;
    c.n_steps = n_steps;
    c.tail = false;
    // Workgroups that work on different weight rows start at different places of the contraction range and wrap around:
    // walking it in step, every workgroup of the launch would ask for the same columns of rows that lie a power of two apart
    // at the same time, which lands on a fraction of the memory channels.  Up-projection: one starting place per tile;
    // down-projection: one per expert and split, so that the workgroups which share a slice of hidden rows walk it in step
    // and find it in L2.  It depends on nothing else: an output element is summed in the same order in every launch of the same
    // number of wavefronts (which sets the rows of a tile) and splits.  (Starting places by weight row, alike for 4 and 8
    // wavefronts: 150 tokens, Mixtral shape, half 16-bit 410 -> 415 us.)
    c.rot = (c.n_steps & 3) ? 0 : 4 * ((UP ? tile_x * 5 : e * 3 + split_z * 5) % (c.n_steps >> 2));
    c.lds = lds;
    c.lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const DevExpert& ee = a.ex.e[e];
    void* out_base = UP ? a.out : (void*)((float*)a.out + split_z * a.split_stride);
    if (ee.resident == kDeferred) return;
    if (!(ee.resident && ee.w1.data && ee.w3.data && ee.w2.data)) {
        leave_out<UP>(c, out_base, a.status, tile_x, NT, kThreads);
        return;
    }
    const int prec = ee.prec;
    if (prec == MOE_PREC_INT4G64) run_chunk<WAVES, UP, MOE_PREC_INT4G64>(c, ee, out_base);
    else if (WIDE && prec == MOE_PREC_INT8G64) run_chunk<WAVES, UP, WIDE ? MOE_PREC_INT8G64 : MOE_PREC_INT4G64>(c, ee, out_base);
    else run_chunk<WAVES, UP, MOE_PREC_FP16>(c, ee, out_base);
}

template <int WAVES, bool UP, bool WIDE>
void launch_prefill_w(const MfmaArgs& a, dim3 grid, hipStream_t st) {
    constexpr size_t lds_bytes = kLdsBytes * WAVES / 8;
    static std::atomic<unsigned long long> configured{0};
    allow_lds((const void*)prefill_kernel<WAVES, UP, WIDE>, lds_bytes, configured);
    prefill_kernel<WAVES, UP, WIDE><<<grid, 64 * WAVES, lds_bytes, st>>>(a);
}

}  // namespace

template <bool UP>
void launch_prefill(const MfmaArgs& a, dim3 grid, hipStream_t st) {
    if (a.waves == 4) {
        if (a.prec8) launch_prefill_w<4, UP, true>(a, grid, st);
        else launch_prefill_w<4, UP, false>(a, grid, st);
    } else {
        if (a.prec8) launch_prefill_w<8, UP, true>(a, grid, st);
        else launch_prefill_w<8, UP, false>(a, grid, st);
    }
}

#if !defined(MOEMIX_MFMA_DOWN)
template void launch_prefill<true>(const MfmaArgs&, dim3, hipStream_t);
#endif
#if !defined(MOEMIX_MFMA_UP)
template void launch_prefill<false>(const MfmaArgs&, dim3, hipStream_t);
#endif

}  // namespace moemix
