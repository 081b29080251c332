// Expert feed-forward layers on many rows (prefill, batched decode): grouped matrix products on the
// matrix cores (paper §1: experts are parallel FF layers; §3: each is 16-bit or 4-bit).
//
//   up  : h[r, n] = silu(sum_c W1[n,c] x_r[c]) * (sum_c W3[n,c] x_r[c])      rows r of one expert, grouped order
//   down: y[s][r, n] = sum_{c in split s} W2[n,c] h[r,c]                      partial sums of the contraction splits
//
// One workgroup = 4 wavefronts = one (expert, tile of weight rows, chunk of activation rows, contraction split).
// Weights are the A operand of v_mfma_f32_16x16x32_f16: lane (r, c) holds 8 contraction elements of weight row r.
// Activations are the B operand, staged in LDS and shared by the 4 wavefronts.  Each lane's 4 accumulators of one
// 16x16 product are 4 consecutive weight rows of one activation row, so results are stored as 8-byte (fp16) or
// 16-byte (fp32) pieces.  4-bit weights travel as codes and are expanded in registers (codes masked into the
// mantissa of an fp16 constant, the constant subtracted, one packed fp16 multiply-add with the group's scale and
// zero); 8-bit codes likewise, with a byte permute in place of the masks.
// tile_body here serves launches with chunks of at most 64 rows, and of 128 where contraction lengths are odd multiples of 64:
// weights are read in whole 128-byte lines (8 lanes per row, 8 rows per load instruction, streamed) and turned into operand
// layout through a small wavefront-private LDS region; activations as a [16*CT, 128*SPB] tile per stage, double-buffered,
// one barrier per stage.  The launches with 128-row chunks of whole steps are in ffn_prefill.hip.
#include <algorithm>
#include <atomic>
#include <cmath>

#include "common.hpp"
#include "kernels.hpp"
#include "mfma_common.hpp"

namespace moemix {

namespace {

// Weights of launches with few activation rows per expert are read once, in whole lines: streamed past the caches'
// replacement order.
constexpr int kTemporalNA = 4;     // A operands per wavefront from which on weight lines are kept for sibling chunks
constexpr int kNASmall = 2;        // A operands per wavefront of launches with at most 32 rows per chunk
constexpr int kSPBMax = 2;         // most 128-column steps per LDS stage
constexpr int spb_for(int ct) { return (8 / ct) < kSPBMax ? (8 / ct) : kSPBMax; }

// Results of one workgroup: lane (r16, c4) holds, for activation row 16 j + r16, weight rows
// 16 tile + 4 c4 + (0..3) of the wavefront's rows.
template <bool UP, int NCT, int NA>
__device__ __forceinline__ void store_results(const TileCtx& c, const float4_t (&acc)[NA][NCT], void* out_base, int wave,
                                              int r16, int c4) {
    constexpr int RW = UP ? 8 * NA : 16 * NA;          // weight rows per wavefront
    const int N = c.N;
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
        const int rr = 16 * j + r16;
        if (rr < c.rows) {
            const size_t g = (size_t)(c.begin + c.m0 + rr);
            if (UP) {
                half_t* h = (half_t*)out_base + g * N;
#pragma unroll
                for (int tile = 0; tile < NA / 2; ++tile) {
                    const int col = c.n0 + wave * RW + tile * 16 + c4 * 4;
                    if (col < N) {
                        half4_t o;
#pragma unroll
                        for (int v = 0; v < 4; ++v) o[v] = (half_t)silu_mul(acc[2 * tile][j][v], acc[2 * tile + 1][j][v]);
                        *(half4_t*)(h + col) = o;
                    }
                }
            } else {
                float* y = (float*)out_base + g * N;
#pragma unroll
                for (int tile = 0; tile < NA; ++tile) {
                    const int col = c.n0 + wave * RW + tile * 16 + c4 * 4;
                    if (col < N) *(float4_t*)(y + col) = acc[tile][j];
                }
            }
        }
    }
}

// The first team's sums become those of all teams, added in the order of the teams.  The others hand theirs over in their
// activation stages (no wavefront reads those any more: every team has passed the last barrier of the range).
template <int KS, int NCT, int NA>
__device__ __forceinline__ void share_sums(const TileCtx& c, float4_t (&acc)[NA][NCT], int wave, int lane) {
    const auto slot = [&](uint8_t* lds, int t, int j) { return (float4_t*)(lds + (((wave * NA + t) * NCT + j) * 64 + lane) * 16); };
    if (c.team) {
#pragma unroll
        for (int t = 0; t < NA; ++t)
#pragma unroll
            for (int j = 0; j < NCT; ++j) *slot(c.lds, t, j) = acc[t][j];
    }
    __syncthreads();
    if (c.team) return;
#pragma unroll
    for (int s = 1; s < KS; ++s)
#pragma unroll
        for (int t = 0; t < NA; ++t)
#pragma unroll
            for (int j = 0; j < NCT; ++j) acc[t][j] += *slot(c.lds + s * c.team_bytes, t, j);
}

// A wavefront holds NA A operands (16-row tiles of weights) per step.  UP: two matrices (w1, w3), NA/2 tiles each
// (workgroup of 4 wavefronts: 32 NA rows); down: one matrix (w2), NA tiles (workgroup: 64 NA rows).  NA = 4 for
// chunks of many activation rows (each B operand read from LDS feeds 4 products), NA = 2 when a chunk holds at
// most 32 rows: the kernel is then bound by its weight stream and a chain of latencies, and half the registers per
// wavefront buy twice the wavefronts per SIMD to hide them.
// NCT = 16-row activation tiles computed (exactly the tiles that hold rows), so the inner loops are
// straight-line code.  SPB = 128-column steps per LDS stage (and per barrier): a launch with few activation
// rows per chunk stages more columns at a time, so that the LDS buffers always hold 128 x 128 elements.
// HALF: rows of an odd multiple of 64 columns.  The last step of the row (c.tail) is half a step: activations past the
// end are zero in LDS, loads past the end of a row repeat its last pieces, and the other operand of those products is
// zero too (quantized weights: the scale and zero of the absent group are zero words out of the byte permute, which
// costs nothing) or the products are left out (16-bit weights: the last two of four sub-steps), so that neither an
// infinity next door nor one in the repeated piece reaches a sum.
//
// KS: the 4 wavefronts are KS teams of 4 / KS, each with a part of the contraction range and LDS of its own, all on the same
// weight rows, 1 / KS as many; c is the team's.  The teams meet at every barrier (c.barriers of them, for the longest part), and
// the first adds up the sums.
template <bool UP, int PREC, int NCT, int SPB, int NA, bool HALF = false, int KS = 1>   // PREC: moe_prec of the expert
__device__ __forceinline__ void tile_body(const TileCtx& c, const DevExpert& ee, void* out_base) {
    constexpr bool INT4 = PREC == MOE_PREC_INT4G64, INT8 = PREC == MOE_PREC_INT8G64, QUANT = INT4 || INT8;
    constexpr int RW = UP ? 8 * NA : 16 * NA;      // weight rows per wavefront: 16 NA / (matrices)
    constexpr int TW = 4 / KS;                     // wavefronts per team
    constexpr int kStride = SPB * kKTile * 2 + 16;     // bytes per activation row of an LDS stage (16 bytes of padding)
    constexpr int PPR = 16 * SPB;                      // 16-byte pieces per row of a stage
    constexpr int RPP = 64 * TW / PPR;                 // rows the threads of a team cover in one pass
    constexpr int NP = NCT * SPB * KS;                 // pieces per thread and stage
    const int tid = threadIdx.x % (64 * TW), lane = tid & 63, r16 = lane & 15, c4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = c.K, N = c.N, n_steps = c.n_steps;
    const int last = n_steps - 1;    // loads that would run past the contraction range repeat the last step instead
    const int buf_bytes = c.mc * kStride;

    // ---- activation pieces this thread stages: column piece tid % PPR of rows tid / PPR + RPP i.
    // Rows past the end of the chunk repeat its last row: their products are computed and never stored.
    const int pcol = tid % PPR, pstep = pcol >> 4;     // pstep: which 128-column step of the stage the piece is in
    const gptr_t xbase = scalar_ptr(c.in + c.k_begin);
    uint32_t xoff[NP];                                 // byte offsets: the input rows of a launch span less than 4 GB
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        int rr = tid / PPR + RPP * i;
        rr = rr < c.rows ? rr : c.rows - 1;
        const int g = c.begin + c.m0 + rr;
        const uint32_t src = (UP && NA == kNASmall && c.tokens) ? (uint32_t)c.tokens[rr]
                           : (UP && c.perm) ? (uint32_t)(c.perm[g] / c.top_k) : (uint32_t)g;
        xoff[i] = src * (uint32_t)K * 2 + (pcol & 15) * 16;
    }
    uint4_t xr[NP];
    const bool tail = HALF && c.tail;
    bool xpast = false;                                // the pieces in xr lie past the end of the rows
    auto load_x = [&](int stage) {
        int step = stage * SPB + pstep;
        step = step < last ? step : last;
        step = step + c.rot < n_steps ? step + c.rot : step + c.rot - n_steps;
        if (HALF) xpast = tail && step == last && (pcol & 8);
        const int byte = step * (kKTile * 2) - (HALF && xpast ? kKTile : 0);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if (HALF) xr[i] = *(const uint4_t MOEMIX_GLOBAL*)(xbase + fresh_offset(xoff[i] + byte));
            else xr[i] = *(const uint4_t MOEMIX_GLOBAL*)(xbase + step * (kKTile * 2) + fresh_offset(xoff[i]));
        }
    };
    auto store_x = [&](int buf) {
        uint8_t* base = c.lds + buf * buf_bytes + (tid / PPR) * kStride + pcol * 16;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            uint4_t v = HALF && xpast ? uint4_t{0u, 0u, 0u, 0u} : xr[i];
            if (INT4) {   // element order (0,4,1,5,2,6,3,7) inside each group of 8, as expand_word delivers codes
                const half8_t h = __builtin_bit_cast(half8_t, v);
                v = __builtin_bit_cast(uint4_t, half8_t{h[0], h[4], h[1], h[5], h[2], h[6], h[3], h[7]});
            }
            *(uint4_t*)(base + i * RPP * kStride) = v;
        }
    };

    // ---- scales and zeros of this lane's weight rows (4-bit): the wavefront owns RW rows from n0 + wave * RW,
    // in tiles of 16; lane (r16, c4) looks after row r16 of each tile
    gptr_t sbase[NA], zbase[NA];                       // uniform bases, one lane offset for both
    uint32_t soff[NA];
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        const int tile = UP ? (t >> 1) : t;                        // up: operands (w1 tile0, w3 tile0, w1 tile1, w3 tile1)
        const DevMat& m = UP ? ((t & 1) ? ee.w3 : ee.w1) : ee.w2;
        int row = c.n0 + wave * RW + tile * 16 + r16;
        row = row < N ? row : N - 1;                               // rows past the end repeat the last row, never stored
        sbase[t] = QUANT ? scalar_ptr(m.scale + (c.k_begin >> 6)) : nullptr;
        zbase[t] = QUANT ? scalar_ptr(m.zero + (c.k_begin >> 6)) : nullptr;
        soff[t] = (uint32_t)row * (uint32_t)(K >> 6) * 2;
    }
    // (what the 128-bit scale loads below ask of the arrays, and of the rows: a range of uneven splits, or a team's part of one, may
    // hold whole fours of steps where rows do not)
    bool sz_aligned16 = K % 512 == 0;
#pragma unroll
    for (int t = 0; t < NA; ++t)
        sz_aligned16 = sz_aligned16 && !(((uintptr_t)sbase[t] | (uintptr_t)zbase[t]) & 15);

    float4_t acc[NA][NCT];
#pragma unroll
    for (int t = 0; t < NA; ++t)
#pragma unroll
        for (int j = 0; j < NCT; ++j) acc[t][j] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

    // B operand of activation tile j, step q of the stage, sub-step s: lane (r16, c4) reads 8 elements of
    // activation row 16 j + r16
    // (quantized weights: a lane owns 32 consecutive columns of the 128-column step, sub-step s its s-th eight of
    // them -- a permutation of the contraction index that the activations follow)
    const int b_lane = r16 * kStride + (QUANT ? c4 * 64 : c4 * 16);
    constexpr int b_sub = QUANT ? 16 : 64;

    // Pipeline: at the first step of a stage the activation data of the next stage goes to the other LDS buffer
    // (its loads were issued a stage earlier) and the loads of the stage after that are issued; weights run three
    // steps (4-bit) or three 32-column sub-steps (16-bit) ahead in a ring of four register buffers; one barrier
    // closes each stage.  Steps are processed in groups of G = max(4, SPB) so that ring slots, the quarter of the
    // scale loads and the place of the barriers are compile-time constants.
    constexpr int G = SPB > 4 ? SPB : 4;
    uint32_t sz_cur[NA][2], sz_next[NA][2];
    const uint32_t sel_full = (c4 >> 1) ? 0x03020302u : 0x01000100u;   // which of the two groups of a 128-column step
    // half a step: its group is the second of the two words fetched for it (load_sz), the other one is absent (the
    // permute's selector 0x0C is a zero byte)
    const uint32_t sel_tail = (c4 >> 1) ? 0x0C0C0C0Cu : 0x03020302u;
    const uint32_t m1024 = vreg_const(0x64006400u), m64 = vreg_const(INT8 ? 0x64646464u : 0x54005400u);
    // scales and zeros of four steps with one load: lane (r16, c4) fetches the pair of groups of step 4 S + c4
    auto load_sz = [&](uint32_t (&dst)[NA][2], int S) {
        int step = 4 * S + c4;
        step = step < last ? step : last;
        step = step + c.rot < n_steps ? step + c.rot : step + c.rot - n_steps;
        if (HALF) {                                    // (the pair of half a step starts one group earlier)
            const uint32_t byte = step * 4 - (tail && step == last ? 2 : 0);
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                dst[t][0] = *(const uint32_half_aligned_t MOEMIX_GLOBAL*)(sbase[t] + fresh_offset(soff[t] + byte));
                dst[t][1] = *(const uint32_half_aligned_t MOEMIX_GLOBAL*)(zbase[t] + fresh_offset(soff[t] + byte));
            }
            return;
        }
#pragma unroll
        for (int t = 0; t < NA; ++t) {
            dst[t][0] = *(const uint32_t MOEMIX_GLOBAL*)(sbase[t] + step * 4 + fresh_offset(soff[t]));
            dst[t][1] = *(const uint32_t MOEMIX_GLOBAL*)(zbase[t] + step * 4 + fresh_offset(soff[t]));
        }
    };
    // 4-bit, at most 32 rows per chunk (the launch is bound by device memory), ranges of a multiple of 4 steps: scales
    // and zeros of sixteen steps with one 128-bit load per lane and array (lane (r16, c4) fetches the eight groups of
    // steps 16 S + 4 c4 .. + 3), so a row's 128-byte line of scales is asked for in two 64-byte requests instead of
    // eight of 16 bytes; with the narrow requests the lines left L2 between requests and a launch fetched 29 % more
    // than its algorithmic bytes.
    constexpr bool kWideSz = INT4 && NA == kNASmall && !HALF;
    const bool wide_sz = kWideSz && !(n_steps & 3) && sz_aligned16;
    uint4_t sq_cur[NA][2], sq_next[NA][2];
    auto load_sq = [&](uint4_t (&dst)[NA][2], int S) {
        int step = 16 * S + 4 * c4;
        step = step < n_steps - 4 ? step : n_steps - 4;            // groups past the end repeat the last one (never used)
        step = step + c.rot < n_steps ? step + c.rot : step + c.rot - n_steps;   // (the rotation is a multiple of 4 steps)
#pragma unroll
        for (int t = 0; t < NA; ++t) {
            dst[t][0] = *(const uint4_t MOEMIX_GLOBAL*)(sbase[t] + step * 4 + fresh_offset(soff[t]));
            dst[t][1] = *(const uint4_t MOEMIX_GLOBAL*)(zbase[t] + step * 4 + fresh_offset(soff[t]));
        }
    };
    auto load_sz_narrow = [&](uint4_t (&dst)[NA][2], int S) {      // the narrow form, kept in word 0 of the same registers
        int step = 4 * S + c4;
        step = step < last ? step : last;
        step = step + c.rot < n_steps ? step + c.rot : step + c.rot - n_steps;
#pragma unroll
        for (int t = 0; t < NA; ++t) {
            dst[t][0][0] = *(const uint32_t MOEMIX_GLOBAL*)(sbase[t] + step * 4 + fresh_offset(soff[t]));
            dst[t][1][0] = *(const uint32_t MOEMIX_GLOBAL*)(zbase[t] + step * 4 + fresh_offset(soff[t]));
        }
    };
    // Weights take a detour through LDS so that device memory is read in whole 128-byte lines: one load instruction
    // fetches, for 8 weight rows, one 128-byte line of each row with 8 lanes per row; the 16-byte pieces are written
    // to a wavefront-private LDS region (slots XOR-swizzled by row so that neither side has bank conflicts) and read
    // back in operand layout.  A staging unit is UB bytes of every row: 4-bit, one line = 256 columns = two steps,
    // lane (r16, c4) takes slot 4 * (step & 1) + c4 as its 32 codes of a step; 16-bit, two lines = 128 columns = one
    // step, lane (r16, c4) takes slot 4 * sb + c4 as its 8 weights of sub-step sb.
    // 8-bit, one line = 128 columns = one step, lane (r16, c4) takes slots 2 c4 and 2 c4 + 1 as its 32 codes.
    constexpr int UL = QUANT ? 1 : 2;    // lines per row and unit
    constexpr int UB = UL * 128;         // bytes per row and unit
    constexpr int UA = QUANT ? 2 : 4;    // operand registers (128-bit) per A operand and unit
    uint4_t stg[NA][2 * UL];             // staged loads of the next unit
    uint4_t apc[NA][UA];                 // the current unit in operand layout
    uint32_t goff[NA][2];                // per-lane byte offsets of the staged rows inside the weight matrix
    gptr_t cbase[NA];                    // uniform: start of the contraction range in the weight matrix
    uint8_t* const wreg = c.lds + 2 * buf_bytes + wave * (NA * c.unit_bytes);
    const int w_wr = (lane >> 3) * UB + (((lane & 7) ^ (lane >> 3)) * 16);
    const int w_rd = r16 * UB;
    const int last_unit = INT4 ? (n_steps + 1) / 2 - 1 : n_steps - 1;
    const int row_end = (INT4 ? (K - c.k_begin) >> 1 : INT8 ? K - c.k_begin : 2 * (K - c.k_begin)) - 16;   // the row's last piece
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        const int tile = UP ? (t >> 1) : t;
        const DevMat& m = UP ? ((t & 1) ? ee.w3 : ee.w1) : ee.w2;
        cbase[t] = scalar_ptr(m.data + (INT4 ? (c.k_begin >> 1) : INT8 ? c.k_begin : c.k_begin * 2));
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
            int row = c.n0 + wave * RW + tile * 16 + 8 * hb + (lane >> 3);
            row = row < N ? row : N - 1;                           // rows past the end repeat the last row, never stored
            goff[t][hb] = (uint32_t)row * (uint32_t)(INT4 ? (K >> 1) : INT8 ? K : 2 * K) + (lane & 7) * 16;
        }
    }
    auto load_unit = [&](int unit) {
        // No loads for a unit past the end (the registers keep what they hold; it is never used).  Repeating the last
        // unit instead looked free and was not: a streamed line has left L2 once it has been read, so every workgroup
        // fetched its last line of every row three times (batched decode: + 11 % of the code bytes).
        if (unit > last_unit) return;
        {   // (a rotated range has an even number of steps: whole units)
            const int urot = INT4 ? c.rot >> 1 : c.rot, units = INT4 ? n_steps >> 1 : n_steps;
            if (c.rot) unit = unit + urot < units ? unit + urot : unit + urot - units;
        }
        // 4-bit, odd number of steps: the last pair's second half would leave the row only in the last row of the
        // last split, so the pair is moved back by one step there (its second half is then never used)
        const int byte0 = (HALF || !INT4 || 2 * unit + 2 <= n_steps) ? unit * UB : unit * UB - 64;
#pragma unroll
        for (int t = 0; t < NA; ++t)
#pragma unroll
            for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                for (int q = 0; q < UL; ++q)
                {
                    // (HALF: pieces past the end of the row repeat its last one)
                    const int lp = (lane & 7) * 16, at = byte0 + q * 128 + lp;
                    const uint4_t MOEMIX_GLOBAL* src =
                        HALF ? (const uint4_t MOEMIX_GLOBAL*)(cbase[t] + fresh_offset(goff[t][hb] + (at < row_end ? at : row_end) - lp))
                             : (const uint4_t MOEMIX_GLOBAL*)(cbase[t] + (byte0 + q * 128) + fresh_offset(goff[t][hb]));
                    // launches with many activation rows per expert run several chunks of one expert side by side on
                    // the same XCD: the second reader of a weight line should find it in L2, so the line is not
                    // marked as used once there
                    // (HALF, quantized: rows are no whole number of lines, so neighbouring units share one; with the
                    // streaming hint it was fetched again for the second: 33 tokens, 4 of 32 8-bit experts of
                    // 2880 x 2880, 213 -> 202 us for the block)
                    stg[t][hb * UL + q] = (NA >= kTemporalNA || (HALF && QUANT)) ? *src : __builtin_nontemporal_load(src);
                }
    };
    auto stage_to_lds = [&]() {
        wave_lds_handover();   // the previous unit has been read by every lane
#pragma unroll
        for (int t = 0; t < NA; ++t)
#pragma unroll
            for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                for (int q = 0; q < UL; ++q)
                    *(uint4_t*)(wreg + t * (16 * UB) + hb * (8 * UB) + q * 128 + w_wr) = stg[t][hb * UL + q];
        wave_lds_handover();
    };
    auto lds_to_operands = [&](int unit) {
        // (4-bit: for the moved-back last pair of an odd range the wanted step sits in the second half)
        const int shift = (HALF || !INT4 || 2 * unit + 2 <= n_steps) ? 0 : 4;
#pragma unroll
        for (int t = 0; t < NA; ++t)
#pragma unroll
            for (int h = 0; h < UA; ++h) {
                const int slot = INT8 ? 2 * c4 + h : (4 * h + c4 + shift) & (8 * UL - 1);
                // the XOR touches the low three bits of the slot only: a piece stays inside its 128-byte line
                apc[t][h] = *(const uint4_t*)(wreg + t * (16 * UB) + w_rd + ((slot ^ (r16 & 7)) * 16));
            }
    };

    load_x(0);
    if (kWideSz && wide_sz) load_sq(sq_cur, 0);
    else if (kWideSz) load_sz_narrow(sq_cur, 0);
    else if (QUANT) load_sz(sz_cur, 0);
    load_unit(0);
    stage_to_lds();
    load_unit(1);
    store_x(0);
    load_x(1);
    __syncthreads();

    for (int base = 0; base < n_steps; base += G) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int step = base + g;
            if (step < n_steps) {                                   // uniform; false only in the last group
                const bool half_step = HALF && tail && step == last;
                const uint32_t sel = half_step ? sel_tail : sel_full;
                const int stage = step / SPB;
                const uint8_t* xb = c.lds + (stage & 1) * buf_bytes + b_lane + (g % SPB) * (kKTile * 2);
                if (g % SPB == 0) {
                    store_x((stage + 1) & 1);                       // past the last stage this writes data nobody reads
                    load_x(stage + 2);
                    // 4-bit, two steps per stage = one unit of codes per stage: the unit that takes the place of the
                    // one used up in the last stage is asked for here, after the activation loads.  Loads return in
                    // the order of their issue, so an activation load (a hit in L2) issued behind a load of weights
                    // from device memory is held back as long as that one takes.
                    if (INT4 && SPB == 2 && step > 0) load_unit(((step - 1) >> 1) + 2);
                }
                if (INT4) {
                    if (kWideSz && wide_sz) {
                        if (g % 4 == 0 && (step & 15) == 0) {
                            if (step > 0) {
#pragma unroll
                                for (int t = 0; t < NA; ++t) { sq_cur[t][0] = sq_next[t][0]; sq_cur[t][1] = sq_next[t][1]; }
                            }
                            if (step + 16 < n_steps) load_sq(sq_next, step / 16 + 1);   // (nothing past the end: see load_unit)
                        }
                    } else if (g % 4 == 0) {
                        if (step > 0) {
#pragma unroll
                            for (int t = 0; t < NA; ++t) {
                                if (kWideSz) { sq_cur[t][0][0] = sq_next[t][0][0]; sq_cur[t][1][0] = sq_next[t][1][0]; }
                                else { sz_cur[t][0] = sz_next[t][0]; sz_cur[t][1] = sz_next[t][1]; }
                            }
                        }
                        if (step + 4 < n_steps) {                   // (nothing past the end: see load_unit)
                            if (kWideSz) load_sz_narrow(sq_next, step / 4 + 1);
                            else load_sz(sz_next, step / 4 + 1);
                        }
                    }
                    if (g % 2 == 0) lds_to_operands(step >> 1);
                    half2_t s2[NA], z2[NA];
                    // the lane of this row that fetched this step's scales: the step's place among four, or (wide
                    // requests) its group of four steps' place among four, where the step's word is g & 3
                    const int src = (r16 + 16 * ((kWideSz && wide_sz) ? (step >> 2) & 3 : g & 3)) * 4;
#pragma unroll
                    for (int t = 0; t < NA; ++t) {
                        const uint32_t sw = !kWideSz ? sz_cur[t][0] : wide_sz ? sq_cur[t][0][g & 3] : sq_cur[t][0][0];
                        const uint32_t zw = !kWideSz ? sz_cur[t][1] : wide_sz ? sq_cur[t][1][g & 3] : sq_cur[t][1][0];
                        const uint32_t sd = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)sw);
                        const uint32_t zd = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)zw);
                        s2[t] = as_half2(__builtin_amdgcn_perm(sd, sd, sel));
                        z2[t] = as_half2(__builtin_amdgcn_perm(zd, zd, sel));
                    }
#pragma unroll
                    for (int sb = 0; sb < 4; ++sb) {
                        half8_t af[NA];
#pragma unroll
                        for (int t = 0; t < NA; ++t) af[t] = expand_word(apc[t][g & 1][sb], s2[t], z2[t], m1024, m64);
#pragma unroll
                        for (int j2 = 0; j2 < NCT; ++j2) {
                            const half8_t b = *(const half8_t*)(xb + j2 * 16 * kStride + sb * b_sub);
#pragma unroll
                            for (int t = 0; t < NA; ++t) acc[t][j2] = mfma16(af[t], b, acc[t][j2]);
                        }
                    }
                    if (g % 2 == 1 || step == last) {               // the pair is used up: the next one takes its place
                        stage_to_lds();
                        if (SPB != 2) load_unit((step >> 1) + 2);   // (two steps per stage: at the next stage's start)
                    }
                } else if (INT8) {
                    if (g % 4 == 0) {
                        if (step > 0) {
#pragma unroll
                            for (int t = 0; t < NA; ++t) { sz_cur[t][0] = sz_next[t][0]; sz_cur[t][1] = sz_next[t][1]; }
                        }
                        if (step + 4 < n_steps) load_sz(sz_next, step / 4 + 1);
                    }
                    lds_to_operands(step);
                    half2_t s2[NA], z2[NA];
                    const int src = (r16 + 16 * (g & 3)) * 4;       // the lane of this row that fetched this step's scales
#pragma unroll
                    for (int t = 0; t < NA; ++t) {
                        const uint32_t sd = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)sz_cur[t][0]);
                        const uint32_t zd = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)sz_cur[t][1]);
                        s2[t] = as_half2(__builtin_amdgcn_perm(sd, sd, sel));
                        z2[t] = as_half2(__builtin_amdgcn_perm(zd, zd, sel));
                    }
#pragma unroll
                    for (int sb = 0; sb < 4; ++sb) {
                        half8_t af[NA];
#pragma unroll
                        for (int t = 0; t < NA; ++t)
                            af[t] = expand_bytes(apc[t][sb >> 1][2 * (sb & 1)], apc[t][sb >> 1][2 * (sb & 1) + 1], s2[t], z2[t],
                                                 m1024, m64);
#pragma unroll
                        for (int j2 = 0; j2 < NCT; ++j2) {
                            const half8_t b = *(const half8_t*)(xb + j2 * 16 * kStride + sb * b_sub);
#pragma unroll
                            for (int t = 0; t < NA; ++t) acc[t][j2] = mfma16(af[t], b, acc[t][j2]);
                        }
                    }
                    stage_to_lds();                                 // the step is used up: the next one takes its place
                    load_unit(step + 2);
                } else {
                    lds_to_operands(step);
#pragma unroll
                    for (int sb = 0; sb < 4; ++sb) {
                        if (HALF && sb == 2 && half_step) break;
#pragma unroll
                        for (int j2 = 0; j2 < NCT; ++j2) {
                            const half8_t b = *(const half8_t*)(xb + j2 * 16 * kStride + sb * b_sub);
#pragma unroll
                            for (int t = 0; t < NA; ++t)
                                acc[t][j2] = mfma16(__builtin_bit_cast(half8_t, apc[t][sb]), b, acc[t][j2]);
                        }
                    }
                    stage_to_lds();                                 // the step is used up: the next one takes its place
                    load_unit(step + 2);
                }
                if (g % SPB == SPB - 1 || step == last) __syncthreads();
            }
        }
    }

    if constexpr (KS > 1) {
        for (int i = (n_steps + SPB - 1) / SPB; i < c.barriers; ++i) __syncthreads();
        share_sums<KS, NCT, NA>(c, acc, wave, lane);
        if (c.team) return;
    }
    store_results<UP, NCT, NA>(c, acc, out_base, wave, r16, c4);
}

// Steps of each of `teams` parts of a range, the last of which may be shorter: whole fours where that comes out even (the wide
// loads of scales), else whole pairs (units of 4-bit codes).
__host__ __device__ inline int team_steps(int steps, int teams) {
    const int unit = steps % (4 * teams) == 0 ? 4 : 2;
    return (steps + teams * unit - 1) / (teams * unit) * unit;
}

// LDS of a workgroup of grouped_mfma_kernel: two activation stages for each team, then weight staging, `unit` bytes for each A operand of
// the 4 wavefronts (c.unit_bytes; a team's part holds its own).
constexpr size_t lds_bytes_for(int ct, int spb, int teams, int unit) {
    return (size_t)teams * 2 * 16 * ct * (spb * kKTile * 2 + 16) + 4 * (ct <= 2 ? kNASmall : 4) * unit;
}
// Four teams with chunks of two tiles leave no room for the staging of 16-bit weights: such launches hold no 16-bit experts (teams_for) and
// have no code for them.
constexpr bool room_for_16bit(int ct, int spb, int teams) {
    return lds_bytes_for(ct, spb, teams, 4096) + (ct <= 2 ? 4 * 16 * ct * sizeof(uint16_t) : 0) <= 160 * 1024;
}

// WIDE: the block holds 8-bit experts as well.  The 8-bit body needs more registers than the other two, and a
// kernel's register count is that of its largest body, so blocks without 8-bit experts get a kernel without it
// (and keep four wavefronts per SIMD at few rows per expert).  In the wide kernel tile_body has variants for 1, 2, 4 and 8
// tiles only.
// HALF: contraction lengths that are odd multiples of 64 (and 128-row chunks whose rows end too close to the reach of 32-bit
// offsets for ffn_prefill.hip), all precisions.  (A wavefront per weight row
// with scalar products, which is what such widths had, took 296 + 190 us for 33 tokens, 4 of 32 experts, d_model and
// d_ff 2880, three quarters of the experts 4-bit; 105 + 54 us here, 4.6 TB/s of stored weights; the rest of the way to the 7 TB/s of a plain read is scales asked for 4 bytes at
// a time and 4-bit rows whose 128-byte requests straddle two lines.)
// SPB: 128-column steps per LDS stage.  Launches with 64-row chunks at whole steps, which hold no 16-bit experts, take one instead
// of two (one_step_per_stage): their stages and weight staging then fit LDS twice (67 KB where two steps want 100), and two
// wavefronts per SIMD are worth more than half the barriers.  Block with 200 tokens, Mixtral shape: 4-bit 359 -> 306 us,
// 8-bit 408 -> 372; 4-bit 2048 x 5632, 160 tokens 117 -> 95.  (Contractions that end with half a step lose 7 %.)
//
// KS: teams that the 4 wavefronts make, which share the contraction range (teams_for).  Launches of few workgroups are bound by
// the chain of steps of each, not by memory: three 4-bit experts of 6784 x 512, 42 tokens, block 64.4 -> 47.5 us with two teams, 38.9 with four; five
// 16-bit ones of 512 x 7808, 8 tokens, 76.6 -> 43.0 with four.
template <bool UP, int CT, bool WIDE, bool HALF, int SPB, int KS>
__global__ __launch_bounds__(256, CT == 4 && SPB == 1 ? 2 : 1) void grouped_mfma_kernel(const MfmaArgs a) {
    constexpr int MC = 16 * CT;                  // activation rows per chunk
    constexpr int NA = CT <= 2 ? kNASmall : 4;   // A operands per wavefront
    constexpr int NT = (UP ? 32 * NA : 64 * NA) / KS;   // weight rows per workgroup
    extern __shared__ __align__(16) uint8_t lds[];   // per team: stages [2][MC][SPB * 256 + 16], weight staging (lds_bytes_for)
    const int tid = threadIdx.x;
    int tile_x, split_z;
    place_workgroup(a.tiles, tile_x, split_z);

    // ---- which expert, which rows
    int k_begin = split_z * a.k_per_split;
    // (the last range of uneven splits is shorter; launches of few pairs only)
    int n_steps = HALF || CT == 1 ? (min(a.k_per_split, a.K - k_begin) + kKTile - 1) / kKTile : a.k_per_split / kKTile;
    int e, begin, cnt, chunk = blockIdx.y;
    TileCtx c;
    c.tokens = nullptr;
    if (a.direct_expert >= 0) {
        e = a.direct_expert; begin = 0; cnt = a.direct_n;
    } else if (CT <= 2 && a.idx) {
        // few pairs: the expert's rows by ballots over the routing result, every wavefront for itself; grouped rows keep
        // increasing pair order, as the grouping kernel has them
        constexpr int NQ = kInlinePairs / 64;
        __shared__ uint16_t tokens[4][MC];
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        int v[NQ];
        load_pairs(a.idx, a.P, lane, v);
        e = -1; begin = 0; cnt = 0;
        for (int i = 0; i < a.E; ++i) {
            int n = 0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) n += __popcll(__ballot(v[q] == i));
            const int nch = (n + MC - 1) / MC;
            if (chunk < nch) { e = i; cnt = n; break; }
            chunk -= nch;
            begin += n;
        }
        if (e < 0) return;
        if (UP) {
            int row = -chunk * MC;                         // of the chunk
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const unsigned long long m = __ballot(v[q] == e);
                const int r = row + __popcll(m & ((1ull << lane) - 1ull));
                if (v[q] == e && r >= 0 && r < MC) tokens[wave][r] = (uint16_t)((64 * q + lane) / a.top_k);
                row += __popcll(m);
            }
            wave_lds_handover();
            c.tokens = tokens[wave];
        }
    } else {
        e = -1; begin = 0; cnt = 0;
        for (int i = 0; i < a.E; ++i) {
            const int b = a.offsets[i], n = a.offsets[i + 1] - b, nch = (n + MC - 1) / MC;
            if (chunk < nch) { e = i; begin = b; cnt = n; break; }
            chunk -= nch;
        }
        if (e < 0) return;
    }
    c.m0 = chunk * MC;
    if (c.m0 >= cnt) return;
    c.in = a.in; c.perm = a.perm; c.top_k = a.top_k; c.K = a.K; c.N = a.N;
    c.begin = begin;
    c.rows = min(MC, cnt - c.m0);
    c.n0 = tile_x * NT;
    c.mc = MC;
    c.unit_bytes = a.unit_bytes;
    c.lds = lds;
    if constexpr (KS > 1) {
        const int part = team_steps(n_steps, KS);
        c.team = __builtin_amdgcn_readfirstlane(tid / (256 / KS));
        c.team_bytes = 2 * MC * (SPB * kKTile * 2 + 16) + 4 / KS * NA * a.unit_bytes;
        c.barriers = (part + SPB - 1) / SPB;
        c.lds = lds + c.team * c.team_bytes;
        k_begin += c.team * part * kKTile;
        n_steps = min(part, n_steps - c.team * part);
    }
    c.k_begin = k_begin;
    c.n_steps = n_steps;
    c.tail = HALF && k_begin + n_steps * kKTile > a.K;
    // Workgroups that work on different weight rows start at different places of the contraction range and wrap
    // around: walking it in step, every workgroup of the launch would ask for the same columns of rows that lie a
    // power of two apart at the same time, which lands on a fraction of the memory channels (measured with a bare
    // read kernel of the same access pattern: 4.3 TB/s in step, 6.0 TB/s staggered).  The offset depends on the
    // tile of weight rows, the expert and the split only: an output element is summed in the same order in every launch
    // with the same rows per tile and splits.
    // Up-projection: one starting place per tile.  Down-projection (rows 7 x 4 KB apart in the Mixtral shape, less
    // prone to the effect): one per expert and contraction split, so that the workgroups which share a slice of the
    // hidden rows walk it in step and find it in L2 (fetched bytes of the prefill down-projection: 1060 MB with one
    // starting place per tile, 781 MB per slice, 637 MB with the slice's workgroups on two XCDs as well).
    c.rot = (HALF || (c.n_steps & 3)) ? 0 : 4 * ((UP ? tile_x * 5 : e * 3 + split_z * 5) % (c.n_steps >> 2));
    const DevExpert& ee = a.ex.e[e];
    void* out_base = UP ? a.out : (void*)((float*)a.out + split_z * a.split_stride);
    if (ee.resident == kDeferred) return;
    if (!(ee.resident && ee.w1.data && ee.w3.data && ee.w2.data)) {
        leave_out<UP>(c, out_base, a.status, tile_x, NT, 256);
        return;
    }
    const int prec = ee.prec;
    const int nct = (c.rows + 15) >> 4;          // 16-row tiles that hold any rows
    // (64-row chunks at whole steps: blocks with 16-bit experts take ffn_prefill.hip)
    constexpr bool k16 = (CT != 4 || HALF) && room_for_16bit(CT, SPB, KS);
    // the straight-line body for exactly the chunk's tiles where the launch can have that many (the clamp keeps
    // the smaller launches from instantiating bodies they never run)
#define MOEMIX_BODY(n)                                                                                          \
    do {                                                                                                        \
        if (prec == MOE_PREC_INT4G64) tile_body<UP, MOE_PREC_INT4G64, ((n) <= CT ? (n) : CT), SPB, NA, HALF, KS>(c, ee, out_base); \
        else if (WIDE && prec == MOE_PREC_INT8G64) tile_body<UP, WIDE ? MOE_PREC_INT8G64 : MOE_PREC_INT4G64, ((n) <= CT ? (n) : CT), SPB, NA, HALF, KS>(c, ee, out_base); \
        else if (k16) tile_body<UP, k16 ? MOE_PREC_FP16 : MOE_PREC_INT4G64, ((n) <= CT ? (n) : CT), SPB, NA, HALF, KS>(c, ee, out_base); \
    } while (0)
    if (WIDE) {
        if (CT >= 8 && nct > 4) MOEMIX_BODY(8);
        else if (CT >= 4 && nct > 2) MOEMIX_BODY(4);
        else if (CT >= 2 && nct > 1) MOEMIX_BODY(2);
        else MOEMIX_BODY(1);
    } else
    if (CT >= 4 && nct > 3) MOEMIX_BODY(4);
    else if (CT >= 4 && nct > 2) MOEMIX_BODY(3);
    else if (CT >= 2 && nct > 1) MOEMIX_BODY(2);
    else MOEMIX_BODY(1);
#undef MOEMIX_BODY
}

template <bool UP, int CT, bool WIDE, bool HALF, int SPB = spb_for(CT), int KS = 1>
void launch_one(const MfmaArgs& a, dim3 grid, hipStream_t st) {
    const size_t lds_max = lds_bytes_for(CT, SPB, KS, room_for_16bit(CT, SPB, KS) ? 4096 : 2048);
    const size_t lds_bytes = lds_bytes_for(CT, SPB, KS, a.unit_bytes);
    static std::atomic<unsigned long long> configured{0};
    allow_lds((const void*)grouped_mfma_kernel<UP, CT, WIDE, HALF, SPB, KS>, lds_max, configured);
    grouped_mfma_kernel<UP, CT, WIDE, HALF, SPB, KS><<<grid, 256, lds_bytes, st>>>(a);
}

bool any_int8(const DevExperts& ex, int E) {
    for (int e = 0; e < E; ++e)
        if (ex.e[e].prec == MOE_PREC_INT8G64) return true;
    return false;
}

// 128-column steps of a contraction, the last of which may be half a one.
int contraction_steps(int f) { return (f + kKTile - 1) / kKTile; }

// Chunks of at most `cap` rows that P pairs over E experts make: half a chunk more per expert than full ones would be.
int likely_chunks(int P, int E, int cap) { return (2 * P / cap + E + 1) / 2; }

// One step per LDS stage lets a second workgroup share a compute unit and fills the first stage sooner; two halve the
// barriers.  So two steps where every workgroup has a compute unit to itself and its range is long.  Launches, one and two
// steps: 79 columns of workgroups x 4 chunks, 12 steps 43.0, 54.7 us; 6 x 4, 79 steps 142.5, 123.6; 32 x 4, 32 steps 55.9, 51.9;
// 11 x 10, 11 steps 27.1, 26.7; 10 x 2, 19 steps 34.2, 31.8; 38 x 2, 9 steps 20.6, 21.7; 8 x 10, 4 steps 14.4, 15.7; of 52
// launches of 60 to 240 tokens the faster one is taken in all but two, where they differ by 1 %.
// (Up-projections and blocks with 4-bit experts come here with more workgroups than compute units only: prefill_waves.)
bool one_step_per_stage(const MfmaArgs& a, dim3 grid, bool up) {
    if (up || !any_int8(a.ex, a.E)) return true;
    const int chunks = a.direct_expert >= 0 ? (int)grid.y : std::min(a.P, likely_chunks(a.P, a.E, 64));
    return grid.x * chunks > kComputeUnits || a.k_per_split / kKTile <= 10;
}

// Chunks of at most `cap` rows that an even load of P pairs over E experts, k of them per token, makes on average: experts
// that get any rows, and those with more than one, two, .. chunks, rows per expert taken as normal about their mean.  (1500 random
// blocks: within 0.91 to 1.12 of the chunks there were in nine of ten; skewed loads of Zipf 0.6 and 1.2 have up to 1.45 times as many in
// chunks of 32, fewer in chunks of 16.)
double expected_chunks(int P, int E, int k, int cap) {
    const double mean = (double)P / E, share = (double)k / E, sd = std::max(std::sqrt(mean * (1.0 - share)), 1e-6);
    const int T = P / k;                                            // most rows of an expert
    double n = 1.0 - std::pow(1.0 - share, T);
    for (int rows = cap; rows < T; rows += cap) {
        const double more = 0.5 * std::erfc((rows + 0.5 - mean) / (sd * std::sqrt(2.0)));
        if (more < 1e-3) break;
        n += more;
    }
    return E * n;
}

// Teams of wavefronts in a workgroup of a launch with a grid for one: `teams` times as many workgroups then walk 1 / teams of the
// range each.  A workgroup alone on its compute unit takes 0.7 to 1 us per step, whatever it reads (it has one wavefront per SIMD, each a
// chain of LDS round trips and expansion), so where compute units have none, chains get shorter; past that every workgroup more
// stages the same activations again and starts again.  1500 random blocks of up to 32 rows per expert, more than half with an even load, the
// others skewed (gating biases of Zipf 0.6 and 1.2); W = workgroups with one team at the expected chunks, W x steps; time of the whole block
// over that with one team (geometric mean, worst), examples with one, two and four teams (us):
//   one tile, four: while every workgroup has a compute unit, W (whole chunks) <= 64, 0.67, 0.94 (two: 0.84); up to 80 0.87, 1.10 (two: 0.86).
//     60 x 44 61.7, 45.1, 38.8; 66 x 49 67.0, 49.1, 55.4; 13 columns of 4.9 chunks, 33 steps 38.0, 31.8, 37.7.
//   one tile, two: while all run at once, three per compute unit without 16-bit experts (2 W <= 768), two with them (2 W <= 512), short of
//     that by what the chunks may be off, less for long chains, which gain more.  Without: chains of up to 12 steps 0.97, 1.03 up to W 350
//     and 1.05, 1.15 up to 450, longer ones 0.93, 1.01 up to 380 and 1.05, 1.15 up to 450 (304 x 33 77.9, 70.7; 380 x 22 60.7, 55.3;
//     400 x 4 34.6, 37.1).  With: 0.94, 1.01 up to 240 and 1.01, 1.13 up to 300 (160 x 33 56.8, 50.0; 300 x 22 60.7, 65.6).
// Chunks of two tiles: W with at least a chunk per expert and one expert with two.
//   four: they fit beside the staging of codes only.  W <= 64 0.74, 0.95 (two: 0.81); up to 80 0.88, 1.13 (two: 0.82).  64 x 60 81.6, 62.5, 54.5.
//   two: the stages of two teams leave room for one workgroup per compute unit, and a second round costs 10 to 20 %.  So while each has one
//     of its own, W <= 128, and if the chain is short (it gains some 5 % then) also with a chunk more than expected: 0.87, even loads at worst
//     1.02, skewed ones 1.14 (they may have more chunks); up to 150 1.02, 1.19; up to 200 1.10, 1.22.  126 x 40 68.8, 53.7; 150 x 18 42.3, 46.3.
// (By the experts' precisions, resident or not: a call that runs some of them later sums in the same order.)
int teams_for(const MfmaArgs& a, int ct, dim3 grid, int splits) {
    if (a.waves || ct > 2) return 1;
    const int steps = contraction_steps(a.k_per_split), units = kComputeUnits;   // (unsplit: k_per_split is K)
    const auto fits = [&](int teams) {   // every part of every range holds two steps at least
        const auto ok = [&](int n) { return n - (teams - 1) * team_steps(n, teams) >= 2; };
        return ok(steps) && ok(contraction_steps(a.K) - (splits - 1) * steps);
    };
    if (!fits(2)) return 1;
    const bool alone = a.direct_expert >= 0, any16 = alone ? (a.prec16 >> a.direct_expert) & 1 : a.prec16 != 0;
    const double expected = alone ? grid.y : expected_chunks(a.P, a.E, a.top_k, 16 * ct);
    const double chunks = ct == 2 && !alone ? std::max(expected, std::min(a.P, a.E) + 1.0) : expected;
    if ((!any16 || room_for_16bit(ct, spb_for(ct), 4)) && 4 * grid.x * std::round(chunks) <= units && fits(4)) return 4;
    if (ct == 1) return grid.x * chunks <= (any16 ? 240 : steps > 12 ? 380 : 350) ? 2 : 1;
    return 2 * grid.x * (!alone && steps <= 10 ? std::max(chunks, expected + 1) : chunks) <= units ? 2 : 1;
}

template <bool UP, bool WIDE, bool HALF>
void launch_ct_w(const MfmaArgs& a, const LaunchForm& form, int teams, dim3 grid, hipStream_t st) {
    switch (form.ct) {
        case 1:
            if (teams == 4) launch_one<UP, 1, WIDE, HALF, spb_for(1), 4>(a, grid, st);
            else if (teams == 2) launch_one<UP, 1, WIDE, HALF, spb_for(1), 2>(a, grid, st);
            else launch_one<UP, 1, WIDE, HALF>(a, grid, st);
            break;
        case 2:
            if (teams == 4) launch_one<UP, 2, WIDE, HALF, spb_for(2), 4>(a, grid, st);
            else if (teams == 2) launch_one<UP, 2, WIDE, HALF, spb_for(2), 2>(a, grid, st);
            else launch_one<UP, 2, WIDE, HALF>(a, grid, st);
            break;
        case 4:
            if (!HALF && (UP || !WIDE || form.steps_per_stage == 1)) launch_one<UP, 4, WIDE, HALF, HALF ? spb_for(4) : 1>(a, grid, st);
            else launch_one<UP, 4, WIDE || !HALF, HALF>(a, grid, st);
            break;
        default: launch_one<UP, 8, true, true>(a, grid, st); break;
    }
}

uint32_t prec_mask(const DevExperts& ex, int E, int prec) {
    uint32_t m = 0;
    for (int e = 0; e < E; ++e) m |= (uint32_t)(ex.e[e].prec == prec) << e;
    return m;
}

// Weight staging needs 4 KB of LDS per A operand for 16-bit experts, 2 KB for 4-bit ones.
int staging_unit_bytes(const DevExperts& ex, int E, const RowMap& rows) {
    if (rows.direct_expert >= 0) return ex.e[rows.direct_expert].prec == MOE_PREC_FP16 ? 4096 : 2048;
    for (int e = 0; e < E; ++e)
        if (ex.e[e].resident == 1 && ex.e[e].prec == MOE_PREC_FP16) return 4096;
    return 2048;
}

// Wavefronts per workgroup of ffn_prefill.hip for a launch of plan `ct` with `columns` tiles of 128 (down: 256) weight rows and
// splits, 0: not for that kernel.  It takes contractions of whole steps and input rows that end a little before the reach of a
// 32-bit byte offset (and that start on 16-byte boundaries, which the callers see to: copies_tokens in api.hip).
//   8: chunks of up to 256 rows, one workgroup per compute unit.
//   4: chunks of up to 128 rows, two workgroups per compute unit with half the weight rows each: they hide each other's
//      beginning and end, and there are more of them; activations go into LDS twice.  Where 8 wavefronts would not give every
//      compute unit a workgroup (600 tokens, 4 experts of 2048 x 2048, top-1, 4-bit 65 -> 60 us; 80 tokens on each of 4 experts
//      of 1024 x 2816, 4-bit 45.7 -> 42.6, 16-bit 50.7 -> 47.9), not where they would (512 tokens, Mixtral shape, 505, 579).
//      Also up to 76 rows per expert (68 rows, Mixtral shape, 4-bit 368 -> 351, 8-bit 438 -> 417, 16-bit 600 -> 562; 75 rows, 32 experts
//      of 2048 x 1408, 4-bit 112 -> 105; 80 rows 367, 368, half 16-bit of 2048 x 5632 214, 220; 100 rows 405, 413).
//      And with 33 to 64 rows per expert, where a chunk of ffn_mfma.hip holds 64: beside 16-bit experts (250 tokens,
//      Mixtral shape, 662 -> 557; 140 tokens 552 -> 524) and where so many experts have more than 64 that they need two such chunks:
//      loads spread by the square root of rows (1 - k / E), and the line lies 1.7 times that below 65 (250 tokens, Mixtral shape,
//      4-bit 414 -> 350, 8-bit 478 -> 415; half of the experts per token, 110 tokens, 8 experts of 1024 x 7168 78, 86).  Else
//      by w, its workgroups at a chunk per expert; all but
//        - up-projections of one and a half to two rounds of 512, or more than 2.7.  The other kernel, half as many workgroups of
//          twice the work, fills one round with the former, and just past two rounds begins its second.  80 launches, the other
//          kernel's time over this one's, whole blocks: w up to 768 1.04, 1.5 to 2 rounds 0.97, up to 2.7 1.05, beyond 0.99.
//        - down-projections of one and a half to two rounds (0.99; 1.06 elsewhere, 1.1 to 1.5 below half a round, where contractions
//          are long), without 4-bit experts half to two if ranges are long (136 tokens, 8 experts of 4992 x 11648, 8-bit 386,
//          397, 4-bit 344, 325), and those of 600 workgroups and more with ranges of up to 3 steps, which end before the
//          rings pay (0.98; 280 tokens, 32 experts of 1536 x 1280, top-4, 4-bit 86, 90).
//        Of 27 to 32 rows (plan_mfma) only the up-projections, and of those ones of short contractions: there the loads past 64 that
//        long chunks are taken for cost least (480 tokens, 32 experts of 768 x 2816, 4-bit 79 -> 73.5; of 3456 x 3840, skewed, 281, 331).
//      240 random blocks of 33 to 64 rows without 16-bit experts, the other kernel, all on this one, as it is: 1, 0.882, 0.878 in
//      the geometric mean.
int prefill_waves(const MfmaArgs& a, int ct, int columns, bool up) {
    if (ct < 4 || a.K % kKTile || (uint64_t)a.P * a.K * 2 + 8192 >= (1ull << 32)) return 0;
    const bool alone = a.direct_expert >= 0;
    const int E = alone ? 1 : a.E, rows = (a.P + E - 1) / E;
    if (ct > 4) return columns * E * ((rows + 127) / 128) <= (int)kComputeUnits || rows <= 76 ? 4 : 8;
    // (by the experts' precisions, resident or not: a call that runs some of them later sums in the same order)
    if (alone ? (a.prec16 >> a.direct_expert) & 1 : a.prec16 != 0) return 4;
    if (rows > 64 || E * (65 - rows) * (65 - rows) < 3 * rows * (E - (alone ? 1 : a.top_k))) return 4;
    if (rows <= 32 && !(up && a.K <= 12 * kKTile)) return 4;
    const bool all8 = alone ? (a.prec8 >> a.direct_expert) & 1 : a.prec8 == (uint32_t)((1ull << a.E) - 1);
    const int w = 2 * columns * E;
    const int from = !up && all8 && a.k_per_split > 24 * kKTile ? 256 : 768;
    if ((w > from && w <= 1024) || (up && w > 1376)) return 0;
    return !up && w >= 600 && a.k_per_split <= 3 * kKTile ? 0 : 4;
}

// Most rows of a 4-bit or 8-bit expert's chunks in ffn_prefill.hip, 0: 128 and no even split (also where that kernel is not
// run), for a launch of `columns` workgroups per chunk.
// Longer chunks save compute-unit time (a workgroup's codes cost it some 6 to 7 tiles of 16 rows, whatever the rows), not
// latency.  So 128 where such chunks all run side by side; else the length for which rounds of workgroups
// times the time of one come out least, the longer one unless a shorter one saves 5 %.  Loads spread around their mean:
// half of the experts are taken to have an eighth more, half an eighth less (none where every token reaches every expert).
// One expert alone: the same from two rounds on.
int quant_chunk_rows(const RowMap& rows, const MfmaArgs& a, int P, int columns) {
    if (a.waves != 8) return 0;
    const auto chunks = [](int n, int cap) { return (n + cap - 1) / cap; };
    const int units = kComputeUnits;
    const bool alone = rows.direct_expert >= 0, exact = alone || rows.top_k == a.E;
    if (alone && columns * chunks(P, 128) < 2 * units) return 0;
    const int E = alone ? 1 : a.E, n16 = alone ? 0 : __builtin_popcount(a.prec16);
    const int n = chunks(P, E);
    const int spread = exact ? 0 : n / 8;
    const auto halves = [&](int cap) { return chunks(n - spread, cap) + chunks(n + spread, cap); };   // chunks of two experts
    if (!alone && columns * E * halves(128) <= 2 * units) return 128;
    if (n <= 128) return kChunkRows;
    int best = 0, least = 0;
    for (int cap = kChunkRows; cap >= 128; cap -= 64) {
        const int wgs = columns * (n16 * halves(kChunkRows) + (E - n16) * halves(cap)) / 2;
        const int cost = chunks(wgs, units) * (40 + 7 * chunks(2 * n / halves(cap), 16));
        if (!best || 20 * cost < 19 * least) { best = cap; least = cost; }
    }
    return best;
}

int chunk_slots(const RowMap& rows, const MfmaArgs& a, int P, int ct) {
    const int mc = a.waves ? 128 : 16 * ct;
    if (rows.direct_expert >= 0) return (rows.direct_n + mc - 1) / mc;
    // every expert may end with one ragged chunk; those of 16-bit experts in ffn_prefill.hip are never shorter than those of
    // the others (a workgroup that finds no chunk costs some 3 us, at the launch's end)
    // (and no chunk is empty: 4 pairs, 32 experts of 1024 x 2816, 16-bit: block 44.8 -> 32.3 us)
    return std::min(P, P / (a.quant_rows ? a.quant_rows : mc) + a.E);
}

struct Launch {
    MfmaArgs a;
    LaunchForm form;
    dim3 grid;
    int teams;    // grouped_mfma_kernel: teams per workgroup
};

LaunchForm form_of(const MfmaArgs& a, int ct, dim3 grid, int splits, bool up) {
    LaunchForm m;
    m.waves = a.waves;
    m.ct = ct;
    m.quant_rows = a.quant_rows;
    m.half = !a.waves && (a.K % kKTile || ct == 8);
    m.steps_per_stage = a.waves ? 0 : ct == 4 && !m.half && one_step_per_stage(a, grid, up) ? 1 : spb_for(ct);
    m.splits = splits;
    m.steps_per_split = a.k_per_split / kKTile;
    return m;
}

template <bool UP>
void launch_ct(const Launch& l, hipStream_t st) {
    if (l.form.waves) launch_prefill<UP>(l.a, l.grid, st);
    else if (l.form.half) launch_ct_w<UP, true, true>(l.a, l.form, l.teams, l.grid, st);
    else if (any_int8(l.a.ex, l.a.E)) launch_ct_w<UP, true, false>(l.a, l.form, l.teams, l.grid, st);
    else launch_ct_w<UP, false, false>(l.a, l.form, l.teams, l.grid, st);
}

// Splits of a contraction of `f` columns into ranges of whole steps, all of one length but the last, which may be shorter.
int steps_per_split(int steps, int splits) { return (steps + splits - 1) / splits; }
// every range holds two steps at least, the last one included
bool splits_ok(int steps, int splits) { return steps - (splits - 1) * steps_per_split(steps, splits) >= 2; }

}  // namespace

// The two projections are separate instantiations of everything above; the build compiles one object for each
// (MOEMIX_MFMA_UP, MOEMIX_MFMA_DOWN; neither: both in one).
#if !defined(MOEMIX_MFMA_DOWN)

// every contraction range must hold at least two 128-column steps (4-bit codes are fetched in pairs of steps)
// (and a weight matrix spans less than 4 GB: rows are addressed with 32-bit byte offsets from the matrix)
bool mfma_shape_ok(int d, int f) {
    return d % kGroup == 0 && f % kGroup == 0 && d >= 2 * kKTile && f >= 2 * kKTile && (uint64_t)d * (uint64_t)f * 2u < (1ull << 32);
}

// The kernels address the rows of their input (tokens, hidden rows) with 32-bit byte offsets from its start.
bool mfma_rows_ok(int rows, int d, int f) {
    return (uint64_t)rows * (uint64_t)(d > f ? d : f) * 2u < (1ull << 32);
}

// Up to so many pairs the widths of odd multiples of 64 are split into ranges of unequal length where the number of steps
// has no divisor: unsplit, a few workgroups walk the whole contraction one step after another, longer than a
// wavefront per output row takes (two tokens, top-1, 16-bit: 960 x 4672 40.1 us with the shape-agnostic kernels, 53.5
// unsplit, 27.4 here; 320 x 9280 49.6, 79.7, 24.5; 704 x 2432 30.9, 35.1, 23.9).  Every pair counts as a chunk there, up to the number
// of experts: with the splits of one chunk, 10 pairs over 32 experts of 2880 x 2880, 4-bit, took 83 us, unsplit 59, with
// those of ten 57.
// (No more than a launch of 16-row chunks has: of the launches of whole steps only those look at where a range ends.)
constexpr int kUnevenPairs = 16;

MfmaPlan plan_mfma(int P, int d, int f, int E, int k, bool any16) {
    MfmaPlan p;
    const int avg = (P + E - 1) / E;              // rows per expert if the load were even
    p.ct = avg <= 16 ? 1 : avg <= 32 ? 2 : avg <= 64 ? 4 : 8;
    // down-projection: split the contraction until there are enough workgroups for 256 compute units
    const int steps = contraction_steps(f);
    const int down_rows = 64 * (p.ct <= 2 ? kNASmall : 4);
    const int tiles = (d + down_rows - 1) / down_rows, base = tiles * (P / (16 * p.ct) + 1);
    int best = 1, best4 = 0;
    for (int s = 1; s <= 16; ++s)
        // (widths that are no multiple of 128: no more scratch than fits the library's own, so that a block which fits
        // with one range per row still does)
        if (splits_ok(steps, s) && base * s <= 640 &&
            (steps % s == 0 || (half_step_width(d, f) && P <= kUnevenPairs && tiles * std::min(P, E) * s <= 640)) &&
            (s == 1 || !half_step_width(d, f) || (size_t)P * ((size_t)4 * s * d + 2 * d + 2 * f + 64) + 4096 <= MOE_STATIC_SCRATCH_BYTES)) {
            best = s;
            if ((steps / s) % 4 == 0) best4 = s;
        }
    // launches with 128-row chunks: ranges of a multiple of 4 steps can be walked from different places (TileCtx::rot), so a
    // split that gives such ranges is preferred if it keeps at least half the workgroups
    p.down_splits = (p.ct == 8 && best4 * 2 >= best) ? best4 : best;
    // Loads spread about their mean, by the square root of avg (1 - k / E): where at least one expert in ten has more rows than
    // a chunk, two tiles per chunk cost less than second chunks (64 tokens, Mixtral shape, 4-bit 236 -> 199 us, 8-bit 357 -> 276,
    // 16-bit 596 -> 447; 52 tokens 200 -> 188, 314 -> 270, 500 -> 446; 40 tokens 177, 180; 268, 265; 429, 439; half of the
    // experts per token: 26 tokens, 8 experts of 3840 x 4480, 16-bit 153, 162).  From a mean of 15 on where all chunks run side by
    // side (8 experts of 1024 x 2816: 52 tokens 39.4, 41.3, 64 tokens 44.3 -> 42.0), never where twice as many would (32 tokens,
    // 4 experts of 640 x 1024, 4-bit 21.1, 22.3).  (The splits, and with them the workspace, stay those of one tile.)
    // Likewise from 32 to 64 rows, unless all chunks run side by side (Mixtral shape, 110 tokens, 4-bit 266 -> 260, 8-bit 357 -> 348,
    // 16-bit 581 -> 505; 126 tokens 287 -> 268, 380 -> 352, 629 -> 507; 8 experts of 1024 x 2816 46.1, 51.3 and 47.6, 48.8); without
    // 16-bit experts only if the workgroups of the down-projection fill the chip too (124 tokens, 8 experts of 2432 x 4864, 8-bit
    // 98.6, 109.9; 232 tokens, 8 of 2176 x 5376, top-1, 8-bit 109 -> 98).
    const int columns = (f + 63) / 64 * E;
    const auto overflows = [&](int rows) { return avg <= rows && 10 * E * (rows + 1 - avg) * (rows + 1 - avg) <= 17 * avg * (E - k); };
    if (p.ct == 2 && overflows(32) && columns > 512 && !half_step_width(d, f) && (any16 || (d + 127) / 128 * p.down_splits * E >= 384))
        p.ct = 4;
    // (chunks of more than one tile take ranges of one length; so few pairs over one expert never get here)
    if (p.ct == 1 && P > kUnevenPairs && overflows(16) && columns > (avg > 14 ? 128 : 512)) p.ct = 2;
    return p;
}

int fewer_splits(int f, int splits, int P) {
    const int steps = contraction_steps(f);
    do --splits;
    while (splits > 1 && !(splits_ok(steps, splits) && (steps % splits == 0 || P <= kUnevenPairs)));
    return splits;
}

namespace {
Launch up_launch(const DevExperts& ex, int E, const RowMap& rows, int P, const half_t* x, int d, int f, half_t* h, int ct,
                 int32_t* status) {
    Launch l;
    MfmaArgs& a = l.a;
    a.ex = ex; a.offsets = rows.offsets; a.perm = rows.perm; a.top_k = rows.top_k;
    a.direct_expert = rows.direct_expert; a.direct_n = rows.direct_n;
    a.idx = rows.idx; a.P = P;
    a.in = x; a.out = h; a.K = d; a.N = f; a.E = E; a.k_per_split = d; a.split_stride = 0; a.status = status;
    a.unit_bytes = staging_unit_bytes(ex, E, rows);
    a.prec16 = prec_mask(ex, E, MOE_PREC_FP16);
    a.prec8 = prec_mask(ex, E, MOE_PREC_INT8G64);
    a.waves = prefill_waves(a, ct, (f + 127) / 128, true);
    const int up_rows = a.waves ? 16 * a.waves : 32 * (ct <= 2 ? kNASmall : 4);
    a.tiles = (f + up_rows - 1) / up_rows;
    a.quant_rows = quant_chunk_rows(rows, a, P, a.tiles);
    l.grid = dim3(a.tiles, chunk_slots(rows, a, P, ct), 1);
    l.form = form_of(a, ct, l.grid, 1, true);
    l.teams = teams_for(a, ct, l.grid, 1);
    if (l.teams > 1) l.grid.x = a.tiles = (f + up_rows / l.teams - 1) / (up_rows / l.teams);
    return l;
}
}  // namespace

LaunchForm up_form(const DevExperts& ex, int E, const RowMap& rows, int P, int d, int f, int ct, int* teams) {
    const Launch l = up_launch(ex, E, rows, P, nullptr, d, f, nullptr, ct, nullptr);
    if (teams) *teams = l.teams;
    return l.form;
}

void launch_ffn_up_mfma(const DevExperts& ex, int E, const RowMap& rows, int P, const half_t* x, int d, int f, half_t* h,
                        int ct, int32_t* status, hipStream_t st) {
    TraceScope trace(kKernelUp, st);
    launch_ct<true>(up_launch(ex, E, rows, P, x, d, f, h, ct, status), st);
}

#endif
#if !defined(MOEMIX_MFMA_UP)

namespace {
Launch down_launch(const DevExperts& ex, int E, const RowMap& rows, int P, const half_t* h, int d, int f, float* y, int ct,
                   int splits, size_t split_stride, int32_t* status) {
    Launch l;
    MfmaArgs& a = l.a;
    a.ex = ex; a.offsets = rows.offsets; a.perm = nullptr; a.top_k = rows.top_k;
    a.direct_expert = rows.direct_expert; a.direct_n = rows.direct_n;
    a.idx = rows.idx; a.P = P;
    a.in = h; a.out = y; a.K = f; a.N = d; a.E = E; a.k_per_split = steps_per_split(contraction_steps(f), splits) * kKTile; a.split_stride = split_stride;
    a.status = status;
    a.unit_bytes = staging_unit_bytes(ex, E, rows);
    a.prec16 = prec_mask(ex, E, MOE_PREC_FP16);
    a.prec8 = prec_mask(ex, E, MOE_PREC_INT8G64);
    a.waves = prefill_waves(a, ct, (d + 255) / 256 * splits, false);
    const int down_rows = a.waves ? 32 * a.waves : 64 * (ct <= 2 ? kNASmall : 4);
    a.tiles = (d + down_rows - 1) / down_rows;
    a.quant_rows = quant_chunk_rows(rows, a, P, a.tiles * splits);
    l.grid = dim3(a.tiles * splits, chunk_slots(rows, a, P, ct), 1);
    l.form = form_of(a, ct, l.grid, splits, false);
    l.teams = teams_for(a, ct, l.grid, splits);
    if (l.teams > 1) {
        a.tiles = (d + down_rows / l.teams - 1) / (down_rows / l.teams);
        l.grid.x = a.tiles * splits;
    }
    return l;
}
}  // namespace

LaunchForm down_form(const DevExperts& ex, int E, const RowMap& rows, int P, int d, int f, int ct, int splits, int* teams) {
    const Launch l = down_launch(ex, E, rows, P, nullptr, d, f, nullptr, ct, splits, 0, nullptr);
    if (teams) *teams = l.teams;
    return l.form;
}

void launch_ffn_down_mfma(const DevExperts& ex, int E, const RowMap& rows, int P, const half_t* h, int d, int f, float* y,
                          int ct, int splits, size_t split_stride, int32_t* status, hipStream_t st) {
    TraceScope trace(kKernelDown, st);
    launch_ct<false>(down_launch(ex, E, rows, P, h, d, f, y, ct, splits, split_stride, status), st);
}

#endif

}  // namespace moemix
