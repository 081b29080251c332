// Host-callable launchers of the moemix kernels (internal to the library).
#pragma once

#include "common.hpp"

namespace moemix {

// How the matrix kernels find their rows.
//   grouped: rows [offsets[e], offsets[e+1]) of the grouped order belong to expert e; grouped row r
//            reads token perm[r] / top_k of x.
//   direct : one given expert, rows 0..n-1 of x in order (moe_expert_ffn_mixed).
struct RowMap {
    const int32_t* offsets;  // device [E+1] or nullptr (direct)
    const int32_t* perm;     // device [P] or nullptr (direct)
    int top_k;
    int direct_expert;       // >= 0: direct mode
    int direct_n;
    // few pairs (group_inline_ok): the routing result [P] itself, from which every workgroup works out the grouping
    // that offsets and perm would tell it (those are not read then)
    const int32_t* idx = nullptr;
};

// Up to kInlinePairs pairs in launches with at most 32 rows per chunk, the kernels that need the grouping work it out
// from the routing result with ballots over up to four 64-lane registers of expert indices: a fraction of a microsecond in
// each of three launches in place of a launch of its own, 2.2 - 4.7 us.  Block with the grouping inside and launched:
// 32 pairs, 1024 x 2816, 30.6, 32.9 us; 128 pairs, 32 experts of 2048 x 1408, 85.0, 86.1; 256 pairs, 8 experts of 1024 x 2816,
// 47.8, 49.5.  The line lies where the gain ends: 256 pairs over 32 experts, a ballot per register and expert in every
// workgroup, 86.7, 86.9 (2048 x 1408) and 32.7, 32.4 (256 x 512).
constexpr int kInlinePairs = 256;
inline bool group_inline_ok(int P, int ct) { return P <= kInlinePairs && ct <= 2; }

// rms_gain != null: the gating input is RMSNorm(x) * rms_gain (fp16).  xn != null: the gating input is also written there [T, d].
void launch_route(const half_t* x, const half_t* wg, const float* bias, int T, int d, int E, int k, int32_t* idx,
                  float* gate, int32_t* idx2, float* gate2, int32_t* status, hipStream_t st,
                  const half_t* rms_gain = nullptr, float eps = 0.0f, half_t* xn = nullptr);
void launch_permute(const int32_t* idx, int P, int E, int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv,
                    int32_t* status, hipStream_t st);

// h[r, :] = silu(W1 x_r) * (W3 x_r) for every row of every expert that has rows.
void launch_ffn_up(const DevExperts& ex, int E, const RowMap& rows, const half_t* x, int d, int f, half_t* h,
                   int32_t* status, hipStream_t st);
// y[r, :] = W2 h[r, :]
void launch_ffn_down(const DevExperts& ex, int E, const RowMap& rows, const half_t* h, int d, int f, float* y,
                     int32_t* status, hipStream_t st);

// Matrix-core path for many rows (contraction lengths multiples of 64, at least 256).  `ct` = 16-row activation tiles per
// chunk (1, 2, 4 or 8); the down-projection splits the contraction `splits` ways and writes one partial
// y per split (`split_stride` elements apart), which launch_combine adds up.
// Widths of odd multiples of 64 (half_step_width) take fewer splits where the workspace at hand has no room for the
// plan's: fewer_splits gives the next smaller number that divides the contraction evenly (any that leaves ranges of two
// steps where the P pairs are few enough for the plan to have such).
struct MfmaPlan {
    int ct;
    int down_splits;
};
bool mfma_shape_ok(int d, int f);
bool mfma_rows_ok(int rows, int d, int f);
// P pairs over E experts, k of them per token; any16: one of them is held in 16 bits.  (The splits do not depend on the last two.)
MfmaPlan plan_mfma(int P, int d, int f, int E, int k, bool any16);
inline bool half_step_width(int d, int f) { return (d | f) % 128 != 0; }
int fewer_splits(int f, int splits, int P);
// (x on a 16-byte boundary if up_form(..).waves)
void launch_ffn_up_mfma(const DevExperts& ex, int E, const RowMap& rows, int P, const half_t* x, int d, int f, half_t* h,
                        int ct, int32_t* status, hipStream_t st);
void launch_ffn_down_mfma(const DevExperts& ex, int E, const RowMap& rows, int P, const half_t* h, int d, int f, float* y,
                          int ct, int splits, size_t split_stride, int32_t* status, hipStream_t st);
// How such a launch runs (asked for by the tests: moemix_launch_form in api.hip).
struct LaunchForm {
    int waves;             // ffn_prefill.hip: wavefronts per workgroup; 0: grouped_mfma_kernel
    int ct;                // 16-row activation tiles per chunk of the plan
    int quant_rows;        // ffn_prefill.hip, 8 wavefronts: most rows of a quantized expert's chunks, 0: 128
    int steps_per_stage;   // grouped_mfma_kernel: 128-column steps per LDS stage
    int half;              // ... the variant that takes contractions of any multiple of 64 and ranges of unequal length
    int splits;            // ranges of the contraction
    int steps_per_split;   // 128-column steps of each, the last one may have fewer where `half` or ct == 1
};
// (teams: grouped_mfma_kernel, teams of wavefronts that share the contraction range of a workgroup)
LaunchForm up_form(const DevExperts& ex, int E, const RowMap& rows, int P, int d, int f, int ct, int* teams = nullptr);
LaunchForm down_form(const DevExperts& ex, int E, const RowMap& rows, int P, int d, int f, int ct, int splits, int* teams = nullptr);

// Batch-1 decode path (one token): shapes it covers, and its two kernels.
bool decode_shape_ok(int d, int f);
// Gating network evaluated inside the up-projection launch (one token): gate matrix [E, d], optional bias,
// optional RMSNorm of the token first (rms_gain != null); the routing result goes to idx_ws / gate_ws [top_k] for
// the down-projection launch and, if wanted, to idx_out / gate_out.  The launch then also clears the status word.
struct GateArgs {
    const half_t* wg;
    const float* bias;
    int E;
    const half_t* rms_gain;
    float eps;
    int32_t* idx_ws;
    float* gate_ws;
    int32_t* idx_out;
    float* gate_out;
};
// gating == null: the routing result is read from idx [top_k].
void launch_decode_up(const DevExperts& ex, const int32_t* idx, const half_t* x, int d, int f, int k, half_t* h,
                      int32_t* status, int blocks, hipStream_t st, const GateArgs* gating = nullptr);
// out32 != null: the result is written there unrounded (fp32) instead of to `out`.
void launch_decode_down(const DevExperts& ex, const int32_t* idx, const float* gate, const half_t* h, int d, int f,
                        int k, const half_t* residual, half_t* out, int32_t* status, hipStream_t st,
                        float* out32 = nullptr);
// Widths that are no multiple of 2048, a slot at a time: slot_sums[s, :] = W2_s h_s for the slots whose expert the table
// marks runnable.  launch_average_slots then gives launch_decode_down's output, bit for bit, from the slots whose
// expert is in `ran` (bit e: expert e).
void launch_decode_down_slots(const DevExperts& ex, const int32_t* idx, const half_t* h, int d, int f, int k, float* slot_sums,
                              int32_t* status, hipStream_t st);
void launch_average_slots(const float* slot_sums, const int32_t* idx, const float* gate, uint32_t ran, int d, int k, half_t* out,
                          hipStream_t st);
// idx[0] = expert, gate[0] = 1: one expert alone through the batch-1 kernels.
void launch_single_route(int32_t* idx, float* gate, int expert, hipStream_t st);

// out[t, :] = fp16( (residual ? residual[t, :] : 0) + sum_s gate[t, s] * sum_p y[p][inv[t*k + s], :] ),
// p over the `splits` partial results, `split_stride` elements apart.
// inv == null: at most kInlinePairs pairs, their places are worked out from the routing result idx [T, k].
void launch_combine(const float* y, int splits, size_t split_stride, const float* gate, const int32_t* inv, int T, int d,
                    int k, const half_t* residual, half_t* out, hipStream_t st, const int32_t* idx = nullptr);
// dst[i] = sum_p y[p][i] for i < n (n a multiple of 4), p over the `splits` partial results `split_stride` elements apart
void launch_reduce_splits(const float* y, int splits, size_t split_stride, size_t n, float* dst, hipStream_t st);
// dst[i] = src[i]; n a multiple of 8, dst on a 16-byte boundary, src anywhere
void launch_copy_halves(const half_t* src, size_t n, half_t* dst, hipStream_t st);
void launch_zero_words(int32_t* p, int n, hipStream_t st);

void launch_dequant_int4(const DevMat& m, int out, int in, half_t* w, hipStream_t st);
void launch_quantize_int4(const half_t* w, int out, int in, uint8_t* packed, half_t* scale, half_t* zero,
                          hipStream_t st);
// Reads `bytes` (a multiple of 16) of device memory once with streamed 128-bit loads.
void launch_stream_read(const void* src, size_t bytes, uint32_t* sink, int blocks, hipStream_t st);
void launch_dequant_int8(const DevMat& m, int out, int in, half_t* w, hipStream_t st);
void launch_quantize_int8(const half_t* w, int out, int in, uint8_t* codes, half_t* scale, half_t* zero, hipStream_t st);
void launch_synth_fill(half_t* dst, size_t n, size_t first, uint64_t seed, uint64_t stream_id, float scale, int kind,
                       hipStream_t st);

}  // namespace moemix

namespace moemix {

// Kernel ids for moe_trace_kernel (same values as MOE_KERNEL_* in the public header).
enum KernelId { kKernelRoute = 0, kKernelPermute = 1, kKernelUp = 2, kKernelDown = 3, kKernelCombine = 4,
                kKernelStreamRead = 5, kKernelCount = 6 };

// One-shot event bracket around the next launch of a given kernel on this thread.
void trace_arm(int kernel, hipEvent_t start, hipEvent_t stop);
void trace_disarm(int kernel);
bool trace_armed(int kernel);
struct TraceScope {
    int kernel;
    hipStream_t st;
    TraceScope(int kernel, hipStream_t st);
    ~TraceScope();
};

}  // namespace moemix
