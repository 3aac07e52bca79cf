// Host-side internal interface between the C ABI (mofq_api.hip) and the kernel
// launchers.  Not part of the public boundary.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/mofq.h"

namespace mofq {

constexpr int kMaxFmt = 2;  // formats scored together in one sweep launch

// Per-unit results of a sweep for up to kMaxFmt formats (device arrays of
// `units` entries each; slot f belongs to fmt[f]).
struct UnitRecords {
  float* scale[kMaxFmt];
  int32_t* clip[kMaxFmt];
  double* err[kMaxFmt];
  double* energy;  // sum x^2 per unit
};

// Codes written by the search itself (per-channel scales, one launch for the whole candidate list):
// every row is emitted while it is at hand, in the format that the tensor's rows favour so far, so
// that the tensor is read once (few rows: each in its own better format); rows whose format turns out not to be the tensor's choice are
// emitted again afterwards (launch_fixup).  What is favoured is a sum over finished rows that
// workgroups read and add to as they come: it decides how many rows are done twice, never the result.
// Every XCD has sums of its own, kTalliesPerXcd of them, so that the traffic stays inside its L2: an
// addition to one place takes some 70 ns and they queue up, and device-wide ones also slow the loads
// (16384 rows: 1.4 ms with one place for the device, 0.30 with 16 such places, 0.25 without).
struct AheadCodes {
  void* codes;              // nullptr: not asked for
  // two formats only (a single one's codes are final):
  uint8_t* tag;             // [rows]: candidate whose codes the row holds
  double* tally;            // [kTallies][kTallyStride]: sums of (error in slot 0 - error in slot 1); zero before the launch.
                            // nullptr: a row takes its own better format
  int32_t cand_of[kMaxFmt]; // launch slot -> candidate index
};

constexpr int kXcds = 8, kTalliesPerXcd = 4, kTallies = kXcds * kTalliesPerXcd;
constexpr int kTallyStride = 16;   // 128 bytes apart

struct SweepParams {
  const void* w;
  int32_t dtype;
  int64_t rows, cols, ld;
  int32_t gran, group;
  int32_t scale_f16;
  int32_t n_clip;
  int32_t n_fmt;          // 1 or 2
  int32_t fmt[kMaxFmt];   // formats, same bit-width
  float clip[MOFQ_MAX_CLIP];
  UnitRecords rec;
  // per-tensor granularity only:
  float* absmax_part;     // [kTensorBlocks]
  double* sse_part;       // [kTensorBlocks][n_fmt][n_clip]
  double* energy_part;    // [kTensorBlocks]
  // per-tensor (INT8, FP8-E4M3) pair with one clip ratio only: the scoring pass also writes
  // the quantized tensor in both formats (dense rows), saving two further reads of the input
  uint8_t* emit_i8;         // int8 codes, or nullptr
  uint8_t* emit_f8;         // e4m3 codes
  // per-channel pair of two different formats (bf16 input) with one clip ratio only: the pass
  // also writes the grid values of format slot f as bf16, dense [rows][cols], to emit_grid[f]
  // (emit_grid_fp8, 4-bit formats: as e4m3 codes, a byte each, at grid_fp8_at() in rows of 2 * cols bytes; emit_grid[f] is the
  // first row's first byte of slot f)
  void* emit_grid[kMaxFmt];
  int32_t emit_grid_fp8;
  AheadCodes ahead;
};

// The grid values of two 4-bit formats as one operand (WA_PAIR_FP8): 128 bytes of a row hold 64 of its columns, the e4m3 codes of the
// first format and then of the second, so that one line of LDS is one step of K.  Pieces of 8 codes; in every second 16 rows the
// two of a 16-byte piece are exchanged: the matrix kernel's reads of 8 bytes by 32 rows then meet no bank twice.
// Byte of a row at which piece c of the first format begins (the second's: 64 further):
constexpr uint32_t grid_fp8_at(uint32_t row, uint32_t c) { return c / 8 * 128 + ((c % 8) ^ (row >> 4 & 1)) * 8; }

constexpr int kTensorBlocks = 1024;  // partial results of per-tensor passes

// Per-tensor scales with one clip ratio (mofq_tensor.hip).
struct TensorParams {
  const void* w;
  int32_t dtype;
  int64_t rows, cols, ld;
  float ratio;
  int32_t scale_f16;
  int32_t n_cand;
  int32_t fmt[MOFQ_MAX_CANDIDATES];
  const float* ext_absmax;       // device, one value, or nullptr: use this magnitude instead of the tensor's own
  float* running;                // device, one value (launch_running_absmax only)
  float* absmax_part;            // scratch, [kTensorBlocks]
  double* sse;                   // scratch, [MOFQ_MAX_CANDIDATES][kTensorBlocks]
  double* energy;                // scratch, [kTensorBlocks]
  mofq_qout_t out;               // members may be nullptr
  mofq_result_t* result;         // optional
  double* tensor_err;            // optional (launch_tensor_quantize)
};
// *running = max(*running, max|x|).
int launch_running_absmax(const TensorParams& p, hipStream_t stream);
// Errors of n_cand formats; then Algorithm 1's select among them, the record and the winner's outputs.
int launch_tensor_scores(const TensorParams& p, hipStream_t stream);
int launch_tensor_pick(const TensorParams& p, hipStream_t stream);
// Codes, scale and error in the one format fmt[0].
int launch_tensor_quantize(const TensorParams& p, hipStream_t stream);

// Enqueue the scale search.  Returns a mofq_status_t.
int launch_sweep(const SweepParams& p, hipStream_t stream);
// Search for groups of 64 and more (4-bit formats, 16-bit inputs) that does not score every element and candidate;
// MOFQ_ERR_UNSUPPORTED (nothing enqueued) elsewhere.
int launch_sweep_group_bits(const SweepParams& p, hipStream_t stream);
// Sort-based search for per-channel 4-bit searches on 16-bit inputs; returns
// MOFQ_ERR_UNSUPPORTED (nothing enqueued) outside that domain.
int launch_sweep_sorted(const SweepParams& p, hipStream_t stream);
// Whether that search takes the histogram kernel (which can write codes ahead).
bool sweep_by_histogram(const SweepParams& p);
// The same for up to kSweepGroupMax tensors of one row length, dtype and configuration in one
// launch (MOFQ_ERR_UNSUPPORTED, nothing enqueued, if they differ or are outside the domain).
constexpr int kSweepGroupMax = 8;
int launch_sweep_sorted_group(const SweepParams* p, int n, hipStream_t stream);
// Scale search of n tensors: one launch where launch_sweep_sorted_group takes them, else one
// launch_sweep per tensor.
int launch_sweep_group(const SweepParams* p, int n, hipStream_t stream);

// Tensor-level reduce + Algorithm 1's strict-less select over n_cand formats
// whose unit errors live in `err[c]` (units entries each).
struct DecideParams {
  int64_t units;
  int32_t n_cand;
  const double* err[MOFQ_MAX_CANDIDATES];
  const double* energy;          // [units] or nullptr
  mofq_result_t* result;         // device, optional
  double* tensor_err_out;        // optional: err of candidate 0 (device) or nullptr
  double* energy_out;            // optional (device) or nullptr
  double* mixed_out;             // optional (device): sum over the units of the smallest candidate's error
  double* part;                  // optional scratch of kDecidePart doubles: with it, many units are
                                 // first reduced by up to kDecideBlocks workgroups
};
constexpr int kDecideBlocks = 256;
constexpr int kDecidePart = (MOFQ_MAX_CANDIDATES + 2) * kDecideBlocks;
int launch_decide(const DecideParams& p, hipStream_t stream);

// Codes and per-unit outputs of up to kEmitBatch tensors of one dtype and candidate list.
struct EmitParams {
  const void* w;
  int32_t dtype;
  int64_t rows, cols, ld;
  int32_t gran, group;
  int32_t scale_f16_out;
  int32_t n_cand;
  int32_t fmt[MOFQ_MAX_CANDIDATES];
  const float* scale[MOFQ_MAX_CANDIDATES];
  const int32_t* clip[MOFQ_MAX_CANDIDATES];
  const double* err[MOFQ_MAX_CANDIDATES];
  DecideParams decide;           // units > 0: the launch takes this reduce + select too and emits its choice; else candidate 0
  const uint8_t* tag;            // launch_fixup: [rows], as the search left it; nullptr with one candidate
  uint8_t* unit_fmt;             // device [units] or nullptr: every unit takes its own best candidate, whose index goes here
  mofq_qout_t out;
  int32_t as_bf16_values;        // out.codes receives the grid values as bf16
};
constexpr int kEmitBatch = 12;
// The same after searches that wrote codes ahead (per-channel scales): per-unit outputs, and the codes
// of the rows whose `tag` is not the choice.
int launch_fixup(const EmitParams* p, int n, int max_blocks, hipStream_t stream);
// Clears the tallies of such searches.
int launch_clear(double* const* p, int n, hipStream_t stream);
// max_blocks: 0, or a cap on the workgroups for emission that runs beside other kernels
int launch_emit(const EmitParams* p, int n, int max_blocks, hipStream_t stream);

// Layer-output error of one linear layer: partial sums per output tile.
// A null xi/wi (or xf/wf) pair skips that format.
// One quantized product of the layer-output kernel: sum_i Gx[t,i] * Gw[o,i], scaled by
// sx * sw[o] in the reduction.  Operand arrays are dense ([M][K] and [N][K]).
enum WaKind : int32_t {
  WA_NONE = 0,
  WA_GRID_BF16 = 1,   // grid values stored as bf16 (exact), bf16 matrix cores
  WA_INT8 = 2,        // int8 codes, int8 matrix cores
  WA_FP8 = 3,         // e4m3 codes, fp8 matrix cores
  WA_PAIR_FP8 = 5,    // both products' w: e4m3 codes of two 4-bit formats in one array (grid_fp8_at), widened as WA_GRID_FP8
  WA_GRID_FP8 = 4,    // e4m3 codes, widened to bf16 on the way to the bf16 matrix cores (exact)
};
struct WaProduct {
  int32_t kind;
  const void* x; const void* w;
  const float* sx;                 // device, one value; nullptr = 1 (unquantized input)
  const float* sw;                 // device, 1 or N values
  double* part;                    // [WaPlan::blocks] squared-difference partials
  // optional second part of the same product (same scales): grid values as bf16, dense
  // [M][kWaSideCols] and [N][kWaSideCols], multiplied on the bf16 matrix cores and added
  const void* xs; const void* ws;
};
struct WaGemmParams {
  const void* x; int64_t ldx;      // bf16 [M][K]
  const void* w; int64_t ldw;      // bf16 [N][K]
  WaProduct q[2];                  // up to two quantized products (kind WA_NONE = unused)
  int32_t w_per_channel;
  int64_t M, N, K;
  double* part_p;                  // [WaPlan::blocks] sum of Y^2
  void* partial;                   // scratch, WaPlan::partial_bytes
};
// How a layer's products are tiled: by its shape alone (the errors' sums depend on it).
struct WaPlan {
  enum : int { kLarge, kMedium, kSmall, kWide };
  int tile;
  bool shared;             // three bf16 products with one X run side by side (wa_gemm_shared_kernel)
  int run;                 // > 0: every product is cut into pieces of up to so many stages (64 sixteen-bit elements of K), each a workgroup's
  int blocks;              // output tiles
  size_t partial_bytes;    // of WaGemmParams::partial
};
WaPlan wa_gemm_plan(int64_t M, int64_t N, int64_t K, int64_t ldx, int64_t ldw);

// The fused weight-activation path (both 8-bit formats as candidates, per-tensor scales)
// works on groups of up to kWaGroup layers: one launch per step for the whole group.
constexpr int kWaGroup = 8;
int launch_wa_gemm(const WaGemmParams& p, hipStream_t stream);
int launch_wa_gemms(const WaGemmParams* p, int n, hipStream_t stream);   // of a group: the layers may share launches

// Pass 1 + 2 over the inputs of the group's layers (up to 2 * kWaGroup tensors, one launch per
// pass): largest magnitude, then both quantized copies and the tensor error of each format.
// A tensor with data == nullptr is skipped (an activation that the previous layer already
// prepared).  The tensor error is left as partial sums over wa_prep_segments() fixed pieces of
// the tensor.
// With the E4M3 codes going to the fp8 matrix cores, the activation's columns of outstanding
// magnitude (outlier channels, Section 3.2) are split off: inside one matrix instruction the
// unit aligns the 8 products of a group of 8 consecutive k to the largest of them and drops
// what falls below its window, so a group that holds an outlier column loses bits of its
// other products.  The split-off columns (at most kWaSideCols) are zeroed in the activation
// operand of the fp8 product and their share of the sum, X[:, cols] W[:, cols]^T, is added by one
// K step on the bf16 matrix cores from the grid values (exact): the same sum, without the loss.
constexpr int kWaSideCols = 64;
struct WaPrepTensor {
  const void* data;          // bf16 [rows][cols], rows `ld` elements apart
  int64_t rows, cols, ld;
  float ratio;               // clip ratio of the scale (1 for activations)
  float* absmax_part;        // [kTensorBlocks]
  double* sse_part;          // [wa_prep_segments(rows, cols)][2]: INT8, E4M3
  uint8_t* q_i8;             // [rows][cols] int8 codes, dense
  uint8_t* q_f8;             // [rows][cols] e4m3 codes, dense
  float* scale;              // [2]: INT8 scale, E4M3 scale
  // column split for the fp8-unit product (all null otherwise)
  int32_t is_x;              // activation: picks the columns; weight: uses its activation's pick
  float* colmax;             // X: [cols] scratch, largest magnitude per column
  uint8_t* col_slot;         // [cols]: slot of a split-off column, 0xFF otherwise (X writes, W reads its X's)
  int32_t* side_cols;        // [kWaSideCols + 1]: the split-off columns in ascending order, then their number
  uint8_t* q_f8_main;        // X: [rows][cols] e4m3 codes with the split-off columns zeroed, dense
  uint16_t* side;            // [rows][kWaSideCols] bf16: e4m3 grid values at the split-off columns, zero beyond their number
};
int wa_prep_segments(int64_t rows, int64_t cols);
int launch_wa_prep(const WaPrepTensor* t, int n, hipStream_t stream);

// After the matrix kernels of a group, one launch: per layer the fixed-order sums of its per-tile partials, Algorithm 1's
// select, the result record, the one-unit outputs (scale, clip index 0, tensor error) of the chosen format for both tensors, and
// its codes into the caller's buffers: a copy of the quantized operand the matrix kernel used (no second quantization).
// Where the chosen format's codes already sit in the destination (src == dst) nothing is moved.
struct WaFinishTensor {
  int32_t n_segments;        // 0: no outputs for this tensor
  const double* sse_part;    // as written by launch_wa_prep
  const float* scale;
  void* out_scales;          // one float; may be nullptr
  int32_t* out_clip;         // may be nullptr
  double* out_unit_err;      // may be nullptr
};
struct WaCopyTensor {
  const uint8_t* src[2];     // INT8 codes, E4M3 codes
  uint8_t* dst;              // nullptr: nothing to do (X only)
  int64_t bytes;             // multiple of 16
};
struct WaFinishParams {
  DecideParams d;                          // err[c] = the tile partials of candidate c's format
  int32_t fmt_slot[MOFQ_MAX_CANDIDATES];   // per candidate: 0 INT8, 1 E4M3
  WaFinishTensor t[2];                     // X, W
  WaCopyTensor codes[2];
};
int launch_wa_finish(const WaFinishParams* p, int n, hipStream_t stream);

inline int hip_status(hipError_t e) { return e == hipSuccess ? MOFQ_OK : MOFQ_ERR_HIP; }

}  // namespace mofq
