/*
 * mofq.h -- C ABI of the MI355X (gfx950) library for the hot path of
 * Mixture-of-Formats Quantization (arXiv 2305.12356): quantize a layer's
 * weights (and, for weight-activation quantization, its input activations) to
 * each candidate format of one bit-width, score each candidate, keep the best.
 *
 * Conventions, valid for every entry point:
 *   - Tensors are row-major with the input dimension contiguous:
 *     W = [out_features, in_features], X = [tokens, in_features]
 *     (the linear layer A_out = W * A_in of Section 3.2).
 *   - Every pointer is a DEVICE pointer unless the comment says HOST.  The
 *     caller owns all memory; the library allocates none, keeps no pointer
 *     after the call and has no global state (two exceptions, stated there:
 *     mofq_select_layer_static and its built-in workspace, and the count that
 *     numbers the calls of mofq_quantize).
 *   - Calls only enqueue work on `stream` (a hipStream_t passed as void*;
 *     NULL = the default stream) and never synchronise: results, including the
 *     chosen format, land in device memory.
 *   - Return value: MOFQ_OK or a negative mofq_status_t.  Arguments are checked
 *     on the host before anything is enqueued, so a failed call has no effect.
 *   - Inputs must be finite; behaviour on NaN/Inf input is unspecified.
 *   - `data` and every output pointer must be 16-byte aligned; `cols` and `ld`
 *     must be multiples of 8 elements.
 *
 * Arithmetic (the paper leaves it open; this is the reading both this library
 * and its CPU oracle implement):
 *   unit   = one tensor, one output channel (row), or `group_size` consecutive
 *            elements of a row;
 *   a      = max |x| over the unit;
 *   s_k    = fl32(fl32(r_k * a) / qmax), qmax = 7 (INT4), 6 (FP4 E2M1),
 *            127 (INT8), 448 (FP8 E4M3); rounded to fp16 (clamped to 65504)
 *            when scale_dtype is MOFQ_F16; a scale below 2^-126 becomes 1;
 *   t      = fl32(x * fl32(1 / s_k));
 *   INT    : q = clamp(round-half-even(t), qmin, qmax), two's-complement code;
 *   FP     : nearest value of the format, ties to the even code, saturating,
 *            sign bit of the code = sign bit of t (E2M1 is Table 1's row without
 *            NaN/Inf: 0 .5 1 1.5 2 3 4 6; E4M3 is the 448-max variant with no
 *            infinity);
 *   error  = sum over the unit of (x - g*s_k)^2 in fp64;
 *   search = first clip candidate with the smallest unit error;
 *   select = first candidate format with the smallest tensor (or layer-output)
 *            error, strict '<' as in Algorithm 1.
 */
#ifndef MOFQ_H_
#define MOFQ_H_

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Candidate formats (Section 3.2: FP4 = E2M1, FP8 = E4M3; Section 4.2 / Table 1
 * for the E2M1 value set). */
typedef enum {
  MOFQ_INT4 = 0,
  MOFQ_FP4_E2M1 = 1,
  MOFQ_INT8 = 2,
  MOFQ_FP8_E4M3 = 3,
  /* The IEEE-aligned FP4 of Table 1 (row "w/ NaN&Inf"): the same codes 0..5 (0 .. 3),
   * codes 6 and 7 are Inf / NaN and never produced; values beyond 3 saturate at 3.
   * The comparison format of Section 4.2. */
  MOFQ_FP4_E2M1_IEEE = 4,
  /* The other 8-bit floating-point option named in Section 2.2: sign / 5 exponent bits
   * (bias 15) / 2 mantissa bits, subnormals m*2^-16, largest finite value 57344;
   * saturating (Inf / NaN codes are never produced).  Scored and emitted like any
   * other format; the W8A8 layer-output metric takes only MOFQ_INT8 / MOFQ_FP8_E4M3. */
  MOFQ_FP8_E5M2 = 5
} mofq_format_t;

typedef enum { MOFQ_F32 = 0, MOFQ_F16 = 1, MOFQ_BF16 = 2 } mofq_dtype_t;

/* Scale granularity: per-tensor (activations, Section 3.2), per-channel
 * (weights, Section 3.2), per-group along the input dimension. */
typedef enum { MOFQ_PER_TENSOR = 0, MOFQ_PER_CHANNEL = 1, MOFQ_PER_GROUP = 2 } mofq_gran_t;

/* Error metric of Algorithm 1's compute_error (Section 4.1): error of the
 * quantized tensor itself, or of the layer output with quantized inputs. */
typedef enum {
  MOFQ_ERR_TENSOR = 0,
  MOFQ_ERR_LAYER_OUTPUT = 1,
  /* Same quantity, but the FP8-E4M3 code product is taken on the fp8 matrix cores
   * instead of being formed from the (bf16-exact) grid values on the bf16 matrix
   * cores: half the matrix time of that product.  Inside one instruction the unit aligns
   * the 8 products of each group of 8 consecutive k to the group's largest exponent sum
   * and drops (towards zero) what lies more than 13 bits below it, which hurts where a group
   * holds an outlier channel of the activation.  With candidates {INT8, FP8_E4M3} and
   * per-tensor weight scales the library therefore splits those columns off (up to 64
   * columns whose largest magnitude is more than 4 times the typical column's) and adds
   * their share of the sum by one exact K step on the bf16 matrix cores: the FP8 error sum
   * is then within 1e-5 of the exact form (measured 4e-7 at most on 2048-token
   * LLaMA-shaped layers, 1e-6 on layers of some ten thousand outputs; layers of a few
   * thousand outputs keep a random part of about 1e-3 / sqrt(tokens * out_features)).
   * With other candidate lists or per-channel weight scales nothing is split off and
   * the deviation is 1e-6 .. 3e-5 at full size, up to 1e-4 on small layers.  The INT8
   * product and the reference energy are exact in both modes. */
  MOFQ_ERR_LAYER_OUTPUT_FP8_UNIT = 2,
  /* Layer-output error of the weight-only case (Section 4.1 names tensor error and
   * layer-output error as the two metrics that suffice there): the input stays in 16
   * bits, only W is quantized: sum (X W^T - X Q(W)^T)^2.  Q(W) is the quantization the
   * tensor-error path produces for the format (scales searched over w_cfg's clip
   * ratios by tensor error). */
  MOFQ_ERR_LAYER_OUTPUT_W_ONLY = 3
} mofq_metric_t;

typedef enum {
  MOFQ_OK = 0,
  MOFQ_ERR_INVALID_ARG = -1, /* null pointer, non-positive size, mixed bit-widths, n_clip < 1 ... */
  MOFQ_ERR_UNSUPPORTED = -2, /* dtype / granularity / shape combination not implemented */
  MOFQ_ERR_MISALIGNED = -3,  /* pointer not 16-byte aligned, cols or ld not a multiple of 8 */
  MOFQ_ERR_WORKSPACE = -4,   /* ws_bytes smaller than mofq_workspace_bytes() */
  MOFQ_ERR_HIP = -5          /* a launch failed */
} mofq_status_t;

#define MOFQ_MAX_CLIP 128      /* most clip candidates per call */
#define MOFQ_MAX_CANDIDATES 4  /* most candidate formats per call */

typedef struct {
  const void* data; /* device, 16-byte aligned */
  int32_t dtype;    /* mofq_dtype_t */
  int64_t rows;     /* out_features (W) or tokens (X) */
  int64_t cols;     /* in_features */
  int64_t ld;       /* elements between consecutive rows, >= cols */
} mofq_tensor_t;

typedef struct {
  int32_t gran;             /* mofq_gran_t */
  int32_t group_size;       /* MOFQ_PER_GROUP only: 32, 64, 128 or 256; cols % group_size == 0 */
  int32_t scale_dtype;      /* MOFQ_F32, or MOFQ_F16: the scale is rounded to fp16 before use */
  int32_t n_clip;           /* 1 .. MOFQ_MAX_CLIP */
  const float* clip_ratios; /* HOST array [n_clip], read during the call; candidate order is
                               the tie order (first smallest wins) */
} mofq_scale_cfg_t;

/* Quantized tensor, all device memory, caller-allocated.  Units are numbered
 * row-major: unit = row (per-channel), row*(cols/group)+group (per-group), 0. */
typedef struct {
  void* codes;       /* 4-bit formats: rows*cols/2 bytes, element 2j of a row in the low nibble
                        of byte j (rows are dense, no padding); 8-bit: rows*cols bytes */
  void* scales;      /* [units] float, or fp16 bits when scale_dtype is MOFQ_F16 */
  int32_t* clip_idx; /* [units] index of the chosen clip ratio; may be NULL */
  double* unit_err;  /* [units] error of the chosen candidate; may be NULL */
} mofq_qout_t;

/* Outcome of Algorithm 1 for one layer; device memory. */
typedef struct {
  int32_t best;       /* index into candidates[] of the chosen format; always in range: 0 when no
                         candidate's error is below +inf (non-finite input) */
  int32_t n;          /* number of candidates */
  double err[MOFQ_MAX_CANDIDATES]; /* error sum of squares per candidate */
  double ref_energy;  /* sum x^2 (tensor metric) or sum (X W^T)^2 (layer-output metric):
                         err/ref_energy is the noise-to-signal power ratio of Section 3.2 */
} mofq_result_t;

/*
 * quantize_layer of Algorithm 1 for one tensor and one format: search the
 * clip ratios per unit, then write codes, scales and (optionally) the chosen
 * indices and unit errors.  `tensor_err` (device, may be NULL) receives the
 * tensor error, the sum of the unit errors.
 *
 * A tensor of up to 163840 elements with one scale and one clip ratio takes one
 * launch whose workgroups hand their error sums over in the workspace, marked with
 * a number that the host draws per call from a process-wide count (atomic, so any
 * thread may call).  Calls on one workspace are to be ordered, as everywhere (see
 * mofq_workspace_bytes); where two such calls overlap on one all the same, the codes
 * are right, but scale, clip index, unit error and tensor error of either can stay
 * unwritten, and no error is returned.
 */
int mofq_quantize(const mofq_tensor_t* t, int32_t format, const mofq_scale_cfg_t* cfg,
                  const mofq_qout_t* out, double* tensor_err,
                  void* ws, size_t ws_bytes, void* stream);

/*
 * compute_error of Algorithm 1 for one candidate format.
 *   metric = MOFQ_ERR_TENSOR       : x must be NULL; *err = sum (W - Q(W))^2 with the
 *                                    scale search of w_cfg; *ref_energy = sum W^2.
 *   metric = MOFQ_ERR_LAYER_OUTPUT : x = A_in; W and X are quantized in `format`
 *                                    (X per-tensor, W per w_cfg, which must have
 *                                    n_clip = 1); *err = sum (X W^T - Q(X) Q(W)^T)^2,
 *                                    *ref_energy = sum (X W^T)^2.  W and X must be
 *                                    MOFQ_BF16 and `format` an 8-bit format.
 *   metric = MOFQ_ERR_LAYER_OUTPUT_W_ONLY : x = A_in stays unquantized (MOFQ_BF16, dense
 *                                    rows: ld = cols); W (MOFQ_BF16) is quantized in
 *                                    `format` (4-bit or 8-bit) per w_cfg (per-tensor or
 *                                    per-channel, any n_clip); *err = sum (X W^T -
 *                                    X Q(W)^T)^2, *ref_energy = sum (X W^T)^2.
 * `err` and `ref_energy` are device pointers (ref_energy may be NULL).
 */
int mofq_score(const mofq_tensor_t* w, const mofq_tensor_t* x, int32_t format, int32_t metric,
               const mofq_scale_cfg_t* w_cfg, double* err, double* ref_energy,
               void* ws, size_t ws_bytes, void* stream);

/*
 * Algorithm 1's loop body for one layer: score every candidate (all of one
 * bit-width, visited in list order), keep the first with the strictly smallest
 * error, and emit the layer quantized in that format.
 *   x == NULL : weight-only; metric must be MOFQ_ERR_TENSOR.
 *   x != NULL : weight-activation; metric must be MOFQ_ERR_LAYER_OUTPUT (or its
 *               _FP8_UNIT variant); W and X share the format (8-bit candidates, both
 *               tensors MOFQ_BF16, cols a multiple of 64, w_cfg per-tensor or
 *               per-channel with n_clip = 1, X per-tensor at ratio 1); x_out (may be
 *               NULL) receives X's codes and its one scale.
 *   x != NULL, metric = MOFQ_ERR_LAYER_OUTPUT_W_ONLY : weight-only select by the layer
 *               output on the 16-bit input x (at most 2 candidates; W and X MOFQ_BF16, X
 *               with ld = cols, cols a multiple of 64, w_cfg per-tensor or per-channel);
 *               x_out is ignored.
 * `candidates` is a HOST array.  `result` is device memory.
 */
int mofq_select_layer(const mofq_tensor_t* w, const mofq_tensor_t* x,
                      const int32_t* candidates, int32_t n_candidates, int32_t metric,
                      const mofq_scale_cfg_t* w_cfg, const mofq_qout_t* w_out,
                      const mofq_qout_t* x_out, mofq_result_t* result,
                      void* ws, size_t ws_bytes, void* stream);

/*
 * mofq_select_layer for callers that cannot allocate or hand over a workspace: code under
 * HIP graph capture, tight serving loops, harnesses that forbid hipMalloc.  Weight-only,
 * tensor error (x = NULL, metric = MOFQ_ERR_TENSOR of mofq_select_layer); same arguments
 * otherwise, same kernels, same results bit for bit.  The workspace is an array of
 * MOFQ_STATIC_WORKSPACE_BYTES inside the library's device image (one copy per GPU, held until
 * the process ends); its address is looked up on the first call on a device.  The call
 * allocates nothing (no hipMalloc / hipFree, no allocating library routine) and enqueues no
 * memset.
 *   - Returns MOFQ_ERR_WORKSPACE, with nothing enqueued, when
 *     mofq_workspace_bytes(w, NULL, n_candidates, MOFQ_ERR_TENSOR, w_cfg) exceeds
 *     MOFQ_STATIC_WORKSPACE_BYTES (per-channel scales: up to about 200 000 rows with two
 *     candidates; groups of 128: up to about 26 M elements).
 *   - Every call on a GPU uses that GPU's one array, which keeps the previous call's
 *     contents; nothing in it has to start at zero (every entry is written before it is
 *     read).  Calls that overlap on one GPU (different streams, or different threads without
 *     ordering) race on it: order them on one stream.
 */
#define MOFQ_STATIC_WORKSPACE_BYTES (8u << 20)
int mofq_select_layer_static(const mofq_tensor_t* w, const int32_t* candidates, int32_t n_candidates,
                             const mofq_scale_cfg_t* w_cfg, const mofq_qout_t* w_out,
                             mofq_result_t* result, void* stream);

/*
 * mofq_select_layer for several weight tensors in one call (weight-only, tensor error;
 * Algorithm 1's loop over the layers of a model): the same results, tensor by tensor, as
 * n_layers calls of mofq_select_layer, but the small dependent steps between the search
 * and the code emission (tensor reduce, select, per-unit outputs) of up to 12 tensors share
 * one launch, so a model-wide pass does not pay their latency per tensor, and the tensors
 * of such a batch that have one row length are searched in one launch.
 *   w, w_out : HOST arrays of n_layers descriptors (device buffers inside, as above).
 *   results  : device array of n_layers records.
 *   ev_begin / ev_end (the _timed variant; may be NULL): HOST arrays of n_layers hipEvent_t,
 *   recorded around the search launches (see mofq_select_layers_search_groups).
 * Workspace: mofq_select_layers_workspace_bytes (the tensors' workspaces side by side).
 * Streams: `side_stream` (a hipStream_t of the caller, default priority; may be NULL or equal
 * to `stream`) lets the select and the code emission of a batch run beside the searches of
 * the next batch, which stay on `stream`.  The side work is ordered after the work already
 * on `stream`, and `stream` waits for it before the call returns, so the caller sees
 * single-stream semantics on `stream`; `side_stream` must not be used by another call at the
 * same time.  The library creates two events for the duration of the call and nothing else.
 */
int mofq_select_layers(int32_t n_layers, const mofq_tensor_t* w, const int32_t* candidates,
                       int32_t n_candidates, const mofq_scale_cfg_t* w_cfg, const mofq_qout_t* w_out,
                       mofq_result_t* results, void* ws, size_t ws_bytes, void* stream,
                       void* side_stream);
int mofq_select_layers_timed(int32_t n_layers, const mofq_tensor_t* w, const int32_t* candidates,
                             int32_t n_candidates, const mofq_scale_cfg_t* w_cfg,
                             const mofq_qout_t* w_out, mofq_result_t* results, void* ws,
                             size_t ws_bytes, void* stream, void* side_stream,
                             void* const* ev_begin, void* const* ev_end);
size_t mofq_select_layers_workspace_bytes(int32_t n_layers, const mofq_tensor_t* w,
                                          int32_t n_candidates, const mofq_scale_cfg_t* w_cfg);
/*
 * How mofq_select_layers groups the searches (host only, enqueues nothing): tensors of one
 * row length (cols) and dtype inside a batch, adjacent or not, are searched together (in one
 * launch where the sort-based per-channel search applies, else in consecutive launches).
 * group_first (HOST, n_layers entries) receives, for every tensor, the index of the first
 * tensor of its group.  The _timed variant records ev_begin[] of that first tensor before the
 * group's launch and ev_end[] of the group's last tensor (the largest index) after it, and
 * leaves the other events of the group alone.  What the events enclose is what those of
 * mofq_select_layer_timed do.
 */
int mofq_select_layers_search_groups(int32_t n_layers, const mofq_tensor_t* w, const int32_t* candidates,
                                     int32_t n_candidates, int32_t* group_first);

/*
 * mofq_select_layer with the layer-output metric of the weight-activation case (Section 3.2,
 * layer analysis; Algorithm 1 with W and X sharing the format) for the linear layers of a
 * model in one call: the same results, layer by layer, as n_layers calls of
 * mofq_select_layer(w[i], x[i], ..., metric, ...).
 *   metric   : MOFQ_ERR_LAYER_OUTPUT or MOFQ_ERR_LAYER_OUTPUT_FP8_UNIT.
 *   w, x, w_out, x_out : HOST arrays of n_layers descriptors (device buffers inside); x_out may
 *              be NULL (no activation outputs), else every entry needs codes and scales.
 *   results  : device array of n_layers records.
 *   ev_begin / ev_end (the _timed variant; may be NULL): HOST arrays of n_layers hipEvent_t,
 *              recorded on `stream` immediately before and after each layer's matrix kernel.
 * With candidates {MOFQ_INT8, MOFQ_FP8_E4M3} (either order) and per-tensor weight scales the
 * layers take a fused path in groups of up to 8 consecutive layers (a decoder block): the X
 * and W of a group go through the quantize passes together (two launches; with the fp8 unit a
 * third before them), then the matrix kernels, in which layers of one tile share a launch (two
 * launches where products are cut into pieces; in the _timed variant with events every layer
 * has its own), then one launch for the selects, the one-unit outputs and the copies of the
 * chosen codes; a layer whose activation descriptor equals the previous layer's (the q/k/v or
 * gate/up projections of a block given the same x) reuses its quantized activation.  During the
 * call w_out[i].codes holds W's E4M3 codes before the select; the chosen format's codes are in
 * place when the call's work has finished.  Other candidate lists and per-channel weight scales
 * go layer by layer through the general path of mofq_select_layer.
 * Workspace: mofq_select_layers_wa_workspace_bytes (one group's operands and, where products
 * are cut into pieces, every layer's partial sums, up to 64 MB a layer; not n_layers').
 * Everything is enqueued on `stream`; the library creates no events and keeps no state.
 */
int mofq_select_layers_wa(int32_t n_layers, const mofq_tensor_t* w, const mofq_tensor_t* x,
                          const int32_t* candidates, int32_t n_candidates, int32_t metric,
                          const mofq_scale_cfg_t* w_cfg, const mofq_qout_t* w_out, const mofq_qout_t* x_out,
                          mofq_result_t* results, void* ws, size_t ws_bytes, void* stream);
int mofq_select_layers_wa_timed(int32_t n_layers, const mofq_tensor_t* w, const mofq_tensor_t* x,
                                const int32_t* candidates, int32_t n_candidates, int32_t metric,
                                const mofq_scale_cfg_t* w_cfg, const mofq_qout_t* w_out,
                                const mofq_qout_t* x_out, mofq_result_t* results, void* ws,
                                size_t ws_bytes, void* stream, void* const* ev_begin, void* const* ev_end);
size_t mofq_select_layers_wa_workspace_bytes(int32_t n_layers, const mofq_tensor_t* w, const mofq_tensor_t* x,
                                             int32_t n_candidates, int32_t metric,
                                             const mofq_scale_cfg_t* w_cfg);

/*
 * Format select at a finer granularity than the layer (Section 4.1 leaves it open, the
 * conclusion lists channel-wise / block-wise selection as future work): weight-only,
 * tensor error; every scale unit of w_cfg (a channel or a group; not per-tensor) takes
 * the candidate with its own smallest error -- Algorithm 1's rule per unit, candidates
 * in list order, strictly smaller wins.
 *   unit_format : device, [units] bytes; receives the index into candidates[] per unit.
 *   w_out       : codes (each unit in its own format; all candidates share the bit
 *                 width, so the layout is that of mofq_quantize), scales, clip indices
 *                 and unit errors of the chosen formats.
 *   result      : device; err[c] = tensor error with candidate c used everywhere and
 *                 best = the layer-wise choice, exactly as mofq_select_layer reports.
 *   mixed_err   : device, one double; the tensor error of the mixed assignment (the sum
 *                 of the per-unit minima, never above err[best]).
 * Workspace: mofq_workspace_bytes(w, NULL, n_candidates, MOFQ_ERR_TENSOR, w_cfg), i.e.
 * mofq_select_units_workspace_bytes() (0 for per-tensor scales, which this call does not take).
 */
int mofq_select_units(const mofq_tensor_t* w, const int32_t* candidates, int32_t n_candidates,
                      const mofq_scale_cfg_t* w_cfg, const mofq_qout_t* w_out,
                      uint8_t* unit_format, mofq_result_t* result, double* mixed_err,
                      void* ws, size_t ws_bytes, void* stream);
size_t mofq_select_units_workspace_bytes(const mofq_tensor_t* w, int32_t n_candidates,
                                         const mofq_scale_cfg_t* w_cfg);

/*
 * Static calibration of a dynamic (activation) tensor (Section 3.2, dynamic tensor
 * analysis): the scale is fixed from calibration batches -- the largest magnitude over
 * all of them -- and then used for batches that were not seen.
 *
 * mofq_calibrate_absmax : *absmax = max(*absmax, max |x|).  `absmax` is one device float
 *   that the caller sets to 0 before the first batch and passes to every further one.
 * mofq_select_calibrated : Algorithm 1's loop body for one tensor whose scale comes from
 *   the calibration: per-tensor scale s_f = fl32(absmax / qmax_f) per candidate (the same
 *   expression as every other scale here, ratio 1; s = 1 if that is below 2^-126), tensor
 *   error sum (x - Q_f(x))^2 with values beyond the calibrated range saturating, first
 *   strictly smallest wins.  x_out (may be NULL) receives the codes and the one scale of
 *   the winner; result as in mofq_select_layer (ref_energy = sum x^2).
 * Workspace of both: mofq_workspace_bytes(x, NULL, n_candidates, MOFQ_ERR_TENSOR, cfg) for
 * a per-tensor cfg with one clip ratio (n_candidates = 1 for the calibration call).
 */
int mofq_calibrate_absmax(const mofq_tensor_t* x, float* absmax, void* ws, size_t ws_bytes,
                          void* stream);
int mofq_select_calibrated(const mofq_tensor_t* x, const int32_t* candidates, int32_t n_candidates,
                           const float* absmax, const mofq_qout_t* x_out, mofq_result_t* result,
                           void* ws, size_t ws_bytes, void* stream);

/*
 * mofq_select_layer with two caller-owned hipEvent_t (passed as void*, either may
 * be NULL) recorded on `stream` immediately before and after the error-scoring
 * kernels (the scale search for the tensor metric, the matrix products for the
 * layer-output metric), so that a harness can time the dominant kernel inside its
 * own timed region.  Everything else is identical: where a per-channel search writes the
 * codes as well (one kernel; from 1024 rows on, 8-bit formats from 2048, and as candidates with
 * several clip ratios from 8192), the events enclose that too.
 */
int mofq_select_layer_timed(const mofq_tensor_t* w, const mofq_tensor_t* x,
                            const int32_t* candidates, int32_t n_candidates, int32_t metric,
                            const mofq_scale_cfg_t* w_cfg, const mofq_qout_t* w_out,
                            const mofq_qout_t* x_out, mofq_result_t* result,
                            void* ws, size_t ws_bytes, void* stream,
                            void* ev_score_begin, void* ev_score_end);

/*
 * What the device in front of us sustains, for reading roofline fractions against (not part
 * of the quantization path; Section 1's motivation is the cost of low-bit arithmetic units,
 * and a measurement harness needs the part's own rates beside the published peaks).  Enqueues
 * one register-only micro-kernel (or `iters` plain copies) on `stream`; the caller times it
 * with events.
 *   kind    : MOFQ_CEILING_COPY      copies the first half of `scratch` to the second half,
 *                                    `iters` times; *work = bytes read + written;
 *             MOFQ_CEILING_READ      reads `scratch` (all but its first 128 KB per compute
 *                                    unit) `iters` times and writes nothing; *work = bytes read;
 *             MOFQ_CEILING_FMA_F32 / _F64   `iters` rounds of 16 independent fused
 *                                    multiply-adds per lane, 32 waves per compute unit;
 *                                    *work = floating-point operations;
 *             MOFQ_CEILING_MFMA_BF16 / _INT8 / _FP8   `iters` rounds of 4 independent 32x32
 *                                    matrix instructions per wave (32x32x16 bf16, 32x32x32
 *                                    int8, 32x32x64 e4m3), 32 waves per compute unit;
 *                                    *work = operations (2 per multiply-add).
 *   scratch : device, 16-byte aligned; at least 8 bytes per lane of the launch (64 KB per
 *             compute unit) for the loop kinds, four times that for the read, any size >= 32
 *             bytes for the copy (copy and read should be given far more than the caches hold
 *             to mean anything).  Contents are
 *             overwritten.
 *   work    : HOST, receives the work of the enqueued launches.
 */
typedef enum {
  MOFQ_CEILING_COPY = 0,
  MOFQ_CEILING_FMA_F32 = 1,
  MOFQ_CEILING_FMA_F64 = 2,
  MOFQ_CEILING_MFMA_BF16 = 3,
  MOFQ_CEILING_MFMA_INT8 = 4,
  MOFQ_CEILING_MFMA_FP8 = 5,
  MOFQ_CEILING_READ = 6
} mofq_ceiling_t;
int mofq_device_ceiling(int32_t kind, void* scratch, size_t scratch_bytes, int32_t iters,
                        double* work, void* stream);

/* Bytes of workspace the three calls above need for these arguments (the
 * largest over the three); 0 on invalid arguments.  Workspace contents are
 * scratch: nothing survives a call, calls sharing a workspace must be ordered
 * on one stream. */
size_t mofq_workspace_bytes(const mofq_tensor_t* w, const mofq_tensor_t* x, int32_t n_candidates,
                            int32_t metric, const mofq_scale_cfg_t* w_cfg);

/* Number of scale units of a tensor under a granularity; -1 if invalid. */
int64_t mofq_num_units(int64_t rows, int64_t cols, int32_t gran, int32_t group_size);

/* Static string for a status code. */
const char* mofq_status_string(int status);

#ifdef __cplusplus
}
#endif
#endif /* MOFQ_H_ */
