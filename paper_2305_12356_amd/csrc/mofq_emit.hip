// Tensor-level reduce + format select (Algorithm 1's strict-less rule), and the
// second quantize_layer call of Algorithm 1: emit the codes of the winning format
// with the scales the search chose.  The decision never leaves device memory,
// so a whole model can be processed without a host synchronisation.
#include <algorithm>

#include "mofq_codes.h"
#include "mofq_internal.h"

namespace mofq {

namespace {

// ---- tensor-level reduce + select ---------------------------------------------------

constexpr int kThreads = 256;
constexpr int kNW = kThreads / 64;

// Sums over the units are taken in two stages of a fixed shape, so that a result depends on the
// number of values alone and not on the launch: consecutive chunks of kChunkUnits values and more (one workgroup each),
// then the chunk sums.  Up to kDirectUnits values there is one stage: reading 16 KB per candidate
// in every emitting workgroup costs less than one more launch (2.5 us of host time, about 2 us on
// the device); beyond, the first stage leaves at most kDecideBlocks values.  Layer selection, us, one stage up to
// 1024 / 2048 / 4096 values: fp32 2048 x 1024, one ratio 13.5 / 11.2 / 11.2; bf16 1237 x 5000, 100 ratios 25.3 / 24.3 / 24.3;
// fp32 4000 x 1024 17.2 / 17.2 / 17.1, 4000 x 4096 34.3 / 34.3 / 35.9.
constexpr int64_t kDirectUnits = 2048, kChunkUnits = 1024;
int64_t partial_chunks(int64_t n) {
  return n <= kDirectUnits ? 0 : std::min<int64_t>(kDecideBlocks, (n + kChunkUnits - 1) / kChunkUnits);
}

// every candidate's error, the energy, the sum of the smallest error of every unit
constexpr int kEnergy = MOFQ_MAX_CANDIDATES, kMixed = kEnergy + 1, kSums = kMixed + 1;

struct SumArrays {
  const double* v[kSums];   // packed: the candidates' errors, then the energy if asked for, then the chunk sums of the mixed error
  int32_t n_cand;
  int32_t n_arr;            // arrays in v
  int32_t has_energy;
  int32_t mixed;            // 1: form the per-unit minimum over the candidates' arrays; 2: v's last array holds its chunk sums
};

// Sums of n values of the first n_arr arrays, and of the per-unit minima if asked for, into s_sum.
// One wave per array: a wave reads 1024 values with 16 loads in flight per lane, so the whole is
// one or two memory latencies for the sizes this is called with (32 loads in flight cost every emission registers:
// fp32 4000 x 1024 17.2 -> 20.7 us), and the order is fixed (lane-strided, then the wave sum).  Valid for every thread.
MOFQ_DEV void block_sums(const SumArrays& a, int n_arr, int64_t lo, int64_t n, bool mixed, double (&s_sum)[kSums]) {
  constexpr int U = 16;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int c = wave; c < n_arr; c += kNW) {
    const double* v = a.v[c] + lo;
    double t = 0.0;
    for (int64_t i0 = lane; i0 < n; i0 += U * 64) {
      double e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) e[u] = v[i0 + u * 64 < n ? i0 + u * 64 : i0];
#pragma unroll
      for (int u = 0; u < U; ++u) t += i0 + u * 64 < n ? e[u] : 0.0;
    }
    t = wave_sum(t);
    if (lane == 0) s_sum[c] = t;
  }
  if (mixed && wave == kNW - 1) {   // the last wave is the one with nothing else to do (two formats and their energy)
    double t = 0.0;
    for (int64_t i = lane; i < n; i += 64) {
      // Algorithm 1's rule for one unit: start at infinity, list order, strictly smaller wins
      double min_err = __builtin_inf(), picked = a.v[0][lo + i];
      for (int c = 0; c < a.n_cand; ++c) {
        const double e = a.v[c][lo + i];
        if (e < min_err) { min_err = e; picked = e; }
      }
      t += picked;
    }
    t = wave_sum(t);
    if (lane == 0) s_sum[kMixed] = t;
  }
  __syncthreads();
}

// First stage for the tensors of a launch: workgroup b of a tensor adds its b-th chunk.
struct PartialTensor {
  SumArrays a;
  double* part;             // [kSums][kDecideBlocks]
  int64_t n, chunk;
};
struct PartialArgs {
  int32_t first_block[kEmitBatch];   // unused entries: INT_MAX
  PartialTensor t[kEmitBatch];
  int32_t n;
};

// Index of the tensor that workgroup `block` belongs to (uniform).
MOFQ_DEV int tensor_of(const int32_t (&first_block)[kEmitBatch], int block) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < kEmitBatch; ++i) k += block >= first_block[i] ? 1 : 0;
  return k;
}

static_assert(sizeof(PartialArgs) <= 4096, "kernel arguments");
__global__ __launch_bounds__(kThreads) void decide_partial_kernel(const PartialArgs args) {
  __shared__ double s_sum[kSums];
  const int k = tensor_of(args.first_block, static_cast<int>(blockIdx.x));
  const PartialTensor& t = args.t[k];
  const int b = static_cast<int>(blockIdx.x) - args.first_block[k];
  const int64_t lo = b * t.chunk;
  const int64_t n = (t.n - lo) < t.chunk ? (t.n - lo) : t.chunk;
  block_sums(t.a, t.a.n_arr, lo, n, t.a.mixed != 0, s_sum);
  const int c = threadIdx.x;   // rows of part in the order of t.a.v
  if (c < t.a.n_arr || (c == kMixed && t.a.mixed)) t.part[c * kDecideBlocks + b] = s_sum[c];
}

// The last stage's input and where the outcome goes.
struct Decision {
  SumArrays a;
  int32_t n;                 // values per array
  mofq_result_t* result;     // each optional
  double* tensor_err_out;
  double* energy_out;
  double* mixed_out;
};

// Last stage and Algorithm 1's select: min_error starts at infinity, candidates in list order, a
// candidate wins only if strictly smaller; the first one where none is below infinity
// (non-finite input), in the record and in what is emitted.  Every workgroup that needs the choice
// calls it; `write`: leave the record too.
MOFQ_DEV int decide(const Decision& d, bool write, double (&s_sum)[kSums]) {
  const int nc = d.a.n_cand;
  block_sums(d.a, write ? d.a.n_arr : nc, 0, d.n, write && d.a.mixed == 1, s_sum);
  double min_err = __builtin_inf();
  int best = 0;
  for (int c = 0; c < nc; ++c)
    if (s_sum[c] < min_err) { min_err = s_sum[c]; best = c; }
  if (write && threadIdx.x == 0) {
    const double energy = d.a.has_energy ? s_sum[nc] : 0.0;
    if (d.result) {
      d.result->best = best;
      d.result->n = nc;
      for (int c = 0; c < MOFQ_MAX_CANDIDATES; ++c) d.result->err[c] = (c < nc) ? s_sum[c] : 0.0;
      d.result->ref_energy = energy;
    }
    if (d.tensor_err_out) *d.tensor_err_out = s_sum[0];
    if (d.energy_out) *d.energy_out = energy;
    if (d.mixed_out) *d.mixed_out = s_sum[d.a.mixed == 2 ? d.a.n_arr - 1 : kMixed];
  }
  return __builtin_amdgcn_readfirstlane(best);
}

__global__ __launch_bounds__(kThreads) void decide_kernel(const Decision d) {
  __shared__ double s_sum[kSums];
  decide(d, true, s_sum);
}

// The weight-activation path after the matrix kernels of a group of layers: select from the per-tile partials, the one-unit
// outputs of the chosen format for X and W, and a copy of its codes (16-byte pieces, grid-stride, four in flight per lane).
// Workgroups are dealt to the tensors in proportion to their sizes; each takes its layer's select anew, as the emission does, and
// the first of a layer writes what is not codes.  (A launch of the selects before the copies cost a single layer 5 us: 777 x 3000 x
// 5056 119.8 us, 116.9 so.)
constexpr int kCopyTensors = 2 * kWaGroup;
struct WaFinishLayer {
  Decision d;
  int32_t fmt_slot[MOFQ_MAX_CANDIDATES];
  WaFinishTensor t[2];
};
struct WaFinishArgs {
  WaFinishLayer p[kWaGroup];
  struct {
    const uint8_t* src[2];
    uint8_t* dst;
    int64_t bytes;
    int32_t layer, writes;   // writes: its first workgroup leaves the layer's other outputs
  } t[kCopyTensors];
  int32_t first_block[kCopyTensors + 1];
  int32_t n;
};
static_assert(sizeof(WaFinishArgs) <= 4096, "kernel arguments");
__global__ __launch_bounds__(kThreads) void wa_finish_kernel(const WaFinishArgs a) {
  __shared__ double s_sum[kSums];
  __shared__ double s_red[kNW];
  int k = 0;
  while (k + 1 < a.n && static_cast<int>(blockIdx.x) >= a.first_block[k + 1]) ++k;   // uniform
  const int b = static_cast<int>(blockIdx.x) - a.first_block[k];
  const int nb = a.first_block[k + 1] - a.first_block[k];
  const auto& copy = a.t[k];
  const WaFinishLayer& l = a.p[copy.layer];
  const bool write = b == 0 && copy.writes != 0;   // uniform
  const int f = l.fmt_slot[decide(l.d, write, s_sum)];
  if (write) {
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      const WaFinishTensor& t = l.t[which];
      if (t.n_segments < 1) continue;   // uniform
      double e = 0.0;
      if (t.out_unit_err) {
        for (int i = threadIdx.x; i < t.n_segments; i += kThreads) e += t.sse_part[2 * i + f];
        e = wave_sum(e);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = e;
        __syncthreads();
        e = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
      }
      if (threadIdx.x == 0) {
        if (t.out_unit_err) *t.out_unit_err = e;
        if (t.out_scales) *static_cast<float*>(t.out_scales) = t.scale[f];
        if (t.out_clip) *t.out_clip = 0;
      }
    }
  }
  const uint8_t* const src = f ? copy.src[1] : copy.src[0];
  if (src == copy.dst) return;   // uniform: the codes are in place
  const u32x4* s4 = reinterpret_cast<const u32x4*>(src);
  u32x4* d4 = reinterpret_cast<u32x4*>(copy.dst);
  const int64_t n = copy.bytes / 16;
  const int64_t stride = static_cast<int64_t>(nb) * kThreads;
  int64_t i = static_cast<int64_t>(b) * kThreads + threadIdx.x;
  for (; i + 3 * stride < n; i += 4 * stride) {
    const u32x4 v0 = s4[i], v1 = s4[i + stride], v2 = s4[i + 2 * stride], v3 = s4[i + 3 * stride];
    d4[i] = v0; d4[i + stride] = v1; d4[i + 2 * stride] = v2; d4[i + 3 * stride] = v3;
  }
  for (; i < n; i += stride) d4[i] = s4[i];
}

// ---- emit -------------------------------------------------------------------------
//
// One launch for up to kEmitBatch tensors does all that follows the search: the select (from the
// unit errors or their chunk sums, redone by every workgroup), the winner's codes and its
// per-unit outputs.  Bound by memory: 2 (4) bytes read and half a byte (one) written per element.
// A workgroup walks segments of consecutive 8-element chunks, so that row, column and unit of a
// chunk follow from one division per segment and a 32-bit multiplication per chunk (a 64-bit
// division per chunk costs more instructions than its quantization); addresses are a uniform base
// plus a 32-bit offset, and the units that open in a segment are written together at its end, a
// thread per unit (as a branch of the chunk loop they cost two dependent loads in every wave).
// Measured: a 7B-shaped block with groups of 128 (202 M elements) 193 us -> 113 us, 4.5 TB/s.

struct EmitTensor {
  const void* w;
  int64_t ld, cols, n_chunks;
  uint32_t cpr, magic;       // 8-element chunks per row; row_of()
  int32_t seg_chunks, n_seg; // chunks per segment
  int32_t gran, group_shift; // log2 of the chunks per group
  const float* scale[MOFQ_MAX_CANDIDATES];
  const int32_t* clip[MOFQ_MAX_CANDIDATES];
  const double* err[MOFQ_MAX_CANDIDATES];
  Decision d;                // d.n = 0: candidate 0
  const uint8_t* tag;        // fixup_kernel: [rows], or nullptr: every row holds its final codes
  uint8_t* unit_fmt;         // PER_UNIT: index of each unit's candidate
  mofq_qout_t out;
};
struct EmitArgs {
  int32_t first_block[kEmitBatch];   // unused entries: INT_MAX
  int32_t n;
  int32_t n_cand;
  int32_t fmt[MOFQ_MAX_CANDIDATES];
  int32_t scale_f16_out;
  int32_t as_bf16_values;   // write grid values (bf16, unscaled) instead of codes
  EmitTensor t[kEmitBatch];
  int32_t fix_rows;         // fixup_kernel: rows a workgroup takes at a time (behind the tensors: in front of them it puts what a single
                            // one's workgroups load first on one cache line more, 0.35 us of a launch)
};

// row, counted from the segment's first, of the chunk `off` chunks behind that row's start
MOFQ_DEV uint32_t row_of(const EmitTensor& t, uint32_t off) {
  if (t.magic) return __umulhi(off, t.magic);         // off * cpr < 2^32: exact
  if (t.cpr == 1) return off;
  return off >= t.cpr ? 1u : 0u;                      // rows longer than a segment
}

// Algorithm 1's rule for one unit: start at infinity, list order, strictly smaller wins
MOFQ_DEV int unit_choice(const EmitTensor& t, int n_cand, int64_t unit) {
  double min_err = __builtin_inf();
  int c = 0;
#pragma unroll
  for (int i = 0; i < MOFQ_MAX_CANDIDATES; ++i)
    if (i < n_cand) {
      const double e = t.err[i][unit];
      if (e < min_err) { min_err = e; c = i; }
    }
  return c;
}

template <int FMT> MOFQ_DEV uint32_t grid_pair_bf16(float t0, float t1) {
  // grid values have at most 7 significant bits: exact in bf16 (top half of fp32)
  return (f2u(Codec<FMT>::grid(t0)) >> 16) | (f2u(Codec<FMT>::grid(t1)) & 0xFFFF0000u);
}

// One 8-element chunk, divided by its unit's scale: quantize and store.
template <int FMT>
MOFQ_DEV void emit_chunk(const EmitArgs& a, void* codes, int64_t c0, uint32_t l, const float (&t)[8]) {   // chunk c0 + l; c0 is uniform
  if (a.as_bf16_values) {
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = grid_pair_bf16<FMT>(t[2 * i], t[2 * i + 1]);
    (static_cast<u32x4*>(codes) + c0)[l] = o;
    return;
  }
  uint32_t words[2];
  encode_scaled8<FMT>(t, words);
  if constexpr (Codec<FMT>::BITS == 4) {
    (static_cast<uint32_t*>(codes) + c0)[l] = words[0];
  } else {
    u32x2 o;
    o[0] = words[0];
    o[1] = words[1];
    (static_cast<u32x2*>(codes) + c0)[l] = o;
  }
}

constexpr int kEmitUnroll = 4;   // chunks per thread and iteration: 16-byte loads in flight per lane
// PER_UNIT: every unit takes its own best candidate (its index goes to unit_fmt), else the tensor's.
// MULTI: more than one tensor; a single one's arguments sit at fixed offsets, so that they all come
// with the first round of scalar loads.  A small launch is a chain of memory latencies, so the
// first chunks and the scales of the first two candidates are requested before the select.
template <typename In, bool PER_UNIT, bool MULTI>
__global__ __launch_bounds__(kThreads) void emit_kernel(const EmitArgs a) {
  __shared__ double s_sum[kSums];
  const int k = MULTI ? tensor_of(a.first_block, static_cast<int>(blockIdx.x)) : 0;
  const EmitTensor& t = a.t[k];
  const int b = static_cast<int>(blockIdx.x) - (MULTI ? a.first_block[k] : 0);
  const int nb = (MULTI && k + 1 < a.n ? a.first_block[k + 1] : static_cast<int>(gridDim.x)) - (MULTI ? a.first_block[k] : 0);
  const bool units_out = PER_UNIT || t.out.scales || t.out.clip_idx || t.out.unit_err;
  const bool per_group = t.gran == MOFQ_PER_GROUP, per_channel = t.gran == MOFQ_PER_CHANNEL;
  const bool dense = t.ld == t.cols;
  int best = -1;

  for (int seg = b; seg < t.n_seg; seg += nb) {
    // everything 64-bit is uniform over the workgroup; lanes add 32-bit offsets
    const int64_t c0 = static_cast<int64_t>(seg) * t.seg_chunks;
    const int64_t row0 = c0 / t.cpr;
    const uint32_t off0 = static_cast<uint32_t>(c0 - row0 * t.cpr);
    const int n = static_cast<int>((t.n_chunks - c0) < t.seg_chunks ? (t.n_chunks - c0) : t.seg_chunks);
    // unit of a chunk: its group (segments start at a group), its row, or 0
    const int64_t unit0 = per_group ? c0 >> t.group_shift : (per_channel ? row0 : 0);
    const int64_t src0 = dense ? c0 * 8 : row0 * t.ld;
    const float* const scale0 = t.scale[0] + unit0;
    const float* const scale1 = t.scale[1] + unit0;
    for (int i0 = 0; i0 < n; i0 += kThreads * kEmitUnroll) {   // uniform
      const int l0 = i0 + static_cast<int>(threadIdx.x);
      Raw8<In> raw[kEmitUnroll];
      float sc0[kEmitUnroll], sc1[kEmitUnroll];
      uint32_t unit[kEmitUnroll];                     // counted from unit0
#pragma unroll
      for (int u = 0; u < kEmitUnroll; ++u) {
        const int l = l0 + u * kThreads < n ? l0 + u * kThreads : n - 1;   // past the end: the last again, not stored
        uint32_t q = 0;
        if (per_channel || !dense) q = row_of(t, off0 + static_cast<uint32_t>(l));
        if (dense) raw[u].load(t.w, src0, static_cast<uint32_t>(l) * 8);
        else raw[u].load(t.w, src0 + static_cast<int64_t>(q) * t.ld, (off0 + static_cast<uint32_t>(l) - q * t.cpr) * 8);
        unit[u] = per_group ? static_cast<uint32_t>(l) >> t.group_shift : (per_channel ? q : 0u);
        sc0[u] = scale0[unit[u]];
        sc1[u] = scale1[unit[u]];
      }
      if (best < 0) best = t.d.n > 0 ? decide(t.d, b == 0, s_sum) : 0;   // uniform
      // candidate c for chunk u, whose format is fmt_c
      auto store = [&](auto fmt_c, const int u, const int c) {
        const float s0 = sc0[u], s1 = sc1[u];
        float s = c == 0 ? s0 : s1;
        if (c > 1) s = t.scale[c][unit0 + unit[u]];
        float scaled[8];
        raw[u].scaled(1.0f / s, scaled);
        emit_chunk<decltype(fmt_c)::value>(a, t.out.codes, c0, static_cast<uint32_t>(l0 + u * kThreads), scaled);   // dense output rows
      };
      if constexpr (PER_UNIT) {
#pragma unroll
        for (int u = 0; u < kEmitUnroll; ++u) {
          if (l0 + u * kThreads >= n) continue;
          const int c = unit_choice(t, a.n_cand, unit0 + unit[u]);
          with_format(a.fmt[c], [&](auto fmt_c) { store(fmt_c, u, c); });
        }
      } else {
        with_format(a.fmt[best], [&](auto fmt_c) {
#pragma unroll
          for (int u = 0; u < kEmitUnroll; ++u)
            if (l0 + u * kThreads < n) store(fmt_c, u, best);
        });
      }
    }
    // outputs of the units that open in this segment, a thread per unit
    if (units_out) {
      const int64_t cpu = per_group ? int64_t{1} << t.group_shift : (per_channel ? t.cpr : t.n_chunks);   // chunks per unit
      const int64_t end = (c0 + n + cpu - 1) / cpu;
      for (int64_t o = (c0 + cpu - 1) / cpu + threadIdx.x; o < end; o += kThreads) {
        int c = best;
        if constexpr (PER_UNIT) {
          c = unit_choice(t, a.n_cand, o);
          t.unit_fmt[o] = static_cast<uint8_t>(c);
        }
        const float s = t.scale[c][o];
        const int32_t clip = t.clip[c][o];
        const double err = t.err[c][o];
        if (t.out.scales) {
          if (a.scale_f16_out)
            static_cast<uint16_t*>(t.out.scales)[o] = __half_as_ushort(__float2half_rn(s));  // exact: s is an fp16 value
          else
            static_cast<float*>(t.out.scales)[o] = s;
        }
        if (t.out.clip_idx) t.out.clip_idx[o] = clip;
        if (t.out.unit_err) t.out.unit_err[o] = err;
      }
    }
  }
}

// After searches that wrote codes ahead (AheadCodes): select, per-unit outputs, and the codes of the
// rows that hold another candidate's.  A workgroup takes fix_rows rows at a time: a thread per row for
// the outputs, then all threads for the chunks of the rows to be done again, as one sequence.  What a row's thread needs of the first two
// candidates is requested before the select.
constexpr int kFixRows = 16;   // at most
template <typename In>
__global__ __launch_bounds__(kThreads) void fixup_kernel(const EmitArgs a) {
  __shared__ double s_sum[kSums];
  __shared__ int s_redo[kFixRows], s_n;
  __shared__ float s_inv[kFixRows];
  const int k = tensor_of(a.first_block, static_cast<int>(blockIdx.x));
  const EmitTensor& t = a.t[k];
  const int b = static_cast<int>(blockIdx.x) - a.first_block[k];
  const int nb = (k + 1 < a.n ? a.first_block[k + 1] : static_cast<int>(gridDim.x)) - a.first_block[k];
  const int64_t rows = t.n_chunks / t.cpr;
  const int tid = threadIdx.x, per = a.fix_rows;
  int best = -1;
  for (int64_t r0 = static_cast<int64_t>(b) * per; r0 < rows; r0 += static_cast<int64_t>(nb) * per) {
    const int64_t o = r0 + tid;
    const bool mine = tid < per && o < rows;
    const int64_t at = mine ? o : r0;
    const float s0 = t.scale[0][at], s1 = t.scale[1][at];
    const int32_t clip0 = t.clip[0][at], clip1 = t.clip[1][at];
    const double err0 = t.err[0][at], err1 = t.err[1][at];
    const int tag = t.tag ? t.tag[at] : 0;
    if (best < 0) best = t.d.n > 0 ? decide(t.d, b == 0, s_sum) : 0;   // uniform
    if (tid < per) {
      bool redo = false;
      float scale = 1.0f;
      if (mine) {
        redo = t.tag && tag != best;
        float s = best == 0 ? s0 : s1;
        int32_t clip = best == 0 ? clip0 : clip1;
        double err = best == 0 ? err0 : err1;
        if (best > 1) { s = t.scale[best][o]; clip = t.clip[best][o]; err = t.err[best][o]; }
        scale = s;
        if (t.out.scales) {
          if (a.scale_f16_out)
            static_cast<uint16_t*>(t.out.scales)[o] = __half_as_ushort(__float2half_rn(s));  // exact: s is an fp16 value
          else
            static_cast<float*>(t.out.scales)[o] = s;
        }
        if (t.out.clip_idx) t.out.clip_idx[o] = clip;
        if (t.out.unit_err) t.out.unit_err[o] = err;
      }
      // the rows to be done again, in any order (per <= 16: one wave)
      const uint64_t again = __builtin_amdgcn_ballot_w64(redo);
      if (redo) {
        const int i = __builtin_popcountll(again & ((uint64_t{1} << tid) - 1));
        s_redo[i] = tid;
        s_inv[i] = 1.0f / scale;
      }
      if (tid == 0) s_n = __builtin_popcountll(again);
    }
    __syncthreads();
    const uint32_t n = static_cast<uint32_t>(s_n) * t.cpr;   // their chunks, one row behind the other
    if (n > 0) {   // uniform
      with_format(a.fmt[best], [&](auto fmt_c) {
        for (uint32_t l0 = tid; l0 < n; l0 += kThreads * kEmitUnroll) {
          Raw8<In> raw[kEmitUnroll];
          uint32_t row[kEmitUnroll], chunk[kEmitUnroll];   // the row's place in the list
#pragma unroll
          for (int u = 0; u < kEmitUnroll; ++u) {
            const uint32_t l = l0 + u * kThreads < n ? l0 + u * kThreads : l0;
            row[u] = t.magic ? __umulhi(l, t.magic) : l / t.cpr;   // l * cpr < 2^32
            chunk[u] = l - row[u] * t.cpr;
            raw[u].load(t.w, (r0 + s_redo[row[u]]) * t.ld, chunk[u] * 8);
          }
#pragma unroll
          for (int u = 0; u < kEmitUnroll; ++u)
            if (l0 + u * kThreads < n) {
              float scaled[8];
              raw[u].scaled(s_inv[row[u]], scaled);
              emit_chunk<decltype(fmt_c)::value>(a, t.out.codes, r0 * t.cpr, static_cast<uint32_t>(s_redo[row[u]]) * t.cpr + chunk[u], scaled);
            }
        }
      });
    }
    __syncthreads();   // s_redo is free again
  }
}

struct ClearArgs {
  double* p[kEmitBatch];
  int32_t n;
};
__global__ __launch_bounds__(kTallies * kTallyStride) void clear_kernel(const ClearArgs a) {   // a workgroup per tensor
  a.p[blockIdx.x][threadIdx.x] = 0.0;
}

}  // namespace

namespace {

// The arrays of a reduce (the unit values), and the last stage's view of it; `partial`: a first
// stage leaves its chunk sums in p.part, one row of kDecideBlocks per array in the same order.
SumArrays sum_arrays(const DecideParams& p) {
  SumArrays a{};
  a.n_cand = p.n_cand;
  for (int c = 0; c < p.n_cand; ++c) a.v[a.n_arr++] = p.err[c];
  if (p.energy) {
    a.v[a.n_arr++] = p.energy;
    a.has_energy = 1;
  }
  a.mixed = p.mixed_out ? 1 : 0;
  return a;
}
Decision decision(const DecideParams& p, bool partial) {
  Decision d{};
  d.a = sum_arrays(p);
  if (partial) {
    for (int c = 0; c < d.a.n_arr; ++c) d.a.v[c] = p.part + c * kDecideBlocks;
    if (d.a.mixed) {
      d.a.v[d.a.n_arr++] = p.part + kMixed * kDecideBlocks;
      d.a.mixed = 2;
    }
  }
  d.n = static_cast<int32_t>(partial ? partial_chunks(p.units) : p.units);
  d.result = p.result;
  d.tensor_err_out = p.tensor_err_out;
  d.energy_out = p.energy_out;
  d.mixed_out = p.mixed_out;
  return d;
}

bool two_stages(const DecideParams& p) { return p.part && partial_chunks(p.units) > 0; }

// First stages of the reduces that have one, in one launch.
int launch_partial(const DecideParams* const* p, int n, hipStream_t st) {
  PartialArgs a{};
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    if (!two_stages(*p[i])) continue;
    PartialTensor& t = a.t[a.n];
    t.a = sum_arrays(*p[i]);
    t.part = p[i]->part;
    t.n = p[i]->units;
    const int64_t nc = partial_chunks(t.n);
    t.chunk = (t.n + nc - 1) / nc;
    a.first_block[a.n++] = blocks;
    // every chunk sum is written, also where rounding the chunk up leaves the last ones empty
    blocks += static_cast<int>(nc);
  }
  for (int i = a.n; i < kEmitBatch; ++i) a.first_block[i] = INT32_MAX;
  if (!a.n) return MOFQ_OK;
  hipLaunchKernelGGL(decide_partial_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

}  // namespace

int launch_wa_finish(const WaFinishParams* p, int n, hipStream_t st) {
  if (!p || n < 1 || n > kWaGroup) return MOFQ_ERR_INVALID_ARG;
  WaFinishArgs a{};
  int64_t want[kCopyTensors];
  int64_t total = 0;
  for (int i = 0; i < n; ++i) {
    const DecideParams& d = p[i].d;
    if (d.units < 1 || d.n_cand < 1 || d.n_cand > MOFQ_MAX_CANDIDATES || !d.result || !p[i].codes[1].dst) return MOFQ_ERR_INVALID_ARG;
    for (int c = 0; c < d.n_cand; ++c) {
      if (!d.err[c] || p[i].fmt_slot[c] < 0 || p[i].fmt_slot[c] > 1) return MOFQ_ERR_INVALID_ARG;
      a.p[i].fmt_slot[c] = p[i].fmt_slot[c];
    }
    a.p[i].d = decision(d, false);
    a.p[i].t[0] = p[i].t[0];
    a.p[i].t[1] = p[i].t[1];
    for (int which = 0; which < 2; ++which) {
      const WaCopyTensor& t = p[i].codes[which];
      if (!t.dst) continue;
      if (t.bytes < 16 || t.bytes % 16 != 0 || !t.src[0] || !t.src[1]) return MOFQ_ERR_INVALID_ARG;
      const int k = a.n++;
      a.t[k] = {{t.src[0], t.src[1]}, t.dst, t.bytes, i, which};
      want[k] = (t.bytes / 16 + kThreads * 4 - 1) / (kThreads * 4);
      total += want[k];
    }
  }
  const int64_t cap = 256 * 8;
  for (int k = 0; k < a.n; ++k) {
    const int64_t nb = total <= cap ? want[k] : std::max<int64_t>(1, want[k] * cap / total);
    a.first_block[k + 1] = a.first_block[k] + static_cast<int32_t>(nb);
  }
  hipLaunchKernelGGL(wa_finish_kernel, dim3(static_cast<unsigned>(a.first_block[a.n])), dim3(kThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

int launch_decide(const DecideParams& p, hipStream_t st) {
  if (p.units < 1 || p.units > (int64_t{1} << 31) * (two_stages(p) ? kChunkUnits : 1) - 1) return MOFQ_ERR_INVALID_ARG;
  const DecideParams* list[1] = {&p};
  const int rc = launch_partial(list, 1, st);
  if (rc != MOFQ_OK) return rc;
  hipLaunchKernelGGL(decide_kernel, dim3(1), dim3(kThreads), 0, st, decision(p, two_stages(p)));
  return hip_status(hipGetLastError());
}

namespace {

// Kernel arguments of an emission (segments and everything else but the workgroups), and the first
// stages of its reduces.
int prepare_emit(const EmitParams* p, int n, EmitArgs& a, hipStream_t st) {
  if (!p || n < 1 || n > kEmitBatch) return MOFQ_ERR_INVALID_ARG;
  static_assert(sizeof(EmitArgs) <= 4096 && MOFQ_MAX_CANDIDATES >= 2, "kernel arguments");
  a = EmitArgs{};
  const DecideParams* dec[kEmitBatch];
  int n_dec = 0;
  // Segments of 512 to 2048 chunks: the largest that still give 1024 workgroups (4 on each of
  // 256 compute units); more of them would only repeat the select more often.
  int64_t total_chunks = 0;
  for (int i = 0; i < n; ++i) total_chunks += p[i].rows * (p[i].cols / 8);
  const int64_t per_thread = std::min<int64_t>(8, std::max<int64_t>(2, total_chunks / (1024 * kThreads)));
  a.n = n;
  a.n_cand = p[0].n_cand;
  a.scale_f16_out = p[0].scale_f16_out;
  a.as_bf16_values = p[0].as_bf16_values;
  for (int c = 0; c < MOFQ_MAX_CANDIDATES; ++c) a.fmt[c] = p[0].fmt[c];
  for (int i = 0; i < n; ++i) {
    const EmitParams& q = p[i];
    if (q.dtype != p[0].dtype || q.n_cand != a.n_cand || q.scale_f16_out != a.scale_f16_out || q.as_bf16_values != a.as_bf16_values || (q.unit_fmt != nullptr) != (p[0].unit_fmt != nullptr) ||
        q.rows < 1 || q.cols < 8 || q.cols % 8 != 0 || !q.out.codes || q.n_cand < 1 || q.n_cand > MOFQ_MAX_CANDIDATES)
      return MOFQ_ERR_INVALID_ARG;
    EmitTensor& t = a.t[i];
    // a dense per-tensor tensor is one run of chunks: rows of one chunk, whatever its shape
    const bool run = q.gran == MOFQ_PER_TENSOR && q.ld == q.cols;
    if (!run && q.cols >= (int64_t{1} << 31)) return MOFQ_ERR_UNSUPPORTED;
    t.w = q.w;
    t.ld = run ? 8 : q.ld;
    t.cols = run ? 8 : q.cols;
    t.cpr = static_cast<uint32_t>(t.cols / 8);
    t.n_chunks = q.rows * (q.cols / 8);
    // exact while off * cpr < 2^32, off < cpr + 2048; longer rows span a segment
    t.magic = (t.cpr > 1 && t.cpr < 32768) ? static_cast<uint32_t>((uint64_t{1} << 32) / t.cpr + 1) : 0;
    t.seg_chunks = static_cast<int32_t>(per_thread * kThreads);
    const int64_t n_seg = (t.n_chunks + t.seg_chunks - 1) / t.seg_chunks;
    if (n_seg >= (int64_t{1} << 31)) return MOFQ_ERR_UNSUPPORTED;
    t.n_seg = static_cast<int32_t>(n_seg);
    t.gran = q.gran;
    if (q.gran == MOFQ_PER_GROUP) {
      if (q.group < 8 || q.group > 4096 || (q.group & (q.group - 1)) != 0) return MOFQ_ERR_UNSUPPORTED;
      while ((8 << t.group_shift) < q.group) ++t.group_shift;   // segments hold whole groups: 512 chunks and more
    }
    for (int c = 0; c < q.n_cand; ++c) { t.scale[c] = q.scale[c]; t.clip[c] = q.clip[c]; t.err[c] = q.err[c]; }
    if (q.n_cand < 2) { t.scale[1] = q.scale[0]; t.clip[1] = q.clip[0]; t.err[1] = q.err[0]; }   // requested early, not used
    if (q.decide.units > 0) {
      t.d = decision(q.decide, two_stages(q.decide));
      dec[n_dec++] = &q.decide;
    }
    t.tag = q.tag;
    t.unit_fmt = q.unit_fmt;
    t.out = q.out;
  }
  for (int i = n; i < kEmitBatch; ++i) a.first_block[i] = INT32_MAX;
  return n_dec ? launch_partial(dec, n_dec, st) : static_cast<int>(MOFQ_OK);
}

// Workgroups: `want` per tensor, or their share of `cap` where they exceed it; returns the total.
unsigned deal_blocks(EmitArgs& a, const int64_t* want, int64_t cap) {
  int64_t total = 0, blocks = 0;
  for (int i = 0; i < a.n; ++i) total += want[i];
  for (int i = 0; i < a.n; ++i) {
    a.first_block[i] = static_cast<int32_t>(blocks);
    blocks += total <= cap ? want[i] : std::max<int64_t>(1, want[i] * cap / total);
  }
  return static_cast<unsigned>(blocks);
}

}  // namespace

int launch_emit(const EmitParams* p, int n, int max_blocks, hipStream_t st) {
  EmitArgs a;
  const int rc = prepare_emit(p, n, a, st);
  if (rc != MOFQ_OK) return rc;
  int64_t want[kEmitBatch];
  for (int i = 0; i < n; ++i) want[i] = a.t[i].n_seg;
  const dim3 grid(deal_blocks(a, want, max_blocks > 0 ? max_blocks : int64_t{1} << 30));
  const bool per_unit = p[0].unit_fmt != nullptr;
#define MOFQ_EMIT(IN)                                                                                                \
  if (per_unit && n == 1) hipLaunchKernelGGL((emit_kernel<IN, true, false>), grid, dim3(kThreads), 0, st, a);          \
  else if (per_unit) return MOFQ_ERR_UNSUPPORTED;                                                                     \
  else if (n == 1) hipLaunchKernelGGL((emit_kernel<IN, false, false>), grid, dim3(kThreads), 0, st, a);                \
  else hipLaunchKernelGGL((emit_kernel<IN, false, true>), grid, dim3(kThreads), 0, st, a);
  switch (p[0].dtype) {
    case MOFQ_F32: MOFQ_EMIT(F32) break;
    case MOFQ_F16: MOFQ_EMIT(F16) break;
    case MOFQ_BF16: MOFQ_EMIT(BF16) break;
    default: return MOFQ_ERR_INVALID_ARG;
  }
#undef MOFQ_EMIT
  return hip_status(hipGetLastError());
}

int launch_fixup(const EmitParams* p, int n, int max_blocks, hipStream_t st) {
  for (int i = 0; i < n; ++i)
    if ((!p[i].tag && p[i].n_cand > 1) || p[i].gran != MOFQ_PER_CHANNEL || p[i].unit_fmt || p[i].as_bf16_values) return MOFQ_ERR_INVALID_ARG;
  EmitArgs a;
  const int rc = prepare_emit(p, n, a, st);
  if (rc != MOFQ_OK) return rc;
  // few rows: fewer at a time, for more workgroups
  int64_t rows = 0, want[kEmitBatch];
  for (int i = 0; i < n; ++i) rows += p[i].rows;
  a.fix_rows = static_cast<int32_t>(std::min<int64_t>(kFixRows, std::max<int64_t>(2, rows / 512)));
  for (int i = 0; i < n; ++i) want[i] = (p[i].rows + a.fix_rows - 1) / a.fix_rows;
  const dim3 grid(deal_blocks(a, want, max_blocks > 0 ? max_blocks : 256 * 8));
  switch (p[0].dtype) {
    case MOFQ_F32: hipLaunchKernelGGL(fixup_kernel<F32>, grid, dim3(kThreads), 0, st, a); break;
    case MOFQ_F16: hipLaunchKernelGGL(fixup_kernel<F16>, grid, dim3(kThreads), 0, st, a); break;
    case MOFQ_BF16: hipLaunchKernelGGL(fixup_kernel<BF16>, grid, dim3(kThreads), 0, st, a); break;
    default: return MOFQ_ERR_INVALID_ARG;
  }
  return hip_status(hipGetLastError());
}

int launch_clear(double* const* p, int n, hipStream_t st) {
  if (!p || n < 1 || n > kEmitBatch) return MOFQ_ERR_INVALID_ARG;
  ClearArgs a{};
  a.n = n;
  for (int i = 0; i < n; ++i) a.p[i] = p[i];
  hipLaunchKernelGGL(clear_kernel, dim3(static_cast<unsigned>(n)), dim3(kTallies * kTallyStride), 0, st, a);
  return hip_status(hipGetLastError());
}

}  // namespace mofq
