// Per-tensor 8-bit quantization of the inputs of linear layers for the layer-output metric of
// the weight-activation case (Section 3.2: A_out = W * A_in with both inputs quantized;
// Section 5: INT8 against FP8-E4M3, activations per tensor).  The activations and weights of a
// group of layers go through every pass together, one launch per pass:
//
//   1. largest magnitude of each tensor (per-workgroup partial maxima);
//   2. both formats at once: the INT8 and the E4M3 codes from one read of the tensor, with
//      the tensor error of each format as partial sums in fp64.
//
// The small dependent steps (folding the partial maxima, the two scales) are redone by every
// workgroup of pass 2 from the partials, so no one-workgroup kernel sits between the passes.
// Nothing is accumulated atomically.  A tensor is cut into a fixed number of segments that
// depends only on its shape; a workgroup takes whole segments and leaves one partial error sum
// per segment, so the sums do not depend on how many workgroups a launch has (which varies
// with how many tensors share it).
#include <algorithm>
#include <type_traits>

#include "mofq_device.h"
#include "mofq_internal.h"

namespace mofq {

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kMaxTensors = 2 * kWaGroup;

struct PrepTensor {
  const uint16_t* data;
  int64_t n_chunks, cpr, ld;   // 8-element chunks in the tensor and per row; elements between rows
  int32_t n_seg;               // segments of the tensor
  int32_t seg_chunks;          // chunks per segment (the last one may be shorter)
  int32_t max_chunks;          // chunks per workgroup of the first pass
  float ratio;                 // clip ratio of the scale
  float* absmax_part;
  int32_t n_absmax;            // partial maxima to fold
  double* sse_part;
  uint8_t* q_i8;
  uint8_t* q_f8;
  float* scale;
  // column split (fp8-unit product); null / 0 otherwise
  int32_t is_x;
  int32_t ld_i32;              // elements between rows (for the column passes)
  int32_t rows_i32, cols_i32;
  float* colmax;
  uint8_t* col_slot;
  int32_t* side_cols;
  uint8_t* q_f8_main;
  uint16_t* side;
};
struct PrepArgs {
  PrepTensor t[kMaxTensors];
  int32_t first_block[kMaxTensors + 1];   // workgroups [first_block[k], first_block[k + 1]) walk tensor k
  int32_t first_side[kMaxTensors + 1];    // quantize pass: behind them, those of the side operands
  int32_t n;
};

// The workgroup's tensor, its index among the tensor's workgroups and their number.
MOFQ_DEV const PrepTensor& my_tensor(const PrepArgs& a, const int32_t (&first)[kMaxTensors + 1], int& k, int& b, int& nb) {
  k = 0;
  while (k + 1 < a.n && static_cast<int>(blockIdx.x) >= first[k + 1]) ++k;   // uniform
  b = static_cast<int>(blockIdx.x) - first[k];
  nb = first[k + 1] - first[k];
  return a.t[k];
}
MOFQ_DEV const PrepTensor& my_tensor(const PrepArgs& a, int& b, int& nb) {
  int k;
  return my_tensor(a, a.first_block, k, b, nb);
}

// Address of chunk c: rows are dense in the outputs, `ld` apart in the input.
MOFQ_DEV const uint16_t* chunk_src(const PrepTensor& t, int64_t c) {
  if (t.ld == t.cpr * 8) return t.data + c * 8;   // uniform: dense input, no division
  const int64_t row = c / t.cpr;
  return t.data + row * t.ld + (c - row * t.cpr) * 8;
}

constexpr int kInFlight = 8;   // 16-byte loads in flight per lane (largest-magnitude pass)

// One chunk in both formats: codes and squared differences.
struct QuantChunk {
  u32x2 i8, f8;
};
MOFQ_DEV QuantChunk quant_chunk(const u32x4 raw, float iA, float iB, double sAd, double sBd, double& accA, double& accB) {
  QuantChunk q;
  float v[8], y[8];
  int wf[2] = {0, 0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = u2f(raw[i] << 16);           // bf16 is the top half of an fp32
    v[2 * i + 1] = u2f(raw[i] & 0xFFFF0000u);
  }
  auto add = [](double& acc, float grid, double s, float x) {
    const double d = __builtin_fma(-static_cast<double>(grid), s, static_cast<double>(x));
    acc = __builtin_fma(d, d, acc);
  };
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    // clamping before rounding gives the same integer; adding 1.5 * 2^23 rounds to nearest even and leaves the
    // two's-complement integer in the low bits (encode_scaled8)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      y[i + h] = med3(v[i + h] * iA, -128.0f, 127.0f) + 12582912.0f;
      add(accA, y[i + h] - 12582912.0f, sAd, v[i + h]);
    }
    // E4M3 through the pack-convert (round to nearest even, subnormals kept; saturating once
    // the input is clamped), which agrees with the codec on every finite fp32 pattern
    const float t0 = med3(v[i] * iB, -448.0f, 448.0f), t1 = med3(v[i + 1] * iB, -448.0f, 448.0f);
    f32x2 g;
    if (i % 4 == 0) {
      wf[i / 4] = __builtin_amdgcn_cvt_pk_fp8_f32(t0, t1, wf[i / 4], false);
      g = __builtin_amdgcn_cvt_pk_f32_fp8(wf[i / 4], false);
    } else {
      wf[i / 4] = __builtin_amdgcn_cvt_pk_fp8_f32(t0, t1, wf[i / 4], true);
      g = __builtin_amdgcn_cvt_pk_f32_fp8(wf[i / 4], true);
    }
    add(accB, g[0], sBd, v[i]);
    add(accB, g[1], sBd, v[i + 1]);
    // one pair at a time: the two fp64 chains are sequential anyway, and scheduling all eight
    // elements of a chunk together costs some 130 registers
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    q.i8[i] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(f2u(y[4 * i + 3]), f2u(y[4 * i + 2]), 0x0C0C0400u),
                                    __builtin_amdgcn_perm(f2u(y[4 * i + 1]), f2u(y[4 * i]), 0x0C0C0400u), 0x05040100u);
    q.f8[i] = static_cast<uint32_t>(wf[i]);
  }
  return q;
}

// E4M3 codes of chunk c less those of the columns that are split off: bit 7 of a column's slot byte set = keep the code
MOFQ_DEV u32x2 without_side(const PrepTensor& t, int64_t c, u32x2 f8) {
  const uint32_t col8 = static_cast<uint32_t>(c) % static_cast<uint32_t>(t.cpr);   // fewer than 2^31 chunks (checked by the host)
  const u32x2 m = reinterpret_cast<const u32x2*>(t.col_slot)[col8];
  u32x2 o;
  o[0] = f8[0] & (((m[0] >> 7) & 0x01010101u) * 0xFFu);
  o[1] = f8[1] & (((m[1] >> 7) & 0x01010101u) * 0xFFu);
  return o;
}
MOFQ_DEV void store_chunk(const PrepTensor& t, int64_t c, const QuantChunk& q) {
  reinterpret_cast<u32x2*>(t.q_i8)[c] = q.i8;
  reinterpret_cast<u32x2*>(t.q_f8)[c] = q.f8;
  if (t.q_f8_main) reinterpret_cast<u32x2*>(t.q_f8_main)[c] = without_side(t, c, q.f8);   // uniform: an activation
}
// Chunks c and c + 1, c even: 16 bytes of codes each
MOFQ_DEV void store_pair(const PrepTensor& t, int64_t c, const QuantChunk& a, const QuantChunk& b) {
  auto both = [](u32x2 p, u32x2 q) { return u32x4{p[0], p[1], q[0], q[1]}; };
  reinterpret_cast<u32x4*>(t.q_i8)[c / 2] = both(a.i8, b.i8);
  reinterpret_cast<u32x4*>(t.q_f8)[c / 2] = both(a.f8, b.f8);
  if (t.q_f8_main) reinterpret_cast<u32x4*>(t.q_f8_main)[c / 2] = both(without_side(t, c, a.f8), without_side(t, c + 1, b.f8));
}

// ---- column split for the fp8-unit product ------------------------------------------------

// Largest magnitude of every column of an activation: a workgroup takes 64 columns, a thread 8
// of them (one 16-byte load per row) on every 32nd row.
__global__ __launch_bounds__(kThreads) void wa_colmax_kernel(const PrepArgs a) {
  __shared__ float s_max[32][65];
  int b, nb;
  const PrepTensor& t = my_tensor(a, b, nb);
  const int tid = threadIdx.x;
  const int cx = tid & 7, ry = tid >> 3;
  const int col0 = b * 64 + cx * 8;          // nb = cols / 64 workgroups
  float m[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) m[i] = 0.0f;
  int r = ry;
  for (; r + 7 * 32 < t.rows_i32; r += 8 * 32) {   // eight loads in flight per lane
    u32x4 raw[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      raw[u] = *reinterpret_cast<const u32x4*>(t.data + static_cast<int64_t>(r + u * 32) * t.ld_i32 + col0);
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        m[2 * i] = __builtin_fmaxf(m[2 * i], __builtin_fabsf(u2f(raw[u][i] << 16)));
        m[2 * i + 1] = __builtin_fmaxf(m[2 * i + 1], __builtin_fabsf(u2f(raw[u][i] & 0xFFFF0000u)));
      }
  }
  for (; r < t.rows_i32; r += 32) {
    float v[8];
    Load8<BF16>::load(t.data + static_cast<int64_t>(r) * t.ld_i32 + col0, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) m[i] = __builtin_fmaxf(m[i], __builtin_fabsf(v[i]));
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) s_max[ry][cx * 8 + i] = m[i];
  __syncthreads();
  if (tid < 64) {
    float r = 0.0f;
#pragma unroll
    for (int y = 0; y < 32; ++y) r = __builtin_fmaxf(r, s_max[y][tid]);
    t.colmax[b * 64 + tid] = r;
  }
}

// Which columns to split off: those whose largest magnitude exceeds kOutlierFactor times the
// typical one, in ascending order, at most kWaSideCols of them.  "Typical" is the mean over the
// columns that do not exceed kOutlierFactor times the mean over all columns, so that the
// outliers themselves do not hide each other where they are many.  One workgroup per
// activation.  (Any choice gives the same sum; the choice only decides how much the fp8 unit's
// alignment can lose.)
constexpr float kOutlierFactor = 4.0f;
//
// A few workgroups beside a pass over the weights, so LDS and registers are left to that: the maxima are read from L2 each time, four
// 16-byte loads in flight per lane.
MOFQ_DEV void pick_columns(const PrepTensor& t) {
  __shared__ double s_sum[2][kThreads / 64];
  __shared__ uint32_t s_cnt[2][kThreads / 64];
  __shared__ float s_amax[kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = t.cols_i32, nv = K / 4;   // K is a multiple of 64
  const u32x4* const col4 = reinterpret_cast<const u32x4*>(t.colmax);
  // f(vector, its four maxima) for the vectors first, first + step, .. of n
  auto each = [&](int first, int step, int n, auto f) {
    for (int i0 = 0; i0 < n; i0 += 4) {
      u32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = col4[i0 + u < n ? first + (i0 + u) * step : first];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u < n) f(first + (i0 + u) * step, v[u]);
    }
  };
  const int strided = tid < nv ? (nv - tid + kThreads - 1) / kThreads : 0;
  double sum = 0.0;
  float amax = 0.0f;
  each(tid, kThreads, strided, [&](int, u32x4 v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sum += static_cast<double>(u2f(v[i]));
      amax = __builtin_fmaxf(amax, u2f(v[i]));
    }
  });
  sum = wave_sum(sum);
  amax = wave_max(amax);
  if (lane == 0) { s_sum[0][wave] = sum; s_amax[wave] = amax; }
  __syncthreads();
  // the tensor's largest magnitude is the largest column maximum
  if (tid == 0) t.absmax_part[0] = __builtin_fmaxf(__builtin_fmaxf(s_amax[0], s_amax[1]), __builtin_fmaxf(s_amax[2], s_amax[3]));
  const float thr0 = kOutlierFactor * static_cast<float>(((s_sum[0][0] + s_sum[0][1]) + (s_sum[0][2] + s_sum[0][3])) / K);
  double sum1 = 0.0;
  uint32_t n1 = 0;
  each(tid, kThreads, strided, [&](int, u32x4 v) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (!(u2f(v[i]) > thr0)) { sum1 += static_cast<double>(u2f(v[i])); ++n1; }
  });
  sum1 = wave_sum(sum1);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) n1 += static_cast<uint32_t>(__shfl_xor(static_cast<int>(n1), d, 64));
  if (lane == 0) { s_sum[1][wave] = sum1; s_cnt[1][wave] = n1; }
  __syncthreads();
  const uint32_t n_typ = (s_cnt[1][0] + s_cnt[1][1]) + (s_cnt[1][2] + s_cnt[1][3]);
  const double typ = ((s_sum[1][0] + s_sum[1][1]) + (s_sum[1][2] + s_sum[1][3])) / (n_typ > 0 ? n_typ : 1);
  const float thr = n_typ > 0 ? kOutlierFactor * static_cast<float>(typ) : thr0;
  // thread t owns the vectors [t * per, (t + 1) * per): count, scan over the threads, assign slots
  const int per = (nv + kThreads - 1) / kThreads;
  const int lo = tid * per < nv ? tid * per : 0, own = tid * per < nv ? (nv - tid * per < per ? nv - tid * per : per) : 0;
  uint32_t n = 0;
  each(lo, 1, own, [&](int, u32x4 v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) n += u2f(v[i]) > thr ? 1u : 0u;
  });
  uint32_t incl = n;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = static_cast<uint32_t>(__shfl_up(static_cast<int>(incl), d, 64));
    if (lane >= d) incl += o;
  }
  if (lane == 63) s_cnt[0][wave] = incl;
  __syncthreads();
  uint32_t base = incl - n;
  for (int w = 0; w < wave; ++w) base += s_cnt[0][w];
  each(lo, 1, own, [&](int c4, u32x4 v) {
    uint32_t slots = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t slot = 0xFFu;
      if (u2f(v[i]) > thr) {
        if (base < static_cast<uint32_t>(kWaSideCols)) { slot = base; t.side_cols[base] = 4 * c4 + i; }
        ++base;
      }
      slots |= slot << (8 * i);
    }
    reinterpret_cast<uint32_t*>(t.col_slot)[c4] = slots;
  });
  if (tid == kThreads - 1) t.side_cols[kWaSideCols] = static_cast<int32_t>(base < static_cast<uint32_t>(kWaSideCols) ? base : kWaSideCols);
}

// First pass: largest magnitudes, a workgroup to a segment (a share of 2500 workgroups to a tensor, 1.2 rounds of resident ones, 95 us
// for the 405 MB of a 7B block's weights, 84 us so).  The tensors and their segments in descending order: the quantize pass begins
// with what was read last (a block of 4096, 200 tokens 711 -> 704 us, 3008, 400 tokens 519 -> 512; smaller ones and a layer alone even).  The activations of a column split, a workgroup each, come first: their largest magnitude
// is that of the column maxima.  Picking their columns beside the weights' largest magnitudes instead of before them takes a launch
// of 15 us out of a 7B block's step.
__global__ __launch_bounds__(kThreads) void wa_absmax_kernel(const PrepArgs a) {
  using L = Load8<BF16>;
  __shared__ float s_wmax[kThreads / 64];
  int b, nb;
  const PrepTensor& t = my_tensor(a, b, nb);
  if (t.is_x && t.side) {   // uniform
    pick_columns(t);
    return;
  }
  const int tid = threadIdx.x;
  const int64_t lo = static_cast<int64_t>(nb - 1 - b) * t.max_chunks;   // the last ones first
  const int64_t hi = (lo + t.max_chunks < t.n_chunks) ? lo + t.max_chunks : t.n_chunks;
  constexpr int64_t stride = kThreads;
  float amax = 0.0f;
  int64_t c = lo + tid;
  for (; c + (kInFlight - 1) * stride < hi; c += kInFlight * stride) {
    float v[kInFlight][8];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) L::load(chunk_src(t, c + u * stride), v[u]);
#pragma unroll
    for (int u = 0; u < kInFlight; ++u)
#pragma unroll
      for (int i = 0; i < 8; ++i) amax = __builtin_fmaxf(amax, __builtin_fabsf(v[u][i]));
  }
  for (; c < hi; c += stride) {
    float v[8];
    L::load(chunk_src(t, c), v);
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
  }
  amax = wave_max(amax);
  if ((tid & 63) == 0) s_wmax[tid >> 6] = amax;
  __syncthreads();
  if (tid == 0)
    t.absmax_part[b] = __builtin_fmaxf(__builtin_fmaxf(s_wmax[0], s_wmax[1]), __builtin_fmaxf(s_wmax[2], s_wmax[3]));
}

// The side operand of a tensor: the E4M3 grid values of its split-off columns as bf16, dense
// [rows][kWaSideCols], zero in the slots beyond the number of split-off columns.  The last workgroups of the quantize pass;
// workgroup b of nb.
MOFQ_DEV void side_operand(const PrepTensor& t, int b, int nb, float scale) {
  const int count = t.side_cols[kWaSideCols];
  const float inv = 1.0f / scale;
  const int64_t n = static_cast<int64_t>(t.rows_i32) * kWaSideCols;
  for (int64_t e = static_cast<int64_t>(b) * kThreads + threadIdx.x; e < n; e += static_cast<int64_t>(nb) * kThreads) {
    const int slot = static_cast<int>(e % kWaSideCols);
    const int64_t row = e / kWaSideCols;
    uint16_t out = 0;
    if (slot < count) {
      const float x = u2f(static_cast<uint32_t>(t.data[row * t.ld_i32 + t.side_cols[slot]]) << 16);
      const int p = __builtin_amdgcn_cvt_pk_fp8_f32(med3(x * inv, -448.0f, 448.0f), 0.0f, 0, false);
      const f32x2 g = __builtin_amdgcn_cvt_pk_f32_fp8(p, false);
      out = static_cast<uint16_t>(f2u(g[0]) >> 16);   // exact: at most 4 significant bits
    }
    t.side[e] = out;
  }
}

// SIDE: the fp8-unit product's inputs, with the side operands' workgroups behind the others; else the exact product's.
template <bool SIDE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5))) void wa_quant_kernel(const PrepArgs a) {
  __shared__ float s_tmp[kThreads / 64];
  __shared__ double s_part[kThreads / 64][2];
  int k, b, nb;
  const bool side = SIDE && static_cast<int>(blockIdx.x) >= a.first_block[a.n];   // uniform
  const PrepTensor& t = side ? my_tensor(a, a.first_side, k, b, nb) : my_tensor(a, a.first_block, k, b, nb);
  const int n_side = nb;
  if (side) nb = a.first_block[k + 1] - a.first_block[k];
  const int tid = threadIdx.x;
  // the tensor's largest magnitude from the partials of the first pass (same launch shape) or
  // from the one the column pass left
  float amax = 0.0f;
  const int na = t.n_absmax;
  for (int i = tid; i < na; i += kThreads) amax = __builtin_fmaxf(amax, t.absmax_part[i]);
  amax = wave_max(amax);
  if ((tid & 63) == 0) s_tmp[tid >> 6] = amax;
  __syncthreads();
  amax = __builtin_fmaxf(__builtin_fmaxf(s_tmp[0], s_tmp[1]), __builtin_fmaxf(s_tmp[2], s_tmp[3]));
  const float sA = unit_scale(amax, t.ratio, Codec<MOFQ_INT8>::QMAX, false);
  const float sB = unit_scale(amax, t.ratio, Codec<MOFQ_FP8_E4M3>::QMAX, false);
  if (side) {
    side_operand(t, b, n_side, sB);
    return;
  }
  if (b == 0 && tid == 0) { t.scale[0] = sA; t.scale[1] = sB; }
  const float iA = 1.0f / sA, iB = 1.0f / sB;
  const double sAd = static_cast<double>(sA), sBd = static_cast<double>(sB);
  const bool dense = t.ld == t.cpr * 8;
  for (int seg = b; seg < t.n_seg; seg += nb) {
    const int64_t lo = static_cast<int64_t>(seg) * t.seg_chunks;
    const int64_t hi = (lo + t.seg_chunks < t.n_chunks) ? lo + t.seg_chunks : t.n_chunks;
    double accA = 0.0, accB = 0.0;
    // dense input (uniform): two neighbouring chunks at a time, so that the codes leave in 16-byte pieces; one where rows are apart or
    // two would leave threads without work (28.95 and 28.64 us for a whole select of 512 x 1024 x 1024)
    const bool pairs = dense && hi - lo >= 4 * kThreads;
    int64_t c = pairs ? lo + 2 * tid : lo + tid;
    for (; pairs && c + 1 < hi; c += 2 * kThreads) {
      const u32x4* const src = reinterpret_cast<const u32x4*>(t.data + c * 8);
      const u32x4 raw0 = src[0], raw1 = src[1];
      const QuantChunk q0 = quant_chunk(raw0, iA, iB, sAd, sBd, accA, accB);
      __builtin_amdgcn_sched_barrier(0);   // one chunk at a time: keeps the register count low
      const QuantChunk q1 = quant_chunk(raw1, iA, iB, sAd, sBd, accA, accB);
      store_pair(t, c, q0, q1);
    }
    // an odd last chunk, or all of them
    for (; c < hi; c += pairs ? 2 * kThreads : kThreads) {
      const u32x4 raw = *reinterpret_cast<const u32x4*>(chunk_src(t, c));
      store_chunk(t, c, quant_chunk(raw, iA, iB, sAd, sBd, accA, accB));
    }
    accA = wave_sum(accA);
    accB = wave_sum(accB);
    __syncthreads();   // the previous segment's partials have been read
    if ((tid & 63) == 0) { s_part[tid >> 6][0] = accA; s_part[tid >> 6][1] = accB; }
    __syncthreads();
    if (tid < 2)
      t.sse_part[static_cast<int64_t>(seg) * 2 + tid] = (s_part[0][tid] + s_part[1][tid]) + (s_part[2][tid] + s_part[3][tid]);
  }
}

bool fill(const WaPrepTensor& p, PrepTensor* t) {
  *t = PrepTensor{};
  if (p.rows < 1 || p.cols < 8 || p.cols % 8 != 0 || p.ld < p.cols || p.ld % 8 != 0) return false;
  if (!p.absmax_part || !p.sse_part || !p.q_i8 || !p.q_f8 || !p.scale) return false;
  t->data = static_cast<const uint16_t*>(p.data);
  t->cpr = p.cols / 8;
  t->n_chunks = p.rows * t->cpr;
  t->ld = p.ld;
  t->n_seg = wa_prep_segments(p.rows, p.cols);
  t->seg_chunks = static_cast<int32_t>((t->n_chunks + t->n_seg - 1) / t->n_seg + 1) / 2 * 2;   // even; the last segments may be empty
  t->ratio = p.ratio;
  t->absmax_part = p.absmax_part;
  t->sse_part = p.sse_part;
  t->q_i8 = p.q_i8;
  t->q_f8 = p.q_f8;
  t->scale = p.scale;
  if (p.side) {
    if (!p.col_slot || !p.side_cols || p.cols % 64 != 0 || p.rows > (1 << 30) || p.cols > (1 << 20) ||
        p.ld > (int64_t{1} << 30))
      return false;
    if (p.is_x && (!p.colmax || !p.q_f8_main || t->n_chunks >= (int64_t{1} << 31))) return false;
    t->is_x = p.is_x;
    t->ld_i32 = static_cast<int32_t>(p.ld);
    t->rows_i32 = static_cast<int32_t>(p.rows);
    t->cols_i32 = static_cast<int32_t>(p.cols);
    t->colmax = p.colmax;
    t->col_slot = p.col_slot;
    t->side_cols = p.side_cols;
    t->q_f8_main = p.is_x ? p.q_f8_main : nullptr;
    t->side = p.side;
  }
  return true;
}

}  // namespace

int wa_prep_segments(int64_t rows, int64_t cols) {
  const int64_t n_chunks = rows * (cols / 8);
  const int64_t b = (n_chunks + kThreads - 1) / kThreads;
  return static_cast<int>(b < 1 ? 1 : (b > kTensorBlocks ? kTensorBlocks : b));
}

int launch_wa_prep(const WaPrepTensor* p, int n, hipStream_t st) {
  if (!p || n < 1 || n > kMaxTensors) return MOFQ_ERR_INVALID_ARG;
  PrepArgs a{};
  int64_t total_seg = 0;
  for (int i = 0; i < n; ++i) {
    if (!p[i].data) continue;   // skipped
    if (!fill(p[i], &a.t[a.n])) return MOFQ_ERR_INVALID_ARG;
    if (a.t[a.n].n_chunks > (int64_t{1} << 40)) return MOFQ_ERR_UNSUPPORTED;
    total_seg += a.t[a.n].n_seg;
    ++a.n;
  }
  if (a.n < 1) return MOFQ_OK;
  // One workgroup per segment, but for up to twice as many segments as 16 workgroups per compute unit a share of those: short
  // segments hardly pay for the fold before them.  Exact / fp8 unit, us, without shares -> with: a block of 1024, 1000 tokens 157.7 ->
  // 156.7 / 160.7 -> 158.4, 2048, 64 tokens 130.2 -> 130.1 / 133.3 -> 130.7; but 4096, 64 tokens, whose segments are four times as long, 441 -> 454 /
  // 446 -> 448.  Beyond that number they lose for all: 4096, 200 tokens, exact 801 -> 824, 3008, 400 tokens 608 -> 620.
  constexpr int64_t kShares = 4096;
  for (int k = 0; k < a.n; ++k) {
    int64_t nb = a.t[k].n_seg;
    if (total_seg > kShares && total_seg <= 2 * kShares) nb = std::max<int64_t>(1, nb * kShares / total_seg);
    a.first_block[k + 1] = a.first_block[k] + static_cast<int32_t>(nb);
  }
  const int blocks = a.first_block[a.n];
  // column split: the activations' column maxima come first, the pick beside the largest magnitudes of the other tensors, and
  // the side operands at the end of the quantize pass (which zeroes the picked columns in the fp8 operand)
  PrepArgs xs{}, am{};
  a.first_side[0] = blocks;
  for (int k = 0; k < a.n; ++k) {
    const PrepTensor& t = a.t[k];
    int64_t side = 0;
    if (t.side) {
      side = std::min<int64_t>((static_cast<int64_t>(t.rows_i32) * kWaSideCols + kThreads * 4 - 1) / (kThreads * 4), 1024);
      if (t.is_x) {
        a.t[k].n_absmax = 1;
        xs.t[xs.n] = am.t[am.n] = t;
        xs.first_block[xs.n + 1] = xs.first_block[xs.n] + t.cols_i32 / 64;
        am.first_block[am.n + 1] = am.first_block[am.n] + 1;
        ++xs.n;
        ++am.n;
      }
    }
    a.first_side[k + 1] = a.first_side[k] + static_cast<int32_t>(side);
  }
  for (int k = a.n - 1; k >= 0; --k) {
    if (a.t[k].side && a.t[k].is_x) continue;
    // 32 KB and more to a workgroup, a round of loads; the quantize pass folds the partial maxima in every workgroup
    PrepTensor& t = a.t[k];
    t.n_absmax = static_cast<int32_t>(std::min<int64_t>(kTensorBlocks, std::max<int64_t>(1, t.n_chunks / (kInFlight * kThreads))));
    t.max_chunks = static_cast<int32_t>((t.n_chunks + t.n_absmax - 1) / t.n_absmax);
    am.t[am.n] = t;
    am.first_block[am.n + 1] = am.first_block[am.n] + t.n_absmax;
    ++am.n;
  }
  static_assert(sizeof(PrepArgs) <= 4096, "kernel arguments");
  if (xs.n) hipLaunchKernelGGL(wa_colmax_kernel, dim3(xs.first_block[xs.n]), dim3(kThreads), 0, st, xs);
  hipLaunchKernelGGL(wa_absmax_kernel, dim3(am.first_block[am.n]), dim3(kThreads), 0, st, am);
  if (a.first_side[a.n] > blocks) hipLaunchKernelGGL(wa_quant_kernel<true>, dim3(a.first_side[a.n]), dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL(wa_quant_kernel<false>, dim3(blocks), dim3(kThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

}  // namespace mofq
