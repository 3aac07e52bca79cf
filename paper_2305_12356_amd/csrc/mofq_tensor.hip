// Per-tensor scales with one candidate ratio (activations: Section 3.2; the absmax scale of a whole
// weight): Algorithm 1's select and the quantization of one tensor in one format.
//
// The passes are bound by memory for large tensors and by launches and memory latencies for small
// ones, so nothing between them gets a launch of its own: the partial maxima and partial error sums
// of a pass (one per workgroup, at most 1024) are folded by every workgroup of the next.
//   select    : largest magnitude | errors of the candidates | select + codes      (3 launches)
//   calibrated: errors of the candidates | select + codes                          (2)
//   quantize  : largest magnitude | codes + error | one-unit outputs               (3), or 1 for small tensors
#include <algorithm>
#include <atomic>
#include <chrono>

#include "mofq_codes.h"
#include "mofq_internal.h"

namespace mofq {

namespace {

constexpr int kThreads = 256;
constexpr int kUnroll = 4;        // 16-byte loads in flight per lane

struct TensorArgs {
  const void* w;
  int64_t n_chunks, cpr, ld;      // 8-element chunks of the tensor and per row; elements between rows
  const float* absmax;            // n_absmax values whose largest is the tensor's magnitude
  int32_t n_absmax;
  int32_t n_blocks;               // workgroups of the passes (partial sums)
  float ratio;
  int32_t scale_f16;
  float* absmax_part;             // [n_blocks]
  float* running;                 // largest-magnitude pass: fold into this value instead
  double* sse;                    // [candidates][kTensorBlocks]
  double* energy;                 // [n_blocks]
  int32_t n_cand;
  int32_t fmt[MOFQ_MAX_CANDIDATES];
  mofq_qout_t out;
  mofq_result_t* result;
  double* tensor_err;
};

// Chunk c: a dense tensor is one run of chunks, rows that lie apart cost a division.
template <typename In> MOFQ_DEV void load_chunk(const TensorArgs& a, int64_t c, Raw8<In>& raw) {
  if (a.ld == a.cpr * 8) {   // uniform
    raw.load(a.w, c * 8, 0);
  } else {
    const int64_t row = c / a.cpr;
    raw.load(a.w, row * a.ld + (c - row * a.cpr) * 8, 0);
  }
}

// f(chunk, its elements) for every chunk of this workgroup, kUnroll loads in flight per lane.
template <typename In, int THREADS = kThreads, typename F> MOFQ_DEV void for_chunks(const TensorArgs& a, F&& f) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * THREADS;
  for (int64_t c = static_cast<int64_t>(blockIdx.x) * THREADS + threadIdx.x; c < a.n_chunks; c += kUnroll * stride) {
    Raw8<In> raw[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) load_chunk<In>(a, c + u * stride < a.n_chunks ? c + u * stride : c, raw[u]);
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (c + u * stride < a.n_chunks) {
        float v[8];
        raw[u].widen(v);
        f(c + u * stride, v);
      }
  }
}

template <int NW> MOFQ_DEV float block_max(float v, float (&s_tmp)[NW]) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) s_tmp[threadIdx.x >> 6] = v;
  __syncthreads();
  v = s_tmp[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) v = __builtin_fmaxf(v, s_tmp[w]);
  return v;
}
template <int NW> MOFQ_DEV double block_sum(double v, double (&s_tmp)[NW]) {   // fixed order
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) s_tmp[threadIdx.x >> 6] = v;
  __syncthreads();
  v = s_tmp[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) v += s_tmp[w];
  return v;
}

// The tensor's magnitude from the previous pass (at most 1024 values) or the calibration (one).
MOFQ_DEV float folded_absmax(const TensorArgs& a, float (&s_tmp)[kThreads / 64]) {
  float m = 0.0f;
#pragma unroll
  for (int u = 0; u < kTensorBlocks / kThreads; ++u) {
    const int i = u * kThreads + static_cast<int>(threadIdx.x);
    m = __builtin_fmaxf(m, a.absmax[i < a.n_absmax ? i : 0]);
  }
  return block_max(m, s_tmp);
}

MOFQ_DEV float format_qmax(int fmt) {
  switch (fmt) {
    case MOFQ_INT4: return Codec<MOFQ_INT4>::QMAX;
    case MOFQ_FP4_E2M1: return Codec<MOFQ_FP4_E2M1>::QMAX;
    case MOFQ_INT8: return Codec<MOFQ_INT8>::QMAX;
    case MOFQ_FP4_E2M1_IEEE: return Codec<MOFQ_FP4_E2M1_IEEE>::QMAX;
    case MOFQ_FP8_E5M2: return Codec<MOFQ_FP8_E5M2>::QMAX;
    default: return Codec<MOFQ_FP8_E4M3>::QMAX;
  }
}

// ---- largest magnitude ----------------------------------------------------------------
// RUNNING: folded into one value that the caller keeps, else one partial maximum per workgroup.
// A running maximum that starts at zero is beaten by every workgroup of the first batch, and a place in memory takes
// an atomic every 4 ns, so that pass has workgroups of 16 waves, a quarter as many: four batches of 2048 x 4096
// bf16 and their select 40.9 -> 34.9 us (8 waves: 35.6), one batch of 4096 x 4096 42.5 -> 31.3.  Partial maxima are
// folded by the next pass, where larger workgroups do not pay: quantizing 4096 x 4096 17.9 us, with them 19.6.
constexpr int kRunningThreads = 1024;
template <typename In, bool RUNNING>
__global__ __launch_bounds__(RUNNING ? kRunningThreads : kThreads) void tensor_max_kernel(const TensorArgs a) {
  constexpr int THREADS = RUNNING ? kRunningThreads : kThreads;
  __shared__ float s_tmp[THREADS / 64];
  float m = 0.0f;
  for_chunks<In, THREADS>(a, [&](int64_t, const float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(v[i]));
  });
  m = block_max(m, s_tmp);
  if (threadIdx.x != 0) return;
  if constexpr (RUNNING) {
    // *running = max(*running, m): magnitudes order like their bit patterns, and most workgroups
    // of a later batch see a value that is large enough already and leave the address alone
    uint32_t* const r = reinterpret_cast<uint32_t*>(a.running);
    if (f2u(m) > __hip_atomic_load(r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      __hip_atomic_fetch_max(r, f2u(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    a.absmax_part[blockIdx.x] = m;
  }
}

// ---- errors of one candidate (FB < 0) or a pair -------------------------------------------
template <typename In, int FA, int FB>
__global__ __launch_bounds__(kThreads) void tensor_errors_kernel(const TensorArgs a, double* sse_a, double* sse_b, int with_energy) {
  constexpr int FBX = FB >= 0 ? FB : FA;
  __shared__ float s_tmp[kThreads / 64];
  __shared__ double s_sum[3][kThreads / 64];
  const float amax = folded_absmax(a, s_tmp);
  const float sA = unit_scale(amax, a.ratio, Codec<FA>::QMAX, a.scale_f16 != 0);
  const float sB = unit_scale(amax, a.ratio, Codec<FBX>::QMAX, a.scale_f16 != 0);
  const float iA = 1.0f / sA, iB = 1.0f / sB;
  const double sAd = static_cast<double>(sA), sBd = static_cast<double>(sB);
  double eA = 0.0, eB = 0.0, en = 0.0;
  uint32_t carry = 0;
  for_chunks<In>(a, [&](int64_t, const float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      score2_f64<FA>(eA, v[i], v[i + 1], iA, sAd, carry);
      if constexpr (FB >= 0) score2_f64<FBX>(eB, v[i], v[i + 1], iB, sBd, carry);
      if (with_energy) {   // uniform
        const double d0 = static_cast<double>(v[i]), d1 = static_cast<double>(v[i + 1]);
        en = __builtin_fma(d0, d0, en);
        en = __builtin_fma(d1, d1, en);
      }
    }
  });
  eA = block_sum(eA, s_sum[0]);
  if constexpr (FB >= 0) eB = block_sum(eB, s_sum[1]);
  en = block_sum(en, s_sum[2]);
  if (threadIdx.x == 0) {
    sse_a[blockIdx.x] = eA;
    if constexpr (FB >= 0) sse_b[blockIdx.x] = eB;
    if (with_energy) a.energy[blockIdx.x] = en;
  }
}

// ---- one-unit outputs -----------------------------------------------------------------------
MOFQ_DEV void write_unit(const TensorArgs& a, float s, double err) {   // one thread
  if (a.out.scales) {
    if (a.scale_f16)
      *static_cast<uint16_t*>(a.out.scales) = __half_as_ushort(__float2half_rn(s));   // exact: s is an fp16 value
    else
      *static_cast<float*>(a.out.scales) = s;
  }
  if (a.out.clip_idx) *a.out.clip_idx = 0;
  if (a.out.unit_err) *a.out.unit_err = err;
  if (a.tensor_err) *a.tensor_err = err;
}

template <int FMT> MOFQ_DEV void store_codes(void* codes, int64_t c, const float (&v)[8], float inv_s) {
  uint32_t words[2];
  encode8<FMT>(v, inv_s, words);
  if constexpr (Codec<FMT>::BITS == 4) {
    static_cast<uint32_t*>(codes)[c] = words[0];
  } else {
    u32x2 o;
    o[0] = words[0];
    o[1] = words[1];
    static_cast<u32x2*>(codes)[c] = o;
  }
}

// Sum of the n_blocks (at most 1024) partial sums by one wave, 16 loads in flight per lane; fixed order.
MOFQ_DEV double wave_partials(const double* v, int n) {
  constexpr int U = kTensorBlocks / 64;
  const int lane = threadIdx.x & 63;
  double e[U], t = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) e[u] = v[lane + u * 64 < n ? lane + u * 64 : 0];
#pragma unroll
  for (int u = 0; u < U; ++u) t += lane + u * 64 < n ? e[u] : 0.0;
  return wave_sum(t);
}

// ---- select + codes of the winner -------------------------------------------------------------
template <typename In>
__global__ __launch_bounds__(kThreads) void tensor_select_kernel(const TensorArgs a) {
  __shared__ float s_tmp[kThreads / 64];
  __shared__ double s_sum[MOFQ_MAX_CANDIDATES + 1];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  static_assert(kThreads / 64 == MOFQ_MAX_CANDIDATES, "a wave per candidate");
  if (wave < a.n_cand) {
    const double t = wave_partials(a.sse + wave * kTensorBlocks, a.n_blocks);
    if ((threadIdx.x & 63) == 0) s_sum[wave] = t;
  }
  if (blockIdx.x == 0 && wave == kThreads / 64 - 1) {
    const double t = wave_partials(a.energy, a.n_blocks);
    if ((threadIdx.x & 63) == 0) s_sum[MOFQ_MAX_CANDIDATES] = t;
  }
  const float amax = folded_absmax(a, s_tmp);   // (its barrier publishes the sums)
  // Algorithm 1: min_error starts at infinity, candidates in list order, strictly smaller wins
  double min_err = __builtin_inf();
  int best = 0;
  for (int c = 0; c < a.n_cand; ++c)
    if (s_sum[c] < min_err) { min_err = s_sum[c]; best = c; }
  best = __builtin_amdgcn_readfirstlane(best);
  const float s = unit_scale(amax, a.ratio, format_qmax(a.fmt[best]), a.scale_f16 != 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (a.result) {
      a.result->best = best;
      a.result->n = a.n_cand;
      for (int c = 0; c < MOFQ_MAX_CANDIDATES; ++c) a.result->err[c] = c < a.n_cand ? s_sum[c] : 0.0;
      a.result->ref_energy = s_sum[MOFQ_MAX_CANDIDATES];
    }
    write_unit(a, s, s_sum[best]);
  }
  if (!a.out.codes) return;   // uniform
  const float inv_s = 1.0f / s;
  with_format(a.fmt[best], [&](auto fmt_c) {
    for_chunks<In>(a, [&](int64_t c, const float (&v)[8]) { store_codes<decltype(fmt_c)::value>(a.out.codes, c, v, inv_s); });
  });
}

// ---- one format: codes and error from one read ---------------------------------------------------
template <typename In, int FMT>
__global__ __launch_bounds__(kThreads) void tensor_quant_kernel(const TensorArgs a) {
  __shared__ float s_tmp[kThreads / 64];
  __shared__ double s_sum[kThreads / 64];
  const float s = unit_scale(folded_absmax(a, s_tmp), a.ratio, Codec<FMT>::QMAX, a.scale_f16 != 0);
  const float inv_s = 1.0f / s;
  const double sd = static_cast<double>(s);
  double e = 0.0;
  uint32_t carry = 0;
  for_chunks<In>(a, [&](int64_t c, const float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 8; i += 2) score2_f64<FMT>(e, v[i], v[i + 1], inv_s, sd, carry);
    store_codes<FMT>(a.out.codes, c, v, inv_s);
  });
  e = block_sum(e, s_sum);
  if (threadIdx.x == 0) a.sse[blockIdx.x] = e;
}
__global__ __launch_bounds__(kThreads) void tensor_unit_kernel(const TensorArgs a) {   // one workgroup
  __shared__ float s_tmp[kThreads / 64];
  const float s = unit_scale(folded_absmax(a, s_tmp), a.ratio, format_qmax(a.fmt[0]), a.scale_f16 != 0);
  if (threadIdx.x < 64) {
    const double e = wave_partials(a.sse, a.n_blocks);
    if (threadIdx.x == 0) write_unit(a, s, e);
  }
}

// Tensors of up to 163840 elements (a few tokens of an activation): one launch.  Every workgroup reads the whole
// tensor (from L2, 8 loads in flight per lane) and finds its magnitude, then writes the codes of its own 8192 elements
// and sums their error; the workgroup that finds everybody's sums in the scratch adds them up.  Up to 65536 elements
// the host bounds the call (5.0 us among others, 15.5 alone), beyond that what one compute unit reads and compares.
// bf16 E4M3, us among others / alone, with all of the error summed by one workgroup -> here: 32768 elements 5.1 / 17.2 ->
// 5.1 / 16.7, 65536 7.5 / 19.8 -> 5.6 / 18.4; in three launches (9.8 / 21.2 whatever the size) -> here: 81920 6.4 / 19.0,
// 131072 7.4 / 19.9, 196608 9.2 / 21.6, 262144 10.9 / 23.6; fp32 65536 7.4 / 20.1 -> 5.9 / 18.6, 131072 8.0 / 20.6.
// In the launches of larger tensors the same meeting would cost more than the third launch: its fence in 1024
// workgroups takes 20 us.
//
// The meeting: workgroup b leaves two words, its sum's bits and the same bits ^ nonce, and reads all of them behind a
// sequentially consistent fence, so the last one in the order of the fences finds them all (a second one that does writes the same
// values; two calls at once on one scratch, which the interface excludes, can lose each other's pairs, and then
// nobody finds all of them).  A pair is complete if it xors to the nonce, which the host draws per call, so the scratch needs no
// clearing; whoever finds all pairs leaves zeros, so that a replay of a captured call, which has the same nonce,
// starts without them.  Torn pairs: (sum, 0) xors to the sum, which is never the nonce (a negative number);
// (0, sum ^ nonce) xors to the nonce only if the sum is 0, the value then read.  Nobody waits for anybody.
constexpr int kSmallThreads = 1024, kSmallLoads = 8, kSmallBlocks = 20;
static_assert(kSmallBlocks <= 64 && 2 * kSmallBlocks <= kTensorBlocks, "a lane and two words of scratch per workgroup");
template <typename In, int FMT>
__global__ __launch_bounds__(kSmallThreads) void tensor_quant_small_kernel(const TensorArgs a, const uint64_t nonce) {
  __shared__ float s_tmp[kSmallThreads / 64];
  __shared__ double s_sum[kSmallThreads / 64];
  const int n = static_cast<int>(a.n_chunks), tid = threadIdx.x;
  const int blocks = gridDim.x, b = blockIdx.x;
  const uint32_t cpr = static_cast<uint32_t>(a.cpr);   // at most n
  const auto load = [&](int c, Raw8<In>& raw) {
    if (a.ld == a.cpr * 8) {   // uniform
      raw.load(a.w, static_cast<int64_t>(c) * 8, 0);
    } else {
      const uint32_t row = static_cast<uint32_t>(c) / cpr;
      raw.load(a.w, row * a.ld + static_cast<int64_t>(static_cast<uint32_t>(c) - row * cpr) * 8, 0);
    }
  };
  float m = 0.0f;
  const auto widest = [&](const Raw8<In>& raw) {
    float v[8];
    raw.widen(v);
#pragma unroll
    for (int i = 0; i < 8; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(v[i]));
  };
  Raw8<In> own;
  const int c_own = b * kSmallThreads + tid;
  load(c_own < n ? c_own : 0, own);   // past the end: chunk 0 again
  for (int j0 = 1; j0 < blocks; j0 += kSmallLoads) {   // the others' chunks, from the next workgroup's on
    Raw8<In> raw[kSmallLoads];
#pragma unroll
    for (int u = 0; u < kSmallLoads; ++u)
      if (j0 + u < blocks) {   // uniform
        const int j = b + j0 + u < blocks ? b + j0 + u : b + j0 + u - blocks;
        const int c = j * kSmallThreads + tid;
        load(c < n ? c : 0, raw[u]);
      }
#pragma unroll
    for (int u = 0; u < kSmallLoads; ++u)
      if (j0 + u < blocks) widest(raw[u]);
  }
  widest(own);
  const float s = unit_scale(block_max(m, s_tmp), a.ratio, Codec<FMT>::QMAX, a.scale_f16 != 0);
  const float inv_s = 1.0f / s;
  const double sd = static_cast<double>(s);
  double e = 0.0;
  if (c_own < n) {
    uint32_t carry = 0;
    float v[8];
    own.widen(v);
#pragma unroll
    for (int i = 0; i < 8; i += 2) score2_f64<FMT>(e, v[i], v[i + 1], inv_s, sd, carry);
    store_codes<FMT>(a.out.codes, c_own, v, inv_s);
  }
  e = block_sum(e, s_sum);
  if (tid >= 64) return;
  if (blocks > 1) {   // uniform
    uint64_t* const place = reinterpret_cast<uint64_t*>(a.sse);   // two words per workgroup
    const auto leave = [&](int i, uint64_t w0, uint64_t w1) {
      __hip_atomic_store(place + 2 * i, w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(place + 2 * i + 1, w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const uint64_t bits = __builtin_bit_cast(uint64_t, e);
    if (tid == 0) leave(b, bits, bits ^ nonce);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "agent");
    const int i = tid < blocks ? tid : 0;
    const uint64_t w0 = __hip_atomic_load(place + 2 * i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t w1 = __hip_atomic_load(place + 2 * i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__ballot((w0 ^ w1) != nonce) != 0) return;   // uniform
    if (tid < blocks) leave(tid, 0, 0);
    e = wave_sum(tid < blocks ? __builtin_bit_cast(double, w0) : 0.0);
  }
  if (tid == 0) write_unit(a, s, e);
}

// A number that no other call of the process has, a count that starts at the time mixed as the SplitMix64 generator
// does (Steele, Lea and Flood 2014; its increment and multipliers): the bits of a finite negative double.
uint64_t next_nonce() {
  static std::atomic<uint64_t> count{static_cast<uint64_t>(std::chrono::system_clock::now().time_since_epoch().count())};
  uint64_t z = count.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (z | 1ull << 63) & ~(1ull << 62);
}

// ---- launches ----------------------------------------------------------------------------------------

// Workgroups of a pass: a chunk per thread, then kUnroll and more, at most kTensorBlocks of them.
int pass_blocks(int64_t n_chunks) {
  return static_cast<int>(std::min<int64_t>(kTensorBlocks, (n_chunks + kThreads - 1) / kThreads));
}

int fill(const TensorParams& p, TensorArgs* a) {
  if (!p.w || p.rows < 1 || p.cols < 8 || p.cols % 8 != 0 || p.ld < p.cols || p.n_cand < 0 || p.n_cand > MOFQ_MAX_CANDIDATES)
    return MOFQ_ERR_INVALID_ARG;
  *a = TensorArgs{};
  a->w = p.w;
  a->cpr = p.cols / 8;
  a->n_chunks = p.rows * a->cpr;
  a->ld = p.rows == 1 ? p.cols : p.ld;
  a->n_blocks = pass_blocks(a->n_chunks);
  a->ratio = p.ratio;
  a->scale_f16 = p.scale_f16;
  a->absmax_part = p.absmax_part;
  a->absmax = p.ext_absmax ? p.ext_absmax : p.absmax_part;
  a->n_absmax = p.ext_absmax ? 1 : a->n_blocks;
  a->running = p.running;
  a->sse = p.sse;
  a->energy = p.energy;
  a->n_cand = p.n_cand;
  for (int c = 0; c < p.n_cand; ++c) a->fmt[c] = p.fmt[c];
  a->out = p.out;
  a->result = p.result;
  a->tensor_err = p.tensor_err;
  return MOFQ_OK;
}

template <typename In> int launch_max(const TensorArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((tensor_max_kernel<In, false>), dim3(a.n_blocks), dim3(kThreads), 0, st, a);
  return hip_status(hipGetLastError());
}
template <typename In> int launch_running(const TensorArgs& a, hipStream_t st) {
  constexpr int per = kRunningThreads / kThreads;
  hipLaunchKernelGGL((tensor_max_kernel<In, true>), dim3((a.n_blocks + per - 1) / per), dim3(kRunningThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

template <typename In> int launch_errors(const TensorArgs& a, hipStream_t st) {
  int c = 0;
  while (c < a.n_cand) {
    double* const sa = a.sse + c * kTensorBlocks;
    double* const sb = sa + kTensorBlocks;
    const int energy = c == 0;
    const int fa = a.fmt[c], fb = c + 1 < a.n_cand ? a.fmt[c + 1] : -1;
    int n = 2;
#define MOFQ_PAIR(A, B, SA, SB)                                                                                        \
  if (fa == (A) && fb == (B))                                                                                          \
    hipLaunchKernelGGL((tensor_errors_kernel<In, MOFQ_MIN2(A, B), MOFQ_MAX2(A, B)>), dim3(a.n_blocks), dim3(kThreads), 0, st, a, SA, SB, energy); \
  else
#define MOFQ_MIN2(A, B) ((A) < (B) ? (A) : (B))
#define MOFQ_MAX2(A, B) ((A) < (B) ? (B) : (A))
    // a pair shares one read; the reversed pair swaps its partial sums
    MOFQ_PAIR(MOFQ_INT4, MOFQ_FP4_E2M1, sa, sb)
    MOFQ_PAIR(MOFQ_FP4_E2M1, MOFQ_INT4, sb, sa)
    MOFQ_PAIR(MOFQ_INT8, MOFQ_FP8_E4M3, sa, sb)
    MOFQ_PAIR(MOFQ_FP8_E4M3, MOFQ_INT8, sb, sa) {
      n = 1;
      switch (fa) {
#define MOFQ_ONE(A) \
  case A: hipLaunchKernelGGL((tensor_errors_kernel<In, A, -1>), dim3(a.n_blocks), dim3(kThreads), 0, st, a, sa, nullptr, energy); break;
        MOFQ_ONE(MOFQ_INT4) MOFQ_ONE(MOFQ_FP4_E2M1) MOFQ_ONE(MOFQ_INT8) MOFQ_ONE(MOFQ_FP8_E4M3)
        MOFQ_ONE(MOFQ_FP4_E2M1_IEEE) MOFQ_ONE(MOFQ_FP8_E5M2)
#undef MOFQ_ONE
        default: return MOFQ_ERR_UNSUPPORTED;
      }
    }
#undef MOFQ_PAIR
#undef MOFQ_MIN2
#undef MOFQ_MAX2
    c += n;
  }
  return hip_status(hipGetLastError());
}

template <typename In> int launch_scores(const TensorArgs& a, hipStream_t st) {
  const int rc = a.absmax == a.absmax_part ? launch_max<In>(a, st) : static_cast<int>(MOFQ_OK);
  return rc ? rc : launch_errors<In>(a, st);
}

template <typename In> int launch_pick(const TensorArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((tensor_select_kernel<In>), dim3(a.out.codes ? a.n_blocks : 1), dim3(kThreads), 0, st, a);
  return hip_status(hipGetLastError());
}

template <typename In, int FMT> int launch_quant_fmt(const TensorArgs& a, hipStream_t st) {
  if (a.n_chunks <= kSmallThreads * kSmallBlocks) {
    const unsigned grid = static_cast<unsigned>((a.n_chunks + kSmallThreads - 1) / kSmallThreads);
    hipLaunchKernelGGL((tensor_quant_small_kernel<In, FMT>), dim3(grid), dim3(kSmallThreads), 0, st, a, next_nonce());
    return hip_status(hipGetLastError());
  }
  const int rc = launch_max<In>(a, st);
  if (rc) return rc;
  hipLaunchKernelGGL((tensor_quant_kernel<In, FMT>), dim3(a.n_blocks), dim3(kThreads), 0, st, a);
  hipLaunchKernelGGL(tensor_unit_kernel, dim3(1), dim3(kThreads), 0, st, a);
  return hip_status(hipGetLastError());
}
template <typename In> int launch_quant(const TensorArgs& a, hipStream_t st) {
  switch (a.fmt[0]) {
    case MOFQ_INT4: return launch_quant_fmt<In, MOFQ_INT4>(a, st);
    case MOFQ_FP4_E2M1: return launch_quant_fmt<In, MOFQ_FP4_E2M1>(a, st);
    case MOFQ_INT8: return launch_quant_fmt<In, MOFQ_INT8>(a, st);
    case MOFQ_FP8_E4M3: return launch_quant_fmt<In, MOFQ_FP8_E4M3>(a, st);
    case MOFQ_FP4_E2M1_IEEE: return launch_quant_fmt<In, MOFQ_FP4_E2M1_IEEE>(a, st);
    case MOFQ_FP8_E5M2: return launch_quant_fmt<In, MOFQ_FP8_E5M2>(a, st);
  }
  return MOFQ_ERR_UNSUPPORTED;
}

}  // namespace

#define MOFQ_BY_DTYPE(CALL)                        \
  switch (p.dtype) {                               \
    case MOFQ_F32: return CALL<F32>(a, st);        \
    case MOFQ_F16: return CALL<F16>(a, st);        \
    case MOFQ_BF16: return CALL<BF16>(a, st);      \
  }                                                \
  return MOFQ_ERR_INVALID_ARG;

int launch_running_absmax(const TensorParams& p, hipStream_t st) {
  TensorArgs a;
  const int rc = fill(p, &a);
  if (rc) return rc;
  if (!a.running) return MOFQ_ERR_INVALID_ARG;
  MOFQ_BY_DTYPE(launch_running)
}

namespace {
int fill_select(const TensorParams& p, TensorArgs* a) {
  const int rc = fill(p, a);
  if (rc) return rc;
  return a->n_cand < 1 || !a->sse || !a->energy || !a->absmax || a->running ? MOFQ_ERR_INVALID_ARG : MOFQ_OK;
}
}  // namespace

int launch_tensor_scores(const TensorParams& p, hipStream_t st) {
  TensorArgs a;
  const int rc = fill_select(p, &a);
  if (rc) return rc;
  MOFQ_BY_DTYPE(launch_scores)
}

int launch_tensor_pick(const TensorParams& p, hipStream_t st) {
  TensorArgs a;
  const int rc = fill_select(p, &a);
  if (rc) return rc;
  MOFQ_BY_DTYPE(launch_pick)
}

int launch_tensor_quantize(const TensorParams& p, hipStream_t st) {
  TensorArgs a;
  const int rc = fill(p, &a);
  if (rc) return rc;
  if (a.n_cand != 1 || !a.sse || !a.absmax_part || a.absmax != a.absmax_part || a.running || !a.out.codes) return MOFQ_ERR_INVALID_ARG;
  MOFQ_BY_DTYPE(launch_quant)
}

}  // namespace mofq
