// Scale search ("sweep"): for every unit of a tensor and every candidate format,
// evaluate all clip ratios and keep the first with the smallest error.
//
// This is the quantize_layer + compute_error pair of Algorithm 1 with the
// tensor-error metric (Section 4.1), evaluated for all scale candidates of a
// unit while the unit's elements sit in registers: the tensor is read from HBM
// once, however many candidates there are.
//
// Work per element and candidate (INT: multiply, round, clamp; FP: multiply,
// clamp, pick spacing, add/subtract rounding constant; then an fp64 residual and
// an fp64 fused multiply-add into the error) is plain vector ALU work: with the
// 100-candidate search the kernel is bound by the vector units, not by HBM.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "mofq_codes.h"
#include "mofq_internal.h"

namespace mofq {

namespace {

struct SweepArgs {
  const void* w;
  int64_t rows, cols, ld;
  int64_t units;
  int32_t group;
  int32_t scale_f16;
  int32_t n_clip;
  UnitRecords rec;
  float* absmax_part;
  double* sse_part;
  double* energy_part;
  int32_t n_blocks;  // per-tensor: blocks of the partial passes
  int32_t k0;                // per-tensor: first clip candidate of this scoring pass
  uint8_t* emit_i8;          // per-tensor 8-bit pair: also write the codes (see SweepParams)
  uint8_t* emit_f8;
  int32_t emit_grid_fp8;
  uint16_t* emit_grid[kMaxFmt];   // per-channel single-candidate pair: grid values as bf16 or e4m3 codes (see SweepParams)
  AheadCodes ahead;
  int32_t bisect;            // 4-bit formats: score candidates by bisection of the clip ratios, which descend
  float clip[MOFQ_MAX_CLIP];
};

// Squared error of one element at one scale: the grid value is chosen in fp32
// (the decision arithmetic), the residual and its square are fp64.
template <int FMT>
MOFQ_DEV void accumulate(double& acc, float x, double xd, float inv_s, double sd) {
  const float t = x * inv_s;
  if constexpr (Codec<FMT>::IS_INT) {
    const double g = static_cast<double>(Codec<FMT>::grid(t));
    const double d = __builtin_fma(-g, sd, xd);
    acc = __builtin_fma(d, d, acc);
  } else {
    // sign-symmetric grid: (|x| - |g| s)^2 == (x - g s)^2
    const double g = static_cast<double>(Codec<FMT>::mag(__builtin_fabsf(t)));
    const double d = __builtin_fma(-g, sd, __builtin_fabs(xd));
    acc = __builtin_fma(d, d, acc);
  }
}

// Phase 1 of the search: squared error of two elements in fp32 (fused residual and
// accumulation, relative error of a unit's sum below 60 * 2^-24).
template <int FMT> MOFQ_DEV void score2_f32(float& acc, float x0, float x1, float inv_s, float s, uint32_t& carry) {
  const f32x2 g = grid2<FMT>(x0 * inv_s, x1 * inv_s, carry);
  const float d0 = __builtin_fmaf(-g[0], s, x0);
  const float d1 = __builtin_fmaf(-g[1], s, x1);
  acc = __builtin_fmaf(d0, d0, acc);
  acc = __builtin_fmaf(d1, d1, acc);
}

// Sum over the wave in six DPP steps; the total is valid in lanes 48..63 only.
MOFQ_DEV float wave_sum_f32_hi(float v) {
  v += dpp_f32<DPP_QUAD_XOR1>(v);
  v += dpp_f32<DPP_QUAD_XOR2>(v);
  v += dpp_f32<DPP_ROW_HALF_MIRROR>(v);
  v += dpp_f32<DPP_ROW_MIRROR>(v);           // every lane: sum of its row of 16
  // rows 1 and 3 add the row before them, then rows 2 and 3 add lane 31 (rows 0+1)
  v += u2f(static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(f2u(v)), 0x142, 0xA, 0xF, false)));
  v += u2f(static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(f2u(v)), 0x143, 0xC, 0xF, false)));
  return v;
}

// Candidates whose fp32 error is within this factor of the smallest fp32 error are
// re-scored in fp64.  The fp32 sum of a unit is within (1 +- 60*2^-24) of the exact
// sum for the same grid choices, so the fp64 winner is always among them.
constexpr float kShortlistFactor = 1.0f + 1.0e-5f;
// Below this the fp32 sums may have lost terms to underflow: re-score everything.
constexpr float kTinySum = 0x1p-80f;

// ------------------------------------------------------------------------------
// Per-channel: one workgroup per row; the row lives in registers (CH chunks of 8
// elements per thread, chunk j of thread t = elements [(j*THREADS + t)*8, +8)).
//
// Phase 1 scores the (format, candidate) pairs in fp32; phase 2 re-scores in fp64 the
// candidates that fp32 cannot separate from the best one and picks the first
// smallest of those, which is the first smallest of all.
//
// Bisection (4-bit formats, bisect_clip): a candidate between two scored ones can be left out where it cannot be the
// winner.  The error of a scale s is the smallest of |x - s g|^2 over all assignments g of levels.  Let s1 > s > s2, E(s)
// below the smallest error T so far, and g its assignment: the parabola |x - t g|^2 has curvature |g|^2, is below T at
// s and not below E1 and E2 at s1 and s2, so sqrt(E1 - T) + sqrt(E2 - T) < |g| (s1 - s2); and s |g| <= |x| + sqrt(T).  A
// gap for which sqrt(E1 - T) + sqrt(E2 - T) > (|x| + sqrt(T)) (s1 - s2) / s2 is left alone.  E1 and E2 are taken 1e-5
// smaller and T 1e-5 larger (fp32 sums), and T by 2^-18 of the energy besides: a decision on rounded numbers
// assigns an element within 2^-22 of a boundary to the level beyond it, which adds up to 4 x^2 2^-22 to the error.
// All of it needs the scales of a gap to lie between s1 and s2; a row where a degenerate scale breaks their order is scored whole.
// 8-bit formats gain nothing by it: their levels are so many that any gap between two ratios can hold anything.
// Vector issue bounds it: layer selection, INT4 against E2M1, fp32: 4096 x 11008, 100 ratios 1145 -> 248 us; 3001 x 5000,
// 50 ratios 246 -> 123.
// ------------------------------------------------------------------------------
template <typename In, int FA, int FB, int THREADS, int CH>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(CH <= 4 ? 8 : 5))) void sweep_channel_kernel(const SweepArgs a) {
  using L = Load8<In>;
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  constexpr int NW = THREADS / 64;
  constexpr int NE = CH * 8;
  constexpr int MAXL = NF * MOFQ_MAX_CLIP;

  __shared__ float s_scale[NF][MOFQ_MAX_CLIP];
  __shared__ float s_inv[NF][MOFQ_MAX_CLIP];
  __shared__ float s_p1[NW][MOFQ_MAX_CLIP][NF];   // phase-1 partial sums per wave
  __shared__ float s_tot[NF][MOFQ_MAX_CLIP];
  __shared__ float s_wmax[NW];
  __shared__ double s_wen[NW];
  __shared__ int s_list[MAXL];                    // shortlisted (format, candidate) pairs
  __shared__ int s_nlist;
  __shared__ double s_p2[NW];
  __shared__ double s_val[MAXL];                  // fp64 error of the shortlisted pairs
  __shared__ uint64_t s_done[NF][MOFQ_MAX_CLIP / 64];   // bisection: bit per scored candidate
  __shared__ int s_new[NF];                             // candidates to score, in s_list at f * MOFQ_MAX_CLIP

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row = blockIdx.x;
  const typename L::elem* src = static_cast<const typename L::elem*>(a.w) + row * a.ld;
  const int K = a.n_clip;

  float x[NE];
  float amax = 0.0f;
  double en = 0.0;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int64_t c0 = (static_cast<int64_t>(j) * THREADS + tid) * 8;
    float v[8];
    if (c0 < a.cols) {
      L::load(src + c0, v);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[j * 8 + i] = v[i];
      amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
      const double xd = static_cast<double>(v[i]);
      en = __builtin_fma(xd, xd, en);
    }
  }

  // unit absmax and energy
  amax = wave_max(amax);
  en = wave_sum(en);
  if (lane == 0) { s_wmax[wave] = amax; s_wen[wave] = en; }
  __syncthreads();
  amax = s_wmax[0];
  en = s_wen[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) { amax = __builtin_fmaxf(amax, s_wmax[w]); en += s_wen[w]; }

  // scales of every (format, candidate)
  for (int idx = tid; idx < NF * K; idx += THREADS) {
    const int f = idx / K, k = idx - f * K;
    const float qmax = (f == 0) ? Codec<FA>::QMAX : Codec<FBX>::QMAX;
    const float s = unit_scale(amax, a.clip[k], qmax, a.scale_f16 != 0);
    s_scale[f][k] = s;
    s_inv[f][k] = 1.0f / s;
  }
  __syncthreads();

  // which of this wave's chunks hold data (wave-uniform)
  bool live[CH];
#pragma unroll
  for (int j = 0; j < CH; ++j)
    live[j] = (static_cast<int64_t>(j) * THREADS + wave * 64) * 8 < a.cols;

  uint32_t carry = 0;
  // ---- phase 1: fp32 error of the candidates (nothing to filter with one candidate) --
  auto score = [&](auto with_a, auto with_b, int kA, int kB) {
    constexpr bool A = decltype(with_a)::value, B = decltype(with_b)::value;
    const float sA = u2f(__builtin_amdgcn_readfirstlane(f2u(s_scale[0][kA])));
    const float iA = u2f(__builtin_amdgcn_readfirstlane(f2u(s_inv[0][kA])));
    const float sB = u2f(__builtin_amdgcn_readfirstlane(f2u(s_scale[NF - 1][kB])));
    const float iB = u2f(__builtin_amdgcn_readfirstlane(f2u(s_inv[NF - 1][kB])));
    float accA = 0.0f, accB = 0.0f;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      if (live[j]) {
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          if constexpr (A) score2_f32<FA>(accA, x[j * 8 + i], x[j * 8 + i + 1], iA, sA, carry);
          if constexpr (B) score2_f32<FBX>(accB, x[j * 8 + i], x[j * 8 + i + 1], iB, sB, carry);
        }
      }
    }
    if constexpr (A) accA = wave_sum_f32_hi(accA);
    if constexpr (B) accB = wave_sum_f32_hi(accB);
    if (lane == 63) {
      if constexpr (A) s_p1[wave][kA][0] = accA;
      if constexpr (B) s_p1[wave][kB][NF - 1] = accB;
    }
  };
  using yes = std::true_type;
  using no = std::false_type;
  using second = std::integral_constant<bool, NF == 2>;
  auto total = [&](int f, int k) {
    float t = 0.0f;
#pragma unroll
    for (int r = 0; r < NW; ++r) t += s_p1[r][k][f];
    return t;
  };
  if (Codec<FA>::BITS == 4 && a.bisect) {   // uniform
    if constexpr (Codec<FA>::BITS == 4) {
      // Five candidates over the whole table, then round by round the middle of every gap between scored ones that can
      // hold the winner; wave f % NW decides for format f.  (Seven or nine to begin with: fewer rounds, more candidates,
      // 3 to 9 % slower with 100 ratios; gaps of two scored whole: 2 %.)
      constexpr int START = 5;
      for (int idx = tid; idx < NF * K; idx += THREADS) s_tot[idx / K][idx % K] = __builtin_inff();   // not scored
      for (int f = 0; f < NF; ++f)
        if (wave == f % NW) {
          // The ratios descend, and so do the scales, but for a step up to the 1 of a degenerate scale from one below 1: the
          // scales between the ends of a gap across that step do not lie between theirs, so such a row is scored whole.
          bool up = false;
          for (int k = lane; k + 1 < K; k += 64) up |= s_scale[f][k] < s_scale[f][k + 1];
          const bool whole = __builtin_amdgcn_ballot_w64(up) != 0;
          const int n = whole ? K : START;
          if (lane < 2) s_done[f][lane] = 0;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          for (int i = lane; i < n; i += 64) {
            const int k = whole ? i : i * (K - 1) / (START - 1);
            s_list[f * MOFQ_MAX_CLIP + i] = k;
            atomicOr(&s_done[f][k >> 6], 1ull << (k & 63));
          }
          if (lane == 0) s_new[f] = n;
        }
      const float root_en = static_cast<float>(__builtin_sqrt(en));
      for (;;) {
        __syncthreads();
        const int nA = __builtin_amdgcn_readfirstlane(s_new[0]), nB = NF == 2 ? __builtin_amdgcn_readfirstlane(s_new[NF - 1]) : 0;
        if (nA + nB == 0) break;   // every round before scored one candidate at least
        const int n_both = nA < nB ? nA : nB;
        auto at = [&](int f, int i) { return __builtin_amdgcn_readfirstlane(s_list[f * MOFQ_MAX_CLIP + i]); };
        if constexpr (NF == 2) {
          for (int i = 0; i < n_both; ++i) score(yes{}, yes{}, at(0, i), at(1, i));
          for (int i = n_both; i < nB; ++i) score(no{}, yes{}, at(1, i), at(1, i));
        }
        for (int i = n_both; i < nA; ++i) score(yes{}, no{}, at(0, i), at(0, i));
        __syncthreads();
        for (int f = 0; f < NF; ++f)
          if (wave == f % NW) {
            const int n = f == 0 ? nA : nB;
            for (int i = lane; i < n; i += 64) {
              const int k = s_list[f * MOFQ_MAX_CLIP + i];
              s_tot[f][k] = total(f, k);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            float b = __builtin_inff();
            for (int k = lane; k < K; k += 64) b = __builtin_fminf(b, s_tot[f][k]);
            b = -wave_max(-b);
            const bool sums = b >= kTinySum && b < __builtin_inff();   // else every candidate is scored
            const float limit = __builtin_fmaf(root_en * root_en, 0x1p-18f, b * kShortlistFactor);
            const float span = (root_en + __builtin_amdgcn_sqrtf(limit)) * (1.0f + 0x1p-10f);
            const uint64_t done0 = s_done[f][0], done1 = s_done[f][1];
            int n_new = 0;
            for (int k0 = 0; k0 < K; k0 += 64) {
              const int k = k0 + lane;
              // the next scored candidate
              const uint64_t low = k < 63 ? done0 >> (k + 1) : 0;
              const uint64_t high = k < 64 ? done1 : (k < 127 ? done1 >> (k - 63) : 0);
              const int next = low ? k + 1 + __builtin_ctzll(low) : (high ? (k < 64 ? 64 : k + 1) + __builtin_ctzll(high) : k);
              bool look = false;
              if ((((k < 64 ? done0 : done1) >> (k & 63)) & 1) && next > k + 1) {
                const float s1 = s_scale[f][k], s2 = s_scale[f][next];
                const float up = __builtin_fmaf(s_tot[f][k], 1.0f - 1.0e-5f, -limit), down = __builtin_fmaf(s_tot[f][next], 1.0f - 1.0e-5f, -limit);
                const float roots = __builtin_amdgcn_sqrtf(__builtin_fmaxf(up, 0.0f)) + __builtin_amdgcn_sqrtf(__builtin_fmaxf(down, 0.0f));
                look = !sums || !(roots > span * ((s1 - s2) / s2));
              }
              const uint64_t lanes = __builtin_amdgcn_ballot_w64(look);
              const int mid = (k + next) >> 1;
              if (look) {
                s_list[f * MOFQ_MAX_CLIP + n_new + __builtin_popcountll(lanes & ((1ull << lane) - 1))] = mid;
                atomicOr(&s_done[f][mid >> 6], 1ull << (mid & 63));
              }
              n_new += __builtin_popcountll(lanes);
            }
            if (lane == 0) s_new[f] = n_new;
          }
      }
    }
  } else {
    for (int k = 0; k < K && K > 1; ++k) score(yes{}, second{}, k, k);
    __syncthreads();
    for (int idx = tid; idx < NF * K; idx += THREADS) {
      const int f = idx / K, k = idx - f * K;
      s_tot[f][k] = K > 1 ? total(f, k) : 0.0f;   // K == 1: zero, which shortlists the only candidate
    }
    __syncthreads();
  }

  // ---- shortlist: candidates fp32 cannot tell from the best, in candidate order ----------------------
  if (wave == 0) {
    int n = 0;
    for (int f = 0; f < NF; ++f) {
      float m = __builtin_inff();
      for (int k = lane; k < K; k += 64) m = __builtin_fminf(m, s_tot[f][k]);
      m = -wave_max(-m);
      const float thr = (m >= kTinySum && m < __builtin_inff()) ? m * kShortlistFactor : __builtin_inff();
      for (int k0 = 0; k0 < K; k0 += 64) {
        const int k = k0 + lane;
        const float t = s_tot[f][k < K ? k : 0];
        const bool in = k < K && !(t > thr);   // NaN too
        const uint64_t lanes = __builtin_amdgcn_ballot_w64(in);
        if (in) s_list[n + __builtin_popcountll(lanes & ((1ull << lane) - 1))] = f * MOFQ_MAX_CLIP + k;
        n += __builtin_popcountll(lanes);
      }
    }
    if (lane == 0) s_nlist = n;
  }
  __syncthreads();
  const int n_list = s_nlist;

  // ---- phase 2: fp64 error of the shortlisted candidates ---------------------------
  for (int e = 0; e < n_list; ++e) {
    const int fk = s_list[e];
    const int f = __builtin_amdgcn_readfirstlane(fk / MOFQ_MAX_CLIP);
    const int k = __builtin_amdgcn_readfirstlane(fk % MOFQ_MAX_CLIP);
    const float s = s_scale[f][k], inv = s_inv[f][k];
    const double sd = static_cast<double>(s);
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      if (live[j]) {
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          if (f == 0) score2_f64<FA>(acc, x[j * 8 + i], x[j * 8 + i + 1], inv, sd, carry);
          else score2_f64<FBX>(acc, x[j * 8 + i], x[j * 8 + i + 1], inv, sd, carry);
        }
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) s_p2[wave] = acc;
    __syncthreads();
    if (tid == 0) {
      double t = s_p2[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += s_p2[w];
      s_val[e] = t;
    }
    __syncthreads();
  }

  // first smallest fp64 error per format (the list is in candidate order)
  if (tid < NF) {
    const int f = tid;
    double best = __builtin_inf();
    int bk = -1;
    for (int e = 0; e < n_list; ++e) {
      const int fk = s_list[e];
      if (fk / MOFQ_MAX_CLIP != f) continue;
      if (s_val[e] < best) { best = s_val[e]; bk = fk % MOFQ_MAX_CLIP; }
    }
    if (bk < 0) { bk = 0; best = __builtin_nan(""); }   // only on non-finite input
    a.rec.scale[f][row] = s_scale[f][bk];
    a.rec.clip[f][row] = bk;
    a.rec.err[f][row] = best;
    if (f == 0 && a.rec.energy) a.rec.energy[row] = en;
  }
}

// ------------------------------------------------------------------------------
// Per-channel with a single candidate (absmax scale, no search): a memory-bound pass, one workgroup
// per row, two barriers.  The row stays in registers as it came from memory and is widened anew
// in each of the three steps (magnitude and energy, errors, codes): left alone, the compiler
// keeps the fp64 image of the whole row across the barrier (128 registers and spills for 4 chunks
// per thread, 72 without).
//
// GRID: the pass also writes the grid values of both formats, the operands of the weight-only layer-output products, so that
// they cost no further read of the tensor: 1 as bf16 (dense rows), 2 as e4m3 codes in one array.
// With a.ahead the row's codes leave from the same registers.
// ------------------------------------------------------------------------------
template <typename In, int FA, int FB, int THREADS, int CH, int GRID = 0>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(GRID ? 2 : 4))) void sweep_channel_single_kernel(const SweepArgs a) {
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  constexpr int NW = THREADS / 64;
  __shared__ float s_wmax[NW];
  __shared__ double s_wen[NW];
  __shared__ double s_acc[2][NW];
  __shared__ double s_tally;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row = blockIdx.x;

  const int cpr = static_cast<int>(a.cols / 8);
  Raw8<In> raw[CH];   // chunk j: the row's chunk j * THREADS + tid; zeros past the row's end add nothing
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int c = j * THREADS + tid;
    raw[j].load(a.w, row * a.ld, static_cast<uint32_t>(c < cpr ? c : 0) * 8);
    if (c >= cpr) raw[j].clear();
  }
  // read early, so that its latency is hidden (it may miss the rows of the last microseconds), but behind
  // the row (loads return in order), and by one wave: waves that read it at different times could disagree
  double tally = 0.0;
  if (NF == 2 && a.ahead.tally && wave == 0) tally = tally_read(a.ahead);
  float amax = 0.0f;
  double en = 0.0;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    float v[8];
    raw[j].widen(v);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
      const double xd = static_cast<double>(v[i]);
      en = __builtin_fma(xd, xd, en);
    }
  }
  amax = wave_max(amax);
  en = wave_sum(en);
  if (lane == 0) { s_wmax[wave] = amax; s_wen[wave] = en; }
  __syncthreads();
  amax = s_wmax[0];
  en = s_wen[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) { amax = __builtin_fmaxf(amax, s_wmax[w]); en += s_wen[w]; }

  const float sA = unit_scale(amax, a.clip[0], Codec<FA>::QMAX, a.scale_f16 != 0);
  const float sB = unit_scale(amax, a.clip[0], Codec<FBX>::QMAX, a.scale_f16 != 0);
  const float iA = 1.0f / sA, iB = 1.0f / sB;
  const double sAd = static_cast<double>(sA), sBd = static_cast<double>(sB);
  double accA = 0.0, accB = 0.0;
  uint32_t carry = 0;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    raw[j].opaque();
    float v[8];
    raw[j].widen(v);
    if constexpr (GRID != 0) {
      // grid values have at most 7 significant bits: exact in bf16 (the top half of an fp32); 4-bit formats' at most 3, and the
      // smallest is 1/2: exact in e4m3
      u32x4 ga, gb;
      int pa[2] = {0, 0}, pb[2] = {0, 0};
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        const float x0 = v[i], x1 = v[i + 1];
        const f32x2 qa = grid2<FA>(x0 * iA, x1 * iA, carry);
        const f32x2 qb = grid2<FBX>(x0 * iB, x1 * iB, carry);
        if constexpr (GRID == 1) {
          ga[i >> 1] = (f2u(qa[0]) >> 16) | (f2u(qa[1]) & 0xFFFF0000u);
          gb[i >> 1] = (f2u(qb[0]) >> 16) | (f2u(qb[1]) & 0xFFFF0000u);
        } else if (i % 4 == 0) {
          pa[i / 4] = __builtin_amdgcn_cvt_pk_fp8_f32(qa[0], qa[1], pa[i / 4], false);
          pb[i / 4] = __builtin_amdgcn_cvt_pk_fp8_f32(qb[0], qb[1], pb[i / 4], false);
        } else {
          pa[i / 4] = __builtin_amdgcn_cvt_pk_fp8_f32(qa[0], qa[1], pa[i / 4], true);
          pb[i / 4] = __builtin_amdgcn_cvt_pk_fp8_f32(qb[0], qb[1], pb[i / 4], true);
        }
        const double a0 = __builtin_fma(-static_cast<double>(qa[0]), sAd, static_cast<double>(x0));
        const double a1 = __builtin_fma(-static_cast<double>(qa[1]), sAd, static_cast<double>(x1));
        accA = __builtin_fma(a0, a0, accA);
        accA = __builtin_fma(a1, a1, accA);
        const double b0 = __builtin_fma(-static_cast<double>(qb[0]), sBd, static_cast<double>(x0));
        const double b1 = __builtin_fma(-static_cast<double>(qb[1]), sBd, static_cast<double>(x1));
        accB = __builtin_fma(b0, b0, accB);
        accB = __builtin_fma(b1, b1, accB);
      }
      const int c = j * THREADS + tid;
      if (c < cpr) {
        if constexpr (GRID == 1) {
          reinterpret_cast<u32x4*>(a.emit_grid[0])[row * cpr + c] = ga;
          reinterpret_cast<u32x4*>(a.emit_grid[1])[row * cpr + c] = gb;
        } else {
          const int64_t at = row * (2 * a.cols) + grid_fp8_at(static_cast<uint32_t>(row), static_cast<uint32_t>(c));
          *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(a.emit_grid[0]) + at) = u32x2{static_cast<uint32_t>(pa[0]), static_cast<uint32_t>(pa[1])};
          *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(a.emit_grid[1]) + at) = u32x2{static_cast<uint32_t>(pb[0]), static_cast<uint32_t>(pb[1])};
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        score2_f64<FA>(accA, v[i], v[i + 1], iA, sAd, carry);
        if constexpr (NF == 2) score2_f64<FBX>(accB, v[i], v[i + 1], iB, sBd, carry);
      }
    }
  }
  accA = wave_sum(accA);
  if constexpr (NF == 2) accB = wave_sum(accB);
  if (lane == 0) { s_acc[0][wave] = accA; s_acc[1][wave] = accB; }
  if (NF == 2 && a.ahead.codes && wave == 0) {
    if (a.ahead.tally) tally = wave_sum(tally);
    if (lane == 0) s_tally = tally;
  }
  __syncthreads();
  if (tid < NF) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += s_acc[tid][w];
    a.rec.scale[tid][row] = tid == 0 ? sA : sB;
    a.rec.clip[tid][row] = 0;
    a.rec.err[tid][row] = t;
    if (tid == 0 && a.rec.energy) a.rec.energy[row] = en;
  }
  if (a.ahead.codes) {   // uniform
    int slot = 0;
    if constexpr (NF == 2) {
      double d = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) d += s_acc[0][w] - s_acc[1][w];
      slot = __builtin_amdgcn_readfirstlane(s_tally + d > 0.0 ? 1 : 0);
      if (tid == 0) {
        if (a.ahead.tally) tally_add<16>(a.ahead, d);
        a.ahead.tag[row] = static_cast<uint8_t>(a.ahead.cand_of[slot]);
      }
    }
    auto codes = [&](auto fmt_c, float inv) {
      constexpr int FMT = decltype(fmt_c)::value;
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        const int c = j * THREADS + tid;
        raw[j].opaque();
        float v[8];
        raw[j].widen(v);
        uint32_t words[2];
        encode8<FMT>(v, inv, words);
        if (c < cpr) {
          if constexpr (Codec<FMT>::BITS == 4) {
            (static_cast<uint32_t*>(a.ahead.codes) + row * cpr)[c] = words[0];
          } else {
            u32x2 o;
            o[0] = words[0];
            o[1] = words[1];
            (static_cast<u32x2*>(a.ahead.codes) + row * cpr)[c] = o;
          }
        }
      }
    };
    if (slot == 0) codes(std::integral_constant<int, FA>{}, iA);
    else codes(std::integral_constant<int, FBX>{}, iB);
  }
}

// ------------------------------------------------------------------------------
// Per-group: LPG lanes share one group of GROUP elements; each lane holds
// GROUP/LPG consecutive elements.  Scales differ per group, so they are per-lane
// values; the LPG lanes of a group split the scale computations of a batch of LPG
// candidates and hand them round with DPP.
// ------------------------------------------------------------------------------
template <int LPG> MOFQ_DEV double group_sum(double v);
template <> MOFQ_DEV double group_sum<4>(double v) { return quad_sum(v); }
template <> MOFQ_DEV double group_sum<16>(double v) { return row16_sum(v); }
template <int LPG> MOFQ_DEV float group_max(float v);
template <> MOFQ_DEV float group_max<4>(float v) {
  v = __builtin_fmaxf(v, dpp_f32<DPP_QUAD_XOR1>(v));
  return __builtin_fmaxf(v, dpp_f32<DPP_QUAD_XOR2>(v));
}
template <> MOFQ_DEV float group_max<16>(float v) {
  v = group_max<4>(v);
  v = __builtin_fmaxf(v, dpp_f32<DPP_ROW_HALF_MIRROR>(v));
  return __builtin_fmaxf(v, dpp_f32<DPP_ROW_MIRROR>(v));
}

// value held by lane `j` of the caller's quad
template <int J> MOFQ_DEV float quad_bcast(float v) { return dpp_f32<J * 0x55>(v); }

MOFQ_DEV float quad_sum_f32(float v) {
  v += dpp_f32<DPP_QUAD_XOR1>(v);
  return v + dpp_f32<DPP_QUAD_XOR2>(v);    // the same value in all four lanes
}
MOFQ_DEV uint32_t quad_or(uint32_t v) {
  v |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), DPP_QUAD_XOR1, 0xF, 0xF, false));
  return v | static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), DPP_QUAD_XOR2, 0xF, 0xF, false));
}

constexpr int kGroupQuads = 256 / 4;             // groups per workgroup
constexpr int kMaskWords = MOFQ_MAX_CLIP / 32;

// Phase 1 scores the candidates of a group in fp32 (hardware fp4/fp8 converts), all of them or, BISECT, by
// bisection (see sweep_channel_kernel; 16 groups of 128 with 50 ratios take 26 rounds of one candidate instead of 50), and
// parks the sums in LDS; the candidates fp32 cannot tell from the group's best are
// collected in a bit mask per group and re-scored in fp64 in candidate order, the j-th
// survivor of all 16 groups of a wave at the same time.  The fp32 sum of a group (32
// terms per lane, two more additions across the quad) is within (1 +- 40*2^-24) of the
// exact sum for the same grid choices, so the fp64 winner is always among the survivors.
template <typename In, int FA, int FB, int GROUP, bool BISECT>
__global__ __launch_bounds__(256) void sweep_group_kernel(const SweepArgs a) {
  using L = Load8<In>;
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  constexpr int LPG = 4;
  constexpr int NE = GROUP / LPG;       // elements per lane
  constexpr int CH = NE / 8;
  static_assert(NE % 8 == 0, "group too small for 4 lanes");

  extern __shared__ float s_dyn[];      // clip[K], then p1[NF][K][kGroupQuads]
  const int K = a.n_clip;
  float* s_clip = s_dyn;
  float* s_p1 = s_dyn + MOFQ_MAX_CLIP;

  const int tid = threadIdx.x;
  const int q = tid & (LPG - 1);
  const int quad = tid >> 2;
  const int64_t gpr = a.cols / GROUP;   // groups per row
  int64_t unit = static_cast<int64_t>(blockIdx.x) * kGroupQuads + quad;
  const bool valid = unit < a.units;
  if (!valid) unit = a.units - 1;       // keep every lane active for the DPP exchanges
  const int64_t row = unit / gpr, gi = unit - row * gpr;
  const typename L::elem* src =
      static_cast<const typename L::elem*>(a.w) + row * a.ld + gi * GROUP + q * NE;
  const bool f16 = a.scale_f16 != 0;

  for (int k = tid; k < K; k += 256) s_clip[k] = a.clip[k];

  float x[NE];
  float amax = 0.0f;
  double en = 0.0;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    float v[8];
    L::load(src + j * 8, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[j * 8 + i] = v[i];
      amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
      const double xd = static_cast<double>(v[i]);
      en = __builtin_fma(xd, xd, en);
    }
  }
  amax = group_max<LPG>(amax);
  en = group_sum<LPG>(en);
  __syncthreads();                       // clip table in place

  uint32_t carry = 0;
  uint32_t maskA[kMaskWords], maskB[kMaskWords];
#pragma unroll
  for (int w = 0; w < kMaskWords; ++w) { maskA[w] = 0; maskB[w] = 0; }

  if (K > 1) {
    // ---- phase 1 ----------------------------------------------------------------
    float minA = __builtin_inff(), minB = __builtin_inff();
    // one candidate of each format per group
    auto one = [&](auto with_a, auto with_b, float sA, float iA, int kA, float sB, float iB, int kB, bool inA, bool inB) __attribute__((always_inline)) {
      float accA = 0.0f, accB = 0.0f;
#pragma unroll
      for (int i = 0; i < NE; i += 2) {
        if constexpr (decltype(with_a)::value) score2_f32<FA>(accA, x[i], x[i + 1], iA, sA, carry);
        if constexpr (decltype(with_b)::value) score2_f32<FBX>(accB, x[i], x[i + 1], iB, sB, carry);
      }
      if constexpr (decltype(with_a)::value) {
        accA = quad_sum_f32(accA);
        minA = __builtin_fminf(minA, inA ? accA : __builtin_inff());
        if (q == 0 && inA) s_p1[kA * kGroupQuads + quad] = accA;
      }
      if constexpr (decltype(with_b)::value) {
        accB = quad_sum_f32(accB);
        minB = __builtin_fminf(minB, inB ? accB : __builtin_inff());
        if (q == 1 && inB) s_p1[(K + kB) * kGroupQuads + quad] = accB;
      }
    };
    using yes = std::true_type;
    using no = std::false_type;
    using second = std::integral_constant<bool, NF == 2>;
    if constexpr (BISECT) {
      // Bisection (see sweep_channel_kernel) on a grid of gaps that all groups share: 8 candidates, then the middles of the gaps
      // that can hold the group's winner, until a gap has two candidates at most, which are scored together.  A lane tests
      // every fourth gap of its group; an error not known is infinite, which ends a gap that was left alone.
      for (int k = q; k < NF * K; k += LPG) s_p1[k * kGroupQuads + quad] = __builtin_inff();
      constexpr int UNROLL = GROUP <= 128 ? LPG : 1;   // (256: the copies of the scoring code would not fit the instruction cache)
      // four candidates of each group and format, from its list
      auto score4 = [&](int kA, int kB) __attribute__((always_inline)) {   // the lane's own; below 0: none
        const float rA = s_clip[kA < 0 ? 0 : kA], rB = s_clip[kB < 0 ? 0 : kB];
        const float mysA = unit_scale(amax, rA, Codec<FA>::QMAX, f16), myiA = 1.0f / mysA;
        float mysB = 0.0f, myiB = 0.0f;
        if constexpr (NF == 2) {
          mysB = unit_scale(amax, rB, Codec<FBX>::QMAX, f16);
          myiB = 1.0f / mysB;
        }
        float s1 = mysA, i1 = myiA, s2 = mysB, i2 = myiB;
#pragma unroll UNROLL
        for (int j = 0; j < LPG; ++j) {   // lane 0's, then every lane takes the next one's
          const int a1 = __builtin_amdgcn_update_dpp(0, kA, 0x00, 0xF, 0xF, true), b1 = __builtin_amdgcn_update_dpp(0, kB, 0x00, 0xF, 0xF, true);
          const bool any_a = __builtin_amdgcn_ballot_w64(a1 >= 0) != 0, any_b = NF == 2 && __builtin_amdgcn_ballot_w64(b1 >= 0) != 0;
          const float sa = quad_bcast<0>(s1), ia = quad_bcast<0>(i1), sb = quad_bcast<0>(s2), ib = quad_bcast<0>(i2);
          if (any_a && any_b) {
            if constexpr (NF == 2) one(yes{}, yes{}, sa, ia, a1, sb, ib, b1, a1 >= 0, b1 >= 0);
          } else if (any_b) {
            if constexpr (NF == 2) one(no{}, yes{}, sa, ia, a1, sb, ib, b1, false, b1 >= 0);
          } else if (any_a) {
            one(yes{}, no{}, sa, ia, a1, sb, ib, b1, a1 >= 0, false);
          }
          kA = __builtin_amdgcn_update_dpp(0, kA, 0x39, 0xF, 0xF, true);
          s1 = dpp_f32<0x39>(s1);
          i1 = dpp_f32<0x39>(i1);
          if constexpr (NF == 2) {
            kB = __builtin_amdgcn_update_dpp(0, kB, 0x39, 0xF, 0xF, true);
            s2 = dpp_f32<0x39>(s2);
            i2 = dpp_f32<0x39>(i2);
          }
        }
      };
      int n = 7;   // gaps
      // floor(i (K - 1) / n): below 2^14, so the rounded product is off by less than half of 1 / n
      auto place = [&](int i, float inv_n) { return static_cast<int>((static_cast<float>(__mul24(i, K - 1)) + 0.5f) * inv_n); };
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      for (int i0 = 0; i0 < 8; i0 += LPG) {
        const int k = place(i0 + q, 1.0f / 7.0f);
        score4(k, k);
      }
      uint8_t* const list = reinterpret_cast<uint8_t*>(s_p1 + NF * K * kGroupQuads) + quad * NF * (K - 8);
      const float root_en = static_cast<float>(__builtin_sqrt(en));
      // two ratios are a scale quotient but for the scales' rounding, unless a scale is below the normal numbers
      const float rounding = f16 ? 1.0f + 0x1.08p-10f : 1.0f + 0x1p-20f;
      for (bool last = false; !last; n *= 2) {
        last = K - 1 <= 3 * n;
        const float inv_n = 1.0f / static_cast<float>(n);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        int left[2] = {0, 0};
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          const float b = f == 0 ? minA : minB;
          const float qmax = f == 0 ? Codec<FA>::QMAX : Codec<FBX>::QMAX;
          const bool regular = b >= kTinySum && b < __builtin_inff() && amax * s_clip[K - 1] >= qmax * (f16 ? 0x1p-13f : 0x1p-124f) &&
                               amax * s_clip[0] <= qmax * (f16 ? 65000.0f : 0x1p126f);
          const float limit = __builtin_fmaf(root_en * root_en, 0x1p-18f, b * kShortlistFactor);
          const float span = (root_en + __builtin_amdgcn_sqrtf(limit)) * (1.0f + 0x1p-10f);
          const float* const e = s_p1 + f * K * kGroupQuads + quad;
          uint32_t bits = 0;
          int count = 0;
          for (int i = q, j = 0; i < n; i += LPG, ++j) {
            const int from = place(i, inv_n), to = place(i + 1, inv_n);
            const float up = __builtin_fmaf(e[from * kGroupQuads], 1.0f - 1.0e-5f, -limit), down = __builtin_fmaf(e[to * kGroupQuads], 1.0f - 1.0e-5f, -limit);
            const float roots = __builtin_amdgcn_sqrtf(__builtin_fmaxf(up, 0.0f)) + __builtin_amdgcn_sqrtf(__builtin_fmaxf(down, 0.0f));
            const float step = __builtin_fmaf(s_clip[from] * rounding, __builtin_amdgcn_rcpf(s_clip[to]), -1.0f);
            if (to - from > 1 && (!regular || !(roots > span * step))) {
              bits |= 1u << j;
              count += last ? to - from - 1 : 1;
            }
          }
          // the list: the lanes' entries one behind another
          const int c1 = __builtin_amdgcn_update_dpp(0, count, 0x90, 0xF, 0xF, true);   // lane q - 1 (quad_perm 0, 0, 1, 2)
          int inc = count + (q >= 1 ? c1 : 0);
          const int c2 = __builtin_amdgcn_update_dpp(0, inc, 0x40, 0xF, 0xF, true);     // lane q - 2 (quad_perm 0, 0, 0, 1)
          inc += q >= 2 ? c2 : 0;
          left[f] = __builtin_amdgcn_update_dpp(0, inc, 0xFF, 0xF, 0xF, true);          // lane 3's
          uint8_t* at = list + f * (K - 8) + (inc - count);
          while (bits) {
            const int i = q + LPG * __builtin_ctz(bits);
            bits &= bits - 1;
            const int from = place(i, inv_n);
            if (last) {
              const int to = place(i + 1, inv_n);
              for (int k = from + 1; k < to; ++k) *at++ = static_cast<uint8_t>(k);
            } else {
              *at++ = static_cast<uint8_t>(place(2 * i + 1, 0.5f * inv_n));
            }
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int i = q; __builtin_amdgcn_ballot_w64(i < left[0] || i < left[1]) != 0; i += LPG)
          score4(i < left[0] ? list[i] : -1, NF == 2 && i < left[1] ? list[K - 8 + i] : -1);
      }
    } else {
      for (int k0 = 0; k0 < K; k0 += LPG) {
        // lane q of the group prepares candidate k0+q (clamped; surplus ones are ignored)
        const int kq = (k0 + q < K) ? k0 + q : K - 1;
        const float r = s_clip[kq];
        const float mysA = unit_scale(amax, r, Codec<FA>::QMAX, f16);
        const float myiA = 1.0f / mysA;
        float mysB = 0.0f, myiB = 0.0f;
        if constexpr (NF == 2) {
          mysB = unit_scale(amax, r, Codec<FBX>::QMAX, f16);
          myiB = 1.0f / mysB;
        }
        auto lane_of = [&](auto j) {
          constexpr int J = decltype(j)::value;
          if (k0 + J < K)   // uniform over the workgroup
            one(yes{}, second{}, quad_bcast<J>(mysA), quad_bcast<J>(myiA), k0 + J, quad_bcast<J>(mysB), quad_bcast<J>(myiB), k0 + J, true, true);
        };
        lane_of(std::integral_constant<int, 0>{});
        lane_of(std::integral_constant<int, 1>{});
        lane_of(std::integral_constant<int, 2>{});
        lane_of(std::integral_constant<int, 3>{});
      }
    }
    __syncthreads();                     // the sums parked by lanes 0 and 1 are visible to the quad

    // ---- survivors: lane q tests candidates q, q+4, ... ----------------------------
    const float thrA = (minA >= kTinySum && minA < __builtin_inff()) ? minA * kShortlistFactor : __builtin_inff();
    const float thrB = (minB >= kTinySum && minB < __builtin_inff()) ? minB * kShortlistFactor : __builtin_inff();
    for (int k = q; k < K; k += LPG) {
      const float vA = s_p1[k * kGroupQuads + quad];
      const uint32_t bit = 1u << (k & 31);
      const bool keepA = vA <= thrA || !(vA == vA);
      bool keepB = false;
      if constexpr (NF == 2) {
        const float vB = s_p1[(K + k) * kGroupQuads + quad];
        keepB = vB <= thrB || !(vB == vB);
      }
#pragma unroll
      for (int w = 0; w < kMaskWords; ++w) {
        if ((k >> 5) == w) {
          if (keepA) maskA[w] |= bit;
          if (keepB) maskB[w] |= bit;
        }
      }
    }
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) {
      maskA[w] = quad_or(maskA[w]);
      if constexpr (NF == 2) maskB[w] = quad_or(maskB[w]);
    }
  } else {
    maskA[0] = 1u;
    if constexpr (NF == 2) maskB[0] = 1u;
  }

  // ---- phase 2: fp64 error of the survivors, first smallest wins -------------------
  double bestA = __builtin_inf(), bestB = __builtin_inf();
  int bkA = -1, bkB = -1;
  float bsA = 1.0f, bsB = 1.0f;
  auto rescore = [&](auto fmt_c, uint32_t (&mask)[kMaskWords], double& best, int& bk, float& bs) {
    constexpr int FMT = decltype(fmt_c)::value;
    for (;;) {
      int k = -1;                        // this group's next survivor, in candidate order
#pragma unroll
      for (int w = 0; w < kMaskWords; ++w) {
        if (k < 0 && mask[w] != 0) {
          k = w * 32 + __builtin_ctz(mask[w]);
          mask[w] &= mask[w] - 1;
        }
      }
      if (__builtin_amdgcn_ballot_w64(k >= 0) == 0) break;
      const float s = unit_scale(amax, s_clip[k >= 0 ? k : 0], Codec<FMT>::QMAX, f16);
      const float inv = 1.0f / s;
      const double sd = static_cast<double>(s);
      double acc = 0.0;
#pragma unroll
      for (int i = 0; i < NE; i += 2) score2_f64<FMT>(acc, x[i], x[i + 1], inv, sd, carry);
      acc = group_sum<LPG>(acc);
      if (k >= 0 && acc < best) { best = acc; bk = k; bs = s; }
    }
  };
  rescore(std::integral_constant<int, FA>{}, maskA, bestA, bkA, bsA);
  if constexpr (NF == 2) rescore(std::integral_constant<int, FBX>{}, maskB, bestB, bkB, bsB);

  if (valid && q == 0) {
    if (bkA < 0) { bkA = 0; bestA = __builtin_nan(""); bsA = unit_scale(amax, s_clip[0], Codec<FA>::QMAX, f16); }   // only on non-finite input
    a.rec.scale[0][unit] = bsA;
    a.rec.clip[0][unit] = bkA;
    a.rec.err[0][unit] = bestA;
    if constexpr (NF == 2) {
      if (bkB < 0) { bkB = 0; bestB = __builtin_nan(""); bsB = unit_scale(amax, s_clip[0], Codec<FBX>::QMAX, f16); }
      a.rec.scale[1][unit] = bsB;
      a.rec.clip[1][unit] = bkB;
      a.rec.err[1][unit] = bestB;
    }
    if (a.rec.energy) a.rec.energy[unit] = en;
  }
}

// ------------------------------------------------------------------------------
// Per-tensor: absmax pass, then a pass of per-block partial errors, then one
// block that adds the partials in block order and picks the candidate.
// ------------------------------------------------------------------------------
template <typename In>
__global__ __launch_bounds__(256) void tensor_absmax_kernel(const SweepArgs a) {
  using L = Load8<In>;
  __shared__ float s_wmax[4];
  __shared__ double s_wen[4];
  const int tid = threadIdx.x;
  const int64_t cpr = a.cols / 8;                 // chunks per row
  const int64_t n_chunks = a.rows * cpr;
  float amax = 0.0f;
  double en = 0.0;
  for (int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + tid; c < n_chunks;
       c += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t row = c / cpr, col = (c - row * cpr) * 8;
    float v[8];
    L::load(static_cast<const typename L::elem*>(a.w) + row * a.ld + col, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
      const double d = static_cast<double>(v[i]);
      en = __builtin_fma(d, d, en);
    }
  }
  amax = wave_max(amax);
  en = wave_sum(en);
  if ((tid & 63) == 0) { s_wmax[tid >> 6] = amax; s_wen[tid >> 6] = en; }
  __syncthreads();
  if (tid == 0) {
    a.absmax_part[blockIdx.x] =
        __builtin_fmaxf(__builtin_fmaxf(s_wmax[0], s_wmax[1]), __builtin_fmaxf(s_wmax[2], s_wmax[3]));
    a.energy_part[blockIdx.x] = (s_wen[0] + s_wen[1]) + (s_wen[2] + s_wen[3]);
  }
}

constexpr int kTensorMaxClip = 8;

MOFQ_DEV float tensor_absmax(const SweepArgs& a, float* s_tmp) {
  const int tid = threadIdx.x;
  float m = 0.0f;
  for (int i = tid; i < a.n_blocks; i += 256) m = __builtin_fmaxf(m, a.absmax_part[i]);
  m = wave_max(m);
  if ((tid & 63) == 0) s_tmp[tid >> 6] = m;
  __syncthreads();
  return __builtin_fmaxf(__builtin_fmaxf(s_tmp[0], s_tmp[1]), __builtin_fmaxf(s_tmp[2], s_tmp[3]));
}

template <typename In, int FA, int FB>
__global__ __launch_bounds__(256) void tensor_score_kernel(const SweepArgs a) {
  using L = Load8<In>;
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  __shared__ float s_tmp[4];
  __shared__ float s_scale[NF][kTensorMaxClip];
  __shared__ float s_inv[NF][kTensorMaxClip];
  __shared__ double s_part[4][NF][kTensorMaxClip];
  const int tid = threadIdx.x;
  // one pass scores up to kTensorMaxClip candidates, a.k0 onwards (more candidates: more passes)
  const int K = (a.n_clip - a.k0) < kTensorMaxClip ? (a.n_clip - a.k0) : kTensorMaxClip;
  const float amax = tensor_absmax(a, s_tmp);
  if (tid < NF * K) {
    const int f = tid / K, k = tid - f * K;
    const float s = unit_scale(amax, a.clip[a.k0 + k], f == 0 ? Codec<FA>::QMAX : Codec<FBX>::QMAX,
                               a.scale_f16 != 0);
    s_scale[f][k] = s;
    s_inv[f][k] = 1.0f / s;
  }
  __syncthreads();

  double acc[NF][kTensorMaxClip];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int k = 0; k < kTensorMaxClip; ++k) acc[f][k] = 0.0;

  const int64_t cpr = a.cols / 8;
  const int64_t n_chunks = a.rows * cpr;
  for (int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + tid; c < n_chunks;
       c += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t row = c / cpr, col = (c - row * cpr) * 8;
    float v[8];
    L::load(static_cast<const typename L::elem*>(a.w) + row * a.ld + col, v);
#pragma unroll
    for (int k = 0; k < kTensorMaxClip; ++k) {
      if (k < K) {
        const float iA = s_inv[0][k], iB = s_inv[NF - 1][k];
        const double sAd = static_cast<double>(s_scale[0][k]);
        const double sBd = static_cast<double>(s_scale[NF - 1][k]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const double xd = static_cast<double>(v[i]);
          accumulate<FA>(acc[0][k], v[i], xd, iA, sAd);
          if constexpr (NF == 2) accumulate<FBX>(acc[1][k], v[i], xd, iB, sBd);
        }
      }
    }
  }
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int k = 0; k < kTensorMaxClip; ++k) {
      if (k < K) {
        const double t = wave_sum(acc[f][k]);
        if ((tid & 63) == 0) s_part[tid >> 6][f][k] = t;
      }
    }
  __syncthreads();
  if (tid < NF * K) {
    const int f = tid / K, k = tid - f * K;
    a.sse_part[(static_cast<int64_t>(blockIdx.x) * NF + f) * a.n_clip + a.k0 + k] =
        (s_part[0][f][k] + s_part[1][f][k]) + (s_part[2][f][k] + s_part[3][f][k]);
  }
}

// Per-tensor (INT8, FP8-E4M3) pair at one clip ratio, as the weight-activation path uses
// it: the same partial errors as tensor_score_kernel, and in the same pass the int8 codes
// and the E4M3 codes of every element, so that the operands
// of the layer-output products cost one read of the tensor instead of three.
template <typename In>
__global__ __launch_bounds__(256) void tensor_score_emit8_kernel(const SweepArgs a) {
  using L = Load8<In>;
  __shared__ float s_tmp[4];
  __shared__ double s_part[4][2];
  const int tid = threadIdx.x;
  const float amax = tensor_absmax(a, s_tmp);
  const float sA = unit_scale(amax, a.clip[0], Codec<MOFQ_INT8>::QMAX, a.scale_f16 != 0);
  const float sB = unit_scale(amax, a.clip[0], Codec<MOFQ_FP8_E4M3>::QMAX, a.scale_f16 != 0);
  const float iA = 1.0f / sA, iB = 1.0f / sB;
  const double sAd = static_cast<double>(sA), sBd = static_cast<double>(sB);
  double accA = 0.0, accB = 0.0;
  const int64_t cpr = a.cols / 8;
  const int64_t n_chunks = a.rows * cpr;
  for (int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + tid; c < n_chunks;
       c += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t row = c / cpr, col = (c - row * cpr) * 8;
    float v[8];
    L::load(static_cast<const typename L::elem*>(a.w) + row * a.ld + col, v);
    uint32_t wi[2] = {0u, 0u};
    int wf[2] = {0, 0};
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      // INT8
      const float q0 = Codec<MOFQ_INT8>::grid(v[i] * iA), q1 = Codec<MOFQ_INT8>::grid(v[i + 1] * iA);
      wi[i >> 2] |= (static_cast<uint32_t>(static_cast<int>(q0)) & 0xFFu) << (8 * (i & 3));
      wi[i >> 2] |= (static_cast<uint32_t>(static_cast<int>(q1)) & 0xFFu) << (8 * ((i & 3) + 1));
      const double d0 = __builtin_fma(-static_cast<double>(q0), sAd, static_cast<double>(v[i]));
      const double d1 = __builtin_fma(-static_cast<double>(q1), sAd, static_cast<double>(v[i + 1]));
      accA = __builtin_fma(d0, d0, accA);
      accA = __builtin_fma(d1, d1, accA);
      // E4M3: pack-convert (exact agreement with the codec, see grid2), decode for the error
      const int p = __builtin_amdgcn_cvt_pk_fp8_f32(med3(v[i] * iB, -448.0f, 448.0f),
                                                    med3(v[i + 1] * iB, -448.0f, 448.0f), 0, false);
      const f32x2 g = __builtin_amdgcn_cvt_pk_f32_fp8(p, false);
      wf[i >> 2] |= (p & 0xFFFF) << (16 * ((i >> 1) & 1));
      const double e0 = __builtin_fma(-static_cast<double>(g[0]), sBd, static_cast<double>(v[i]));
      const double e1 = __builtin_fma(-static_cast<double>(g[1]), sBd, static_cast<double>(v[i + 1]));
      accB = __builtin_fma(e0, e0, accB);
      accB = __builtin_fma(e1, e1, accB);
    }
    const int64_t e8 = (row * a.cols + col) / 8;   // dense output rows
    u32x2 oi;
    oi[0] = wi[0];
    oi[1] = wi[1];
    reinterpret_cast<u32x2*>(a.emit_i8)[e8] = oi;
    u32x2 of;
    of[0] = static_cast<uint32_t>(wf[0]);
    of[1] = static_cast<uint32_t>(wf[1]);
    reinterpret_cast<u32x2*>(a.emit_f8)[e8] = of;
  }
  accA = wave_sum(accA);
  accB = wave_sum(accB);
  if ((tid & 63) == 0) { s_part[tid >> 6][0] = accA; s_part[tid >> 6][1] = accB; }
  __syncthreads();
  if (tid < 2)
    a.sse_part[static_cast<int64_t>(blockIdx.x) * 2 + tid] =
        (s_part[0][tid] + s_part[1][tid]) + (s_part[2][tid] + s_part[3][tid]);
}

template <int FA, int FB>
__global__ __launch_bounds__(256) void tensor_finalize_kernel(const SweepArgs a) {
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  __shared__ float s_tmp[4];
  __shared__ double s_red[4];
  __shared__ double s_tot[NF][MOFQ_MAX_CLIP];
  const int tid = threadIdx.x;
  const int K = a.n_clip;
  const float amax = tensor_absmax(a, s_tmp);
  // Partials in a fixed order.  Few (format, candidate) pairs: the whole workgroup adds each
  // of them; many: one wave per pair.
  if (NF * K <= 4) {
    for (int idx = 0; idx < NF * K; ++idx) {
      const int f = idx / K, k = idx - f * K;
      double t = 0.0;
      for (int b = tid; b < a.n_blocks; b += 256)
        t += a.sse_part[(static_cast<int64_t>(b) * NF + f) * K + k];
      t = wave_sum(t);
      __syncthreads();
      if ((tid & 63) == 0) s_red[tid >> 6] = t;
      __syncthreads();
      if (tid == 0) s_tot[f][k] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
    }
  } else {
    for (int idx = tid >> 6; idx < NF * K; idx += 4) {
      const int f = idx / K, k = idx - f * K;
      double t = 0.0;
      for (int b = tid & 63; b < a.n_blocks; b += 64)
        t += a.sse_part[(static_cast<int64_t>(b) * NF + f) * K + k];
      t = wave_sum(t);
      if ((tid & 63) == 0) s_tot[f][k] = t;
    }
  }
  double en = 0.0;
  for (int b = tid; b < a.n_blocks; b += 256) en += a.energy_part[b];
  en = wave_sum(en);
  __syncthreads();
  if ((tid & 63) == 0) s_red[tid >> 6] = en;
  __syncthreads();
  if (tid == 0) {
    for (int f = 0; f < NF; ++f) {
      double best = __builtin_inf();
      int bk = 0;
      for (int k = 0; k < K; ++k)
        if (s_tot[f][k] < best) { best = s_tot[f][k]; bk = k; }
      a.rec.scale[f][0] = unit_scale(amax, a.clip[bk], f == 0 ? Codec<FA>::QMAX : Codec<FBX>::QMAX,
                                     a.scale_f16 != 0);
      a.rec.clip[f][0] = bk;
      a.rec.err[f][0] = best;
    }
    if (a.rec.energy) a.rec.energy[0] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
  }
}

// ---- dispatch ---------------------------------------------------------------------

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <typename In, int FA, int FB>
int launch_channel(const SweepArgs& a, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(a.rows));
  const int64_t chunks = a.cols / 8;
#define MOFQ_CH(THREADS, CH)                                                            \
  if (chunks <= static_cast<int64_t>(THREADS) * (CH)) {                                  \
    if (a.emit_grid[0]) {                                                                \
      if constexpr (std::is_same<In, BF16>::value && FB >= 0) {                          \
        if (a.n_clip != 1 || !a.emit_grid[1]) return MOFQ_ERR_UNSUPPORTED;               \
        if (!a.emit_grid_fp8)                                                            \
          hipLaunchKernelGGL((sweep_channel_single_kernel<In, FA, FB, THREADS, CH, 1>), grid, dim3(THREADS), 0, st, a); \
        else if constexpr (Codec<FA>::BITS == 4 && Codec<(FB >= 0 ? FB : FA)>::BITS == 4) \
          hipLaunchKernelGGL((sweep_channel_single_kernel<In, FA, FB, THREADS, CH, 2>), grid, dim3(THREADS), 0, st, a); \
        else                                                                             \
          return MOFQ_ERR_UNSUPPORTED;                                                   \
      } else {                                                                           \
        return MOFQ_ERR_UNSUPPORTED;                                                     \
      }                                                                                  \
    } else if (a.n_clip == 1)                                                            \
      hipLaunchKernelGGL((sweep_channel_single_kernel<In, FA, FB, THREADS, CH>), grid, dim3(THREADS), 0, st, a); \
    else                                                                                 \
      hipLaunchKernelGGL((sweep_channel_kernel<In, FA, FB, THREADS, CH>), grid, dim3(THREADS), 0, st, a); \
    return hip_status(hipGetLastError());                                                \
  }
  // 32 to 48 elements per lane: enough work per candidate to amortise the cross-lane
  // reduction, few enough registers for many waves per SIMD
  MOFQ_CH(64, 1)     //   512 columns
  MOFQ_CH(64, 4)     //  2048
  MOFQ_CH(128, 4)    //  4096
  MOFQ_CH(256, 4)    //  8192
  MOFQ_CH(256, 6)    // 12288
  MOFQ_CH(512, 4)    // 16384
  MOFQ_CH(512, 6)    // 24576
  MOFQ_CH(1024, 4)   // 32768
#undef MOFQ_CH
  return MOFQ_ERR_UNSUPPORTED;
}

template <typename In, int FA, int FB>
int launch_group(const SweepArgs& a, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(ceil_div(a.units, kGroupQuads)));
  constexpr int NF = (FB >= 0) ? 2 : 1;
  const size_t lds = sizeof(float) * (MOFQ_MAX_CLIP + static_cast<size_t>(NF) * a.n_clip * kGroupQuads) +
                     (Codec<FA>::BITS == 4 && a.bisect ? static_cast<size_t>(NF) * (a.n_clip - 8) * kGroupQuads : 0);   // bisection: lists of candidates beyond the first 8
  switch (a.group) {
#define MOFQ_G(G)                                                                        \
  case G:                                                                                \
    if constexpr (Codec<FA>::BITS == 4)                                                   \
      if (a.bisect) {                                                                    \
        hipLaunchKernelGGL((sweep_group_kernel<In, FA, FB, G, true>), grid, dim3(256), lds, st, a);  \
        return hip_status(hipGetLastError());                                            \
      }                                                                                  \
    hipLaunchKernelGGL((sweep_group_kernel<In, FA, FB, G, false>), grid, dim3(256), lds, st, a);  \
    return hip_status(hipGetLastError());
    MOFQ_G(32)
    MOFQ_G(64)
    MOFQ_G(128)
    MOFQ_G(256)
#undef MOFQ_G
  }
  return MOFQ_ERR_UNSUPPORTED;
}

template <typename In, int FA, int FB>
int launch_tensor(SweepArgs a, hipStream_t st) {
  const int64_t n_chunks = a.rows * (a.cols / 8);
  a.n_blocks = static_cast<int32_t>(std::min<int64_t>(kTensorBlocks, ceil_div(n_chunks, 256)));
  hipLaunchKernelGGL((tensor_absmax_kernel<In>), dim3(a.n_blocks), dim3(256), 0, st, a);
  if constexpr (FA == MOFQ_INT8 && FB == MOFQ_FP8_E4M3) {
    if (a.emit_i8 && a.emit_f8 && a.n_clip == 1) {
      hipLaunchKernelGGL((tensor_score_emit8_kernel<In>), dim3(a.n_blocks), dim3(256), 0, st, a);
      hipLaunchKernelGGL((tensor_finalize_kernel<FA, FB>), dim3(1), dim3(256), 0, st, a);
      return hip_status(hipGetLastError());
    }
  }
  if (a.emit_i8 || a.emit_f8) return MOFQ_ERR_UNSUPPORTED;
  for (a.k0 = 0; a.k0 < a.n_clip; a.k0 += kTensorMaxClip)
    hipLaunchKernelGGL((tensor_score_kernel<In, FA, FB>), dim3(a.n_blocks), dim3(256), 0, st, a);
  a.k0 = 0;
  hipLaunchKernelGGL((tensor_finalize_kernel<FA, FB>), dim3(1), dim3(256), 0, st, a);
  return hip_status(hipGetLastError());
}

template <typename In, int FA, int FB>
int launch_gran(const SweepParams& p, const SweepArgs& a, hipStream_t st) {
  switch (p.gran) {
    case MOFQ_PER_CHANNEL: return launch_channel<In, FA, FB>(a, st);
    case MOFQ_PER_GROUP: return launch_group<In, FA, FB>(a, st);
    case MOFQ_PER_TENSOR: return launch_tensor<In, FA, FB>(a, st);
  }
  return MOFQ_ERR_INVALID_ARG;
}

// From how many descending clip ratios on bisection scores a 4-bit format's candidates.  On rows it scores 12 of 20, 17 of
// 50, 19 of 100 of them, but in five dependent rounds, which a row of few elements per wave or a tensor of few workgroups
// waits for; a wave of 16 groups takes as many rounds of four as the worst of them, 16 to 20 candidates of 20, 20 to 29 of 50.
// Layer selection, us, fp32, all candidates / bisection: rows: 4096 x 4096, 12: 88.8 / 87.4, 16: 105.9 / 96.2; 3001 x
// 5000, 10: 78.4 / 78.3, 14: 94.5 / 87.9; 2000 x 1024, 28: 31.8 / 32.3, 32: 34.4 / 32.5; few rows: 512 x 8192, 16: 33.9 /
// 34.2, 20: 38.5 / 37.4; 256 x 16384, 14: 33.6 / 34.5, 18: 38.2 / 37.1; 1000 x 600, 32: 26.0 / 26.9, 40: 30.0 / 29.7; 256 x
// 1024, 40: 28.0 / 28.8.  Groups, 2048 x 4096: 32, 18: 75.0 / 75.5, 20: 78.9 / 77.2, 50: 157 / 126; 64, 14: 56.7 / 56.6, 16:
// 60.9 / 58.5, 50: 140 / 97; 128, 16: 55.6 / 55.1, 18: 60.1 / 58.7, 50: 130 / 88; 256, 18: 62.6 / 62.5, 20: 67.1 / 66.6, 50:
// 133 / 96.  Fewer groups than are resident at once: 400 x 2048: 32, 32: 26.3 / 27.1, 40: 29.6 / 28.5; 64, 40: 28.6 / 29.2, 50:
// 33.0 / 32.7; 128, 28: 31.9 / 32.4, 32: 34.7 / 34.1; 256, 24: 43.2 / 44.0, 28: 48.0 / 46.3; 100 x 1024: 32, 50: 26.4 / 28.5.
int bisect_clip(const SweepParams& p) {
  if (p.gran == MOFQ_PER_TENSOR) return MOFQ_MAX_CLIP + 1;
  if (p.gran == MOFQ_PER_GROUP) {
    const int64_t groups = mofq_num_units(p.rows, p.cols, p.gran, p.group);
    const int g = p.group == 32 ? 0 : (p.group == 64 ? 1 : (p.group == 128 ? 2 : 3));
    static constexpr int64_t resident[4] = {65536, 65536, 49152, 32768};   // groups resident at once
    static constexpr int many[4] = {20, 16, 18, 20}, few[4] = {40, 40, 32, 28};
    if (groups >= resident[g]) return many[g];
    return g == 0 && groups < 16384 ? 64 : few[g];
  }
  if (p.cols <= 2048) return p.rows >= 1024 ? 32 : 44;
  return p.rows >= 1024 ? 12 : 18;
}

template <typename In>
int launch_fmt(const SweepParams& p, const SweepArgs& a, hipStream_t st) {
  const int fa = p.fmt[0], fb = p.n_fmt == 2 ? p.fmt[1] : -1;
#define MOFQ_F(A, B) \
  if (fa == (A) && fb == (B)) return launch_gran<In, A, B>(p, a, st);
  MOFQ_F(MOFQ_INT4, -1)
  MOFQ_F(MOFQ_FP4_E2M1, -1)
  MOFQ_F(MOFQ_INT8, -1)
  MOFQ_F(MOFQ_FP8_E4M3, -1)
  MOFQ_F(MOFQ_FP4_E2M1_IEEE, -1)
  MOFQ_F(MOFQ_FP8_E5M2, -1)
  MOFQ_F(MOFQ_INT4, MOFQ_FP4_E2M1)   // pairs come in (INT, FP) order; the caller maps slots
  MOFQ_F(MOFQ_INT8, MOFQ_FP8_E4M3)
#undef MOFQ_F
  return MOFQ_ERR_UNSUPPORTED;
}

}  // namespace

int launch_sweep(const SweepParams& p, hipStream_t st) {
  {
    const int rc = p.gran == MOFQ_PER_GROUP ? launch_sweep_group_bits(p, st) : launch_sweep_sorted(p, st);
    if (rc != MOFQ_ERR_UNSUPPORTED) return rc;
  }
  SweepArgs a{};
  a.w = p.w;
  a.rows = p.rows;
  a.cols = p.cols;
  a.ld = p.ld;
  a.group = p.group;
  a.scale_f16 = p.scale_f16;
  a.n_clip = p.n_clip;
  a.rec = p.rec;
  a.absmax_part = p.absmax_part;
  a.sse_part = p.sse_part;
  a.energy_part = p.energy_part;
  if (p.emit_i8 || p.emit_f8) {
    if (p.gran != MOFQ_PER_TENSOR) return MOFQ_ERR_UNSUPPORTED;
    a.emit_i8 = p.emit_i8;
    a.emit_f8 = p.emit_f8;
  }
  if (p.emit_grid[0] || p.emit_grid[1]) {
    if (p.gran != MOFQ_PER_CHANNEL || p.n_clip != 1 || p.n_fmt != 2) return MOFQ_ERR_UNSUPPORTED;
    a.emit_grid[0] = static_cast<uint16_t*>(p.emit_grid[0]);
    a.emit_grid[1] = static_cast<uint16_t*>(p.emit_grid[1]);
    a.emit_grid_fp8 = p.emit_grid_fp8;
    if (p.emit_grid_fp8 && p.cols % 64 != 0) return MOFQ_ERR_UNSUPPORTED;
  }
  if (p.ahead.codes) {
    if (p.gran != MOFQ_PER_CHANNEL || p.n_clip != 1 || (p.n_fmt == 2 && !p.ahead.tag)) return MOFQ_ERR_UNSUPPORTED;
    a.ahead = p.ahead;
  }
  a.units = mofq_num_units(p.rows, p.cols, p.gran, p.group);
  a.bisect = p.n_clip >= bisect_clip(p);
  for (int k = 0; k < p.n_clip; ++k) {
    a.clip[k] = p.clip[k];
    if (!(p.clip[k] > 0.0f) || !std::isfinite(p.clip[k]) || (k > 0 && p.clip[k] > p.clip[k - 1])) a.bisect = 0;
  }
  if (a.units <= 0) return MOFQ_ERR_INVALID_ARG;
  // same format twice in one launch is handled as two single launches by the caller
  switch (p.dtype) {
    case MOFQ_F32: return launch_fmt<F32>(p, a, st);
    case MOFQ_F16: return launch_fmt<F16>(p, a, st);
    case MOFQ_BF16: return launch_fmt<BF16>(p, a, st);
  }
  return MOFQ_ERR_INVALID_ARG;
}

int launch_sweep_group(const SweepParams* p, int n, hipStream_t st) {
  if (n > 1) {
    const int rc = launch_sweep_sorted_group(p, n, st);
    if (rc != MOFQ_ERR_UNSUPPORTED) return rc;
  }
  for (int i = 0; i < n; ++i) {
    const int rc = launch_sweep(p[i], st);
    if (rc != MOFQ_OK) return rc;
  }
  return MOFQ_OK;
}

}  // namespace mofq
