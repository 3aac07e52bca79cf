// Per-channel scale search on bf16 rows, 4-bit and 8-bit formats, and on fp16 rows, 8-bit formats: the histogram search of
// mofq_sweep_hist.hip with a prefix for every bit pattern.  A bf16 magnitude has 128 patterns per
// binade, so the patterns between the smallest threshold of any candidate and the row's largest magnitude
// are few (about 760 for INT4 / E2M1 over ratios in [0.5, 1], about 2600 for E4M3, whose
// subnormals reach 20 binades down) and the count and the sum of magnitudes of the elements below
// each of them fit in LDS, packed into 64 bits: count << 48 | sum in units of the first counted
// pattern's ulp.  Both are exact.  A look-up (candidate, level boundary) is then the boundary's pattern (patterns_below), one
// 8-byte read and three integer operations, 8 vector instructions in all against 22 of the group
// records, which makes the 127 boundaries of an 8-bit format cheap: scoring every (element, candidate)
// pair takes 4.8 instructions per element, candidate and format (240 000 per wave lane for a row of
// 5000 elements and 50 candidates; here a wave issues 1780 instructions in all).  Bound by vector issue and, at 8 bits, by the LDS reads of the look-ups beside it (their
// bank conflicts take 41 % of the LDS's cycles).
// The error that leaves for an 8-bit format is the winner's element-wise sum (finish_row): the look-ups
// choose it, and their difference of large sums would keep four digits fewer (1e-12 instead of 1e-15 on 5000 elements).
// The prefixes lie over the counters they are formed from (a thread holds its share in registers meanwhile), so that
// six workgroups of the 8-bit search fit a compute unit instead of five.
// Measured, layer selection: INT8 against E4M3, 3001 x 5000, 50 ratios 277 -> 69.8 -> 66.0 (prefixes over
// the counters) -> 62.0 (patterns_below, weights of the counts by dot products: 13 -> 8 instructions a look-up) -> 60.5 (RowCounters) ->
// 58 us (both winners summed in one pass, a thread's own prefixes in registers, scans by data-parallel-primitive moves); 4096 x 11008, 100 ratios 1294 -> 141 us; INT4 against E2M1, 1237 x 5000, 100 ratios: 28.2 -> 25.6 -> 23.4 us.
//
// fp16 rows (8-bit formats) have eight times the patterns, up to 20300 below the largest for E4M3: a prefix per group of
// 8, packed alike, and a look-up adds the group's first counters, 36 instructions.  Counters and prefixes take 61 KB, so
// two workgroups of 8 waves to a compute unit, and only the patterns that lie below the row's largest are summed up.
// Bound by vector issue and, for few ratios, by the steps of a row with so few rows resident.  Layer selection, INT8
// against E4M3, scored directly -> here: 3001 x 5000, 50 ratios 267 -> 159 us; 4096 x 11008, 100 ratios 1302 -> 280;
// 300 x 11008, 60 ratios 133 -> 33.
//
// INT8's levels are spaced evenly; E4M3's evenly inside runs of 8 codes (a binade; the subnormals are the
// first run): per run the level sums are d sum_i S_i and d^2 sum_i (2 (base + i) + 1) C_i with d the run's
// spacing.  Boundaries beyond the largest level count everything (threshold infinity) and cancel against the
// last level's weight.
#include "mofq_search_common.h"

namespace mofq {

namespace {

constexpr int kMaxBins = 4096, kMaxTailBins = 1024;             // bf16
constexpr int kMaxHalfBins = 24576, kMaxHalfTailBins = 2048;    // fp16
constexpr int kRuns = 16;   // runs of 8 boundaries of an 8-bit format

// Decision thresholds of the formats' boundaries: level magnitude m_b or below <=> t <= thr; est: a
// shade below, edge: decision_edge(thr) (counters_below).  Run r, boundary i between code 8 r + i and the next; ties to the even code.
struct Boundary {
  float est, thr;
  double edge;
};
struct BoundaryTable {
  Boundary b[kRuns][8];
};
constexpr double kInfinity = __builtin_inf();
constexpr float prev_float(float x) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) - 1u); }   // x > 0
constexpr Boundary boundary(double mid, bool up_is_even) {
  const float m = static_cast<float>(mid);   // exact
  const float thr = up_is_even ? prev_float(m) : m;
  return Boundary{static_cast<float>(thr * (1.0 - 0x1p-21)), thr, decision_edge(thr)};
}
constexpr Boundary kBeyond{static_cast<float>(kInfinity), static_cast<float>(kInfinity), kInfinity};
constexpr BoundaryTable int8_table() {
  BoundaryTable t{};
  for (int r = 0; r < kRuns; ++r)
    for (int i = 0; i < 8; ++i) {
      const int b = 8 * r + i;
      t.b[r][i] = b < 127 ? boundary(b + 0.5, b % 2 == 1) : kBeyond;
    }
  return t;
}
constexpr double e4m3_mag(int c) {
  double m = c < 8 ? c : 8 + (c & 7);
  for (int e = c < 8 ? 0 : (c >> 3) - 1; e < 9; ++e) m *= 0.5;
  for (int e = 9; e < (c < 8 ? 0 : (c >> 3) - 1); ++e) m *= 2.0;
  return m;
}
constexpr BoundaryTable e4m3_table() {
  BoundaryTable t{};
  for (int r = 0; r < kRuns; ++r)
    for (int i = 0; i < 8; ++i) {
      const int c = 8 * r + i;
      t.b[r][i] = c < 126 ? boundary(0.5 * (e4m3_mag(c) + e4m3_mag(c + 1)), c % 2 == 1) : kBeyond;
    }
  return t;
}
static_assert(e4m3_mag(126) == 448.0 && e4m3_mag(8) == 0x1p-6 && e4m3_mag(1) == 0x1p-9 && e4m3_mag(127) == 480.0, "E4M3 magnitudes");
__device__ const BoundaryTable kInt8Boundaries = int8_table();
__device__ const BoundaryTable kE4m3Boundaries = e4m3_table();

template <int FMT> struct Runs;
template <> struct Runs<MOFQ_INT8> {
  static constexpr double LAST = 128.0;   // the level after the last run
  MOFQ_DEV static const BoundaryTable& table() { return kInt8Boundaries; }
  MOFQ_DEV static double spacing(int) { return 1.0; }
  MOFQ_DEV static int base(int r) { return 8 * r; }
};
template <> struct Runs<MOFQ_FP8_E4M3> {
  static constexpr double LAST = 512.0;
  MOFQ_DEV static const BoundaryTable& table() { return kE4m3Boundaries; }
  MOFQ_DEV static double spacing(int r) { return __builtin_bit_cast(double, static_cast<uint64_t>(1023 - 9 + (r > 0 ? r - 1 : 0)) << 52); }   // 2^(max(r, 1) - 10)
  MOFQ_DEV static int base(int r) { return r > 0 ? 8 : 0; }
};

MOFQ_DEV int clamped(int x, int lo, int hi) {   // one instruction
  int r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "s"(lo), "v"(hi));
  return r;
}

// Exclusive prefixes over the counters, P[0 .. nbin], packed count << 48 | sum.  Thread `id` of
// NW waves takes the counters [id pp, (id + 1) pp), pp even and at most 2 PWMAX.  NW > 1: by the whole workgroup, with
// barriers; a thread's counters stay in its registers over the first, behind which P may lie over them.
template <int NW, int PWMAX>
MOFQ_DEV void packed_prefixes(const uint32_t* counters, uint64_t* P, int lo, int nbin, uint64_t* s_wave) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int id = NW > 1 ? tid : lane;
  const int pw = (nbin / 2 + NW * 64 - 1) / (NW * 64);   // words per thread
  const int e_lo = exponent_of<BF16>(lo);
  const int w0 = id * pw, w1 = (w0 + pw < nbin / 2) ? w0 + pw : nbin / 2;
  uint32_t c2[PWMAX];
#pragma unroll
  for (int j = 0; j < PWMAX; ++j) c2[j] = j < pw && w0 + j < w1 ? counters[w0 + j] : 0u;
  auto add = [&](int j, uint64_t& acc, auto between) {
    uint32_t m, shift;
    mant_shift<BF16>(static_cast<uint32_t>(lo + 2 * (w0 + j)), e_lo, m, shift);   // lo is even: both patterns share the exponent
    acc += static_cast<uint64_t>(m << shift) * (c2[j] & 0xFFFFu) + (static_cast<uint64_t>(c2[j] & 0xFFFFu) << 48);
    between();
    acc += static_cast<uint64_t>((m + 1) << shift) * (c2[j] >> 16) + (static_cast<uint64_t>(c2[j] >> 16) << 48);
  };
  constexpr bool KEEP = PWMAX <= 6;   // the thread's own prefixes in registers, else formed again behind the scan
  uint64_t own[KEEP ? 2 * PWMAX : 1];
  uint64_t acc = 0;
#pragma unroll
  for (int j = 0; j < PWMAX; ++j) {
    if constexpr (KEEP) {
      own[2 * j] = acc;
      add(j, acc, [&] { own[2 * j + 1] = acc; });   // (counters past the end are zero)
    } else if (j < pw) {   // uniform; words past the end count nothing
      add(j, acc, [] {});
    }
  }
  // exclusive scan over the threads (sums of the two fields do not meet: the sum stays below 2^48)
  const uint64_t inc = wave_incl_scan_u64(acc);
  uint64_t at = inc - acc;
  if constexpr (NW > 1) {
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    for (int w = 0; w < wave; ++w) at += s_wave[w];
  }
#pragma unroll
  for (int j = 0; j < PWMAX; ++j)
    if (j < pw) {
      uint64_t first = at, second = 0;
      if constexpr (KEEP) {
        first += own[2 * j];
        second = at + own[2 * j + 1];
      } else {
        add(j, at, [&] { second = at; });
      }
      if (w0 + j < w1) {
        P[2 * (w0 + j)] = first;
        P[2 * (w0 + j) + 1] = second;
      }
    }
  if (id == NW * 64 - 1) P[nbin] = KEEP ? at + acc : at;
  if constexpr (NW > 1) __syncthreads();
}

// fp16: exclusive prefixes over groups of 8 counters, P[0 .. nbin / 8], packed alike.
MOFQ_DEV uint64_t packed_group(const u32x4 w, int first, int e_first) {   // of the counters from pattern `first` on, a multiple of 8
  uint32_t c, weighted, m, shift;
  count8<false>(w, c, weighted);
  mant_shift<F16>(static_cast<uint32_t>(first), e_first, m, shift);   // a group shares its exponent
  return (static_cast<uint64_t>(__umul24(m, c) + weighted) << shift) + (static_cast<uint64_t>(c) << 48);
}
template <int NW, int GPMAX>
MOFQ_DEV void group_prefixes(const uint32_t* counters, uint64_t* P, int lo, int nbin, uint64_t* s_wave) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int id = NW > 1 ? tid : lane;
  const int ng = nbin >> 3, gp = (ng + NW * 64 - 1) / (NW * 64);   // groups per thread
  const int e_lo = exponent_of<F16>(lo);
  uint64_t v[GPMAX], acc = 0;
#pragma unroll
  for (int i = 0; i < GPMAX; ++i) {
    const int g = id * gp + i;
    v[i] = 0;
    if (i < gp && g < ng) v[i] = packed_group(reinterpret_cast<const u32x4*>(counters)[g], lo + 8 * g, e_lo);
    acc += v[i];
  }
  const uint64_t inc = wave_incl_scan_u64(acc);
  uint64_t at = inc - acc;
  if constexpr (NW > 1) {
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    for (int w = 0; w < wave; ++w) at += s_wave[w];
  }
#pragma unroll
  for (int i = 0; i < GPMAX; ++i) {
    const int g = id * gp + i;
    if (i < gp && g < ng) P[g] = at;
    at += v[i];
  }
  if (id == NW * 64 - 1) P[ng] = at;
  if constexpr (NW > 1) __syncthreads();
}

MOFQ_DEV double sum_of(uint64_t p) {   // the low 48 bits
  return __builtin_fma(static_cast<double>(static_cast<uint32_t>(p >> 32) & 0xFFFFu), 0x1p32, static_cast<double>(static_cast<uint32_t>(p)));
}
MOFQ_DEV uint32_t count_of(uint64_t p) { return static_cast<uint32_t>(p >> 48); }

template <typename In> constexpr int kThreadsOf = std::is_same<In, BF16>::value ? 256 : 512;
template <typename In, int FA, int FB, int CH>
__global__ __launch_bounds__(kThreadsOf<In>) __attribute__((amdgpu_waves_per_eu(std::is_same<In, BF16>::value && CH <= 6 ? 5 : 4)))
void sweep_pattern_kernel(const SortedArgs a) {
  constexpr bool HALF = std::is_same<In, F16>::value;
  constexpr int kThreads = kThreadsOf<In>, kNW = kThreads / 64;
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  constexpr bool TAIL_A = Codec<FA>::IS_INT, TAIL_B = (FB >= 0) && Codec<FBX>::IS_INT;   // the level one beyond the positive ones
  constexpr bool ANY_TAIL = TAIL_A || TAIL_B;
  constexpr bool EIGHT = Codec<FA>::BITS == 8;

  // dynamic LDS: [prefixes, before them the counters in the same place | of the negative elements | their counters]
  extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
  int nbin = a.nbin;   // multiples of 8
  const int ntbin = ANY_TAIL ? a.ntbin : 0;
  // fp16: [prefixes of the groups | of the negative elements' | masks | counters | theirs | 16 bytes]
  int n_rec = HALF ? nbin >> 3 : nbin;
  const int n_trec = HALF ? ntbin >> 3 : ntbin;   // (before the counters the spare ones)
  uint64_t* const P = reinterpret_cast<uint64_t*>(s_dyn);
  uint64_t* const TP = P + (n_rec + 1);
  u32x4* const keep = reinterpret_cast<u32x4*>(s_dyn + (static_cast<uint32_t>(n_rec + n_trec + 2) * 8 + 15) / 16 * 16);   // fp16: of the first c of 8 counters
  uint32_t* const counters = (HALF ? reinterpret_cast<uint32_t*>(keep + 8) : reinterpret_cast<uint32_t*>(s_dyn)) + kSpare / 2;
  uint32_t* const tcounters = HALF ? counters + nbin / 2 : reinterpret_cast<uint32_t*>(TP + (ntbin + 1));

  __shared__ RowSearch<NF, kNW> sh;
  __shared__ float s_wmax[kNW];
  __shared__ double s_wsum[kNW];
  __shared__ uint64_t s_wave[kNW];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t tensor = 0;                                                    // wave-uniform
#pragma unroll
  for (int i = 1; i < kSweepGroupMax; ++i) tensor += (blockIdx.x >= a.row0[i]);
  const int64_t row = blockIdx.x - a.row0[tensor];
  const SortedTensor& T = a.t[tensor];
  const uint16_t* src = static_cast<const uint16_t*>(T.w) + row * T.ld;
  const int K = a.n_clip;
  const int n = static_cast<int>(a.cols);

  // ---- load the row, clear the counters; largest magnitude and energy ------------------------------
  Raw8<In> raw[CH];
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int c = (j * kThreads + tid) * 8;
    raw[j].load(src, 0, static_cast<uint32_t>(c < n ? c : 0));
    if (c >= n) raw[j].clear();
  }
  // what the tensor's finished rows favour: behind the row (loads return in order), by one wave (waves that
  // read it at different times could disagree)
  double tally = 0.0;
  if (NF == 2 && T.ahead.tally && wave == kNW - 1) tally = tally_read(T.ahead);
  {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int i = tid; i < nbin / 8; i += kThreads) reinterpret_cast<u32x4*>(counters)[i] = zero;
    for (int i = tid; i < ntbin / 8; i += kThreads) reinterpret_cast<u32x4*>(tcounters)[i] = zero;
    if (HALF && tid < 32) {   // word tid % 4 of the mask of the first tid / 4 counters
      const int c = tid >> 2, i = tid & 3;
      reinterpret_cast<uint32_t*>(keep)[tid] = (c >= 2 * i + 2) ? 0xFFFFFFFFu : ((c == 2 * i + 1) ? 0x0000FFFFu : 0u);
    }
  }
  float amax = 0.0f;
  double en = 0.0;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    float v[8];
    raw[j].widen(v);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
      const double d = static_cast<double>(v[i]);
      en = __builtin_fma(d, d, en);
    }
  }
  amax = wave_max(amax);
  en = wave_sum(en);
  if (lane == 0) { s_wmax[wave] = amax; s_wsum[wave] = en; }
  __syncthreads();   // also: the counters are clear
  amax = s_wmax[0];
  en = s_wsum[0];
#pragma unroll
  for (int w = 1; w < kNW; ++w) {
    amax = __builtin_fmaxf(amax, s_wmax[w]);
    en += s_wsum[w];
  }
  {   // thread f * MOFQ_MAX_CLIP + k
    const int f = tid / MOFQ_MAX_CLIP, k = tid % MOFQ_MAX_CLIP;
    const float qmax = (f == 0) ? Codec<FA>::QMAX : Codec<FBX>::QMAX;
    if (f < NF && k < K) sh.scale[f][k] = unit_scale(amax, a.clip[k], qmax, a.scale_f16 != 0);
  }
  static_assert(2 * MOFQ_MAX_CLIP <= kThreads, "one thread per (format, candidate)");

  // ---- count the nbin patterns up to the largest magnitude's (a non-finite element lands in the last
  // counter: the row's error is non-finite anyway) ---------------------------------------------------
  const int hmax = __builtin_amdgcn_readfirstlane(static_cast<int>(pattern_rtz<In>(__builtin_fminf(amax, 3.4028234e38f))));   // exact for a finite amax
  const int lo = (((hmax + 1 - nbin) > 0 ? (hmax + 1 - nbin) : 0) + 7) & ~7;
  const int tlo = (((hmax + 1 - ntbin) > 0 ? (hmax + 1 - ntbin) : 0) + 7) & ~7;
  if constexpr (HALF) {   // fp16 rarely has as many patterns below the largest
    nbin = min(nbin, (hmax + 1 - lo + 7) & ~7);
    n_rec = nbin >> 3;
  }
  {
    const RowCounters row_counters(counters, lo, nbin);
    const uint32_t tat = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_u32*)tcounters));
#pragma unroll
    for (int j0 = 0; j0 < CH; j0 += 4) {
      constexpr int PART = CH < 4 ? CH : 4;
      uint32_t noted = 0;
#pragma unroll
      for (int j = j0; j < j0 + PART; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t w = j < CH ? raw[j].w[i] : 0;
          if (j < CH) row_counters.count_pair(w);   // whatever lies below every threshold has no counter, padding (zero) neither unless they reach that far down (E4M3 on fp16)
          if constexpr (ANY_TAIL) note_negative(noted, w, tlo, 4 * (j - j0) + i);
        }
      if constexpr (ANY_TAIL) count_noted<kThreads * 16>(noted, src, static_cast<uint32_t>(j0 * kThreads + tid) * 16, tlo, ntbin, tat);
    }
  }
  __syncthreads();

  if constexpr (HALF) {
    if constexpr (ANY_TAIL)
      if (wave == kNW - 1) group_prefixes<1, kMaxHalfTailBins / 8 / 64>(tcounters, TP, tlo, ntbin, s_wave);
    group_prefixes<kNW, kMaxHalfBins / 8 / kThreads>(counters, P, lo, nbin, s_wave);
  } else {
    if constexpr (ANY_TAIL)
      if (wave == kNW - 1) {
        if (ntbin <= 256) packed_prefixes<1, 2>(tcounters, TP, tlo, ntbin, s_wave);
        else packed_prefixes<1, kMaxTailBins / 128>(tcounters, TP, tlo, ntbin, s_wave);
      }
    // (the short ones of the 4-bit formats in code of their own: 1237 x 5000 took 0.6 us more in the other's)
    if (nbin <= 4 * kThreads) packed_prefixes<kNW, 2>(counters, P, lo, nbin, s_wave);
    else if (nbin <= 12 * kThreads) packed_prefixes<kNW, 6>(counters, P, lo, nbin, s_wave);
    else packed_prefixes<kNW, kMaxBins / 2 / kThreads>(counters, P, lo, nbin, s_wave);
  }
  const uint64_t total = P[n_rec];
  const float v_lo = bits_to_float<In>(static_cast<uint32_t>(lo));
  const double unit = static_cast<double>(bits_to_float<In>(static_cast<uint32_t>(lo) + 1) - v_lo);   // an ulp at lo
  const double s_total = sum_of(total);
  const double c_total = static_cast<double>(count_of(total));

  // ---- level boundaries: one lane per candidate; a wave takes (format, 64 candidates, part of the runs) ----
  {
    // A candidate's scale, and what its boundaries are looked for with.
    struct Candidate {
      float s, inv;
      double per_edge;
    };
    auto candidate = [&](int f, int k) {
      const float s = sh.scale[f][k < K ? k : K - 1];
      const float inv = HALF ? reciprocal(s) : 1.0f / s;
      return Candidate{s, inv, edge_unit(s, inv)};
    };
    const int before_lo = pattern_before<In>(lo), before_tlo = pattern_before<In>(tlo);
    // H = the largest pattern h with fl32(v(h) * inv) <= thr, as in the histogram kernel.  Returns H - first + 1 as
    // a number of counters; negative numbers are large ones to the unsigned minimum.  Where subnormals are counted: the
    // pattern of est * s rounded toward zero passes, one decision on the next tells.
    auto counters_below = [](auto normal_tag, const Boundary& b, const Candidate& c, int first, int before) {
      if constexpr (decltype(normal_tag)::value) return patterns_below<In>(b.edge, c.per_edge, before);
      if constexpr (HALF) {
        const int h = static_cast<int>(pattern_rtz<F16>(b.est * c.s));
        return h + (1 - first) + (scaled<F16>(static_cast<uint32_t>(h + 1), c.inv) <= b.thr ? 1 : 0);
      }
      const uint32_t x1 = f2u(b.est * c.s) + 0x10000u;
      const bool above = u2f(x1 & 0xFFFF0000u) * c.inv <= b.thr;
      return static_cast<int>(x1 >> 16) - first + (above ? 1 : 0);
    };
    // count and sum of the elements in the first n1 counters
    auto first_counters = [&](const uint64_t* R, const uint32_t* cells, int first, uint32_t n1) {
      if constexpr (HALF) {
        const uint32_t g = n1 >> 3;
        return R[g] + packed_group(reinterpret_cast<const u32x4*>(cells)[g] & keep[n1 & 7], first + 8 * static_cast<int>(g), exponent_of<F16>(first));
      } else {
        return R[n1];
      }
    };
    // those in the counters below a boundary of the row; below_first: the boundary lies beneath all of them
    const uint32_t cells_at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint64_t*)P)) - 8u * static_cast<uint32_t>(before_lo);
    auto up_to = [&](auto normal_tag, const Boundary& b, const Candidate& c, bool& below_first) {
      if constexpr (decltype(normal_tag)::value && !HALF) {   // the difference of the patterns is in the address
        const int top = pattern_top<In>(b.edge, c.per_edge);
        below_first = top < before_lo;
        return *(__attribute__((address_space(3))) uint64_t*)static_cast<uintptr_t>(cells_at + 8u * static_cast<uint32_t>(clamped(top, before_lo, before_lo + nbin)));
      }
      const int n1 = counters_below(normal_tag, b, c, lo, before_lo);
      below_first = n1 < 0;
      return first_counters(P, counters, lo, min(static_cast<uint32_t>(n1), static_cast<uint32_t>(nbin)));
    };
    const int chunks = (K + 63) >> 6;
    // few units: the runs of an 8-bit format are dealt to all waves, whose partial sums meet in LDS
    const int parts = EIGHT ? kNW / (NF * chunks) : 1;   // 4, 2 or 1
    double A = 0.0, B = 0.0, ca_tail = 0.0;
    bool bad = false;
    int cb_tail = 0;
    auto tail = [&](auto normal_tag, const int first_level, const Boundary& b, const Candidate& c) {
      // negative elements beyond the last positive level's upper boundary sit one level further
      const int n1 = counters_below(normal_tag, b, c, tlo, before_tlo);
      bad |= n1 < 0;
      const uint64_t above = TP[n_trec] - first_counters(TP, tcounters, tlo, min(static_cast<uint32_t>(n1), static_cast<uint32_t>(ntbin)));
      const float v_tlo = bits_to_float<In>(static_cast<uint32_t>(tlo));
      ca_tail = sum_of(above) * static_cast<double>(bits_to_float<In>(static_cast<uint32_t>(tlo) + 1) - v_tlo);
      cb_tail = static_cast<int>(count_of(above)) * (2 * first_level + 1);
    };
    auto finish = [&](const int f, const int k, float s, double last) {
      if (k < K) {
        const double At = __builtin_fma(unit, A + last * s_total, ca_tail);
        const double Bt = B + static_cast<double>(cb_tail) + last * last * c_total;
        const double sc = static_cast<double>(s);
        const double v = (en - 2.0 * sc * At) + sc * sc * Bt;   // filtered error
        sh.fast[f][k] = bad ? __builtin_nan("") : v;
      }
    };
    auto search8 = [&](auto normal_tag, auto fmt_c, const int f, const int k, const int part) {
      constexpr int FMT = decltype(fmt_c)::value;
      const Candidate c = candidate(f, k);
      A = B = ca_tail = 0.0;
      bad = false;
      cb_tail = 0;
      const BoundaryTable& t = Runs<FMT>::table();
      const int runs = kRuns / parts;
      for (int r = part * runs; r < (part + 1) * runs; ++r) {
        uint64_t sums = 0;
        uint32_t ib = 0;
        const uint32_t base2 = 2 * Runs<FMT>::base(r) + 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          bool below_first;
          const uint64_t p = up_to(normal_tag, t.b[r][i], c, below_first);
          // the smallest threshold: nothing uncounted above it, and no subnormal product (too coarse an estimate)
          if (i == 0 && r == 0) bad = below_first || (!decltype(normal_tag)::value && !(t.b[0][0].est * c.s >= 0x1p-126f));
          sums += p;      // (the counts overflow out of the word)
          ib = dot2(static_cast<uint32_t>(p >> 32), (base2 + 2 * i) << 16, ib);   // the count, in the upper half, times its weight
        }
        const double d = Runs<FMT>::spacing(r);
        A = __builtin_fma(-d, sum_of(sums), A);
        B = __builtin_fma(-d * d, static_cast<double>(static_cast<int>(ib)), B);
      }
      if constexpr (Codec<FMT>::IS_INT)
        if (part == 0) tail(normal_tag, 127, boundary(127.5, true), c);
      if (parts == 1) finish(f, k, c.s, Runs<FMT>::LAST);
    };
    auto search4 = [&](auto normal_tag, auto fmt_c, const int f, const int k) {
      constexpr int FMT = decltype(fmt_c)::value;
      const Candidate c = candidate(f, k);
      A = B = ca_tail = 0.0;
      bad = false;
      cb_tail = 0;
      // In half levels: sum_b (sum up to boundary b) 2 (m_{b+1} - m_b), steps of 1, 2 or 4 (pattern_search_fits: below 2^48),
      // and sum_b (count up to boundary b) 4 (m_{b+1}^2 - m_b^2)
      uint64_t sums = 0;
      uint32_t cb4 = 0;
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        bool below_first;
        const uint64_t p = up_to(normal_tag, Boundary{a.thr_est[f][q], a.thr[f][q], a.thr_edge[f][q]}, c, below_first);
        if (q == 0) bad = below_first;
        sums += p << half_steps_log2<FMT>(q);
        cb4 = dot2(static_cast<uint32_t>(p >> 32), static_cast<uint32_t>(-a.dg2q[f][q]) << 16, cb4);
      }
      A = -0.5 * sum_of(sums);
      B = -0.25 * static_cast<double>(static_cast<int>(cb4));
      if constexpr (Codec<FMT>::IS_INT) tail(normal_tag, 7, Boundary{a.thr_est[f][7], a.thr[f][7], a.thr_edge[f][7]}, c);
      finish(f, k, c.s, static_cast<double>(a.g_last[f]));
    };
    auto search = [&](auto normal_tag) {
      for (int u = wave; u < NF * chunks * parts; u += kNW) {   // wave-uniform
        const int part = u % parts, fc = u / parts;
        const int f = fc / chunks;
        const int k = (fc - f * chunks) * 64 + lane;
        if constexpr (EIGHT) {
          if (f == 0) search8(normal_tag, std::integral_constant<int, FA>{}, f, k, part);
          else search8(normal_tag, std::integral_constant<int, FBX>{}, f, k, part);
        } else {
          if (f == 0) search4(normal_tag, std::integral_constant<int, FA>{}, f, k);
          else search4(normal_tag, std::integral_constant<int, FBX>{}, f, k);
        }
      }
    };
    if (lo >= (1 << Pattern<In>::MANT)) search(std::true_type{});   // no subnormal has a counter
    else search(std::false_type{});
    if constexpr (EIGHT) {
      if (parts > 1) {   // one unit per wave: its sums are still in its registers
        double* const s_part = reinterpret_cast<double*>(P);   // [wave][64][2], over the prefixes
        __syncthreads();
        s_part[tid * 2] = A;
        s_part[tid * 2 + 1] = B;
        __syncthreads();
        if (wave % parts == 0) {
          const int fc = wave / parts, f = fc / chunks;
          const int k = (fc - f * chunks) * 64 + lane;
          for (int p = 1; p < parts; ++p) {
            A += s_part[(tid + 64 * p) * 2];
            B += s_part[(tid + 64 * p) * 2 + 1];
          }
          finish(f, k, sh.scale[f][k < K ? k : K - 1], f == 0 ? Runs<FA>::LAST : Runs<FBX>::LAST);
        }
      }
    }
  }
  __syncthreads();

  // ---- winners (the re-scored values lie over the prefixes, which are no longer needed), codes --------
  finish_row<In, FA, FB, kThreads, CH, true>(sh, reinterpret_cast<double*>(P), src, n, K, en, unit * s_total, a.g_absmax, T.rec, row);
  if (T.ahead.codes) emit_row_ahead<In, FA, FB, kThreads, CH>(sh, T.ahead, tally, raw, src, n, row);   // uniform
}

template <typename In> size_t lds_bytes(const SortedArgs& a) {
  if (std::is_same<In, F16>::value) return (static_cast<size_t>(a.nbin / 8 + a.ntbin / 8 + 2) * 8 + 15) / 16 * 16 + 128 + 2 * static_cast<size_t>(kSpare + a.nbin + a.ntbin) + 16;
  const size_t prefixes = std::max<size_t>(8 * static_cast<size_t>(a.nbin + 1 + a.ntbin + 1), 2 * MOFQ_MAX_CLIP * sizeof(double));
  return prefixes + 2 * static_cast<size_t>(a.ntbin);
}

template <typename In, int FA, int FB>
int launch_shape(const SortedArgs& a, int64_t total_rows, hipStream_t st) {
  constexpr int THREADS = kThreadsOf<In>;
  const dim3 grid(static_cast<unsigned>(total_rows));
  const int64_t chunks = a.cols / 8;
#define MOFQ_PATTERN(CH)                                                                        \
  if (chunks <= THREADS * (CH)) {                                                               \
    hipLaunchKernelGGL((sweep_pattern_kernel<In, FA, FB, CH>), grid, dim3(THREADS), lds_bytes<In>(a), st, a); \
    return hip_status(hipGetLastError());                                                       \
  }
  MOFQ_PATTERN(1)   //  2048 columns of bf16, 4096 of fp16
  MOFQ_PATTERN(2)   //  4096, 8192
  MOFQ_PATTERN(3)   //  6144, 12288
  MOFQ_PATTERN(4)   //  8192, 16384
  if constexpr (std::is_same<In, BF16>::value) {
    MOFQ_PATTERN(6)   // 12288
    MOFQ_PATTERN(12)  // 24576
  }
#undef MOFQ_PATTERN
  return MOFQ_ERR_UNSUPPORTED;
}

}  // namespace

// The packed prefixes hold it: sums below 2^45 units (an element is below 2^(1 + mantissa bits + binades); eight prefixes
// are added up in 48 bits, those of a 4-bit format with weights of 14 together); LDS for three workgroups (fp16: two); room for the partial sums of a divided search.
bool pattern_search_fits(const SweepParams& p, int nbin, int ntbin) {
  const bool eight = p.fmt[0] == MOFQ_INT8 || p.fmt[0] == MOFQ_FP8_E4M3;
  if (p.dtype == MOFQ_F16) {
    if (!eight || nbin < 4096 || nbin > kMaxHalfBins || ntbin > kMaxHalfTailBins || p.cols > 16384) return false;
    const int span = (std::max(nbin, ntbin) + 1023) / 1024;
    return (p.cols << (11 + span)) <= (int64_t{1} << 45);
  }
  if (p.dtype != MOFQ_BF16 || nbin <= 0 || nbin > kMaxBins || ntbin > kMaxTailBins) return false;
  const int span = (std::max(nbin, ntbin) + 127) / 128;
  if (eight && nbin < 512) return false;
  return span <= 22 && (p.cols << (8 + span)) <= (int64_t{1} << (eight ? 45 : 44)) && p.cols <= 24576;
}

int launch_sweep_pattern(const SweepParams& p, const SortedArgs& a, int64_t total_rows, hipStream_t st) {
  if (!pattern_search_fits(p, a.nbin, a.ntbin)) return MOFQ_ERR_UNSUPPORTED;
  const int fa = p.fmt[0], fb = p.n_fmt == 2 ? p.fmt[1] : -1;
  if (p.dtype == MOFQ_F16) {
#define MOFQ_F(A, B) \
  if (fa == (A) && fb == (B)) return launch_shape<F16, A, B>(a, total_rows, st);
    MOFQ_F(MOFQ_INT8, MOFQ_FP8_E4M3)
    MOFQ_F(MOFQ_INT8, -1)
    MOFQ_F(MOFQ_FP8_E4M3, -1)
#undef MOFQ_F
    return MOFQ_ERR_UNSUPPORTED;
  }
#define MOFQ_F(A, B) \
  if (fa == (A) && fb == (B)) return launch_shape<BF16, A, B>(a, total_rows, st);
  MOFQ_F(MOFQ_INT4, MOFQ_FP4_E2M1)
  MOFQ_F(MOFQ_INT4, -1)
  MOFQ_F(MOFQ_FP4_E2M1, -1)
  MOFQ_F(MOFQ_INT8, MOFQ_FP8_E4M3)
  MOFQ_F(MOFQ_INT8, -1)
  MOFQ_F(MOFQ_FP8_E4M3, -1)
#undef MOFQ_F
  return MOFQ_ERR_UNSUPPORTED;
}

}  // namespace mofq
