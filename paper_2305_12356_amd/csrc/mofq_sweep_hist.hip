// Per-channel scale search from a histogram of the magnitudes' bit patterns: Algorithm 1's
// quantize_layer + compute_error with the tensor-error metric (Section 4.1) for per-channel weight
// scales over a table of clip ratios, INT4 against FP4-E2M1 (Table 1).  The formulation, the filter
// and the shortlist are described at the top of mofq_sweep_sorted.hip, whose kernel this one replaces
// wherever its histogram fits.
//
// The decision "fl32(|x| * inv) <= threshold" is monotone in the magnitude's bit pattern, so for
// every (candidate, boundary) there is one largest pattern H that passes, and the elements on
// level magnitudes up to m_b are those with pattern <= H.  Instead of sorting the row, the kernel
// counts the elements per pattern (16-bit counters, two per word, LDS adds), forms count and
// magnitude-sum prefixes over groups of 8 patterns (a group shares its exponent, so its elements'
// magnitudes are v0 + i ulp and its sum is v0 C + ulp sum i c_i, exact in fp64), finds H from
// a product in fp64 (patterns_below), and reads count and sum up to H from the group
// prefix and one 16-byte read of the group's counters.  Only the patterns between the smallest
// threshold and the row's largest magnitude get a counter: elements below every threshold sit on
// level 0 for every candidate and drop out of both level sums.  How many patterns that is
// depends on the clip ratios alone, so the host sizes the histogram (dynamic LDS) and uses the
// sorting kernel where it would not fit.  INT4's negative elements beyond its extra boundary
// are counted in a second, short histogram over the top of the range.
//
// Where the counted patterns span few enough binades, sums of magnitudes are 32-bit integers in units
// of the first counted pattern's ulp (exact, and a third of the instructions of fp64 sums); else fp64.
//
// Bound by vector issue: 904 instructions per wave on rows of 4096 elements (INT4 / E2M1, 100 ratios, codes
// included): 215 to count, 160 for the prefixes, 205 for the look-ups; they take nine tenths of the clocks.  Two blocks of the 65B shape 2295 -> 2222 us, eight of the 7B shape 3094 -> 2957 us with the
// negative elements' counting behind the loop (note_negative), the halves of a word selected by
// the instructions that use them (count_pair) and one weighted sum per group (count8); 2218 -> 2161 and 2953 -> 2845 us
// with look-ups of 22 instead of 32 instructions (patterns_below instead of an estimate and a decision, weights that are zero
// where masks were) whose reads are requested one look-up ahead (in a loop, a look-up at a time: 2190 and 2884); 2120 and 2818 us with
// spare counters instead of branches (RowCounters), notes that hold the word's place, scales by a multiplication and the codes'
// widening and product in one instruction; 2725 us on the 7B blocks with rows of up to 4096 columns kept in registers for their codes.
//
// Filter, shortlist and exact fp64 re-score are those of the sorting kernel; the re-score reads
// the row again.  With AheadCodes the row's codes are written at the end, from registers or a further read that
// comes from L2.
#include "mofq_search_common.h"

namespace mofq {

namespace {

// ---- prefixes -----------------------------------------------------------------------------
// Exclusive prefix of count and magnitude sum per group of 8 counters, one record per group, the
// totals in record ng.  A group's patterns share the exponent: pattern lo + 8 g + i has the magnitude
// (m + i) << shift in units of the ulp of pattern lo (Narrow) or v0 + i ulp (Wide).
struct Narrow {
  using sum_t = uint32_t;
  uint32_t sum, word;   // word: count (16 bits) | m (11) | shift (5: where a shift takes its amount from)
};
struct Wide {
  using sum_t = double;
  double sum;
  uint32_t cnt, unused;
};

// Count and magnitude sum of the elements in the histogram's first n1 counters, 0 <= n1 <= nbin:
// the record of group n1 / 8 plus the first n1 % 8 counters of that group (n1 = nbin reads the 16
// bytes after the counters, which are inside the workgroup's LDS, and masks them all).
// Eight counters, two per word, of which the first c count: their number and index-weighted number are dot products with
// weights that are zero for the others, from a table in LDS (Weights: the rows of c).  JOINT: both in one sum (count8).
struct Weights {
  uint32_t w[2][8][4];   // [0]: the index (JOINT: 2^15 more); [1], not with JOINT: 1
};
template <bool JOINT> MOFQ_DEV void fill_weights(Weights& t, int tid) {   // threads 0 .. 31
  const int c = tid >> 2, i = tid & 3;
  const uint32_t mask = (c >= 2 * i + 2) ? 0xFFFFFFFFu : ((c == 2 * i + 1) ? 0x0000FFFFu : 0u);
  t.w[0][c][i] = ((JOINT ? 0x80008000u : 0u) + static_cast<uint32_t>(2 * i) + (static_cast<uint32_t>(2 * i + 1) << 16)) & mask;
  if constexpr (!JOINT) t.w[1][c][i] = 0x00010001u & mask;
}
// A look-up's reads, and what they come to.
template <typename Rec, bool JOINT> struct LookUp {
  u32x4 w, wi, w1;
  Rec r;
  uint32_t g;
  MOFQ_DEV void read(const uint32_t* hist, const Rec* rec, const Weights& t, uint32_t n1) {
    g = n1 >> 3;
    asm("" : "+v"(g));   // opaque: both addresses are one shift-add of g (of n1 they would be a shift, a mask and an addition)
    w = *reinterpret_cast<const u32x4*>(hist + 4 * g);
    wi = *reinterpret_cast<const u32x4*>(t.w[0][n1 & 7]);
    if constexpr (!JOINT) w1 = *reinterpret_cast<const u32x4*>(t.w[1][n1 & 7]);
    r = rec[g];
  }
  MOFQ_DEV void counts(uint32_t& cin, uint32_t& win) const {
    uint32_t s = 0, n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s = dot2(w[j], wi[j], s);
      if constexpr (!JOINT) n = dot2(w[j], w1[j], n);
    }
    cin = JOINT ? s >> 15 : n;
    win = JOINT ? s & 0x7FFFu : s;
  }
};
template <typename In, bool JOINT> MOFQ_DEV void hist_prefix(const LookUp<Narrow, JOINT>& l, int, uint32_t& C, uint32_t& S) {
  uint32_t cin, win;
  l.counts(cin, win);
  S = l.r.sum + ((__umul24(__builtin_amdgcn_ubfe(l.r.word, 5u, 11u), cin) + win) << (l.r.word & 31u));
  C = (l.r.word >> 16) + cin;
}
template <typename In, bool JOINT> MOFQ_DEV void hist_prefix(const LookUp<Wide, JOINT>& l, int lo, uint32_t& C, double& S) {
  uint32_t cin, win;
  l.counts(cin, win);
  const float v0 = bits_to_float<In>(static_cast<uint32_t>(lo) + 8 * l.g);
  const float ulp = bits_to_float<In>(static_cast<uint32_t>(lo) + 8 * l.g + 1) - v0;   // exact
  const double s = __builtin_fma(static_cast<double>(v0), static_cast<double>(cin), l.r.sum);
  S = __builtin_fma(static_cast<double>(ulp), static_cast<double>(win), s);
  C = l.r.cnt + cin;
}

// One group's own count and sum, and its record.
template <typename In, bool JOINT> MOFQ_DEV void group_sum(const Narrow*, u32x4 w, int lo, int g, uint32_t& c, uint32_t& s, uint32_t& aux) {
  uint32_t wsum, m, shift;
  count8<JOINT>(w, c, wsum);
  mant_shift<In>(static_cast<uint32_t>(lo + 8 * g), exponent_of<In>(lo), m, shift);
  s = (__umul24(m, c) + wsum) << shift;
  aux = (m << 5) | shift;
}
template <typename In, bool JOINT> MOFQ_DEV void group_sum(const Wide*, u32x4 w, int lo, int g, uint32_t& c, double& s, uint32_t& aux) {
  uint32_t wsum;
  count8<JOINT>(w, c, wsum);
  const float v0 = bits_to_float<In>(static_cast<uint32_t>(lo + 8 * g));
  const float ulp = bits_to_float<In>(static_cast<uint32_t>(lo + 8 * g + 1)) - v0;
  s = __builtin_fma(static_cast<double>(ulp), static_cast<double>(wsum), static_cast<double>(v0) * static_cast<double>(c));
  aux = 0;
}
MOFQ_DEV Narrow make_record(const Narrow*, uint32_t c, uint32_t s, uint32_t aux) { return Narrow{s, (c << 16) | aux}; }
MOFQ_DEV Wide make_record(const Wide*, uint32_t c, double s, uint32_t) { return Wide{s, c, 0}; }
MOFQ_DEV uint32_t record_count(const Narrow& r) { return r.word >> 16; }
MOFQ_DEV uint32_t record_count(const Wide& r) { return r.cnt; }
MOFQ_DEV uint32_t wave_excl_scan(uint32_t v, uint32_t& total) { return wave_excl_scan_u32(v, total); }
MOFQ_DEV double wave_excl_scan(double v, double& total) { return wave_excl_scan_f64(v, total); }

// The records of all groups: lane `id` of `lanes` takes the groups [id gp, (id + 1) gp), gp <= GPMAX.
// NW > 1: by all threads of the workgroup (three barriers); NW = 1: by one wave alone, without
// barriers, for a short histogram: the caller's next barrier publishes the result.
template <typename In, bool JOINT, int NW, int GPMAX, typename Rec>
MOFQ_DEV void hist_records(const uint32_t* hist, Rec* rec, int lo, int ng, uint32_t* s_wc, typename Rec::sum_t* s_ws) {
  using sum_t = typename Rec::sum_t;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int id = NW > 1 ? tid : lane;
  const int gp = (ng + NW * 64 - 1) / (NW * 64);
  uint32_t c8[GPMAX], aux[GPMAX];
  sum_t s8[GPMAX];
  uint32_t ct = 0;
  sum_t st = 0;
#pragma unroll
  for (int i = 0; i < GPMAX; ++i) {
    const int g = id * gp + i;
    c8[i] = 0;
    s8[i] = 0;
    aux[i] = 0;
    if (i < gp && g < ng) {
      group_sum<In, JOINT>(rec, *reinterpret_cast<const u32x4*>(hist + 4 * g), lo, g, c8[i], s8[i], aux[i]);
      ct += c8[i];
      st += s8[i];
    }
  }
  uint32_t wct;
  sum_t wst;
  uint32_t cb = wave_excl_scan(ct, wct);
  sum_t sb = wave_excl_scan(st, wst);
  if constexpr (NW > 1) {
    if (lane == 0) { s_wc[wave] = wct; s_ws[wave] = wst; }
    __syncthreads();
    for (int w = 0; w < wave; ++w) { cb += s_wc[w]; sb += s_ws[w]; }
  }
#pragma unroll
  for (int i = 0; i < GPMAX; ++i) {
    const int g = id * gp + i;
    if (i < gp && g < ng) rec[g] = make_record(rec, cb, sb, aux[i]);
    cb += c8[i];
    sb += s8[i];
  }
  if (id == NW * 64 - 1) rec[ng] = make_record(rec, cb, sb, 0);
  if constexpr (NW > 1) __syncthreads();
}

template <typename In, int FA, int FB, int CH, typename Rec>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CH <= 2 ? 5 : (CH <= 6 ? 4 : 3))))
void sweep_hist_kernel(const SortedArgs a) {
  using L = Load8<In>;
  constexpr int THREADS = 256;
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  constexpr int NW = THREADS / 64;
  constexpr bool ANY_TAIL = FA == MOFQ_INT4 || FBX == MOFQ_INT4;
  constexpr int GPMAX = kHistMaxBins / 8 / THREADS;   // groups per thread at most

  constexpr bool JOINT = CH <= 2;   // 4096 elements at most
  static_assert(CH > 2 || CH * THREADS * 8 <= 4096, "count8");
  using sum_t = typename Rec::sum_t;

  // dynamic LDS: [records | the short histogram's | spare counters | counters | the short histogram's | 16 bytes]
  extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
  const int nbin = a.nbin, ntbin = ANY_TAIL ? a.ntbin : 0;   // multiples of 8
  const int ng = nbin >> 3, ntg = ntbin >> 3;
  Rec* const rec = reinterpret_cast<Rec*>(s_dyn);
  Rec* const trec = rec + (ng + 1);
  uint32_t* const hist = reinterpret_cast<uint32_t*>(s_dyn + (static_cast<size_t>((ng + 1) + (ntg + 1)) * sizeof(Rec) + 15) / 16 * 16 + 2 * kSpare);
  uint32_t* const thist = hist + (nbin >> 1);   // (counts stay below 2^16: a row has at most 24576 elements)

  __shared__ RowSearch<NF, NW> sh;
  __shared__ float s_wmax[NW];
  __shared__ double s_wsum[NW];
  __shared__ uint32_t s_wc[NW];
  __shared__ sum_t s_ws[NW];
  __shared__ __attribute__((aligned(16))) Weights s_weights;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t tensor = 0;                                                    // wave-uniform
#pragma unroll
  for (int i = 1; i < kSweepGroupMax; ++i) tensor += (blockIdx.x >= a.row0[i]);
  const int64_t row = blockIdx.x - a.row0[tensor];
  const SortedTensor& T = a.t[tensor];
  const typename L::elem* src = static_cast<const typename L::elem*>(T.w) + row * T.ld;
  const int K = a.n_clip;
  const int n = static_cast<int>(a.cols);
  if (tid < 32) fill_weights<JOINT>(s_weights, tid);

  // ---- load the row (it stays in registers until it is counted): absmax, energy; clear the counters ---
  u32x4 rawv[CH];
  float amax = 0.0f;
  uint32_t amax2 = 0;   // fp16 rows: running maximum of |x| in both halves of a register
  double en = 0.0;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int64_t c0 = (static_cast<int64_t>(j) * THREADS + tid) * 8;
    u32x4 raw = {0u, 0u, 0u, 0u};
    if (c0 < a.cols) raw = *reinterpret_cast<const u32x4*>(src + c0);
    rawv[j] = raw;
  }
  // what the tensor's finished rows favour: behind the row (loads return in order), by one wave (waves that
  // read it at different times could disagree)
  double tally = 0.0;
  if (NF == 2 && T.ahead.tally && wave == NW - 1) tally = tally_read(T.ahead);
  {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int i = tid; i < ng + ntg; i += THREADS) reinterpret_cast<u32x4*>(hist)[i] = zero;   // hist and thist are adjacent
  }
#pragma unroll
  for (int j = 0; j < CH; ++j) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t h0 = rawv[j][i] & 0xFFFFu, h1 = rawv[j][i] >> 16;
      const float v0 = bits_to_float<In>(h0), v1 = bits_to_float<In>(h1);
      if constexpr (std::is_same<In, F16>::value) {
        amax2 = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(f16x2, amax2),
                                                                       __builtin_bit_cast(f16x2, rawv[j][i] & 0x7FFF7FFFu)));
      } else {
        amax = __builtin_fmaxf(amax, __builtin_fmaxf(__builtin_fabsf(v0), __builtin_fabsf(v1)));
      }
      const double d0 = static_cast<double>(v0), d1 = static_cast<double>(v1);
      en = __builtin_fma(d0, d0, en);
      en = __builtin_fma(d1, d1, en);
    }
  }
  if constexpr (std::is_same<In, F16>::value)
    amax = __builtin_fmaxf(bits_to_float<In>(amax2 & 0xFFFFu), bits_to_float<In>(amax2 >> 16));
  amax = wave_max(amax);
  en = wave_sum(en);
  if (lane == 0) { s_wmax[wave] = amax; s_wsum[wave] = en; }
  __syncthreads();   // also: the counters are clear
  amax = s_wmax[0];
  en = s_wsum[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    amax = __builtin_fmaxf(amax, s_wmax[w]);
    en += s_wsum[w];
  }
  if (tid < 2 * MOFQ_MAX_CLIP) {   // thread f * MOFQ_MAX_CLIP + k
    const int f = __builtin_amdgcn_readfirstlane(tid / MOFQ_MAX_CLIP), k = tid % MOFQ_MAX_CLIP;
    const float qmax = (f == 0) ? Codec<FA>::QMAX : Codec<FBX>::QMAX;
    if (f < NF && k < K) {
      if (std::is_same<In, F16>::value && amax <= 65504.0f) {   // uniform
        const float ra = a.clip[k] * amax;
        sh.scale[f][k] = f == 0 ? search_scale<FA>(ra, a.scale_f16 != 0) : search_scale<FBX>(ra, a.scale_f16 != 0);
      } else {
        sh.scale[f][k] = unit_scale(amax, a.clip[k], qmax, a.scale_f16 != 0);
      }
    }
  }
  static_assert(2 * MOFQ_MAX_CLIP <= THREADS, "one thread per (format, candidate)");

  // ---- the histogram covers the nbin patterns up to the largest magnitude's (a non-finite
  // element lands in the last counter: the row's error is non-finite anyway) --------------------
  const int hmax = __builtin_amdgcn_readfirstlane(static_cast<int>(pattern_rtz<In>(__builtin_fminf(amax, 3.4028234e38f))));   // exact for a finite amax
  const int lo = (((hmax + 1 - nbin) > 0 ? (hmax + 1 - nbin) : 0) + 7) & ~7;
  const int tlo = (((hmax + 1 - ntbin) > 0 ? (hmax + 1 - ntbin) : 0) + 7) & ~7;
  {
    const RowCounters counters(hist, lo, nbin);
    const uint32_t thist_at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_u32*)thist));   // LDS byte address, a multiple of 16
#pragma unroll
    for (int j0 = 0; j0 < CH; j0 += 4) {
      constexpr int PART = CH < 4 ? CH : 4;
      uint32_t noted = 0;
#pragma unroll
      for (int j = j0; j < j0 + PART; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t w = j < CH ? rawv[j][i] : 0;
          // padding (zero) and whatever lies below every threshold has no counter
          if (j < CH) counters.count_pair(w);
          if constexpr (ANY_TAIL) note_negative(noted, w, tlo, 4 * (j - j0) + i);
        }
      if constexpr (ANY_TAIL) count_noted<THREADS * 16>(noted, src, static_cast<uint32_t>(j0 * THREADS + tid) * 16, tlo, ntbin, thist_at);
    }
  }
  __syncthreads();

  // ---- group prefixes ----------------------------------------------------------------------------
  // (the short histogram by the last wave alone, before the barriers of the long one's prefixes)
  if constexpr (ANY_TAIL)
    if (wave == NW - 1) hist_records<In, JOINT, 1, kHistMaxTailBins / 8 / 64>(thist, trec, tlo, ntg, s_wc, s_ws);
  hist_records<In, JOINT, NW, GPMAX>(hist, rec, lo, ng, s_wc, s_ws);
  const uint32_t c_total = record_count(rec[ng]);
  // sums are in units of this (1 where they are fp64 magnitudes)
  const float v_lo = bits_to_float<In>(static_cast<uint32_t>(lo));
  const double sum_unit = std::is_same<Rec, Narrow>::value ? static_cast<double>(bits_to_float<In>(static_cast<uint32_t>(lo) + 1) - v_lo) : 1.0;
  const double s_total = static_cast<double>(rec[ng].sum);
  // sum |x| enters the rounding bounds only: the counted elements' sum (raised beyond its rounding)
  // plus, for every other element, the magnitude of the first counted pattern, which exceeds its own
  const double l1 = sum_unit * s_total * (1.0 + 0x1p-40) + static_cast<double>(n) * static_cast<double>(v_lo);

  // ---- level boundaries of every candidate: one lane per candidate, one wave per (format, 64
  // candidates) --------------------------------------------------------------------------------
  {
    const int chunks = (K + 63) >> 6;
    const int before_lo = pattern_before<In>(lo), before_tlo = pattern_before<In>(tlo);
    auto unit = [&](auto normal_tag, auto fmt_c, const int f, const int k) {
      constexpr int FMT = decltype(fmt_c)::value;
      constexpr bool NORMAL = decltype(normal_tag)::value, TAIL = FMT == MOFQ_INT4;
      const float s = sh.scale[f][k < K ? k : K - 1];
      const float inv = std::is_same<In, F16>::value ? reciprocal(s) : 1.0f / s;
      // H = the largest pattern h with fl32(v(h) * inv) <= thr; returns H - first + 1.  Where subnormals are
      // counted: inv and the product are each off by at most 2^-24, so the decision flips between thr s (1 - 2^-22)
      // and thr s (1 + 2^-22); thr_est is thr (1 - 2^-21) (to 2^-24), so the pattern of thr_est s rounded toward zero passes,
      // and the second pattern above it, at least 2^-11 larger, does not: one decision, on the first, tells.
      const double per_edge = edge_unit(s, inv);
      auto counters_below = [&](const int q, const int first, const int before) {
        if constexpr (NORMAL) return patterns_below<In>(a.thr_edge[f][q], per_edge, before);
        const int est = static_cast<int>(pattern_rtz<In>(a.thr_est[f][q] * s));
        const bool above = scaled<In>(static_cast<uint32_t>(est + 1), inv) <= a.thr[f][q];
        return est + (1 - first) + (above ? 1 : 0);
      };
      // counters at or below H, as a number of counters: H - lo + 1 within [0, nbin].  A threshold
      // more than one pattern below the histogram's range sends the candidate to the exact pass:
      // uncounted elements might lie above it.  The first boundary's is the smallest (and a negative
      // number is a large one to the unsigned minimum, so addresses stay inside).
      int fewest = 0;
      double ca = 0.0, ca_tail = 0.0;
      uint32_t cb4 = 0;   // 4 sum_b (count up to boundary b) (m_{b+1}^2 - m_b^2): an integer below 2^31
      using Look = LookUp<Rec, JOINT>;
      auto look_up = [&](Look& l, const int q) {
        const int n1 = counters_below(q, lo, before_lo);
        fewest = n1;
        l.read(hist, rec, s_weights, min(static_cast<uint32_t>(n1), static_cast<uint32_t>(nbin)));
      };
      auto look_up_tail = [&](Look& l) {
        const int n1 = counters_below(7, tlo, before_tlo);
        fewest = min(fewest, n1);
        l.read(thist, trec, s_weights, min(static_cast<uint32_t>(n1), static_cast<uint32_t>(ntbin)));
      };
      auto add = [&](const Look& l, const double step, const uint32_t weight) {
        uint32_t C;
        sum_t S;
        hist_prefix<In, JOINT>(l, lo, C, S);
        ca = __builtin_fma(static_cast<double>(S), -step, ca);
        cb4 = __umul24(C, weight) + cb4;
        asm volatile("" : "+v"(ca), "+v"(cb4));   // worked out here and not where the sums are used
      };
      auto add_tail = [&](const Look& l) {
        // negative elements with a pattern above H: the short histogram's totals less its prefix
        uint32_t C;
        sum_t S;
        hist_prefix<In, JOINT>(l, tlo, C, S);
        ca_tail = static_cast<double>(trec[ntg].sum - S);
        if constexpr (std::is_same<Rec, Narrow>::value) {
          const float v_tlo = bits_to_float<In>(static_cast<uint32_t>(tlo));
          ca_tail *= static_cast<double>(bits_to_float<In>(static_cast<uint32_t>(tlo) + 1) - v_tlo);
        }
        cb4 -= __umul24(record_count(trec[ntg]) - C, quad_step<FMT>(7));
      };
      if constexpr (NORMAL) {
        // one look-up's reads under way while the one before is worked out (all eight at once cost some 80 registers)
        Look l[2];
        look_up(l[0], 6);
#pragma unroll
        for (int q = 6; q >= 0; --q) {   // the first boundary last
          __builtin_amdgcn_sched_barrier(0);
          if (q > 0) look_up(l[(7 - q) & 1], q - 1);
          else if constexpr (TAIL) look_up_tail(l[1]);
          __builtin_amdgcn_sched_barrier(0);
          add(l[(6 - q) & 1], 0.5 * (1 << half_steps_log2<FMT>(q)), quad_step<FMT>(q));
        }
        if constexpr (TAIL) add_tail(l[1]);
      } else {
#pragma unroll 1
        for (int q = 6; q >= 0; --q) {
          Look l;
          look_up(l, q);
          add(l, -a.dgd[f][q], static_cast<uint32_t>(-a.dg2q[f][q]));
        }
        if constexpr (TAIL) {
          Look l;
          look_up_tail(l);
          add_tail(l);
        }
      }
      if (k < K) {
        const double gl = static_cast<double>(a.g_last[f]);
        const double A = __builtin_fma(sum_unit, ca + gl * s_total, ca_tail);
        const double B = -0.25 * static_cast<double>(static_cast<int>(cb4)) + gl * gl * static_cast<double>(c_total);
        const double sc = static_cast<double>(s);
        const double v = (en - 2.0 * sc * A) + sc * sc * B;   // filtered error
        sh.fast[f][k] = fewest < 0 ? __builtin_nan("") : v;
      }
    };
    auto units = [&](auto normal_tag) {
      for (int u = wave; u < NF * chunks; u += NW) {
        const int f = u / chunks;                         // wave-uniform
        const int k = (u - f * chunks) * 64 + lane;
        if (f == 0) unit(normal_tag, std::integral_constant<int, FA>{}, 0, k);
        else unit(normal_tag, std::integral_constant<int, FBX>{}, NF - 1, k);
      }
    };
    if (lo >= (1 << Pattern<In>::MANT)) units(std::true_type{});   // no subnormal has a counter
    else units(std::false_type{});
  }
  __syncthreads();

  // ---- winners.  With 32-bit sums everything but the energy is exact; fp64 sums: a group's sum is exact
  // (products and sum of fewer than 2^27 units of one ulp), a group prefix adds at most GPMAX of them
  // in a thread, 6 levels of the wave scan and the waves before, and a look-up adds two exact products:
  // fewer than 16 roundings, whatever the row's length.  The re-scored values lie over the records,
  // which are no longer needed (the host sizes the dynamic LDS for it).
  static_assert(GPMAX + 6 + NW + 2 <= 16, "depth of the prefix sums");
  finish_row<In, FA, FB, THREADS, CH, std::is_same<Rec, Narrow>::value>(sh, reinterpret_cast<double*>(s_dyn), src, n, K, en, l1, a.g_absmax, T.rec, row);
  Raw8<In> kept[CH];
#pragma unroll
  for (int j = 0; j < CH; ++j) kept[j].w = rawv[j];
  if (T.ahead.codes) emit_row_ahead<In, FA, FB, THREADS, CH>(sh, T.ahead, tally, kept, src, n, row);   // uniform
}

// Dynamic LDS: the records and counters of both histograms; the shortlist's re-scored values lie
// over their start later.
template <typename In, int FA, int FB, typename Rec>
int launch_hist_shape(const SortedArgs& a, int64_t total_rows, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(total_rows));
  const int64_t chunks = a.cols / 8;
  const int ng = a.nbin / 8, ntg = a.ntbin / 8;
  const size_t lds = std::max<size_t>((static_cast<size_t>((ng + 1) + (ntg + 1)) * sizeof(Rec) + 15) / 16 * 16 + 2 * static_cast<size_t>(kSpare + a.nbin + a.ntbin) + 16,
                                      2 * MOFQ_MAX_CLIP * sizeof(double));   // at least the shortlist's values
#define MOFQ_HIST(CH)                                                                         \
  if (chunks <= 256 * (CH)) {                                                                  \
    hipLaunchKernelGGL((sweep_hist_kernel<In, FA, FB, CH, Rec>), grid, dim3(256), lds, st, a);  \
    return hip_status(hipGetLastError());                                                      \
  }
  MOFQ_HIST(1)   //  2048 columns
  MOFQ_HIST(2)   //  4096
  MOFQ_HIST(4)   //  8192
  MOFQ_HIST(6)   // 12288
  MOFQ_HIST(12)  // 24576
#undef MOFQ_HIST
  return MOFQ_ERR_UNSUPPORTED;
}

// 32-bit sums where they cannot overflow: the counted patterns reach at most `span` binades above
// the first one's, so a magnitude is below 2^(MANT + 1 + span) units.
template <typename In, int FA, int FB>
int launch_hist_sums(const SortedArgs& a, int64_t total_rows, hipStream_t st) {
  constexpr int ppb = 1 << Pattern<In>::MANT;
  const int span = (std::max(a.nbin, a.ntbin) + ppb - 1) / ppb;
  if constexpr (std::is_same<In, F16>::value)   // (bf16 rows with so few patterns have their own kernel)
    if (span <= 16 && (a.cols << (Pattern<In>::MANT + 1 + span)) < (int64_t{1} << 32)) return launch_hist_shape<In, FA, FB, Narrow>(a, total_rows, st);
  return launch_hist_shape<In, FA, FB, Wide>(a, total_rows, st);
}

}  // namespace

int launch_sweep_hist(const SweepParams& p, const SortedArgs& a, int64_t total_rows, hipStream_t st) {
  if (a.nbin <= 0 || (p.dtype != MOFQ_F16 && p.dtype != MOFQ_BF16)) return MOFQ_ERR_UNSUPPORTED;
  if (pattern_search_fits(p, a.nbin, a.ntbin)) return launch_sweep_pattern(p, a, total_rows, st);
  const int fa = p.fmt[0], fb = p.n_fmt == 2 ? p.fmt[1] : -1;
  const bool h = p.dtype == MOFQ_F16;
  if (fa == MOFQ_INT4 && fb == MOFQ_FP4_E2M1)
    return h ? launch_hist_sums<F16, MOFQ_INT4, MOFQ_FP4_E2M1>(a, total_rows, st) : launch_hist_sums<BF16, MOFQ_INT4, MOFQ_FP4_E2M1>(a, total_rows, st);
  if (fa == MOFQ_INT4 && fb == -1)
    return h ? launch_hist_sums<F16, MOFQ_INT4, -1>(a, total_rows, st) : launch_hist_sums<BF16, MOFQ_INT4, -1>(a, total_rows, st);
  if (fa == MOFQ_FP4_E2M1 && fb == -1)
    return h ? launch_hist_sums<F16, MOFQ_FP4_E2M1, -1>(a, total_rows, st) : launch_hist_sums<BF16, MOFQ_FP4_E2M1, -1>(a, total_rows, st);
  return MOFQ_ERR_UNSUPPORTED;
}

}  // namespace mofq
