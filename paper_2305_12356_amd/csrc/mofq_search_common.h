// Shared by the per-channel searches that do not score every (element, candidate) pair
// (mofq_sweep_sorted.hip: sort the row and search it; mofq_sweep_hist.hip and mofq_sweep_bf16.hip: count the
// row's bit patterns): their kernel arguments and the device helpers they use.
#pragma once
#include <cmath>
#include <type_traits>

#include "mofq_codes.h"
#include "mofq_internal.h"

namespace mofq {

// One launch searches up to kSweepGroupMax tensors of one row length, dtype and configuration:
// the rows of all tensors are numbered through, one workgroup per row.
struct SortedTensor {
  const void* w;
  int64_t ld;
  UnitRecords rec;
  AheadCodes ahead;   // histogram kernels only
};
struct SortedArgs {
  SortedTensor t[kSweepGroupMax];
  uint32_t row0[kSweepGroupMax];   // number of the first row of tensor i (unused entries: 0xFFFFFFFF)
  int64_t cols;                    // of every tensor
  int32_t scale_f16, n_clip;
  int32_t nbin, ntbin;             // histogram kernel: counters of the row's histogram and of INT4's negative elements
  float clip[MOFQ_MAX_CLIP];
  // per format slot: level magnitudes 0 = m_0 < m_1 < ... < m_7;  |level|(t) <= m_b  <=>  t <= thr[b]
  // for b = 0..6.  Entry 7 is INT4's extra boundary (|t| below it: a negative element stays on -7)
  // with the weights of the step from 7 to 8; unused (zero weights) for E2M1.
  float thr[2][8];
  float thr_est[2][8];   // histogram kernels: a shade below thr
  double thr_edge[2][8]; // histogram kernels: between the last product that rounds to thr and the first beyond (decision_edge)
  double dgd[2][8];   // m_b - m_{b+1};  entry 7: 8 - 7
  int32_t dg2q[2][8]; // 4 (m_b^2 - m_{b+1}^2): an integer for every 4-bit format;  entry 7: 4 (64 - 49)
  float g_last[2];    // m_7
  float g_absmax[2];  // largest |level|
};

// Where the exact products |x| * inv that round to thr or below end, as a number that none of them is near: half an ulp above
// thr, which itself rounds to the even neighbour, moved by 2^-40 to the side that the tie belongs to.  A product has 35 bits
// at most and that midpoint 25, so products other than the tie are 2^-36 and more away from it.
constexpr double decision_edge(float thr) {
  const uint32_t u = __builtin_bit_cast(uint32_t, thr);
  const double mid = 0.5 * (static_cast<double>(thr) + static_cast<double>(__builtin_bit_cast(float, u + 1u)));
  return mid * (u & 1u ? 1.0 - 0x1p-40 : 1.0 + 0x1p-40);
}

// How many bit patterns lie between a threshold t = c * amax and amax at most: a pattern is
// (exponent, mantissa) read as an integer, i.e. PPB * (log2 of the value + a term in [0, 0.0861))
// up to a constant, so two values a factor 1 / c apart are at most PPB * (log2(1 / c) + 0.0861) + 1
// patterns apart (fewer among subnormals).  The scale's own roundings move a threshold by less than
// a pattern; the kernel rounds the first counter's pattern up to a multiple of 8.
inline int hist_bins(double ratio_amax_over_threshold, int ppb) {
  const double lg = std::log2(ratio_amax_over_threshold);
  const double bins = ppb * ((lg > 0.0 ? lg : 0.0) + 0.09) + 24.0;
  if (!(bins < 1.0e6)) return 1 << 20;
  return (static_cast<int>(std::ceil(bins)) + 7) / 8 * 8;
}

constexpr int kHistMaxBins = 8192;      // histogram kernel: patterns with a counter at most (16 KB)
constexpr int kHistMaxTailBins = 2048;  // of INT4's negative elements

// The histogram kernel for arguments with nbin > 0 (mofq_sweep_hist.hip).
int launch_sweep_hist(const SweepParams& p, const SortedArgs& a, int64_t total_rows, hipStream_t st);
// The one of bf16 rows and of 8-bit formats (mofq_sweep_bf16.hip), and whether these histograms fit it.
int launch_sweep_pattern(const SweepParams& p, const SortedArgs& a, int64_t total_rows, hipStream_t st);
bool pattern_search_fits(const SweepParams& p, int nbin, int ntbin);

namespace {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// ---- sort keys ------------------------------------------------------------------------
// The key of an element is the low 15 bits of its own 16-bit pattern (the magnitude; fp16 and
// bf16 magnitudes order like their patterns); the sign bit rides along untouched.
typedef short i16x2 __attribute__((ext_vector_type(2)));
MOFQ_DEV uint32_t sign_fill2(uint32_t w) {   // each half: 0xFFFF where its top bit is set, else 0
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, w) >> 15);
}

template <typename In> MOFQ_DEV float bits_to_float(uint32_t h);
template <> MOFQ_DEV float bits_to_float<F16>(uint32_t h) {
  return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(h)));
}
template <> MOFQ_DEV float bits_to_float<BF16>(uint32_t h) { return u2f(h << 16); }

// fl32(|x| * inv) for the element with bit pattern h.  For fp16 the widening and the product are
// one mixed-precision fused multiply-add with a zero addend: the same single rounding of the
// exact product.
template <typename In> MOFQ_DEV float scaled(uint32_t h, float inv);
template <> MOFQ_DEV float scaled<F16>(uint32_t h, float inv) {
  return __builtin_fmaf(__builtin_fabsf(static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(h)))), inv, 0.0f);
}
template <> MOFQ_DEV float scaled<BF16>(uint32_t h, float inv) { return __builtin_fabsf(u2f(h << 16)) * inv; }

// x plus the value the data-parallel-primitive control CTRL brings from another lane (0 where
// the control has no source lane or ROW_MASK excludes the row)
template <int CTRL, int ROW_MASK> MOFQ_DEV uint32_t dpp_add_u32(uint32_t x) {
  return x + static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROW_MASK, 0xf, false));
}
// exclusive prefix over the wave and the wave total: shifts by 1, 2, 4, 8 inside each row of
// 16 lanes, then lane 15 of a row into the next row, then lane 31 into the upper half
MOFQ_DEV uint32_t wave_excl_scan_u32(uint32_t v, uint32_t& total) {
  uint32_t inc = v;
  inc = dpp_add_u32<0x111, 0xf>(inc);   // row_shr:1
  inc = dpp_add_u32<0x112, 0xf>(inc);   // row_shr:2
  inc = dpp_add_u32<0x114, 0xf>(inc);   // row_shr:4
  inc = dpp_add_u32<0x118, 0xf>(inc);   // row_shr:8
  inc = dpp_add_u32<0x142, 0xa>(inc);   // row_bcast:15 into rows 1 and 3
  inc = dpp_add_u32<0x143, 0xc>(inc);   // row_bcast:31 into rows 2 and 3
  total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), 63));
  return inc - v;
}
// the same for 64-bit integers: each step moves the two halves of the running sum separately
template <int CTRL, int ROW_MASK> MOFQ_DEV uint64_t dpp_add_u64(uint64_t x) {
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(x)), CTRL, ROW_MASK, 0xf, false));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(x >> 32)), CTRL, ROW_MASK, 0xf, false));
  return x + ((static_cast<uint64_t>(hi) << 32) | lo);
}
MOFQ_DEV uint64_t wave_incl_scan_u64(uint64_t v) {
  v = dpp_add_u64<0x111, 0xf>(v);   // row_shr:1
  v = dpp_add_u64<0x112, 0xf>(v);   // row_shr:2
  v = dpp_add_u64<0x114, 0xf>(v);   // row_shr:4
  v = dpp_add_u64<0x118, 0xf>(v);   // row_shr:8
  v = dpp_add_u64<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  return dpp_add_u64<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
}
// and for doubles
template <int CTRL, int ROW_MASK> MOFQ_DEV double dpp_add_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(u)), CTRL, ROW_MASK, 0xf, false));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(u >> 32)), CTRL, ROW_MASK, 0xf, false));
  return x + __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);   // +0.0 where nothing arrives
}
MOFQ_DEV double wave_excl_scan_f64(double v, double& total) {
  double inc = v;
  inc = dpp_add_f64<0x111, 0xf>(inc);   // row_shr:1
  inc = dpp_add_f64<0x112, 0xf>(inc);   // row_shr:2
  inc = dpp_add_f64<0x114, 0xf>(inc);   // row_shr:4
  inc = dpp_add_f64<0x118, 0xf>(inc);   // row_shr:8
  inc = dpp_add_f64<0x142, 0xa>(inc);   // row_bcast:15 into rows 1 and 3
  inc = dpp_add_f64<0x143, 0xc>(inc);   // row_bcast:31 into rows 2 and 3
  total = __shfl(inc, 63, 64);
  return inc - v;
}

// sum over the wave in fp32 (uniform result)
MOFQ_DEV float wave_sum_f32(float v) {
  v += dpp_f32<DPP_QUAD_XOR1>(v);
  v += dpp_f32<DPP_QUAD_XOR2>(v);
  v += dpp_f32<DPP_ROW_HALF_MIRROR>(v);
  v += dpp_f32<DPP_ROW_MIRROR>(v);
  const float a = u2f(__builtin_amdgcn_readlane(static_cast<int>(f2u(v)), 0));
  const float b = u2f(__builtin_amdgcn_readlane(static_cast<int>(f2u(v)), 16));
  const float c = u2f(__builtin_amdgcn_readlane(static_cast<int>(f2u(v)), 32));
  const float d = u2f(__builtin_amdgcn_readlane(static_cast<int>(f2u(v)), 48));
  return (a + b) + (c + d);
}

// bit pattern of x >= 0 rounded toward zero to the input type
template <typename In> MOFQ_DEV uint32_t pattern_rtz(float x);
template <> MOFQ_DEV uint32_t pattern_rtz<F16>(float x) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(x, 0.0f));   // the high half is +0
}
template <> MOFQ_DEV uint32_t pattern_rtz<BF16>(float x) { return f2u(x) >> 16; }
template <typename In> struct Pattern;
template <> struct Pattern<F16> { static constexpr int MANT = 10, BIAS = 15; };
template <> struct Pattern<BF16> { static constexpr int MANT = 7, BIAS = 127; };

// 4-bit formats: log2 of twice the step from level q to the next, and 4 (m_{q+1}^2 - m_q^2)
template <int FMT> constexpr int half_steps_log2(int q) { return FMT == MOFQ_INT4 ? 1 : (q < 4 ? 0 : (q < 6 ? 1 : 2)); }
template <int FMT> constexpr uint32_t quad_step(int q) {
  constexpr uint32_t e2m1[7] = {1, 3, 5, 7, 20, 28, 80};
  return FMT == MOFQ_INT4 ? 8u * static_cast<uint32_t>(q) + 4u : (q < 7 ? e2m1[q] : 0u);
}

// ra / QMAX by one multiplication and Markstein's correction: the correctly rounded quotient for 7 and 6 (all mantissas
// checked) wherever it is at least 2^-126.
template <int FMT> MOFQ_BOTH float over_qmax(float ra) {
  constexpr float d = Codec<FMT>::QMAX, r = 1.0f / d;
  const float q = ra * r;
  return __builtin_fmaf(__builtin_fmaf(-d, q, ra), r, q);
}
// unit_scale of a search for a finite absmax, ra = ratio * absmax; a non-finite unit comes out as 1.
template <int FMT> MOFQ_DEV float search_scale(float ra, bool f16) {
  float s = over_qmax<FMT>(ra);
  if (f16) s = round_fp16_clamped(s);
  if (!(s >= 0x1p-126f)) s = 1.0f;
  return s;
}

// ---- the largest pattern that a decision passes --------------------------------------------------------
// fl32(|x| * inv) <= thr, inv = fl32(1 / s): the elements that pass are those up to decision_edge(thr) / inv, and
// 1 / inv = s + s (1 - s inv) to 2^-48 (|1 - s inv| <= 2^-24; both steps are exact but for the last rounding).  The
// quotient in fp64 is cut off at the input type's mantissa by taking the top of its bits: exponent and mantissa
// are the pattern but for the difference of the biases.  Three instructions a boundary, against seven for a rounded
// estimate and the decision itself on the next pattern.  Holds for normal numbers of the input type; a quotient
// below the smallest one gives a number below its pattern.
MOFQ_BOTH double edge_unit(float s, float inv) {
  const double sd = static_cast<double>(s);
  return __builtin_fma(sd, __builtin_fma(-sd, static_cast<double>(inv), 1.0), sd);
}
template <typename In> constexpr int kPatternBase = (1023 - Pattern<In>::BIAS) << Pattern<In>::MANT;
// How many patterns from one on pass; before: pattern_before of that one.
template <typename In> MOFQ_DEV int pattern_before(int first) {
  int b = __builtin_amdgcn_readfirstlane(first + kPatternBase<In> - 1);
  asm("" : "+s"(b));   // opaque: one subtraction
  return b;
}
template <typename In> MOFQ_BOTH int pattern_top(double edge, double unit) {
  return static_cast<int>(static_cast<uint32_t>(__builtin_bit_cast(uint64_t, edge * unit) >> 32) >> (20 - Pattern<In>::MANT));
}
template <typename In> MOFQ_DEV int patterns_below(double edge, double unit, int before) { return pattern_top<In>(edge, unit) - before; }

// 1 / s, correctly rounded for s in [2^-126, 2^125] (all of them checked): the hardware's reciprocal and one step of
// Newton's iteration r + r (1 - s r).
MOFQ_DEV float reciprocal(float s) {
  const float r = __builtin_amdgcn_rcpf(s);
  return __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);
}

// Lexicographic minimum of (value, index) over the wave by data-parallel-primitive moves: the
// smallest value (no NaN among the inputs), then the smallest index among the lanes that hold it.
template <int CTRL> MOFQ_DEV int dpp_i32(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true); }
MOFQ_DEV void wave_argmin_dpp(double& v, int& idx) {
  double m = v;
  m = __builtin_fmin(m, dpp_f64<DPP_QUAD_XOR1>(m));
  m = __builtin_fmin(m, dpp_f64<DPP_QUAD_XOR2>(m));
  m = __builtin_fmin(m, dpp_f64<DPP_ROW_HALF_MIRROR>(m));
  m = __builtin_fmin(m, dpp_f64<DPP_ROW_MIRROR>(m));
  m = __builtin_fmin(__builtin_fmin(readlane_f64(m, 0), readlane_f64(m, 16)), __builtin_fmin(readlane_f64(m, 32), readlane_f64(m, 48)));
  int c = (v == m) ? idx : 0x7FFFFFFF;
  c = min(c, dpp_i32<DPP_QUAD_XOR1>(c));
  c = min(c, dpp_i32<DPP_QUAD_XOR2>(c));
  c = min(c, dpp_i32<DPP_ROW_HALF_MIRROR>(c));
  c = min(c, dpp_i32<DPP_ROW_MIRROR>(c));
  idx = min(min(__builtin_amdgcn_readlane(c, 0), __builtin_amdgcn_readlane(c, 16)),
            min(__builtin_amdgcn_readlane(c, 32), __builtin_amdgcn_readlane(c, 48)));
  v = m;
}


// m and shift of the group at pattern p (subnormals: the first normal binade's ulp, no leading bit)
template <typename In> MOFQ_DEV void mant_shift(uint32_t p, int e_lo, uint32_t& m, uint32_t& shift) {
  constexpr int MANT = Pattern<In>::MANT;
  const uint32_t e1 = __builtin_elementwise_sub_sat(p >> MANT, 1u);                   // exponent field less one, 0 for subnormals
  // mantissa with its leading bit: p - (e1 << MANT) (as a shift and a subtraction it costs one instruction more)
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(m) : "v"(e1), "s"(-(1 << MANT)), "v"(p));
  int first = __builtin_amdgcn_readfirstlane(e_lo - 1);
  asm("" : "+s"(first));   // opaque: one subtraction
  shift = e1 - static_cast<uint32_t>(first);
}
template <typename In> MOFQ_DEV int exponent_of(int p) { const int e = p >> Pattern<In>::MANT; return e > 1 ? e : 1; }

// ---- counting a row's bit patterns ---------------------------------------------------------------------
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

MOFQ_DEV uint32_t dot2(uint32_t a, uint32_t b, uint32_t c) {   // a.lo b.lo + a.hi b.hi + c
  return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b), c, false);
}

// count and index-weighted count of eight counters, two per word.  JOINT: rows of up to 4096 elements, whose
// weighted count stays below 7 * 2^12 < 2^15: one sum with the weights 2^15 + i (two instructions fewer).
template <bool JOINT> MOFQ_DEV void count8(const u32x4 w, uint32_t& c, uint32_t& wsum) {
  constexpr uint32_t base = JOINT ? 0x80008000u : 0u;
  uint32_t s = 0;
  c = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if constexpr (!JOINT) c = dot2(w[j], 0x00010001u, c);
    s = dot2(w[j], base + (static_cast<uint32_t>(2 * j) | (static_cast<uint32_t>(2 * j + 1) << 16)), s);
  }
  if constexpr (JOINT) c = s >> 15;
  wsum = JOINT ? s & 0x7FFFu : s;
}

// One counter (16 bits, two per word) at LDS byte address base + byte_off (a multiple of 4) more: the low half
// of the word for an even counter number, else the high half.
MOFQ_DEV void count_at(uint32_t base, uint32_t byte_off, uint32_t parity16, uint32_t one = 1u) {
  // 1 or 65536: the shift takes the low five bits of its operand, which is 16 times the counter number
  __hip_atomic_fetch_add((lds_u32*)static_cast<uintptr_t>(base + byte_off), one << (parity16 & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The counters of a row, with kSpare counters before them that nobody reads: an element below the counted patterns goes to
// one of those, a lane to its own (one for all serialises the additions), which costs one instruction for two elements instead of a
// comparison and a change of the active lanes for each.
constexpr int kSpare = 16;
struct RowCounters {
  uint32_t at, one;        // LDS byte address of the spare ones; 1 in a register of its own (the half-selecting shift takes no constant)
  i16x2 first, last, spare;
  MOFQ_DEV RowCounters(const uint32_t* counters, int lo, int nbin)
      : at(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_u32*)counters)) - 2 * kSpare), one(1) {
    const short f = static_cast<short>(lo - kSpare), l = static_cast<short>(nbin - 1 + kSpare), s = static_cast<short>(threadIdx.x & (kSpare - 1));
    first = i16x2{f, f};
    last = i16x2{l, l};
    spare = i16x2{s, s};
    asm("" : "+v"(one), "+v"(spare));
  }
  // both halves of a word of two elements at once: signed 16-bit differences to the first pattern (patterns are below 2^15),
  // clamped to the last counter (a non-finite element's row has a non-finite error anyway)
  MOFQ_DEV void count_pair(uint32_t w) const {
    const i16x2 b2 = __builtin_elementwise_max(__builtin_elementwise_min(__builtin_bit_cast(i16x2, w & 0x7FFF7FFFu) - first, last), spare);
    uint32_t off2 = __builtin_bit_cast(uint32_t, b2 << static_cast<short>(1)) & 0xFFFCFFFCu;
    uint32_t par2 = __builtin_bit_cast(uint32_t, b2 << static_cast<short>(4));
    // opaque: the halves are then selected by the instructions that use them instead of masked first
    asm("" : "+v"(off2), "+v"(par2));
    count_at(at, off2 & 0xFFFFu, par2, one);
    count_at(at, off2 >> 16, par2 >> 16, one);
  }
};

// The counters of a row's negative elements at or above pattern tlo, counted apart from the others.  They are
// few (the boundary lies half way up to the row's largest magnitude), but among the 128 elements of a wave's
// word there is nearly always one: as a branch of the counting loop they cost every word 15 instructions.
// So the loop only notes them, 3 instructions per word, and they are read again (they come from
// L2) once the loop is done: a lane has two at most in most rows.
// A mask holds the words of four 16-byte chunks: bits t and 16 + t the halves of word t.
MOFQ_DEV void note_negative(uint32_t& mask, uint32_t w, int tlo, int t) {
  const unsigned short below = static_cast<unsigned short>(0x8000 + tlo - 1);
  const u16x2 below2 = {below, below}, one = {1, 1};
  uint32_t over = __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, w), below2));   // sign and magnitude as one number
  asm("" : "+v"(over));   // opaque: else two comparisons and selects
  mask |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, over), one)) << t;
}
// chunk0: byte offset of the lane's first chunk of the mask; its chunks are STRIDE bytes apart.
template <uint32_t STRIDE>
MOFQ_DEV void count_noted(uint32_t mask, const uint16_t* src, uint32_t chunk0, int tlo, int ntbin, uint32_t at) {
  static_assert(STRIDE % 4 == 0, "chunks");
  while (mask) {
    const uint32_t p = static_cast<uint32_t>(__builtin_ctz(mask));
    mask &= mask - 1;
    const uint32_t off = (p & 12u) * (STRIDE / 4) + (p & 3u) * 4 + (p >> 4) * 2 + chunk0;
    const int b = min((*reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(src) + off) & 0x7FFF) - tlo, ntbin - 1);
    count_at(at, (static_cast<uint32_t>(b) >> 1) << 2, static_cast<uint32_t>(b) << 4);
  }
}


// ---- what follows the filtered errors of a row: shortlist, exact re-score, the winners -----------------
// Shared memory of these steps (the filtered errors are the caller's to fill).
template <int NF, int NW> struct RowSearch {
  float scale[NF][MOFQ_MAX_CLIP];
  double fast[NF][MOFQ_MAX_CLIP];       // filtered errors; NaN: has to be scored exactly
  double thr[NF], p2[NW], p2b[NW], best[NF], tally;
  float best_scale[NF];
  int direct[NF];                       // the winning candidate where no element-wise pass is needed, else -1
  int nlist;
  uint8_t list[NF * MOFQ_MAX_CLIP];     // format * MOFQ_MAX_CLIP + candidate
};

// Shortlist margin and rounding bound of the filtered error v = (en - 2 s A) + s^2 B.
// EXACT_SUMS: A and B are exact but for one addition.  The error of a candidate is at most the energy (0 is a
// grid value, and clipping moves an element towards itself), so s^2 B <= (|x| + |x - s g|)^2 <= 4 en and
// 2 s A <= 5 en; en itself comes from a summation tree of depth E + 14, and six operations round on terms
// of at most 6 en: |v - exact| <= u (E + 48) en =: beta.  The margin 2^-40 en is far above 2 beta.
// Otherwise prefix sums are off by up to D u sum|x| (fewer than D roundings each): the bound is the sorting
// kernel's.
struct FilterBounds {
  double margin, beta;
};
// 8-bit formats: B is exact (an integer below 2^51 in units of the smallest level's square), A takes fewer than
// 24 roundings on terms of at most 512 sum|x|.
template <int E, bool EXACT_SUMS, int BITS>
MOFQ_DEV FilterBounds filter_bounds(double en, double l1, double smax, double gmax, double n) {
  if constexpr (EXACT_SUMS && BITS == 8) {
    const double beta = 0x1p-53 * ((E + 48) * en + 48.0 * 512.0 * smax * l1);
    return {__builtin_fmax(0x1p-40 * en, 4.0 * beta), beta};
  } else if constexpr (EXACT_SUMS) {
    return {0x1p-40 * en, 0x1p-53 * (E + 48) * en};
  } else {
    constexpr double D = 16.0;
    const double mag = en + 2.0 * smax * gmax * l1 + smax * smax * gmax * gmax * n;
    return {0x1p-33 * mag, 0x1p-53 * (40.0 * D * 2.0 * smax * l1 + (E + 32) * en + 8.0 * smax * smax * gmax * gmax * n)};
  }
}

// From the filtered errors (published by a barrier) to the winner of each format: rec of the row, and
// sh.best / sh.best_scale (for the caller to publish).  The row at src is read again where the filter cannot
// separate the candidates; s_val: MOFQ_MAX_CLIP doubles per format of LDS that is free by then.
template <typename In, int FA, int FB, int THREADS, int CH, bool EXACT_SUMS>
MOFQ_DEV void finish_row(RowSearch<(FB >= 0 ? 2 : 1), THREADS / 64>& sh, double* s_val, const uint16_t* src, int n, int K, double en, double l1,
                         const float (&g_absmax)[2], const UnitRecords& rec, int64_t row) {
  constexpr int NF = (FB >= 0) ? 2 : 1, FBX = (FB >= 0) ? FB : FA, NW = THREADS / 64, E = CH * 8;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int f = wave; f < NF; f += NW) {
    double m = __builtin_inf();
    int km = 0;
    float smax = 0.0f;
    for (int k = lane; k < K; k += 64) {
      const double v = sh.fast[f][k];
      if (v < m) { m = v; km = k; }
      smax = __builtin_fmaxf(smax, sh.scale[f][k]);
    }
    wave_argmin_dpp(m, km);
    if constexpr (!EXACT_SUMS || Codec<FA>::BITS == 8) smax = wave_max(smax);
    const FilterBounds fb = filter_bounds<E, EXACT_SUMS, Codec<FA>::BITS>(en, l1, static_cast<double>(smax), static_cast<double>(g_absmax[f]), static_cast<double>(n));
    const double thr = m + fb.margin;   // more than twice the bound: both values carry the error
    int cnt = 0;
    for (int k0 = 0; k0 < K; k0 += 64) {
      const int k = k0 + lane;
      cnt += __builtin_popcountll(__ballot(k < K && !(sh.fast[f][k < K ? k : 0] > thr)));
    }
    // 4-bit formats: one whose shortlist is one candidate with a provably accurate error is done; false for a zero
    // or non-finite error.  An 8-bit format's error is some 1e-4 of what its filter cancels, four digits of the
    // reported error, so its winner is scored element by element too (a pass of 10 instructions per element beside
    // the 13 per look-up and boundary).
    const bool direct = Codec<FA>::BITS == 4 && cnt == 1 && fb.beta <= 0x1p-34 * m;
    if (lane == 0) { sh.thr[f] = thr; sh.direct[f] = direct ? km : -1; }
  }
  if (tid == 0) sh.nlist = 0;
  __syncthreads();
#pragma unroll
  for (int f = 0; f < NF; ++f)
    if (sh.direct[f] < 0)   // uniform
      for (int k = tid; k < K; k += THREADS)
        if (!(sh.fast[f][k] > sh.thr[f])) sh.list[atomicAdd(&sh.nlist, 1)] = static_cast<uint8_t>(f * MOFQ_MAX_CLIP + k);   // any order
  __syncthreads();
  const int n_list = sh.nlist;

  // exact fp64 re-score of the shortlist, element by element
  uint32_t carry = 0;
  // An 8-bit search nearly always has its two winners here: both formats from one read of the row
  const bool both = Codec<FA>::BITS == 8 && NF == 2 && n_list == 2 && sh.list[0] / MOFQ_MAX_CLIP != sh.list[1] / MOFQ_MAX_CLIP;   // uniform
  if (both) {
    const int first = sh.list[0] / MOFQ_MAX_CLIP;   // place of format 0 in the list
    const float s0 = sh.scale[0][sh.list[first] % MOFQ_MAX_CLIP], s1 = sh.scale[NF - 1][sh.list[1 - first] % MOFQ_MAX_CLIP];
    const float i0 = 1.0f / s0, i1 = 1.0f / s1;
    const double d0 = static_cast<double>(s0), d1 = static_cast<double>(s1);
    double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int c = (j * THREADS + tid) * 8;
      Raw8<In> raw;
      raw.clear();                   // padding is zero and scores zero
      if (c < n) raw.load(src, 0, static_cast<uint32_t>(c));
      float v[8];
      raw.widen(v);
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        score2_f64<FA>(acc0, v[i], v[i + 1], i0, d0, carry);
        score2_f64<FBX>(acc1, v[i], v[i + 1], i1, d1, carry);
      }
    }
    acc0 = wave_sum(acc0);
    acc1 = wave_sum(acc1);
    if (lane == 0) { sh.p2[wave] = acc0; sh.p2b[wave] = acc1; }
    __syncthreads();
    if (tid < 2) {
      const double* const p = tid == first ? sh.p2 : sh.p2b;
      double t = p[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += p[w];
      s_val[tid] = t;
    }
    __syncthreads();
  }
  for (int e = both ? n_list : 0; e < n_list; ++e) {
    const int fk = sh.list[e];
    const int f = __builtin_amdgcn_readfirstlane(fk / MOFQ_MAX_CLIP);
    const int k = __builtin_amdgcn_readfirstlane(fk % MOFQ_MAX_CLIP);
    const float s = sh.scale[f][k], inv = 1.0f / s;
    const double sd = static_cast<double>(s);
    double acc = 0.0;
    auto score = [&](auto fmt_c) {
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        const int c = (j * THREADS + tid) * 8;
        Raw8<In> raw;
        raw.clear();                   // padding is zero and scores zero
        if (c < n) raw.load(src, 0, static_cast<uint32_t>(c));
        float v[8];
        raw.widen(v);
#pragma unroll
        for (int i = 0; i < 8; i += 2) score2_f64<decltype(fmt_c)::value>(acc, v[i], v[i + 1], inv, sd, carry);
      }
    };
    if (f == 0) score(std::integral_constant<int, FA>{});
    else score(std::integral_constant<int, FBX>{});
    acc = wave_sum(acc);
    if (lane == 0) sh.p2[wave] = acc;
    __syncthreads();
    if (tid == 0) {
      double t = sh.p2[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += sh.p2[w];
      s_val[e] = t;
    }
    __syncthreads();
  }

  if (tid < NF) {
    const int f = tid;
    double best = __builtin_inf();
    int bk = sh.direct[f];
    if (bk >= 0) best = sh.fast[f][bk];
    for (int e = 0; e < n_list; ++e) {   // smallest error, then smallest index: the first smallest
      const int fk = sh.list[e];
      if (fk / MOFQ_MAX_CLIP != f) continue;
      const int k = fk % MOFQ_MAX_CLIP;
      if (s_val[e] < best || (s_val[e] == best && k < bk)) { best = s_val[e]; bk = k; }
    }
    if (bk < 0) { bk = 0; best = __builtin_nan(""); }   // only on non-finite input
    rec.scale[f][row] = sh.scale[f][bk];
    rec.clip[f][row] = bk;
    rec.err[f][row] = best;
    if (f == 0 && rec.energy) rec.energy[row] = en;
    sh.best[f] = best;
    sh.best_scale[f] = sh.scale[f][bk];
  }
}

// The row's codes (AheadCodes) after finish_row, in the format that the tensor's rows favour so far.
// `tally`: what tally_read gave the last wave.  Rows of up to kKeptChunks chunks a thread stay in its registers (`kept`) from
// the first pass on; longer ones are read again, from L2.
constexpr int kKeptChunks = 3;
template <typename In, int FA, int FB, int THREADS, int CH>
MOFQ_DEV void emit_row_ahead(RowSearch<(FB >= 0 ? 2 : 1), THREADS / 64>& sh, const AheadCodes& ahead, double tally, const Raw8<In> (&kept)[CH],
                             const uint16_t* src, int n, int64_t row) {
  constexpr int NF = (FB >= 0) ? 2 : 1, FBX = (FB >= 0) ? FB : FA, NW = THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (NF == 2 && wave == NW - 1) {
    if (ahead.tally) tally = wave_sum(tally);   // uniform
    if (lane == 0) sh.tally = tally;
  }
  Raw8<In> raw[CH];
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int c = (j * THREADS + tid) * 8;
    if constexpr (Codec<FA>::BITS == 4 && CH <= kKeptChunks) {
      raw[j] = kept[j];
      raw[j].opaque();   // nothing widened from it is kept
    } else {
      raw[j].load(src, 0, static_cast<uint32_t>(c < n ? c : 0));
    }
  }
  __syncthreads();
  int slot = 0;
  if constexpr (NF == 2) {
    const double d = sh.best[0] - sh.best[1];
    slot = __builtin_amdgcn_readfirstlane(sh.tally + d > 0.0 ? 1 : 0);
    if (tid == 0) {
      if (ahead.tally) tally_add<4>(ahead, d);
      ahead.tag[row] = static_cast<uint8_t>(ahead.cand_of[slot]);
    }
  }
  const float inv = 1.0f / sh.best_scale[slot];
  const int64_t row_chunks = row * (n / 8);
  auto emit = [&](auto fmt_c) {
    constexpr int FMT = decltype(fmt_c)::value;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int c = j * THREADS + tid;
      float t[8];
      raw[j].scaled(inv, t);
      uint32_t words[2];
      encode_scaled8<FMT>(t, words);
      if (c * 8 < n) {
        if constexpr (Codec<FMT>::BITS == 4) {
          (static_cast<uint32_t*>(ahead.codes) + row_chunks)[c] = words[0];
        } else {
          u32x2 o;
          o[0] = words[0];
          o[1] = words[1];
          (static_cast<u32x2*>(ahead.codes) + row_chunks)[c] = o;
        }
      }
    }
  };
  if (slot == 0) emit(std::integral_constant<int, FA>{});
  else emit(std::integral_constant<int, FBX>{});
}

}  // namespace

}  // namespace mofq
