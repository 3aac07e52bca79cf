// Group-wise scale search for the 4-bit formats on 16-bit weights: Algorithm 1's quantize_layer +
// compute_error with the tensor-error metric (Section 4.1) per group of consecutive elements (Section 5),
// over a table of clip ratios.  The formulation is that of the per-channel searches (mofq_sweep_sorted.hip):
// the error of a candidate follows from the number and the sum of magnitudes of the elements below each of its
// 7 level boundaries (INT4: 8), and the decision is monotone in the magnitude's bit pattern.  Scoring a group
// of 128 directly (sweep_group_kernel) costs 9.6 vector instructions per element and candidate for the format
// pair, 960 wave instructions per group with 50 ratios plus a second pass in fp64; a look-up costs 16,
// whatever the group's size.
//
// One wave takes 64 / LPG groups, LPG = GROUP / 8 lanes each, and shares nothing with other waves:
//   1. a bit per pattern that occurs, over the patterns between the smallest threshold of any candidate and
//      the group's largest magnitude (fp16: about 5700 bits, bf16: 720), 32 to an LDS word, beside each word the number
//      of distinct patterns before it;
//   2. per distinct pattern the count and the sum of magnitudes (integers, in ulps of the first pattern) of its
//      elements, and of its negative elements for INT4's extra level; prefix sums of both.  Count and
//      sum share a word of 32 bits where they fit (those of the negative elements in the upper half of 64), else 64;
//   3. a lane per candidate: the largest pattern below each boundary (an fp32 estimate and one exact decision), its
//      rank among the distinct patterns (a population count), count and sum up to it: two LDS reads; long tables that
//      descend are searched coarsely first, then the gaps that can hold the winner;
//   4. the smallest error and, for the winner alone, the sum of its residuals element by element: that sum is what
//      leaves (the difference of sums keeps two digits fewer).  Where a second candidate is too close, or a scale is
//      out of range (non-finite or nearly exact groups), all candidates of the group are scored that way, in fp64.
//
// Bound by vector issue and latency together: 1356 instructions per wave of four groups of 128 with 50 ratios take 77 % of
// the clocks (130 of them the winners' own sums; the direct kernel: 4360); 11 KB of LDS leave 3.5 waves per SIMD, so
// registers are spent on look-ups in flight (with a scheduler that kept to 63 registers for 8 waves per SIMD the same
// instructions took 1425 us instead of 1230).  Measured, layer selection of the seven linears of a
// 7B block, fp16 groups of 128, 50 ratios: 3003 us (direct) -> 1434 -> 1230 (every candidate looked up) -> 1143 us (the gaps
// searched).  A wave that walks several tiles with the next one's elements requested ahead: 1413 (its share is fixed).
#include <algorithm>
#include <cmath>

#include "mofq_search_common.h"

namespace mofq {

namespace {

struct GroupArgs {
  const void* w;
  int64_t cols, ld, units;
  int32_t scale_f16, n_clip;
  int32_t nbin;                // patterns with a bit, a multiple of 32
  int32_t descending;          // the ratios: none larger than the one before
  UnitRecords rec;
  float clip[MOFQ_MAX_CLIP];
};

// Level magnitudes m_0 .. m_7 (INT4: and 8 on the negative side), decision thresholds as in fill_levels
constexpr float below(float x) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) - 1u); }   // x > 0
template <int FMT> struct Levels {
  static constexpr int N = FMT == MOFQ_INT4 ? 8 : 7;   // boundaries
  static constexpr float mag(int b) {
    constexpr float e2m1[8] = {0.0f, 0.5f, 1.0f, 1.5f, 2.0f, 3.0f, 4.0f, 6.0f};
    return FMT == MOFQ_INT4 ? static_cast<float>(b) : e2m1[b < 8 ? b : 7];
  }
  static constexpr float thr(int b) {   // ties to the even code
    const float mid = 0.5f * (mag(b) + mag(b + 1));
    return b % 2 == 1 ? below(mid) : mid;
  }
  static constexpr float over(int b) { return static_cast<float>(thr(b) * (1.0 + 0x1p-21)); }
  static constexpr uint32_t step2(int b) { return static_cast<uint32_t>(2.0f * (mag(b + 1) - mag(b))); }   // an integer
  static constexpr uint32_t dg2q(int b) { return static_cast<uint32_t>(4.0f * (mag(b + 1) * mag(b + 1) - mag(b) * mag(b))); }
  static constexpr float kBelow = 1.0f / (over(6) * (1.0f + 0x1p-20f));    // a scale of amax times this: boundary 6 is below amax
  static constexpr float kAbove = (1.0f + 0x1p-20f) / over(0);             // of v times this: boundary 0 is not below v
  // a lane's own boundary, the same numbers: byte tables of 4 (m_q + m_{q+1}) / 2 and of the weights (E2M1 has no
  // eighth boundary: no weight)
  MOFQ_DEV static float thr_of(uint32_t q) {
    const float mid = FMT == MOFQ_INT4 ? static_cast<float>(q) + 0.5f : 0.25f * static_cast<float>(static_cast<uint32_t>(0x14140E0A07050301ull >> (8 * q)) & 0xFFu);
    return u2f(f2u(mid) - (q & 1u));
  }
  MOFQ_DEV static uint32_t step2_of(uint32_t q) { return FMT == MOFQ_INT4 ? 2u : static_cast<uint32_t>(0x0004020201010101ull >> (8 * q)) & 0xFFu; }
  MOFQ_DEV static uint32_t dg2q_of(uint32_t q) { return FMT == MOFQ_INT4 ? 8 * q + 4 : static_cast<uint32_t>(0x00501C1407050301ull >> (8 * q)) & 0xFFu; }
};

// count << B | sum
template <bool WIDE> struct Cell {
  using word = uint32_t;
  static constexpr int B = 24;
  MOFQ_DEV static uint32_t sum(word w) { return w & 0xFFFFFFu; }
  MOFQ_DEV static int count(word w) { return static_cast<int>(w >> 24); }
};
template <> struct Cell<true> {
  using word = uint64_t;
  static constexpr int B = 48;
  MOFQ_DEV static uint64_t sum(word w) { return w & 0xFFFFFFFFFFFFull; }
  MOFQ_DEV static int count(word w) { return static_cast<int>(w >> 48); }
};

// what a lane of the wave wrote to LDS is there for the others: LDS operations of a wave are in order
MOFQ_DEV void wave_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

template <typename T> MOFQ_DEV uint32_t lds_address(T* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) T*)p));
}

// over the LPG adjacent lanes of a group (8, 16 or 32)
template <int LPG, typename T, typename Op> MOFQ_DEV T group_reduce(T v, Op op) {
  auto dpp = [](T x, auto ctrl_c) {
    constexpr int CTRL = decltype(ctrl_c)::value;
    if constexpr (sizeof(T) == 8) return dpp_f64<CTRL>(x);
    else if constexpr (std::is_same<T, float>::value) return dpp_f32<CTRL>(x);
    else return static_cast<T>(dpp_i32<CTRL>(static_cast<int>(x)));
  };
  v = op(v, dpp(v, std::integral_constant<int, DPP_QUAD_XOR1>{}));
  v = op(v, dpp(v, std::integral_constant<int, DPP_QUAD_XOR2>{}));
  v = op(v, dpp(v, std::integral_constant<int, DPP_ROW_HALF_MIRROR>{}));
  if constexpr (LPG >= 16) v = op(v, dpp(v, std::integral_constant<int, DPP_ROW_MIRROR>{}));
  if constexpr (LPG >= 32) v = op(v, __shfl_xor(v, 16, 64));
  return v;
}
// of the next lane (0 behind the last)
MOFQ_DEV float next_lane(float x) { return u2f(static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(f2u(x)), 0x130, 0xf, 0xf, false))); }   // wave_shl:1
// sum over N adjacent lanes (2, 4 or 8)
template <int N, typename T> MOFQ_DEV T lanes_sum(T v) {
  auto from = [](T x, auto ctrl_c) {
    constexpr int CTRL = decltype(ctrl_c)::value;
    auto half = [](uint32_t h) { return static_cast<uint32_t>(dpp_i32<CTRL>(static_cast<int>(h))); };
    if constexpr (sizeof(T) == 8) return (static_cast<T>(half(static_cast<uint32_t>(x >> 32))) << 32) | half(static_cast<uint32_t>(x));
    else return half(x);
  };
  v += from(v, std::integral_constant<int, DPP_QUAD_XOR1>{});
  if constexpr (N >= 4) v += from(v, std::integral_constant<int, DPP_QUAD_XOR2>{});
  if constexpr (N >= 8) v += from(v, std::integral_constant<int, DPP_ROW_HALF_MIRROR>{});
  return v;
}
// x of the lane that control CTRL names, 0 where there is none or ROW_MASK leaves the row out
template <int CTRL, int ROW_MASK, typename T> MOFQ_DEV T dpp_or_zero(T x) {
  auto half = [](uint32_t v) { return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROW_MASK, 0xf, false)); };
  if constexpr (sizeof(T) == 4) return static_cast<T>(half(static_cast<uint32_t>(x)));
  else return static_cast<T>(half(static_cast<uint32_t>(x))) | (static_cast<T>(half(static_cast<uint32_t>(static_cast<uint64_t>(x) >> 32))) << 32);
}
// exclusive prefix over the group's lanes
template <int LPG, typename T> MOFQ_DEV T group_excl(T v, int l) {
  T inc = v;
  auto step = [&](auto ctrl_c, int d) {   // row_shr: inside rows of 16 lanes
    const T o = dpp_or_zero<decltype(ctrl_c)::value, 0xf>(inc);
    inc += (LPG >= 16 || l >= d) ? o : 0;
  };
  step(std::integral_constant<int, 0x111>{}, 1);
  step(std::integral_constant<int, 0x112>{}, 2);
  step(std::integral_constant<int, 0x114>{}, 4);
  if constexpr (LPG >= 16) step(std::integral_constant<int, 0x118>{}, 8);
  if constexpr (LPG >= 32) inc += dpp_or_zero<0x142, 0xa>(inc);   // row_bcast:15 into rows 1 and 3
  return inc - v;
}

// LDS of a wave: bit words and ranks of each group, then of each group the words of the distinct patterns: one array with
// both halves (narrow with INT4), or an array each.  The lanes of a group look at neighbouring candidates and read
// neighbouring places, about the same ones in every group, so the groups' arrays begin in different banks: the tables
// 256 / GPW bytes apart modulo 256 (an odd number of entries per lane), and so the words.
template <int GROUP, bool WIDE, bool TAIL> struct GroupLayout {
  static constexpr int LPG = GROUP / 8, GPW = 64 / LPG;
  static constexpr bool JOINED = TAIL && !WIDE;
  using store = std::conditional_t<WIDE || JOINED, uint64_t, uint32_t>;
  static constexpr int STRIDE = sizeof(store);
  static constexpr int SHIFT = 256 / GPW;
  static constexpr int CELLS = (STRIDE * (GROUP + 1) - SHIFT + 255) / 256 * 256 + SHIFT;   // GROUP + 1 of them are used
  static constexpr int entries(int nbin) { return ((nbin / 32 + 1 + LPG - 1) / LPG) | 1; }   // per lane; odd: lanes' pieces in different banks
  static constexpr int table(int nbin) { return entries(nbin) * LPG * 8; }
  static constexpr int bytes(int nbin) { return GPW * (table(nbin) + CELLS * (TAIL && !JOINED ? 2 : 1)); }   // pieces of 16
  // behind them: the clip ratios, and per format and group the candidates to look at in the gaps
  static constexpr bool gaps(int K) { return K > 2 * LPG; }
  static constexpr int lists(int K, int nf) { return gaps(K) ? nf * GPW * (K - LPG) : 0; }
  static constexpr int all_bytes(int nbin, int K, int nf) { return bytes(nbin) + 4 * K + lists(K, nf); }
};

// Waves per SIMD that the registers are shared out for.  LDS leaves 3.5 (fp16, groups of 128, 50 ratios): what registers
// are free then hold look-ups in flight.  bf16 has an eighth of the bits and room for more waves: 4096 x 4096, groups
// of 128, 50 ratios 95.6 us with 4, 92.0 with 5, 89.8 with 6, 91.4 with 8 (before the gaps were searched, with 8: 107.8);
// with 64-bit words 4: groups of 256 111 us, with 6 115.
template <typename In, bool WIDE> constexpr int kWaves = std::is_same<In, BF16>::value && !WIDE ? 6 : 4;

template <typename In, int FA, int FB, int GROUP, bool WIDE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<In, WIDE>, kWaves<In, WIDE>))) void sweep_group_bits_kernel(const GroupArgs a) {
  constexpr int NF = (FB >= 0) ? 2 : 1;
  constexpr int FBX = (FB >= 0) ? FB : FA;
  constexpr int LPG = GROUP / 8, GPW = 64 / LPG;
  constexpr bool TAIL = FA == MOFQ_INT4 || FBX == MOFQ_INT4;
  using Lay = GroupLayout<GROUP, WIDE, TAIL>;
  using C = Cell<WIDE>;
  using word = typename C::word;
  typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
  typedef __attribute__((address_space(3))) word lds_word;

  extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
  const int K = a.n_clip, nbin = a.nbin;
  const int lane = threadIdx.x, l = lane % LPG, g = lane / LPG;
  const int epl = Lay::entries(nbin);
  u32x2* const tbl = reinterpret_cast<u32x2*>(s_dyn + g * Lay::table(nbin));           // bits, distinct patterns before them
  using store = typename Lay::store;
  store* const P = reinterpret_cast<store*>(s_dyn + GPW * Lay::table(nbin) + g * Lay::CELLS);
  store* const PN = P + GPW * Lay::CELLS / Lay::STRIDE;   // not where they are joined
  float* const s_clip = reinterpret_cast<float*>(s_dyn + Lay::bytes(nbin));
  uint8_t* const list = reinterpret_cast<uint8_t*>(s_clip + K) + g * (K - LPG);   // of format 0; format 1: GPW (K - LPG) further

  const int64_t gpr = a.cols / GROUP;   // groups per row
  int64_t unit = static_cast<int64_t>(blockIdx.x) * GPW + g;
  const bool valid = unit < a.units;
  if (!valid) unit = a.units - 1;
  int64_t at0 = unit * GROUP;
  if (a.ld != a.cols) {   // uniform
    const int64_t row = unit / gpr;
    at0 = row * a.ld + (unit - row * gpr) * GROUP;
  }
  const uint16_t* const src = static_cast<const uint16_t*>(a.w) + at0 + l * 8;
  const bool f16 = a.scale_f16 != 0;

  Raw8<In> raw;
  raw.load(src, 0, 0);
  for (int k = lane; k < K; k += 64) s_clip[k] = a.clip[k];
  {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int i = lane; i < Lay::bytes(nbin) / 16; i += 64) reinterpret_cast<u32x4*>(s_dyn)[i] = zero;
  }
  float x[8], amax = 0.0f;
  raw.widen(x);
  double en = 0.0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[i] = __builtin_fabsf(x[i]);
    amax = __builtin_fmaxf(amax, x[i]);
    const double xd = static_cast<double>(x[i]);
    en = __builtin_fma(xd, xd, en);
  }
  amax = group_reduce<LPG>(amax, [](float p, float q) { return __builtin_fmaxf(p, q); });
  en = group_reduce<LPG>(en, [](double p, double q) { return p + q; });
  // the counted patterns; whatever lies below them is on level 0 for every candidate
  const int hmax = static_cast<int>(pattern_rtz<In>(__builtin_fminf(amax, 3.4028234e38f)));
  const int lo = (hmax + 1 - nbin) > 0 ? hmax + 1 - nbin : 0;

  // ---- 1. bits ----------------------------------------------------------------------------------------
  wave_fence();
  const uint32_t tbl_at = lds_address(tbl), p_at = lds_address(P), pn_at = Lay::JOINED ? p_at + 4 : lds_address(PN);
  auto entry_at = [&](uint32_t n) {   // of pattern number n
    uint32_t e = n >> 5;
    asm("" : "+v"(e));   // a shift-and-add
    return (e << 3) + tbl_at;
  };
  // (no branches around the LDS operations of the elements below the counted patterns: these set and add nothing)
  // Pattern numbers of two elements at once, 0 .. nbin - 1 (a non-finite element gets the last: the group's error is
  // non-finite anyway), and 1 for the counted ones.
  uint32_t at2[4], in2[4], at[8];   // at: LDS address of the entry
  const i16x2 lo2 = {static_cast<short>(lo), static_cast<short>(lo)}, last2 = {static_cast<short>(nbin - 1), static_cast<short>(nbin - 1)}, zero2 = {0, 0};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const i16x2 n2 = __builtin_elementwise_min(__builtin_bit_cast(i16x2, raw.w[j] & 0x7FFF7FFFu) - lo2, last2);
    at2[j] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(n2, zero2));
    in2[j] = (~__builtin_bit_cast(uint32_t, n2) >> 15) & 0x00010001u;
    asm("" : "+v"(at2[j]), "+v"(in2[j]));   // opaque: the halves are taken by the instructions that use them
    uint32_t e0 = __builtin_amdgcn_ubfe(at2[j], 5u, 11u), e1 = at2[j] >> 21;
    asm("" : "+v"(e0), "+v"(e1));
    at[2 * j] = (e0 << 3) + tbl_at;
    at[2 * j + 1] = (e1 << 3) + tbl_at;
    __hip_atomic_fetch_or((lds_u32*)static_cast<uintptr_t>(at[2 * j]), (in2[j] & 0xFFFFu) << (at2[j] & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or((lds_u32*)static_cast<uintptr_t>(at[2 * j + 1]), (in2[j] >> 16) << ((at2[j] >> 16) & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  wave_fence();
  {
    uint32_t n = 0;
    for (int e = 0; e < epl; ++e) n += __builtin_popcount(tbl[l * epl + e][0]);
    uint32_t base = group_excl<LPG>(n, l);
    for (int e = 0; e < epl; ++e) {
      const uint32_t bits = tbl[l * epl + e][0];
      tbl[l * epl + e][1] = base;
      base += __builtin_popcount(bits);
    }
  }
  wave_fence();
  // distinct patterns among the first n 
  auto rank_at = [&](uint32_t at, uint32_t n) {
    uint32_t r;
    const u32x2 t = *(lds_u32x2*)static_cast<uintptr_t>(at);
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(__builtin_amdgcn_ubfe(t[0], 0u, n)), "v"(t[1]));   // (the width's low 5 bits count)
    return r;
  };
  auto rank = [&](uint32_t n) { return rank_at(entry_at(n), n); };
  auto cell = [](uint32_t at, uint32_t r) { return *(lds_word*)static_cast<uintptr_t>(at + r * Lay::STRIDE); };

  // ---- 2. count and sum per distinct pattern, prefixes -----------------------------------------------
  constexpr int kUlp = std::is_same<In, F16>::value ? 25 : 134;   // exponent field of the pattern whose ulp is 1
  const int e_lo = exponent_of<In>(lo);
  uint32_t d[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) d[i] = rank_at(at[i], i % 2 == 0 ? at2[i / 2] : at2[i / 2] >> 16);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bool counted = (in2[i / 2] & (i % 2 == 0 ? 1u : 0x10000u)) != 0;
    const word one = counted ? (static_cast<word>(1) << C::B) + static_cast<word>(static_cast<uint32_t>(__builtin_ldexpf(x[i], kUlp - e_lo))) : 0;
    const store neg = (raw.w[i / 2] & (i % 2 == 0 ? 0x8000u : 0x80000000u)) != 0 ? static_cast<store>(one) : 0;
    if constexpr (Lay::JOINED) {
      __hip_atomic_fetch_add(P + d[i], one | (neg << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
      __hip_atomic_fetch_add(P + d[i], one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if constexpr (TAIL) __hip_atomic_fetch_add(PN + d[i], neg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  wave_fence();
  auto prefix = [&](store* cells) {   // (no carry from one half to the other)
    store v[8], sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = cells[l * 8 + i];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const store c = v[i];
      v[i] = sum;
      sum += c;
    }
    const store base = group_excl<LPG>(sum, l);
#pragma unroll
    for (int i = 0; i < 8; ++i) cells[l * 8 + i] = base + v[i];
    if (l == LPG - 1) cells[GROUP] = base + sum;
  };
  prefix(P);
  if constexpr (TAIL && !Lay::JOINED) prefix(PN);
  wave_fence();
  const word total = cell(p_at, GROUP);
  const word n_total = TAIL ? cell(pn_at, GROUP) : 0;
  const float v_lo = bits_to_float<In>(static_cast<uint32_t>(lo));
  const double four_ulp = 4.0 * static_cast<double>(bits_to_float<In>(static_cast<uint32_t>(lo) + 1) - v_lo);   // ulps at lo
  const double en4 = 4.0 * en;

  // ---- 3. candidates -----------------------------------------------------------------------------
  double best[NF], second[NF];
  bool bad = !(amax <= 0x1p127f);   // the group has to be scored exactly (here: scales may leave the reciprocal's range)
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    best[f] = second[f] = __builtin_inf();
  }
  int before_lo = -lo;
  asm("" : "+v"(before_lo));   // opaque: pattern, this and the carry of the decision are one addition
  const float v_max = bits_to_float<In>(static_cast<uint32_t>(hmax));
  // What the search of the gaps needs of the lane's candidate: 4 (error), 4 (sum of squared levels), scale.
  struct Coarse {
    double v;
    float b4, s;
  } coarse[NF];
  // Candidate k (any valid number where there is none, !in), PER adjacent lanes to each, which share its boundaries.
  auto candidate = [&](auto fmt_c, auto per_c, int k, bool in, int f) {
    constexpr int FMT = decltype(fmt_c)::value, PER = decltype(per_c)::value;
    using Lv = Levels<FMT>;
    const float s0 = search_scale<FMT>(s_clip[k] * amax, f16);   // (a non-finite group comes out as 1 and is scored exactly later)
    // No boundary but the eighth beyond the counted patterns: a scale that rounding to fp16 moved so far sends the group
    // to the exact pass.  (The patterns span more than the boundaries do, so the lower limit is the smaller one.)
    const float s = med3(s0, v_lo * Lv::kAbove, v_max * Lv::kBelow);
    bad |= s != s0;
    const float inv = reciprocal(s);   // (a group with a larger scale than that takes is scored exactly, with the division)
    // The largest pattern at or below the boundary (threshold t s): the pattern of t s (1 + 2^-21) rounded toward
    // zero or the one before it, as the exact decision on the first tells; patterns above are beyond t s (1 + 2^-22), those
    // below short of t s (1 - 2^-22), whatever the rounding of 1 / s and of the product.
    auto distinct = [&](float over, float thr, bool last) {
      const uint32_t e = pattern_rtz<In>(over * s);
      const bool at_most = scaled<In>(e, inv) <= thr;
      uint32_t n = e + static_cast<uint32_t>(before_lo) + (at_most ? 1u : 0u);
      if (last) n = min(n, static_cast<uint32_t>(nbin));
      return rank(n);
    };
    // Sums in half levels and 4 times the sum of squares, less those of all elements on level 7 (INT4: all its
    // negative ones on -8, one level further): what is missing below the boundaries.
    word A = -static_cast<word>(2.0f * Lv::mag(7)) * C::sum(total);
    uint32_t b4 = -static_cast<uint32_t>(4.0f * Lv::mag(7) * Lv::mag(7)) * static_cast<uint32_t>(C::count(total));
    if constexpr (FMT == MOFQ_INT4) {
      A -= 2 * C::sum(n_total);
      b4 -= 60u * static_cast<uint32_t>(C::count(n_total));
    }
    if constexpr (PER > 1)   // once
      if (l % PER != 0) { A = 0; b4 = 0; }
    auto add = [&](word p, uint32_t step2, uint32_t dg2q) {
      if constexpr (WIDE) {
        A += C::sum(p) * step2;
        b4 += __umul24(static_cast<uint32_t>(C::count(p)), dg2q);
      } else {
        A += __umul24(p, step2);   // the low 24 bits
        b4 = __builtin_amdgcn_udot4(p, dg2q << 24, b4, false);
      }
    };
    if constexpr (PER == 1) {
      uint32_t r[Lv::N];
#pragma unroll
      for (int q = 0; q < Lv::N; ++q) r[q] = distinct(Lv::over(q), Lv::thr(q), q == 7);
#pragma unroll
      for (int q = 0; q < Lv::N; ++q) {
        const word p = cell(q == 7 ? pn_at : p_at, r[q]);
        if constexpr (WIDE) add(p, Lv::step2(q), Lv::dg2q(q));
        else {
          asm("v_mad_u32_u24 %0, %1, %2, %0" : "+v"(A) : "v"(p), "n"(Lv::step2(q)));   // the low 24 bits
          b4 = __builtin_amdgcn_udot4(p, Lv::dg2q(q) << 24, b4, false);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8 / PER; ++i) {
        const uint32_t q = static_cast<uint32_t>(l % PER + i * PER);
        const float thr = Lv::thr_of(q);
        const uint32_t r = distinct(thr * (1.0f + 0x1p-21f), thr, FMT == MOFQ_INT4 && i == 8 / PER - 1);
        const word p = cell(FMT == MOFQ_INT4 && i == 8 / PER - 1 && q == 7 ? pn_at : p_at, r);
        add(p, Lv::step2_of(q), Lv::dg2q_of(q));
      }
      A = lanes_sum<PER>(A);
      b4 = lanes_sum<PER>(b4);
    }
    // 4 (error): exact scaling
    const double sd = static_cast<double>(s);
    const double Ad = static_cast<double>(static_cast<std::make_signed_t<word>>(A)), bd = static_cast<double>(static_cast<int>(b4));
    // the candidate rides in the lowest bits: 2^-45 of the error, far below the margin
    const double v0 = __builtin_fma(sd, __builtin_fma(-sd, bd, Ad * four_ulp), en4);
    const double v = __builtin_bit_cast(double, (__builtin_bit_cast(uint64_t, v0) & ~uint64_t{127}) | static_cast<uint32_t>(k));
    if (in) {
      second[f] = __builtin_fmin(second[f], __builtin_fmax(v, best[f]));
      best[f] = __builtin_fmin(best[f], v);
    }
    coarse[f] = Coarse{v, -static_cast<float>(bd), s};
  };
  auto both = [&](auto what) {
    what(std::integral_constant<int, FA>{}, 0);
    if constexpr (NF == 2) what(std::integral_constant<int, FBX>{}, NF - 1);
  };
  using one_lane = std::integral_constant<int, 1>;
  const double margin = 4.0 * filter_bounds<GROUP, true, 4>(en, 0.0, 0.0, 0.0, 0.0).margin;
  if (Lay::gaps(K) && a.descending) {   // uniform
    // LPG candidates over the whole table first, then the ones in the gaps that can be the winner.  The error of a scale
    // s is the smallest of |x - s g|^2 over all assignments g of levels, so in a gap s2 < s < s1 it lies above some
    // parabola of curvature |g|^2 <= B, B that at s2 (a smaller scale, larger levels), which at s1 and s2 is not below the errors E1
    // and E2 there.  The smallest value of such a parabola is below T only if sqrt(E1 - T) + sqrt(E2 - T) < sqrt(B) (s1 - s2).
    // T: the smallest error so far, twice the filter's margin, and 2^-18 of the energy: a decision on rounded
    // numbers assigns an element within 2^-22 of a boundary to the level beyond it, which adds up to 4 x^2 2^-22 to the
    // error (and takes such elements' levels out of B where the gap is that small).  The rest is rounded in favour of
    // looking.  On LLaMA-like groups of 128 with 50 ratios 4 and 3 of the 34 candidates in the gaps are left.
    auto place = [&](int i) { return static_cast<int>(static_cast<uint32_t>(i * (K - 1)) / static_cast<uint32_t>(LPG - 1)); };
    const int mine = place(l), next = place(l + 1);
    both([&](auto fmt_c, int f) { candidate(fmt_c, one_lane{}, mine, true, f); });
    uint32_t left[NF];
    const int gap = (K - 1 + LPG - 2) / (LPG - 1) - 1;   // the most candidates in one
    // bf16: magnitudes whose squares leave fp32 are scaled by a power of two
    const int e = std::is_same<In, F16>::value ? 0 : -__builtin_amdgcn_frexp_expf(amax);
    both([&](auto, int f) {
      const Coarse& c = coarse[f];
      const double m = group_reduce<LPG>(c.v, [](double p, double q) { return __builtin_fmin(p, q); });
      double above = c.v - (m + 2.0 * margin + 0x1p-18 * en4);
      float ds = c.s - next_lane(c.s);
      if constexpr (!std::is_same<In, F16>::value) {
        above = __builtin_amdgcn_ldexp(above, 2 * e);
        ds = __builtin_amdgcn_ldexpf(ds, e);
      }
      const float root = __builtin_amdgcn_sqrtf(__builtin_fmaxf(static_cast<float>(above), 0.0f));   // of 4 (E - T)
      // (the lanes' values are moved by all of them: one that is switched off has none for its neighbour)
      const float roots = root + next_lane(root), reach = __builtin_amdgcn_sqrtf(next_lane(c.b4)) * ds * (1.0f + 0x1p-12f);
      const bool look = l < LPG - 1 && !(roots > reach);
      const uint32_t n = look ? static_cast<uint32_t>(next - mine - 1) : 0u;
      const uint32_t first = group_excl<LPG>(n, l);
      left[f] = group_reduce<LPG>(n, [](uint32_t p, uint32_t q) { return p + q; });
      for (uint32_t j = 0; j < static_cast<uint32_t>(gap); ++j)
        if (j < n) list[f * GPW * (K - LPG) + first + j] = static_cast<uint8_t>(mine + 1 + j);
    });
    wave_fence();
    both([&](auto fmt_c, int f) {
      for (uint32_t i = 0; __builtin_amdgcn_ballot_w64(i < left[f]) != 0; i += LPG) {
        const bool in = i + l < left[f];
        candidate(fmt_c, one_lane{}, in ? list[f * GPW * (K - LPG) + i + l] : 0, in, f);
      }
    });
  } else {
    int k0 = 0;
    for (; k0 + LPG <= K; k0 += LPG) both([&](auto fmt_c, int f) { candidate(fmt_c, one_lane{}, k0 + l, true, f); });
    // The rest of them: several lanes to a candidate where there are enough (two candidates on 16 lanes take
    // 143 instructions instead of a round's 242).
    const int rest = K - k0;   // uniform
    auto shared = [&](auto per_c) {
      const int k = k0 + l / decltype(per_c)::value;
      both([&](auto fmt_c, int f) { candidate(fmt_c, per_c, min(k, K - 1), k < K, f); });
    };
    if (rest > 0) {
      if (rest * 8 <= LPG) shared(std::integral_constant<int, 8>{});
      else if (rest * 4 <= LPG) shared(std::integral_constant<int, 4>{});
      else if (rest * 2 <= LPG) shared(std::integral_constant<int, 2>{});
      else shared(one_lane{});
    }
  }

  // ---- 4. winners.  Count and sum are exact and the error takes two roundings (filter_bounds): a candidate that
  // is the smallest by more than the margin is the winner, and its own error is then summed element by element, for
  // en - 2 s A + s^2 B keeps two digits fewer than that sum. -------------------------------------------------
  const bool exact = group_reduce<LPG>(bad ? 1 : 0, [](int p, int q) { return p | q; }) != 0;
  int win[NF];
  bool sure[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    auto least = [](double p, double q) { return __builtin_fmin(p, q); };
    const double m = group_reduce<LPG>(best[f], least);
    win[f] = static_cast<int>(__builtin_bit_cast(uint64_t, m) & 127u);
    const double m2 = group_reduce<LPG>(best[f] == m ? second[f] : best[f], least);   // candidates of one lane are its own
    sure[f] = !exact && m2 > m + margin;   // false for a zero or non-finite error
  }
  raw.opaque();
  raw.widen(x);
  uint32_t carry = 0;
  auto residuals = [&](auto fmt_c, float s, float inv) {
    constexpr int FMT = decltype(fmt_c)::value;
    const double sd = static_cast<double>(s);
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 8; i += 2) score2_f64<FMT>(acc, x[i], x[i + 1], inv, sd, carry);
    return group_reduce<LPG>(acc, [](double p, double q) { return p + q; });
  };
  float s_win[NF];
  double err[NF];
  auto winner = [&](auto fmt_c, int f) {
    win[f] = win[f] < K ? win[f] : 0;   // none on non-finite input
    s_win[f] = unit_scale(amax, s_clip[win[f]], Codec<decltype(fmt_c)::value>::QMAX, f16);
    err[f] = residuals(fmt_c, s_win[f], reciprocal(s_win[f]));
  };
  winner(std::integral_constant<int, FA>{}, 0);
  if constexpr (NF == 2) winner(std::integral_constant<int, FBX>{}, NF - 1);
  auto finish = [&](auto fmt_c, int f) {
    if (__builtin_amdgcn_ballot_w64(!sure[f] && valid) != 0) {
      double eb = __builtin_inf();
      int ek = -1;
      for (int c = 0; c < K; ++c) {
        const float s = unit_scale(amax, s_clip[c], Codec<decltype(fmt_c)::value>::QMAX, f16);
        const double e = residuals(fmt_c, s, 1.0f / s);
        if (e < eb) { eb = e; ek = c; }
      }
      if (!sure[f]) {
        err[f] = ek < 0 ? __builtin_nan("") : eb;   // only on non-finite input
        win[f] = ek < 0 ? 0 : ek;
        s_win[f] = unit_scale(amax, s_clip[win[f]], Codec<decltype(fmt_c)::value>::QMAX, f16);
      }
    }
    if (valid && l == 0) {
      a.rec.scale[f][unit] = s_win[f];
      a.rec.clip[f][unit] = win[f];
      a.rec.err[f][unit] = err[f];
    }
  };
  finish(std::integral_constant<int, FA>{}, 0);
  if constexpr (NF == 2) finish(std::integral_constant<int, FBX>{}, NF - 1);
  if (valid && l == 0 && a.rec.energy) a.rec.energy[unit] = en;
}

template <typename In, int FA, int FB, int GROUP>
int launch_size(const GroupArgs& a, hipStream_t st) {
  constexpr int GPW = 64 / (GROUP / 8), MANT = Pattern<In>::MANT;
  constexpr bool TAIL = FA == MOFQ_INT4 || FB == MOFQ_INT4;
  // A magnitude is below 2^bits ulps of the first pattern: an integer of 32 bits, whose sum over a group of 256
  // fits the wide cell's 48; the narrow cell holds sums below 2^24 and counts below 2^8.  More binades than that are
  // the direct kernel's (bf16 from ratios below about 2e-6 on; an fp16 table ends at 8).
  const int bits = MANT + 1 + ((a.nbin + (1 << MANT) - 1) >> MANT);
  if (bits > 32) return MOFQ_ERR_UNSUPPORTED;
  const dim3 grid(static_cast<unsigned>((a.units + GPW - 1) / GPW));
  if (GROUP <= 128 && bits < 24 && ((GROUP - 1) >> (24 - bits)) == 0) {
    const size_t lds = static_cast<size_t>(GroupLayout<GROUP, false, TAIL>::all_bytes(a.nbin, a.n_clip, FB >= 0 ? 2 : 1));
    hipLaunchKernelGGL((sweep_group_bits_kernel<In, FA, FB, GROUP, false>), grid, dim3(64), lds, st, a);
  } else {
    const size_t lds = static_cast<size_t>(GroupLayout<GROUP, true, TAIL>::all_bytes(a.nbin, a.n_clip, FB >= 0 ? 2 : 1));
    hipLaunchKernelGGL((sweep_group_bits_kernel<In, FA, FB, GROUP, true>), grid, dim3(64), lds, st, a);
  }
  return hip_status(hipGetLastError());
}

template <typename In, int FA, int FB>
int launch_fmt(const SweepParams& p, const GroupArgs& a, hipStream_t st) {
  switch (p.group) {
    case 64: return launch_size<In, FA, FB, 64>(a, st);
    case 128: return launch_size<In, FA, FB, 128>(a, st);
    case 256: return launch_size<In, FA, FB, 256>(a, st);
  }
  return MOFQ_ERR_UNSUPPORTED;
}

template <typename In>
int launch_type(const SweepParams& p, const GroupArgs& a, hipStream_t st) {
  const int fa = p.fmt[0], fb = p.n_fmt == 2 ? p.fmt[1] : -1;
  if (fa == MOFQ_INT4 && fb == MOFQ_FP4_E2M1) return launch_fmt<In, MOFQ_INT4, MOFQ_FP4_E2M1>(p, a, st);
  if (fa == MOFQ_INT4 && fb == -1) return launch_fmt<In, MOFQ_INT4, -1>(p, a, st);
  if (fa == MOFQ_FP4_E2M1 && fb == -1) return launch_fmt<In, MOFQ_FP4_E2M1, -1>(p, a, st);
  return MOFQ_ERR_UNSUPPORTED;
}

// From how many clip ratios on this kernel is the faster one: building the table costs what scoring that many candidates
// costs (the direct kernel scores all of them up to 15 to 19, beyond by bisection). The pair shares one table and a format
// alone has it to itself; INT4's takes the negative elements' words as well (E2M1 alone needs neither them nor their
// prefixes); bf16 has an eighth of fp16's bits to clear and to walk; a group of 64 has a table of its own like any other;
// one of 256 takes 64-bit words. kNever: bisection is faster up to MOFQ_MAX_CLIP. Measured at the lines, layer selection,
// 4096 x 4096, type and group, ratios: us scored directly / by look-up: INT4 and E2M1: fp16 64, 56: 170.0 / 174.3, 64:
// 193.4 / 182.3; fp16 128, 12: 79.6 / 78.0; fp16 256, 22: 113.3 / 111.8; bf16 64, 10: 76.9 / 74.7; bf16 128, 9: 66.5 /
// 65.6; bf16 256, 18: 102.5 / 100.4. INT4: fp16 64, 128: 154.2 / 193.6; fp16 128, 27: 71.6 / 70.4; fp16 256, 128: 121.6 /
// 142.3; bf16 64, 18: 64.6 / 63.0; bf16 128, 18: 60.3 / 58.4; bf16 256, 56: 92.5 / 109.1, 128: 120.8 / 130.1. E2M1: fp16
// 64, 128: 144.4 / 170.0; fp16 128, 15: 57.5 / 56.6; fp16 256, 22: 65.2 / 63.1; bf16 64, 12: 53.3 / 52.7; bf16 128, 11:
// 47.8 / 46.7; bf16 256, 17: 58.6 / 58.2.
// Tensors of fewer than kFewElements: bisection's rounds wait for each other where few groups are resident, so there the
// lines are those to scoring all candidates (the pair, fp16 64, layer selection: 400 x 2048, 24: 22.3 / 22.2, 32: 25.6 / 20.7;
// 500 x 4096, 24: 29.7 / 29.7; 1000 x 4096, 32: 55.0 / 52.1; 2048 x 4096, 30: 75.4 / 88.5).
constexpr int kNever = MOFQ_MAX_CLIP + 1;
constexpr int64_t kFewElements = 6 << 20;
int min_clip(const SweepParams& p) {
  static constexpr int lines[2][2][3][3] = {   // [many, few elements][fp16, bf16][64, 128, 256][pair, INT4, E2M1]
      {{{60, kNever, kNever}, {12, 27, 15}, {22, kNever, 22}}, {{10, 17, 12}, {9, 18, 11}, {18, kNever, 17}}},
      {{{23, 48, 28}, {12, 25, 15}, {21, 39, 20}}, {{10, 19, 13}, {9, 19, 11}, {18, 37, 17}}}};
  const int which = p.n_fmt == 2 ? 0 : (p.fmt[0] == MOFQ_INT4 ? 1 : 2);
  return lines[p.rows * p.cols < kFewElements ? 1 : 0][p.dtype == MOFQ_F16 ? 0 : 1][p.group == 64 ? 0 : (p.group == 128 ? 1 : 2)][which];
}

}  // namespace

int launch_sweep_group_bits(const SweepParams& p, hipStream_t st) {
  if (p.gran != MOFQ_PER_GROUP || (p.dtype != MOFQ_F16 && p.dtype != MOFQ_BF16) || p.n_clip < min_clip(p)) return MOFQ_ERR_UNSUPPORTED;
  GroupArgs a{};
  a.w = p.w;
  a.cols = p.cols;
  a.ld = p.ld;
  a.units = mofq_num_units(p.rows, p.cols, p.gran, p.group);
  if (a.units <= 0) return MOFQ_ERR_INVALID_ARG;
  a.scale_f16 = p.scale_f16;
  a.n_clip = p.n_clip;
  a.rec = p.rec;
  float r_min = INFINITY;
  a.descending = 1;
  for (int k = 0; k < p.n_clip; ++k) {
    if (!(p.clip[k] > 0.0f) || !std::isfinite(p.clip[k])) return MOFQ_ERR_UNSUPPORTED;
    r_min = std::fmin(r_min, p.clip[k]);
    a.clip[k] = p.clip[k];
    if (k > 0 && p.clip[k] > p.clip[k - 1]) a.descending = 0;
  }
  const bool e2m1 = p.fmt[0] == MOFQ_FP4_E2M1 || (p.n_fmt == 2 && p.fmt[1] == MOFQ_FP4_E2M1);
  a.nbin = (hist_bins((e2m1 ? 24.0 : 14.0) / r_min, p.dtype == MOFQ_F16 ? 1024 : 128) + 31) / 32 * 32;
  if (a.nbin > 8192) return MOFQ_ERR_UNSUPPORTED;   // 2 KB of bits per group
  return p.dtype == MOFQ_F16 ? launch_type<F16>(p, a, st) : launch_type<BF16>(p, a, st);
}

}  // namespace mofq
