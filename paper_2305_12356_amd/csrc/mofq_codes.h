// Device helpers shared by the kernels that score and write codes: grid values and codes through the
// gfx950 pack-convert instructions, elements kept as they come from memory.
#pragma once
#include <type_traits>

#include "mofq_device.h"
#include "mofq_internal.h"

namespace mofq {

namespace {

// ---- grid value of a scaled element, two elements at a time ---------------------
//
// FP formats use the gfx950 pack-convert instructions (round to nearest even,
// subnormals, saturation); they agree with Codec<>::mag / code on every finite fp32
// bit pattern (checked exhaustively on the part), and cost about half the vector
// cycles of the add/subtract-constant form.
typedef float f32x2 __attribute__((ext_vector_type(2)));

// `carry` is the register the fp4 encode merges its byte into; its other bytes are
// never read, so it is simply handed from call to call (no clearing instruction).
template <int FMT> MOFQ_DEV f32x2 grid2(float t0, float t1, uint32_t& carry) {
  f32x2 g;
  if constexpr (FMT == MOFQ_FP4_E2M1) {
    carry = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(carry, t0, t1, 1.0f, 0);
    g = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(carry, 1.0f, 0);
  } else if constexpr (FMT == MOFQ_FP4_E2M1_IEEE) {
    // the same grid below 3: clamp, then the same convert
    carry = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(carry, med3(t0, -3.0f, 3.0f), med3(t1, -3.0f, 3.0f), 1.0f, 0);
    g = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(carry, 1.0f, 0);
  } else if constexpr (FMT == MOFQ_FP8_E4M3) {
    const int p = __builtin_amdgcn_cvt_pk_fp8_f32(med3(t0, -448.0f, 448.0f), med3(t1, -448.0f, 448.0f), 0, false);
    g = __builtin_amdgcn_cvt_pk_f32_fp8(p, false);
  } else {
    g[0] = Codec<FMT>::grid(t0);
    g[1] = Codec<FMT>::grid(t1);
  }
  return g;
}

// Squared error of two elements, the residual and its square in fp64.
template <int FMT> MOFQ_DEV void score2_f64(double& acc, float x0, float x1, float inv_s, double sd, uint32_t& carry) {
  const f32x2 g = grid2<FMT>(x0 * inv_s, x1 * inv_s, carry);
  const double d0 = __builtin_fma(-static_cast<double>(g[0]), sd, static_cast<double>(x0));
  const double d1 = __builtin_fma(-static_cast<double>(g[1]), sd, static_cast<double>(x1));
  acc = __builtin_fma(d0, d0, acc);
  acc = __builtin_fma(d1, d1, acc);
}

// Codes of 8 scaled elements (Raw8::scaled).  4-bit: one word, element 2j in the low nibble of byte j;
// 8-bit: two words, one byte per element.  The FP formats use the gfx950 pack-convert
// instructions (round to nearest even, subnormals kept, saturating; the E4M3 convert
// needs its input clamped to +-448 first), which agree with Codec<>::code on every
// finite fp32 bit pattern.
template <int FMT>
MOFQ_DEV void encode_scaled8(const float (&t)[8], uint32_t (&words)[2]) {
  if constexpr (FMT == MOFQ_FP4_E2M1) {
    uint32_t w = 0;
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, t[0], t[1], 1.0f, 0);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, t[2], t[3], 1.0f, 1);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, t[4], t[5], 1.0f, 2);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, t[6], t[7], 1.0f, 3);
    words[0] = w;
    words[1] = 0;
  } else if constexpr (FMT == MOFQ_FP8_E4M3) {
    float c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = med3(t[i], -448.0f, 448.0f);
    int w0 = 0, w1 = 0;
    w0 = __builtin_amdgcn_cvt_pk_fp8_f32(c[0], c[1], w0, false);
    w0 = __builtin_amdgcn_cvt_pk_fp8_f32(c[2], c[3], w0, true);
    w1 = __builtin_amdgcn_cvt_pk_fp8_f32(c[4], c[5], w1, false);
    w1 = __builtin_amdgcn_cvt_pk_fp8_f32(c[6], c[7], w1, true);
    words[0] = static_cast<uint32_t>(w0);
    words[1] = static_cast<uint32_t>(w1);
  } else if constexpr (FMT == MOFQ_INT4 || FMT == MOFQ_INT8) {
    // Clamping before rounding gives the same integer (the bounds are integers); adding 1.5 * 2^23
    // rounds to nearest even and leaves the two's-complement integer in the low bits.
    constexpr float lo = FMT == MOFQ_INT4 ? -8.0f : -128.0f, hi = FMT == MOFQ_INT4 ? 7.0f : 127.0f;
    uint32_t y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = f2u(med3(t[i], lo, hi) + 12582912.0f);
    if constexpr (FMT == MOFQ_INT4) {
      uint32_t b[4];   // two codes in the low byte
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = (y[2 * i] & 0xFu) | ((y[2 * i + 1] << 4) & ~0xFu);
      words[0] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0C0C0400u), __builtin_amdgcn_perm(b[1], b[0], 0x0C0C0400u), 0x05040100u);
      words[1] = 0;
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        words[i] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(y[4 * i + 3], y[4 * i + 2], 0x0C0C0400u),
                                         __builtin_amdgcn_perm(y[4 * i + 1], y[4 * i], 0x0C0C0400u), 0x05040100u);
    }
  } else if constexpr (Codec<FMT>::BITS == 4) {
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) w |= Codec<FMT>::code(t[i]) << (4 * i);
    words[0] = w;
    words[1] = 0;
  } else {
    uint32_t w0 = 0, w1 = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w0 |= Codec<FMT>::code(t[i]) << (8 * i);
      w1 |= Codec<FMT>::code(t[4 + i]) << (8 * i);
    }
    words[0] = w0;
    words[1] = w1;
  }
}

template <int FMT> MOFQ_DEV void encode8(const float (&v)[8], float inv_s, uint32_t (&words)[2]) {
  float t[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] = v[i] * inv_s;
  encode_scaled8<FMT>(t, words);
}

// What the finished rows of a tensor favour (AheadCodes): read by one wave (a lane per place; the sum
// is over the wave), added to by one thread of one row in EVERY.  Workgroup ids go round the XCDs;
// workgroup scope keeps both in the XCD's own L2.  Stale or missed values only cost a row done twice.
MOFQ_DEV double tally_read(const AheadCodes& a) {
  const int lane = threadIdx.x & 63;
  const double* const t = a.tally + ((blockIdx.x % kXcds) * kTalliesPerXcd + lane) * kTallyStride;
  return lane < kTalliesPerXcd ? __hip_atomic_load(t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0.0;
}
// (loads queue behind the additions: the shorter a row's work, the fewer of them)
template <unsigned EVERY> MOFQ_DEV void tally_add(const AheadCodes& a, double d) {
  const unsigned n = blockIdx.x / kXcds;   // this row's number in its XCD
  if (n / kTalliesPerXcd % EVERY == 0)
    __hip_atomic_fetch_add(a.tally + ((blockIdx.x % kXcds) * kTalliesPerXcd + n % kTalliesPerXcd) * kTallyStride, d, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

// 8 elements as they come from memory, widened where they are used
template <typename In> struct Raw8 {
  u32x4 w;
  // element i0 + i; i0 is uniform
  MOFQ_DEV void load(const void* base, int64_t i0, uint32_t i) {
    w = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(base) + i0 + i);
  }
  MOFQ_DEV void clear() { w = u32x4{0u, 0u, 0u, 0u}; }
  MOFQ_DEV void opaque() { asm volatile("" : "+v"(w)); }   // what was computed from it is not kept for later uses
  MOFQ_DEV void widen(float (&v)[8]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (std::is_same<In, F16>::value) {
        v[2 * i] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w[i])));
        v[2 * i + 1] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w[i] >> 16)));
      } else {
        v[2 * i] = u2f(w[i] << 16);
        v[2 * i + 1] = u2f(w[i] & 0xFFFF0000u);
      }
    }
  }
  // fl32(x * inv).  fp16: widening and product are one mixed-precision fused multiply-add, the same single rounding of
  // the exact product; the addend -0 leaves a zero's sign.
  MOFQ_DEV void scaled(float inv, float (&t)[8]) const {
    widen(t);
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = std::is_same<In, F16>::value ? __builtin_fmaf(t[i], inv, -0.0f) : t[i] * inv;
  }
};
template <> struct Raw8<F32> {
  u32x4 w[2];
  MOFQ_DEV void load(const void* base, int64_t i0, uint32_t i) {
    const u32x4* p = reinterpret_cast<const u32x4*>(static_cast<const float*>(base) + i0 + i);
    w[0] = p[0];
    w[1] = p[1];
  }
  MOFQ_DEV void clear() { w[0] = w[1] = u32x4{0u, 0u, 0u, 0u}; }
  MOFQ_DEV void opaque() { asm volatile("" : "+v"(w[0]), "+v"(w[1])); }
  MOFQ_DEV void widen(float (&v)[8]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] = u2f(w[0][i]); v[4 + i] = u2f(w[1][i]); }
  }
  MOFQ_DEV void scaled(float inv, float (&t)[8]) const {
    widen(t);
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] *= inv;
  }
};

template <typename F> MOFQ_DEV void with_format(int fmt, F&& f) {
  switch (fmt) {
    case MOFQ_INT4: f(std::integral_constant<int, MOFQ_INT4>{}); break;
    case MOFQ_FP4_E2M1: f(std::integral_constant<int, MOFQ_FP4_E2M1>{}); break;
    case MOFQ_INT8: f(std::integral_constant<int, MOFQ_INT8>{}); break;
    case MOFQ_FP4_E2M1_IEEE: f(std::integral_constant<int, MOFQ_FP4_E2M1_IEEE>{}); break;
    case MOFQ_FP8_E5M2: f(std::integral_constant<int, MOFQ_FP8_E5M2>{}); break;
    default: f(std::integral_constant<int, MOFQ_FP8_E4M3>{}); break;
  }
}

}  // namespace

}  // namespace mofq
