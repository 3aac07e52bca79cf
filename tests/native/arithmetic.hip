// The searches' arithmetic as the kernels have it, for the tests: on the host what host code can run, on the device the rest.
#include "../../paper_2305_12356_amd/csrc/mofq_search_common.h"

using namespace mofq;

namespace {

template <typename In> void patterns(const float* thr, int n, float s, float inv, int first, int32_t* out) {
  const double unit = edge_unit(s, inv);
  for (int i = 0; i < n; ++i) out[i] = pattern_top<In>(decision_edge(thr[i]), unit) - (first + kPatternBase<In> - 1);   // patterns_below
}

// reciprocal() of `count` floats from the bit pattern `first` on; a quotient rounded to 53 bits rounds to the same 24.
__global__ __launch_bounds__(256) void reciprocal_kernel(uint32_t first, uint32_t count, uint32_t* bad) {
  uint32_t n = 0;
  for (uint64_t i = blockIdx.x * 256u + threadIdx.x; i < count; i += gridDim.x * 256u) {
    const float s = u2f(first + static_cast<uint32_t>(i));
    n += f2u(reciprocal(s)) != f2u(static_cast<float>(1.0 / static_cast<double>(s))) ? 1u : 0u;
  }
  if (n) atomicAdd(bad, n);
}

}  // namespace

extern "C" {

// out[i]: how many patterns from `first` on are at or below the level boundary with decision threshold thr[i].
void arithmetic_patterns(int bf16, const float* thr, int n, float s, float inv, int first, int32_t* out) {
  if (bf16) patterns<BF16>(thr, n, s, inv, first, out);
  else patterns<F16>(thr, n, s, inv, first, out);
}

// How many of `count` floats from the bit pattern `first` on have another quotient than fp32 division.
uint32_t arithmetic_quotients(int e2m1, uint32_t first, uint32_t count) {
  uint32_t bad = 0;
  for (uint32_t i = 0; i < count; ++i) {
    const float ra = __builtin_bit_cast(float, first + i);
    const float want = ra / (e2m1 ? 6.0f : 7.0f);
    bad += (e2m1 ? over_qmax<MOFQ_FP4_E2M1>(ra) : over_qmax<MOFQ_INT4>(ra)) != want;
  }
  return bad;
}

// `bad`: on the device, added to.
int arithmetic_reciprocals(uint32_t first, uint32_t count, uint32_t* bad, void* stream) {
  hipLaunchKernelGGL(reciprocal_kernel, dim3(2048), dim3(256), 0, static_cast<hipStream_t>(stream), first, count, bad);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // extern "C"
