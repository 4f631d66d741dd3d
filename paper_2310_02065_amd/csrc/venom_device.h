// Device code that the product kernels share: operand types, the 2:4 matrix instruction, the activations.
#pragma once

#include "venom_internal.h"

namespace venom {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half16 __attribute__((ext_vector_type(16)));
typedef _Float16 half2 __attribute__((ext_vector_type(2)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

#define LDS_PTR(T) T __attribute__((address_space(3)))*

// GELU(x) = x * Phi(x) = max(x, 0) - |x| Q(|x|), Q the upper tail of the normal distribution, as 2^P(|x|): log2 Q is
// smooth, so one exponential and no reciprocal, and x < 0 gets its tail by a product, not as a difference.  P(0) = -1, and
// each P is the polynomial of its degree with the smallest largest error (a linear program), counted in units of E as
// error of |x| Q and, for |x| > 4, in units of 2e-4 (|x| - 2.5)^2 as relative error of Q (0.6 to 0.9 of that of the
// rational-times-Gaussian formula 7.1.26 of Abramowitz & Stegun, which served here before):
//   fp16 output: degree 8 on |x| <= 5.9, E = 2e-8; from there on P stays below -29 and falls, and the output is zero.
//     Its leading coefficient is negative, so that no clamp is needed.  Of all fp16 x 53 round another way than
//     the exact value, by one unit in the last place (256 with 7.1.26, 332 with x/2 + |x| (1/2 - Q)).
//   fp32 output: degree 11 on |x| <= 13, E = 5e-9, as there the tail is seen down to x = -12.9, where 2^P underflows.  |x| is
//     clamped where it is multiplied, too: no 0 x Inf.  3e-8 in norm on N(0, 1/4) .. N(0, 9) (7.1.26: 5e-8 to 1e-7), on no
//     interval worse than 7.1.26 or x/2 + |x| (1/2 - Q).
// `on` is 1 for x > 0 and 0 for x < 0 (in between it is multiplied by next to nothing), one multiplication with the
// clamp of its result; infinities and NaN come out as from x * Phi(x).  11 and 15 full-rate instructions and one transcendental
// (7.1.26: 15 and two).  The output stage evaluates it 128 times per lane on the waves that the matrix instructions
// then wait for: 4096 x 1024 x 16384 at 128:2:16 with bias, us per call, 7.1.26 -> now, fp16 73 -> 65, fp32 91 -> 90; as
// token-major layer 93 -> 90 and 117 -> 113.
template <bool OUT_F32>
__device__ __forceinline__ float gelu_by_definition(float x) {
  const float on = __builtin_amdgcn_fmed3f(x * 0x1p126f, 0.f, 1.f);
  if constexpr (OUT_F32) {
    const float a = __builtin_amdgcn_fmed3f(fabsf(x), 0.f, 13.5f);
    float p = fmaf(5.57935698e-10f, a, -3.05136716e-08f);
    p = fmaf(p, a, 6.97282076e-07f);
    p = fmaf(p, a, -8.63450987e-06f);
    p = fmaf(p, a, 6.18117556e-05f);
    p = fmaf(p, a, -2.28697128e-04f);
    p = fmaf(p, a, -1.04886603e-04f);
    p = fmaf(p, a, 7.07445014e-03f);
    p = fmaf(p, a, -5.25283851e-02f);
    p = fmaf(p, a, -4.59191263e-01f);
    p = fmaf(p, a, -1.15110779f);
    p = fmaf(p, a, -1.f);
    return fmaf(-a, __builtin_amdgcn_exp2f(p), x * on);
  } else {
    const float a = fabsf(x);
    float p = fmaf(-1.12579994e-06f, a, 1.83935899e-05f);
    p = fmaf(p, a, -8.35712781e-05f);
    p = fmaf(p, a, -3.9356359e-04f);
    p = fmaf(p, a, 7.4137128e-03f);
    p = fmaf(p, a, -5.27529866e-02f);
    p = fmaf(p, a, -4.59116608e-01f);
    p = fmaf(p, a, -1.15111709f);
    p = fmaf(p, a, -1.f);
    return x * fabsf(on - __builtin_amdgcn_exp2f(p));
  }
}
// The tanh form x/2 * (1 + tanh u), u = sqrt(2/pi) (x + 0.044715 x^3), written as x / (1 + e^(-2u)); the exponent of 2
// is x (A + B x^2), A = -2 log2(e) sqrt(2/pi), B = 0.044715 A.
__device__ __forceinline__ float gelu_tanh_form(float x) {
  const float e = __builtin_amdgcn_exp2f(x * fmaf(x * x, -0.10294324f, -2.30220818f));
  return x * __builtin_amdgcn_rcpf(1.f + e);
}

template <int ABID>
__device__ __forceinline__ floatx16 smfmac(half8 a, half16 b, floatx16 c, int idx) {
  return __builtin_amdgcn_smfmac_f32_32x32x32_f16(a, b, c, idx, 0, ABID);
}

}  // namespace venom
