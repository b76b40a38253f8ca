// mlp_kernels.hpp -- ensemble MLP surrogate for <v>(a, omega, F, D, gamma):
// members of 5 -> 256 -> 256 -> 256 -> 1 with tanh-GELU, BF16 weights and FP32
// accumulation.  The two 256 x 256 layers (99% of the work) run on
// v_mfma_f32_16x16x32_bf16; the 5-input and 1-output layers are FP32 FMAs on the same
// BF16 weights.  Layout of the parameters and the element-wise functions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bm {
namespace mlp {

constexpr int IN = 5;
constexpr int H = 256;
// FP32 parameter block of one member (row-major [out][in] weights):
constexpr int OFF_W1 = 0;                 // [256][5]
constexpr int OFF_B1 = OFF_W1 + H * IN;   // [256]
constexpr int OFF_W2 = OFF_B1 + H;        // [256][256]
constexpr int OFF_B2 = OFF_W2 + H * H;    // [256]
constexpr int OFF_W3 = OFF_B2 + H;        // [256][256]
constexpr int OFF_B3 = OFF_W3 + H * H;    // [256]
constexpr int OFF_W4 = OFF_B3 + H;        // [256]
constexpr int OFF_B4 = OFF_W4 + H;        // [1]
constexpr int NPARAM = OFF_B4 + 1;        // 133377
// BF16 weight block of one member: W1 | W2 | W3 | W4 (biases stay FP32)
constexpr int BOFF_W1 = 0;
constexpr int BOFF_W2 = BOFF_W1 + H * IN;
constexpr int BOFF_W3 = BOFF_W2 + H * H;
constexpr int BOFF_W4 = BOFF_W3 + H * H;
constexpr int NBF = BOFF_W4 + H;          // 132608

typedef uint16_t bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (NaN kept quiet).
__device__ __forceinline__ bf16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (bf16_t)((u >> 16) | 0x0040u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float((uint32_t)b << 16); }

// tanh-GELU: 0.5 z (1 + tanh u), u = c (z + 0.044715 z^3), c = sqrt(2 / pi).
// Since 0.5 (1 + tanh u) = 1 / (1 + e^{-2u}), gelu = z sigma with
// sigma = 1 / (1 + 2^{-2 c log2(e) z (1 + 0.044715 z^2)}) on the hardware exp2 and
// reciprocal (1 ulp each); sigma saturates to 0 / 1 for large |u|.  t = tanh u.
__device__ __forceinline__ float gelu_t(float z, float &t)
{
    const float k = -2.0f * 0.7978845608028654f * 1.4426950408889634f;   // -2 c log2(e)
    const float w = z * fmaf(k * 0.044715f, z * z, k);
    const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(w));
    t = fmaf(2.0f, sg, -1.0f);
    return z * sg;
}
__device__ __forceinline__ float gelu(float z)
{
    float t;
    return gelu_t(z, t);
}
// d gelu / dz = 0.5 (1 + t) + 0.5 z (1 - t^2) c (1 + 3 * 0.044715 z^2)
__device__ __forceinline__ float gelu_grad(float z)
{
    float t;
    (void)gelu_t(z, t);
    const float c = 0.7978845608028654f;
    return 0.5f * (1.0f + t) + 0.5f * z * (1.0f - t * t) * c * fmaf(0.134145f, z * z, 1.0f);
}

// Input normalisation to [-1, 1] over the surrogate's domain:
// a in [0, 8], omega in [1, 10], F in [-0.5, 0.5], log10 D in [-4, -1], gamma in [0.5, 2].
__device__ __forceinline__ void normalise(const float *x, float u[IN])
{
    u[0] = x[0] * 0.25f - 1.0f;
    u[1] = (x[1] - 5.5f) * (1.0f / 4.5f);
    u[2] = x[2] * 2.0f;
    u[3] = (log10f(x[3]) + 2.5f) * (1.0f / 1.5f);
    u[4] = (x[4] - 1.25f) * (1.0f / 0.75f);
}

} // namespace mlp
} // namespace bm
