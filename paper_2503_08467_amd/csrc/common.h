// Internal device helpers shared by the MoE layer kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe {

typedef uint16_t bf16_t;  // raw bfloat16 bits
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// float -> bfloat16, round to nearest even (gfx950 converts in hardware: v_cvt_pk_bf16_f32).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return __builtin_bit_cast(bf16_t, static_cast<__bf16>(f)); }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const bf16x2_t v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Lanes of this wave whose expert equals this lane's (valid lanes only), from nbits ballots
// over the id bits (E <= 2^nbits).
__device__ __forceinline__ uint64_t same_expert_lanes(int e, bool valid, int nbits) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
        const bool bit = valid && ((e >> b) & 1);
        const uint64_t m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    return peers;
}

// Activations of the expert FFN (fp32).
__device__ __forceinline__ float act_gelu(float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752f)); }

__device__ __forceinline__ float act_gelu_tanh(float u) {
    const float c = 0.79788456080286536f;  // sqrt(2/pi)
    return 0.5f * u * (1.0f + tanhf(c * (u + 0.044715f * u * u * u)));
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

// Fast activations for the bf16 epilogues (their error is far below bf16 rounding).
//
// GELU(u) = u Phi(u) = max(u, 0) - |u| Q(|u|) with Q(a) = Phi(-a) = 2^p(a); p, the base-2
// logarithm of the normal tail, is smooth, and its degree-8 fit here (least largest error of
// a Q(a) over [0, 9], by linear programming, subject to the relative errors of the tail) leaves
// |GELU error| <= 2.6e-7 in fp32 (3.9e-8 root mean square over N(0, 1)) and in the negative
// tail relative errors of at most 2.6e-3 down to -7 and 1.2e-2 down to -9, where the values
// are 1e-18; past that the leading coefficient takes 2^p to 0.  One exponential and ten plain
// instructions, where Abramowitz & Stegun 7.1.26 (3.3e-7, 5.5e-8, 6.5e-3 and 1.5e-2) took a
// reciprocal, an exponential and fourteen.
__device__ __forceinline__ float act_gelu_fast(float u) {
    const float a = fabsf(u);
    float p = -1.76333070e-07f;
    p = fmaf(p, a, 2.71696660e-06f);
    p = fmaf(p, a, 1.74325122e-05f);
    p = fmaf(p, a, -7.24288286e-04f);
    p = fmaf(p, a, 8.01050460e-03f);
    p = fmaf(p, a, -5.33516148e-02f);
    p = fmaf(p, a, -4.58798370e-01f);
    p = fmaf(p, a, -1.15119599e+00f);
    p = fmaf(p, a, -9.99993450e-01f);
    // max(u, 0) as a median: one instruction (fmaxf would quiet u first)
    return fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_amdgcn_fmed3f(u, 0.f, __builtin_inff()));
}

// act_gelu_fast with p of degree 10: 2.4e-7 at most and 2.1e-8 root mean square, where
// 0.5 u (1 + erff) has 4.5e-7 and 2.5e-8 and no digit left in the tail.  An infinity gives itself
// or, below zero, NaN, as it does there.
__device__ __forceinline__ float act_gelu_near(float u) {
    const float a = fabsf(u);
    float p = -7.46755095e-09f;
    p = fmaf(p, a, 2.90787827e-07f);
    p = fmaf(p, a, -4.67541513e-06f);
    p = fmaf(p, a, 3.87351075e-05f);
    p = fmaf(p, a, -1.46217167e-04f);
    p = fmaf(p, a, -2.85693500e-04f);
    p = fmaf(p, a, 7.31283934e-03f);
    p = fmaf(p, a, -5.27087918e-02f);
    p = fmaf(p, a, -4.59119996e-01f);
    p = fmaf(p, a, -1.15111982e+00f);
    p = fmaf(p, a, -9.99999538e-01f);
    const float r = fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_amdgcn_fmed3f(u, 0.f, __builtin_inff()));
    return a < __builtin_inff() ? r : u * __builtin_amdgcn_fmed3f(u, 0.f, 1.f);
}

// 0.5 u (1 + tanh(z)) = u / (1 + e^(-2 z)), z = sqrt(2 / pi) (u + 0.044715 u^3), with the
// hardware exponential and reciprocal: no cancellation in the negative tail (relative errors
// there below 4e-6 down to -6, where 1 + tanhf leaves no digit; root mean square over N(0, 1)
// 3.0e-8 against tanhf's 2.5e-8).
__device__ __forceinline__ float act_gelu_tanh_fast(float u) {
    const float c = -2.0f * 0.79788456080286536f * 1.4426950408889634f;  // -2 sqrt(2 / pi) log2(e)
    const float z = u * fmaf(u * u, c * 0.044715f, c);
    return u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z));
}

// silu(z) = z / (1 + e^-z) with the hardware exponential and reciprocal (about 1 ulp each).
__device__ __forceinline__ float silu_fast(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

__host__ __device__ constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
__host__ __device__ constexpr int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

}  // namespace moe
