// bf16 -> e4m3 coding shared by the activation and the weight quantisation kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe355 {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ inline float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ inline float clamp448(float v) { return fminf(fmaxf(v, -448.f), 448.f); }

// largest magnitude of 8 bf16 values (a NaN does not count)
__device__ inline float bf16x8_amax(const u32x4& u) {
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) amax = fmaxf(amax, fmaxf(fabsf(bf16lo(u[i])), fabsf(bf16hi(u[i]))));
    return amax;
}

// v / s from an estimate of 1/s: the reciprocal refined once, then the quotient estimate corrected by its exact remainder
// (Markstein's correction); signs are arranged so that -0 stays -0.  For every bf16 significand over every scale amax/448 with a
// bf16 amax, and an estimate up to 2 ulp off, it equals the division (tests/test_quotient_host.py compiles these two functions).
__host__ __device__ inline float refined_reciprocal(float s, float estimate) { return fmaf(fmaf(-s, estimate, 1.0f), estimate, estimate); }
__host__ __device__ inline float corrected_quotient(float v, float s, float inv) {
    const float q0 = v * inv;
    return fmaf(-fmaf(q0, s, -v), inv, q0);
}

// Codes of 8 bf16 values over the group's scale s = amax/448 (1 for an all-zero group).
// A true division is some ten instructions and made the quantisation kernels bound by the vector ALU (weights: 4.4 TB/s,
// against 5.8 with this form).  In the stated range of s no remainder of a quotient that can reach a non-zero code underflows;
// outside it (and for an infinite s) the division itself is taken.
constexpr float SCALE_MID_MIN = 1e-25f, SCALE_MID_MAX = 1e25f;
struct E4m3Coder {
    float s, inv;
    bool mid_range;
    __device__ explicit E4m3Coder(float scale) : s(scale) {
        inv = refined_reciprocal(s, __builtin_amdgcn_rcpf(s));
        mid_range = s > SCALE_MID_MIN && s < SCALE_MID_MAX;
    }
    __device__ float quotient(float v) const { return corrected_quotient(v, s, inv); }
    // four codes, a in the low byte.  |v| <= amax, so the quotient is at most 448 up to one rounding, which the conversion
    // rounds back; the lower bound stays because it is what makes a NaN -448.
    __device__ uint32_t pack4(float a, float b, float c, float d) const {
        int p = 0;
        if (mid_range) {
            p = __builtin_amdgcn_cvt_pk_fp8_f32(fmaxf(quotient(a), -448.f), fmaxf(quotient(b), -448.f), p, false);
            p = __builtin_amdgcn_cvt_pk_fp8_f32(fmaxf(quotient(c), -448.f), fmaxf(quotient(d), -448.f), p, true);
        } else {
            p = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a / s), clamp448(b / s), p, false);
            p = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(c / s), clamp448(d / s), p, true);
        }
        return (uint32_t)p;
    }
    __device__ u32x2 pack8(const u32x4& u) const {
        u32x2 c;
        c[0] = pack4(bf16lo(u[0]), bf16hi(u[0]), bf16lo(u[1]), bf16hi(u[1]));
        c[1] = pack4(bf16lo(u[2]), bf16hi(u[2]), bf16lo(u[3]), bf16hi(u[3]));
        return c;
    }
};

}  // namespace moe355
