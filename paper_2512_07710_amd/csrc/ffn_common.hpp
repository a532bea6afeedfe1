// What the block-scaled FP8 GEMMs share: the big tiles (ffn.hip) and the weight-streaming kernels (ffn_stream.hip, ffn_flow.hip, ffn_few.hip).
#pragma once
#include "lanes.hpp"
#include "moe_internal.hpp"

namespace moe355 {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int KB = QBLOCK;                        // K bytes per stage (= one scale block)

// Direct global -> LDS copies.  Lane i of the wave deposits its bytes at lds_addr + i*size;
// the global address is sbase + voff (per lane).  Completion is tracked by vmcnt; the
// compiler does not see these as memory operations of its own, so every wait on them is
// written out explicitly by the kernels.  (The big tiles issue most of theirs under scalar conditions, in ffn.hip.)
__device__ inline void dma16(uint32_t lds_addr, uint32_t voff, const void* sbase) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
}
// the same for bytes that nothing else will read
__device__ inline void dma16_once(uint32_t lds_addr, uint32_t voff, const void* sbase) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
}
__device__ inline void dma4(uint32_t lds_addr, uint32_t voff, const void* sbase) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
}

// a < b ? -1 : 0 for wave-uniform values, in a scalar register whatever the compiler makes of the comparison
__device__ __forceinline__ int all_ones_if_less(int a, int b) {
    int r;
    asm("s_cmp_lt_i32 %1, %2\n\ts_cselect_b32 %0, -1, 0" : "=s"(r) : "s"(a), "s"(b) : "scc");
    return r;
}

// the 32 K-bytes a lane feeds to one 32x32x64 MFMA, from its row's two swizzled 16-byte chunks at LDS addresses c0, c1
typedef __attribute__((address_space(3))) const v4i* lds_v4i;
__device__ inline v8i lds_operand(uint32_t c0, uint32_t c1, int plus) {
    const v4i lo = *reinterpret_cast<lds_v4i>(c0 + plus), hi = *reinterpret_cast<lds_v4i>(c1 + plus);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// h / sc, correctly rounded, for many values over one scale: a reciprocal refined once, then the quotient estimate corrected by
// its exact remainder (three instructions instead of a full division each; equal to the division wherever sc is far from the
// ends of the fp32 range, and the plain division elsewhere).  |h / sc| <= 448 up to one rounding, so no clamp.
struct Quotient {
    float sc, inv;
    bool mid_range;
    __device__ explicit Quotient(float s) : sc(s) {
        inv = __builtin_amdgcn_rcpf(sc);
        inv = fmaf(fmaf(-sc, inv, 1.0f), inv, inv);
        mid_range = sc > 1e-30f && sc < 1e30f;
    }
    __device__ float operator()(float hv) const {
        const float q0 = hv * inv;
        return mid_range ? fmaf(fmaf(-q0, sc, hv), inv, q0) : hv / sc;
    }
};
__device__ inline uint32_t e4m3_codes4(const Quotient& q, float a, float b, float c, float d) {
    int code = 0;
    code = __builtin_amdgcn_cvt_pk_fp8_f32(q(a), q(b), code, false);
    code = __builtin_amdgcn_cvt_pk_fp8_f32(q(c), q(d), code, true);
    return (uint32_t)code;
}
// silu(g)*u with the hardware reciprocal (1 ulp): far below the matrix cores' own error
__device__ inline float swiglu(float g, float u) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u; }

}  // namespace moe355
