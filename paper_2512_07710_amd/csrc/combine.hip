// Weighted combine of the expert outputs back to token order.
//
// Each thread gathers its columns of the k expert-ordered fp32 rows named by inv_perm,
// accumulates w[t,j]*row in slot order with fp32 fused multiply-adds and rounds to
// bf16 once.  A gather per output token needs no atomics and is deterministic.
#include "moe_internal.hpp"

namespace moe355 {
namespace {

__device__ inline uint32_t f32_to_bf16_rne(float v) {
    uint32_t b = __float_as_uint(v);
    if ((b & 0x7FFFFFFFu) > 0x7F800000u) return (b >> 16) | 0x40;   // NaN stays NaN
    return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int COMBINE_THREADS = 256;

// One thread owns four columns of one token, so a block covers up to 1024 columns and a token takes ceil(d/1024) blocks of equal
// width: each wave issues its k row reads once and is replaced by a fresh one.  KT > 0: k known at compile time, so that the k reads are
// all in flight before the first multiply-add; KT == 0: any k up to MAX_K.
//
// Bound by the bytes of the expert rows, each read exactly once: they go past the caches (non-temporal), and so does y.  One block per
// token that walked the row (4096 x 5120, k = 8): 144 us = 5.0 TB/s, with non-temporal reads 131; in this form 139 without
// and 119 (6.0 TB/s) with them; 32768 x 7168: 1.58 -> 1.38 ms.  The same for rows that the last-level cache could hold: layers on buffers
// of their own taken in turns, us, one block per token / through the caches / past them: 1901 x 1920, k = 6 (88 MB of rows) 104.6 / 102.4 /
// 93.6, 2000 x 2048, k = 4 109 / 106 / 100, 1233 x 1792, k = 7 84 / 83 / 78.  A single layer repeated on the same buffers with nothing
// between is the exception (92.9 / 91.1 / 95.8, 92.5 / 89.8 / 93.0, 77.8 / 76.5 / 80.6).
// Equal widths: 1152 columns as blocks of 1024 and 128 left seven eighths of every second block idle (layers of 6000 x 1152, k = 4
// 122.2, with equal ones 120.3, of 8600 x 1152, k = 1 74.6 / 71.4).
template <int KT>
__global__ __launch_bounds__(COMBINE_THREADS) void combine_kernel(const float* __restrict__ y_perm,
                                                                  const int32_t* __restrict__ inv_perm,
                                                                  const float* __restrict__ topk_w, int d, int k_rt,
                                                                  int parts, uint16_t* __restrict__ y,
                                                                  float* __restrict__ y_f32) {
    const int t = blockIdx.x / parts;
    const int c4 = (blockIdx.x % parts) * blockDim.x + threadIdx.x;
    if (c4 >= d / 4) return;
    const int k = KT > 0 ? KT : k_rt;
    const int32_t* const rows = inv_perm + (size_t)t * k;      // block-uniform: scalar loads
    const float* const w = topk_w + (size_t)t * k;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto load = [&](int row) {
        return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(y_perm + (size_t)row * d + (size_t)c4 * 4));
    };
    auto add = [&](float wj, const f32x4& v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = fmaf(wj, v[i], acc[i]);
    };
    if (KT > 0) {
        constexpr int KU = KT > 0 ? KT : 1;
        f32x4 v[KU];
        int row[KU];
#pragma unroll
        for (int j = 0; j < KU; ++j) {
            row[j] = rows[j];                                  // < 0: the slot's expert id was invalid, it adds nothing
            v[j] = load(max(row[j], 0));
        }
#pragma unroll
        for (int j = 0; j < KU; ++j)
            if (row[j] >= 0) add(w[j], v[j]);
    } else {
        for (int j = 0; j < k; ++j) {
            const int row = rows[j];
            if (row >= 0) add(w[j], load(row));
        }
    }
    u32x2 o;
    o[0] = f32_to_bf16_rne(acc[0]) | (f32_to_bf16_rne(acc[1]) << 16);
    o[1] = f32_to_bf16_rne(acc[2]) | (f32_to_bf16_rne(acc[3]) << 16);
    __builtin_nontemporal_store(o, reinterpret_cast<u32x2*>(y + (size_t)t * d + (size_t)c4 * 4));
    if (y_f32) *reinterpret_cast<f32x4*>(y_f32 + (size_t)t * d + (size_t)c4 * 4) = acc;   // the sums before rounding
}

}  // namespace

hipError_t launch_combine(moe_ctx* c, const float* y_perm, const int32_t* inv_perm, const float* topk_w,
                          uint16_t* y, float* y_f32) {
    const moe_dims& D = c->dims;
    const int parts = (D.d / 4 + COMBINE_THREADS - 1) / COMBINE_THREADS;
    const int threads = ((D.d / 4 + parts - 1) / parts + 63) / 64 * 64;
#define MOE_COMBINE(KT_)                                                                                             \
    hipLaunchKernelGGL(combine_kernel<KT_>, dim3((unsigned)(D.T * parts)), dim3(threads), 0, c->stream, y_perm, \
                       inv_perm, topk_w, D.d, D.k, parts, y, y_f32)
    switch (D.k) {
        case 1: MOE_COMBINE(1); break;
        case 2: MOE_COMBINE(2); break;
        case 3: MOE_COMBINE(3); break;
        case 4: MOE_COMBINE(4); break;
        case 5: MOE_COMBINE(5); break;
        case 6: MOE_COMBINE(6); break;
        case 7: MOE_COMBINE(7); break;
        case 8: MOE_COMBINE(8); break;
        default: MOE_COMBINE(0); break;
    }
#undef MOE_COMBINE
    return hipGetLastError();
}

}  // namespace moe355
