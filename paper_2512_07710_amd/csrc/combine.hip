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
constexpr int64_t LAYER_CACHED_BYTES = 192ll << 20, ROWS_CACHED_BYTES = 96ll << 20;

// One thread owns four columns of one token, so a block covers up to 1024 columns and a token takes ceil(d/1024) blocks of equal
// width: each wave issues its k row reads once and is replaced by a fresh one.  KT > 0: k known at compile time, so that the k reads are
// all in flight before the first multiply-add; KT == 0: any k up to MAX_K.
//
// Bound by the bytes of the expert rows, each read exactly once.  PAST: they go past the caches (non-temporal), and so does y.  One block
// per token that walked the row (4096 x 5120, k = 8): 144 us = 5.0 TB/s, with non-temporal reads 131; in this form 139
// without and 119 (6.0 TB/s) with them; 32768 x 7168: 1.58 -> 1.38 ms.
// Not PAST: a layer whose weights and rows stay in the last-level cache together.  Non-temporal reads are then at the mercy of where the
// rows lie: 88 MB of them (1901 x 1920, k = 6) copied in, combined and y read back 44 or 51 us, through the caches 44; layers of 1233 x
// 1792, k = 7 (62 MB) 80.6 / 76.5, of 1901 x 2048, k = 6 (93 MB) 100.9 / 95.2.  y stays near for its reader: 7168 columns x k = 1 and
// 50 MB of rows in the same sequence 39.7 / 37.4.  Other layers are faster PAST: 777 x 2176, k = 5 with 351 MB of weights 117 us,
// y through the caches 119.5, the rows as well 125; 123 MB of rows 151 / 159, 295 MB 254 / 270.
// Equal widths: 1152 columns as blocks of 1024 and 128 left seven eighths of every second block idle (10850 rows, k = 1, in the same
// sequence 43.3, now 38.6; one block per token 36.9.  The layers around such rows: 75.3 us with one block per token, now 72.9).
template <int KT, bool PAST>
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
        const f32x4* const from = reinterpret_cast<const f32x4*>(y_perm + (size_t)row * d + (size_t)c4 * 4);
        return PAST ? __builtin_nontemporal_load(from) : *from;
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
    u32x2* const to = reinterpret_cast<u32x2*>(y + (size_t)t * d + (size_t)c4 * 4);
    if (PAST) __builtin_nontemporal_store(o, to);
    else *to = o;
    if (y_f32) *reinterpret_cast<f32x4*>(y_f32 + (size_t)t * d + (size_t)c4 * 4) = acc;   // the sums before rounding
}

}  // namespace

hipError_t launch_combine(moe_ctx* c, const float* y_perm, const int32_t* inv_perm, const float* topk_w,
                          uint16_t* y, float* y_f32) {
    const moe_dims& D = c->dims;
    const int parts = (D.d / 4 + COMBINE_THREADS - 1) / COMBINE_THREADS;
    const int threads = ((D.d / 4 + parts - 1) / parts + 63) / 64 * 64;
    const int64_t row_bytes = (int64_t)D.T * D.k * D.d * (int64_t)sizeof(float), weight_bytes = 3ll * D.E * D.d * D.F;
    const bool past = row_bytes > ROWS_CACHED_BYTES || row_bytes + weight_bytes > LAYER_CACHED_BYTES;
#define MOE_COMBINE_AS(KT_, PAST_)                                                                                         \
    hipLaunchKernelGGL((combine_kernel<KT_, PAST_>), dim3((unsigned)(D.T * parts)), dim3(threads), 0, c->stream, y_perm, \
                       inv_perm, topk_w, D.d, D.k, parts, y, y_f32)
#define MOE_COMBINE(KT_)                     \
    do {                                     \
        if (past) MOE_COMBINE_AS(KT_, true); \
        else MOE_COMBINE_AS(KT_, false);     \
    } while (0)
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
#undef MOE_COMBINE_AS
    return hipGetLastError();
}

}  // namespace moe355
