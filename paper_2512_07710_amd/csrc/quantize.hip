// Per-row, per-128-column FP8 (e4m3) quantisation of bf16 activations, with optional
// fan-out of each quantised row to several output rows (the expert-ordered layout).
//
// A block takes 32 rows of one 128-column group.  Sixteen lanes own one row of it: each loads 8 bf16
// (16 bytes), the group maximum is reduced with four xor-shuffles, scale = amax/448 is a
// correctly rounded fp32 division and x/scale its correctly rounded quotient, so the codes are
// reproducible bit for bit.  The row is read once and written `fanout` times.  Scales are stored K-block
// major, scales[group][output row]: the layout the grouped GEMM reads them in.
//
// Bound by HBM (3 bytes per element).  With one row per block the scales left as single words, each in a cache line
// of its own, and every element paid a true division: 17.8 us for 4096 x 5120 and 37.2 for 8192 x 7168, against
// 14.4 and 29.4 (6.0 TB/s) in this form; 16 rows per block take 14.6 and 30.5, 64 rows 15.1 and 31.2.  Non-temporal loads
// would be 11 % faster at 32768 x 7168 but slower at 8192 and below, where x is still in the last-level cache.
#include "e4m3.hpp"
#include "moe_internal.hpp"

namespace moe355 {
namespace {

constexpr int Q_PASSES = 2;                            // rows per thread
constexpr int Q_ROWS = 16 * Q_PASSES;                  // rows per block
constexpr int64_t Q_MAX_GRID = 1 << 22;

__global__ __launch_bounds__(256) void quantize_rows_kernel(const uint16_t* __restrict__ x, int64_t rows_in,
                                                            int cols, const int32_t* __restrict__ dst_rows,
                                                            int fanout, uint8_t* __restrict__ q,
                                                            float* __restrict__ scales) {
    const int64_t rows_out = dst_rows ? rows_in * fanout : rows_in;
    const int groups = cols / QBLOCK;
    const int64_t units = (rows_in + Q_ROWS - 1) / Q_ROWS * groups;
    const int sub = threadIdx.x & 15;
    for (int64_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
        const int g = (int)(unit % groups);            // neighbouring blocks read neighbouring groups of the same rows
        const int64_t r0 = unit / groups * Q_ROWS + (threadIdx.x >> 4);
        const size_t col = (size_t)g * QBLOCK + sub * 8;
        u32x4 raw[Q_PASSES];
#pragma unroll
        for (int i = 0; i < Q_PASSES; ++i) {
            const int64_t r = r0 + i * 16;
            raw[i] = u32x4{0u, 0u, 0u, 0u};
            if (r < rows_in) raw[i] = *reinterpret_cast<const u32x4*>(x + r * cols + col);
        }
#pragma unroll
        for (int i = 0; i < Q_PASSES; ++i) {
            const int64_t r = r0 + i * 16;             // the 16 lanes of a group share it
            float amax = bf16x8_amax(raw[i]);
            amax = fmaxf(amax, __shfl_xor(amax, 1));
            amax = fmaxf(amax, __shfl_xor(amax, 2));
            amax = fmaxf(amax, __shfl_xor(amax, 4));
            amax = fmaxf(amax, __shfl_xor(amax, 8));
            if (r >= rows_in) continue;
            const E4m3Coder coder((amax == 0.f) ? 1.0f : amax / 448.0f);
            const u32x2 codes = coder.pack8(raw[i]);
            for (int j = 0; j < fanout; ++j) {
                const int64_t orow = dst_rows ? (int64_t)dst_rows[r * fanout + j] : r;
                if (orow < 0) continue;               // assignment skipped by the permutation
                *reinterpret_cast<u32x2*>(q + orow * cols + col) = codes;
                if (sub == 0) scales[(int64_t)g * rows_out + orow] = coder.s;
            }
        }
    }
}

}  // namespace

hipError_t launch_quantize(hipStream_t s, const uint16_t* x, int64_t rows_in, int32_t cols,
                           const int32_t* dst_rows, int32_t fanout, uint8_t* q, float* scales) {
    const int64_t units = (rows_in + Q_ROWS - 1) / Q_ROWS * (cols / QBLOCK);
    const int grid = (int)(units < Q_MAX_GRID ? units : Q_MAX_GRID);
    hipLaunchKernelGGL(quantize_rows_kernel, dim3(grid), dim3(256), 0, s, x, rows_in, cols, dst_rows, fanout, q,
                       scales);
    return hipGetLastError();
}

}  // namespace moe355
