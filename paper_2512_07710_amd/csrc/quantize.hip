// Per-row, per-128-column FP8 (e4m3) quantisation of bf16 activations, with optional
// fan-out of each quantised row to several output rows (the expert-ordered layout).
//
// A block takes 16 * PASSES rows of one 128-column group.  Sixteen lanes own one row of it: each loads 8 bf16
// (16 bytes), the group maximum is reduced with four xor-shuffles, scale = amax/448 is a
// correctly rounded fp32 division and x/scale its correctly rounded quotient, so the codes are
// reproducible bit for bit.  The row is read once and written `fanout` times.  Scales are stored K-block
// major, scales[group][output row]: the layout the grouped GEMM reads them in.
//
// Bound by HBM (3 bytes per element).  With one row per block the scales left as single words, each in a cache line
// of its own, and every element paid a true division: 15.6 us for 4096 x 5120 and 36.1 for 8192 x 7168 called in a row, against
// 12.4 and 28.2 (6.2 TB/s) with 32 rows per block.  Non-temporal loads
// would be 11 % faster at 32768 x 7168 but slower at 8192 and below, where x is still in the last-level cache.
#include "quantize_rows.hpp"

namespace moe355 {
namespace {

constexpr int64_t Q_MAX_GRID = 1 << 22;
// Fanned out, a block's work is its stores, fanout rows for each it reads, and a small batch in 32-row blocks leaves them to a few
// CUs, one round trip (index of the output row, store) after another: 69 x 1536 to 8 rows each took 5.9 us, one row per block 3.5.
// Below this many blocks of 32 rows it therefore runs in blocks of 16, four stores behind four indices that were requested with the
// row itself: 3.6 us, 256 x 4096 to 6 rows 5.1 -> 4.1.  Large batches are faster in the long blocks and with one store at a time,
// which keeps to fewer output rows at once: 16384 x 7168 to 8 rows 262 us against 324, 8192 x 4096 to 1 19.4 / 22.8;
// 4096 x 5120 to 8 (5120 blocks of 32 rows) level.
constexpr int64_t Q_LONG_MIN_BLOCKS = 8192;

template <int PASSES>                                  // rows per thread
__global__ __launch_bounds__(256) void quantize_rows_kernel(const uint16_t* __restrict__ x, int64_t rows_in,
                                                            int cols, const int32_t* __restrict__ dst_rows,
                                                            int fanout, uint8_t* __restrict__ q,
                                                            float* __restrict__ scales) {
    constexpr int AT_ONCE = PASSES == 1 ? 4 : 1;       // stores of a fanned-out row in flight
    const int64_t rows_out = dst_rows ? rows_in * fanout : rows_in;
    const int groups = cols / QBLOCK;
    const int64_t units = (rows_in + 16 * PASSES - 1) / (16 * PASSES) * groups;
    const int sub = threadIdx.x & 15;
    for (int64_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
        const int g = (int)(unit % groups);            // neighbouring blocks read neighbouring groups of the same rows
        const int64_t r0 = unit / groups * (16 * PASSES) + (threadIdx.x >> 4);
        const size_t col = (size_t)g * QBLOCK + sub * 8;
        u32x4 raw[PASSES];
        int32_t dst[PASSES];                           // lane `sub` of a row's sixteen: where slot `sub` of it goes
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int64_t r = r0 + i * 16;
            raw[i] = u32x4{0u, 0u, 0u, 0u};
            dst[i] = -1;
            if (r < rows_in) {
                raw[i] = *reinterpret_cast<const u32x4*>(x + r * cols + col);
                if (dst_rows && sub < fanout) dst[i] = dst_rows[r * fanout + sub];
            }
        }
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int64_t r = r0 + i * 16;             // the 16 lanes of a group share it
            const E4m3Coder coder = group_coder(raw[i]);
            if (r >= rows_in) continue;
            const u32x2 codes = coder.pack8(raw[i]);
            auto put = [&](int64_t orow) {
                if (orow < 0) return;                  // assignment skipped by the permutation
                *reinterpret_cast<u32x2*>(q + orow * cols + col) = codes;
                if (sub == 0) scales[(int64_t)g * rows_out + orow] = coder.s;
            };
            if (!dst_rows) {
                put(r);
                continue;
            }
            for (int j0 = 0; j0 < fanout; j0 += 16) {
                if (j0 > 0) dst[i] = j0 + sub < fanout ? dst_rows[r * fanout + j0 + sub] : -1;
                for (int j = 0; j < 16 && j0 + j < fanout; j += AT_ONCE) {
                    int32_t to[AT_ONCE];               // (slots past the fan-out hold -1)
#pragma unroll
                    for (int u = 0; u < AT_ONCE; ++u) to[u] = __shfl(dst[i], j + u, 16);
#pragma unroll
                    for (int u = 0; u < AT_ONCE; ++u) put(to[u]);
                }
            }
        }
    }
}

}  // namespace

hipError_t launch_quantize(hipStream_t s, const uint16_t* x, int64_t rows_in, int32_t cols,
                           const int32_t* dst_rows, int32_t fanout, uint8_t* q, float* scales) {
    auto blocks = [&](int rows) { return (rows_in + rows - 1) / rows * (cols / QBLOCK); };
    auto launch = [&](auto kernel, int64_t units) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(units < Q_MAX_GRID ? units : Q_MAX_GRID)), dim3(256), 0, s, x, rows_in, cols,
                           dst_rows, fanout, q, scales);
        return hipGetLastError();
    };
    return dst_rows && blocks(32) < Q_LONG_MIN_BLOCKS ? launch(quantize_rows_kernel<1>, blocks(16)) : launch(quantize_rows_kernel<2>, blocks(32));
}

}  // namespace moe355
