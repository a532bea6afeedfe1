// Block-wise FP8 (e4m3) quantisation of a bf16 weight matrix: one fp32 scale per 128x128 block.
//
// One workgroup of 512 threads per block.  Sixteen lanes own one row of the block, 8 columns (16 bytes) each, so that a
// wave's load instruction reads four whole 256-byte row pieces and its stores write four whole 128-byte ones; a thread
// holds the same 8 columns of four rows, 32 rows apart.  The block maximum goes through a wave reduction and eight LDS
// words; scale = amax/448 is a correctly rounded fp32 division and w/scale its correctly rounded quotient, so that codes
// and scales are reproducible bit for bit.  Each element is read once and written once: 3 bytes of HBM traffic per weight,
// which bound the kernel.  Neither the weights nor the codes are touched again soon: both go past the caches.
//
// 196608 x 5120 weights: 690 us (4.4 TB/s) with 64 contiguous elements per thread and true divisions; 571 with 256 threads
// in this arrangement and the shorter quotient, 532 with non-temporal loads and stores, 521 (5.8 TB/s) with 512 threads.
#include "e4m3.hpp"
#include "moe_internal.hpp"

namespace moe355 {
namespace {

constexpr int WQ_THREADS = 512;
constexpr int WQ_ROWS = WQ_THREADS / 16;               // rows of the block per pass
constexpr int WQ_PASSES = QBLOCK / WQ_ROWS;

__global__ __launch_bounds__(WQ_THREADS) void quantize_blocks_kernel(const uint16_t* __restrict__ w, int64_t rows, int cols,
                                                                     uint8_t* __restrict__ q,
                                                                     float* __restrict__ scales) {
    __shared__ float s_max[WQ_THREADS / 64];
    const int bj = blockIdx.x, tid = threadIdx.x;
    const int64_t bi = blockIdx.y;
    const size_t off = (size_t)(bi * QBLOCK + (tid >> 4)) * cols + (size_t)bj * QBLOCK + (tid & 15) * 8;
    u32x4 raw[WQ_PASSES];
#pragma unroll
    for (int v = 0; v < WQ_PASSES; ++v)
        raw[v] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(w + off + (size_t)v * WQ_ROWS * cols));
    float amax = 0.f;
#pragma unroll
    for (int v = 0; v < WQ_PASSES; ++v) amax = fmaxf(amax, bf16x8_amax(raw[v]));
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) amax = fmaxf(amax, __shfl_xor(amax, m));
    if ((tid & 63) == 0) s_max[tid >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WQ_THREADS / 64; ++i) amax = fmaxf(amax, s_max[i]);
    const E4m3Coder coder((amax == 0.f) ? 1.0f : amax / 448.0f);
    if (tid == 0) scales[(size_t)bi * (cols / QBLOCK) + bj] = coder.s;
#pragma unroll
    for (int v = 0; v < WQ_PASSES; ++v)
        __builtin_nontemporal_store(coder.pack8(raw[v]), reinterpret_cast<u32x2*>(q + off + (size_t)v * WQ_ROWS * cols));
    (void)rows;
}

}  // namespace

hipError_t launch_quantize_weights(hipStream_t s, const uint16_t* w, int64_t rows, int32_t cols, uint8_t* q,
                                   float* scales) {
    hipLaunchKernelGGL(quantize_blocks_kernel, dim3(cols / QBLOCK, (unsigned)(rows / QBLOCK)), dim3(WQ_THREADS), 0, s, w,
                       rows, cols, q, scales);
    return hipGetLastError();
}

}  // namespace moe355
