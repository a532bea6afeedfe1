// Block-wise FP8 (e4m3) quantisation of a bf16 weight matrix: one fp32 scale per 128x128 block.
//
// One workgroup of 512 threads per block, or of 1024 for two neighbouring ones.  Sixteen lanes own one row of a block, 8 columns (16 bytes) each,
// so that a wave's load instruction reads whole row pieces of 256 (pair: 512) bytes and its stores write whole ones of half that; a thread
// holds the same 8 columns of four rows, 32 rows apart.  The block maximum goes through a wave reduction and a few
// LDS words; scale = amax/448 is a correctly rounded fp32 division and w/scale its correctly rounded quotient, so that codes
// and scales are reproducible bit for bit.  Each element is read once and written once: 3 bytes of HBM traffic per weight,
// which bound the kernel.  Neither the weights nor the codes are touched again soon: both go past the caches.
//
// 196608 x 5120 weights: 690 us (4.4 TB/s) with 64 contiguous elements per thread and true divisions; 571 with 256 threads in this arrangement and
// the shorter quotient, 532 with non-temporal loads and stores, 521 (5.8 TB/s) with 512 threads, 501 (6.0) in pairs.  Pairs on 512 threads 504, on
// 256 510, four blocks on 1024 565; loads through the caches 519, stores 527; an eighth of the matrix to each XCD 504; fewer workgroups to a CU 505
// to 630.
#include "e4m3.hpp"
#include "moe_internal.hpp"

namespace moe355 {
namespace {

constexpr int WQ_ROWS = 32;                            // rows of a block per pass
constexpr int WQ_PASSES = QBLOCK / WQ_ROWS;

template <int B>                                       // neighbouring blocks that a workgroup takes
__global__ __launch_bounds__(512 * B) void quantize_blocks_kernel(const uint16_t* __restrict__ w, int cols, uint8_t* __restrict__ q,
                                                                  float* __restrict__ scales) {
    constexpr int LANES = 16 * B, WAVES = 8 * B;       // lanes of a row; waves
    __shared__ float s_max[B][WAVES];
    const int tid = threadIdx.x, sub = tid % LANES, mine = sub >> 4;           // which of the blocks
    const int bj = blockIdx.x * B + mine;
    const int64_t bi = blockIdx.y;
    const size_t off = (size_t)(bi * QBLOCK + tid / LANES) * cols + (size_t)bj * QBLOCK + (sub & 15) * 8;
    u32x4 raw[WQ_PASSES];
#pragma unroll
    for (int v = 0; v < WQ_PASSES; ++v)
        raw[v] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(w + off + (size_t)v * WQ_ROWS * cols));
    float amax = 0.f;
#pragma unroll
    for (int v = 0; v < WQ_PASSES; ++v) amax = fmaxf(amax, bf16x8_amax(raw[v]));
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        if (m < 16 || m >= LANES) amax = fmaxf(amax, __shfl_xor(amax, m));     // (not with another block's lanes)
    if ((tid & 63) < LANES && (sub & 15) == 0) s_max[mine][tid >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WAVES; ++i) amax = fmaxf(amax, s_max[mine][i]);
    const E4m3Coder coder((amax == 0.f) ? 1.0f : amax / 448.0f);
    if (tid < LANES && (sub & 15) == 0) scales[(size_t)bi * (cols / QBLOCK) + bj] = coder.s;
#pragma unroll
    for (int v = 0; v < WQ_PASSES; ++v)
        __builtin_nontemporal_store(coder.pack8(raw[v]), reinterpret_cast<u32x2*>(q + off + (size_t)v * WQ_ROWS * cols));
}

}  // namespace

// Pairs, where a row is a whole number of them and the matrix is more than the last-level cache holds (us, single blocks / pairs): 262144 x 7168 975
// / 922, 262144 x 1536 203 / 194, 131072 x 3072 201 / 195, 32768 x 4096 (256 MB of weights) 65.8 / 64.5; 16384 x 4096 33.4 / 33.6, 8192 x 4096 18.0 /
// 18.2; rows that end in half a pair, whose pieces are then not aligned to their size, 32768 x 7040 104.7 / 110.9, 131072 x 2944 177.7 / 186.5.
static constexpr int64_t PAIRS_FROM_BYTES = 256ll << 20;

hipError_t launch_quantize_weights(hipStream_t s, const uint16_t* w, int64_t rows, int32_t cols, uint8_t* q,
                                   float* scales) {
    auto launch = [&](auto kernel, int blocks) {
        hipLaunchKernelGGL(kernel, dim3(cols / QBLOCK / blocks, (unsigned)(rows / QBLOCK)), dim3(512 * blocks), 0, s, w, cols, q, scales);
    };
    if (cols % (2 * QBLOCK) == 0 && rows * cols * 2 >= PAIRS_FROM_BYTES) launch(quantize_blocks_kernel<2>, 2);
    else launch(quantize_blocks_kernel<1>, 1);
    return hipGetLastError();
}

}  // namespace moe355
