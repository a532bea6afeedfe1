// The quantisation of a group of 128 columns, shared by the quantisation's own kernel (quantize.hip) and those that carry the
// token-order quantisation along in blocks of their own.
#pragma once
#include "e4m3.hpp"
#include "moe_internal.hpp"

namespace moe355 {

// Sixteen lanes own one 128-column group, 8 bf16 each: its maximum, reduced with four xor-shuffles, makes the scale.  All sixteen
// call it.
__device__ inline E4m3Coder group_coder(const u32x4& raw) {
    float amax = bf16x8_amax(raw);
    amax = fmaxf(amax, __shfl_xor(amax, 1));
    amax = fmaxf(amax, __shfl_xor(amax, 2));
    amax = fmaxf(amax, __shfl_xor(amax, 4));
    amax = fmaxf(amax, __shfl_xor(amax, 8));
    return E4m3Coder((amax == 0.f) ? 1.0f : amax / 448.0f);
}

// Group g of row r in token order.  All sixteen lanes of a live row call it.  Codes and scales go past the caches: they are read next
// by the CUs of other XCDs, from which lines that are still dirty in this one's L2 come slowly (gate/up projection of 3584 tokens x 1 of
// 64 experts, 7168 x 512, behind this: 92 us / 79 past the caches, 777 x 5 of 60, 2176 x 896 49.5 / 48.9; larger batches level).
__device__ inline void quantize_row_group(const token_quant& t, int64_t r, int g, int sub) {
    const size_t at = (size_t)r * t.cols + (size_t)g * QBLOCK + sub * 8;
    const u32x4 raw = *reinterpret_cast<const u32x4*>(t.x + at);
    const E4m3Coder coder = group_coder(raw);
    __builtin_nontemporal_store(coder.pack8(raw), reinterpret_cast<u32x2*>(t.q + at));
    if (sub == 0) __builtin_nontemporal_store(coder.s, t.scales + (size_t)g * t.rows + r);
}

// block `unit` of THREADS threads: TOKEN_QUANT_ROWS rows of THREADS/(16*TOKEN_QUANT_ROWS) groups at a time (scales leave in runs of
// 32 words)
constexpr int TOKEN_QUANT_ROWS = 32;
template <int THREADS, int PASSES>
__device__ inline void quantize_block(const token_quant& t, uint32_t unit) {
    constexpr int RPP = TOKEN_QUANT_ROWS / PASSES;             // rows per pass
    constexpr int GPB = THREADS / 16 / RPP;                    // groups per block
    const int groups = t.cols / QBLOCK, per_row = (groups + GPB - 1) / GPB;
    const int g = (int)(unit % per_row) * GPB + (int)(threadIdx.x >> 4) / RPP;
    const int64_t r0 = (int64_t)(unit / per_row) * TOKEN_QUANT_ROWS + (threadIdx.x >> 4) % RPP;
#pragma unroll
    for (int i = 0; i < PASSES; ++i)
        if (g < groups && r0 + i * RPP < t.rows) quantize_row_group(t, r0 + i * RPP, g, threadIdx.x & 15);
}
template <int THREADS, int PASSES>
inline int64_t quantize_blocks(const token_quant& t) {
    constexpr int GPB = THREADS / 16 / (TOKEN_QUANT_ROWS / PASSES);
    return t.x ? (t.rows + TOKEN_QUANT_ROWS - 1) / TOKEN_QUANT_ROWS * ((t.cols / QBLOCK + GPB - 1) / GPB) : 0;
}

}  // namespace moe355
