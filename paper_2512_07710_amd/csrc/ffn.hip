// Grouped block-scaled FP8 SwiGLU expert FFN on the CDNA4 matrix cores.
//
// Work unit: a tile of up to TOK_TILE (256) expert-sorted rows x 256 staged weight rows.  A
// small kernel turns offsets[] into the list of work units (expert, first row, feature tile,
// rows), so ragged experts need no host round trip, and orders it so that units sharing a
// weight tile are adjacent; blocks map onto the list so that each XCD (blockIdx % 8) walks a
// contiguous range, of equal numbers of units or, where the slowest XCD gains by it, of equal cost, and its L2 sees
// every weight tile once (ffn_rules.hpp).
//
// Main loop, one iteration per 128-wide K block (= one scale block):
//   * both operand tiles are copied global -> LDS by direct-to-LDS loads (no staging
//     registers) into rings of three (weights) and two (activations) 32 KiB buffers, 16-byte
//     chunks XOR-swizzled by row so that the operand reads spread over all 64 banks;
//   * partial = W_tile * X_tile^T with one v_mfma_f32_16x16x128_f8f6f4 per 16x16 sub-tile (narrow
//     tiles: two v_mfma_f32_32x32x64_f8f6f4 per 32x32 sub-tile; same sums);
//   * acc += (xs[kb][row] * ws[feature block,kb]) * partial in fp32.
// The product is taken as (features x tokens): in the accumulator layout a lane then
// owns ONE token column and 4 (16) feature rows, so the activation scale is one scalar per lane
// and sub-tile, and the 128-wide amax of the epilogue is a lane-local reduction plus two
// (one) shuffles and one exchange between the four waves that share a token.
// Activation scales are K-block major ([K/128][rows]): the lanes of a wave read
// consecutive floats of one plane.
//
// Eight waves per block: wave (wt, wf) owns 64 staged weight rows x half of the tile's groups of 32
// tokens (4 x 8 sub-tiles in a full tile: 12 operand sub-tiles feed 32 products).  The two waves of
// a SIMD, w and w + 4, take the two halves, so a tile of n groups costs every SIMD n/8 of a full
// tile's matrix work.  The K loop is instantiated for 1 to 4 groups per wave.
//
// GEMM1: staged rows of wave wf are [32 gate rows | 32 up rows] of the same features;
//        epilogue h = silu(g)*u, re-quantised to e4m3 with one scale per (row, 128 features).
// GEMM2: staged rows are 256 consecutive output features; epilogue: fp32 rows, turned through LDS so
//        that every row is stored in contiguous 256-byte pieces.
#include "ffn_common.hpp"
#include "ffn_rules.hpp"

#include <type_traits>

namespace moe355 {
namespace {

constexpr int W_ROWS = 256;                       // staged weight rows per block
constexpr int X_ROWS = TOK_TILE;                  // staged activation rows per block (256)
constexpr int W_TILE = W_ROWS * KB;                // 32 KiB: one K block of the weight tile
constexpr int X_TILE = X_ROWS * KB;                // 32 KiB: one K block of the activation tile
constexpr int NW_BUF = 3, NX_BUF = 2;              // LDS ring depths
constexpr int X_RING = NW_BUF * W_TILE;            // byte offset of the activation ring
constexpr int NTHREADS = 512;
constexpr int CODES_LD = 128 + 16;                  // bytes from row to row of the LDS tile of hidden codes
// ------------------------------------------------------------------ work list
// An expert with c rows gets ceil(c/h) row tiles, h the launch's tile height, ordered (expert, feature tile, row tile).  Units
// that share a weight tile are thus neighbours and, when they do the same amount of work, the blocks
// that run them side by side on one XCD advance in step and hit each other's lines in that XCD's L2
// (a few K steps of skew already exceed what the L2 retains, and the shared tile is then fetched
// again from HBM).
// The lanes of a wave as deal() wants them: lane x has XCD x's number, lane NXCD the one after the last.
struct WaveLanes {
    int lane;
    template <class F, class... A>
    __device__ auto each(F f, A... a) const { return f(min(lane, NXCD), a...); }
    __device__ int next(int v) const { return from_lanes<0x101, 0xf>(v); }       // row_shl 1
    __device__ int last(int v) const { return __builtin_amdgcn_readlane(v, NXCD); }
    __device__ float most(float t) const {                     // row_shr 1, 2, 4: lane 7 has the largest of the eight (none is negative)
        t = fmaxf(t, __int_as_float(from_lanes<0x111, 0xf>(__float_as_int(t))));
        t = fmaxf(t, __int_as_float(from_lanes<0x112, 0xf>(__float_as_int(t))));
        t = fmaxf(t, __int_as_float(from_lanes<0x114, 0xf>(__float_as_int(t))));
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), NXCD - 1));
    }
    __device__ int sum(int v) const { return __builtin_amdgcn_readlane(wave_scan(v), NXCD - 1); }
    __device__ bool any(bool b) const { return (__ballot(b) & ((1ull << NXCD) - 1)) != 0; }
    __device__ void put(int32_t* to, int v, int n) const {
        if (lane < n) to[lane] = v;
    }
};
// What every block of a list works out for itself from the rows of all experts (thread tid has those of expert tid): the height of the
// tiles, and how many there are.  empty: list 1 stays so unless the batch is concentrated, see DOWN_SKEW_UNITS.
struct ListPlan { int h, tiles; bool empty; };
__device__ inline ListPlan plan_list(int rows_t, int list, const ListShape& shape, bool choose) {
    constexpr int SUMS = HEIGHTS + 2, WAVES = MAX_E / 64;      // tiles at each height, groups of 32 rows, tiles of 64
    __shared__ int32_t s_sums[WAVES][SUMS];
    const int tid = threadIdx.x;
#pragma unroll
    for (int j = 0; j < SUMS; ++j) {
        if (shape.one_height && j > 0 && j <= HEIGHTS) continue;
        const int h = j < HEIGHTS ? tile_height(j) : j == HEIGHTS ? 32 : STREAM_ROWS;
        const int sum = wave_scan((rows_t + h - 1) / h);
        if ((tid & 63) == 63) s_sums[tid >> 6][j] = sum;
    }
    __syncthreads();
    int sums[SUMS], tiles[HEIGHTS];
#pragma unroll
    for (int j = 0; j < SUMS; ++j) sums[j] = s_sums[0][j] + s_sums[1][j] + s_sums[2][j] + s_sums[3][j];
#pragma unroll
    for (int j = 0; j < HEIGHTS; ++j) tiles[j] = sums[j];
    const int h = list_height(shape, tiles, sums[HEIGHTS]);
    int total = tiles[0];                                      // at the chosen height
#pragma unroll
    for (int j = 1; j < HEIGHTS; ++j) total = h == tile_height(j) ? tiles[j] : total;
    return {h, total, choose && list == 1 && sums[HEIGHTS + 1] <= 2 * tiles[0]};
}
// One block for each list l (0: gate/up, 1: down) deals it to the XCDs, beside the blocks that write its units (the first expert's block
// dealing before it wrote its own: passes of 656 x 4 tokens of 32 experts, 1024 x 512, 40.6 us / 40.0 with a block for it, 600 x 4 39.5 /
// 39.0, 2000 x 4 of 16, 1536 x 1024 93.3 / 92.9; without any dealing 39.5, 38.8 and 92.7).
__device__ inline void deal_list(const int32_t* __restrict__ offsets, int E, int list, const ListShape& shape, bool choose,
                                 Queue* __restrict__ queue, Rest* __restrict__ rest) {
    constexpr int WAVES = MAX_E / 64;
    __shared__ int32_t s_scan[WAVES], s_cost[WAVES];
    __shared__ Cuts s_cuts;
    const int tid = threadIdx.x, wave = tid >> 6, n_ft = shape.n_ft;
    const int rows_t = tid < E ? offsets[tid + 1] - offsets[tid] : 0;
    const ListPlan plan = plan_list(rows_t, list, shape, choose);
    if (plan.empty) {
        if (tid < NXCD) queue->fixed[tid] = 0;
        if (tid == 0) queue->total = queue->helpers = 0;
        return;
    }
    const int units = plan.tiles * n_ft;
    if (units > CUS) {                                         // (a round or less is dealt by numbers: no cuts)
        const int nt_t = (rows_t + plan.h - 1) / plan.h, cost_t = tiles_share(nt_t, (rows_t + 31) / 32);
        int tiles_to = wave_scan(nt_t), cost_to = wave_scan(cost_t), cost_all = 0;    // up to and with expert tid, first in its wave
        if ((tid & 63) == 63) {
            s_scan[wave] = tiles_to;
            s_cost[wave] = cost_to;
        }
        if (tid <= NXCD) no_cut(s_cuts, tid, units);
        __syncthreads();
        for (int w = 0; w < WAVES; ++w) {
            if (w < wave) tiles_to += s_scan[w];
            if (w < wave) cost_to += s_cost[w];
            cost_all += s_cost[w];
        }
        if (nt_t > 0) cut_expert(s_cuts, nt_t, tiles_to, cost_t, cost_to, cost_all, n_ft, units);
        __syncthreads();
    }
    if (wave == 0) deal(WaveLanes{tid}, s_cuts, units, list_blocks(shape.capacity) / NXCD, *queue);
    if (tid < NXCD) rest[tid].taken = 0;
}
// Block (e, l) writes the units of expert e into list l; every block recomputes the tile counts of all experts for its base index and
// the height.
__device__ inline void build_work(const int32_t* __restrict__ offsets, int E, int e, int list, const ListShape& shape, bool choose,
                                  Work* __restrict__ work) {
    constexpr int WAVES = MAX_E / 64;
    __shared__ int32_t s_scan[WAVES], s_base;
    const int tid = threadIdx.x, wave = tid >> 6;
    const int n_ft = shape.n_ft;
    const int rows_t = tid < E ? offsets[tid + 1] - offsets[tid] : 0;
    const ListPlan plan = plan_list(rows_t, list, shape, choose);
    if (plan.empty) return;
    const int h = plan.h, before = wave_scan((rows_t + h - 1) / h);    // tiles up to expert tid, in its wave
    if ((tid & 63) == 63) s_scan[wave] = before;
    __syncthreads();
    if (tid == e) {
        int base = before - (rows_t + h - 1) / h;
        for (int w = 0; w < wave; ++w) base += s_scan[w];
        s_base = base;
    }
    __syncthreads();
    const int start = offsets[e], cnt = offsets[e + 1] - start;
    const int nt = (cnt + h - 1) / h;
    if (nt == 0) return;
    const int base = s_base * n_ft;
    for (int idx = tid; idx < nt * n_ft; idx += 256) {
        const int f = idx / nt, i = idx - f * nt;
        Work w;
        split_rows(cnt, nt, i, w);
        w.expert = e;
        w.row0 += start;
        w.ft = f;
        work[base + idx] = w;
    }
}

struct RestCounts {
    Rest* rest;
    __device__ int take(int x) const { return __hip_atomic_fetch_add(&rest[x].taken, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ int taken(int y) const { return __hip_atomic_load(&rest[y].taken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

// ------------------------------------------------------------------ helpers
// The matrix instructions are written as volatile asm so that they stay exactly where the
// source puts them: the schedule below relies on it.  A product over a whole K block at once, or over its first half (new) and
// its second (acc).
__device__ inline void mfma_16(v4f& t, const v8i& a, const v8i& b) {
    // "+v", although t is only written: the product registers then stay where they are through the whole K loop
    asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, 0" : "+v"(t) : "v"(a), "v"(b) : "memory");
}
__device__ inline void mfma_new(v16f& t, const v8i& a, const v8i& b) {
    asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, 0" : "=&v"(t) : "v"(a), "v"(b) : "memory");
}
__device__ inline void mfma_acc(v16f& t, const v8i& a, const v8i& b) {
    asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, %0" : "+v"(t) : "v"(a), "v"(b) : "memory");
}
// An empty volatile asm that "rewrites" x: uses of x after it cannot move above it, and
// values feeding x cannot move below it.
#define PIN(x) asm volatile("" : "+v"(x))

// A tile's hidden codes go out through LDS, 128 contiguous bytes of a row from 8 lanes: straight from the accumulator layout a
// store instruction carries 8 bytes for each of 32 rows (gate/up, us: 64 experts x 5120 x 1536 at 1030 rows 964 / 951, 128 x 2048 x 768
// at 420 198 / 190, 16 x 3072 x 2048 at 224 58.9 / 55.8, of which 0.5..1.5 % is the earlier start of the first weights).
__device__ inline void store_codes(uint8_t* __restrict__ hq, const uint8_t* s_codes, const Work& wk, int f0, int NOUT, int tid) {
    for (int i = tid; i < wk.nrows * 8; i += NTHREADS)
        *reinterpret_cast<uint4*>(hq + (size_t)(wk.row0 + (i >> 3)) * NOUT + f0 + (i & 7) * 16) =
            *reinterpret_cast<const uint4*>(s_codes + (i >> 3) * CODES_LD + (i & 7) * 16);
}

// sixteen bytes of an output row, past the caches or through them
template <bool PAST>
__device__ inline void put_row(float* dst, const v4f& v) {
    if (PAST) __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(dst));
    else *reinterpret_cast<v4f*>(dst) = v;
}

// ------------------------------------------------------------------ operand copies
// What one wave brings of every K block: staged weight rows [32w, 32w+32) and staged activation rows [32w, 32w+32).
struct Feed {
    uint32_t lds_rows;                                         // LDS address of this wave's rows in ring slot 0
    uint32_t w_off[2], x_off[4];                               // per lane: byte offset of its 16-byte chunk in copies 0,1 / 0..3
    const uint8_t* w_base[2];                                  // weight copies 0,1 and copies 2,3 (the same lane offsets again)
    const uint8_t* x_base;
    int x_copies;                                              // activation copies that carry rows of the tile
};

// Copy J of K block kb goes out if J < n.  The condition is a scalar branch inside the asm: the compiler's control flow
// stays a straight line, which the register allocation of the K loop depends on (with C++ conditions around the copies
// the loop spills).
#define COPY_IF(J, N, LDS, VOFF, SBASE, CACHE)                                                             \
    asm volatile("s_mov_b32 m0, %0\n\ts_cmp_gt_i32 %3, %4\n\ts_cbranch_scc0 .Lskip%=\n\t"                  \
                 "global_load_lds_dwordx4 %1, %2" CACHE "\n.Lskip%=:"                                              \
                 :: "s"(LDS), "v"(VOFF), "s"(SBASE), "s"(N), "n"(J) : "memory", "scc")
// ONCE: weights that few other tiles read go past the caches (non-temporal: a block stream of 128-byte row pieces into LDS reaches
// 6.0..6.6 TB/s that way and 5.3..5.9 through them)
template <bool ONCE, int J>
__device__ __forceinline__ void copy_w1(const Feed& f, int kb, int wslot, int n) {
    if (ONCE) COPY_IF(J, n, f.lds_rows + wslot * W_TILE + J * 8 * KB, f.w_off[J & 1], f.w_base[J >> 1] + (size_t)kb * KB, " nt");
    else COPY_IF(J, n, f.lds_rows + wslot * W_TILE + J * 8 * KB, f.w_off[J & 1], f.w_base[J >> 1] + (size_t)kb * KB, "");
}
template <int J>
__device__ __forceinline__ void copy_x1(const Feed& f, int kb, int xslot, int n) {
    COPY_IF(J, n, f.lds_rows + X_RING + xslot * X_TILE + J * 8 * KB, f.x_off[J], f.x_base + (size_t)kb * KB, "");
}
#undef COPY_IF
template <bool ONCE>
__device__ __forceinline__ void copy_w(const Feed& f, int kb, int wslot, int n = 4) {
    copy_w1<ONCE, 0>(f, kb, wslot, n);
    copy_w1<ONCE, 1>(f, kb, wslot, n);
    copy_w1<ONCE, 2>(f, kb, wslot, n);
    copy_w1<ONCE, 3>(f, kb, wslot, n);
}
__device__ __forceinline__ void copy_x(const Feed& f, int kb, int xslot) {
    copy_x1<0>(f, kb, xslot, f.x_copies);
    copy_x1<1>(f, kb, xslot, f.x_copies);
    copy_x1<2>(f, kb, xslot, f.x_copies);
    copy_x1<3>(f, kb, xslot, f.x_copies);
}

// ------------------------------------------------------------------ K loop of a full tile
struct Tile {
    uint32_t lds0;                                             // LDS address of ring slot 0
    int nkb;
    uint32_t a_row, b_row;                                     // LDS byte offset of the lane's row in weight / activation slot 0
    int l16, quad;                                             // row of a 16-row operand tile; quarter of its K block
    int row, n_rows;                                           // the wave's first token row, plus the lane; rows of a scale plane
    const uint8_t* act_s;
    const float *sa, *sb;                                      // weight scales of the wave's gate / up rows (or both the same)
};

// The products of a K block, four tiles of 16 weight rows x two tiles of 16 tokens for each group of 32, in the order they are made: token
// tile by token tile, the weights forwards and backwards in turn, so that each product shares an operand with the one before (energy,
// see k_loop).  Forwards by the first token tile and by the last: the last one's weights are replaced in the order in which the next K
// block wants them.
struct Product { int weights, tokens; };
constexpr Product product(int m) {
    const int tokens = m >> 2, j = m & 3;
    return {tokens > 0 && tokens % 2 == 0 ? 3 - j : j, tokens};
}

// One wave: 64 staged weight rows (four tiles of 16) x NTS groups of 32 tokens (two tiles each), 8*NTS products per K block, one
// v_mfma_f32_16x16x128_f8f6f4 and four multiply-adds a lane each.
//
// With many rows this kernel runs at the power cap, so what counts is the energy of a product.  From registers alone, with the
// multiply-adds, codes of quantised Gaussians, TFLOP/s: pairs of 32x32x64 3500 in any order, 16x16x128 3725 to 3790, in the order above
// 3822 (3680 to 3730 on random bits: mfma_loop in probe.hip, where pairs of 32x32x64 reached 3460).  Here, with the same
// sums bit for bit (inside an instruction the lane groups get their 16-byte chunks in the order in which two 32x32x64 meet them, as in
// ffn_few.hip), against pairs of 32x32x64, us: linear 8192 x 7168 x 8192 486 / 475; 32768 tokens of
// 7168 x 2048, 256 experts, gate/up 6940 / 6915, down 4370 / 4335; 4096 tokens of 5120 x 1536, 128 experts of 257..261 rows, 544 /
// 546 and 350 / 343; 3000 x 6 of 2048 x 768 102.0 / 100.5 and 77.6 / 75.9.  The clock rises by what the energy falls, less 5 % more
// cycles for twice the instructions and for handing out the scales.  Tried and level or worse: weight tile by weight tile, operands
// requested eleven products ahead instead of seven, a raised wave priority around the matrix instructions (1..3 %).
//
// Pipeline.  K block kb of the weight tile lives in ring slot kb % 3, of the activation tile in slot kb % 2.  Each wave
// passes ONE barrier per K block, after its last LDS read of block kb, behind the first product of its last token group: the pipe
// has that one to work on while the waves meet (in front of it: 1.2 % more cycles).  Behind the barrier block kb+1 is complete in LDS
// and the slots of block kb are free.  The copies that
// refill them follow: activation block kb+2, then weight block kb+3 - always in that order, so that "all but the newest
// four copies have landed" is exactly "everything but the weight block two steps ahead".  They go out one behind every
// second product (activations over the last group, weights over the first group of the next step; NTS = 1 has
// no products to spare and sends the weights at the end of the step), so that the wave does not sit at the issue of a
// copy while the queue drains (in two bursts of four the gate/up projection ran 4 % slower).  The last group's products
// already fetch the first operands of block kb+1 into registers: the weight operands a[] stay for a whole step and are replaced one
// by one behind their last product, the token operands go through two register sets in turn (three for NTS = 3, so that a step always
// starts with set 0).
template <int NTS, bool GATED, bool ONCE>
__device__ __forceinline__ void k_loop(const Tile& t, const Feed& f, v4f (&acc)[4][8]) {
    const int nkb = t.nkb;
    // LDS byte address of a lane's first operand chunk relative to a ring slot; its second is four chunks on, that address with bit 6
    // flipped (the swizzle is an exclusive or of the chunk number)
    const int first = (t.quad & 1) * 2 + (t.quad >> 1);
    const uint32_t off0 = (uint32_t)(first ^ (t.l16 & 7) ^ ((t.l16 >> 3) & 1)) << 4;
    const uint32_t a00 = t.lds0 + t.a_row + off0, b00 = t.lds0 + t.b_row + off0;
    auto read_op = [&](v8i& o, uint32_t at, int plus) { o = lds_operand(at, at ^ 64, plus); };
    auto read_group = [&](v8i (&o)[2], uint32_t at, int plus) {
        read_op(o[0], at, plus);
        read_op(o[1], at, plus + 16 * KB);
    };
    // activation scales of this wave's token columns (K-block major: one plane per K block), by buffer loads whose
    // range check covers the token columns past the end of the plane (they read 0 and are never stored): one address
    // register for all groups.  Issued as asm; the data is only touched behind a vmcnt wait.
    // A load fetches the scales of 64 tokens, four tiles; each tile's sixteen are then handed to all four lane groups by swaps of rows
    // and of halves.
    constexpr int NXS = (NTS + 1) / 2;
    const uint32_t xs_at = 4u * (uint32_t)t.row;
    const size_t plane = (size_t)t.n_rows * 4;
    float xs_n[NXS], xs[NXS * 4];
#pragma unroll
    for (int i = 0; i < NXS; ++i) xs_n[i] = 0.f;
    auto xs_load = [&](int kb, int go) {                       // scalar condition inside the asm, as in COPY_IF
        const uint64_t base = (uint64_t)(uintptr_t)(t.act_s + (size_t)kb * plane);
        v4i rsrc;
        rsrc[0] = (int)(uint32_t)base;
        rsrc[1] = (int)(uint32_t)((base >> 32) & 0xFFFFu);
        rsrc[2] = (int)(uint32_t)min(plane, (size_t)0xFFFFFFFFu);
        rsrc[3] = 0x00020000;                                  // raw 32-bit data
#pragma unroll
        for (int i = 0; i < NXS; ++i)
            asm volatile("s_cmp_lg_u32 %3, 0\n\ts_cbranch_scc0 .Lskip%=\n\tbuffer_load_dword %0, %1, %2, 0 offen offset:%4\n.Lskip%=:"
                         : "+v"(xs_n[i]) : "v"(xs_at), "s"(rsrc), "s"(go), "n"(i * 256) : "memory", "scc");
    };
    auto xs_take = [&]() {
#pragma unroll
        for (int i = 0; i < NXS; ++i)
            asm volatile("v_mov_b32 %0, %4\n\tv_mov_b32 %1, %4\n\ts_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\t"
                         "s_nop 1\n\tv_mov_b32 %2, %0\n\tv_mov_b32 %3, %1\n\ts_nop 1\n\t"
                         "v_permlane32_swap_b32 %0, %2\n\tv_permlane32_swap_b32 %1, %3"
                         : "=&v"(xs[4 * i]), "=&v"(xs[4 * i + 1]), "=&v"(xs[4 * i + 2]), "=&v"(xs[4 * i + 3]) : "v"(xs_n[i]));
    };
    xs_load(0, 1);
    if (nkb > 1) {                                             // weight block 1 is not waited for
        copy_w<ONCE>(f, 1, 1);
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    xs_take();
    if (nkb > 1) {
        xs_load(1, 1);
        copy_x(f, 1, 1);
    }
    if (nkb > 2) copy_w<ONCE>(f, 2, 2);
    constexpr int NB = NTS == 3 ? 3 : 2;                      // register sets of token operands
    v8i a[4], b[NB][2];
    read_group(b[0], b00, 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) read_op(a[s], a00, s * 16 * KB);
    float wsc[2];                                              // weight scales of the block being folded, in scalar registers
    asm volatile("s_load_dword %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0\n\ts_waitcnt lgkmcnt(0)"
                 : "=&s"(wsc[0]), "=&s"(wsc[1]) : "s"(t.sa), "s"(t.sb) : "memory");
    auto load_wsc = [&](float (&w)[2], int kb) {               // issued by hand; complete at the barrier that follows
        const float *const at_a = t.sa + kb, *const at_b = t.sb + kb;
        asm volatile("s_load_dword %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0" : "=&s"(w[0]), "=&s"(w[1]) : "s"(at_a), "s"(at_b) : "memory");
    };
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int tt = 0; tt < 2 * NTS; ++tt)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[s][tt][r] = 0.f;
    // product m is held in T[m & 3] until it is folded behind product m + 2; the last two of a K block behind the first two of the next
    // (at first: zeros, folded with scale 0)
    v4f T[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) T[s][r] = 0.f;
    float sc = 0.f;                                            // scale being folded with

    auto scale = [&](float x, float w) {                       // w * x at this place (see PIN)
        float r;
        asm volatile("v_mul_f32 %0, %1, %2" : "=v"(r) : "s"(w), "v"(x));
        return r;
    };
    // fold the product of weight tile S and token tile TT, held in T[J], into its accumulator
#define FOLD(J, S, TT, SCV)                                                                     \
    do {                                                                                        \
        const float scv_ = (SCV);                                                               \
        PIN(T[J]);                                                                              \
        _Pragma("unroll") for (int r = 0; r < 4; ++r)                                           \
            acc[S][TT][r] = fmaf(scv_, T[J][r], acc[S][TT][r]);                                 \
        PIN(acc[S][TT]);                                                                        \
    } while (0)

    int wslot = 0;                                             // ring slot of weight block kb
    int kb = 0;
    // Where a loop lies is worth up to 6 % either way, and what other code of the kernel happens to make of it changes with every edit.  So
    // gate/up loops start on a multiple of 64 bytes, the others 28 bytes past one, with four groups 36.  us at 0 / 20 / 24 / 28 past: down
    // projection of 16 experts, 2048 x 2048, of 150 rows 30.0 / 30.1 / 30.0 / 29.2 (where an edit elsewhere left it 30.0), of 165 rows 30.1 /
    // 30.3 / 30.0 / 29.5; linear 473 x 3712 x 9216 31.0 / 31.7 / 31.8 / 30.8, 700 x 4096 x 8192 34.7 / 35.3 / 35.5 / 34.5.  Where they lay
    // before / at 28 / with four groups at 36: linear 170 x 7168 x 32768 62.9 / 60.6 / 60.5, 12727 x 4864 x 14208 832 / 838 / 833; layers
    // of 250 rows an expert and more level.
    if (GATED) asm volatile(".p2align 6");
    else asm volatile(".p2align 6\n\t.rept %0\n\ts_nop 0\n\t.endr" :: "n"(NTS < 4 ? 7 : 9));
    do {                                                       // (K >= 128: at least one block)
        const int wnext = (wslot == NW_BUF - 1) ? 0 : wslot + 1;
        const int wprev = (wslot == 0) ? NW_BUF - 1 : wslot - 1;             // slot of block kb-1 = of block kb+2
        const uint32_t sX = b00 + (kb & 1) * X_TILE;                         // block kb
        const uint32_t sWn = a00 + wnext * W_TILE;                           // block kb+1
        const uint32_t sXn = b00 + ((kb & 1) ^ 1) * X_TILE;                  // block kb+1
        const int kn = min(kb + 1, nkb - 1);
        float wsc_n[2];                                        // weight scales of block kb+1
        const int more = all_ones_if_less(kb + 2, nkb);        // is there a block kb+2?
        const int nx = f.x_copies & more;                      // copies of activation block kb+2
        const int nw = 4 & more & all_ones_if_less(0, kb);     // copies of weight block kb+2 (the prologue sent block 2)
#pragma unroll
        for (int m = 0; m < 8 * NTS; ++m) {
            const int ts = m >> 3, q = m & 7;
            const int bi = ts % NB, bnext = ts + 1 < NTS ? (ts + 1) % NB : NTS == 1 ? 1 : 0;
            const bool last = ts == NTS - 1;
            if (NTS == 1 && m == 0) load_wsc(wsc_n, kn);
            mfma_16(T[m & 3], a[product(m).weights], b[bi][q >> 2]);
            if (last && q == 0) {
                // all of this wave's reads of block kb have been issued; wait for them and for the
                // copies that must be complete (all of them in the last two steps), then meet the other waves
                asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 .Lmore%=\n\t"
                             "s_waitcnt vmcnt(0)\n.Lmore%=:" :: "s"(more) : "memory", "scc");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if (NTS > 1 && m == 0) copy_w1<ONCE, 0>(f, kb + 2, wprev, nw);
            if (NTS > 1 && m == 2) copy_w1<ONCE, 1>(f, kb + 2, wprev, nw);
            if (NTS > 1 && m == 4) copy_w1<ONCE, 2>(f, kb + 2, wprev, nw);
            if (NTS > 1 && m == 6) copy_w1<ONCE, 3>(f, kb + 2, wprev, nw);
            if (!last && q == 1) read_group(b[bnext], sX, (ts + 1) * 32 * KB);
            if (last && q == 1) read_group(b[bnext], sXn, 0);
            if (NTS > 1 && m == (NTS > 2 ? 9 : 1)) {
                // behind operand reads that are not waited for until six products later (a scalar load in
                // flight turns the next wait for an LDS read into a wait for everything)
                load_wsc(wsc_n, kn);
            }
            if (last && q == 1) copy_x1<0>(f, kb + 2, kb & 1, nx);
            if (last && q == 3) copy_x1<1>(f, kb + 2, kb & 1, nx);
            if (last && q == 5) copy_x1<2>(f, kb + 2, kb & 1, nx);
            if (last && q == 7) copy_x1<3>(f, kb + 2, kb & 1, nx);
            if (last && q >= 4) read_op(a[q - 4], sWn, (q - 4) * 16 * KB);   // its last product is on its way
            // The four multiply-adds of product m-2 sit behind product m: its result has left the matrix pipe (two more
            // instructions have been issued since), and the vector ALU works in the shadow of the one just issued.
            if (m < 2) {
                FOLD(m + 2, m + 2, 2 * NTS - 1, sc);
            } else {
                const Product p = product(m - 2), before = product(m < 3 ? 0 : m - 3);
                if (((m - 2) & 3) == 0 || (GATED && p.weights / 2 != before.weights / 2))
                    sc = scale(xs[p.tokens], wsc[GATED ? p.weights / 2 : 0]);
                FOLD((m - 2) & 3, p.weights, p.tokens, sc);
            }
            if (m == 8 * NTS - 1) {
                if (GATED) sc = scale(xs[2 * NTS - 1], wsc[1]);
                xs_take();                                     // block kb+1: landed before the barrier above
                asm volatile("s_mov_b32 %0, %2\n\ts_mov_b32 %1, %3" : "=&s"(wsc[0]), "=&s"(wsc[1]) : "s"(wsc_n[0]), "s"(wsc_n[1]));
                xs_load(kb + 2, more);
                if (NTS == 1) {
                    copy_w<ONCE>(f, kb + 3, wslot, 4 & all_ones_if_less(kb + 3, nkb));
                    b[0][0] = b[1][0];
                    b[0][1] = b[1][1];
                }
            }
        }
        wslot = wnext;
    } while (++kb < nkb);
    // the last two products: wait out the matrix pipe, then fold them
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
    FOLD(2, 2, 2 * NTS - 1, sc);
    FOLD(3, 3, 2 * NTS - 1, sc);
#undef FOLD
}

// ------------------------------------------------------------------ GEMM kernel
// GATED = true : Wa = W1, Wb = W3 [E, NOUT, K]; feature tile = 128 features (gate + up rows)
// GATED = false: Wa = W2 [E, NOUT, K]; feature tile = 256 output features
// act [N, K] u8 are the expert-sorted activations; act_s [K/128][N] f32 their scales, K-block major.
// GATHER (gate/up only): act [n_tok, K] is in TOKEN order and sorted row p reads the codes of token
// perm[p] / fan (clamped to the last token, so that a foreign perm cannot address outside act): the
// expert-ordered copy of the codes is never materialised.  The scales act_s
// [K/128][n_rows] are in sorted order in both cases (they are 1/128 of the data; a lane-scattered
// scale read per K step would cost more than it saves).
// PAST: y_perm goes past the caches (down_goes_past, linear_goes_past).  An instance of its own: with both forms in one, the layers of the other took
// 0.3 % longer.
template <bool GATED, bool GATHER, bool LINEAR, bool PAST = false>
__global__ __launch_bounds__(NTHREADS, 1) void ffn_gemm(const uint8_t* __restrict__ act,
                                                        const float* __restrict__ act_s, int n_rows,
                                                        const int32_t* __restrict__ perm, int fan, int n_tok,
                                                        const Work* __restrict__ work,
                                                        const Queue* __restrict__ queue,
                                                        Rest* __restrict__ rest,
                                                        const uint8_t* __restrict__ Wa,
                                                        const uint8_t* __restrict__ Wb,
                                                        const float* __restrict__ sa,
                                                        const float* __restrict__ sb, int K, int NOUT,
                                                        uint8_t* __restrict__ hq, float* __restrict__ hs,
                                                        float* __restrict__ y_perm) {
    constexpr int FT = GATED ? 128 : 256;                      // output features per tile
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    // [3][256 weight rows][128 B] then [2][256 activation rows][128 B]: all 160 KiB.  The amax
    // exchange of the epilogue reuses the first bytes once the main loop is over.
    float* const s_amax = reinterpret_cast<float*>(smem);

    // ---- which work unit: XCD x (= blockIdx % 8) walks the contiguous range of the list that it has been dealt, and then helps the others
    const int xcd = blockIdx.x % NXCD, slot = blockIdx.x / NXCD;
    Work wk;
    if (LINEAR) {
        // one "expert" owns all n_rows rows in `fan` row tiles, and the unit is worked out here instead of read from a list
        const int tiles = fan, total = tiles * ((NOUT + FT - 1) / FT), chunk = (total + NXCD - 1) / NXCD;
        const int wi = xcd * chunk + slot;
        if (slot >= chunk || wi >= total) return;
        wk.expert = 0;
        wk.ft = wi / tiles;
        split_rows(n_rows, tiles, wi - wk.ft * tiles, wk);
    } else {
        // read together, not each where the compiler finds it needed: a round trip less at the start of every unit (passes, us, one after
        // another / this: 656 x 4 tokens of 32 experts, 1024 x 512 40.3 / 39.9, 777 x 5 of 60, 2176 x 896 107.2 / 106.5)
        int begin = queue->begin[xcd], fixed = queue->fixed[xcd], helpers = queue->helpers;
        asm volatile("" : "+s"(begin), "+s"(fixed), "+s"(helpers));
        int wi = own_unit(begin, fixed, helpers, slot);
        if (wi == NO_UNIT) return;
        if (wi == LOOK) {
            int32_t& s_unit = *reinterpret_cast<int32_t*>(smem + X_RING - 16);
            if (threadIdx.x == 0) s_unit = take_rest(*queue, RestCounts{rest}, xcd);
            __syncthreads();                                   // (the last weight slot, first copied to behind another barrier)
            wi = __builtin_amdgcn_readfirstlane(s_unit);
            if (wi < 0) return;
        }
        wk = work[wi];
    }
    const int e = wk.expert;
    const int row_end = wk.row0 + wk.nrows;                    // this tile's rows only
    const int f0 = wk.ft * FT;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int wt = wave >> 2, wf = wave & 3;                   // token half, weight-row quarter (64 rows)
    const int nkb = K / KB;
    const int nblk_out = NOUT / QBLOCK;

    // ---- copy plan: wave w brings staged weight rows [32w, 32w+32) and staged activation rows
    //      [32w, 32w+32) of every K block, 4 + 4 instructions of 8 rows each; lane i -> row i/8,
    //      LDS chunk slot i%8 which receives global chunk slot ^ (row & 7) ^ ((row >> 3) & 1): with that
    //      swizzle the operand reads below touch all 64 LDS banks evenly.
    //      Staged weight row r: GATED: features f0 + (r/64)*32 + r%32, gate (Wa) if (r/32)%2 == 0 else up (Wb).
    //      NARROW tiles (at most 64 rows, or 96, see below): wave w's 32 staged rows are 32 consecutive features of the tile
    //      (down projection) or, GATED, [16 gate rows | 16 up rows] of features f0 + 16w .. 16w+15.
    // (LINEAR: a product of 129..160 rows can have a tile as short beside a taller one; k_loop<1> in both halves, their waves in step)
    const bool narrow = !LINEAR && narrow_tile(wk);            // block-uniform
    const bool once = !LINEAR && wk.tiles <= (GATED ? GATE_UP_ONCE_TILES : DOWN_ONCE_TILES);   // as is this
    // A wave whose features all lie beyond NOUT (down projection, NOUT an odd multiple of 128: feature tile half empty)
    // copies the last 32 features again; they are multiplied and not stored.
    Feed feed;
    auto weights = [&](int kb, int slot) {
        if (once) copy_w<true>(feed, kb, slot);
        else copy_w<false>(feed, kb, slot);
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
    feed.lds_rows = lds0 + wave * 32 * KB;                     // this wave's rows inside a tile buffer
    {
        const int sub = lane >> 3, cslot = lane & 7;
        const int f_wave = GATED ? (narrow ? f0 + wave * 16 : f0 + (wave >> 1) * 32) : min(f0 + wave * 32, NOUT - 32);
        const size_t w0 = ((size_t)e * NOUT + f_wave) * (size_t)K;
        const bool split = GATED && narrow;                    // copies 0,1 gate rows and 2,3 up rows of the same features
        feed.w_base[0] = ((GATED && !narrow && (wave & 1)) ? Wb : Wa) + w0;
        feed.w_base[1] = split ? Wb + w0 : feed.w_base[0] + (size_t)16 * K;
        uint32_t chunk[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = wave * 32 + j * 8 + sub;
            chunk[j] = (cslot ^ (r & 7) ^ ((r >> 3) & 1)) << 4;
            if (j < 2) feed.w_off[j] = (uint32_t)(j * 8 + sub) * (uint32_t)K + chunk[j];
        }
        // the weights of K block 0 are on their way before the rows' tokens have been looked up
        weights(0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = min(wk.row0 + wave * 32 + j * 8 + sub, row_end - 1);   // rows past the tile repeat its last row
            const int src = GATHER ? (int)min((uint32_t)perm[p] / (uint32_t)fan, (uint32_t)(n_tok - 1)) : p - wk.row0;
            feed.x_off[j] = (uint32_t)src * (uint32_t)K + chunk[j];
        }
    }
    feed.x_base = GATHER ? act : act + (size_t)wk.row0 * K;

    // 8-row activation copies that lie wholly beyond the tile's last row are not issued at all
    // (a ragged tile then moves only the rows it has); wave-uniform
    feed.x_copies = __builtin_amdgcn_readfirstlane(max(0, min(4, (row_end - wk.row0 - wave * 32 + 7) / 8)));

    // ---- weight scales of this wave's rows (wave-uniform -> scalar loads)
    const int blk_a = GATED ? wk.ft : min(wk.ft * 2 + (narrow ? wave >> 2 : wf >> 1), nblk_out - 1);
    const float* sa_e = sa + ((size_t)e * nblk_out + blk_a) * nkb;
    const float* sb_e = GATED ? sb + ((size_t)e * nblk_out + blk_a) * nkb : sa_e;

    copy_x(feed, 0, 0);
    if (narrow) {
        // ---- NARROW tile: at most 64 rows, or 96 that are all of their expert's.  In the layout above a wave has one or two groups of tokens
        //      to multiply, the two waves of a SIMD often not the same, behind a schedule made for eight groups.  Here
        //      wave w multiplies the 32 staged weight rows it copies itself by the tile's two or three groups of 32 token
        //      columns (two matrix instructions each per K block), so the matrix work is spread over every wave
        //      and the tile runs at the speed its weight tile streams in.  Same rings, same copy order, same
        //      barrier per K block as the full tiles; nothing is overlapped by hand - the copies are the bound.
        //      Two groups against k_loop<1> and weights through the caches, us: gate/up of 64 experts x 4096 x 1408 at 24 rows 117 / 137, at
        //      58 125 / 145, 256 x 7168 x 2048 at 12 rows 1101 / 1260; down at 50 rows 83 / 88 and 754 / 799.  Three groups against
        //      k_loop<2> beside k_loop<1>, gate/up | down: 60 experts x 2176 x 896 at 65 rows 52.5 / 54.2 | 39.8 / 40.9, 64 x 4096 x 1408
        //      at 62 132.6 / 136.8 | 84.2 / 84.6, at 80 148.9 / 152.2 | 90.1 / 91.9, 256 x 7168 x 2048 at 94 1346 / 1361 | 809 / 826.  Four
        //      are no better (at 106 rows 164.2 / 160.0 | 105.9 / 98).
        const uint32_t off00 = (uint32_t)((half * 2) ^ (l32 & 7) ^ ((l32 >> 3) & 1)) << 4;
        const uint32_t a00 = lds0 + (uint32_t)(wave * 32 + l32) * KB + off00;
        const uint32_t b00 = lds0 + (uint32_t)(X_RING + l32 * KB) + off00;
        auto run = [&](auto groups) __attribute__((always_inline)) {
            constexpr int NG = decltype(groups)::value;
            uint32_t xs_i[NG];
#pragma unroll
            for (int ts = 0; ts < NG; ++ts) xs_i[ts] = 4u * (uint32_t)min(wk.row0 + ts * 32 + l32, n_rows - 1);
            const size_t plane = (size_t)n_rows * 4;
            auto xs_load = [&](float& dst, int kb, int ts) {
                const uint8_t* const at = reinterpret_cast<const uint8_t*>(act_s) + (size_t)kb * plane;
                const uint32_t off = xs_i[ts];
                asm volatile("global_load_dword %0, %1, %2" : "=v"(dst) : "v"(off), "s"(at) : "memory");
            };
            float xs_n[NG], xs_cur[NG];
            auto xs_loads = [&](int kb) {
#pragma unroll
                for (int ts = 0; ts < NG; ++ts) xs_load(xs_n[ts], kb, ts);
            };
            xs_loads(0);
            if (nkb > 1) {
                weights(1, 1);
                asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int ts = 0; ts < NG; ++ts) asm volatile("v_mov_b32 %0, %1" : "=v"(xs_cur[ts]) : "v"(xs_n[ts]));
            if (nkb > 1) {
                xs_loads(1);
                copy_x(feed, 1, 1);
            }
            if (nkb > 2) weights(2, 2);
            v16f an[NG];
#pragma unroll
            for (int ts = 0; ts < NG; ++ts)
#pragma unroll
                for (int r = 0; r < 16; ++r) an[ts][r] = 0.f;
            int wslot = 0;
            for (int kb = 0; kb < nkb; ++kb) {
                const uint32_t sW = a00 + wslot * W_TILE, sX = b00 + (kb & 1) * X_TILE;
                v8i a[2], b[NG][2];
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    a[ks] = lds_operand(sW ^ (ks * 64), sW ^ (ks * 64 + 16), 0);
#pragma unroll
                    for (int ts = 0; ts < NG; ++ts) b[ts][ks] = lds_operand(sX ^ (ks * 64), sX ^ (ks * 64 + 16), ts * 32 * KB);
                }
                float wsa, wsb;                                    // complete at the barrier below
                asm volatile("s_load_dword %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0"
                             : "=&s"(wsa), "=&s"(wsb) : "s"(sa_e + kb), "s"(sb_e + kb) : "memory");
                v16f T[NG];
#pragma unroll
                for (int ts = 0; ts < NG; ++ts) {
                    mfma_new(T[ts], a[0], b[ts][0]);
                    mfma_acc(T[ts], a[1], b[ts][1]);
                }
                // this wave's reads of block kb are done (the operands are in registers): wait for the copies that must be
                // complete (all but the weight block two steps ahead), meet the other waves, refill the freed slots
                if (kb + 2 < nkb) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                asm volatile("" : "+s"(wsa), "+s"(wsb));           // not used above this point
                float x[NG];
#pragma unroll
                for (int ts = 0; ts < NG; ++ts) {
                    x[ts] = xs_cur[ts];
                    asm volatile("v_mov_b32 %0, %1" : "=v"(xs_cur[ts]) : "v"(xs_n[ts]));
                }
                if (kb + 2 < nkb) {
                    xs_loads(kb + 2);
                    copy_x(feed, kb + 2, kb & 1);
                }
                if (kb + 3 < nkb) weights(kb + 3, wslot);
                // the matrix instructions have left the pipe by now; a few wait states more cost nothing here
                asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
                for (int ts = 0; ts < NG; ++ts) PIN(T[ts]);
                // accumulator rows 0..15 of the product (registers 0..7) are gate rows, 16..31 (registers 8..15) up rows
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float w = (GATED && r >= 8) ? wsb : wsa;
#pragma unroll
                    for (int ts = 0; ts < NG; ++ts) an[ts][r] = fmaf(x[ts] * w, T[ts][r], an[ts][r]);
                }
#pragma unroll
                for (int ts = 0; ts < NG; ++ts) PIN(an[ts]);
                wslot = (wslot == NW_BUF - 1) ? 0 : wslot + 1;
            }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();                          // every wave is done with the operand rings
            asm volatile("" ::: "memory");
            // ---- narrow epilogue.  Register r of an[ts] belongs to token row0 + ts*32 + l32 and staged row
            //      32w + (r/4)*8 + half*4 + r%4 of this wave.
            if (GATED) {
                // registers 0..7: gate of features f0 + 16w + (r/4)*8 + half*4 + r%4, registers 8..15: up of the same
                float h[NG][8];
                float amax[NG];
#pragma unroll
                for (int ts = 0; ts < NG; ++ts) {
                    amax[ts] = 0.f;
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const float v = swiglu(an[ts][r], an[ts][r + 8]);
                        h[ts][r] = v;
                        amax[ts] = fmaxf(amax[ts], fabsf(v));
                    }
                    amax[ts] = fmaxf(amax[ts], __shfl_xor(amax[ts], 32));
                    if (half == 0) s_amax[wave * NARROW_ROWS + ts * 32 + l32] = amax[ts];
                }
                __syncthreads();                                   // the 128 features of a token's group live in all 8 waves
                uint8_t* const s_codes = smem + 8 * NARROW_ROWS * 4;       // out through LDS, as from a full tile
#pragma unroll
                for (int ts = 0; ts < NG; ++ts) {
                    const int trow = ts * 32 + l32;
                    const int p = wk.row0 + trow;
                    float am = 0.f;
#pragma unroll
                    for (int w = 0; w < 8; ++w) am = fmaxf(am, s_amax[w * NARROW_ROWS + trow]);
                    const float sc = (am == 0.f) ? 1.0f : am / 448.0f;
                    const Quotient q(sc);
                    uint8_t* const dst = s_codes + trow * CODES_LD + wave * 16 + half * 4;
#pragma unroll
                    for (int r4 = 0; r4 < 2; ++r4)
                        *reinterpret_cast<uint32_t*>(dst + r4 * 8) =
                            e4m3_codes4(q, h[ts][r4 * 4], h[ts][r4 * 4 + 1], h[ts][r4 * 4 + 2], h[ts][r4 * 4 + 3]);
                    if (half == 0 && wave == 0 && p < row_end) hs[(size_t)wk.ft * n_rows + p] = sc;
                }
                __syncthreads();
                store_codes(hq, s_codes, wk, f0, NOUT, tid);
            } else {
                // a group's 32 features x 32 rows go through a region of the wave's own, so that eight lanes write 128 contiguous bytes of a
                // row (straight from the accumulators 16 bytes for each of 64: the down projections above 42.8, 86.6, 93.4 and 829 us)
                constexpr int LD = 36;
                float* const stage = reinterpret_cast<float*>(smem) + wave * (32 * LD);
                if (f0 + wave * 32 < NOUT) {
#pragma unroll
                    for (int ts = 0; ts < NG; ++ts) {
#pragma unroll
                        for (int r4 = 0; r4 < 4; ++r4)
                            *reinterpret_cast<v4f*>(stage + l32 * LD + r4 * 8 + half * 4) =
                                v4f{an[ts][r4 * 4], an[ts][r4 * 4 + 1], an[ts][r4 * 4 + 2], an[ts][r4 * 4 + 3]};
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // as in the full tiles' epilogue
                        v4f v[4];
#pragma unroll
                        for (int it = 0; it < 4; ++it) v[it] = *reinterpret_cast<const v4f*>(stage + (it * 8 + (lane >> 3)) * LD + (lane & 7) * 4);
                        const int p = wk.row0 + ts * 32 + (lane >> 3);
                        float* const dst = y_perm + (size_t)p * NOUT + f0 + wave * 32 + (lane & 7) * 4;
#pragma unroll
                        for (int it = 0; it < 4; ++it)
                            if (p + it * 8 < row_end) put_row<PAST>(dst + (size_t)(it * 8) * NOUT, v[it]);
                    }
                }
            }
        };
        if (wk.nrows <= 64) run(std::integral_constant<int, 2>{});
        else run(std::integral_constant<int, 3>{});
        return;
    }
    // ---- full tile: 32-row token groups n = ceil(rows / 32) of 3..8 (LINEAR: 2..8); waves 0..3 (token half 0) take the first ceil(n/2)
    //      of them, waves 4..7 the others.  Wave w and wave w + 4 share a SIMD, so every SIMD multiplies n groups: the
    //      matrix time of a tile follows its height in steps of 32 rows.
    const int n_grp = (wk.nrows + 31) >> 5;
    const int grp0 = wt == 0 ? 0 : (n_grp + 1) >> 1;           // this wave's first token group
    const int nts = wt == 0 ? (n_grp + 1) >> 1 : n_grp >> 1;   // and how many it has (1..4), wave-uniform
    const int l16 = lane & 15, quad = lane >> 4;
    v4f acc[4][8];                                             // k_loop<nts> defines the first 2*nts of each
    Tile tile;
    tile.lds0 = lds0;
    tile.nkb = nkb;
    tile.a_row = (uint32_t)(wf * 64 + l16) * KB;
    tile.b_row = (uint32_t)(X_RING + (grp0 * 32 + l16) * KB);
    tile.l16 = l16;
    tile.quad = quad;
    tile.row = wk.row0 + grp0 * 32 + lane;
    tile.n_rows = n_rows;
    tile.act_s = reinterpret_cast<const uint8_t*>(act_s);
    tile.sa = sa_e;
    tile.sb = sb_e;
#define LOOP(NTS)                                              \
    do {                                                       \
        if (once) k_loop<NTS, GATED, true>(tile, feed, acc);   \
        else k_loop<NTS, GATED, false>(tile, feed, acc);       \
    } while (0)
    switch (nts) {
        case 4: LOOP(4); break;
        case 3: LOOP(3); break;
        case 2: LOOP(2); break;
        default: LOOP(1); break;
    }
#undef LOOP
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                              // every wave is done with the operand rings
    asm volatile("" ::: "memory");

    // ---- epilogue.  Accumulator (s, tt, r) of this lane belongs to token
    //      row0 + grp0*32 + tt*16 + l16 and staged weight row wf*64 + s*16 + quad*4 + r.
    if (GATED) {
        // s = 0, 1 gate, s = 2, 3 up of features f0 + wf*32 + (s%2)*16 + quad*4 + r
        float h[8][8];
#pragma unroll
        for (int tt = 0; tt < 8; ++tt) {
            if (tt >= 2 * nts) break;
            float am = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float v = swiglu(acc[i >> 2][tt][i & 3], acc[2 + (i >> 2)][tt][i & 3]);
                h[tt][i] = v;
                am = fmaxf(am, fabsf(v));
            }
            am = fmaxf(am, __shfl_xor(am, 16));                // the four lane groups cover 32 features
            am = fmaxf(am, __shfl_xor(am, 32));
            if (quad == 0) s_amax[wf * X_ROWS + grp0 * 32 + tt * 16 + l16] = am;
        }
        __syncthreads();                                       // the other 96 features live in the other three waves of wt
        uint8_t* const s_codes = smem + 4 * X_ROWS * 4;        // [X_ROWS][CODES_LD], behind s_amax
#pragma unroll
        for (int tt = 0; tt < 8; ++tt) {
            if (tt >= 2 * nts) break;
            const int trow = grp0 * 32 + tt * 16 + l16;
            const int p = wk.row0 + trow;
            const float am = fmaxf(fmaxf(s_amax[trow], s_amax[X_ROWS + trow]),
                                   fmaxf(s_amax[2 * X_ROWS + trow], s_amax[3 * X_ROWS + trow]));
            const float sc = (am == 0.f) ? 1.0f : am / 448.0f;
            const Quotient q(sc);
            uint8_t* const dst = s_codes + trow * CODES_LD + wf * 32 + quad * 4;
#pragma unroll
            for (int s = 0; s < 2; ++s)
                *reinterpret_cast<uint32_t*>(dst + s * 16) =
                    e4m3_codes4(q, h[tt][s * 4], h[tt][s * 4 + 1], h[tt][s * 4 + 2], h[tt][s * 4 + 3]);
            if (quad == 0 && wf == 0 && p < row_end) hs[(size_t)wk.ft * n_rows + p] = sc;
        }
        __syncthreads();
        store_codes(hq, s_codes, wk, f0, NOUT, tid);
    } else {
        // A store instruction straight from the accumulators would carry 64 bytes for each of 16 different rows in 16-byte pieces, which the
        // memory pipeline takes as separate requests.  Each wave therefore turns its 64 x 32-token blocks through a
        // private LDS region (the operand rings are free now), two regions in turn, and writes 256 contiguous
        // bytes of a row with every 16 lanes.
        constexpr int TS_STRIDE = 68;                          // floats per staged token row: 64 + 4 of padding
        const int fcol = f0 + wf * 64;
        if (fcol < NOUT) {
#pragma unroll
            for (int ts = 0; ts < 4; ++ts) {
                if (ts >= nts) break;
                float* const stage = reinterpret_cast<float*>(smem) + (wave * 2 + (ts & 1)) * (32 * TS_STRIDE);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        *reinterpret_cast<v4f*>(stage + (h * 16 + l16) * TS_STRIDE + s * 16 + quad * 4) = acc[s][2 * ts + h];
                // the lanes of a wave run in step: once its own LDS writes have completed, every lane's have (and the
                // reads of the region used two groups ago have been consumed by their stores)
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                v4f v[8];
#pragma unroll
                for (int it = 0; it < 8; ++it)
                    v[it] = *reinterpret_cast<const v4f*>(stage + (it * 4 + (lane >> 4)) * TS_STRIDE + (lane & 15) * 4);
                const int p = wk.row0 + (grp0 + ts) * 32 + (lane >> 4);
                float* const dst = y_perm + (size_t)p * NOUT + fcol + (lane & 15) * 4;
#pragma unroll
                for (int it = 0; it < 8; ++it)
                    if (p + it * 4 < row_end) put_row<PAST>(dst + (size_t)(it * 4) * NOUT, v[it]);
            }
        }
    }
}

constexpr size_t SMEM_BYTES = NW_BUF * W_TILE + NX_BUF * X_TILE;   // 160 KiB

}  // namespace

// length of the gate/up projection's work list, behind which the down projection's lies; and room for both
static int64_t gate_up_list(const moe_dims* D) { return gate_up_streams(D) ? 0 : gate_up_units(D); }
size_t ffn_work_bytes(const moe_dims* D) {
    if (gate_up_flows(D)) return sizeof(Work);                 // (then neither projection needs a list)
    return sizeof(Work) * (size_t)(gate_up_list(D) + (down_form(D) == Down::STREAM ? 0 : down_big_units(D)) + 1);
}
size_t ffn_queue_bytes() { return 2 * (sizeof(Queue) + NXCD * sizeof(Rest)); }
size_t ffn_ticket_bytes(const moe_dims* D) { return gate_up_streams(D) && !gate_up_flows(D) ? sizeof(int32_t) * (size_t)gate_up_units(D) : 0; }
size_t ffn_h_rows_bytes(const moe_dims* D) {
    return gate_up_streams(D) && !gate_up_flows(D) ? sizeof(float) * (size_t)((int64_t)D->T * D->k) * (size_t)D->F : 0;
}

static hipError_t set_lds_limits() {
    static bool attr_set = false;
    if (attr_set) return hipSuccess;
    const void* kernels[6] = {reinterpret_cast<const void*>(&ffn_gemm<true, false, false>),
                              reinterpret_cast<const void*>(&ffn_gemm<true, true, false>),
                              reinterpret_cast<const void*>(&ffn_gemm<false, false, false>),
                              reinterpret_cast<const void*>(&ffn_gemm<false, false, false, true>),
                              reinterpret_cast<const void*>(&ffn_gemm<false, false, true>),
                              reinterpret_cast<const void*>(&ffn_gemm<false, false, true, true>)};
    for (const void* k : kernels) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SMEM_BYTES);
        if (e != hipSuccess) return e;
    }
    hipError_t e = set_stream_lds_limits();
    if (e == hipSuccess) e = set_few_lds_limits();
    if (e == hipSuccess) e = set_flow_lds_limits();
    if (e != hipSuccess) return e;
    attr_set = true;
    return hipSuccess;
}

// What the big tiles need before they start, in one launch (two took 2..3 us more of every layer): how the lists are dealt (one block
// each), the work lists (the next E*lists blocks) and, with perm, the scales of the expert-sorted rows from the per-token scales:
// out[g][p] = in[g][perm[p] / fan].
__global__ __launch_bounds__(256) void prepare_big_tiles(const int32_t* __restrict__ offsets, int E, int lists, ListShape shape0,
                                                         ListShape shape1, bool choose, Work* __restrict__ work0,
                                                         Work* __restrict__ work1, Queue* __restrict__ queues, Rest* __restrict__ rests,
                                                         const float* __restrict__ in, int T, const int32_t* __restrict__ perm,
                                                         int fan, int N, float* __restrict__ out) {
    if ((int)blockIdx.x < lists) {
        const int list = blockIdx.x;
        deal_list(offsets, E, list, list == 0 ? shape0 : shape1, choose, queues + list, rests + list * NXCD);
        return;
    }
    const int block = blockIdx.x - lists;
    if (block < E * lists) {
        const int list = block / E;
        build_work(offsets, E, block % E, list, list == 0 ? shape0 : shape1, choose, list == 0 ? work0 : work1);
        return;
    }
    const uint32_t b = block - E * lists, row_blocks = (uint32_t)((N + 255) / 256);
    const size_t g = b / row_blocks;
    const int p = (int)(b % row_blocks) * 256 + (int)threadIdx.x;
    if (p >= N) return;
    const uint32_t t = min((uint32_t)perm[p] / (uint32_t)fan, (uint32_t)(T - 1));
    out[g * N + p] = in[g * T + t];
}

// perm == nullptr: xq/xs are the expert-ordered activations [N,d], [d/128][N].
// perm != nullptr: xq/xs are in token order [T,d], [d/128][T]; sorted row p reads token perm[p] / k
//                  (the scales are first brought into sorted order in the context's workspace).
hipError_t launch_expert_ffn(moe_ctx* c, const uint8_t* xq, const float* xs, const int32_t* perm, const int32_t* offsets,
                             const uint8_t* W1, const uint8_t* W3, const uint8_t* W2, const float* s1,
                             const float* s3, const float* s2, float* y_perm) {
    const moe_dims& D = c->dims;
    hipError_t ea = set_lds_limits();
    if (ea != hipSuccess) return ea;
    Work* work = reinterpret_cast<Work*>(c->tiles);
    hipEvent_t* ev = nullptr;
    if (c->profiling && c->prof_calls < PROF_MAX_CALLS) ev = c->prof_events + 3 * c->prof_calls++;

    const int N = (int)((int64_t)D.T * D.k);
    const bool flow1 = gate_up_flows(&D), flow2 = down_flows(&D), stream1 = !flow1 && gate_up_streams(&D);
    const Down down = down_form(&D);
    const int units1 = (int)gate_up_units(&D);
    Work* work2 = work + gate_up_list(&D);                     // the down projection's list
    Queue* const queues = reinterpret_cast<Queue*>(c->queues); // and how each of them is dealt to the XCDs
    Rest* const rests = reinterpret_cast<Rest*>(queues + 2);
    if (!stream1 && !flow1) {                                  // (the streaming kernels need neither list nor sorted scales)
        const int lists = down == Down::STREAM ? 1 : 2;
        const int64_t gather = perm ? (int64_t)((N + 255) / 256) * (D.d / QBLOCK) : 0;
        hipLaunchKernelGGL(prepare_big_tiles, dim3((unsigned)((D.E + 1) * lists + gather)), dim3(256), 0, c->stream, offsets, D.E, lists,
                           gate_up_shape(&D), down_shape(&D), down == Down::EITHER,
                           work, work2, queues, rests, xs, D.T, perm, D.k, N, c->xs_sorted);
    }
    if (ev) (void)hipEventRecord(ev[0], c->stream);          // the timed interval is the GEMM kernel alone
    if (flow1) {
        hipError_t e = launch_flow_gate_up(c, xq, xs, perm, offsets, W1, W3, s1, s3);
        if (e != hipSuccess) return e;
    } else if (gate_up_few(&D)) {
        hipError_t e = launch_few_gate_up(c, xq, xs, perm, offsets, (int)max_row_tiles(&D, FEW_ROWS), W1, W3, s1, s3);
        if (e != hipSuccess) return e;
    } else if (stream1) {
        hipError_t e = launch_stream_gate_up(c, xq, xs, perm, offsets, units1, W1, W3, s1, s3);
        if (e != hipSuccess) return e;
    } else {
        auto launch = [&](auto kernel, const float* scales, int fan, int n_tok) {
            hipLaunchKernelGGL(kernel, dim3(list_blocks(units1)), dim3(NTHREADS), SMEM_BYTES, c->stream, xq, scales, N, perm, fan, n_tok, work,
                               queues, rests, W1, W3, s1, s3, D.d, D.F, c->hq, c->hs, (float*)nullptr);
        };
        if (perm) launch(ffn_gemm<true, true, false>, c->xs_sorted, D.k, D.T);
        else launch(ffn_gemm<true, false, false>, xs, 1, 1);
    }
    if (ev) (void)hipEventRecord(ev[1], c->stream);
    if (flow2) {
        hipError_t e = launch_flow_down(c, offsets, W2, s2, y_perm);
        if (e != hipSuccess) return e;
    } else if (down_few(&D)) {
        hipError_t e = launch_few_down(c, offsets, (int)max_row_tiles(&D, FEW_ROWS), W2, s2, y_perm);
        if (e != hipSuccess) return e;
    } else if (down != Down::BIG) {
        hipError_t e = launch_stream_down(c, offsets, (int)down_stream_units(&D), down == Down::EITHER ? &queues[1].total : nullptr, W2, s2, y_perm);
        if (e != hipSuccess) return e;
    }
    if (down != Down::STREAM && !flow2) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(list_blocks((int)down_big_units(&D))), dim3(NTHREADS), SMEM_BYTES, c->stream, c->hq, c->hs, N,
                               (const int32_t*)nullptr, 1, 1, work2, queues + 1, rests + NXCD, W2, (const uint8_t*)nullptr, s2,
                               (const float*)nullptr, D.F, D.d, (uint8_t*)nullptr, (float*)nullptr, y_perm);
        };
        if (down_goes_past(&D)) launch(ffn_gemm<false, false, false, true>);
        else launch(ffn_gemm<false, false, false>);
    }
    if (ev) (void)hipEventRecord(ev[2], c->stream);
    return hipGetLastError();
}

// Dense block-scaled FP8 linear layer: the down-projection kernel with a single "expert" that owns all rows.  It needs no work list:
// the two launches that made one took 10 us of the 490 of 8192 rows x 7168 x 8192.
hipError_t launch_linear(moe_ctx* c, const uint8_t* xq, const float* xs, int32_t rows, int32_t K, const uint8_t* Wq,
                         const float* ws, int32_t NOUT, float* y) {
    hipError_t ea = set_lds_limits();
    if (ea != hipSuccess) return ea;
    if (few_linear_groups(rows, NOUT)) return launch_few_linear(c, xq, xs, rows, K, Wq, ws, NOUT, y);
    if (linear_streams(rows, NOUT)) return launch_stream_linear(c, xq, xs, rows, K, Wq, ws, NOUT, y);
    const int nft = (NOUT + 255) / 256, tiles = linear_tiles(rows, nft, K / KB);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((tiles * nft + NXCD - 1) / NXCD * NXCD), dim3(NTHREADS), SMEM_BYTES,
                           c->stream, xq, xs, rows, (const int32_t*)nullptr, tiles, 1, (const Work*)nullptr,
                           (const Queue*)nullptr, (Rest*)nullptr, Wq, (const uint8_t*)nullptr, ws, (const float*)nullptr, K, NOUT,
                           (uint8_t*)nullptr, (float*)nullptr, y);
    };
    if (linear_goes_past(rows, K, NOUT)) launch(ffn_gemm<false, false, true, true>);
    else launch(ffn_gemm<false, false, true>);
    return hipGetLastError();
}

}  // namespace moe355
