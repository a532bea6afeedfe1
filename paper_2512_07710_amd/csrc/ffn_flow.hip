// Block-scaled FP8 GEMMs for up to a few dozen rows per expert in persistent blocks: one continuous stream of weights per CU.
//
// The unit of work is that of the big tiles' narrow form (ffn.hip): up to 96 rows of an expert x 256 staged weight rows, eight waves,
// each of which multiplies the 32 staged rows that it brings itself (gate/up: 16 gate rows and the 16 up rows of the same features).
// What is different is what happens between units.  There a block ends: its last copies drain, its results leave, the next block finds
// its unit, looks its rows up and waits for its first weights.  Here a block of each CU walks its units, and the copies run D - 1 K blocks
// ahead of the products across the end of a unit: the next unit's first weights and rows are on their way while this one's last K
// blocks are multiplied and its results are stored.
//   * K blocks pass through a ring of D stages, 256 staged weight rows, the tile's rows and their scales, all by direct-to-LDS copies;
//     one barrier for each K block, behind which the stage before it is refilled.
//   * The tiles are worked out from the offsets in registers (ffn_rows.hpp) and the scales gathered straight from the token-order
//     planes, so that neither list nor sorted scales are needed: a launch less in front of the projection.
//   * What a unit looks up (its weight scales, which tokens its rows are) comes by copies of its own while the unit before is
//     multiplied.
//   * 16x16x128 products in ffn_few.hip's byte order, so the bits are those of the other kernels; a tile's time follows its rows in
//     steps of 16.
// The K loop has to be a straight line.  With C++ conditions around the copies (which weights go past the caches, which waves bring
// rows and which scales) the same schedule took 600 instead of 440 us for 16 tokens x 8 of 256 experts, 7168 x 2048: at 1.2 us for
// a stage of 32 KB whatever stands between a barrier and the copies behind it is time without requests.
// Bound by the weights: 16 x 8 of 256, 7168 x 2048 6.8 TB/s, 256 x 6 of 64, 4096 x 1408 6.5 TB/s.  Gate/up, us, big tiles or streaming kernel (with
// the launch that makes lists) / here: 256 tokens x 6 of 64, 4096 x 1408 124 / 114, 300 x 5 of 112, 1152 x 1280 71 / 55, 335 x 2 of 40, 3072 x 512
// 32.2 / 27.4, 16 x 8 of 256, 7168 x 2048 445 / 442; whole layers of random shapes in ffn_rules.hpp.  Four stages with tiles of 64 or 32 rows, row
// lookups behind the first weights, and waits that leave a unit's stores outstanding: level.
#include "ffn_rows.hpp"
#include "ffn_rules.hpp"

#include <type_traits>

namespace moe355 {
namespace {

constexpr int NTHR = 512;
constexpr int TILES = FLOW_ROWS / 16;                 // groups of 16 rows
constexpr int D = 3;                                  // stages
constexpr int W_STAGE = 256 * KB;                     // one K block of a unit's 256 staged weight rows
constexpr int X_STAGE = FLOW_ROWS * KB;               // of its rows
constexpr int X_COPIES = FLOW_ROWS / 8, S_COPIES = (FLOW_ROWS + 63) / 64;      // copies of the rows, and of their scales, in a stage
constexpr int AUX = X_COPIES + S_COPIES;
constexpr int NA = (AUX + 7) / 8;                     // of which a wave has so many, or one less
constexpr int STAGE = W_STAGE + X_STAGE + S_COPIES * 256;
constexpr int WS_ROW = FLOW_MAX_KB * 4;           // a row of weight scales; a unit has two
constexpr int WS_AT = D * STAGE, PERM_AT = WS_AT + 4 * WS_ROW;                 // two units' weight scales; the next unit's rows
constexpr int LDS_BYTES = PERM_AT + S_COPIES * 256;
constexpr int Y_LD = 36;                              // floats from row to row of a wave's LDS tile of outputs: 32 + 4
// copies newer than those of the K block that has to have landed, of a wave with na copies besides its weights
constexpr int newer(int na) { return (D - 2) * (4 + na); }
static_assert(FLOW_ROWS % 16 == 0 && LDS_BYTES <= 160 * 1024 && newer(NA) <= 63, "fits a CU's LDS; wait counts fit the 6-bit field");

template <class T>
__device__ inline const T* scalar(const T* p) {                // a wave-uniform pointer, in scalar registers whatever it was made of
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<const T*>((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)v) |
                                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32);
}

// The rows' K must be of D + 1 to FLOW_MAX_KB K blocks: a unit's lookups are asked for in its predecessor's first K block and read D - 1 before
// the last.
template <bool GATED, bool GATHER>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(2))) void ffn_flow(StreamArgs g) {
    constexpr int FT = GATED ? 128 : 256;                      // output features per unit
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int32_t* const s_perm = reinterpret_cast<const int32_t*>(smem + PERM_AT);

    // ---- XCD x (= blockIdx % 8) has a contiguous eighth of the units, and its blocks take them in turn
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nft = (g.NOUT + FT - 1) / FT;
    const RowTiles<true, FLOW_ROWS, 16> tiles(g, lane);
    const int total = tiles.total * nft, chunk = (total + NXCD - 1) / NXCD;
    const int xcd = blockIdx.x % NXCD, slots = gridDim.x / NXCD;
    int unit = xcd * chunk + (int)(blockIdx.x / NXCD);
    const int unit_end = min(total, (xcd + 1) * chunk);
    if (unit >= unit_end) return;

    const int l16 = lane & 15, quad = lane >> 4;
    const int sub = lane >> 3, cslot = lane & 7;
    const int nkb = g.K / KB, nblk_out = g.NOUT / QBLOCK;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
    const uint32_t sw[2] = {(uint32_t)(cslot ^ sub) << 4, (uint32_t)(cslot ^ sub ^ 1) << 4};
    const uint32_t w_off[2] = {(uint32_t)sub * (uint32_t)g.K + sw[0], (uint32_t)(8 + sub) * (uint32_t)g.K + sw[1]};
    const uint32_t plane = (uint32_t)(GATHER ? g.n_tok : g.n_rows) * 4u;
    const int full_aux = all_ones_if_less(wave, AUX - 8 * (NA - 1));            // does the wave have NA of them?

    // ---- where the copies come from
    const uint8_t *w_base[2], *a_base[NA];                     // of the K block that is copied next
    uint32_t aux_off[NA];
    uint32_t aux_step[NA];
    int once;
    auto weights_of = [&](const Tile& t, const uint8_t* (&base)[2]) {
        const int f_wave = GATED ? t.ft * FT + wave * 16 : min(t.ft * FT + wave * 32, g.NOUT - 32);
        const size_t w0 = ((size_t)t.expert * g.NOUT + f_wave) * (size_t)g.K;
        base[0] = scalar(g.Wa + w0);
        base[1] = scalar(GATED ? g.Wb + w0 : g.Wa + w0 + (size_t)16 * g.K);
    };
    auto aim_rows = [&](const Tile& t, auto perm_at) {         // perm_at(r): perm of the tile's row r < nrows
#pragma unroll
        for (int j = 0; j < NA; ++j) {
            const int a = wave + 8 * j;
            const bool rows = a < X_COPIES;
            const int r = min(rows ? a * 8 + sub : (a - X_COPIES) * 64 + lane, t.nrows - 1);
            const uint32_t row = GATHER ? min((uint32_t)perm_at(r) / (uint32_t)g.fan, (uint32_t)(g.n_tok - 1)) : (uint32_t)r;
            a_base[j] = scalar((rows ? g.act : reinterpret_cast<const uint8_t*>(g.act_s)) + (GATHER ? 0 : (size_t)t.row0 * (rows ? g.K : 4)));
            aux_off[j] = rows ? row * (uint32_t)g.K + sw[a & 1] : 4u * row;
        }
    };
#pragma unroll
    for (int j = 0; j < NA; ++j) aux_step[j] = __builtin_amdgcn_readfirstlane(wave + 8 * j < X_COPIES ? (uint32_t)KB : plane);
    // one K block of the wave's weights, and of its share of rows and scales; the conditions inside the asm, so that the K loop is a
    // straight line
    auto issue = [&](int slot) {
        const uint32_t st = lds0 + slot * STAGE;
#pragma unroll
        for (int j = 0; j < NA; ++j) {
            const int a = wave + 8 * j;
            const uint32_t to = st + W_STAGE + (a < X_COPIES ? a * 1024 : X_STAGE + (a - X_COPIES) * 256);
            if (8 * j + 8 <= X_COPIES) dma16(to, aux_off[j], a_base[j]);
            else
                asm volatile("s_mov_b32 m0, %0\n\ts_cmp_lt_i32 %3, %4\n\ts_cbranch_scc0 .Lscale%=\n\tglobal_load_lds_dwordx4 %1, %2\n\t"
                             "s_branch .Lend%=\n.Lscale%=:\n\ts_cmp_lt_i32 %3, %5\n\ts_cbranch_scc0 .Lend%=\n\t"
                             "global_load_lds_dword %1, %2\n.Lend%=:"
                             :: "s"(to), "v"(aux_off[j]), "s"(a_base[j]), "s"(a), "n"(X_COPIES), "n"(AUX) : "memory", "scc");
            a_base[j] += aux_step[j];
        }
        asm volatile("s_mov_b32 m0, %0\n\ts_cmp_lg_u32 %5, 0\n\ts_cbranch_scc0 .Lcached%=\n\t"
                     "global_load_lds_dwordx4 %1, %3 nt\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3 nt\n\t"
                     "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4 nt\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %4 nt\n\ts_branch .Lend%=\n.Lcached%=:\n\t"
                     "global_load_lds_dwordx4 %1, %3\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\t"
                     "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %4\n.Lend%=:"
                     :: "s"(st + wave * (32 * KB)), "v"(w_off[0]), "v"(w_off[1]), "s"(w_base[0]), "s"(w_base[1]), "s"(once) : "memory", "scc");
        w_base[0] += KB;
        w_base[1] += KB;
    };
    // what a unit has to look up, brought by waves 5 to 7: its two rows of weight scales, and which tokens its rows are
    auto look_up = [&](const Tile& t, int buffer) {
        const uint32_t at = lds0 + WS_AT + buffer * (2 * WS_ROW);
        if (wave == 5 || wave == 6) {
            const int row = GATED ? t.ft : min(t.ft * 2 + wave - 5, nblk_out - 1);
            const float* const s = (GATED && wave == 6 ? g.sb : g.sa) + ((size_t)t.expert * nblk_out + row) * nkb;
            for (int k0 = 0; k0 < nkb; k0 += 64) dma4(at + (wave - 5) * WS_ROW + k0 * 4, 4u * (uint32_t)min(k0 + lane, nkb - 1), scalar(s));
        }
        if (GATHER && wave == 7) {
#pragma unroll
            for (int j = 0; j < S_COPIES; ++j) dma4(lds0 + PERM_AT + j * 256, 4u * (uint32_t)min(j * 64 + lane, t.nrows - 1), scalar(g.perm + t.row0));
        }
    };

    auto tile_of = [&](int u) {                                // in scalar registers, whatever the compiler makes of find's division
        const Tile t = tiles.find(g, u, nft);
        return Tile{__builtin_amdgcn_readfirstlane(t.expert), __builtin_amdgcn_readfirstlane(t.ft), __builtin_amdgcn_readfirstlane(t.row0),
                    __builtin_amdgcn_readfirstlane(t.nrows), __builtin_amdgcn_readfirstlane(t.tiles)};
    };
    Tile cur = tile_of(unit), next = cur;
    int buffer = 0;
    const uint8_t* w_next[2];
    weights_of(cur, w_base);
    once = all_ones_if_less(cur.tiles, 2);
    aim_rows(cur, [&](int r) { return g.perm[cur.row0 + r]; });
    look_up(cur, 0);
#pragma unroll
    for (int i = 0; i < D - 1; ++i) issue(i);
    int rslot = 0;                                             // stage of the K block that is multiplied next
    auto free_slot = [&]() { return rslot == 0 ? D - 1 : rslot - 1; };
    bool more = false;                                         // is there a unit behind this one?

    const int first = (quad & 1) * 2 + (quad >> 1);
    const uint32_t off0 = (uint32_t)(first ^ (l16 & 7) ^ ((l16 >> 3) & 1)) << 4;
    const uint32_t a0 = lds0 + (wave * 32 + l16) * KB + off0, b0 = lds0 + W_STAGE + l16 * KB + off0;
    const uint32_t x0 = lds0 + W_STAGE + X_STAGE + l16 * 4;

    auto run = [&](auto tiles_of_16) {
        constexpr int N = decltype(tiles_of_16)::value;
        constexpr bool LATE = N <= 4;                          // a product is folded while the next K block's operands are read
        v4f acc[2][N], T[2][N];
        float sc[2][N];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < N; ++t) {
                sc[s][t] = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[s][t][r] = T[s][t][r] = 0.f;
            }
        auto fold = [&]() {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int t = 0; t < N; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[s][t][r] = fmaf(sc[s][t], T[s][t][r], acc[s][t][r]);
        };
        uint32_t ws_at = lds0 + WS_AT + buffer * (2 * WS_ROW) + (GATED ? 0 : (wave >> 2) * WS_ROW);
        auto multiply = [&]() {
            const uint32_t st = (uint32_t)(rslot * STAGE);
            rslot = rslot == D - 1 ? 0 : rslot + 1;
            v8i a[2], b[N];
            float x[N], ws[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) a[s] = lds_operand(a0 + st, (a0 + st) ^ 64, s * 16 * KB);
#pragma unroll
            for (int t = 0; t < N; ++t) {
                b[t] = lds_operand(b0 + st, (b0 + st) ^ 64, t * 16 * KB);
                x[t] = *reinterpret_cast<__attribute__((address_space(3))) const float*>(x0 + st + t * 64);
            }
            ws[0] = *reinterpret_cast<__attribute__((address_space(3))) const float*>(ws_at);
            ws[1] = GATED ? *reinterpret_cast<__attribute__((address_space(3))) const float*>(ws_at + WS_ROW) : ws[0];
            ws_at += 4;
            if (LATE) fold();                                  // the K block before
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const v4f z = {0.f, 0.f, 0.f, 0.f};
                    T[s][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a[s], b[t], z, 0, 0, 0, 0, 0, 0);
                    sc[s][t] = x[t] * ws[s];
                }
            if (!LATE) fold();
        };
        // The K block to be multiplied has landed for everybody, and everybody is done with the one before, whose slots are free.
        auto meet = [&]() {
            asm volatile("s_waitcnt vmcnt(%1) lgkmcnt(0)\n\ts_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 .Lfull%=\n\ts_waitcnt vmcnt(%2)\n.Lfull%=:"
                         :: "s"(full_aux), "n"(newer(NA)), "n"(newer(NA - 1)) : "memory", "scc");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
#pragma unroll 1
        for (int kb = 0; kb < nkb - (D - 1); ++kb) {
            meet();
            issue(free_slot());
            if (kb == 0 && more) {
                next = tile_of(unit + slots);
                weights_of(next, w_next);
                look_up(next, buffer ^ 1);
            }
            multiply();
        }
#pragma unroll
        for (int i = 0; i < D - 1; ++i) {                      // the copies go on with the next unit
            if (i == 0 || more) {
                meet();
            } else {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if (more) {
                if (i == 0) {
                    w_base[0] = w_next[0];
                    w_base[1] = w_next[1];
                    once = all_ones_if_less(next.tiles, 2);
                    aim_rows(next, [&](int r) { return s_perm[r]; });
                }
                issue(free_slot());
            }
            multiply();
        }
        if (LATE) fold();
        uint8_t* const s_epi = smem + free_slot() * STAGE;     // the stage multiplied last: refilled behind the next barrier but the epilogue's
        if (GATED) {
            // a wave's largest values and codes lie where its weights were
            auto s_amax = [&](int w) { return reinterpret_cast<float*>(s_epi + w * (32 * KB)); };
            auto s_codes = [&](int w) { return s_epi + w * (32 * KB) + FLOW_ROWS * 4; };
            float h[N][4];
#pragma unroll
            for (int t = 0; t < N; ++t) {
                float am = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    h[t][r] = swiglu(acc[0][t][r], acc[1][t][r]);
                    am = fmaxf(am, fabsf(h[t][r]));
                }
                am = fmaxf(am, __shfl_xor(am, 16));
                am = fmaxf(am, __shfl_xor(am, 32));
                if (quad == 0) s_amax(wave)[t * 16 + l16] = am;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int t = 0; t < N; ++t) {
                const int r = t * 16 + l16;
                float am = 0.f;
#pragma unroll
                for (int w = 0; w < 8; ++w) am = fmaxf(am, s_amax(w)[r]);
                const float scale = (am == 0.f) ? 1.0f : am / 448.0f;
                *reinterpret_cast<uint32_t*>(s_codes(wave) + r * 16 + quad * 4) =
                    e4m3_codes4(Quotient(scale), h[t][0], h[t][1], h[t][2], h[t][3]);
                if (quad == 0 && wave == 0 && r < cur.nrows) g.hs[(size_t)cur.ft * g.n_rows + cur.row0 + r] = scale;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            for (int r = tid >> 3; r < cur.nrows; r += NTHR / 8)
                *reinterpret_cast<uint4*>(g.hq + (size_t)(cur.row0 + r) * g.NOUT + cur.ft * FT + cslot * 16) =
                    *reinterpret_cast<const uint4*>(s_codes(cslot) + r * 16);
        } else {
            float* const s_y = reinterpret_cast<float*>(s_epi + wave * (32 * KB));
            const int f = cur.ft * FT + wave * 32;
            if (f < g.NOUT) {
#pragma unroll
                for (int t = 0; t < N; ++t) {
#pragma unroll
                    for (int s = 0; s < 2; ++s) *reinterpret_cast<v4f*>(s_y + l16 * Y_LD + s * 16 + quad * 4) = acc[s][t];
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    v4f v[2];
#pragma unroll
                    for (int it = 0; it < 2; ++it) v[it] = *reinterpret_cast<const v4f*>(s_y + (it * 8 + sub) * Y_LD + cslot * 4);
#pragma unroll
                    for (int it = 0; it < 2; ++it) {
                        const int r = t * 16 + it * 8 + sub;
                        if (r < cur.nrows) *reinterpret_cast<v4f*>(g.y + (size_t)(cur.row0 + r) * g.NOUT + f + cslot * 4) = v[it];
                    }
                    asm volatile("" ::: "memory");
                }
            }
        }
    };
    for (;;) {
        more = unit + slots < unit_end;
        switch ((cur.nrows + 15) >> 4) {
            case 1: run(std::integral_constant<int, 1>{}); break;
            case 2: run(std::integral_constant<int, 2>{}); break;
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 4: run(std::integral_constant<int, 4>{}); break;
            case 5: run(std::integral_constant<int, 5>{}); break;
            default: run(std::integral_constant<int, TILES>{}); break;
        }
        if (!more) break;
        cur = next;
        unit += slots;
        buffer ^= 1;
    }
}

template <bool GATED, bool GATHER>
hipError_t launch(hipStream_t stream, const StreamArgs& a) {
    hipLaunchKernelGGL((ffn_flow<GATED, GATHER>), dim3(CUS), dim3(NTHR), LDS_BYTES, stream, a);
    return hipGetLastError();
}
template <bool GATED, bool GATHER>
hipError_t allow_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&ffn_flow<GATED, GATHER>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
}

}  // namespace

hipError_t set_flow_lds_limits() {
    hipError_t e = allow_lds<true, true>();
    if (e == hipSuccess) e = allow_lds<true, false>();
    if (e == hipSuccess) e = allow_lds<false, false>();
    return e;
}

hipError_t launch_flow_gate_up(moe_ctx* c, const uint8_t* xq, const float* xs, const int32_t* perm, const int32_t* offsets,
                               const uint8_t* W1, const uint8_t* W3, const float* s1, const float* s3) {
    const moe_dims& m = c->dims;
    const StreamArgs a{xq, xs, m.T * m.k, perm, m.k, m.T, offsets, m.E, nullptr, nullptr, W1, W3, s1, s3, m.d, m.F,
                       true, nullptr, c->hq, c->hs, nullptr};
    return perm ? launch<true, true>(c->stream, a) : launch<true, false>(c->stream, a);
}

hipError_t launch_flow_down(moe_ctx* c, const int32_t* offsets, const uint8_t* W2, const float* s2, float* y_perm) {
    const moe_dims& m = c->dims;
    const StreamArgs a{c->hq, c->hs, m.T * m.k, nullptr, 1, 1, offsets, m.E, nullptr, nullptr, W2, nullptr, s2, nullptr, m.F, m.d,
                       true, nullptr, nullptr, nullptr, y_perm};
    return launch<false, false>(c->stream, a);
}

}  // namespace moe355
