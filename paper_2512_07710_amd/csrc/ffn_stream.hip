// Block-scaled FP8 GEMMs for few rows per expert: the weight-streaming form of the grouped GEMM in ffn.hip.
//
// With a few dozen rows per expert the time is that of bringing every weight in once, and what matters is how many bytes are
// in flight and how evenly the weights are spread over the chip.  The big-tile kernel holds 160 KiB of LDS per block: one block
// per CU, nothing overlaps a tile's prologue and epilogue, and a single sequence's few tiles leave most CUs idle.  Here a
// work unit (a tile of up to 64 rows x 128 gated / 256 plain output features) is cut into S = 8/NW blocks of NW waves,
// small enough that several share a CU:
//   * wave g of the unit's eight multiplies 32 staged weight rows (gate/up: 16 gate rows and the 16 up rows of the same
//     features, so that SwiGLU is lane-local) by the tile's one or two groups of 32 token columns, as the narrow tiles of
//     ffn.hip do, with the same instructions in the same order: the results are bit-identical;
//   * weights, activations and activation scales all come by direct-to-LDS copies into a ring of D stages (K blocks), D - 2 of
//     them in flight behind the one being multiplied, one barrier per K block;
//   * a product is folded into its accumulators while the next K block's operands are read, so that a K step is not a chain
//     of barrier, operand reads, matrix instructions and multiply-adds (a second set of operand registers, read a K block
//     ahead, was slower: the register copies cost more than the overlap);
//   * activation scales are gathered straight from the token-order planes (a few dozen rows: no sorted copy needed).
// Gate/up: the scale of a token's 128 hidden features spans the unit's S blocks.  Each block puts its h (fp32) into the
// context's workspace; the last of the S to arrive (an atomic ticket per unit) takes the maximum and writes the codes.  Nobody waits.
#include "ffn_rows.hpp"

#include <type_traits>

namespace moe355 {
namespace {

constexpr int W_WAVE = 32 * KB;                       // one K block of a wave's 32 staged weight rows
constexpr int X_STAGE = STREAM_ROWS * KB;             // one K block of the tile's rows
constexpr int XS_STAGE = STREAM_ROWS * 4;             // and of their scales

constexpr int stage_bytes(int nw) { return nw * W_WAVE + X_STAGE + XS_STAGE; }

// CHOSEN: the kernel that made the work lists has counted the tiles and may have given the batch to the big tiles
template <int NW, int D, bool GATED, bool GATHER, bool GROUPED, bool CHOSEN>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2))) void ffn_stream(StreamArgs g) {
    constexpr int S = 8 / NW;                                  // blocks per unit
    constexpr int FT = GATED ? 128 : 256;                      // output features per unit
    constexpr int STAGE = stage_bytes(NW);
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

    if (CHOSEN && *g.big_units != 0) return;
    // ---- which block of which unit: XCD x (= blockIdx % 8) walks a contiguous eighth of the units, a unit's blocks side by side
    const int tid = threadIdx.x, lane = tid & 63;
    const int nft = (g.NOUT + FT - 1) / FT;
    const RowTiles<GROUPED, STREAM_ROWS, 32> tiles(g, lane);
    const int total = tiles.total * nft * S;
    const int chunk = (total + NXCD - 1) / NXCD;
    const int slot = blockIdx.x / NXCD;
    const int u = (int)(blockIdx.x % NXCD) * chunk + slot;
    if (slot >= chunk || u >= total) return;
    const int unit = u / S;
    const Tile wk = tiles.find(g, unit, nft);
    const int row_end = wk.row0 + wk.nrows;
    const int f0 = wk.ft * FT;

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gw = (u % S) * NW + wave;                        // wave of the unit
    const int l32 = lane & 31, half = lane >> 5;
    const int nkb = g.K / KB;
    const int nblk_out = g.NOUT / QBLOCK;
    if (!GATED && f0 + (u % S) * NW * 32 >= g.NOUT) return;    // the empty half of an odd last feature tile

    // ---- copy plan, 8 rows x 128 bytes per instruction: lane i -> row i/8, LDS chunk slot i%8, which receives global 16-byte
    //      chunk slot ^ (row & 7) ^ ((row >> 3) & 1), so that the operand reads touch all 64 LDS banks evenly
    const int sub = lane >> 3, cslot = lane & 7;
    const uint32_t sw[2] = {(uint32_t)(cslot ^ sub) << 4, (uint32_t)(cslot ^ sub ^ 1) << 4};   // even / odd groups of 8 rows
    const int f_wave = GATED ? f0 + gw * 16 : min(f0 + gw * 32, g.NOUT - 32);
    const size_t w0 = ((size_t)wk.expert * g.NOUT + f_wave) * (size_t)g.K;
    const uint8_t* const w_base[2] = {g.Wa + w0, GATED ? g.Wb + w0 : g.Wa + w0 + (size_t)16 * g.K};
    const uint32_t w_off[2] = {(uint32_t)sub * (uint32_t)g.K + sw[0], (uint32_t)(8 + sub) * (uint32_t)g.K + sw[1]};
    auto token = [&](int r) {                                  // the activation row of tile row r (past the end: the last one)
        const int p = min(wk.row0 + r, row_end - 1);
        return GATHER ? (int)min((uint32_t)g.perm[p] / (uint32_t)g.fan, (uint32_t)(g.n_tok - 1)) : p;
    };
    const uint8_t* const x_base = GATHER ? g.act : g.act + (size_t)wk.row0 * g.K;
    const size_t plane = (size_t)(GATHER ? g.n_tok : g.n_rows) * 4;
    const uint32_t xs_off = 4u * (uint32_t)token(lane);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;

    // ---- weight scales: lane i keeps those of K blocks 64*n + i, broadcast one at a time
    const int blk = GATED ? wk.ft : min(wk.ft * 2 + (gw >> 2), nblk_out - 1);
    const float* const sa_e = g.sa + ((size_t)wk.expert * nblk_out + blk) * nkb;
    const float* const sb_e = GATED ? g.sb + ((size_t)wk.expert * nblk_out + blk) * nkb : sa_e;

    v16f acc[2];
#pragma unroll
    for (int ts = 0; ts < 2; ++ts)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ts][r] = 0.f;

    auto k_loop = [&](auto groups, auto once) {
        constexpr bool ONCE = decltype(once)::value;           // no other row tile reads these weights
        constexpr int TS = decltype(groups)::value;            // groups of 32 token columns
        constexpr int XC = TS * 4 / NW > 0 ? TS * 4 / NW : 1;  // activation copies per wave and stage
        constexpr int C = 4 + XC + 1;                          // copies per wave and stage
        static_assert((D - 2) * C <= 63, "wait counts fit the 6-bit field");
        uint32_t x_off[XC];
#pragma unroll
        for (int j = 0; j < XC; ++j) {
            const int grp = (wave * XC + j) % (TS * 4);        // NW > 4*TS: two waves bring the same rows
            const int src = token(grp * 8 + sub);
            x_off[j] = (uint32_t)(GATHER ? src : src - wk.row0) * (uint32_t)g.K + sw[grp & 1];
        }
        auto issue = [&](int kb, int islot) {
            const uint32_t st = lds0 + islot * STAGE;
            const size_t k0 = (size_t)kb * KB;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t at = st + wave * W_WAVE + j * 1024;
                if (ONCE) dma16_once(at, w_off[j & 1], w_base[j >> 1] + k0);
                else dma16(at, w_off[j & 1], w_base[j >> 1] + k0);
            }
#pragma unroll
            for (int j = 0; j < XC; ++j)
                dma16(st + NW * W_WAVE + ((wave * XC + j) % (TS * 4)) * 1024, x_off[j], x_base + k0);
            // every wave brings the same scales to the same place: the wait counts of all waves stay alike
            dma4(st + NW * W_WAVE + X_STAGE, xs_off, reinterpret_cast<const uint8_t*>(g.act_s) + (size_t)kb * plane);
        };
        float wsa_l = 0.f, wsb_l = 0.f;
        auto load_ws = [&](int kb) {
            const int at = min(kb + lane, nkb - 1);
            wsa_l = sa_e[at];
            if (GATED) wsb_l = sb_e[at];
            // waited for here: the compiler would otherwise wait for every copy in flight at the use, in every K step
            asm volatile("s_waitcnt vmcnt(0)" : "+v"(wsa_l), "+v"(wsb_l) :: "memory");
        };
        load_ws(0);
        int islot = 0;
#pragma unroll
        for (int i = 0; i < D - 1; ++i) {
            if (i < nkb) issue(i, i);
            islot = i + 1;                                     // D - 1 after the prologue
        }
        // LDS byte address of a lane's first operand chunk relative to a stage; chunk (ks, j) is that address with bits
        // 6 and 4 flipped by ks and j (the swizzle is an exclusive or of the chunk number)
        const uint32_t off00 = (uint32_t)((half * 2) ^ (l32 & 7) ^ ((l32 >> 3) & 1)) << 4;
        const uint32_t a00 = lds0 + (uint32_t)(wave * W_WAVE + l32 * KB) + off00;
        const uint32_t b00 = lds0 + (uint32_t)(NW * W_WAVE + l32 * KB) + off00;
        const uint32_t x00 = lds0 + (uint32_t)(NW * W_WAVE + X_STAGE + l32 * 4);
        v16f T[TS];
        float sc_a[TS], sc_b[TS];
#pragma unroll
        for (int ts = 0; ts < TS; ++ts) {
            sc_a[ts] = sc_b[ts] = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) T[ts][r] = 0.f;
        }
        // accumulator registers 0..7 are gate rows, 8..15 up rows
        auto fold = [&]() {
#pragma unroll
            for (int ts = 0; ts < TS; ++ts)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[ts][r] = fmaf((GATED && r >= 8) ? sc_b[ts] : sc_a[ts], T[ts][r], acc[ts][r]);
        };
        int rslot = 0;
        for (int kb = 0; kb < nkb; ++kb) {
            if (kb != 0 && (kb & 63) == 0) load_ws(kb);
            // stage kb has landed when at most the D - 2 newer ones are outstanding (near the end fewer were issued); the
            // barrier makes it everybody's, and says that all are done with stage kb - 1, whose slot is refilled
            if (kb + D - 2 < nkb) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((D - 2) * C) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kb + D - 1 < nkb) issue(kb + D - 1, islot);
            islot = islot == D - 1 ? 0 : islot + 1;
            const uint32_t st = (uint32_t)(rslot * STAGE);
            rslot = rslot == D - 1 ? 0 : rslot + 1;
            v8i a[2], b[TS][2];
            float x[TS];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const uint32_t sA = (a00 + st), sB = (b00 + st);
                a[ks] = lds_operand(sA ^ (ks * 64), sA ^ (ks * 64 + 16), 0);
#pragma unroll
                for (int ts = 0; ts < TS; ++ts) b[ts][ks] = lds_operand(sB ^ (ks * 64), sB ^ (ks * 64 + 16), ts * 32 * KB);
            }
#pragma unroll
            for (int ts = 0; ts < TS; ++ts)
                x[ts] = *reinterpret_cast<__attribute__((address_space(3))) const float*>(x00 + st + ts * 128);
            fold();                                            // K block kb - 1
            const float wsa = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wsa_l), kb & 63));
            const float wsb = GATED ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wsb_l), kb & 63)) : wsa;
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) {
                v16f z;
#pragma unroll
                for (int r = 0; r < 16; ++r) z[r] = 0.f;
                T[ts] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[0], b[ts][0], z, 0, 0, 0, 0, 0, 0);
                T[ts] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[1], b[ts][1], T[ts], 0, 0, 0, 0, 0, 0);
                sc_a[ts] = x[ts] * wsa;
                sc_b[ts] = x[ts] * wsb;
            }
        }
        fold();
    };
    const int n_grp = wk.nrows > 32 ? 2 : 1;
    // non-temporal weight copies where no other row tile of the expert reads them
    const bool once = g.once && wk.tiles == 1;
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    if (once) {
        if (n_grp == 1) k_loop(one, std::true_type{});
        else k_loop(two, std::true_type{});
    } else {
        if (n_grp == 1) k_loop(one, std::false_type{});
        else k_loop(two, std::false_type{});
    }

    // ---- register r of acc[ts] belongs to token row0 + ts*32 + l32 and staged row (r/4)*8 + half*4 + r%4 of this wave
    if (!GATED) {
#pragma unroll
        for (int ts = 0; ts < 2; ++ts) {
            const int p = wk.row0 + ts * 32 + l32;
            if (p >= row_end) continue;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int fcol = f0 + gw * 32 + r4 * 8 + half * 4;
                if (fcol < g.NOUT)
                    *reinterpret_cast<float4*>(g.y + (size_t)p * g.NOUT + fcol) =
                        make_float4(acc[ts][r4 * 4], acc[ts][r4 * 4 + 1], acc[ts][r4 * 4 + 2], acc[ts][r4 * 4 + 3]);
            }
        }
        return;
    }
    // registers 0..7: gate of features f0 + 16*gw + (r/4)*8 + half*4 + r%4, registers 8..15: up of the same.  h goes through
    // LDS, so that it leaves in runs of the block's 16*NW features (straight from the registers it would be 8-byte pieces,
    // each a memory transaction of its own), and stays there for the block's own share of the codes.
    constexpr int HW = NW * 16, HP = HW + 4;                   // features per block, and the padded row of the LDS tile
    float* const s_h = reinterpret_cast<float*>(smem);         // [STREAM_ROWS][HP]
    int32_t* const s_ticket = reinterpret_cast<int32_t*>(smem) + STREAM_ROWS * HP;
    static_assert((STREAM_ROWS * HP + 1) * 4 <= D * STAGE, "the tile fits the ring");
    const int sub_f = (u % S) * HW;                            // the block's first feature in the unit
    __syncthreads();                                           // every wave is done with the ring
#pragma unroll
    for (int ts = 0; ts < 2; ++ts)
#pragma unroll
        for (int r4 = 0; r4 < 2; ++r4)
            *reinterpret_cast<float4*>(s_h + (ts * 32 + l32) * HP + wave * 16 + r4 * 8 + half * 4) =
                make_float4(swiglu(acc[ts][r4 * 4], acc[ts][r4 * 4 + 8]), swiglu(acc[ts][r4 * 4 + 1], acc[ts][r4 * 4 + 9]),
                            swiglu(acc[ts][r4 * 4 + 2], acc[ts][r4 * 4 + 10]), swiglu(acc[ts][r4 * 4 + 3], acc[ts][r4 * 4 + 11]));
    __syncthreads();
    float* const rows = g.h_rows + (size_t)wk.row0 * g.NOUT + f0;
    if (S > 1) {
        for (int i = tid; i < wk.nrows * (HW / 2); i += NW * 64) {
            const int r = i / (HW / 2), c = i % (HW / 2) * 2;
            put2(rows + (size_t)r * g.NOUT + sub_f + c, s_h[r * HP + c], s_h[r * HP + c + 1]);
        }
        if (!last_block(g.tickets + unit, S, *s_ticket)) return;
    }
    // the unit's last block: 16 lanes per row, 8 features each
    for (int r = tid >> 4; r < wk.nrows; r += NW * 4) {        // (the 16 lanes of a row share r)
        const int c = (tid & 15) * 8;
        float h[8];
        if (S == 1 || c / HW == u % S) {
#pragma unroll
            for (int i = 0; i < 8; ++i) h[i] = s_h[r * HP + c - sub_f + i];
        } else {
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                const float2 v = get2(rows + (size_t)r * g.NOUT + c + i);
                h[i] = v.x;
                h[i + 1] = v.y;
            }
        }
        put_hidden_row(g, wk.row0 + r, wk.ft, tid & 15, h);
    }
}

// Four waves and three stages: two blocks of 75 KB share a CU.  On the same buffers (gate/up, 64 experts x 4096 x 1408 and more):
// two waves and three or four stages measure the same with few units and 5 % more time in a full grid, one wave 10 % more,
// five stages (one block per CU) the same or worse.
constexpr int NW = 4, D = 3;
// A dense product of at most 64 units leaves half of the CUs idle in blocks of four waves: two waves and four stages
// (40 x 4096 x 10240, 40 units, 18.3 -> 14.0 us, 40 x 7168 x 12288 30.5 -> 22.3, 256 x 4096 x 4096, 64 units, 15.8 -> 13.5; 128 units:
// 22.3 -> 24.0).
constexpr int NW_FEW = 2, D_FEW = 4, FEW_UNITS = 64;
// Weights that are read once go past the caches: a whole layer's experts never stay in the 256 MB last-level cache until the
// next step of a model (one sequence, 104 MB of weights, after other data: 76 us for the layer through the caches, 67 past
// them).  That holds for small layers as well when other data comes between two passes (layers of 100, 201 and 170 MB of weights taken
// in turns on several sets of weights and inputs: 39.8, 51.4, 57.3 us through the caches, 37.4, 49.2, 53.0 past them); repeated on
// the same weights with nothing between they pay for it (256 tokens x 2 of 2048 x 1024, 16 experts 35.2 / 36.1, 128 x 2 of 4096 x
// 2048, 8 experts 48.2 / 57.2, the form before either 63.6), which no model does.
// A dense matrix of up to this size may well stay (40 rows x 4096 x 6144, in this kernel: 25.4 and 24.4 us after other data, 16.6
// and 17.0 when it is still there), beyond it cannot.
constexpr int64_t LINEAR_ONCE_BYTES = 256ll << 20;

template <int WAVES, int STAGES, bool GATED, bool GATHER, bool GROUPED, bool CHOSEN = false>
hipError_t launch(hipStream_t stream, const StreamArgs& a, int max_units) {
    const int grid = (max_units * (8 / WAVES) + NXCD - 1) / NXCD * NXCD;
    hipLaunchKernelGGL((ffn_stream<WAVES, STAGES, GATED, GATHER, GROUPED, CHOSEN>), dim3(grid), dim3(WAVES * 64), STAGES * stage_bytes(WAVES), stream, a);
    return hipGetLastError();
}

template <int WAVES, int STAGES, bool GATED, bool GATHER, bool GROUPED, bool CHOSEN = false>
hipError_t allow_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&ffn_stream<WAVES, STAGES, GATED, GATHER, GROUPED, CHOSEN>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, STAGES * stage_bytes(WAVES));
}

}  // namespace

// all instances at once, so that any first call (before a capture, say) covers every later one
hipError_t set_stream_lds_limits() {
    hipError_t e = allow_lds<NW, D, true, true, true>();
    if (e == hipSuccess) e = allow_lds<NW, D, true, false, true>();
    if (e == hipSuccess) e = allow_lds<NW, D, false, false, true>();
    if (e == hipSuccess) e = allow_lds<NW, D, false, false, true, true>();
    if (e == hipSuccess) e = allow_lds<NW, D, false, false, false>();
    if (e == hipSuccess) e = allow_lds<NW_FEW, D_FEW, false, false, false>();
    return e;
}

hipError_t launch_stream_gate_up(moe_ctx* c, const uint8_t* xq, const float* xs, const int32_t* perm, const int32_t* offsets,
                                 int max_units, const uint8_t* W1, const uint8_t* W3, const float* s1, const float* s3) {
    const moe_dims& m = c->dims;
    const StreamArgs a{xq, xs, m.T * m.k, perm, m.k, m.T, offsets, m.E, nullptr, c->tickets, W1, W3, s1, s3, m.d, m.F,
                       true, c->h_rows, c->hq, c->hs, nullptr};
    return perm ? launch<NW, D, true, true, true>(c->stream, a, max_units) : launch<NW, D, true, false, true>(c->stream, a, max_units);
}

hipError_t launch_stream_down(moe_ctx* c, const int32_t* offsets, int max_units, const int32_t* big_units, const uint8_t* W2,
                              const float* s2, float* y_perm) {
    const moe_dims& m = c->dims;
    const StreamArgs a{c->hq, c->hs, m.T * m.k, nullptr, 1, 1, offsets, m.E, big_units, nullptr, W2, nullptr, s2, nullptr, m.F, m.d,
                       true, nullptr, nullptr, nullptr, y_perm};
    return big_units ? launch<NW, D, false, false, true, true>(c->stream, a, max_units) : launch<NW, D, false, false, true>(c->stream, a, max_units);
}

hipError_t launch_stream_linear(moe_ctx* c, const uint8_t* xq, const float* xs, int32_t rows, int32_t K, const uint8_t* Wq,
                                const float* ws, int32_t NOUT, float* y) {
    const StreamArgs a{xq, xs, rows, nullptr, 1, 1, nullptr, 1, nullptr, nullptr, Wq, nullptr, ws, nullptr, K, NOUT,
                       rows <= STREAM_ROWS && (int64_t)K * NOUT > LINEAR_ONCE_BYTES, nullptr, nullptr, nullptr, y};
    const int units = (rows + STREAM_ROWS - 1) / STREAM_ROWS * ((NOUT + 255) / 256);
    return units <= FEW_UNITS ? launch<NW_FEW, D_FEW, false, false, false>(c->stream, a, units)
                              : launch<NW, D, false, false, false>(c->stream, a, units);
}

}  // namespace moe355
