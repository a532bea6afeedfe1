// What the weight-streaming GEMMs share (ffn_stream.hip, ffn_flow.hip, ffn_few.hip): their arguments, and the row tiles worked out on the device.
#pragma once
#include "ffn_common.hpp"
#include "ffn_rules.hpp"
#include "ticket.hpp"

namespace moe355 {

// relaxed device-scope accesses: they go to the point where all XCDs' L2 caches agree
__device__ inline void put2(float* p, float a, float b) {
    const uint64_t v = (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32);
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline float2 get2(const float* p) {
    const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

struct StreamArgs {
    const uint8_t* act;            // GATHER: [n_tok, K] codes in token order; else [n_rows, K] in sorted order
    const float* act_s;            // their scales, [K/128][n_tok] or [K/128][n_rows]
    int n_rows;
    const int32_t* perm;           // GATHER: sorted row p is token perm[p] / fan
    int fan, n_tok;
    const int32_t* offsets;        // GROUPED: [E+1], of the experts' rows
    int E;
    const int32_t* big_units;      // CHOSEN: nothing to do where it is not zero
    int32_t* tickets;              // GATED: one per unit, zero before and after the launch
    const uint8_t *Wa, *Wb;
    const float *sa, *sb;
    int K, NOUT;
    bool once;                     // may the weights go past the caches?
    float* h_rows;                 // GATED: [n_rows][NOUT] h before its codes
    uint8_t* hq;
    float* hs;
    float* y;
};

// ---- hidden rows of a unit whose 128 features are spread over S blocks
// Every wave's part of h has been put; the last of the unit's blocks (last_block) can read all of it with get2.
// Sixteen lanes own row p of feature tile ft, lane `sub` features 8*sub .. 8*sub+7 in h: their scale and codes.
__device__ inline void put_hidden_row(const StreamArgs& g, int p, int ft, int sub, const float (&h)[8]) {
    float am = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) am = fmaxf(am, fabsf(h[i]));
    am = fmaxf(am, __shfl_xor(am, 1));
    am = fmaxf(am, __shfl_xor(am, 2));
    am = fmaxf(am, __shfl_xor(am, 4));
    am = fmaxf(am, __shfl_xor(am, 8));
    const float sc = (am == 0.f) ? 1.0f : am / 448.0f;
    const Quotient q(sc);
    uint2 codes;
    codes.x = e4m3_codes4(q, h[0], h[1], h[2], h[3]);
    codes.y = e4m3_codes4(q, h[4], h[5], h[6], h[7]);
    *reinterpret_cast<uint2*>(g.hq + (size_t)p * g.NOUT + ft * 128 + sub * 8) = codes;
    if (sub == 0) g.hs[(size_t)ft * g.n_rows + p] = sc;
}

// The row tiles of all experts and the units made of them, ordered (expert, feature tile, row tile) as in the big-tile kernel's
// work list.  Every wave works them out from the offsets in registers: lane l keeps experts 4l .. 4l+3.  (A list written by a
// kernel of its own costs a launch, 4..5 us of a decode step, and two dependent loads here instead of one.)
struct Tile { int expert, ft, row0, nrows, tiles; };            // tiles: row tiles of the expert
template <bool GROUPED, int ROWS, int GROUP>                   // !GROUPED: one "expert" owns all n_rows rows
struct RowTiles {
    int off[5];                                                // offsets of the lane's experts
    int before, total;                                         // tiles of the experts before the lane's; of all
    __device__ RowTiles(const StreamArgs& g, int lane) {
        if (!GROUPED) {
            total = (g.n_rows + ROWS - 1) / ROWS;
            return;
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) off[i] = g.offsets[min(lane * 4 + i, g.E)];
        int mine = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) mine += count(i);
        const int incl = wave_scan(mine);
        before = incl - mine;
        total = __builtin_amdgcn_readlane(incl, 63);
    }
    __device__ int count(int i) const { return (off[i + 1] - off[i] + ROWS - 1) / ROWS; }
    __device__ Tile find(const StreamArgs& g, int unit, int nft) const {
        Tile t;
        if (!GROUPED) {
            t.expert = 0;
            t.tiles = total;
            t.ft = unit / total;
            t.row0 = (unit - t.ft * total) * ROWS;
            t.nrows = min(ROWS, g.n_rows - t.row0);
            return t;
        }
        const int at = unit / nft;                             // a tile of the unit's expert (an expert has tiles * nft units)
        int end = before + count(0) + count(1) + count(2) + count(3);
        const int l = __builtin_ctzll(__ballot(end > at));     // at < total: some lane has it
        int base = __builtin_amdgcn_readlane(before, l), start = 0, cnt = 0;
        t.expert = 4 * l;
        t.tiles = 0;
        bool found = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = __builtin_amdgcn_readlane(off[i], l), n = __builtin_amdgcn_readlane(off[i + 1], l) - o;
            const int nt = (n + ROWS - 1) / ROWS;
            if (!found && at < base + nt) {
                found = true;
                t.expert = 4 * l + i;
                t.tiles = nt;
                start = o;
                cnt = n;
            }
            if (!found) base += nt;
        }
        const int r = unit - base * nft;
        t.ft = r / t.tiles;
        const int i = r - t.ft * t.tiles;
        // groups of GROUP rows dealt out evenly over the expert's tiles
        const int G = (cnt + GROUP - 1) / GROUP;
        const int lo = min(cnt, GROUP * (i * G / t.tiles)), hi = min(cnt, GROUP * ((i + 1) * G / t.tiles));
        t.row0 = start + lo;
        t.nrows = hi - lo;
        return t;
    }
};

}  // namespace moe355
