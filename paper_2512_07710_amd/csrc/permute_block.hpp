// The whole permutation of a small batch in one block: shared by the permutation's own launch and the router's last one.
#pragma once
#include "lanes.hpp"
#include "moe_internal.hpp"

namespace moe355 {

// Up to one_block_max_n assignments: the three steps of permute.hip in one block and one launch, where the launches themselves are most of the
// time.  Sixteen waves rank STEPS times 64 entries each in the manner of chunk_hist_rank, then scan over the experts and scatter
// from registers; bound by its chain of barriers and memory round trips.
// Whole calls in a row, us, this form / the two launches: replay of 2100 assignments k = 6 6.3 / 9.9, 4000 k = 2 7.3 / 10.0, 4096 k = 8 7.6 / 10.1,
// k = 16 7.7 / 10.9, 4500 k = 6 10.6 / 10.2, 4800 11.4 / 10.4, 5000 k = 2 10.0 / 10.0, 5120 k = 8 10.9 / 10.5, k = 16 10.6 / 11.1, 8100 k = 1 11.9 /
// 10.1 (beyond the line, before the other form lost a launch: 6000 k = 6 11.9 / 11.2, 8000 k = 16 13.3 / 12.0); replayed layers of 512 x 8 of 64,
// 2048 x 512 65.0 / 68.6, 750 x 6 of 32, 1024 x 512 48.5 / 48.2, 800 x 6 of 64, 4096 x 512 132.7 / 131.9, 640 x 8 of 128, 2048 x 768 145.4 / 145.8,
// 320 x 16 of 64, 2048 x 512 74.1 / 74.7, 8100 x 1 of 16 85.4 / 85.3.  Ids from the router itself: layers of 750 x 6 55.0 / 56.7, 640 x 8 156.8 /
// 158.1, 4500 x 1 of 32, 2048 x 512 89.3 / 92.4, 8100 x 1 105.7 / 107.4.
constexpr int ONE_BLOCK_WAVES = 16;
constexpr int ONE_BLOCK_MAX_STEPS = 8;

// id_at(i): the expert of assignment i < N; every thread of the block calls it
template <int STEPS, class IdAt>
__device__ inline void permute_block(IdAt id_at, int N, int E, int32_t* __restrict__ ids_copy, const float* __restrict__ w_in,
                                     float* __restrict__ w_copy, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
                                     int32_t* __restrict__ inv_perm, int k, bool check_dups, int32_t* __restrict__ flags) {
    constexpr int PER_WAVE = STEPS * 64;
    __shared__ int32_t s_cnt[ONE_BLOCK_WAVES][MAX_E];
    __shared__ int32_t s_off[MAX_E];                  // exclusive scan of the expert totals
    __shared__ int32_t s_part[MAX_E / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int32_t my_id[STEPS], my_rank[STEPS];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int i = wave * PER_WAVE + st * 64 + lane;
        my_id[st] = -1;
        if (i < N) {
            my_id[st] = id_at(i);
            if (w_copy) w_copy[i] = w_in[i];
        }
    }
    for (int i = tid; i < ONE_BLOCK_WAVES * MAX_E; i += ONE_BLOCK_WAVES * 64) (&s_cnt[0][0])[i] = 0;
    __syncthreads();
    const uint64_t lower = (1ull << lane) - 1ull;
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int i = wave * PER_WAVE + st * 64 + lane;
        const int32_t v = my_id[st];
        if (ids_copy && i < N) ids_copy[i] = v;
        const bool valid = v >= 0 && v < E;
        const int key = v & (MAX_E - 1);
        uint64_t same = __ballot(valid);
        if (!valid) same = ~same;
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t bal = __ballot((key >> bit) & 1);
            same &= ((key >> bit) & 1) ? bal : ~bal;
        }
        const int before = s_cnt[wave][key];
        my_rank[st] = before + __popcll(same & lower);
        if (valid && (same & lower) == 0ull) s_cnt[wave][key] = before + __popcll(same);
        // A repeat of an earlier slot of the same token: among the 64 that are looked at together the ballots have found it; slots before them are
        // read, by the few lanes whose token begins there.
        if (check_dups && valid) {
            const int slot = i % k, here = lane < slot ? lane : slot;
            bool dup = ((same & lower) >> (lane - here)) != 0ull;
            for (int q = i - slot; q < i - here; ++q) dup |= id_at(q) == v;
            if (dup) flags[1] = 1;
        }
    }
    __syncthreads();
    int total = 0, incl = 0;
    if (tid < MAX_E) {                                // thread e: per-wave bases and the total of expert e
#pragma unroll
        for (int w = 0; w < ONE_BLOCK_WAVES; ++w) {
            const int c = s_cnt[w][tid];
            s_cnt[w][tid] = total;
            total += c;
        }
        if (tid >= E) total = 0;
        incl = total;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            incl += lane >= off ? v : 0;
        }
        if (lane == 63) s_part[wave] = incl;
    }
    __syncthreads();
    if (tid < MAX_E) {
        for (int w = 0; w < wave; ++w) incl += s_part[w];
        s_off[tid] = incl - total;
        if (tid < E) offsets[tid + 1] = incl;
        if (tid == 0) offsets[0] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int i = wave * PER_WAVE + st * 64 + lane;
        if (i >= N) continue;
        const int e = my_id[st];
        if (e < 0 || e >= E) {
            flags[0] = 1;
            inv_perm[i] = -1;
            continue;
        }
        const int pos = s_off[e] + s_cnt[wave][e] + my_rank[st];
        inv_perm[i] = pos;
        perm[pos] = i;
    }
}

// The same for up to 64 assignments by one wave: lane i ranks assignment i among the wave's, nothing is left to count.
template <class IdAt>
__device__ inline void permute_wave(IdAt id_at, int N, int E, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
                                    int32_t* __restrict__ inv_perm, int k, bool check_dups, int32_t* __restrict__ flags) {
    __shared__ int32_t s_of[MAX_E];                   // rows of each expert, then where they start
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < MAX_E / 64; ++i) s_of[i * 64 + lane] = 0;
    const int e = lane < N ? id_at(lane) : -1;
    const bool valid = e >= 0 && e < E;
    const int key = e & (MAX_E - 1);
    uint64_t same = __ballot(valid);
    if (!valid) same = ~same;
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        const uint64_t bal = __ballot((key >> bit) & 1);
        same &= ((key >> bit) & 1) ? bal : ~bal;
    }
    const uint64_t before = same & ((1ull << lane) - 1ull);
    // LDS operations of a wave execute in order
    if (valid && before == 0ull) s_of[key] = __popcll(same);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    int n[MAX_E / 64], mine = 0;                      // lane l has experts 4l .. 4l+3
#pragma unroll
    for (int i = 0; i < MAX_E / 64; ++i) {
        n[i] = s_of[lane * (MAX_E / 64) + i];
        mine += n[i];
    }
    int at = wave_scan(mine) - mine;
#pragma unroll
    for (int i = 0; i < MAX_E / 64; ++i) {
        const int expert = lane * (MAX_E / 64) + i;
        s_of[expert] = at;
        at += n[i];
        if (expert < E) offsets[expert + 1] = at;
    }
    if (lane == 0) offsets[0] = 0;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (lane >= N) return;
    if (!valid) {
        flags[0] = 1;
        inv_perm[lane] = -1;
        return;
    }
    if (check_dups) {
        // earlier slots of the same token with the same id
        if (before >> (lane - lane % k)) flags[1] = 1;
    }
    const int pos = s_of[key] + __popcll(before);
    inv_perm[lane] = pos;
    perm[pos] = lane;
}

}  // namespace moe355
