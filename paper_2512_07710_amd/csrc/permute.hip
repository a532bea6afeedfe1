// Stable counting sort of the T*k (token, slot) assignments by expert id.
//
// Two kernels:
//   1. chunk_hist_rank: each block ranks PERM_CHUNK ids with wave ballots and per-wave
//      running counts in LDS, which yields the chunk's histogram and every entry's rank
//      among earlier equal ids of the chunk.
//      Its last block turns the per-chunk histograms into exclusive prefix
//      sums over chunks (per expert) and the expert totals into offsets[0..E] (scan_chunks).
//   2. scatter: position = offsets[e] + prefix[chunk][e] + rank; writes perm/inv_perm.  Ids that come
//      from a log are also checked here: an id outside [0,E) raises flags[0], an id that repeats an
//      earlier slot of the same token raises flags[1] (the permutation is still the stable sort of
//      what was given).
// The result is unique (stable), so it can be compared bit for bit.  Batches of at most one_block_max_n
// assignments take one fused launch instead (permute_one_block).
#include "permute_block.hpp"
#include "ticket.hpp"
#include "quantize_rows.hpp"

#include <mutex>

namespace moe355 {
namespace {

// Scratch of moe_route_replay_noalloc: the per-chunk histograms of the two-kernel permutation, then two flag
// words and a ticket.  A file-scope device array (every GPU the library runs on holds its own copy until the process ends)
// instead of a hipMalloc'ed workspace, so that the call allocates nothing.
constexpr int NOALLOC_MAX_N = 1 << 20;                                  // assignments (T*k) per call
constexpr int NOALLOC_COUNT_INTS = (NOALLOC_MAX_N / PERM_CHUNK) * MAX_E; // 512 chunks x 256 experts
constexpr int NOALLOC_FLAG_INTS = 64;
static __device__ __align__(256) int32_t scratch[NOALLOC_COUNT_INTS + NOALLOC_FLAG_INTS];   // 512.25 KiB

// Host code never passes `scratch` itself to a kernel (there the name is a host-side stand-in): the device
// address is asked for once per device and kept here.
constexpr int MAX_DEVICES = 64;
int32_t* scratch_addr[MAX_DEVICES] = {};
std::mutex scratch_mutex;

hipError_t scratch_on_current_device(int32_t** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        scratch_addr[dev] = static_cast<int32_t*>(p);
    }
    *out = scratch_addr[dev];
    return hipSuccess;
}

// Per-chunk histograms -> their exclusive prefix sums over chunks (per expert), and the experts' totals -> offsets[0..E].  One block, whose
// launch's other blocks have put the histograms.
__device__ inline void scan_chunks(int32_t* __restrict__ chunk_counts, int n_chunks, int E, int32_t* __restrict__ offsets) {
    __shared__ int32_t s_part[MAX_E / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto count = [&](int c) {
        return __hip_atomic_load(chunk_counts + (size_t)c * E + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    int run = 0;
    if (tid < E) {
        int c = 0;
        for (; c + 16 <= n_chunks; c += 16) {
            int v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = count(c + u);
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                chunk_counts[(size_t)(c + u) * E + tid] = run;
                run += v[u];
            }
        }
        for (; c < n_chunks; ++c) {
            const int v = count(c);
            chunk_counts[(size_t)c * E + tid] = run;
            run += v;
        }
    }
    int incl = wave_scan(run);
    if (lane == 63) s_part[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += s_part[w];
    if (tid < E) offsets[tid + 1] = incl;
    if (tid == 0) offsets[0] = 0;
}

// Each of the four waves ranks a quarter of the chunk, 64 entries at a time: eight ballots (one per
// bit of the expert id) give every lane the set of lanes that hold the same id, its rank among them is
// a population count of the lower lanes, and the lowest lane of each set advances that expert's running
// count, kept per wave in LDS (read by the whole set, then written by one lane: LDS operations of a wave
// execute in order).  A second pass turns the per-wave counts into the chunk histogram and the per-wave
// bases.  Ids outside [0,E) are ranked among themselves; that rank is never used.
// The last block to arrive (ticket.hpp) scans the histograms; nobody waits.  In a launch of its own the scan came behind the tokens' quantisation
// that rides in this one (us, two launches / this: 8000 assignments of 64 experts 7.4 + 2.7 / 9.0, 12000 of 16 6.6 + 4.6 / 8.8, 262144 of 256 11.6 +
// 20.2 / 28.4; layers of 1000 x 8 of 64, 1024 x 512 61.4 / 60.2, 6000 x 2 of 16, 3072 x 2048 337.0 / 334.8, 4096 x 8 of 128, 5120 x 1536 1093 /
// 1091).
__global__ __launch_bounds__(256) void chunk_hist_rank(const int32_t* __restrict__ ids, int N, int E,
                                                       int32_t* __restrict__ chunk_counts,
                                                       int32_t* __restrict__ rank_out,
                                                       int32_t* __restrict__ ids_copy, int n_chunks,
                                                       int32_t* __restrict__ offsets, int32_t* __restrict__ ticket,
                                                       token_quant tokens) {
    if ((int)blockIdx.x >= n_chunks) {                // (as in permute_one_block)
        quantize_block<256, 2>(tokens, blockIdx.x - n_chunks);
        return;
    }
    constexpr int PER_WAVE = PERM_CHUNK / 4;          // 512 entries, 8 steps of 64
    __shared__ int32_t s_cnt[4][MAX_E];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int base = blockIdx.x * PERM_CHUNK;
    for (int i = tid; i < 4 * MAX_E; i += 256) (&s_cnt[0][0])[i] = 0;
    __syncthreads();
    int32_t my_id[PER_WAVE / 64], my_rank[PER_WAVE / 64];
    const uint64_t lower = (1ull << lane) - 1ull;
#pragma unroll
    for (int st = 0; st < PER_WAVE / 64; ++st) {
        const int i = base + wave * PER_WAVE + st * 64 + lane;
        int32_t v = -1;
        if (i < N) {
            v = ids[i];
            if (ids_copy) ids_copy[i] = v;
        }
        const bool valid = v >= 0 && v < E;           // entries past the end and bad ids form a class of their own
        my_id[st] = v;
        const int key = v & (MAX_E - 1);
        uint64_t same = __ballot(valid);              // lanes past the end never match a valid lane
        if (!valid) same = ~same;
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t bal = __ballot((key >> bit) & 1);
            same &= ((key >> bit) & 1) ? bal : ~bal;
        }
        const int before = s_cnt[wave][key];
        my_rank[st] = before + __popcll(same & lower);
        if (valid && (same & lower) == 0ull) s_cnt[wave][key] = before + __popcll(same);
    }
    __syncthreads();
    // thread e: per-wave bases (exclusive over waves) and the chunk total of expert e
    if (tid < MAX_E) {
        int run = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int c = s_cnt[w][tid];
            s_cnt[w][tid] = run;
            run += c;
        }
        if (tid < E)
            __hip_atomic_store(chunk_counts + (size_t)blockIdx.x * E + tid, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < PER_WAVE / 64; ++st) {
        const int i = base + wave * PER_WAVE + st * 64 + lane;
        if (i < N) rank_out[i] = my_rank[st] + s_cnt[wave][my_id[st] & (MAX_E - 1)];
    }
    __shared__ int32_t s_ticket;
    if (!last_block(ticket, n_chunks, s_ticket)) return;
    scan_chunks(chunk_counts, n_chunks, E, offsets);
}

__global__ __launch_bounds__(256) void scatter(const int32_t* __restrict__ ids, int N, int E,
                                               const int32_t* __restrict__ chunk_prefix,
                                               const int32_t* __restrict__ offsets,
                                               const float* __restrict__ w_in, float* __restrict__ w_copy,
                                               int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                                               int k, bool check_dups, int32_t* __restrict__ flags) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    if (w_copy) w_copy[i] = w_in[i];
    const int e = ids[i];
    if (e < 0 || e >= E) {
        flags[0] = 1;                                   // plain store; any writer stores the same value
        inv_perm[i] = -1;
        return;
    }
    if (check_dups) {
        const int first = i - i % k;                    // slot 0 of this assignment's token
        bool dup = false;
        for (int q = first; q < i; ++q) dup |= ids[q] == e;
        if (dup) flags[1] = 1;
    }
    const int chunk = i / PERM_CHUNK;
    const int pos = offsets[e] + chunk_prefix[(size_t)chunk * E + e] + inv_perm[i];   // inv_perm holds the rank
    // (within the rows unless calls overlapped that must not: then at least nothing outside is written, or read by the combine)
    const bool inside = (uint32_t)pos < (uint32_t)N;
    inv_perm[i] = inside ? pos : -1;
    if (inside) perm[pos] = i;
}

constexpr int ONE_BLOCK_MAX_N = ONE_BLOCK_WAVES * ONE_BLOCK_MAX_STEPS * 64;
constexpr int ONE_BLOCK_CHECKED_MAX_N = 5120;
static_assert(ONE_BLOCK_CHECKED_MAX_N <= ONE_BLOCK_MAX_N, "the block holds that many");
inline int one_block_max_n(bool check_dups, int k) { return check_dups && k > 1 ? ONE_BLOCK_CHECKED_MAX_N : ONE_BLOCK_MAX_N; }

// The quantisation of the same batch's tokens, which waits for nobody, may come along in blocks of its own (block 0 permutes): beside
// one busy block the rest of the chip is idle, and a launch less (777 tokens x 2176: 9.2 + 4.9 us one after the other).
template <int STEPS>
__global__ __launch_bounds__(ONE_BLOCK_WAVES * 64) void permute_one_block(
    const int32_t* __restrict__ ids, int N, int E, int32_t* __restrict__ ids_copy, const float* __restrict__ w_in,
    float* __restrict__ w_copy, int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
    int k, bool check_dups, int32_t* __restrict__ flags, token_quant tokens) {
    if (blockIdx.x > 0) {
        quantize_block<ONE_BLOCK_WAVES * 64, 1>(tokens, blockIdx.x - 1);
        return;
    }
    permute_block<STEPS>([&](int i) { return ids[i]; }, N, E, ids_copy, w_in, w_copy, offsets, perm, inv_perm, k, check_dups, flags);
}

__global__ void fill_i32(int32_t* __restrict__ p, int n, int32_t v) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void clear_flags(int32_t* __restrict__ flags, int32_t* __restrict__ ticket, int32_t* __restrict__ offsets, int E) {
    if ((int)threadIdx.x <= E) offsets[threadIdx.x] = 0;
    if (threadIdx.x < 2) flags[threadIdx.x] = 0;
    if (threadIdx.x == 2) *ticket = 0;
}

}  // namespace

// a fill kernel, not hipMemsetAsync: it stays correct when a caller records the call into a HIP graph
hipError_t launch_fill_i32(hipStream_t stream, int32_t* p, int n, int32_t v) {
    if (n > 0) hipLaunchKernelGGL(fill_i32, dim3((n + 255) / 256), dim3(256), 0, stream, p, n, v);
    return hipGetLastError();
}

hipError_t launch_permute(const permute_args& a, const int32_t* ids_in, int32_t* ids_copy, const float* w_in,
                          float* w_copy, int32_t* offsets, int32_t* perm, int32_t* inv_perm, const token_quant& tokens) {
    const int N = a.T * a.k;
    const int n_chunks = (N + PERM_CHUNK - 1) / PERM_CHUNK;
    if (N > 0 && N <= one_block_max_n(a.check_dups, a.k)) {
#define MOE_ONE_BLOCK(STEPS_)                                                                                              \
    hipLaunchKernelGGL(permute_one_block<STEPS_>, dim3(grid), dim3(ONE_BLOCK_WAVES * 64), 0, a.stream, ids_in, N, a.E, ids_copy, \
                       w_in, w_copy, offsets, perm, inv_perm, a.k, a.check_dups, a.flags, tokens)
        const unsigned grid = (unsigned)(1 + quantize_blocks<ONE_BLOCK_WAVES * 64, 1>(tokens));
        const int steps = (N + ONE_BLOCK_WAVES * 64 - 1) / (ONE_BLOCK_WAVES * 64);
        if (steps == 1) MOE_ONE_BLOCK(1);
        else if (steps == 2) MOE_ONE_BLOCK(2);
        else if (steps <= 4) MOE_ONE_BLOCK(4);
        else MOE_ONE_BLOCK(ONE_BLOCK_MAX_STEPS);
#undef MOE_ONE_BLOCK
        return hipGetLastError();
    }
    if (N > 0)
        hipLaunchKernelGGL(chunk_hist_rank, dim3((unsigned)(n_chunks + quantize_blocks<256, 2>(tokens))), dim3(256), 0, a.stream, ids_in,
                           N, a.E, a.chunk_counts, inv_perm, ids_copy, n_chunks, offsets, a.ticket, tokens);
    if (N > 0)
        hipLaunchKernelGGL(scatter, dim3((N + 255) / 256), dim3(256), 0, a.stream, ids_in, N, a.E,
                           a.chunk_counts, offsets, w_in, w_copy, perm, inv_perm, a.k, a.check_dups, a.flags);
    return hipGetLastError();
}

// Router Replay (copy of the log + stable permutation) whose only workspace is the static device array above.
// Overlapping calls on one GPU (two streams, two threads) share that array and race.
int route_replay_noalloc(hipStream_t stream, int32_t T, int32_t E, int32_t k, const int32_t* logged_idx,
                         const float* logged_w, int32_t* topk_idx, float* topk_w, int32_t* offsets, int32_t* perm,
                         int32_t* inv_perm, int32_t* id_flags) {
    if (T < 0 || E < 1 || E > MAX_E || k < 1 || k > E || k > MAX_K) return MOE_EINVAL;
    if ((int64_t)T * k > NOALLOC_MAX_N) return MOE_EINVAL;             // beyond the scratch array's capacity
    if (!offsets) return MOE_EINVAL;
    if (T > 0 && (!logged_idx || !logged_w || !topk_idx || !topk_w || !perm || !inv_perm)) return MOE_EINVAL;
    int32_t* base = nullptr;
    if (scratch_on_current_device(&base) != hipSuccess) return MOE_EHIP;
    int32_t* flags = id_flags ? id_flags : base + NOALLOC_COUNT_INTS;
    int32_t* const ticket = base + NOALLOC_COUNT_INTS + 2;
    // the flags must start at zero, and so must the ticket, whatever calls that overlapped have left in it (their counts differ from
    // batch to batch); offsets, so that such a call leaves experts without rows and not what was there before (the histograms need no
    // clearing: every chunk in use is rewritten in full)
    hipLaunchKernelGGL(clear_flags, dim3(1), dim3((MAX_E + 64) / 64 * 64), 0, stream, flags, ticket, offsets, E);
    if (hipGetLastError() != hipSuccess) return MOE_EHIP;
    if (T == 0) return MOE_OK;
    const permute_args a{stream, T, E, k, base, flags, ticket, true};
    int32_t* idx_copy = (topk_idx == logged_idx) ? nullptr : topk_idx;
    float* w_copy = (topk_w == logged_w) ? nullptr : topk_w;
    return launch_permute(a, logged_idx, idx_copy, logged_w, w_copy, offsets, perm, inv_perm, token_quant{}) == hipSuccess ? MOE_OK
                                                                                                                          : MOE_EHIP;
}

}  // namespace moe355
