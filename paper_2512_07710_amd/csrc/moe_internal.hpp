// Internal declarations shared by the HIP translation units of libmoe355.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "moe355.h"

namespace moe355 {

constexpr int QBLOCK = 128;        // quantisation group (activations 1x128, weights 128x128)
constexpr int PERM_CHUNK = 2048;   // assignments handled by one block of the permutation kernels
constexpr int TOK_TILE = 256;      // expert-sorted rows per GEMM tile
constexpr int STREAM_ROWS = 64;    // expert-sorted rows per tile of the weight-streaming GEMMs
constexpr int FEW_ROWS = 16;       // expert-sorted rows per tile of the small-block GEMMs
constexpr int MAX_E = 256;
constexpr int MAX_K = 16;
constexpr int PROF_MAX_CALLS = 512;
constexpr int ROUTE_TICKET = 32, FLAG_INTS = 33;   // (the ticket has a cache line of its own)


}  // namespace moe355

struct moe_ctx {
    moe_dims dims;
    hipStream_t stream;
    int device;
    int n_chunks;            // ceil(N / PERM_CHUNK)
    int32_t* chunk_counts;   // [n_chunks][E] per-chunk histograms, then their exclusive scans
    void* tiles;             // GEMM work lists (gate/up list, then down list)
    void* queues;            // [2] their lengths and how they are dealt to the XCDs
    int32_t* tickets;        // streaming gate/up projection only: one per unit, zero between launches
    int32_t* flags;          // [0] != 0: an expert id outside [0,E) was met; [1] != 0: a logged id repeated inside a token;
                             //     [ROUTE_TICKET] ticket of the router and the permutation, zero between launches
    float* h_rows;           // streaming gate/up projection only: [N][F] hidden activations before their codes
    float* xs_sorted;        // [d/128][N] activation scales in sorted order (gathered FFN only)
    uint16_t* router_planes; // router weights split into three bf16 planes, matrix-core order
    float* route_partial;    // [splits][T padded to 32][E padded] partial logits of the split router (small batches only)
    uint8_t* hq;             // [N][F]
    float* hs;               // [N][F/128]
    // optional kernel timing: three events per recorded expert-FFN call
    bool profiling;
    int prof_calls;
    hipEvent_t* prof_events; // [3 * PROF_MAX_CALLS], created on first enable
};

namespace moe355 {

// Token-order quantisation that a permutation's launch takes along: rows of `cols` bf16 -> codes and [cols/128][rows] scales.
// x == nullptr: none.
struct token_quant {
    const uint16_t* x = nullptr;
    int64_t rows = 0;
    int32_t cols = 0;
    uint8_t* q = nullptr;
    float* scales = nullptr;
};
// logged_idx == nullptr: top-k selection; otherwise the ids are given (and searched for repeats) and only the gate weights are
// computed.  Router, then the permutation, with `tokens` quantised along the way.
hipError_t launch_route(moe_ctx* c, const uint16_t* x, const float* W_r, const float* bias, const int32_t* logged_idx,
                        int32_t* topk_idx, float* topk_w, int32_t* offsets, int32_t* perm, int32_t* inv_perm,
                        const token_quant& tokens);
// Permutation of T*k assignments over E experts on `stream`.  chunk_counts: ceil(T*k / PERM_CHUNK) * E ints of
// scratch; flags: two ints, [0] raised by an id outside [0,E), [1] (check_dups only) by a repeat inside a token.
struct permute_args {
    hipStream_t stream;
    int T, E, k;
    int32_t* chunk_counts;
    int32_t* flags;
    int32_t* ticket;             // zero between launches
    bool check_dups;
};
hipError_t launch_permute(const permute_args& a, const int32_t* ids_in, int32_t* ids_copy, const float* w_in,
                          float* w_copy, int32_t* offsets, int32_t* perm, int32_t* inv_perm, const token_quant& tokens);
inline permute_args permute_args_of(moe_ctx* c, bool check_dups) {
    return permute_args{c->stream, c->dims.T, c->dims.E, c->dims.k, c->chunk_counts, c->flags, c->flags + ROUTE_TICKET, check_dups};
}
// Router Replay with every byte of workspace in a static device array (permute.hip)
int route_replay_noalloc(hipStream_t stream, int32_t T, int32_t E, int32_t k, const int32_t* logged_idx,
                         const float* logged_w, int32_t* topk_idx, float* topk_w, int32_t* offsets, int32_t* perm,
                         int32_t* inv_perm, int32_t* id_flags);
hipError_t launch_probe_copy(hipStream_t stream, const void* src, void* dst, size_t bytes);
hipError_t launch_probe_mfma(hipStream_t stream, int blocks, int steps, bool scaled, float* sink);
hipError_t launch_fill_i32(hipStream_t stream, int32_t* p, int n, int32_t v);
hipError_t launch_quantize(hipStream_t s, const uint16_t* x, int64_t rows_in, int32_t cols,
                           const int32_t* dst_rows, int32_t fanout, uint8_t* q, float* scales);
hipError_t launch_expert_ffn(moe_ctx* c, const uint8_t* xq, const float* xs, const int32_t* perm, const int32_t* offsets,
                             const uint8_t* W1, const uint8_t* W3, const uint8_t* W2,
                             const float* s1, const float* s3, const float* s2, float* y_perm);
hipError_t launch_linear(moe_ctx* c, const uint8_t* xq, const float* xs, int32_t rows, int32_t K,
                         const uint8_t* Wq, const float* ws, int32_t NOUT, float* y);
hipError_t launch_quantize_weights(hipStream_t s, const uint16_t* w, int64_t rows, int32_t cols, uint8_t* q,
                                   float* scales);
size_t ffn_work_bytes(const moe_dims* D);
size_t ffn_queue_bytes();
size_t ffn_ticket_bytes(const moe_dims* D);
size_t ffn_h_rows_bytes(const moe_dims* D);
// The weight-streaming GEMMs (ffn_stream.hip).  perm as in launch_expert_ffn
hipError_t set_stream_lds_limits();
hipError_t launch_stream_gate_up(moe_ctx* c, const uint8_t* xq, const float* xs, const int32_t* perm, const int32_t* offsets,
                                 int max_units, const uint8_t* W1, const uint8_t* W3, const float* s1, const float* s3);
// big_units, if given: nothing to do where it is not zero (the big tiles take the batch)
hipError_t launch_stream_down(moe_ctx* c, const int32_t* offsets, int max_units, const int32_t* big_units, const uint8_t* W2,
                              const float* s2, float* y_perm);
hipError_t launch_stream_linear(moe_ctx* c, const uint8_t* xq, const float* xs, int32_t rows, int32_t K, const uint8_t* Wq,
                                const float* ws, int32_t NOUT, float* y);
// The GEMMs in small blocks for products that do not fill the chip (ffn_few.hip), tiles of FEW_ROWS rows in the grouped ones
hipError_t set_few_lds_limits();
hipError_t launch_few_gate_up(moe_ctx* c, const uint8_t* xq, const float* xs, const int32_t* perm, const int32_t* offsets,
                              int max_tiles, const uint8_t* W1, const uint8_t* W3, const float* s1, const float* s3);
hipError_t launch_few_down(moe_ctx* c, const int32_t* offsets, int max_tiles, const uint8_t* W2, const float* s2, float* y_perm);
hipError_t launch_few_linear(moe_ctx* c, const uint8_t* xq, const float* xs, int32_t rows, int32_t K, const uint8_t* Wq,
                             const float* ws, int32_t NOUT, float* y);
// The GEMMs in persistent blocks (ffn_flow.hip)
hipError_t set_flow_lds_limits();
hipError_t launch_flow_gate_up(moe_ctx* c, const uint8_t* xq, const float* xs, const int32_t* perm, const int32_t* offsets,
                               const uint8_t* W1, const uint8_t* W3, const float* s1, const float* s3);
hipError_t launch_flow_down(moe_ctx* c, const int32_t* offsets, const uint8_t* W2, const float* s2, float* y_perm);
size_t route_workspace_bytes(int E, int d);
size_t route_partial_bytes(int T, int E);
hipError_t launch_combine(moe_ctx* c, const float* y_perm, const int32_t* inv_perm,
                          const float* topk_w, uint16_t* y, float* y_f32);

}  // namespace moe355
