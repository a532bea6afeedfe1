// Scans over the lanes of a wave.
#pragma once
#include <hip/hip_runtime.h>

namespace moe355 {

// inclusive prefix sum over the wave, by lane shifts
template <int CTRL, int ROWS>
__device__ inline int from_lanes(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }
__device__ inline int wave_scan(int v) {
    v += from_lanes<0x111, 0xf>(v);                            // row_shr 1, 2, 4, 8: rows of 16 lanes
    v += from_lanes<0x112, 0xf>(v);
    v += from_lanes<0x114, 0xf>(v);
    v += from_lanes<0x118, 0xf>(v);
    v += from_lanes<0x142, 0xa>(v);                            // row_bcast 15, 31: over the rows
    v += from_lanes<0x143, 0xc>(v);
    return v;
}

}  // namespace moe355
