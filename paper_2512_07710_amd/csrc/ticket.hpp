// Which of the blocks that work on the same thing is the last to arrive: an atomic ticket, nobody waits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe355 {

// A ticket is one wrapping increment and always of the same n, so any number of whole launches leaves it at zero.  That holds for launches that
// overlapped as well, which a context does not allow: what they computed is undefined, but the calls behind them find their last block again.  (An
// add, with the last block's store of zero behind it, lost the arrivals between the two, and no later launch on the ticket had a last block.)
template <class Count>             // increment(limit): the value before; from `limit` the count goes to zero
__host__ __device__ inline bool last_to_arrive(const Count& count, int n) { return count.increment(n - 1) == n - 1; }

struct DeviceCount {
    int32_t* at;
    __device__ int increment(int limit) const { return (int)atomicInc(reinterpret_cast<unsigned*>(at), (unsigned)limit); }
};

// The whole block calls it, behind the stores that the last block will read: relaxed device-scope ones, which go to the point where all
// XCDs' L2 caches agree.  s_last: LDS.
__device__ inline bool last_block(int32_t* ticket, int n, int32_t& s_last) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");            // every wave's stores have reached that point
    __syncthreads();
    if (threadIdx.x == 0) s_last = last_to_arrive(DeviceCount{ticket}, n);
    __syncthreads();
    return s_last != 0;
}

}  // namespace moe355
