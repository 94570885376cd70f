// Device side of the completion flags (not installed): how the last launch of a call tells the waiting
// host that its results are in pinned memory, and the fold of workgroup records that such launches
// begin with.
//
// hipStreamSynchronize returns about 5 us after the kernel has ended (11.3 us for one empty launch and
// the wait; 6.1 us when the kernel stores a word the host polls), which is most of a small call.  The
// last launch therefore stores its call's sequence number into one flag per workgroup.
#pragma once
#include "bsse_internal.h"
#include <limits.h>

namespace bsse {

// By every thread of the workgroup, when all of its results have been written.
__device__ __forceinline__ void signal_done(const Done &d, unsigned slot)
{
    // Every wavefront's stores have left it; then one write-back of the caches and the flag.  (A system
    // fence in every wavefront instead is a write-back each: 45 us instead of 27 for 256 workgroups of
    // eight.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(d.flag + slot, d.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace bsse
