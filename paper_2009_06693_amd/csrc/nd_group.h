// Groups of lanes that work on one sample: half a wavefront, a wavefront, or a workgroup of several.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nd {

template <int THREADS>
__device__ __forceinline__ void group_sync() {
    if (THREADS > 64) {
        __syncthreads();
    } else {  // part of one wavefront: its LDS operations complete in order; keep the compiler from moving them
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}
// true when x is non-zero in any lane of the group; group_lanes: the group's lanes within its wavefront
template <int THREADS>
__device__ __forceinline__ int group_or(int x, uint64_t group_lanes) {
    if (THREADS > 64) return __syncthreads_or(x);
    group_sync<THREADS>();
    const int r = (__ballot(x != 0) & group_lanes) != 0ull;
    group_sync<THREADS>();
    return r;
}
// true when x is true in any lane of a group inside one wavefront; orders nothing
template <int THREADS>
__device__ __forceinline__ bool group_any(bool x, uint64_t group_lanes) {
    static_assert(THREADS <= 64, "groups of more than a wavefront do not call it");
    return (__ballot(x) & group_lanes) != 0ull;
}
// A queue place for every lane with flag set (any order).  A group inside one wavefront counts in a
// register (*fill, the same in all its lanes); a group of several wavefronts counts in LDS (*fill_lds).
// Every lane of the group calls it, in converged code.
template <int THREADS>
__device__ __forceinline__ uint32_t group_reserve(bool flag, uint64_t group_lanes, uint32_t* fill, uint32_t* fill_lds) {
    const uint64_t votes = __ballot(flag) & group_lanes;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t before =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(votes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)votes, 0u));
    const uint32_t n = (uint32_t)__popcll(votes);
    if (THREADS > 64) {
        uint32_t base = 0;
        if (lane == 0 && n > 0) base = atomicAdd(fill_lds, n);
        base = (uint32_t)__shfl((int)base, 0, 64);
        return base + before;
    }
    const uint32_t base = *fill;
    *fill = base + n;
    return base + before;
}

}  // namespace nd
