// Rays dealt to the waves of the query kernels.
#pragma once
#include "nif_device.hpp"

namespace nif {

// First of the n tickets that the wave takes from a range's counter, for all its lanes (they call it
// together); `size`, the range's rays, or more if none is left.  Other waves take tickets meanwhile, so
// two lanes' readings of the counter can differ: the leader's counts, or some lanes would leave out
// rays that the wave has taken and others repeat rays.  look: read the counter before the atomic, as
// the atomics of a launch's waves on one counter go one after the other (3,072 waves past 8 ranges
// without a ray: 300 us).
__device__ __forceinline__ int64_t take_tickets(int64_t* counter, int64_t size, int n, int leader, bool look) {
    unsigned long long* c = reinterpret_cast<unsigned long long*>(counter);
    bool left = size > 0;
    if (left && look) {
        const int64_t at = (int64_t)__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        left = ballot(at < size) >> leader & 1;
    }
    unsigned long long base = (unsigned long long)size;
    if (lane_id() == leader && left) base = atomicAdd(c, (unsigned long long)n);
    return left ? (int64_t)__shfl(base, leader) : size;
}

}  // namespace nif
