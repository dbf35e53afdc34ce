// Device helpers shared by the forest rounds and the half-precision engine: per-component minima and list appends with one
// atomic per wavefront or workgroup.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace slhc {

// atomicMin that first looks: the per-component minima only decrease, so a value that does not beat
// what is already there never needs the atomic (a stale, larger value read here only costs an atomic).  In late rounds one component holds most vertices and
// unfiltered atomics on its single word serialise (measured 6 ms per round at N = 1M).
__device__ inline void min_into(uint32_t* slot, uint32_t v)
{
    if (v < *reinterpret_cast<volatile uint32_t*>(slot)) atomicMin(slot, v);
}
__device__ inline void min_into(unsigned long long* slot, unsigned long long v)
{
    if (v < *reinterpret_cast<volatile unsigned long long*>(slot)) atomicMin(slot, v);
}

// Minimum of `v` over the lanes that share a component, one atomic per component and wavefront.  In the
// late rounds most vertices belong to a few large components, and one atomic per vertex on those few
// words serialises (measured: 0.7 ms for one kernel at N = 1M).  The first two distinct colours of the
// wavefront are reduced across lanes; lanes of any further colour fall back to their own atomic, so a
// wavefront of 64 different colours (the first round) costs two short passes, not 64.
__device__ inline void wave_min_into(uint32_t* slots, int c, uint32_t v, bool active)
{
    const int lane = threadIdx.x & 63;
    unsigned long long todo = __ballot(active);
#pragma unroll 1
    for (int pass = 0; pass < 2 && todo; ++pass) {
        const int leader = __builtin_ctzll(todo);
        const int c0 = __shfl(c, leader);
        const bool mine = active && c == c0;
        uint32_t m = mine ? v : 0xffffffffu;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t other = (uint32_t)__shfl_xor((int)m, o);
            m = other < m ? other : m;
        }
        if (lane == leader) min_into(&slots[c0], m);
        const unsigned long long served = __ballot(mine);
        todo &= ~served;
        active = active && !mine;
    }
    if (active) min_into(&slots[c], v);
}

// Slot of this thread among the threads of the grid that pass `mine`, behind *counter: one atomic per
// workgroup (per-vertex or per-wavefront atomics on the one counter word serialise: 15 600 of them took
// 0.18 ms at N = 1M).  Every thread of the workgroup must call it.
template <int THREADS>
__device__ inline int block_append(bool mine, int32_t* counter)
{
    __shared__ int wave_count[THREADS / 64];
    __shared__ int wave_base[THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long mask = __ballot(mine);
    if (lane == 0) wave_count[wave] = __popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
        for (int w = 0; w < THREADS / 64; ++w) { wave_base[w] = total; total += wave_count[w]; }
        const int base = total > 0 ? atomicAdd(counter, total) : 0;
        for (int w = 0; w < THREADS / 64; ++w) wave_base[w] += base;
    }
    __syncthreads();
    const int pre = __builtin_amdgcn_mbcnt_hi((unsigned int)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)mask, 0u));
    return mine ? wave_base[wave] + pre : -1;
}

}  // namespace slhc
