// Device helpers: reductions over the lanes of a wavefront; for the forest rounds and the half-precision engine per-component minima and
// list appends with one atomic per wavefront or workgroup.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace slhc {

// The two children of a merge: a caller's array, which may begin at any word.
typedef int v2i_word __attribute__((ext_vector_type(2), aligned(4)));

// One step of a reduction: op(x, x of lane ^ O), op commutative.  From 4 on the lanes of an aligned group of O have to hold the same value, as
// they do after the steps 1, 2, .. O / 2: within 16 lanes the mirrored lane stands in for lane ^ O.  Vector instructions of 4 cycles, where
// __shfl_xor goes through LDS and waits for it.
template <int O, typename F>
__device__ inline unsigned int lanes_step(unsigned int x, F&& op)
{
    static_assert(O == 1 || O == 2 || O == 4 || O == 8 || O == 16 || O == 32, "");
    if constexpr (O <= 8) {
        constexpr int CTRL = O == 1 ? 0xb1 : O == 2 ? 0x4e : O == 4 ? 0x141 : 0x140;     // quad_perm 1 0 3 2, 2 3 0 1, row_half_mirror, row_mirror
        return op(x, (unsigned int)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true));
    } else {
        // (both halves of every pair of rows, or of the wavefront, to either of them)
        const auto r = O == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false) : __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return op((unsigned int)r[0], (unsigned int)r[1]);
    }
}
template <int O> __device__ inline float lanes_add(float x)
{
    return __uint_as_float(lanes_step<O>(__float_as_uint(x), [](unsigned int a, unsigned int b) { return __float_as_uint(__uint_as_float(a) + __uint_as_float(b)); }));
}
template <int O> __device__ inline float lanes_min(float x)
{
    return __uint_as_float(lanes_step<O>(__float_as_uint(x), [](unsigned int a, unsigned int b) { return __float_as_uint(fminf(__uint_as_float(a), __uint_as_float(b))); }));
}
template <int O> __device__ inline float lanes_max(float x)
{
    return __uint_as_float(lanes_step<O>(__float_as_uint(x), [](unsigned int a, unsigned int b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); }));
}
template <int O> __device__ inline unsigned int lanes_min(unsigned int x)
{
    return lanes_step<O>(x, [](unsigned int a, unsigned int b) { return a < b ? a : b; });
}
template <int O> __device__ inline int lanes_or(int x)
{
    return (int)lanes_step<O>((unsigned int)x, [](unsigned int a, unsigned int b) { return a | b; });
}
template <int O> __device__ inline unsigned long long lanes_min(unsigned long long x)
{
    if constexpr (O <= 8) {
        const unsigned int lo = lanes_step<O>((unsigned int)x, [](unsigned int, unsigned int b) { return b; });
        const unsigned int hi = lanes_step<O>((unsigned int)(x >> 32), [](unsigned int, unsigned int b) { return b; });
        const unsigned long long other = ((unsigned long long)hi << 32) | lo;
        return other < x ? other : x;
    } else {
        const unsigned int lo = (unsigned int)x, hi = (unsigned int)(x >> 32);
        const auto l = O == 16 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false) : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = O == 16 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false) : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        const unsigned long long a = ((unsigned long long)(unsigned int)h[0] << 32) | (unsigned int)l[0], b = ((unsigned long long)(unsigned int)h[1] << 32) | (unsigned int)l[1];
        return a < b ? a : b;
    }
}
// over FROM, 2 FROM, .. lanes apart: of FROM = 1 all 64 lanes, every lane holds the result
template <int FROM = 1, typename T> __device__ inline T wave_min(T x)
{
    if constexpr (FROM < 64) return wave_min<2 * FROM>(lanes_min<FROM>(x));
    else return x;
}
template <int FROM = 1> __device__ inline float wave_max(float x)
{
    if constexpr (FROM < 64) return wave_max<2 * FROM>(lanes_max<FROM>(x));
    else return x;
}
// the sum of 8 neighbouring lanes' values, added in a tree of neighbours, pairs and fours
__device__ inline float lanes_add8(float x) { return lanes_add<4>(lanes_add<2>(lanes_add<1>(x))); }

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
        const uint32_t m = wave_min(mine ? v : 0xffffffffu);
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
