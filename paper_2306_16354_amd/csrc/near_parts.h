// Device parts that the passes of the half-precision engine share: bounds between product values and distances, the search for
// the k-th largest of a wavefront's values, loads into LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "near_kernels.h"
#include "wave_ops.h"

namespace slhc {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f_word __attribute__((ext_vector_type(4), aligned(4)));      // global loads of 16 bytes need the alignment of a word only

constexpr int TILE = 128;
constexpr int FRAG_STEP = 4096;            // bytes of a tile per 16 columns
constexpr int REG_STEPS = 8;               // up to 128 columns the query fragments stay in registers
constexpr float F16_LIMIT = 60000.f;       // larger values (after scaling) do not fit
constexpr float F16_FLUSH = 6.103515625e-05f;   // 2^-14: smaller ones are rounded to 0, so no subnormal is ever multiplied
constexpr float INF = __builtin_inff();
constexpr float LOWEST = -3.4028234663852886e38f;      // a bound every product value of a real row reaches
#define NEVER __builtin_nanf("")                       // a bound nothing reaches, +inf included

// What the arithmetic on the rounded rows can be off by.  An instruction aligns its 16 products and the accumulator
// to the largest magnitude, one bit below its last place, cuts the rest off, adds and rounds: at most 18 units of
// 2^-24 of that magnitude (6.0 measured at most, over 3 million sums against 64 bits: test_f16_mfma_error_stays_within_the_budget).
// The accumulator starts at minus half the candidate's squared norm n_c.  With a, b the first columns of the query and of the
// candidate, a . b = (|a|^2 + |b|^2 - |a - b|^2) / 2, so a partial sum lies between -n_c / 2 - D^2 / 2 and n_q / 2 for rows a distance
// D apart; and all products together have at most the magnitude (n_q + n_c) / 2.  After `steps` instructions the value is off by at most
//     kappa (steps (max(n_q, n_c) / 2 + D^2 / 2) + (n_q + n_c) / 2),   kappa = 18 2^-24,
// and since |n_q - n_c| <= D (2 |x_q| + D), by at most e (n_q + n_c) + f (D |x_q| / 2 + 5/4 D^2) with e = kappa (steps / 4 + 1 / 2) and
// f = kappa steps, for either row in the role of the query: a pair's one product may serve both (pairs_kernels.hip).
// (Counting every partial sum as n_c + n_q / 2 instead: 1M x 128 in the row order evaluated 46.9 pairs per row exactly instead of 43.8.)
// nu: the relative error of a squared norm (8 ceil(steps / 8) + 8 rounded additions).  The stored half norms are lowered by what
// belongs to the candidate: a value `acc` is never below the true one by more than e n_q + f (...).
struct NearBoundArgs { float e, f, nu, h_of_n, eps, delta, gamma, tiny; };
static float near_kappa() { return 9.f * 1.02f * 1.1920928955078125e-07f; }
static float near_e(int steps) { return near_kappa() * (0.25f * (float)steps + 0.5f); }
static float near_nu(int steps) { return (float)(8 * ((steps + 7) / 8) + 8) * 5.9604644775390625e-08f; }

// The product value any row within (scaled, squared) distance t2 of the query reaches; h: the query's stored half norm.
// (8 units of 2^-24 of n for the roundings here and of limits and values that have h added or taken off)
__device__ inline float near_bound_at(float t2, float h, const NearBoundArgs& a)
{
    const float n = h / a.h_of_n;
    const float norm = __builtin_sqrtf(n);
    // what the exact evaluation's own rounding can hide, and underflow of its squares
    const float t = __builtin_sqrtf(t2 * (1.f + a.gamma) + a.tiny);
    const float rho_q = a.eps * norm + a.delta;
    // a candidate within t of the query has a norm of at most norm + t + both displacements
    const float rho_c = (a.eps * (norm + t + rho_q) + a.delta) * (1.f + 1e-3f);
    const float reach = (t + rho_q + rho_c) * (1.f + 1e-6f);
    return n * (0.5f - 0.5f * a.nu - a.e - 4.8e-7f) - 0.5f * reach * (reach * (1.f + 2e-6f + 2.5f * a.f) + a.f * norm);
}
// From a product value some candidate shows: an upper bound of that candidate's distance (its squared norm n_c is at
// most (|x_q| + D)^2 <= 9/8 n_q + 9 D^2, and D |x_q| at most n_q / 8 + 2 D^2), and from it the bound for all candidates that
// may be as near.
__device__ inline float near_distance_from(float acc, float h, const NearBoundArgs& a)
{
    const float n = h / a.h_of_n;
    const float norm = __builtin_sqrtf(n);
    const float of_c = 4.f * a.e + 2.f * a.nu, of_d = 4.5f * a.f + 9.f * of_c;
    if (of_d > 0.9f) return INF;                                // (hundreds of thousands of columns)
    const float d2 = fmaxf(0.f, n * (1.f + a.nu + 2.f * a.e + 1.125f * of_c + 0.125f * a.f + 9.6e-7f) - 2.f * acc) / (1.f - of_d) * (1.f + 1e-6f);
    const float dd = __builtin_sqrtf(d2);
    const float rho_q = a.eps * norm + a.delta;
    const float rho_c = (a.eps * (norm + dd) + a.delta) * (1.f + 1e-3f);
    return (dd + rho_q + rho_c) * (1.f + 1e-6f);
}
__device__ inline float near_bound_from(float acc, float h, const NearBoundArgs& a)
{
    const float t = near_distance_from(acc, h, a);
    return t < INF ? near_bound_at(t * t * (1.f + a.gamma), h, a) : LOWEST;
}
// near_bound_at the other way round: no row whose product value is `acc` at most is within this (scaled, squared) distance.
__device__ inline float near_lower_from(float acc, float h, const NearBoundArgs& a)
{
    const float n = h / a.h_of_n;
    const float norm = __builtin_sqrtf(n);
    const float rho_q = a.eps * norm + a.delta;
    const float reach2 = (2.f * (n * (0.5f - 0.5f * a.nu - a.e - 4.8e-7f) * (1.f - 1e-6f) - acc) - 0.125f * a.f * n) / (1.f + 4.5f * a.f) * (1.f - 6e-6f);
    const float reach = __builtin_sqrtf(fmaxf(0.f, reach2)) * (1.f - 4e-6f);
    const float t = (reach - rho_q - (a.eps * (norm + rho_q) + a.delta) * (1.f + 2e-3f)) / (1.f + a.eps * (1.f + 2e-3f)) * (1.f - 4e-6f);
    return t > 0.f ? fmaxf(0.f, (t * t * (1.f - 4e-6f) - a.tiny) / (1.f + a.gamma) * (1.f - 4e-6f)) : 0.f;
}

__device__ inline NearBoundArgs near_args(const NearScale* sc, int steps, int d, float e, float nu)
{
    NearBoundArgs a;
    a.e = e; a.nu = nu;
    a.f = 9.f * 1.02f * 1.1920928955078125e-07f * (float)steps;
    a.h_of_n = 0.5f - 0.5f * nu - e;
    a.eps = fminf(__uint_as_float(sc->eps_bits), 4.8876e-4f) * (1.f + 1e-3f);      // 2^-11 at most
    a.delta = F16_FLUSH * __builtin_sqrtf((float)d);
    a.gamma = (float)(2 * (d + 16)) * 1.1920928955078125e-07f;
    a.tiny = (float)d * 2.350988701644575e-38f * sc->scale * sc->scale;            // d * 2^-125
    return a;
}

__device__ inline float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

__device__ inline unsigned int ordered_bits(float x)
{
    const unsigned int b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
// A value that at least kk of the wavefront's values v(i), i < n, reach, and not many more: bisection between the
// smallest and the largest of them.  Values that are not finite do not count.  Returns LOWEST when fewer than kk are.
// BISECT_FAR: where the ends may be a thousand times farther apart than the values in question and a list overflows for it (one
// group of a sample without a row of the query's cluster).
constexpr int BISECT = 13, BISECT_FAR = 20;
template <typename V>
__device__ inline float near_kth(int n, int kk, V&& value)
{
    float lo = INF, hi = -INF;
    int have = 0;
    for (int i = 0; i < n; i += 64) {
        const float x = value(i);
        const bool fine = fabsf(x) < INF;
        have += __popcll(__ballot(fine));
        lo = fine ? fminf(lo, x) : lo;
        hi = fine ? fmaxf(hi, x) : hi;
    }
    if (have < kk) return LOWEST;
    lo = wave_min(lo); hi = wave_max(hi);
    for (int it = 0; it < BISECT; ++it) {
        const float mid = 0.5f * lo + 0.5f * hi;
        int reach = 0;
        for (int i = 0; i < n; i += 64) {
            const float x = value(i);
            reach += __popcll(__ballot(x >= mid && x < INF));
        }
        if (reach >= kk) lo = mid; else hi = mid;
    }
    return lo;
}

// The same of at most 64 W values, kept in registers on the way.
template <int W, typename V>
__device__ inline float near_kth_of(int n, int kk, V&& value)
{
    float v[W], lo = INF, hi = -INF;
    int have = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) v[j] = value(64 * j);
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const bool fine = fabsf(v[j]) < INF;
        have += __popcll(__ballot(fine));
        lo = fine ? fminf(lo, v[j]) : lo;
        hi = fine ? fmaxf(hi, v[j]) : hi;
        v[j] = fine ? v[j] : -INF;
    }
    if (have < kk) return LOWEST;
    lo = wave_min(lo); hi = wave_max(hi);
    for (int it = 0; it < BISECT; ++it) {
        const float mid = 0.5f * lo + 0.5f * hi;
        int reach = 0;
#pragma unroll
        for (int j = 0; j < W; ++j) reach += __popcll(__ballot(v[j] >= mid));
        if (reach >= kk) lo = mid; else hi = mid;
    }
    return lo;
}

// 64 consecutive quads, or words `stride` bytes apart, from `at` bytes behind `base` (both the same for all lanes) to LDS, one a lane.
// As buffer loads: with the same loads as global_load_lds, which count as accesses through flat addresses, the compiler has every wait for
// an LDS read wait for all of them (lgkmcnt(0)), and the fragments of the next step, read ahead of a step's multiplies, are waited for before these.
// Clustering 250k x 784 130 -> 121 ms, cross 1-NN 10 000 in 100 000 x 64 255 -> 248 us, 100k x 64 5.86 -> 5.80 ms; 1M x 128 as it was.
__device__ inline void near_lds_load(const void* base, unsigned int at, void* l, bool quad, int stride = 4)
{
    const int lane = threadIdx.x & 63;
    at = __builtin_amdgcn_readfirstlane(at);           // (the compiler may keep it in a vector register, and would loop over its values)
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, -1, 0x00020000);      // (raw words, no end)
    if (quad)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)l, 16, lane * 16, at, 0, 0);
    else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)l, 4, lane * stride, at, 0, 0);
}
// A quad of each lane's own.  Past the compiler, see near_lds_load; who waits for the tile waits for these loads too.
__device__ inline void near_lds_gather(const void* g, void* l)
{
    unsigned int m0;                             // (the compiler's)
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0) : "s"((unsigned int)(uintptr_t)(__attribute__((address_space(3))) void*)l), "v"(g) : "memory");
}

// Waits for this wavefront's loads into LDS, then for the other wavefronts.
__device__ inline void near_lds_ready()
{
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Beyond 128 columns a step of the pipeline is a chunk of 32 columns of both sides, 32 KiB, in one of four buffers: the loads run three chunks ahead, and the
// fragments of a chunk's first 16 columns are read while the last ones of the chunk before are multiplied, so that after a barrier there is
// something to multiply at once.  250k x 784, the pass for the k-NN graph and that for the first connection round: 48.6 and 49.1 ms with chunks of 64
// columns in two buffers, every fragment read after the chunk's barrier and all reads waited for at once; 44.8 and 46.4 so (1.09 PFLOP/s of
// products made once; the matrix pipe 60 % of the busy cycles, 51 to 54 before, at 1.8 to 1.9 GHz, to which it throttles, 1.9 to 2.0 before).
constexpr int CHUNK_STEPS = 2;
constexpr int CHUNK_TILE = CHUNK_STEPS * FRAG_STEP;
constexpr int CHUNK_SIDE = 2 * CHUNK_TILE;
constexpr int CHUNK = 2 * CHUNK_SIDE;
constexpr int CHUNKS = 4;                                               // buffers

// In the pass over a chunk, before its second step is read.  The next chunk is in LDS once all of this wavefront's loads are done but the
// four of the chunk after that (one_after: there is one), and every wavefront has read the chunk before this one, whose buffer is filled next:
// what may still be on its way are the six fragments of this chunk's first step.
__device__ inline void near_chunk_ready(bool one_after)
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (one_after) __builtin_amdgcn_s_waitcnt(0x0674);     // vmcnt(4) lgkmcnt(6)
    else __builtin_amdgcn_s_waitcnt(0x0670);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Where the rows of a matrix lie in a copy that is not in their order: row b * tiles + i, i < tiles, in tile i + near_shift(b) and there, in
// the same 32 as place b, at place b - near_turn(tile), both round and round.  So a tile has one row of every stretch of `tiles` rows and is
// an even sample of them, whatever order they are in.  The shift: where row i is of cluster i % n, and n and `tiles` have a divisor in
// common, tile i would have the rows of a few clusters only.  The turn: where rows lie in the order of their clusters, the same place of all
// tiles would have the rows of one, and the groups that a sample's maxima are taken of are places of 32.  (Turned by up to 128, short rows
// that share a cache line are read by workgroups of several XCDs: near_make of 400 000 x 8 40.4 us, 37.8 so.)
__device__ inline int near_turn(int tile) { return (int)(((unsigned int)tile * 0x9e3779b1u) >> 27); }
__device__ inline int near_shift(int b, int tiles) { return (int)__umulhi((unsigned int)b * 0x9e3779b1u, (unsigned int)tiles); }
__device__ inline long long near_row(int pos, int tiles, int in_order)
{
    if (in_order) return pos;
    const int t = pos >> 7, b = (pos & 96) | ((pos + near_turn(t)) & 31), i = t - near_shift(b, tiles);
    return (long long)b * tiles + (i < 0 ? i + tiles : i);
}
__device__ inline int near_pos(int row, int tiles)             // (not in order)
{
    const int b = row / tiles, i = row - b * tiles + near_shift(b, tiles), t = i < tiles ? i : i - tiles;
    return t * TILE + ((b & 96) | ((b - near_turn(t)) & 31));
}

// A panel of 128 rows goes to the list kernels, known before what is there of its rows' lists is looked through.
constexpr int PANEL_GONE = 2;
__device__ inline void near_panel_gone(int32_t* todo, int32_t* todo_mark, int panel)
{
    // (a hundred thousand rows may say so of forty panels, one exchange after another: 5000 x 12 of 2000 copies each 4.8 ms, 4.2 with the look)
    if (__hip_atomic_load(todo_mark + panel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == PANEL_GONE) return;
    if (atomicExch(todo_mark + panel, PANEL_GONE) == 0) todo[2 + atomicAdd(todo, 1)] = panel;
}

// i * near_spread(n) % n for i = 0, 1, ...: the numbers below n in an order whose every stretch is spread evenly over them (n times the
// golden ratio, or the next number that has no divisor in common with n).  Products below 2^32: up to n = 2^17, beyond that as they are.
inline int near_spread(int n)
{
    if (n > 1 << 17) return 1;
    int m = (int)(0.6180339887498949 * n);
    for (m = m < 1 ? 1 : (m > 32000 ? 32000 : m);; ++m) {
        int a = m, b = n;
        while (b) { const int r = a % b; a = b; b = r; }
        if (a == 1) return m;
    }
}
__device__ inline int near_spread_at(int i, int spread, int n) { return (int)((unsigned int)i * (unsigned int)spread % (unsigned int)n); }

}  // namespace slhc
