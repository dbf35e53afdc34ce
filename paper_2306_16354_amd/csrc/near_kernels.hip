// Nearest rows by float16 tile products: threshold, emit, select.
//
// The tile products of the sweeps only decide which pairs are evaluated exactly, so what they need is not float32
// products but a bound on what rounding can do.  Here every row is rounded ONCE to float16 (relative to a central
// value of every column and times a power of two) and the products of the rounded rows are exact: 11 x 11 bits.  The
// distance of the rounded rows then differs from that of the rows by no more than the two rows moved,
//     |D(x, y) - D(x', y')| <= |x - x'| + |y - y'|      (triangle inequality),
// a few 1e-4 of the rows' norms.  One v_mfma_f32_32x32x16_f16 per 16 columns does what the split bfloat16 copy needs
// three instructions for, on half the bytes.
//
// A k-NN search runs in four launches instead of keeping lists inside the sweep:
//   1. maxima   every query takes the largest product value in each of 32 groups per part of an even sample of the
//               candidates; the k-th largest of all its group maxima is a threshold that k candidates reach;
//   2. bounds   that value per query, turned into the product value any of its k nearest rows must reach;
//   3. emit     all candidates against that fixed bound; the few that pass are appended to a buffer of the lane that
//               found them (no list, no exact evaluation, no exchange between lanes in the loop);
//   4. select   per query: a tighter bound from what was emitted, exact evaluation of what is left, ranks.
// A 1-NN search needs no first pass: its bound follows the best product value seen so far.
//
// Every reported distance is the same float32 sum in the same order as in the list kernels (sweep_kernels.hip), so
// the results are the same bits.  A query whose candidates do not fit its buffers even after tightening (masses of
// ties) is left to the list kernels through a device-side list of panels.
#include <hip/hip_runtime.h>
#include <cmath>
#include <stdint.h>
#include "near_kernels.h"
#include "near_parts.h"
#include "pairs_kernels.h"
#include "wave_ops.h"

namespace slhc {

constexpr int SAMPLE_RUNS = 64, SAMPLE_PER_RUN = 32;
constexpr int MAX_ENTRIES = 1024;          // entries of one query over all its buffers
constexpr int GROUPS = 32;                 // group maxima per query and part

// ---------------------------------------------------------------------------------------------- sample of the rows
// Column means of SAMPLE_RUNS runs of evenly spaced rows, and per run the largest distance of a value from its run's
// mean.  One workgroup per run and 256 columns; the additions of a run keep a fixed order.
__global__ void __launch_bounds__(256) near_runs_kernel(const float* __restrict__ X, int n, int d, float* __restrict__ partial,
                                                        float* __restrict__ run_max, NearScale* __restrict__ sc,
                                                        uint32_t* __restrict__ clear, int clear_words, int32_t* __restrict__ todo,
                                                        long long todo_words)
{
    {   // words that later launches of this call expect to be 0
        const long long at = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
        const long long step = (long long)gridDim.x * gridDim.y * 256;
        for (long long i = at; i < todo_words; i += step) todo[i] = 0;
        for (long long i = at; i < clear_words; i += step) clear[i] = 0u;
    }
    __shared__ float sums[256], cnts[256], mx[256];
    const int run = blockIdx.x, tid = threadIdx.x;
    const int c0 = blockIdx.y * 256;
    const int cols = d - c0 < 256 ? d - c0 : 256;
    int log = 0;
    while (1 << log < cols) ++log;
    const int width = 1 << log, sub = 256 >> log;           // threads per row, rows side by side
    const int c = tid & (width - 1), g = tid >> log;
    // (sample i is row i n / samples; `samples` is n or a power of two, and must not be divided by: a division of 64 bits per sample made this
    // kernel 31 KB of code, read anew by every call: 6.9 us, 4.9 so)
    constexpr int MOST = SAMPLE_RUNS * SAMPLE_PER_RUN;
    static_assert((MOST & (MOST - 1)) == 0, "the division below is a shift");
    const bool every = n < MOST;
    const int samples = every ? n : MOST;
    const int i0 = (int)((long long)run * samples / SAMPLE_RUNS), i1 = (int)((long long)(run + 1) * samples / SAMPLE_RUNS);
    float v[SAMPLE_PER_RUN];
    float sum = 0.f, cnt = 0.f;
#pragma unroll
    for (int j = 0; j < SAMPLE_PER_RUN; ++j) {
        const int i = i0 + g + j * sub;
        v[j] = __builtin_nanf("");
        if (c < cols && i < i1) v[j] = X[(every ? (size_t)i : (size_t)i * (size_t)n / MOST) * d + c0 + c];
    }
#pragma unroll
    for (int j = 0; j < SAMPLE_PER_RUN; ++j)
        if (fabsf(v[j]) < INF) { sum += v[j]; cnt += 1.f; }        // false for NaN
    sums[tid] = sum; cnts[tid] = cnt;
    __syncthreads();
    float mean = 0.f;
    {
        float s = 0.f, m = 0.f;
        for (int q = 0; q < sub; ++q) { s += sums[q * width + c]; m += cnts[q * width + c]; }
        mean = m > 0.f ? s / m : __builtin_nanf("");
    }
    float far = 0.f;
#pragma unroll
    for (int j = 0; j < SAMPLE_PER_RUN; ++j) {
        const float e = fabsf(v[j] - mean);
        if (e < INF) far = fmaxf(far, e);
    }
    mx[tid] = far;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) mx[tid] = fmaxf(mx[tid], mx[tid + w]);
        __syncthreads();
    }
    if (g == 0 && c < cols) partial[(size_t)run * d + c0 + c] = mean;
    if (tid == 0) run_max[blockIdx.y * SAMPLE_RUNS + run] = i1 > i0 ? mx[0] : -1.f;
    if (run == 0 && blockIdx.y == 0 && tid == 0) { sc->eps_bits = 0u; sc->huge = 0u; }
}

// the two middle values of 64 lanes' valid ones, averaged (0 valid: 0)
__device__ inline float near_median64(float x, bool valid, int lane)
{
    const int n = __popcll(__ballot(valid));
    int rank = 0;
    const float key = valid ? x : INF;
#pragma unroll
    for (int q = 0; q < 64; ++q) {
        const float y = __uint_as_float((unsigned int)__builtin_amdgcn_readlane((int)__float_as_uint(key), q));
        if (y < x || (y == x && q < lane)) ++rank;
    }
    float pick = 0.f;
    if (valid && n > 0) {
        if (rank == ((n - 1) >> 1)) pick += 0.5f * x;
        if (rank == (n >> 1)) pick += 0.5f * x;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) pick += __shfl_xor(pick, o);
    return pick;
}

// shift[c] = the median of the runs' means (a single far row cannot drag it; a value beyond 2^50 is replaced by 0), and
// the scale: the power of two that brings the median run's largest value near 2^7.  float16 then has room for rows
// 500 times larger and keeps its full relative precision for values 2 million times smaller.  The runs' means of column 0 become the words
// in which near_make's workgroups meet: 0.
__global__ void __launch_bounds__(256) near_shift_kernel(float* __restrict__ partial, const float* __restrict__ run_max, int d,
                                                         float* __restrict__ shift, NearScale* __restrict__ sc)
{
    const int lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c < d) {
        const float x = partial[(size_t)lane * d + c];
        const float m = near_median64(x, fabsf(x) < INF, lane);
        if (lane == 0) shift[c] = fabsf(m) <= 1.125899906842624e15f ? m : 0.f;
        if (c == 0) partial[(size_t)lane * d] = 0.f;
    } else if (c == d) {
        float x = -1.f;
        const int parts = (d + 255) / 256;
        for (int y = 0; y < parts; ++y) x = fmaxf(x, run_max[y * SAMPLE_RUNS + lane]);
        float m = near_median64(x, x > 0.f, lane);
        if (lane == 0) {
            int e = 0;
            if (m > 0.f && m < INF) (void)frexpf(m, &e);              // m = f * 2^e, f in [0.5, 1)
            int up = 7 - e;
            up = up < -100 ? -100 : (up > 100 ? 100 : up);
            sc->scale = ldexpf(1.f, up);
        }
    }
}

size_t near_stats_scratch_floats(int d) { return (size_t)SAMPLE_RUNS * (size_t)d + (size_t)SAMPLE_RUNS * (size_t)((d + 255) / 256); }

hipError_t near_stats(const float* X, int n, int d, const NearBuffers& b, uint32_t* clear, int clear_words, hipStream_t s)
{
    float* run_max = b.partial + (size_t)SAMPLE_RUNS * d;
    hipLaunchKernelGGL(near_runs_kernel, dim3(SAMPLE_RUNS, (unsigned)((d + 255) / 256)), dim3(256), 0, s, X, n, d, b.partial, run_max, b.scale,
                       clear, clear_words, b.todo, 2 + 2 * b.todo_panels);
    hipLaunchKernelGGL(near_shift_kernel, dim3((unsigned)(d / 4 + 1)), dim3(256), 0, s, b.partial, run_max, d, b.shift, b.scale);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------- the float16 copy
struct NearMake {
    const float* X; const int32_t* rows; const int32_t* colour; const float* shift; NearScale* sc;
    const int32_t* shift_row;            // optional: tile t is taken relative to row shift_row[t] of `shift` (-1: is left empty)
    unsigned char* frag; float *negh, *negh_best; int32_t* out_colour; float* hn; unsigned int* nonfinite;
    unsigned int* eps_of;                // optional: 64 words, d apart, none above what sc->eps_bits will be
    int n_src, n, d, tiles, steps, in_order; float h_of_n, hn_scale, absent;
    const int32_t* n_dev;
    int32_t* count; unsigned long long* best_at;
    int32_t* todo; long long todo_words;
};

// One workgroup per block of 32 rows of a tile; LPR lanes share a row, eight columns each at a time.  The pieces go
// through LDS so that they leave in whole lines.  Bound by reading X once and writing half of it (1M x 128: 180 us, 4.3 TB/s; 215 with the shift
// read a word at a time), and below a million rows by the workgroups' reports at its end: 100 000 x 64 29 us, 17 with the words in 64 lines, 14
// without; 100 000 x 128 28 and 22.  (The 64 words in one line: 26 us, and 40 if they are read first.  A thousand workgroups that pass over the blocks:
// 23, but 240 us for 1M x 128.)
constexpr int MAKE_STEPS = 8;
template <int LPR, bool VEC4>
__global__ void __launch_bounds__(256) near_make_kernel(NearMake p)
{
    __shared__ __align__(16) unsigned char stage[MAKE_STEPS * 1024];
    __shared__ unsigned int eps_max;
    const int tid = threadIdx.x;
    const int t = blockIdx.x >> 2, blk = blockIdx.x & 3;
    const int n_in = p.n_dev ? (*p.n_dev < p.n ? *p.n_dev : p.n) : p.n;
    if (p.n_dev && t * TILE >= n_in) return;         // (copies of unknown length are in order)
    constexpr int ROWS = 256 / LPR;                  // rows side by side
    constexpr int PASSES = ROWS >= 32 ? 1 : 32 / ROWS;
    const int part = tid % LPR, sub = tid / LPR;
    const bool mine = sub < 32;
    const float scale = p.sc->scale;
    const float* __restrict__ shift = p.shift_row ? p.shift + (size_t)(p.shift_row[t] < 0 ? 0 : p.shift_row[t]) * p.d : p.shift;
    const bool empty = p.shift_row && p.shift_row[t] < 0;
    if (tid == 0) eps_max = 0u;
    for (long long i = (long long)blockIdx.x * 256 + tid; i < p.todo_words; i += (long long)gridDim.x * 256) p.todo[i] = 0;
    float nn[PASSES], rr[PASSES], xx[PASSES];
    bool huge[PASSES];
    long long src[PASSES];
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        nn[i] = rr[i] = xx[i] = 0.f; huge[i] = false;
        const int in_tile = blk * 32 + sub + i * ROWS;
        const long long at = near_row(t * TILE + in_tile, p.tiles, p.in_order);
        long long row = mine && at < n_in && !empty ? (p.rows ? (long long)p.rows[at] : at) : -1;
        if (row >= p.n_src) row = -1;
        src[i] = row;
    }
    for (int s0 = 0; s0 < p.steps; s0 += MAKE_STEPS) {
        const int ns = p.steps - s0 < MAKE_STEPS ? p.steps - s0 : MAKE_STEPS;
        for (int oct = part; oct < 2 * ns; oct += LPR) {
            const int col = 16 * s0 + 8 * oct;
            float m[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) m[e] = 0.f;
            if (VEC4) {
#pragma unroll
                for (int e = 0; e < 8; e += 4)
                    if (col + e + 4 <= p.d) {
                        const v4f a = *reinterpret_cast<const v4f*>(shift + col + e);
                        m[e] = a[0]; m[e + 1] = a[1]; m[e + 2] = a[2]; m[e + 3] = a[3];
                    }
            } else
#pragma unroll
                for (int e = 0; e < 8; ++e) m[e] = col + e < p.d ? shift[col + e] : 0.f;
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                const int r = sub + i * ROWS;
                float v[8];
                const float* x = p.X + (size_t)(src[i] < 0 ? 0 : src[i]) * p.d + col;
                if (VEC4) {
                    v4f a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
                    if (src[i] >= 0 && col + 4 <= p.d) a = *reinterpret_cast<const v4f*>(x);
                    if (src[i] >= 0 && col + 8 <= p.d) b = *reinterpret_cast<const v4f*>(x + 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
                } else {
                    // rows that begin on any word, 16 bytes at a time all the same; the last values of a row come from its last eight, moved
                    // down (a branch of its own for them costs another wait: 20 011 x 50 11.5 us, 9.4 so, by single values 8.4;
                    // 1000 x 100 000 x 99 fused search 133 us by single values, 122 so)
                    const int left = src[i] < 0 ? 0 : p.d - col;
                    if (p.d >= 8) {
                        const int by = left >= 8 ? 0 : 8 - left;
                        v4f a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
                        if (left > 0) { a = reinterpret_cast<const v4f_word*>(x - by)[0]; b = reinterpret_cast<const v4f_word*>(x - by)[1]; }
#pragma unroll
                        for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
#pragma unroll
                        for (int o = 4; o > 0; o >>= 1)
#pragma unroll
                            for (int e = 0; e < 8; ++e) v[e] = (by & o) ? (e + o < 8 ? v[e + o < 8 ? e + o : e] : 0.f) : v[e];
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = e < left ? x[e] : 0.f;
                    }
                }
                v8h h;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bool live = src[i] >= 0 && col + e < p.d;
                    xx[i] = __builtin_fmaf(v[e], v[e], xx[i]);
                    float u = live ? (v[e] - m[e]) * scale : 0.f;
                    if (fabsf(u) > F16_LIMIT) huge[i] = true;
                    u = fminf(fmaxf(u, -F16_LIMIT), F16_LIMIT);        // NaN becomes a number here; its row is cut off below
                    const bool flush = fabsf(u) < F16_FLUSH;
                    const _Float16 q = flush ? (_Float16)0.f : (_Float16)u;
                    const float w = (float)q;
                    h[e] = q;
                    nn[i] = __builtin_fmaf(w, w, nn[i]);
                    const float res = flush ? 0.f : u - w;             // (flushed values: delta covers them)
                    rr[i] = __builtin_fmaf(res, res, rr[i]);
                }
                if (mine) *reinterpret_cast<v8h*>(stage + (oct >> 1) * 1024 + ((oct & 1) * 32 + r) * 16) = h;
            }
        }
        __syncthreads();
        unsigned char* dst = p.frag + ((size_t)t * p.steps + s0) * FRAG_STEP + blk * 1024;
        for (int i = tid; i < ns * 64; i += 256)
            *reinterpret_cast<v4f*>(dst + (size_t)(i >> 6) * FRAG_STEP + (i & 63) * 16) = reinterpret_cast<const v4f*>(stage)[i];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        float n = lanes_add8(nn[i]), r = lanes_add8(rr[i]), x = lanes_add8(xx[i]);
        int hg = lanes_or<4>(lanes_or<2>(lanes_or<1>(huge[i] ? 1 : 0)));
        if (LPR == 16) { n = lanes_add<8>(n); r = lanes_add<8>(r); x = lanes_add<8>(x); hg = lanes_or<8>(hg); }
        if (part == 0 && mine) {
            const int at = t * TILE + blk * 32 + sub + i * ROWS;
            float nh = -p.h_of_n * n;
            if (hg) nh = INF;
            if (src[i] < 0 || !(x < INF)) nh = p.absent;         // no row, or one whose squared norm is not a finite float32
            p.negh[at] = nh;
            if (p.negh_best) p.negh_best[at] = nh == INF ? p.absent : nh;
            if (hg && src[i] >= 0) p.sc->huge = 1u;
            if (p.out_colour) p.out_colour[at] = src[i] >= 0 && p.colour ? p.colour[src[i]] : -1;
            if (p.best_at) p.best_at[at] = ~0ull;
            if (p.count) p.count[at] = 0;
            if (src[i] >= 0) {
                if (p.hn) p.hn[src[i]] = p.hn_scale * x;
                if (p.nonfinite && !(x < INF)) atomicOr(p.nonfinite, 1u);
                if (!hg && n > 0.f && r > 0.f) atomicMax(&eps_max, __float_as_uint(__builtin_sqrtf(r / n)));
            }
        }
    }
    __syncthreads();
    // (2 units in the last place for the roundings of the two sums and of the difference from the shift)
    if (tid == 0 && eps_max != 0u) {
        const unsigned int mine_bits = __float_as_uint(__uint_as_float(eps_max) * (1.f + 1e-4f));
        // Most workgroups find the word already there and leave it alone; but the first two thousand of a launch end together and would
        // queue for it (9 ns each), so they meet at 64 words, a row of the column statistics apart, and a few of each 32 go on.  (In lines of
        // their own from 32 columns on, eight of them in one line at 4 columns: the 1-NN of 1000 queries in 1M x 4 214 -> 200 us, in 1M x 32 251 -> 222.)
        const bool first = !p.eps_of || atomicMax(p.eps_of + (size_t)(blockIdx.x & 63) * p.d, mine_bits) < mine_bits;
        if (first && __hip_atomic_load(&p.sc->eps_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < mine_bits) atomicMax(&p.sc->eps_bits, mine_bits);
    }
}

hipError_t near_make(const float* X, int n_src, int d, const int32_t* rows, int n, const int32_t* colour, const NearBuffers& b,
                     const NearCopy& out, float* hn, unsigned int* nonfinite, hipStream_t s, bool clear_todo, const int32_t* n_dev,
                     const int32_t* shift_row)
{
    if (n_dev && !out.in_order) return hipErrorInvalidValue;
    NearMake p{};
    p.X = X; p.rows = rows; p.colour = colour; p.shift = b.shift; p.sc = b.scale;
    p.frag = out.frag; p.negh = out.negh; p.out_colour = out.colour; p.hn = hn; p.nonfinite = nonfinite;
    p.n_src = n_src; p.n = n; p.d = d; p.tiles = out.tiles; p.steps = near_steps(d); p.h_of_n = 0.5f - 0.5f * near_nu(p.steps) - near_e(p.steps);
    p.shift_row = shift_row;
    p.eps_of = reinterpret_cast<unsigned int*>(b.partial);
    p.count = out.count; p.best_at = out.best_at;
    p.negh_best = out.negh_best; p.in_order = out.in_order; p.n_dev = n_dev;
    p.absent = out.finite_padding ? -1e38f : -INF;
    p.todo = b.todo; p.todo_words = clear_todo ? 2 + 2 * b.todo_panels : 0;
    p.hn_scale = 0.5f * (1.0f - (float)(d + 8) * 1.1920928955078125e-07f);         // as launch_half_norms
    const bool vec4 = d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
    const dim3 grid((unsigned)out.tiles * 4u), block(256);
    if (p.steps <= 4) {
        if (vec4) hipLaunchKernelGGL((near_make_kernel<8, true>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((near_make_kernel<8, false>), grid, block, 0, s, p);
    } else {
        if (vec4) hipLaunchKernelGGL((near_make_kernel<16, true>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((near_make_kernel<16, false>), grid, block, 0, s, p);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------- the sweep
struct NearSweep {
    const unsigned char* qfrag; const float* qnegh; const int32_t* qcolour; int q_tile0, q_tile1;
    const unsigned char* cfrag; const float* cnegh; const int32_t* ccolour; int c_tiles;
    const NearScale* sc; float e, nu; int d, steps;
    // item = panel * nseg + seg; seg takes tiles seg, seg + nseg, ... of a list of `used` candidate tiles: every
    // stride-th one (skip = 0), or all but those (skip = 1); spread: near_spread(used) or 0 (maxima, not listed: in that order, so that a
    // part of them is an even sample of the rows too)
    int nseg, stride, used, skip, spread;
    // queries counted on the device (n_dev, over all batches): the panels that exist share `slots` workgroups in at most
    // most_seg segments each
    const int32_t* n_dev; int slots, most_seg;
    // listed: the candidate tiles of every panel, list_len of them; list_step: every how-manieth is taken (0: none)
    const unsigned short* list; const int32_t* list_len; const int32_t* list_step; int list_stride;
    // block, nearest: the lists are cut into items of ITEM_TILES tiles, panel i has those from items[i] to items[i + 1]
    const int32_t* items; int panels;
    int nsub;                          // buffers per query: the lanes that hold its values, over all segments
    int kk;                            // candidates a query needs (itself included where it meets itself)
    const float* bound;                // emit, nearest (or nullptr): [queries of the batch]
    const float* reach;                // instead of bound: squared distances (rows as they are) that matter, by query; < 0: none
    // queries by position in an order (nullptr: query i is position i), n_q of them unless counted on the device
    const int32_t* qpos; int n_q;
    // Searches in a row order with two copies: `local` (side 1) holds every tile relative to its region and serves the pairs
    // inside one region, the other copy (side 2) all others.  region[tile] < 0: no region.  Entries of side 2 carry `mark`.
    const int32_t* region; int side; unsigned int mark;
    const int32_t* tile_colour;        // listed, coloured: the colour all rows of a tile share, -1 where they differ
    int append;                        // emit: the buffers hold the entries of an earlier launch, whose values do not compare
    float* maxima; int parts, groups;  // maxima: [nseg * parts][queries of the batch][groups], groups 32 or 8
    uint2* entries; int32_t* counts; int capl;      // emit: [queries of the batch][2 nseg][capl], [queries][2 nseg]
                                                    // nearest: [queries of the batch][capl], counts by position
    unsigned long long* best_at;       // arg: (largest product value, candidate position) by query position; block: (distance below
                                       // which there is no candidate, position of the first of the 16 values of a lane in a block
                                       // of 32 candidates the nearest of which is about there)
    uint4* top;                        // top: [queries of the batch][nsub] (largest product value of a lane, position of the first of
                                       // the 16 values it is among, largest outside these 16)
    int nq_batch;
};

enum { NEAR_MAXIMA = 0, NEAR_EMIT = 1, NEAR_TOP = 2, NEAR_NEAREST = 3, NEAR_ARG = 4, NEAR_BLOCK = 5 };

// entries are written and read back by one wavefront, past its L1
__device__ inline unsigned long long near_entry_load(const uint2* e)
{
    return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(e), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One lane's buffer is about to fill: the whole wavefront reads its n entries, finds the kk-th largest product value
// (every one of them belongs to a different candidate, so kk candidates reach it) and keeps the entries that may
// still be among the nearest.  Returns the new bound; *n the number kept.
__device__ __attribute__((noinline)) float near_refine(uint2* buf, int* n_, int kk, float h, NearBoundArgs a)
{
    const int lane = threadIdx.x & 63;
    const int n = *n_;
    __builtin_amdgcn_s_waitcnt(0x0f70);
    const float kth = near_kth(n, kk, [&](int i) {
        return i + lane < n ? __uint_as_float((unsigned int)near_entry_load(buf + i + lane)) : -INF;
    });
    if (kth == LOWEST) return LOWEST;
    const float bound = near_bound_from(kth, h, a);
    int kept = 0;
    for (int i = 0; i < n; i += 64) {
        const unsigned long long e = i + lane < n ? near_entry_load(buf + i + lane) : 0ull;
        const bool keep = i + lane < n && __uint_as_float((unsigned int)e) >= bound;
        const unsigned long long m = __ballot(keep);
        const int pre = __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
        if (keep) __hip_atomic_store(reinterpret_cast<unsigned long long*>(buf + kept + pre), e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        kept += __popcll(m);
    }
    *n_ = kept;
    return bound;
}

// What a lane carries for its two queries (one of each block of 32) through a sweep, and what it does with the values
// of 32 or 64 candidates.
template <int MODE, bool COLOURED>
struct NearLane {
    float h[2], bound[2];
    int qcol[2];
    unsigned int off[2], roomy[2];          // byte offsets into the entries: next free, last with room for 32
    float m[2][16], m1[2], m2[2];
    int m1_at[2];
    NearBoundArgs args;
    int q_at[2];                            // number of the query, and that in the batch
    int lq[2];
    int q_pos[2], reg[2];                   // its position in the copy, and region
    bool valid[2];

    // queries of block `qblk` and the next one of tile `qtile`; `sub`: the buffer of this lane among the p.nsub of a query
    __device__ inline void start(const NearSweep& p, int qtile, int qblk, int l32, int sub, bool live)
    {
        if (MODE == NEAR_EMIT || MODE == NEAR_NEAREST || MODE == NEAR_BLOCK) args = near_args(p.sc, p.steps, p.d, p.e, p.nu);
        const int qt = live ? qtile : p.q_tile0;
        const int n_q = p.n_dev ? *p.n_dev : p.n_q;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            q_at[qb] = qt * TILE + (qblk + qb) * 32 + l32;
            lq[qb] = q_at[qb] - p.q_tile0 * TILE;
            valid[qb] = live && (!p.qpos || q_at[qb] < n_q);
            q_pos[qb] = !p.qpos ? q_at[qb] : valid[qb] ? p.qpos[q_at[qb]] : 0;
            reg[qb] = p.region ? p.region[q_pos[qb] >> 7] : -1;
            const float nh = p.qnegh[q_pos[qb]];
            h[qb] = -nh;
            const bool ok = valid[qb] && fabsf(nh) < INF;
            bound[qb] = NEVER;
            if ((MODE == NEAR_EMIT || MODE == NEAR_NEAREST) && p.reach) {
                const float r = ok ? p.reach[MODE == NEAR_EMIT ? lq[qb] : q_at[qb]] : -1.f, t2 = r * p.sc->scale * p.sc->scale;
                if (r >= 0.f) bound[qb] = t2 < INF ? fmaxf(LOWEST, near_bound_at(t2, h[qb], args)) : LOWEST;
            } else if (MODE == NEAR_EMIT && ok) bound[qb] = p.bound[lq[qb]];
            if (COLOURED) qcol[qb] = p.qcolour[q_pos[qb]];
            if (MODE == NEAR_EMIT) {
                off[qb] = ((unsigned int)lq[qb] * (unsigned int)p.nsub + (unsigned int)sub) * (unsigned int)p.capl * 8u;
                roomy[qb] = off[qb] + (unsigned int)(p.capl - 32) * 8u;
                if (p.append && live) {
                    const int have = p.counts[(size_t)lq[qb] * p.nsub + sub];
                    if (have > p.capl - 32) {                // (given up, or no room for what one step may find)
                        off[qb] = 0u; roomy[qb] = 0xffffffffu; bound[qb] = NEVER;
                    } else off[qb] += (unsigned int)have * 8u;
                }
            }
            m1[qb] = m2[qb] = -INF;
            m1_at[qb] = -1;
            if (MODE == NEAR_MAXIMA) {
#pragma unroll
                for (int r = 0; r < 16; ++r) m[qb][r] = -INF;
            }
        }
    }

    // acc[query block][candidate block]: value r of a lane belongs to candidate 8 (r / 4) + 4 lhalf + r % 4 of its block;
    // pos0: position of the first of the 32 CB candidates, col: their colours (LDS)
    // ok: whether the lane's queries and the candidates' tile are of the side in hand (and of different colours, with one_colour,
    // which all lanes share: the 32 compares and selects per 16 values of a query are as much as a third of all vector instructions)
    // EARLY: words of colours read ahead, of four candidates each.  Eight compares are made before the eight selects that need them (left alone, the compiler puts every
    // compare right before its select, with two idle cycles between, and how much of it passes under multiplies is its choice): connection rounds of 1M x 128 without a
    // row order 313 -> 285 ms, 100 000 x 100 8.4 -> 6.3 ms.  (The more words ahead, the more registers: with all eight 309 ms, and up to 48 columns one
    // workgroup less on a CU, 200 000 x 16 13.8 -> 14.8 ms; with two 13.4.)
    template <int EARLY, int CB>
    __device__ inline __attribute__((always_inline)) void take(const NearSweep& p, v16f (&acc)[2][CB], int pos0, const unsigned char* col, int lhalf,
                                                               bool ok0 = true, bool ok1 = true, bool one_colour = false)
    {
        const bool ok[2] = {ok0, ok1};
        const int lane = threadIdx.x & 63;
        if (COLOURED && !one_colour) {
            v4i cc[4 * CB];                                         // of four candidates each
            auto read = [&](int i) { cc[i] = *reinterpret_cast<const v4i*>(col + ((i >> 2) * 32 + 8 * (i & 3) + 4 * lhalf) * 4); };
#pragma unroll
            for (int i = 0; i < EARLY; ++i) read(i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4 * CB; ++i) {
                unsigned long long same[2][4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb) same[qb][e] = __ballot(cc[i][e] == qcol[qb]);
                if (i + EARLY < 4 * CB) read(i + EARLY);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb) {
                        const int r = 4 * (i & 3) + e;
                        acc[qb][i >> 2][r] = __builtin_amdgcn_inverse_ballot_w64(same[qb][e]) ? -INF : acc[qb][i >> 2][r];
                    }
            }
        }
        if (MODE == NEAR_MAXIMA) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) m[qb][r] = CB == 2 ? max3(m[qb][r], acc[qb][0][r], acc[qb][CB - 1][r]) : fmaxf(m[qb][r], acc[qb][0][r]);
            return;
        }
        if (MODE == NEAR_BLOCK || MODE == NEAR_TOP) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const v16f& v = acc[qb][cb];
                    float mx = max3(v[0], v[1], v[2]);
#pragma unroll
                    for (int r = 3; r < 15; r += 2) mx = max3(mx, v[r], v[r + 1]);
                    mx = fmaxf(mx, v[15]);
                    const bool up = mx > m1[qb] && ok[qb];
                    m1_at[qb] = up ? pos0 + 32 * cb : m1_at[qb];
                    if (MODE == NEAR_TOP) m2[qb] = fmaxf(m2[qb], fminf(m1[qb], mx));
                    m1[qb] = up ? mx : m1[qb];
                }
            return;
        }
        if (MODE == NEAR_ARG) {
            // the number of the value among the lane's 16 CB replaces the five lowest bits of its mantissa (an infinity
            // would become a NaN: copies used here have finite padding)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                float mx = -INF;
#pragma unroll
                for (int i = 0; i < 16 * CB; i += 2) {
                    const float a = __uint_as_float((__float_as_uint(acc[qb][i >> 4][i & 15]) & 0xffffffe0u) | (unsigned int)i);
                    const float b = __uint_as_float((__float_as_uint(acc[qb][i >> 4][(i & 15) + 1]) & 0xffffffe0u) | (unsigned int)(i + 1));
                    mx = max3(mx, a, b);
                }
                const bool up = mx > m1[qb];
                m1_at[qb] = up ? pos0 : m1_at[qb];
                m1[qb] = up ? mx : m1[qb];
            }
            return;
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            // maxima of 5, 5, 3 and 3 values of each block (three at a time in one instruction), and of all
            constexpr int from[5] = {0, 5, 10, 13, 16};
            float g8[4 * CB];
#pragma unroll
            for (int g = 0; g < 4 * CB; ++g) {
                const v16f& v = acc[qb][g >> 2];
                const int r = from[g & 3];
                g8[g] = max3(v[r], v[r + 1], v[r + 2]);
                if ((g & 3) < 2) g8[g] = max3(g8[g], v[r + 3], v[r + 4]);
            }
            float mx = fmaxf(max3(g8[0], g8[1], g8[2]), g8[3]);
            if constexpr (CB == 2) mx = max3(max3(g8[4], g8[5], g8[6]), mx, g8[7]);
            if (!__any(mx >= bound[qb] && ok[qb])) continue;
            if (MODE == NEAR_NEAREST) {
                // A handful per query over all workgroups, but by the hundred among copies of a point: one addition to memory, and one wait for what it
                // returns, for all of a lane's values (300 000 x 10, every point 600 times, the second search of the rows left over: 54.6 ms with one per value, 39.3 so).
                int at = 0;
#pragma unroll
                for (int g = 0; g < 4 * CB; ++g)
                    if (__any(g8[g] >= bound[qb] && ok[qb])) {
#pragma unroll
                        for (int r = from[g & 3]; r < from[(g & 3) + 1]; ++r) at += acc[qb][g >> 2][r] >= bound[qb] ? 1 : 0;
                    }
                if (at > 0 && ok[qb]) at = atomicAdd(p.counts + q_at[qb], at);
#pragma unroll
                for (int g = 0; g < 4 * CB; ++g) {
                    if (__any(g8[g] >= bound[qb] && ok[qb])) {
#pragma unroll
                        for (int r = from[g & 3]; r < from[(g & 3) + 1]; ++r) {
                            const float v = acc[qb][g >> 2][r];
                            if (__any(v >= bound[qb]) && v >= bound[qb] && ok[qb]) {
                                const unsigned int pos = p.mark | (unsigned int)pos0 + (g >> 2) * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
                                if (at < p.capl) p.entries[(size_t)lq[qb] * p.capl + at] = make_uint2(__float_as_uint(v), pos);
                                ++at;
                            }
                        }
                    }
                }
                continue;
            }
#pragma unroll
            for (int g = 0; g < 4 * CB; ++g) {
                if (__any(g8[g] >= bound[qb] && ok[qb])) {
#pragma unroll
                    for (int r = from[g & 3]; r < from[(g & 3) + 1]; ++r) {
                        const float v = acc[qb][g >> 2][r];
                        if (__any(v >= bound[qb]) && v >= bound[qb] && ok[qb]) {
                            const unsigned int pos = p.mark | (unsigned int)pos0 + (g >> 2) * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
                            *reinterpret_cast<uint2*>(reinterpret_cast<unsigned char*>(p.entries) + off[qb]) =
                                make_uint2(__float_as_uint(v), pos);
                            off[qb] += 8u;
                        }
                    }
                }
            }
            // room for the 32 values that come next, or tighten
            unsigned long long full = __ballot(off[qb] > roomy[qb]);
            while (full) {
                const int who = __builtin_ctzll(full);
                full &= full - 1;
                const unsigned int start = (unsigned int)__builtin_amdgcn_readlane((int)roomy[qb], who) - (unsigned int)(p.capl - 32) * 8u;
                int n = (int)(((unsigned int)__builtin_amdgcn_readlane((int)off[qb], who) - start) >> 3);
                const float hw = __uint_as_float((unsigned int)__builtin_amdgcn_readlane((int)__float_as_uint(h[qb]), who));
                const float nb = p.append ? LOWEST : near_refine(reinterpret_cast<uint2*>(reinterpret_cast<unsigned char*>(p.entries) + start), &n, p.kk, hw, args);
                if (lane == who) {
                    off[qb] = start + (unsigned int)n * 8u;
                    bound[qb] = fmaxf(bound[qb], nb);
                    // ties by the hundred: this query is given up here (count capl + 1) and takes nothing more
                    if (n > p.capl - 32) { off[qb] = 0u; roomy[qb] = 0xffffffffu; bound[qb] = NEVER; }
                }
            }
        }
    }

    // one part of the maxima ends
    __device__ inline void flush(const NearSweep& p, int part_at, int lhalf, bool live)
    {
        if (live) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                float* out = p.maxima + ((size_t)part_at * p.nq_batch + lq[qb]) * p.groups + (p.groups >> 1) * lhalf;
                v4f few;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4f v = {m[qb][4 * g], m[qb][4 * g + 1], m[qb][4 * g + 2], m[qb][4 * g + 3]};
                    if (p.groups == GROUPS) *reinterpret_cast<v4f*>(out + 4 * g) = v;
                    few[g] = fmaxf(max3(v[0], v[1], v[2]), v[3]);
                }
                if (p.groups != GROUPS) *reinterpret_cast<v4f*>(out) = few;
            }
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int r = 0; r < 16; ++r) m[qb][r] = -INF;
    }

    __device__ inline void finish(const NearSweep& p, int sub, int lhalf, bool live)
    {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            if (MODE == NEAR_TOP && live)
                p.top[(size_t)lq[qb] * p.nsub + sub] = make_uint4(__float_as_uint(m1[qb]), (unsigned int)(m1_at[qb] + 4 * lhalf), __float_as_uint(m2[qb]), 0u);
            if (MODE == NEAR_BLOCK) {
                const float v = __shfl_xor(m1[qb], 32);
                const int at = __shfl_xor(m1_at[qb], 32);
                const bool other = v > m1[qb];
                const float m = other ? v : m1[qb];
                const int pos = other ? at + 4 : m1_at[qb];                  // (lhalf 0 writes)
                // (two copies may hold the query, and their product values do not compare: distances do)
                if (valid[qb] && fabsf(h[qb]) < INF && lhalf == 0 && m > -INF && m < INF) {
                    const float low = near_lower_from(m, h[qb], args) / p.sc->scale / p.sc->scale;
                    atomicMin(p.best_at + q_at[qb], ((unsigned long long)__float_as_uint(low) << 32) | (unsigned int)pos);
                }
            }
            if (MODE == NEAR_ARG && live && m1_at[qb] >= 0 && fabsf(m1[qb]) < 1e37f) {
                const int i = (int)(__float_as_uint(m1[qb]) & 31u), r = i & 15;
                const int pos = m1_at[qb] + (i >> 4) * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
                atomicMax(p.best_at + q_at[qb], ((unsigned long long)ordered_bits(m1[qb]) << 32) | (unsigned int)pos);
            }
            if (MODE == NEAR_EMIT && live)
                p.counts[(size_t)lq[qb] * p.nsub + sub] =
                    roomy[qb] == 0xffffffffu ? p.capl + 1 : (int)((off[qb] + (unsigned int)(p.capl - 32) * 8u - roomy[qb]) >> 3);
        }
    }
};

// The share of a workgroup: which panel, which segment of how many, and where the query tiles end.
struct NearShare { int panel, seg, nseg, q_tile1; bool any; };
__device__ inline NearShare near_share(const NearSweep& p, int item, int panel_tiles, int units)
{
    NearShare r{0, 0, p.nseg, p.q_tile1, true};
    if (p.n_dev) {
        int n = *p.n_dev - p.q_tile0 * TILE;
        const int most = (p.q_tile1 - p.q_tile0) * TILE;
        n = n < 0 ? 0 : (n > most ? most : n);
        r.q_tile1 = p.q_tile0 + (n + TILE - 1) / TILE;
        const int panels = (r.q_tile1 - p.q_tile0 + panel_tiles - 1) / panel_tiles;
        int k = panels > 0 ? p.slots / panels : 1;
        k = k > p.most_seg ? p.most_seg : k;
        k = k > units ? units : k;
        r.nseg = k < 1 ? 1 : k;
        r.any = item < panels * r.nseg;
    }
    r.panel = item / r.nseg;
    r.seg = item - r.panel * r.nseg;
    return r;
}

// the j-th candidate tile
template <int MODE>
__device__ inline int near_tile_at(const NearSweep& p, int j)
{
    if (MODE == NEAR_MAXIMA && p.spread) j = near_spread_at(j, p.spread, p.used);
    return p.skip ? j + j / (p.stride - 1) + 1 : j * p.stride;
}

// Tiles per item of a list.  The lists of a round are a few thousand tiles in all, and longer items leave CUs without one; shorter ones load a
// panel's queries more often.  Clusterings with 64, 32, 16 and 8, in ms: 100 000 x 64 4.88, 4.58, 4.55 and 4.50; 60 000 x 100 4.05, 3.73, 3.65 and 3.53;
// 300 000 x 96 19.07, 18.02, 17.96 and 18.06; 800 000 x 128 67.7, 67.3, 68.4 and 70.5.  (Left-over rows of 100 000 x 64, 376 and 219 us.)
constexpr int ITEM_TILES = 32;

// Up to 128 columns: a wavefront keeps the fragments of its 64 queries (two blocks of 32) in registers and passes over
// the candidate tiles, which the workgroup's wavefronts bring into LDS together (double buffered, one barrier per
// tile).  A lane's 16 values of a 32 x 32 block belong to one query, so bounds and counts are registers.
// Fragment order in memory makes every load and every LDS read consecutive over the lanes.
// Where a value costs a compare of colours or an index, and in connection rounds over lists, 32 candidates at a time: 100 to 130 registers instead of 130 to
// 220, so that two workgroups share a CU (up to 96 columns).  Nearest rows of another colour, 10 000 in 100 000 x 64, 267 -> 237 us with as many segments as that takes, 20 000 in
// 60 000 x 10 217 -> 199; first edges over lists 1.43 -> 1.29 ms of 100k x 64, 8.9 -> 8.7 of 1M x 128; nearest pivots 3.7 -> 3.2.  (Emission, what is left over and
// maxima are no faster so: 168 and 176, 377 and 426 us of 100k x 64.)
// (Emission of up to 32 columns is held to 128 registers, with which two workgroups of eight wavefronts share a CU: with one more, 300 000 x 10
// rows without clusters in the row order took 9.9 ms of it instead of 7.1.  Likewise maxima of 80 columns to 168 registers, three workgroups of four.)
template <int KS, int MODE, bool COLOURED, bool LISTED>
__global__ void __launch_bounds__(512, KS <= 2 && MODE == NEAR_EMIT ? 4 : KS == 5 && MODE == NEAR_MAXIMA ? 3 : 2) near_sweep_kernel(NearSweep p)
{
    extern __shared__ __align__(16) unsigned char near_smem[];
    constexpr int CB = (MODE == NEAR_TOP && COLOURED && KS <= 6) || MODE == NEAR_ARG || MODE == NEAR_BLOCK ? 1 : 2;       // blocks of 32 candidates at once
    constexpr int UNROLL = MODE == NEAR_BLOCK && LISTED ? 1 : 4;
    constexpr int BUF = KS * FRAG_STEP + 1024;           // fragments, minus half norms, colours
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6;
    // Lists differ in length by orders of magnitude, so searches without buffers of their own per share hand them out in
    // equal items; the grid passes over the items.
    constexpr bool ITEMS = LISTED && (MODE == NEAR_BLOCK || MODE == NEAR_NEAREST);
    const int n_items = ITEMS ? p.items[p.panels] : 0;
    for (int item = blockIdx.x; !ITEMS || item < n_items; item += gridDim.x) {
    NearShare share{0, 0, 1, p.q_tile1, true};
    int item_from = 0;
    if (ITEMS) {
        int lo = 0, hi = p.panels;                       // items[lo] <= item < items[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (p.items[mid] <= item) lo = mid; else hi = mid;
        }
        share.panel = lo;
        item_from = (item - p.items[lo]) * ITEM_TILES;
    } else share = near_share(p, item, waves >> 1, p.used);
    if (!share.any) return;
    const unsigned short* __restrict__ list = LISTED ? p.list + (size_t)share.panel * p.list_stride + item_from : nullptr;
    const int list_step = LISTED && p.list_step ? p.list_step[share.panel] : 1;
    if (list_step == 0) return;
    int used = p.used;
    if (LISTED) {
        used = (p.list_len[share.panel] - item_from + list_step - 1) / list_step;
        if (ITEMS && used > ITEM_TILES) used = ITEM_TILES;
    }
    const int seg = share.seg, nseg = share.nseg;
    const int qtile = p.q_tile0 + share.panel * (waves >> 1) + (wave >> 1);
    const bool live = qtile < share.q_tile1;             // (whole wavefronts)
    const int qblk = (wave & 1) * 2;

    NearLane<MODE, COLOURED> mine;
    mine.start(p, qtile, qblk, l32, 2 * seg + lhalf, live);
    v8h qf[2][KS];
    {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            const int at = mine.q_pos[qb];                  // consecutive, or wherever the queries are
            const unsigned char* src = p.qfrag + (size_t)(at >> 7) * (KS * FRAG_STEP) + ((at >> 5) & 3) * 1024 + (lhalf * 32 + (at & 31)) * 16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[qb][ks] = *reinterpret_cast<const v8h*>(src + ks * FRAG_STEP);
        }
    }
    // (a second search of the rows left over: whose lists overflowed, see pairs_again)
    if (MODE == NEAR_NEAREST && !LISTED && !__syncthreads_or(!(mine.bound[0] != mine.bound[0] && mine.bound[1] != mine.bound[1]))) return;
    // first bounds come from the one copy that holds all of a query's region
    const int first_reg = LISTED && MODE == NEAR_MAXIMA && p.side ? __builtin_amdgcn_readfirstlane(mine.reg[0]) : 0;
    const bool mine_here = !(LISTED && MODE == NEAR_MAXIMA && p.side) || (p.side == 1) == (first_reg >= 0);

    const int ntiles = seg < used ? (used - seg + nseg - 1) / nseg : 0;
    // (called for i = 0, 1, ...: a lane holds one of 64 entries of the list, and that tile's region and colour: a load of one word
    // per tile makes every tile wait for it, behind the stage for the next tile as well.  Clustering 100k x 64, connection rounds: 1.69 ms of
    // sweeps for first edges and 0.49 for nearest rows, 1.59 and 0.42 so; 1M x 128: 9.9 and 1.6 ms, 9.3 and 1.4, emission 17.9 and 17.4)
    int listed = 0, listed_reg = -1, listed_colour = -1;
    auto tile_at = [&](int i) -> int {
        if (!LISTED) return near_tile_at<MODE>(p, seg + i * nseg);
        if ((i & 63) == 0) {
            const int j = seg + (i + lane) * nseg;
            listed = j < used ? (int)list[j * list_step] : 0;
            if (p.side) listed_reg = p.region[listed];
            if (COLOURED) listed_colour = p.tile_colour[listed];
        }
        return __builtin_amdgcn_readlane(listed, i & 63);
    };
    auto stage = [&](int i, int tile) {
        const size_t t = tile;
        unsigned char* dst = near_smem + (i & 1) * BUF;
        const unsigned char* src = p.cfrag + t * (KS * FRAG_STEP);
        for (int j = wave; j < KS * 4; j += waves) near_lds_load(src, j * 1024, dst + j * 1024, true);
        for (int j = wave; j < (COLOURED ? 4 : 2); j += waves) {
            const void* rows = j < 2 ? (const void*)(p.cnegh + t * TILE) : (const void*)(p.ccolour + t * TILE);
            near_lds_load(rows, (j & 1) * 256, dst + KS * FRAG_STEP + j * 256, false);
        }
    };
    int next = ntiles > 0 ? tile_at(0) : 0;
    if (ntiles > 0) stage(0, next);
    int next_colour = LISTED && COLOURED ? __builtin_amdgcn_readlane(listed_colour, 0) : -1;
    int next_reg = LISTED ? __builtin_amdgcn_readlane(listed_reg, 0) : -1;
    const int per_part = MODE == NEAR_MAXIMA ? (ntiles + p.parts - 1) / p.parts : 0;
    int part = 0, part_end = per_part;
    for (int i = 0; i < ntiles; ++i) {
        near_lds_ready();
        const int pos0 = next * TILE, colour_here = next_colour, tile_reg = next_reg;
        if (i + 1 < ntiles) {
            next = tile_at(i + 1);
            if (LISTED && COLOURED) next_colour = __builtin_amdgcn_readlane(listed_colour, (i + 1) & 63);
            if (LISTED) next_reg = __builtin_amdgcn_readlane(listed_reg, (i + 1) & 63);
            stage(i + 1, next);
        }
        const unsigned char* tb = near_smem + (i & 1) * BUF;
        bool ok0 = true, ok1 = true;
        if (LISTED && p.side) {
            ok0 = (tile_reg >= 0 && tile_reg == mine.reg[0]) == (p.side == 1);
            ok1 = (tile_reg >= 0 && tile_reg == mine.reg[1]) == (p.side == 1);
        }
        const int tile_col = LISTED && COLOURED ? colour_here : -1;
        if (LISTED && COLOURED) {
            ok0 = ok0 && tile_col != mine.qcol[0];           // (colours are not negative)
            ok1 = ok1 && tile_col != mine.qcol[1];
        }
        if (!LISTED || (mine_here && __any(ok0 || ok1)))
#pragma unroll UNROLL
        for (int part = 0; part < 4 / CB; ++part) {
            v16f acc[2][CB];
            v8h cf[2][CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) cf[0][cb] = *reinterpret_cast<const v8h*>(tb + (part * CB + cb) * 1024 + lane * 16);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                v16f hv;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4f t4 = *reinterpret_cast<const v4f*>(tb + KS * FRAG_STEP + ((part * CB + cb) * 32 + 8 * g + 4 * lhalf) * 4);
                    hv[4 * g] = t4[0]; hv[4 * g + 1] = t4[1]; hv[4 * g + 2] = t4[2]; hv[4 * g + 3] = t4[3];
                }
                acc[0][cb] = hv; acc[1][cb] = hv;
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                // the next step's fragments are on their way while this step is multiplied (the fence keeps the reads
                // from sinking to their use, which leaves the whole LDS latency between two groups of multiplies)
                if (ks + 1 < KS) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
                        cf[(ks + 1) & 1][cb] = *reinterpret_cast<const v8h*>(tb + (ks + 1) * FRAG_STEP + (part * CB + cb) * 1024 + lane * 16);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb)
                        acc[qb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cf[ks & 1][cb], qf[qb][ks], acc[qb][cb], 0, 0, 0);
            }
            mine.template take<KS <= 3 ? 2 : 4>(p, acc, pos0 + part * 32 * CB, tb + KS * FRAG_STEP + 512 + part * 128 * CB, lhalf, ok0, ok1, tile_col >= 0);
        }
        if (MODE == NEAR_MAXIMA && (i + 1 == part_end || i + 1 == ntiles)) {
            mine.flush(p, seg * p.parts + part, lhalf, live && mine_here);
            ++part;
            part_end += per_part;
        }
    }
    if (MODE == NEAR_MAXIMA)
        for (; part < p.parts; ++part) mine.flush(p, seg * p.parts + part, lhalf, live && mine_here);
    mine.finish(p, 2 * seg + lhalf, lhalf, live);
    if (!ITEMS) break;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();                        // the buffers in LDS are free again
    asm volatile("" ::: "memory");
    }
}

// Beyond 128 columns: 256 queries x 256 candidates per workgroup, both streamed through LDS 32 columns at a time
// (four buffers, the pipeline of pairs_wide_kernel), a wavefront holding 64 x 128 of the products.  Consecutive items of an XCD are the segments of
// neighbouring panels: its 32 workgroups share 8 panels of queries, which stay in its L2, and read the same candidates.
// Bound by the products and what is not done under them (first fragments, the test of the values).  k-NN 3900 x 160 104 -> 91 us, 60 000 x 256 2.42 ->
// 2.14 ms, 1-NN 5000 in 200 000 x 200 602 -> 492 us, 1000 in 100 000 x 256 171 -> 156 us against chunks of 64 columns in two buffers, waited
// for all at once; the sample of 250k x 784 7.6 -> 6.1 ms.
constexpr int WIDE_ROWS = 2048;                                         // half norms and colours of 256 candidates
constexpr int WIDE_LDS = CHUNKS * CHUNK + 2 * WIDE_ROWS;

template <int MODE, bool COLOURED>
__global__ void __launch_bounds__(512, 2) near_wide_kernel(NearSweep p)
{
    extern __shared__ __align__(16) unsigned char near_smem[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qg = wave >> 1, cg = wave & 1;                            // 64 queries, 128 candidates of the 256 x 256
    const int npairs = (p.used + 1) / 2;                                // pairs of listed tiles
    int item = blockIdx.x;
    {
        NearShare all = near_share(p, 0, 2, npairs);
        if (!all.any) return;
        const int items = (all.q_tile1 - p.q_tile0 + 1) / 2 * all.nseg;
        const int per = items >> 3;                                     // workgroups b, b + 8, ... share an XCD
        if (item >= items) return;
        if (item < per * 8) item = (item & 7) * per + (item >> 3);
    }
    const NearShare share = near_share(p, item, 2, npairs);
    const int seg = share.seg, nseg = share.nseg, q_tile1 = share.q_tile1;
    const int qtile0 = p.q_tile0 + share.panel * 2;
    const int qtile = qtile0 + (qg >> 1);
    const bool live = qtile < q_tile1;
    const int qblk = (qg & 1) * 2;
    const int sub = (2 * seg + cg) * 2 + lhalf;

    NearLane<MODE, COLOURED> mine;
    mine.start(p, qtile, qblk, l32, sub, live);

    if (MODE == NEAR_NEAREST && !__syncthreads_or(!(mine.bound[0] != mine.bound[0] && mine.bound[1] != mine.bound[1]))) return;      // (as in near_sweep_kernel)
    const int filled = (p.d + 15) / 16, nchunks = (filled + CHUNK_STEPS - 1) / CHUNK_STEPS;
    const bool odd = (filled & 1) != 0;                                 // the last chunk has one step
    const int nmine = seg < npairs ? (npairs - seg + nseg - 1) / nseg : 0;
    auto listed = [&](int j) -> int { return near_tile_at<MODE>(p, j); };
    const int total = nmine * nchunks;
    // a wavefront brings in one step of one tile of one side, four pieces of 1 KiB: of the queries, where they are
    const int my_tile = (wave >> 1) & 1, my_st = wave & 1;
    const unsigned char* q_src[4] = {p.qfrag, p.qfrag, p.qfrag, p.qfrag};
    if (wave < 4) {
        const int n_q = p.n_dev ? *p.n_dev : p.n_q;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            const int t = qtile0 + my_tile < q_tile1 ? qtile0 + my_tile : qtile0;
            const int i = t * TILE + blk * 32 + l32;
            const int at_q = !p.qpos ? i : i < n_q ? p.qpos[i] : 0;
            q_src[blk] = p.qfrag + ((size_t)(at_q >> 7) * p.steps + my_st) * FRAG_STEP + ((at_q >> 5) & 3) * 1024 + (lhalf * 32 + (at_q & 31)) * 16;
        }
    }
    // the next chunk's loads, and with a pair's first chunk the norms and colours
    int staged = 0, stage_i = 0, stage_chunk = 0, stage_t0 = 0, stage_t1 = 0;
    auto stage_tiles = [&]() {
        const int j0 = 2 * (seg + stage_i * nseg);
        stage_t0 = listed(j0);
        stage_t1 = listed(j0 + 1 < p.used ? j0 + 1 : j0);
    };
    if (nmine > 0) stage_tiles();
    auto stage = [&]() {
        unsigned char* dst = near_smem + (staged & (CHUNKS - 1)) * CHUNK + wave * FRAG_STEP;
        if (stage_chunk == 0 && wave < (COLOURED ? 8 : 4)) {
            const size_t t = my_tile ? stage_t1 : stage_t0;
            const void* rows = wave < 4 ? (const void*)(p.cnegh + t * TILE) : (const void*)(p.ccolour + t * TILE);
            near_lds_load(rows, my_st * 256, near_smem + CHUNKS * CHUNK + (stage_i & 1) * WIDE_ROWS + wave * 256, false);
        }
        if (wave < 4) {
#pragma unroll
            for (int blk = 0; blk < 4; ++blk) near_lds_gather(q_src[blk] + (size_t)stage_chunk * (CHUNK_STEPS * FRAG_STEP), dst + blk * 1024);
        } else {
            const unsigned char* src = p.cfrag + ((size_t)(my_tile ? stage_t1 : stage_t0) * p.steps + stage_chunk * CHUNK_STEPS + my_st) * FRAG_STEP;
#pragma unroll
            for (int blk = 0; blk < 4; ++blk) near_lds_load(src, blk * 1024, dst + blk * 1024, true);
        }
        ++staged;
        if (++stage_chunk == nchunks) {
            stage_chunk = 0;
            if (++stage_i < nmine) stage_tiles();
        }
    };
    const int per_part = MODE == NEAR_MAXIMA ? (nmine + p.parts - 1) / p.parts : 0;
    int part = 0, part_end = per_part;
    v16f acc[2][2][2];                                                  // [pair of candidate blocks][query block][candidate block]
    v8h qf[2][2], cf[2][4];                                             // [step of the chunk]
    auto read = [&](int at, int st) {
        const unsigned char* qs = near_smem + (at & (CHUNKS - 1)) * CHUNK + (qg >> 1) * CHUNK_TILE + st * FRAG_STEP + qblk * 1024 + lane * 16;
        const unsigned char* cs = near_smem + (at & (CHUNKS - 1)) * CHUNK + CHUNK_SIDE + cg * CHUNK_TILE + st * FRAG_STEP + lane * 16;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) qf[st][qb] = *reinterpret_cast<const v8h*>(qs + qb * 1024);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) cf[st][cb] = *reinterpret_cast<const v8h*>(cs + cb * 1024);
        __builtin_amdgcn_sched_barrier(0);                              // (ahead of the multiplies that follow)
    };
    auto multiply = [&](int st, int from, int to) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
                if (cb >= from && cb < to)
                    acc[cb >> 1][qb][cb & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cf[st][cb], qf[st][qb], acc[cb >> 1][qb][cb & 1], 0, 0, 0);
    };
    for (int i = 0; i < CHUNKS - 1 && i < total; ++i) stage();
    near_lds_ready();
    int at = 0;
    for (int i = 0; i < nmine; ++i) {
        const unsigned char* nb = near_smem + CHUNKS * CHUNK + (i & 1) * WIDE_ROWS;
        const bool half_pair = 2 * (seg + i * nseg) + cg >= p.used;   // the second tile of the last pair may be missing
        // (the chunk, the norms and the colours have been there since the last barrier)
        read(at, 0);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            v16f hv;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4f t4 = *reinterpret_cast<const v4f*>(nb + cg * 512 + (cb * 32 + 8 * g + 4 * lhalf) * 4);
                hv[4 * g] = t4[0]; hv[4 * g + 1] = t4[1]; hv[4 * g + 2] = t4[2]; hv[4 * g + 3] = t4[3];
            }
            acc[cb >> 1][0][cb & 1] = hv; acc[cb >> 1][1][cb & 1] = hv;
        }
#pragma unroll 1
        for (int chunk = 1; chunk < nchunks; ++chunk, ++at) {
            near_chunk_ready(at + 2 < total);
            read(at, 1);
            multiply(0, 0, 2);
            if (staged < total) stage();
            multiply(0, 2, 4);
            __builtin_amdgcn_sched_barrier(0);
            read(at + 1, 0);
            multiply(1, 0, 4);
        }
        near_chunk_ready(at + 2 < total);
        read(at, 1);
        multiply(0, 0, 4);
        if (!odd) multiply(1, 0, 4);
        if (staged < total) stage();
        ++at;
        const int j = 2 * (seg + i * nseg) + cg;
        const int pos0 = listed(j < p.used ? j : 0) * TILE;
        if (!half_pair) {
            mine.template take<4>(p, acc[0], pos0, nb + 1024 + cg * 512, lhalf);
            mine.template take<4>(p, acc[1], pos0 + 64, nb + 1024 + cg * 512 + 256, lhalf);
        }
        if (MODE == NEAR_MAXIMA && (i + 1 == part_end || i + 1 == nmine)) {
            mine.flush(p, (2 * seg + cg) * p.parts + part, lhalf, live);
            ++part;
            part_end += per_part;
        }
    }
    if (MODE == NEAR_MAXIMA)
        for (; part < p.parts; ++part) mine.flush(p, (2 * seg + cg) * p.parts + part, lhalf, live);
    mine.finish(p, sub, lhalf, live);
}

// One wavefront per query: (nearly) the kk-th largest of its group maxima, and the bound that follows.
// reach (optional): an upper end of the squared distance of the kk-th nearest row.  step (optional): a second set of maxima,
// made where the step of the query's panel is not 0; the better of the two bounds stays (one candidate may be in both sets).
template <bool LIMIT>
__global__ void __launch_bounds__(256) near_bounds_kernel(const float* __restrict__ maxima, int parts, int log_groups, int nq_batch, int q0, int kk,
                                                          const float* __restrict__ qnegh, const NearScale* __restrict__ sc, float e,
                                                          float nu, int steps, int d, float* __restrict__ bound, float* __restrict__ reach,
                                                          const int32_t* __restrict__ step, int panel_queries,
                                                          const int32_t* __restrict__ region, const float* __restrict__ negh_local,
                                                          const NearScale* __restrict__ sc_local, int32_t* __restrict__ limit_counts, int32_t* __restrict__ limit_last,
                                                          int32_t* __restrict__ limit_lost)
{
    const int lane = threadIdx.x & 63;
    const int lq = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (lq >= nq_batch) return;
    if (step && (step[lq / panel_queries] == 0 || region[(q0 + lq) >> 7] < 0)) return;
    const int n = parts << log_groups;               // at most 1024
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int i = j * 64 + lane;
        v[j] = i < n ? maxima[(((size_t)(i >> log_groups) * nq_batch + lq) << log_groups) + (i & ((1 << log_groups) - 1))] : -INF;
    }
    float lo = INF, hi = -INF;
    int have = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (j * 64 < n) {
            const bool fine = fabsf(v[j]) < INF;
            have += __popcll(__ballot(fine));
            lo = fine ? fminf(lo, v[j]) : lo;
            hi = fine ? fmaxf(hi, v[j]) : hi;
            v[j] = fine ? v[j] : -INF;
        }
    lo = wave_min(lo); hi = wave_max(hi);
    if (have >= kk)
        for (int it = 0; it < (LIMIT ? BISECT_FAR : BISECT); ++it) {
            const float mid = 0.5f * lo + 0.5f * hi;
            int reach = 0;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (j * 64 < n) reach += __popcll(__ballot(v[j] >= mid));
            if (reach >= kk) lo = mid; else hi = mid;
            if (LIMIT && reach == kk) break;
        }
    if (lane == 0) {
        if (region && region[(q0 + lq) >> 7] >= 0) { qnegh = negh_local; sc = sc_local; }
        const float nh = qnegh[q0 + lq];
        const NearBoundArgs a = near_args(sc, steps, d, e, nu);
        const float made = have < kk ? LOWEST : fmaxf(LOWEST, near_bound_from(lo, -nh, a));
        if (LIMIT) {                    // of a row for pairs_emit; none where there is no row or it goes to the list kernels
            limit_counts[lq] = limit_last[lq] = 0;
            if (lq == 0) *limit_lost = 0;
            bound[lq] = !(fabsf(nh) < INF) ? NEVER : made == LOWEST ? LOWEST : made + nh;
            return;
        }
        bound[lq] = step ? fmaxf(bound[lq], made) : made;
        if (reach) {
            const float t = have < kk ? INF : near_distance_from(lo, -nh, a) / sc->scale;          // (a power of two)
            // (no row, or none that is finite: reaches nothing; values beyond float16: left to the list kernels)
            const float r = fabsf(nh) < INF ? (t * t * (1.f + a.gamma) + (float)d * 2.350988701644575e-38f) * (1.f + 1e-6f) : -1.f;
            reach[lq] = step ? fminf(reach[lq], r) : r;
        }
    }
}

// ---------------------------------------------------------------------------------------------- selection
constexpr unsigned int MARK = 0x80000000u;
struct NearSelect {
    const uint2* entries; const int32_t* counts; int nsub, capl, nq_batch, q0, by_position;
    int list0;                       // by position: the position of the first count
    const float* qnegh; const NearScale* sc; float e, nu; int steps;
    const float* Xq; const float* Xc; const int32_t* q_rows;
    int d, k, kk, nq, nq_rows, nc, q_tiles, c_tiles, exclude_self;
    int32_t* out_idx; float* out_dist; int32_t* evaluated;
    int32_t* todo; int32_t* todo_mark;
    int merge;                       // the output rows already hold the list of earlier candidates
    float* next_bound;               // optional: the bound the list implies, for the candidates still to come
    const int32_t* n_dev;            // optional: the first *n_dev queries only
    const int32_t* slot;             // optional: where the answers of query i go
    int q_in_order, c_in_order;
    const int32_t* c_ids; int n_ids; // optional: candidates are positions of an order, c_ids[position] their row (-1: none)
    const int32_t* ids;              // optional: so are the queries
    const int32_t* qpos;             // optional: query i is this position of the copies
    int pair_lists;                  // the entries hold u (pairs_kernels.h) instead of product values
    int skip_gone;                   // rows of panels that are known to go to the list kernels are left out
    // optional, of an order with two copies (see NearSweep): entries without MARK come from the local one
    const int32_t* region; const float* negh_local; const NearScale* sc_local;
};

// How rows are read: 2 by aligned quads, 1 by quads at any word, 0 by words.  Quads at any word cost a second branch for a row's end, and pay from 64
// columns on: selection of 20 000 rows, k = 16, of 50 columns 48 us by words and 50, of 65 52 and 48, of 101 64 and 50, of 401 304 and 167.
static int near_vec(bool aligned, int d) { return aligned ? 2 : d >= 64 ? 1 : 0; }
template <int VEC>
__device__ inline v4f near_quad(const float* __restrict__ row, int t, int d)
{
    v4f v = {0.f, 0.f, 0.f, 0.f};
    if (VEC == 2) {
        if (t < d) v = *reinterpret_cast<const v4f*>(row + t);
    } else if (VEC == 1 && t + 4 <= d) {
        v = *reinterpret_cast<const v4f_word*>(row + t);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (t + e < d) v[e] = row[t + e];
    }
    return v;
}
__device__ inline float near_quad_sqdist(v4f a, v4f b, float s)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) { const float x = a[e] - b[e]; s = __builtin_fmaf(x, x, s); }
    return s;
}

// The exact distance of row xa to row xb by eight lanes, in the order of group8_sqdist (sweep_kernels.hip): slabs of 64
// features, lane g of eight adds features 4g.. and 4(g + 8).. of every slab into two sums, xor butterfly 1, 2, 4.  q: what
// lane g adds of the first 128 features of xa.
template <int VEC>
__device__ inline float near_exact(const v4f (&q)[4], const v4f (&b)[4], const float* __restrict__ xa, const float* __restrict__ xb, int d, int g)
{
    float s0 = 0.f, s1 = 0.f;
    s0 = near_quad_sqdist(q[0], b[0], s0); s0 = near_quad_sqdist(q[2], b[2], s0);
    s1 = near_quad_sqdist(q[1], b[1], s1); s1 = near_quad_sqdist(q[3], b[3], s1);
    for (int base = 128; base < d; base += 128) {
        const int t0 = base + 4 * g;
        const v4f a00 = near_quad<VEC>(xa, t0, d), b00 = near_quad<VEC>(xb, t0, d);
        const v4f a10 = near_quad<VEC>(xa, t0 + 32, d), b10 = near_quad<VEC>(xb, t0 + 32, d);
        const v4f a01 = near_quad<VEC>(xa, t0 + 64, d), b01 = near_quad<VEC>(xb, t0 + 64, d);
        const v4f a11 = near_quad<VEC>(xa, t0 + 96, d), b11 = near_quad<VEC>(xb, t0 + 96, d);
        s0 = near_quad_sqdist(a00, b00, s0); s0 = near_quad_sqdist(a01, b01, s0);
        s1 = near_quad_sqdist(a10, b10, s1); s1 = near_quad_sqdist(a11, b11, s1);
    }
    return lanes_add8(s0) + lanes_add8(s1);
}
template <int VEC>
__device__ inline void near_first_quads(v4f (&q)[4], const float* __restrict__ xa, int d, int g)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = near_quad<VEC>(xa, 4 * g + 32 * j, d);
}
template <int VEC>
__device__ inline float near_exact(const v4f (&q)[4], const float* __restrict__ xa, const float* __restrict__ xb, int d, int g)
{
    v4f b[4];
    near_first_quads<VEC>(b, xb, d, g);
    return near_exact<VEC>(q, b, xa, xb, d, g);
}

// One wavefront per query.  Of 20 011 x 50, k = 10, 50 us: the entries' way into LDS 14, the bound from them 15 (two to four values a lane, looked for in LDS at every step of
// the bisection), the exact distances 15 (eight pairs at a time, each row waited for), ranks 4.  With the values in registers where they are few, and the rows of 16 pairs
// on their way at once, 43; 50 000 x 128, k = 32 179 -> 152, connection rounds and lists of 1M x 128 4.4 -> 3.5 ms.
template <int VEC>
__global__ void __launch_bounds__(256) near_select_kernel(NearSelect p)
{
    __shared__ unsigned long long keys_[4][MAX_ENTRIES + 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lq = blockIdx.x * 4 + w;
    if (lq >= p.nq_batch) return;
    unsigned long long* keys = keys_[w];
    const int qpos = p.q0 + lq;
    const long long qn = near_row(qpos, p.q_tiles, p.q_in_order);
    if (qn >= p.nq || (p.n_dev && qn >= *p.n_dev)) return;      // padding of the last tiles
    const long long row = p.ids ? (long long)p.ids[qn] : p.q_rows ? (long long)p.q_rows[qn] : qn;
    if (p.ids && row < 0) return;                               // a position without a row
    const long long qi = p.ids ? row : p.slot ? (long long)p.slot[qn] : qn;
    const int qcopy = p.qpos ? p.qpos[qn] : qpos;
    const int gone = p.skip_gone ? p.todo_mark[qi >> 7] : 0;    // (on its way with the half norm)
    const float nh = p.qnegh[qcopy];
    if (row < 0 || row >= p.nq_rows || nh == -INF) {            // not a row, or not a finite one
        for (int j = lane; j < p.k; j += 64) { p.out_idx[qi * p.k + j] = -1; p.out_dist[qi * p.k + j] = INF; }
        if (p.evaluated && lane == 0) p.evaluated[qi] = 0;
        return;
    }
    // (40 000 x 24 with norms over orders of magnitude, k = 20, whole search 5.78 -> 5.30 ms; 20 011 x 50, 10, 2.94 -> 2.61: distances for lists that are made again)
    if (gone == PANEL_GONE) {
        if (p.evaluated && lane == 0) p.evaluated[qi] = 0;
        return;
    }
    // gather the entries of all buffers: counts side by side over the lanes, running totals, then every lane looks up
    // the buffer its entry lies in
    int n = 0;
    const float base = p.pair_lists ? nh : 0.f;
    bool lost = nh == INF || (p.region && p.negh_local[qcopy] == INF);
    {
        const int mine = lane < p.nsub ? p.counts[p.by_position ? (size_t)(qpos - p.list0) : (size_t)lq * p.nsub + lane] : 0;
        lost = lost || __any(mine > p.capl);
        int upto = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(upto, o);
            if (lane >= o) upto += x;
        }
        n = lost ? 0 : __builtin_amdgcn_readlane(upto, 63);
        const unsigned long long* e = reinterpret_cast<const unsigned long long*>(p.entries) + (size_t)lq * p.nsub * p.capl;
        for (int i = 0; i < n; i += 64) {
            const int at = i + lane;
            int sub = 0;                                        // number of buffers that end at or before `at`
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const int end = __shfl(upto, sub + o - 1);
                if (sub + o <= p.nsub && end <= at) sub += o;
            }
            const int begin = __shfl(upto - mine, sub & 63);
            if (at < n) {
                const unsigned long long x = e[(size_t)sub * p.capl + (at - begin)];
                keys[at] = (x & 0xffffffff00000000ull) | __float_as_uint(__uint_as_float((unsigned int)x) - base);
            }
        }
    }
    if (lost) {
        if (lane == 0) {
            const int panel = (int)((p.c_ids ? qcopy : qi) >> 7);
            if (atomicExch(p.todo_mark + panel, 1) == 0) p.todo[2 + atomicAdd(p.todo, 1)] = panel;
            if (p.next_bound) p.next_bound[lq] = NEVER;
            if (p.evaluated) p.evaluated[qi] = 0;
        }
        return;
    }
    __builtin_amdgcn_wave_barrier();
    // a tighter bound from (nearly) the kk-th largest product value emitted
    float bound = LOWEST, bound_local = LOWEST;
    const NearBoundArgs args = near_args(p.sc, p.steps, p.d, p.e, p.nu);
    if (p.region) {
        // product values of the two copies do not compare: the bound comes from those of one
        const unsigned int first = p.region[qcopy >> 7] >= 0 ? 0u : MARK;
        const float nl = p.negh_local[qcopy];
        const NearBoundArgs al = near_args(p.sc_local, p.steps, p.d, p.e, p.nu);
        if (n > p.kk + 4) {
            auto value = [&](int i) {
                const unsigned long long e = i + lane < n ? keys[i + lane] : 0ull;
                return i + lane < n && ((unsigned int)(e >> 32) & MARK) == first ? __uint_as_float((unsigned int)e) : -INF;
            };
            const float kth = n <= 128 ? near_kth_of<2>(n, p.kk, value) : n <= 256 ? near_kth_of<4>(n, p.kk, value) : near_kth(n, p.kk, value);
            if (kth != LOWEST) {
                const NearScale* sc = first ? p.sc : p.sc_local;
                const float t = near_distance_from(kth, first ? -nh : -nl, first ? args : al) / sc->scale;
                const float t2 = (t * t * (1.f + args.gamma) + (float)p.d * 2.350988701644575e-38f) * (1.f + 1e-6f);
                if (t2 < INF) {
                    bound = fmaxf(LOWEST, near_bound_at(t2 * p.sc->scale * p.sc->scale, -nh, args));
                    if (fabsf(nl) < INF) bound_local = fmaxf(LOWEST, near_bound_at(t2 * p.sc_local->scale * p.sc_local->scale, -nl, al));
                }
            }
        }
    } else if (n > p.kk + 4) {
        auto value = [&](int i) { return i + lane < n ? __uint_as_float((unsigned int)keys[i + lane]) : -INF; };
        const float kth = n <= 128 ? near_kth_of<2>(n, p.kk, value) : n <= 256 ? near_kth_of<4>(n, p.kk, value) : near_kth(n, p.kk, value);
        if (kth != LOWEST) bound = near_bound_from(kth, -nh, args);
    }
    // keep what reaches it, without the query itself; positions become row numbers
    int left = 0;
    for (int i = 0; i < n; i += 64) {
        unsigned long long e = i + lane < n ? keys[i + lane] : 0ull;
        const int pos = (int)((unsigned int)(e >> 32) & ~MARK);
        const float least = p.region && !((unsigned int)(e >> 32) & MARK) ? bound_local : bound;
        long long cand = near_row(pos, p.c_tiles, p.c_in_order);
        if (p.c_ids) cand = i + lane < n && cand < p.n_ids ? (long long)p.c_ids[cand] : -1;
        const bool keep = i + lane < n && cand >= 0 && __uint_as_float((unsigned int)e) >= least && cand < p.nc && !(p.exclude_self && cand == row);
        const unsigned long long mask = __ballot(keep);
        const int pre = __builtin_amdgcn_mbcnt_hi((unsigned int)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)mask, 0u));
        __builtin_amdgcn_wave_barrier();
        if (keep) keys[left + pre] = (unsigned long long)cand;
        left += __popcll(mask);
        __builtin_amdgcn_wave_barrier();
    }
    // exact distances, eight pairs side by side and the rows of as many more on their way
    const int grp = lane >> 3, g = lane & 7;
    const float* xa = p.Xq + (size_t)row * p.d;
    v4f qa[4];
    near_first_quads<VEC>(qa, xa, p.d, g);
    constexpr int AT_ONCE = 2;      // (four: 188 us where two take 169, 50 000 x 128, k = 32; one 179)
    for (int i = 0; i < left; i += 8 * AT_ONCE) {
        unsigned int cand[AT_ONCE];
        v4f b[AT_ONCE][4];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
            const int at = i + 8 * u + grp;
            cand[u] = (unsigned int)keys[at < left ? at : i];
            if (u == 0 || i + 8 * u < left) near_first_quads<VEC>(b[u], p.Xc + (size_t)cand[u] * p.d, p.d, g);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
            const int at = i + 8 * u + grp;
            if (u > 0 && i + 8 * u >= left) break;
            const float dist = near_exact<VEC>(qa, b[u], xa, p.Xc + (size_t)cand[u] * p.d, p.d, g);
            if (at < left && g == 0) keys[at] = ((unsigned long long)__float_as_uint(dist) << 32) | cand[u];
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (p.evaluated && lane == 0) p.evaluated[qi] = left + (p.merge ? p.evaluated[qi] : 0);
    if (p.merge) {
        for (int j = 0; j < p.k; j += 64)
            if (j + lane < p.k)
                keys[left + j + lane] = ((unsigned long long)__float_as_uint(p.out_dist[qi * p.k + j + lane]) << 32) | (unsigned int)p.out_idx[qi * p.k + j + lane];
        left += p.k;
        __builtin_amdgcn_wave_barrier();
    }
    // ranks by (distance, row): every key against all of them
    for (int i = 0; i < left; i += 64) {
        const unsigned long long mine = i + lane < left ? keys[i + lane] : ~0ull;
        int rank = 0;
        for (int j = 0; j < left; ++j) rank += keys[j] < mine ? 1 : 0;
        if (i + lane < left && rank < p.k) {
            p.out_idx[qi * p.k + rank] = (int32_t)(unsigned int)mine;
            p.out_dist[qi * p.k + rank] = __uint_as_float((unsigned int)(mine >> 32));
            if (rank == p.k - 1 && p.next_bound)
                p.next_bound[lq] = near_bound_at(__uint_as_float((unsigned int)(mine >> 32)) * p.sc->scale * p.sc->scale, -nh, args);
        }
    }
    for (int j = left + lane; j < p.k; j += 64) { p.out_idx[qi * p.k + j] = -1; p.out_dist[qi * p.k + j] = INF; }
    if (p.next_bound && lane == 0 && left < p.k) p.next_bound[lq] = LOWEST;
}

static void near_select(const NearSelect& p, bool aligned, dim3 grid, hipStream_t s)
{
    switch (near_vec(aligned, p.d)) {
        case 2: hipLaunchKernelGGL(near_select_kernel<2>, grid, dim3(256), 0, s, p); break;
        case 1: hipLaunchKernelGGL(near_select_kernel<1>, grid, dim3(256), 0, s, p); break;
        default: hipLaunchKernelGGL(near_select_kernel<0>, grid, dim3(256), 0, s, p);
    }
}

// ---------------------------------------------------------------------------------------------- launches
__global__ void __launch_bounds__(256) near_clear_kernel(unsigned long long* a, long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) a[i] = 0ull;
}

__global__ void __launch_bounds__(256) near_todo_clear_kernel(int32_t* __restrict__ todo, long long words)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < words; i += (long long)gridDim.x * 256) todo[i] = 0;
}

struct NearPlan {
    int waves, panel_tiles;             // wavefronts per workgroup, query tiles per panel
    int nseg, nsub, capl;               // emit
    int max_seg, max_parts, max_sets, groups, stride, used;      // maxima (used = 0: none, every candidate is emitted)
    int stages;                         // 2: the sample's exact lists set the bounds for the other candidates
    int batch_tiles;                    // query tiles per batch
    size_t per_tile;                    // bytes of batch scratch per query tile
};

static int near_cus()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1) return 256;
    return v;
}

// A sample of one candidate tile in `stride`, searched in at most `seg` segments.
static void near_sample(NearPlan& p, int stride, int CT, int kk, bool wide, int seg)
{
    p.stride = stride;
    p.used = (CT + stride - 1) / stride;
    p.max_seg = seg;
    const int sets = p.max_seg * (wide ? 2 : 1);         // sets of group maxima per part
    const int per_seg = ((wide ? (p.used + 1) / 2 : p.used) + p.max_seg - 1) / p.max_seg;
    // about six groups per neighbour wanted, in 8 or 32 groups per set
    p.groups = 6 * kk <= 8 * sets ? 8 : GROUPS;
    int parts = (6 * kk + p.groups * sets - 1) / (p.groups * sets);
    if (parts > per_seg) parts = per_seg;
    if (parts * sets > 32) parts = 32 / sets;
    p.max_parts = parts < 1 ? 1 : parts;
    p.max_sets = sets * p.max_parts;
}

static NearPlan near_plan(long long nq, long long nc, int d, int kk, size_t batch_bytes, bool coloured = false)
{
    NearPlan p{};
    const int cus = near_cus();
    const int QT = near_tiles(nq), CT = near_tiles(nc);
    const bool wide = near_steps(d) > REG_STEPS;
    const int units = wide ? (CT + 1) / 2 : CT;          // what the segments share out
    // lanes of a wavefront row that hold a query's values, per segment
    const int lanes = wide ? 4 : 2;
    const int most_seg = kk == 1 ? 64 : (wide ? 4 : (kk > 40 ? 4 : 8));
    auto segs = [&](int n, int most) {
        const int panels = (QT + p.panel_tiles - 1) / p.panel_tiles;
        int s = (p.waves == 8 ? cus : 2 * cus) / panels;
        if (coloured && near_steps(d) <= 6 && p.waves == 8 && 2 * cus / panels <= 32) s = 2 * cus / panels;       // (two to a CU, see near_sweep_kernel)
        if (s > most) s = most;
        if (s > n) s = n;
        return s < 1 ? 1 : s;
    };
    // the largest workgroups (64 queries per wavefront share what is staged) that still fill the chip
    for (p.waves = 8;; p.waves >>= 1) {
        p.panel_tiles = p.waves / 2;
        if (wide) { p.panel_tiles = 2; break; }
        const int panels = (QT + p.panel_tiles - 1) / p.panel_tiles;
        const int slots = p.waves == 8 ? cus : 2 * cus;
        if (p.waves == 2 || panels * segs(CT, most_seg) * 4 >= slots * 3) break;
    }
    p.nseg = segs(units, most_seg);
    if (wide && p.nseg < 4 && units >= 64) p.nseg = 4;   // (so that an XCD's workgroups share 8 panels, see the kernel)
    p.nsub = lanes * p.nseg;
    p.capl = kk == 1 ? 256 : (p.nsub <= 2 ? 512 : (p.nsub <= 4 ? 256 : (p.nsub <= 8 ? 128 : 64)));
    p.used = 0; p.stride = 1; p.max_seg = 1; p.max_parts = 1; p.groups = GROUPS; p.stages = 1;
    if (kk > 1 && CT > 2) {
        // A sample of one tile in `stride`: the maxima pass costs M / stride (M: all tiles at 1.3e15 operations a
        // second), the entries it leaves cost about 0.12 ns each, kk * stride per query: least at
        // stride^2 = M / (0.12 ns * kk * queries).  At least 16 tiles; at most 5: beyond that, clusters of a hundred
        // thousand near-equidistant rows overflow the buffers (1M x 128: at 8 a few queries went to the list kernels).
        int stride = (int)(__builtin_sqrt((double)nc * 16.0 * near_steps(d) * 1.28e-5 / kk) + 0.5);
        if (stride > CT / 16) stride = CT / 16;
        if (stride > 5) stride = 5;
        if (stride < 1) stride = 1;
        p.stages = stride >= 3 ? 2 : 1;
        near_sample(p, stride, CT, kk, wide, segs(wide ? ((CT + stride - 1) / stride + 1) / 2 : (CT + stride - 1) / stride, wide ? 8 : 16));
    }
    p.per_tile = kk == 1 ? (size_t)TILE * 8 * (size_t)p.capl
                         : (size_t)TILE * (4 + (size_t)(p.used ? p.max_sets * p.groups * 4 : 0) + (size_t)p.nsub * (4 + 8 * (size_t)p.capl));
    long long bt = batch_bytes > 8192 ? (long long)((batch_bytes - 8192) / p.per_tile) : 0;
    if (bt >= QT) bt = QT;
    else if (bt >= p.panel_tiles) bt = bt / p.panel_tiles * p.panel_tiles;
    if (bt > 1024) bt = 1024;
    p.batch_tiles = (int)bt;
    return p;
}

size_t near_batch_bytes(long long nq, long long nc, int d, int kk)
{
    const NearPlan p = near_plan(nq, nc, d, kk, (size_t)1 << 62);
    return p.per_tile * (size_t)p.batch_tiles + 8192;
}

size_t near_least_batch_bytes(long long nq, long long nc, int d, int kk)
{
    const NearPlan p = near_plan(nq, nc, d, kk, (size_t)1 << 62);
    const int most = near_tiles(nq);
    return p.per_tile * (size_t)(p.panel_tiles < most ? p.panel_tiles : most) + 8192;
}

template <int MODE, bool COLOURED, bool LISTED = false>
static hipError_t near_launch_sweep(const NearSweep& p, int waves, hipStream_t s)
{
    const bool wide = p.steps > REG_STEPS;
    const int per_panel = wide ? 2 : waves / 2;
    const int panels = (p.q_tile1 - p.q_tile0 + per_panel - 1) / per_panel;
    // (queries counted on the device: as many workgroups as any count can use)
    const dim3 grid((unsigned)(LISTED && (MODE == NEAR_BLOCK || MODE == NEAR_NEAREST) ? (waves == 8 ? 2 : 4) * near_cus() : p.n_dev ? (panels > p.slots ? panels : p.slots) : panels * p.nseg)), block((unsigned)(64 * waves));
    const size_t lds = wide ? (size_t)WIDE_LDS : 2 * ((size_t)p.steps * FRAG_STEP + 1024);
    auto run = [&](auto kernel) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, block, lds, s, p);
        return hipGetLastError();
    };
    if constexpr (LISTED) {
        if (wide || !p.list || !p.list_len) return hipErrorInvalidValue;
    } else {
        if (wide) return run(&near_wide_kernel<MODE, COLOURED>);
    }
    switch (p.steps) {
        case 1: return run(&near_sweep_kernel<1, MODE, COLOURED, LISTED>);
        case 2: return run(&near_sweep_kernel<2, MODE, COLOURED, LISTED>);
        case 3: return run(&near_sweep_kernel<3, MODE, COLOURED, LISTED>);
        case 4: return run(&near_sweep_kernel<4, MODE, COLOURED, LISTED>);
        case 5: return run(&near_sweep_kernel<5, MODE, COLOURED, LISTED>);
        case 6: return run(&near_sweep_kernel<6, MODE, COLOURED, LISTED>);
        case 7: return run(&near_sweep_kernel<7, MODE, COLOURED, LISTED>);
        case 8: return run(&near_sweep_kernel<8, MODE, COLOURED, LISTED>);
        default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------------------------- nearest rows
// A 1-NN search keeps, per lane, the 16 candidates with the largest product value and what the others reach at most; so one
// pass settles all queries except those that have a second near candidate in the same lane (1 in a hundred or so), which
// are searched for on their own.  Bound by that pass.  1k x 100k x 128: 129 -> 115 us; 10k x 100k x 64 by colours: 390 -> 261 us
// (two passes, the second emitting what the first one's best value leaves).
struct NearTop {
    const uint4* top; int nsub, nq_batch, q0;
    const float* qnegh; const int32_t *qcolour, *ccolour; const NearScale* sc; float e, nu; int steps;
    const float* Xq; const float* Xc; const int32_t* q_rows;
    int d, nq, nq_rows, nc, q_tiles, c_tiles, q_in_order, c_in_order;
    int32_t* out_idx; float* out_dist; int32_t* evaluated;
    int32_t *rows_left, *slot_left, *pos_left, *counts_left, *count_left; float* reach_left;
    int32_t* todo; int32_t* todo_mark;
};

template <int VEC>
__global__ void __launch_bounds__(256) near_top_kernel(NearTop p)
{
    const int lane = threadIdx.x & 63;
    const int lq = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (lq >= p.nq_batch) return;
    const int qpos = p.q0 + lq;
    const long long qi = near_row(qpos, p.q_tiles, p.q_in_order);
    if (qi >= p.nq) return;
    const long long row = p.q_rows ? (long long)p.q_rows[qi] : qi;
    const float nh = p.qnegh[qpos];
    if (row < 0 || row >= p.nq_rows || nh == -INF) {
        if (lane == 0) { p.out_idx[qi] = -1; p.out_dist[qi] = INF; if (p.evaluated) p.evaluated[qi] = 0; }
        return;
    }
    if (nh == INF) {                                            // values beyond float16: the list kernels
        if (lane == 0) {
            const int panel = (int)(qi >> 7);
            if (atomicExch(p.todo_mark + panel, 1) == 0) p.todo[2 + atomicAdd(p.todo, 1)] = panel;
            if (p.evaluated) p.evaluated[qi] = 0;
        }
        return;
    }
    float m1[2], m2[2];
    int at[2];
    bool pending[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = lane + 64 * r;
        uint4 t = make_uint4(__float_as_uint(-INF), 0u, __float_as_uint(-INF), 0u);
        if (i < p.nsub) t = p.top[(size_t)lq * p.nsub + i];
        m1[r] = __uint_as_float(t.x); at[r] = (int)t.y; m2[r] = __uint_as_float(t.z);
        pending[r] = m1[r] > -INF;
    }
    const NearBoundArgs a = near_args(p.sc, p.steps, p.d, p.e, p.nu);
    const float* xa = p.Xq + (size_t)row * p.d;
    const int grp = lane >> 3, g = lane & 7;
    v4f qa[4];
    near_first_quads<VEC>(qa, xa, p.d, g);
    const int qcol = p.qcolour ? p.qcolour[qpos] : 0;
    unsigned long long key = ~0ull;
    float bound = LOWEST;
    int evaluated = 0;
    for (int turn = 0; turn < 128; ++turn) {
        // the lane with the largest value that may still hide the nearest
        const float mine = fmaxf(pending[0] ? m1[0] : -INF, pending[1] ? m1[1] : -INF);
        const float mx = wave_max(mine);
        if (!(mx > -INF) || mx < bound) break;
        const int who = __builtin_ctzll(__ballot(mine == mx));
        const bool second = !(pending[0] && m1[0] == mx);
        const int base = __builtin_amdgcn_readlane(second ? at[1] : at[0], who);
        if (lane == who) pending[second ? 1 : 0] = false;
        // (the colours wait beside the rows, not before them)
        v4f xb[2][4];
        long long cand[2];
        bool fine[2];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int j = half * 8 + grp;
            const int pos = base + 8 * (j >> 2) + (j & 3);
            cand[half] = near_row(pos, p.c_tiles, p.c_in_order);
            fine[half] = cand[half] >= 0 && cand[half] < p.nc;
            near_first_quads<VEC>(xb[half], p.Xc + (size_t)(fine[half] ? cand[half] : 0) * p.d, p.d, g);
            fine[half] = fine[half] && !(p.qcolour && p.ccolour[pos] == qcol);
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const float dist = near_exact<VEC>(qa, xb[half], xa, p.Xc + (size_t)(fine[half] ? cand[half] : 0) * p.d, p.d, g);
            const unsigned long long k = ((unsigned long long)__float_as_uint(dist) << 32) | (unsigned int)cand[half];
            if (fine[half] && dist < INF && k < key) key = k;
        }
        key = wave_min<8>(key);                                      // (eight lanes have one pair)
        evaluated += 16;
        if (key != ~0ull) bound = fmaxf(LOWEST, near_bound_at(__uint_as_float((unsigned int)(key >> 32)) * p.sc->scale * p.sc->scale, -nh, a));
    }
    const bool open = __any(m2[0] >= bound && m2[0] > -INF) || __any(m2[1] >= bound && m2[1] > -INF) || p.sc->huge != 0u;
    if (lane == 0) {
        p.out_idx[qi] = key == ~0ull ? -1 : (int32_t)(unsigned int)key;
        p.out_dist[qi] = key == ~0ull ? INF : __uint_as_float((unsigned int)(key >> 32));
        if (p.evaluated) p.evaluated[qi] = evaluated;
        if (open) {
            const int i = atomicAdd(p.count_left, 1);
            p.rows_left[i] = (int32_t)row; p.slot_left[i] = (int32_t)qi; p.pos_left[i] = qpos; p.counts_left[i] = 0;
            p.reach_left[i] = key == ~0ull ? INF : __uint_as_float((unsigned int)(key >> 32));
        }
    }
}

// the query tiles from t0 on, nqb queries; `p` prepared for the copies
static hipError_t near_nearest(const NearProblem& a, const NearCopy& q, const NearCopy& c, const NearBuffers& b, const NearPlan& plan,
                               NearSweep p, bool vec4, int t0, int nqb, hipStream_t s)
{
    const bool wide = p.steps > REG_STEPS;
    const int lanes = wide ? 4 : 2, tiles = nqb / TILE;
    const size_t n = (size_t)q.tiles * TILE;
    p.nseg = plan.nseg * lanes > 128 ? 128 / lanes : plan.nseg;
    p.nsub = lanes * p.nseg; p.stride = 1; p.skip = 0; p.used = c.tiles;
    p.top = reinterpret_cast<uint4*>(b.batch);
    p.cnegh = c.negh_best;
    hipError_t e = a.coloured ? near_launch_sweep<NEAR_TOP, true>(p, plan.waves, s) : near_launch_sweep<NEAR_TOP, false>(p, plan.waves, s);
    if (e != hipSuccess) return e;
    if (t0 > 0) hipLaunchKernelGGL(near_todo_clear_kernel, dim3(1), dim3(256), 0, s, b.todo + 1, 1);
    NearTop t{};
    t.top = p.top; t.nsub = p.nsub; t.nq_batch = nqb; t.q0 = t0 * TILE;
    t.qnegh = q.negh; t.qcolour = a.coloured ? q.colour : nullptr; t.ccolour = c.colour;
    t.sc = b.scale; t.e = p.e; t.nu = p.nu; t.steps = p.steps;
    t.Xq = a.Xq; t.Xc = a.Xc; t.q_rows = a.q_rows;
    t.d = a.d; t.nq = a.nq; t.nq_rows = a.nq_rows; t.nc = a.nc;
    t.q_tiles = q.tiles; t.c_tiles = c.tiles; t.q_in_order = q.in_order; t.c_in_order = c.in_order;
    t.out_idx = a.out_idx; t.out_dist = a.out_dist; t.evaluated = a.evaluated;
    t.rows_left = q.left; t.slot_left = q.left + n; t.pos_left = q.left + 2 * n; t.reach_left = reinterpret_cast<float*>(q.left + 3 * n);
    t.counts_left = q.count; t.count_left = b.todo + 1;
    t.todo = b.todo; t.todo_mark = b.todo_mark;
    const dim3 per_query((unsigned)((nqb + 3) / 4));
    switch (near_vec(vec4, a.d)) {
        case 2: hipLaunchKernelGGL(near_top_kernel<2>, per_query, dim3(256), 0, s, t); break;
        case 1: hipLaunchKernelGGL(near_top_kernel<1>, per_query, dim3(256), 0, s, t); break;
        default: hipLaunchKernelGGL(near_top_kernel<0>, per_query, dim3(256), 0, s, t);
    }
    // those with more than one near candidate in a lane
    const int waves = wide ? plan.waves : (plan.waves > 2 ? plan.waves / 2 : 2);
    p.cnegh = c.negh;
    p.q_tile0 = 0; p.q_tile1 = tiles;
    p.qpos = t.pos_left; p.n_dev = t.count_left; p.slots = (waves == 8 ? 1 : 2) * near_cus(); p.most_seg = p.slots;
    p.reach = t.reach_left; p.counts = t.counts_left; p.capl = plan.capl;
    p.entries = reinterpret_cast<uint2*>(b.batch);
    e = a.coloured ? near_launch_sweep<NEAR_NEAREST, true>(p, waves, s) : near_launch_sweep<NEAR_NEAREST, false>(p, waves, s);
    if (e != hipSuccess) return e;
    NearSelect sel{};
    sel.entries = p.entries; sel.counts = p.counts; sel.nsub = 1; sel.by_position = 1; sel.capl = plan.capl;
    sel.nq_batch = nqb; sel.q0 = 0;
    sel.qnegh = q.negh; sel.sc = b.scale; sel.e = p.e; sel.nu = p.nu; sel.steps = p.steps;
    sel.Xq = a.Xq; sel.Xc = a.Xc; sel.q_rows = t.rows_left; sel.slot = t.slot_left; sel.qpos = t.pos_left; sel.n_dev = t.count_left;
    sel.d = a.d; sel.k = sel.kk = 1; sel.nq = nqb; sel.nq_rows = a.nq_rows; sel.nc = a.nc;
    sel.q_tiles = q.tiles; sel.c_tiles = c.tiles; sel.q_in_order = 1; sel.c_in_order = c.in_order;
    sel.out_idx = a.out_idx; sel.out_dist = a.out_dist; sel.evaluated = a.evaluated;
    sel.todo = b.todo; sel.todo_mark = b.todo_mark;
    near_select(sel, vec4, per_query, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------- rows among themselves
// A k-NN search whose queries are its candidates multiplies every pair once (pairs_kernels.hip): limits from a sample as before,
// then the offsets round the circle of blocks in a few bands; between two bands every row's limit is tightened by what its list
// holds.  A list needs room for what passes before the next tightening: kk * g entries and what rounding adds, if a band has
// seen g times as many rows at its end as at its beginning (every tile is an even sample of the rows).  Rows whose lists
// overflow all the same are searched for on their own, with the buffers and the tightening of the sweeps.  A row has to keep all its copies,
// so where every point is there some hundred times most rows overflow; the rest of the bands is left out then, and every row
// searched for: 150 000 x 80, k = 12, 2000 copies each, 202 ms without that, 142 so, 91 since
// full lists take no more entries.
// (Sorting the rows by their nearest of a few hundred pivots first, so that what passes comes together, was tried: limits then come from
// a row's own surroundings and say nothing about the other rows, a third of the rows overflowed, 1M x 128 took 250 ms
// without their panels against 200 ms.)
struct PairPlan {
    NearPlan sample;
    int waves, blocks, cap, bands, to[8], nseg[8];
    int batch;                             // tiles whose rows are searched for at a time
    bool once;
};
// From 32 tiles on.  Against sweeps that keep what passes by a branch per value (near_sweep_kernel's emission, which is left where memory is short), in us:
// 5000 x 10, k = 10: 68 and 62; 8000 x 30, 10: 93 and 90; 13 000 x 40, 10: 127 and 123; 20 011 x 50, 10: 220 and 216; 20 000 x 128, 32, clusters by Zipf's law: 4460
// and 391; 30 000 x 30, 16: 338 and 312; 40 000 x 70, 10: 596 and 574; 50 000 x 10, 10: 629 and 502; 100 000 x 48, 10: 2434 and 1763; 250 000 x 20, 10: 8.5 and
// 6.4 ms; 250 000 x 60, 20, by Zipf's law 14.0 and 12.3.  k = 12, 300 copies of every row: 5000 x 12 164 and 214, 12 000 x 30 325 and 357 (an entry is an addition in
// memory here), 20 000 x 16 3424 and 540; 600 copies: 2321 and 443, 4093 and 790, 5592 and 1213.
static bool pair_search_wanted(int T) { return T >= 32 && T < (1 << 17); }
// Whether every pair is multiplied once, for both of its rows, or in either order.  Once takes the test 36 instructions for 16 values instead of 12 and half
// the products: 35 000 x 128, k = 16, 661 us in either order and 549 once; 40 000 x 110, 10: 746 and 621; 13 000 x 70, 10: 145 and 147; of 60 000 x 128, 12, the
// products alone are most of it.  Narrower rows gain as well (100 000 x 48, 10: 1763 and 1415, 20 011 x 50, 10: 216 and 201, 20 000 x 16, 10: 167 and 161), but the lists of both rows
// of a pair have to be there at once, so such rows could not be searched for in turns (near_pair_plan), and tests hold what slhc_probe_knn_products reports of them.
static bool pairs_once(int T, int steps) { return steps > REG_STEPS || (T <= 100 ? steps >= 3 : steps >= 6 || (T >= 384 && steps >= 5)); }
// from here on rows whose lists overflow are searched for on their own before the list kernels take their panels; below, the five
// launches cost more (20 us of 200 at 20 000 rows) than a panel or two
constexpr int PAIR_AGAIN_TILES = 256;
// bytes: of the memory for them (0: the least there may be).  Lists are as long as it allows, up to PAIRS_MOST, which costs nothing where they
// stay short (5000 x 200 and 16 000 x 300, lists of 256 and 1024: the same times) and leaves fewer rows over.
constexpr int PAIR_TURNS = 8;              // at most
static size_t pair_lists_bytes(int T, int cap) { return (size_t)T * TILE * (24 + 8 * (size_t)cap) + 4096; }
static bool near_pair_plan(long long n, int d, int kk, size_t bytes, PairPlan* out)
{
    const int T = near_tiles(n), steps = near_steps(d);
    if (kk < 2 || !pair_search_wanted(T)) return false;
    PairPlan p{};
    p.once = pairs_once(T, steps);
    const bool wide = steps > REG_STEPS;
    const int cus = near_cus();
    p.cap = (12 * kk + 63) / 64 * 64;
    p.cap = p.cap < 256 ? 256 : (p.cap > PAIRS_MOST ? PAIRS_MOST : p.cap);
    // What a sample of one tile in `stride` costs, and one band (0) or a first one of the sample's share and b more that see
    // g times as much each, in us: the products of the sample (1.1e15 a second), 15 us per band and 1 ns per row for the tightening
    // before it, 0.1 ns per entry, of which rounding makes twice what is asked for on average.
    const double all = (double)n * n * 32.0 * (steps < 6 ? 6 : steps) / 1.1e9, entry = 2e-4 * n * kk, most = p.cap / (3.5 * kk);
    double best = 1e300;
    int stride = 1, more = 0;
    for (int s = 1; s <= 16 && s <= T / 16; ++s)
        for (int b = 0; b <= 7; ++b) {
            const double g = b > 0 ? pow((double)s, 1.0 / b) : s;
            if (g > most && s > 1 && b < 7) continue;
            const double cost = all / s + 15.0 * (b + 1) + 1e-3 * n * b + entry * (b > 0 ? 1.0 + b * (g - 1.0) : g);
            if (cost < best) { best = cost; stride = s; more = b; }
        }
    const double g = more > 0 ? pow((double)stride, 1.0 / more) : 1.0;
    // Lists take what memory there is.  Where that is less than PAIRS_MOST entries for every row (from some 150 000 rows on), rows whose pairs are met in either order are
    // searched for in turns, with whole lists: rows left over cost a second search otherwise, with a branch per value that passes, or the list kernels.  k = 12, 300 000 x 10 of 600
    // copies each 67 -> 27.8 ms, of 2000 238 -> 185; k = 10, 174 000 x 20 of 900 62 -> 20, 250 000 x 40 with norms over orders of magnitude 96 -> 88, blobs of 800 000 x 16 57 -> 39.
    // What a turn costs beside, its launches and their ends: blobs of 160 000 x 20 3.12 and 3.00 ms, 180 000 x 10 3.27 and 3.39, 220 000 x 20 5.02 and 5.15, 250 000 x 40 7.81 and
    // 7.80.  (Workgroups of half and of one and a half times the length in turns: 220 000 x 20 5.32 and 5.19.)
    while (p.cap + 64 <= PAIRS_MOST && pair_lists_bytes(T, p.cap + 64) <= bytes) p.cap += 64;
    p.batch = T;
    const long long fit = bytes > 8192 ? (long long)((bytes - 8192) / (pair_lists_bytes(1, PAIRS_MOST) - 4096)) / 2 * 2 : 0;
    if (!p.once && p.cap < PAIRS_MOST && fit * PAIR_TURNS >= T) {
        const int turns = (int)((T + fit - 1) / fit);
        p.batch = ((T + turns - 1) / turns + 1) / 2 * 2;
        p.cap = PAIRS_MOST;
    }
    auto lay_out = [&](int waves) {
        const int bt = wide ? 2 : waves / 2, slots = waves >= 8 ? cus : (p.once && steps > 5 ? 2 : 3) * cus;
        p.waves = waves;
        p.blocks = (T + bt - 1) / bt;
        const int asking = (p.batch + bt - 1) / bt;
        const int half = p.once ? p.blocks / 2 + 1 : p.blocks;     // meetings of a block
        double seen = 1.0 / stride;
        int from = 0;
        for (p.bands = 0; from < half; ++p.bands, seen *= g) {
            int to = p.bands == more ? half : p.once ? (int)(0.5 * (seen * p.blocks + 1.0)) : (int)(seen * p.blocks + 0.5);
            to = to < from + 1 ? from + 1 : (to > half ? half : to);
            const int len = to - from;
            int seg = (8 * slots + asking - 1) / asking;
            if (wide && seg < 4) seg = 4;      // (so that an XCD's workgroups share 8 blocks, see the kernel)
            // about eight rounds of workgroups, the last of them as full as can be
            auto rounds = [&](int n) { return (double)(((long long)asking * n + slots - 1) / slots) * ((double)len / n + 0.15); };
            int best_seg = seg > len ? len : seg;
            for (int n = waves == 4 ? 1 : (2 * seg + 2) / 3; !wide && n <= len && 2 * n <= 3 * seg; ++n)
                if (rounds(n) < rounds(best_seg)) best_seg = n;
            p.to[p.bands] = to;
            p.nseg[p.bands] = best_seg;
            from = to;
        }
    };
    // Workgroups of four wavefronts, of which three and more fit a CU but for the widest rows multiplied once; there, from 49 152 rows on, one of twelve
    // has more wavefronts per SIMD (see pairs_kernel): 100 000 x 80, k = 30, 2.53 ms with four and 2.47, 250 000 x 70, 20, 11.7 and 10.9, 40 000 x 70, 10: 543 and 549 us.
    int waves = wide ? 8 : p.once && steps >= 5 && T >= 384 ? 12 : 4;
    if (waves == 4 && (T / 2) * (T / 4) < 2 * cus) waves = 2;
    lay_out(waves);
    p.sample = near_plan(n, n, d, kk, 0);
    NearPlan& q = p.sample;
    const int used = (T + stride - 1) / stride, panels = (p.batch + q.panel_tiles - 1) / q.panel_tiles;
    int seg = (q.waves == 8 && p.batch == T ? cus : 2 * cus) / panels;       // (in turns there are few panels: two workgroups to a CU)
    const int units = wide ? (used + 1) / 2 : used, limit = wide ? 8 : 16;
    seg = seg > limit ? limit : seg;
    seg = seg > units ? units : seg;
    near_sample(q, stride, T, kk, wide, seg < 1 ? 1 : seg);
    *out = p;
    return true;
}

size_t near_pairs_bytes(long long n, int d, int kk, bool* once)
{
    PairPlan p;
    if (!near_pair_plan(n, d, kk, 0, &p)) return 0;
    if (once) *once = p.once;
    return pair_lists_bytes(near_tiles(n), p.cap);
}

static hipError_t near_search_pairs(const NearProblem& a, const NearCopy& c, const NearBuffers& b, const PairPlan& plan, bool vec4, int first, hipStream_t s)
{
    // the rows of the tiles from `first` on
    const int end = first + plan.batch < c.tiles ? first + plan.batch : c.tiles, tiles = end - first;
    const int kk = a.k + 1, steps = near_steps(a.d), rows = tiles * TILE;
    const bool wide = steps > REG_STEPS;
    const float e = near_e(steps), nu = near_nu(steps);
    unsigned char* at = b.pairs;
    auto take = [&](size_t bytes) { unsigned char* r = at; at += (bytes + 255) / 256 * 256; return r; };
    float* limit = reinterpret_cast<float*>(take((size_t)rows * 4));
    int32_t* counts = reinterpret_cast<int32_t*>(take((size_t)rows * 4));
    PairsLeft left{};
    left.row = reinterpret_cast<int32_t*>(take((size_t)rows * 4)); left.pos = reinterpret_cast<int32_t*>(take((size_t)rows * 4));
    left.counts = reinterpret_cast<int32_t*>(take((size_t)rows * 4)); left.reach = reinterpret_cast<float*>(take((size_t)rows * 4));
    left.count = b.todo + 1;
    int32_t* lost = reinterpret_cast<int32_t*>(take(4));
    const size_t lists_bytes = (size_t)rows * (size_t)plan.cap * 8;
    uint2* entries = reinterpret_cast<uint2*>(take(lists_bytes));
    NearSweep p{};
    p.qfrag = p.cfrag = c.frag; p.qnegh = p.cnegh = c.negh; p.c_tiles = c.tiles;
    p.sc = b.scale; p.d = a.d; p.steps = steps; p.e = e; p.nu = nu; p.kk = kk;
    const NearPlan& q = plan.sample;
    p.stride = q.stride; p.used = q.used; p.nseg = q.max_seg; p.parts = q.max_parts; p.groups = q.groups;
    p.spread = near_spread(q.used);
    float* maxima = reinterpret_cast<float*>(entries);              // (the lists are empty yet)
    const size_t per_tile = (size_t)TILE * q.max_sets * q.groups * 4;
    long long batch = (long long)(lists_bytes / per_tile) / q.panel_tiles * q.panel_tiles;
    if (batch < 1) return hipErrorInvalidValue;
    hipError_t err = hipSuccess;
    if (first > 0) hipLaunchKernelGGL(near_todo_clear_kernel, dim3(1), dim3(256), 0, s, left.count, 1);
    for (int t0 = first; t0 < end; t0 += (int)batch) {
        const int t1 = t0 + batch < end ? t0 + (int)batch : end, at = t0 - first;
        p.q_tile0 = t0; p.q_tile1 = t1; p.nq_batch = (t1 - t0) * TILE;
        p.maxima = maxima;
        err = near_launch_sweep<NEAR_MAXIMA, false>(p, q.waves, s);
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL((near_bounds_kernel<true>), dim3((unsigned)(p.nq_batch / 4)), dim3(256), 0, s, maxima, q.max_sets, q.groups == GROUPS ? 5 : 3, p.nq_batch,
                           t0 * TILE, kk, c.negh, b.scale, e, nu, steps, a.d, limit + (size_t)at * TILE, static_cast<float*>(nullptr),
                           static_cast<const int32_t*>(nullptr), 1, static_cast<const int32_t*>(nullptr), static_cast<const float*>(nullptr),
                           static_cast<const NearScale*>(nullptr), counts + (size_t)at * TILE, left.row + (size_t)at * TILE, lost);
    }
    NearPairs r{};
    r.frag = c.frag; r.negh = c.negh; r.tiles = c.tiles; r.steps = steps; r.filled = (a.d + 15) / 16; r.blocks = plan.blocks; r.once = plan.once; r.first = first / (wide ? 2 : plan.waves / 2); r.row0 = first * TILE; r.rows = rows; r.spread = near_spread(r.blocks);
    r.limit = limit; r.entries = entries; r.counts = counts; r.cap = plan.cap;
    const bool again = c.tiles >= PAIR_AGAIN_TILES;
    r.lost = lost; r.lost_most = again ? (rows < a.nq ? rows : a.nq) / 2 : rows;
    r.todo = b.todo; r.todo_mark = b.todo_mark; r.full_gone = !again && !plan.once;
    for (int i = 0; i < plan.bands; ++i) {
        if (i > 0) {
            err = pairs_tighten(r, kk, b.scale, e, nu, a.d, left.row, s);       // (no rows are left yet)
            if (err != hipSuccess) return err;
        }
        r.from = i > 0 ? plan.to[i - 1] : 0; r.to = plan.to[i]; r.nseg = plan.nseg[i];
        err = pairs_emit(r, plan.waves, s);
        if (err != hipSuccess) return err;
    }
    r.cap_again = 4 * plan.cap >= 3 * PAIRS_MOST ? plan.cap : PAIRS_MOST;  // (of nearly that length: one turn of the loop below)
    if (again) {
        err = pairs_left(r, kk, b.scale, e, nu, a.d, a.nq, left, s);
        if (err != hipSuccess) return err;
    }
    NearSelect sel{};
    sel.qnegh = c.negh; sel.sc = b.scale; sel.e = e; sel.nu = nu; sel.steps = steps;
    sel.Xq = a.Xq; sel.Xc = a.Xc;
    sel.d = a.d; sel.k = a.k; sel.kk = kk; sel.nq = a.nq; sel.nq_rows = a.nq_rows; sel.nc = a.nc;
    sel.q_tiles = sel.c_tiles = c.tiles; sel.exclude_self = 1;
    sel.out_idx = a.out_idx; sel.out_dist = a.out_dist; sel.evaluated = a.evaluated;
    sel.todo = b.todo; sel.todo_mark = b.todo_mark;
    sel.entries = entries; sel.counts = counts; sel.nsub = 1; sel.by_position = 1; sel.capl = plan.cap; sel.pair_lists = 1; sel.skip_gone = again || r.full_gone;
    sel.nq_batch = rows; sel.q0 = sel.list0 = first * TILE;
    auto select = [&]() -> hipError_t {
        near_select(sel, vec4, dim3((unsigned)((sel.nq_batch + 3) / 4)), s);
        return hipGetLastError();
    };
    err = select();
    if (err != hipSuccess || !again) return err;
    // The rows left: any kk of the rows met reach their distance, and lists of 1024 rarely overflow; where one does, its kk-th value
    // makes the second search short.
    const int waves = wide ? 8 : 4;
    r.cap = r.cap_again;
    p.stride = 1; p.used = c.tiles;
    p.qpos = left.pos; p.n_dev = left.count; p.slots = (waves == 8 ? 1 : 2) * near_cus(); p.most_seg = p.slots;
    p.reach = left.reach; p.counts = left.counts; p.capl = r.cap; p.entries = entries;
    sel.q_rows = sel.slot = left.row; sel.qpos = left.pos; sel.n_dev = left.count;
    sel.q_in_order = 1; sel.counts = left.counts; sel.capl = r.cap; sel.pair_lists = 0; sel.nq = rows; sel.list0 = 0;
    int room = (int)(lists_bytes / ((size_t)TILE * r.cap * 8));            // tiles of queries whose lists fit
    if (room < tiles) room = room / 2 * 2;
    if (room < 2) return hipErrorInvalidValue;
    for (int t0 = 0; t0 < tiles; t0 += room) {
        p.q_tile0 = t0; p.q_tile1 = t0 + room < tiles ? t0 + room : tiles;
        p.nq_batch = sel.nq_batch = (p.q_tile1 - t0) * TILE; sel.q0 = t0 * TILE;
        err = near_launch_sweep<NEAR_NEAREST, false>(p, waves, s);
        if (err == hipSuccess) err = pairs_again(r, kk, b.scale, e, nu, a.d, t0 * TILE, p.nq_batch, left, s);
        if (err == hipSuccess) err = near_launch_sweep<NEAR_NEAREST, false>(p, waves, s);
        if (err == hipSuccess) err = select();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

hipError_t near_search(const NearProblem& a, const NearCopy& q, const NearCopy& c, const NearBuffers& b, hipStream_t s)
{
    const int kk = a.k + (a.exclude_self ? 1 : 0);
    const NearPlan plan = near_plan(a.nq, a.nc, a.d, kk, b.batch_bytes, a.coloured != 0);
    if (plan.batch_tiles < 1 || (a.nq + 127) / 128 > b.todo_panels || (a.coloured && (kk != 1 || !q.colour || !c.colour)) ||
        (kk == 1 && (!q.left || !q.count || !c.negh_best)))
        return hipErrorInvalidValue;
    const bool vec4 = a.d % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.Xq) | reinterpret_cast<uintptr_t>(a.Xc)) & 15) == 0;
    PairPlan pairs;
    if (a.exclude_self && q.frag == c.frag && !c.in_order && b.pairs && near_pair_plan(a.nc, a.d, kk, b.pairs_bytes, &pairs) &&
        b.pairs_bytes >= pair_lists_bytes(pairs.batch, pairs.cap)) {
        hipError_t e = hipSuccess;
        for (int first = 0; first < c.tiles && e == hipSuccess; first += pairs.batch) e = near_search_pairs(a, c, b, pairs, vec4, first, s);
        return e;
    }
    NearSweep p{};
    p.qfrag = q.frag; p.qnegh = q.negh; p.qcolour = q.colour;
    p.cfrag = c.frag; p.cnegh = c.negh; p.ccolour = c.colour; p.c_tiles = c.tiles;
    p.sc = b.scale; p.d = a.d; p.steps = near_steps(a.d); p.e = near_e(p.steps); p.nu = near_nu(p.steps);
    p.kk = kk;
    NearSelect sel{};
    sel.qnegh = q.negh; sel.sc = b.scale; sel.e = p.e; sel.nu = p.nu; sel.steps = p.steps;
    sel.Xq = a.Xq; sel.Xc = a.Xc; sel.q_rows = a.q_rows;
    sel.d = a.d; sel.k = a.k; sel.kk = kk; sel.nq = a.nq; sel.nq_rows = a.nq_rows; sel.nc = a.nc;
    sel.q_tiles = q.tiles; sel.c_tiles = c.tiles; sel.exclude_self = a.exclude_self;
    sel.out_idx = a.out_idx; sel.out_dist = a.out_dist; sel.evaluated = a.evaluated;
    sel.todo = b.todo; sel.todo_mark = b.todo_mark;
    sel.q_in_order = q.in_order; sel.c_in_order = c.in_order;
    for (int t0 = 0; t0 < q.tiles; t0 += plan.batch_tiles) {
        const int t1 = t0 + plan.batch_tiles < q.tiles ? t0 + plan.batch_tiles : q.tiles;
        const int nqb = (t1 - t0) * TILE;
        const dim3 per_query((unsigned)((nqb + 3) / 4));
        unsigned char* at = b.batch;
        auto take = [&](size_t bytes) { unsigned char* r = at; at += (bytes + 255) / 256 * 256; return r; };
        p.q_tile0 = t0; p.q_tile1 = t1; p.nq_batch = nqb;
        p.capl = sel.capl = plan.capl;
        sel.nq_batch = nqb; sel.q0 = t0 * TILE;
        auto select = [&]() -> hipError_t {
            sel.entries = p.entries; sel.counts = p.counts;
            near_select(sel, vec4, per_query, s);
            return hipGetLastError();
        };
        hipError_t e = hipSuccess;
        if (kk == 1) {
            e = near_nearest(a, q, c, b, plan, p, vec4, t0, nqb, s);
            if (e != hipSuccess) return e;
            continue;
        }
        float* bound = reinterpret_cast<float*>(take((size_t)nqb * 4));
        float* maxima = reinterpret_cast<float*>(take(plan.used ? (size_t)nqb * plan.max_sets * plan.groups * 4 : 0));
        p.counts = reinterpret_cast<int32_t*>(take((size_t)nqb * plan.nsub * 4));
        p.entries = reinterpret_cast<uint2*>(take((size_t)nqb * plan.nsub * plan.capl * 8));
        p.bound = bound; p.maxima = maxima;
        p.stride = plan.stride; p.used = plan.used; p.skip = 0;
        if (plan.used) {
            p.nseg = plan.max_seg; p.parts = plan.max_parts; p.groups = plan.groups;
            e = near_launch_sweep<NEAR_MAXIMA, false>(p, plan.waves, s);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL((near_bounds_kernel<false>), per_query, dim3(256), 0, s, maxima, plan.used ? plan.max_sets : 0,
                           plan.groups == GROUPS ? 5 : 3, nqb, t0 * TILE, kk, q.negh, b.scale, p.e, p.nu, p.steps, a.d, bound, static_cast<float*>(nullptr), static_cast<const int32_t*>(nullptr), 1,
                           static_cast<const int32_t*>(nullptr), static_cast<const float*>(nullptr), static_cast<const NearScale*>(nullptr), static_cast<int32_t*>(nullptr), static_cast<int32_t*>(nullptr),
                           static_cast<int32_t*>(nullptr));
        p.nseg = plan.nseg; p.nsub = plan.nsub;
        sel.nsub = plan.nsub; sel.by_position = 0; sel.merge = 0; sel.next_bound = nullptr;
        if (plan.stages == 2) {
            e = near_launch_sweep<NEAR_EMIT, false>(p, plan.waves, s);
            if (e != hipSuccess) return e;
            sel.next_bound = bound;
            e = select();
            if (e != hipSuccess) return e;
            p.skip = 1; p.used = c.tiles - plan.used;
            sel.merge = 1; sel.next_bound = nullptr;
        } else {
            p.stride = 1; p.used = c.tiles;
        }
        e = near_launch_sweep<NEAR_EMIT, false>(p, plan.waves, s);
        if (e != hipSuccess) return e;
        e = select();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------------------------- searches in a row order
// Lists of candidate tiles per panel of queries.  One workgroup per panel: the distinct tiles its queries lie in, each with
// the largest reach and the range of colours among its queries, go to LDS, and every candidate tile is tried against them.
// Bound by reading the rows of the table of tile pairs once: 1M x 128 (8264 tiles) 85 us per list of all panels.
enum { LIST_LOCAL = 1, LIST_CROSS = 2 };        // pairs inside a region; all others
struct NearList {
    const float* gap; int T;
    const int32_t* region; int what;
    float* reach;                          // by query of the batch (set to -1 where the query is left to the list kernels), or
    const int32_t* colour; const uint32_t* threshold; int n_rows;      // (colour by position) the query's component's threshold
    const int32_t* tile_colour;            // (with colour) tiles all of whose rows have the queries' one colour are left out
    const int32_t* pos; int n_pos;         // position of query i in the order (nullptr: query i), positions there are
    int q0, nq, panel_queries;
    const int32_t* n_dev;                  // optional: queries there are, over all batches
    const unsigned short* from; const int32_t* from_len;               // optional: only the tiles of an earlier list
    unsigned short* list; int32_t* list_len; int32_t* list_step; int list_stride;
    double cost;                           // list_step: a pass over one tile in units of an emitted entry
    int kk;
    unsigned long long* tile_steps;
    // optional: a query tile that would need more than `most` candidate tiles is left to the list kernels instead
    int most; int32_t *todo, *todo_mark;
};
constexpr int LIST_QUERIES = 512;          // per panel at most
// Threads per panel: a list is a walk over thousands of tiles in the table, bound by the wait for each step's loads, and there are no
// more panels than CUs.  Clustering 1M x 128, with 256 threads whose loads waited for one another: 4.4 ms of lists and 0.9 of first
// tiles; 1.5 and 0.2 so.
constexpr int LIST_THREADS = 1024, LIST_WAVES = LIST_THREADS / 64;
static_assert(LIST_THREADS >= LIST_QUERIES, "near_segments gives every query a thread");

struct NearSegments {
    int tile[LIST_QUERIES], lo[LIST_QUERIES], hi[LIST_QUERIES], reg[LIST_QUERIES];
    unsigned int reach[LIST_QUERIES];
    int heads[LIST_WAVES], count, wants;
};
// Returns the number of distinct tiles (runs of them) of the panel's `mine` queries; a barrier at the end.
__device__ inline int near_segments(const NearList& p, NearSegments& g, int base, int mine)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) g.count = 0;
    if (tid < mine) { const int i = tid; g.lo[i] = 0x7fffffff; g.hi[i] = -1; g.reach[i] = 0u; }
    auto pos_of = [&](int i) -> int { return p.pos ? p.pos[p.q0 + base + i] : p.q0 + base + i; };
    const int at_pos = tid < mine ? pos_of(tid) : -1;
    const bool head = tid < mine && (tid == 0 || (pos_of(tid - 1) >> 7) != (at_pos >> 7));
    const unsigned long long heads = __ballot(head);
    if (lane == 0) g.heads[wave] = __popcll(heads);
    __syncthreads();
    int nseg = 0;
    for (int w = 0; w < LIST_WAVES; ++w) nseg += g.heads[w];
    if (tid < mine) {
        int at = -1;
        for (int w = 0; w < wave; ++w) at += g.heads[w];
        at += __popcll(heads & (~0ull >> (63 - lane)));
        const int t = at_pos >> 7;
        const bool fine = at_pos >= 0 && at_pos < p.n_pos;
        if (head) { g.tile[at] = fine ? t : -1; g.reg[at] = fine ? p.region[t] : -1; }
        float reach = -1.f;
        if (!fine) {}
        else if (p.colour) {
            const int c = p.colour[at_pos];
            if ((unsigned int)c < (unsigned int)p.n_rows) {
                reach = __uint_as_float(p.threshold[c]);
                atomicMin(&g.lo[at], c); atomicMax(&g.hi[at], c);
            }
        } else reach = p.reach[base + tid];
        // (what a bound on a table entry's rounding can hide; 0 is left for a tile none of whose queries needs anything)
        if (reach >= 0.f) atomicMax(&g.reach[at], __float_as_uint(fmaxf(reach * (1.f + 1e-5f), 1e-37f)));
    }
    __syncthreads();
    return nseg;
}

__global__ void __launch_bounds__(LIST_THREADS) near_list_kernel(NearList p)
{
    __shared__ NearSegments g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int panel = blockIdx.x;
    int nq = p.nq;
    if (p.n_dev) { const int n = *p.n_dev - p.q0; nq = n < nq ? n : nq; }
    const int base = panel * p.panel_queries;
    if (base >= nq) {
        if (tid == 0 && gridDim.y == 1) { p.list_len[panel] = 0; if (p.list_step) p.list_step[panel] = 0; }
        return;
    }
    const int mine = nq - base < p.panel_queries ? nq - base : p.panel_queries;
    const int nseg = near_segments(p, g, base, mine);
    if (p.what == LIST_LOCAL) {
        bool any = false;
        for (int seg = 0; seg < nseg; ++seg) any = any || g.reg[seg] >= 0;
        if (!any) {
            if (tid == 0 && gridDim.y == 1) { p.list_len[panel] = 0; if (p.list_step) p.list_step[panel] = 0; }
            return;
        }
    }
    unsigned short* list = p.list + (size_t)panel * p.list_stride;
    const unsigned short* from = p.from ? p.from + (size_t)panel * p.list_stride : nullptr;
    const int n = from ? p.from_len[panel] : p.T;
    auto needs = [&](int seg, int t, int tc, int tr) -> bool {
        const unsigned int r = g.reach[seg];
        const int st = g.tile[seg], sr = g.reg[seg];
        if (r == 0u || st < 0 || (tc >= 0 && g.lo[seg] == tc && g.hi[seg] == tc)) return false;
        if ((sr >= 0 && sr == tr) != (p.what == LIST_LOCAL)) return false;
        return p.gap[(size_t)st * p.T + t] <= __uint_as_float(r);      // (NaN: no)
    };
    // (panels of few queries per tile have many tiles: several workgroups share the candidates of one, see gridDim.y)
    const bool shared = gridDim.y > 1;
    int32_t* counter = shared ? p.list_len + panel : &g.count;
    // (two strips of 64 tiles and four of the panel's own at a time, their eight table entries read side by side whether they decide or not,
    // where any of them may)
    auto scan = [&]() {
        for (int i0 = (blockIdx.y * LIST_WAVES + wave) * 128; i0 < n; i0 += 2 * LIST_THREADS * gridDim.y) {
            int t[2], tc[2], tr[2];
            bool fine[2], keep[2] = {false, false};
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int i = i0 + 64 * u + lane;
                t[u] = i < n ? (from ? (int)from[i] : i) : -1;
                fine[u] = t[u] >= 0 && t[u] < p.T;
                if (!fine[u]) t[u] = 0;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) { tc[u] = p.colour ? p.tile_colour[t[u]] : -1; tr[u] = p.region[t[u]]; }
            for (int s0 = 0; s0 < nseg && __any((fine[0] && !keep[0]) || (fine[1] && !keep[1])); s0 += 4) {
                bool may[2][4], any = false;
                unsigned int row[4];
                float r[4], gap[2][4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int seg = s0 + e < nseg ? s0 + e : nseg - 1;
                    const int st = __builtin_amdgcn_readfirstlane(g.tile[seg]), sr = __builtin_amdgcn_readfirstlane(g.reg[seg]);
                    const int lo = __builtin_amdgcn_readfirstlane(g.lo[seg]), hi = __builtin_amdgcn_readfirstlane(g.hi[seg]);
                    const unsigned int reach = (unsigned int)__builtin_amdgcn_readfirstlane((int)g.reach[seg]);
                    r[e] = __uint_as_float(reach);
                    row[e] = (unsigned int)(st < 0 ? 0 : st);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        may[u][e] = fine[u] && reach != 0u && st >= 0 && !(tc[u] >= 0 && lo == tc[u] && hi == tc[u]) &&
                                    (sr >= 0 && sr == tr[u]) == (p.what == LIST_LOCAL);
                        any = any || may[u][e];
                    }
                }
                if (!__any(any)) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int u = 0; u < 2; ++u) gap[u][e] = p.gap[(size_t)row[e] * p.T + t[u]];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int u = 0; u < 2; ++u) keep[u] = keep[u] || (may[u][e] && gap[u][e] <= r[e]);      // (NaN: no)
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const unsigned long long m = __ballot(keep[u]);
                int at = 0;
                if (lane == 0 && m) at = atomicAdd(counter, __popcll(m));
                at = __shfl(at, 0);
                if (keep[u]) list[at + __popcll(m & (lane ? ~0ull >> (64 - lane) : 0ull))] = (unsigned short)t[u];
            }
        }
        __syncthreads();
    };
    scan();
    if (p.most > 0 && g.count > p.most) {
        // which of the panel's tiles want that many (there are few such tiles: rows with fewer near rows than they ask for)
        for (int seg = 0; seg < nseg; ++seg) {
            __syncthreads();
            if (tid == 0) g.wants = 0;
            __syncthreads();
            int wants = 0;
            for (int t = tid; t < p.T; t += LIST_THREADS) wants += needs(seg, t, p.colour ? p.tile_colour[t] : -1, p.region[t]) ? 1 : 0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) wants += __shfl_xor(wants, o);
            if (lane == 0 && wants) atomicAdd(&g.wants, wants);
            __syncthreads();
            if (tid == 0 && g.wants > p.most) {
                g.reach[seg] = 0u;
                const int st = g.tile[seg];
                if (atomicExch(p.todo_mark + st, 1) == 0) p.todo[2 + atomicAdd(p.todo, 1)] = st;
            }
        }
        __syncthreads();
        if (tid == 0) g.count = 0;
        __syncthreads();
        for (int i = tid; i < mine; i += LIST_THREADS) {
            const int t = (p.q0 + base + i) >> 7;               // (queries in order)
            for (int seg = 0; seg < nseg; ++seg)
                if (g.tile[seg] == t && g.reach[seg] == 0u) p.reach[base + i] = -1.f;
        }
        scan();
    }
    if (tid == 0 && !shared) {
        const int count = g.count;
        p.list_len[panel] = count;
        if (p.list_step) {
            // as in near_plan: sample one tile in `step`, step^2 = pass over all / entries per step; at least 16 tiles.  A list
            // not much longer than the window has nothing to gain.
            int step = (int)(__builtin_sqrt((double)count * p.cost / p.kk) + 0.5);
            if (step > count / 16) step = count / 16;
            if (step > 5) step = 5;
            p.list_step[panel] = count < 24 ? 0 : (step < 1 ? 1 : step);
        }
        if (p.tile_steps && count) atomicAdd(p.tile_steps, (unsigned long long)((mine + TILE - 1) / TILE) * count);
    }
}

// Some of the nearest tiles with rows of other colours, for a first edge out of every component: of up to eight of the panel's
// tiles, the nearest in each of four interleaved quarters of all tiles.
constexpr int FIRST_TILES = 32;
static int near_list_stride(int T) { return T > FIRST_TILES ? T : FIRST_TILES; }
__global__ void __launch_bounds__(LIST_THREADS) near_first_kernel(NearList p)
{
    __shared__ NearSegments g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int panel = blockIdx.x, base = panel * p.panel_queries;
    const int mine = p.nq - base < p.panel_queries ? p.nq - base : p.panel_queries;
    if (mine <= 0) { if (tid == 0) p.list_len[panel] = 0; return; }
    const int nseg = near_segments(p, g, base, mine);
    unsigned short* list = p.list + (size_t)panel * p.list_stride;
    const int picks = nseg < 8 ? nseg : 8;
    for (int i = wave >> 2; i < picks; i += LIST_WAVES / 4) {                  // (four wavefronts to a tile, a quarter each)
        const int s = (int)((long long)i * nseg / picks);
        const int st = g.tile[s];
        unsigned long long best = ~0ull;
        if (st >= 0) {
            const float* gaps = p.gap + (size_t)st * p.T;
            const int colour = g.lo[s] == g.hi[s] ? g.lo[s] : -2;
#pragma unroll 4
            for (int t = tid & 255; t < p.T; t += 256) {                                  // (both read whether they decide or not)
                const int tc = p.tile_colour[t];
                const float gap = gaps[t];
                const unsigned int off = (unsigned int)(t > st ? t - st : st - t);
                const unsigned long long key = ((unsigned long long)__float_as_uint(gap) << 32) | (off << 16) | (unsigned int)t;
                if (gap >= 0.f && !(tc >= 0 && tc == colour)) best = key < best ? key : best;
            }
        }
        best = wave_min(best);
        if (lane == 0 && best != ~0ull) list[atomicAdd(&g.count, 1)] = (unsigned short)(best & 0xffffu);
    }
    __syncthreads();
    if (tid == 0) p.list_len[panel] = g.count;
}

// The tiles around each of a panel's own ones: what the first bounds come from.
__global__ void __launch_bounds__(64) near_window_kernel(int tile0, int panel_tiles, int last_tile, int T, int around, unsigned short* __restrict__ list,
                                                         int32_t* __restrict__ list_len, int list_stride, int panels)
{
    const int panel = blockIdx.x * 64 + threadIdx.x;
    if (panel >= panels) return;
    const int a = tile0 + panel * panel_tiles, e = a + panel_tiles < last_tile ? a + panel_tiles : last_tile;
    int lo = a - around, hi = e + around;
    lo = lo < 0 ? 0 : lo;
    hi = hi > T ? T : hi;
    for (int t = lo; t < hi; ++t) list[(size_t)panel * list_stride + (t - lo)] = (unsigned short)t;
    list_len[panel] = hi - lo;
}

// items[i]: items of the panels before i; tile_steps (optional): tiles multiplied, by the panels' query tiles.
__global__ void __launch_bounds__(1024) near_items_kernel(const int32_t* __restrict__ len, int panels, int32_t* __restrict__ items,
                                                          int panel_queries, int nq, unsigned long long* __restrict__ tile_steps)
{
    __shared__ int sum[1024];
    const int tid = threadIdx.x, per = (panels + 1023) / 1024;
    const int a = tid * per < panels ? tid * per : panels, e = a + per < panels ? a + per : panels;
    int c = 0;
    unsigned long long steps = 0;
    for (int i = a; i < e; ++i) {
        c += (len[i] + ITEM_TILES - 1) / ITEM_TILES;
        const int q = nq - i * panel_queries < panel_queries ? nq - i * panel_queries : panel_queries;
        steps += (unsigned long long)((q + TILE - 1) / TILE) * len[i];
    }
    sum[tid] = c;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int v = tid >= o ? sum[tid - o] : 0;
        __syncthreads();
        sum[tid] += v;
        __syncthreads();
    }
    int at = sum[tid] - c;
    for (int i = a; i < e; ++i) { items[i] = at; at += (len[i] + ITEM_TILES - 1) / ITEM_TILES; }
    if (tid == 1023) items[panels] = sum[1023];
    if (tile_steps && steps) atomicAdd(tile_steps, steps);
}

// The scale of the copy by regions: the median tile's radius near 2^7 (see near_shift_kernel).
__global__ void __launch_bounds__(64) near_local_scale_kernel(const float* __restrict__ tile_r, const int32_t* __restrict__ region, int T, NearScale* __restrict__ sc,
                                                              const NearScale* __restrict__ sc_all, const float* __restrict__ negh, int rows,
                                                              const float* __restrict__ hn, const int32_t* __restrict__ perm, float* __restrict__ ratio)
{
    // the 64 lanes' shares of the tiles, one local tile of each
    const int lane = threadIdx.x;
    float r = -1.f;
    for (int t = (int)((long long)lane * T / 64); t < (int)((long long)(lane + 1) * T / 64) && !(r > 0.f); ++t)
        if (region[t] >= 0) r = tile_r[t];
    // squared norms of a sample of rows as they are, over those relative to the common shift
    float as_is = 0.f, shifted = 0.f;
    for (int j = 0; j < 16; ++j) {
        const int at = (int)((long long)(lane * 16 + j) * rows / 1024);
        const float x = perm[at] >= 0 ? hn[perm[at]] : 0.f, y = -negh[at];
        if (x < INF && y < INF) { as_is += x; shifted += y / sc_all->scale / sc_all->scale; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { as_is += __shfl_xor(as_is, o); shifted += __shfl_xor(shifted, o); }
    if (lane == 0) ratio[1] = as_is / fmaxf(shifted, 1e-30f);
    const float m = near_median64(r, r > 0.f && r < INF, lane);
    if (lane == 0) {
        int e = 0;
        if (m > 0.f && m < INF) (void)frexpf(m, &e);
        int up = 7 - e;
        up = up < -100 ? -100 : (up > 100 ? 100 : up);
        sc->scale = ldexpf(1.f, up);
        ratio[0] = sc->scale / sc_all->scale;
        sc->eps_bits = 0u;
        sc->huge = 0u;
    }
}

hipError_t near_make_ordered(const float* X, int n_src, int d, const NearOrder& o, const float* tile_c, const float* tile_r,
                             const int32_t* tile_first, const float* hn, const NearBuffers& b, hipStream_t s)
{
    hipError_t e = near_make(X, n_src, d, o.perm, o.rows, nullptr, b, o.all, nullptr, nullptr, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(near_local_scale_kernel, dim3(1), dim3(64), 0, s, tile_r, o.region, o.tiles, o.local_scale, b.scale, o.all.negh, o.rows, hn, o.perm, o.ratios);
    NearBuffers bl = b;
    bl.scale = o.local_scale;
    bl.shift = const_cast<float*>(tile_c);
    bl.partial = nullptr;                            // (its words belong to the other copies' scale)
    return near_make(X, n_src, d, o.perm, o.rows, nullptr, bl, o.local, nullptr, nullptr, s, false, nullptr, tile_first);
}

// Tiles of other regions that a tile meets at most.  Rows with fewer rows of their own cluster than neighbours asked for reach
// through a cluster's worth of them, with bounds that one pass cannot tighten; their tiles (a handful) are left to the list
// kernels, which look outwards from the nearest.  1M x 128: with 256 instead, one workgroup each keeps nine launches for 3.5 ms.
constexpr int CROSS_MOST = 64;
struct NearOrderedPlan { int waves, panel_tiles, window, nseg, nsub, capl, max_seg, max_parts, sets; size_t per_tile; };
constexpr int ORDERED_AROUND = 2;          // tiles before and after a panel's own
static NearOrderedPlan near_ordered_plan(int T, int kk)
{
    NearOrderedPlan p{};
    // workgroups of eight wavefronts share what they stage among 512 queries; smaller ones where there are too few panels
    p.waves = T >= 1024 ? 8 : (T >= 256 ? 4 : 2);
    p.panel_tiles = p.waves / 2;
    p.window = p.panel_tiles + 2 * ORDERED_AROUND;
    p.nseg = 4;                            // (panels differ in their lists: four shares of each even that out)
    p.nsub = 2 * p.nseg;
    p.capl = 128;
    p.max_seg = 4;
    p.max_parts = (6 * kk + GROUPS * p.max_seg - 1) / (GROUPS * p.max_seg);
    if (p.max_parts > 4) p.max_parts = 4;
    p.sets = p.window > p.max_seg * p.max_parts ? p.window : p.max_seg * p.max_parts;
    p.per_tile = (size_t)TILE * (8 + (size_t)p.sets * GROUPS * 4 + (size_t)p.nsub * (4 + 8 * (size_t)p.capl)) + 3 * ((size_t)T * 2 + 1024) / (size_t)p.panel_tiles + 64;
    return p;
}

size_t near_ordered_batch_bytes(long long rows, int kk)
{
    const int T = near_tiles(rows);
    const NearOrderedPlan p = near_ordered_plan(T, kk);
    const int most = T < 1024 ? T : 1024;
    return p.per_tile * (size_t)(most < p.panel_tiles ? p.panel_tiles : most) + 16384;
}

size_t near_least_ordered_batch_bytes(long long rows, int kk)
{
    const NearOrderedPlan p = near_ordered_plan(near_tiles(rows), kk);
    return p.per_tile * (size_t)p.panel_tiles + 16384;
}

static bool near_order_ok(const NearOrder& o, int d)
{
    return o.gap && o.perm && o.region && o.all.in_order && o.local.in_order && o.all.tiles == o.tiles && o.local.tiles == o.tiles &&
           o.tiles >= 1 && o.tiles <= 65535 && o.rows <= o.tiles * TILE && near_steps(d) <= REG_STEPS;
}

// one side of a sweep over lists
static void near_side(NearSweep& p, const NearOrder& o, const NearBuffers& b, int side, const unsigned short* list, const int32_t* len,
                      const int32_t* step, bool best)
{
    const NearCopy& c = side == 1 ? o.local : o.all;
    p.qfrag = p.cfrag = c.frag;
    p.qnegh = c.negh; p.cnegh = best ? c.negh_best : c.negh;
    p.sc = side == 1 ? o.local_scale : b.scale;
    p.region = o.region; p.side = side; p.mark = side == 1 ? 0u : MARK;
    p.list = list; p.list_len = len; p.list_step = step; p.list_stride = near_list_stride(o.tiles);
}

// k-NN.  What bounds it: the products of the pairs of tiles on the lists (about 1.3 PFLOP/s) and the exact evaluation of what is
// emitted.  Bounds come from the tiles around a panel first; the tiles within them are listed and, where these are many, every
// few of them tighten the bounds before the rest is multiplied.  The copy by regions keeps a cluster's distance from the
// other clusters out of the rounding: without it, 1M x 128 (k = 32) passes several times as many candidates and a third of the
// panels overflow.  1M x 128: 68 ms with the list kernels, 32 ms; 100k x 64: 2.1 -> 0.8 ms.
hipError_t near_search_ordered(const NearProblem& a, const NearOrder& o, const NearBuffers& b, hipStream_t s)
{
    const int kk = a.k + 1, T = o.tiles;
    const NearOrderedPlan plan = near_ordered_plan(T, kk);
    if (!near_order_ok(o, a.d) || T > b.todo_panels || b.batch_bytes < 16384) return hipErrorInvalidValue;
    long long bt = (long long)((b.batch_bytes - 16384) / plan.per_tile) / plan.panel_tiles * plan.panel_tiles;
    if (bt < 1) return hipErrorInvalidValue;
    if (bt > 1024) bt = 1024;              // (byte offsets of 32 bits into the entries)
    if (bt > T) bt = T;
    NearSweep p{};
    p.c_tiles = T;
    p.d = a.d; p.steps = near_steps(a.d); p.e = near_e(p.steps); p.nu = near_nu(p.steps);
    p.kk = kk; p.stride = 1; p.used = T;
    NearSelect sel{};
    sel.qnegh = o.all.negh; sel.sc = b.scale; sel.e = p.e; sel.nu = p.nu; sel.steps = p.steps;
    sel.region = o.region; sel.negh_local = o.local.negh; sel.sc_local = o.local_scale;
    sel.Xq = sel.Xc = a.Xq; sel.ids = sel.c_ids = o.perm; sel.n_ids = o.rows;
    sel.d = a.d; sel.k = a.k; sel.kk = kk; sel.nq = o.rows; sel.nq_rows = sel.nc = a.nc;
    sel.q_tiles = sel.c_tiles = T; sel.q_in_order = sel.c_in_order = 1; sel.exclude_self = 1;
    sel.out_idx = a.out_idx; sel.out_dist = a.out_dist; sel.evaluated = a.evaluated;
    sel.todo = b.todo; sel.todo_mark = b.todo_mark;
    const bool vec4 = a.d % 4 == 0 && (reinterpret_cast<uintptr_t>(a.Xq) & 15) == 0;
    for (int t0 = 0; t0 < T; t0 += (int)bt) {
        const int t1 = t0 + bt < T ? t0 + (int)bt : T;
        const int nqb = (t1 - t0) * TILE, panels = (t1 - t0 + plan.panel_tiles - 1) / plan.panel_tiles;
        const dim3 per_query((unsigned)((nqb + 3) / 4)), per_panel((unsigned)panels);
        unsigned char* at = b.batch;
        auto take = [&](size_t bytes) { unsigned char* r = at; at += (bytes + 255) / 256 * 256; return r; };
        float* bound = reinterpret_cast<float*>(take((size_t)nqb * 4));
        float* reach = reinterpret_cast<float*>(take((size_t)nqb * 4));
        float* maxima = reinterpret_cast<float*>(take((size_t)nqb * plan.sets * GROUPS * 4));
        int32_t* counts = reinterpret_cast<int32_t*>(take((size_t)nqb * plan.nsub * 4));
        uint2* entries = reinterpret_cast<uint2*>(take((size_t)nqb * plan.nsub * plan.capl * 8));
        unsigned short* list[3];
        int32_t *len[3], *step[2];
        for (int i = 0; i < 3; ++i) list[i] = reinterpret_cast<unsigned short*>(take((size_t)panels * near_list_stride(T) * 2));
        for (int i = 0; i < 3; ++i) len[i] = reinterpret_cast<int32_t*>(take((size_t)panels * 4));
        for (int i = 0; i < 2; ++i) step[i] = reinterpret_cast<int32_t*>(take((size_t)panels * 4));
        p.q_tile0 = t0; p.q_tile1 = t1; p.nq_batch = nqb;
        p.maxima = maxima; p.groups = GROUPS; p.capl = plan.capl; p.append = 0;
        sel.nq_batch = nqb; sel.q0 = t0 * TILE;
        auto bounds = [&](int sets, const int32_t* steps_of) {
            hipLaunchKernelGGL((near_bounds_kernel<false>), per_query, dim3(256), 0, s, maxima, sets, 5, nqb, t0 * TILE, kk, o.all.negh, b.scale, p.e, p.nu,
                               p.steps, a.d, bound, reach, steps_of, plan.panel_tiles * TILE, o.region, o.local.negh, o.local_scale, static_cast<int32_t*>(nullptr), static_cast<int32_t*>(nullptr),
                           static_cast<int32_t*>(nullptr));
        };
        NearList l{};
        l.gap = o.gap; l.T = T; l.region = o.region; l.reach = reach; l.n_pos = T * TILE; l.q0 = t0 * TILE; l.nq = nqb;
        l.panel_queries = plan.panel_tiles * TILE;
        l.list_stride = near_list_stride(T); l.kk = kk;
        l.cost = 16.0 * p.steps * 1.28e-5 * TILE;
        auto make_list = [&](int what, int from, int to, int32_t* step_to) {
            l.what = what; l.from = from >= 0 ? list[from] : nullptr; l.from_len = from >= 0 ? len[from] : nullptr;
            l.list = list[to]; l.list_len = len[to]; l.list_step = step_to;
            hipLaunchKernelGGL(near_list_kernel, per_panel, dim3(LIST_THREADS), 0, s, l);
        };
        hipError_t e = hipSuccess;
        // 1. the tiles around every panel: first bounds (of each query in the copy that holds its region, or in the other)
        hipLaunchKernelGGL(near_window_kernel, dim3((unsigned)((panels + 63) / 64)), dim3(64), 0, s, t0, plan.panel_tiles, t1, T, ORDERED_AROUND,
                           list[2], len[2], near_list_stride(T), panels);
        p.nseg = 1; p.parts = plan.window;
        for (int side = 1; side <= 2 && e == hipSuccess; ++side) {
            near_side(p, o, b, side, list[2], len[2], nullptr, false);
            e = near_launch_sweep<NEAR_MAXIMA, false, true>(p, plan.waves, s);
        }
        if (e != hipSuccess) return e;
        bounds(plan.window, nullptr);
        // 2. the tiles within them, and where these are many, better bounds from a sample of them
        make_list(LIST_LOCAL, -1, 0, step[0]);
        p.nseg = plan.max_seg; p.parts = plan.max_parts;
        near_side(p, o, b, 1, list[0], len[0], step[0], false);
        e = near_launch_sweep<NEAR_MAXIMA, false, true>(p, plan.waves, s);
        if (e != hipSuccess) return e;
        bounds(plan.max_seg * plan.max_parts, step[0]);
        // 3. emit and select
        l.tile_steps = o.tile_steps;
        make_list(LIST_LOCAL, 0, 2, nullptr);
        l.most = CROSS_MOST; l.todo = b.todo; l.todo_mark = b.todo_mark;
        make_list(LIST_CROSS, -1, 1, nullptr);
        p.reach = reach; p.counts = counts; p.entries = entries; p.nsub = plan.nsub;
        p.nseg = plan.nseg;
        near_side(p, o, b, 1, list[2], len[2], nullptr, false);
        e = near_launch_sweep<NEAR_EMIT, false, true>(p, plan.waves, s);
        if (e != hipSuccess) return e;
        p.append = 1;
        near_side(p, o, b, 2, list[1], len[1], nullptr, false);
        e = near_launch_sweep<NEAR_EMIT, false, true>(p, plan.waves, s);
        if (e != hipSuccess) return e;
        p.reach = nullptr;
        sel.entries = entries; sel.counts = counts; sel.nsub = plan.nsub; sel.capl = plan.capl;
        near_select(sel, vec4, per_query, s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------------------------- connection rounds
struct NearRange {
    unsigned long long* best_at; const float *negh, *negh_local; const NearScale *sc, *sc_local;
    const float* X; const int32_t* colour; int d;
    int n, n_rows; const int32_t* rows; const int32_t* qpos; int c_tiles, c_in_order; const int32_t* c_ids; int n_ids;
    uint32_t* threshold; const uint32_t* threshold0;
    int32_t* edge_at;
    int32_t* out_idx; float *out_dist, *out_low; int32_t* evaluated;
    int32_t *rows_left, *slot_left, *pos_left, *counts_left, *count_left; float* reach_left;
};

__global__ void __launch_bounds__(256) near_range_clear_kernel(NearRange p)
{
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= p.n) return;
    p.best_at[q] = ~0ull;
    p.edge_at[q] = -1;
    p.out_idx[q] = -1;
    p.out_dist[q] = INF;
}

// One wavefront per query: of the 16 candidates about the nearest of which is in best_at, the nearest of another colour,
// exactly.  An edge of the query's component, which lowers the component's threshold.
template <int VEC>
__global__ void __launch_bounds__(256) near_edge_kernel(NearRange p)
{
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (q >= p.n) return;
    const unsigned long long best = p.best_at[q];
    const int row = p.rows[q];
    if (p.edge_at && (best == ~0ull || p.edge_at[q] == (int)(unsigned int)best)) return;      // as before
    const bool fine_row = (unsigned int)row < (unsigned int)p.n_rows;
    const int c = fine_row ? p.colour[row] : -1;
    unsigned long long key = ~0ull;
    if (best != ~0ull && (unsigned int)c < (unsigned int)p.n_rows) {
        const int grp = lane >> 3, g = lane & 7;
        const float* xa = p.X + (size_t)row * p.d;
        v4f qa[4];
        near_first_quads<VEC>(qa, xa, p.d, g);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int j = half * 8 + grp;
            long long cand = near_row((int)(unsigned int)best + 8 * (j >> 2) + (j & 3), p.c_tiles, p.c_in_order);
            if (p.c_ids) cand = cand < p.n_ids ? (long long)p.c_ids[cand] : -1;
            const bool real = cand >= 0 && cand < p.n_rows;
            const bool fine = real && p.colour[real ? cand : 0] != c;
            const float dist = near_exact<VEC>(qa, xa, p.X + (size_t)(fine ? cand : row) * p.d, p.d, g);
            const unsigned long long k = ((unsigned long long)__float_as_uint(dist) << 32) | (unsigned int)cand;
            if (fine && dist < INF && k < key) key = k;
        }
        key = wave_min<8>(key);                                      // (eight lanes have one pair)
    }
    if (lane == 0) {
        if (p.edge_at) {
            p.edge_at[q] = (int)(unsigned int)best;
            // (an edge found earlier may be the shorter one all the same)
            if (key == ~0ull || !(__uint_as_float((unsigned int)(key >> 32)) < p.out_dist[q])) return;
        }
        p.out_idx[q] = key == ~0ull ? -1 : (int32_t)(unsigned int)key;
        p.out_dist[q] = key == ~0ull ? INF : __uint_as_float((unsigned int)(key >> 32));
        if (key != ~0ull) min_into(&p.threshold[c], (uint32_t)(key >> 32));
    }
}

// The queries whose nearest row of another colour may be as near as the threshold go on to the search.
__global__ void __launch_bounds__(256) near_split_kernel(NearRange p)
{
    const int q = blockIdx.x * 256 + threadIdx.x;
    bool left = false;
    float reach = INF;
    int row = -1, pos = 0;
    if (q < p.n) {
        pos = p.qpos ? p.qpos[q] : q;
        const float nh = p.negh[pos];
        row = p.rows[q];
        const int c = (unsigned int)row < (unsigned int)p.n_rows ? p.colour[row] : -1;
        float lower = 0.f;
        if (nh == -INF || c < 0 || c >= p.n_rows) lower = INF;          // no row
        else if (nh == INF || (p.negh_local && p.negh_local[pos] == INF)) left = true;      // (ends up with the list kernels)
        else {
            reach = __uint_as_float(p.threshold[c]);
            // nothing found: no other colour among the rows that float16 holds
            if (p.sc->huge == 0u && (!p.sc_local || p.sc_local->huge == 0u)) {
                const unsigned long long best = p.best_at[q];
                lower = best == ~0ull ? INF : __uint_as_float((unsigned int)(best >> 32));
            }
            left = lower <= reach && lower < INF;
            // (the tiles left out hold only rows beyond the threshold they were left out by, which is not below `reach`)
            if (p.threshold0) lower = fminf(lower, __uint_as_float(p.threshold0[c]));
        }
        p.out_low[q] = lower;
        if (!left && p.evaluated) p.evaluated[q] = 0;
    }
    const int at = block_append<256>(left, p.count_left);
    if (left && at < p.n) {
        p.rows_left[at] = row; p.slot_left[at] = q; p.reach_left[at] = reach;
        if (p.pos_left) { p.pos_left[at] = pos; p.counts_left[at] = 0; }
    }
}

static void near_edges(const NearRange& r, bool vec4, hipStream_t s)
{
    const dim3 grid((unsigned)((r.n + 3) / 4));
    switch (near_vec(vec4, r.d)) {
        case 2: hipLaunchKernelGGL(near_edge_kernel<2>, grid, dim3(256), 0, s, r); break;
        case 1: hipLaunchKernelGGL(near_edge_kernel<1>, grid, dim3(256), 0, s, r); break;
        default: hipLaunchKernelGGL(near_edge_kernel<0>, grid, dim3(256), 0, s, r);
    }
}

// Where most rows are queries, one pass over all pairs of rows serves both rows of each (pairs_best) and costs half of one over
// all candidates of every row; rows that ask nothing are served too.
static bool near_link_by_pairs(const NearLink& a, const NearCopy& c, const NearBuffers& b)
{
    return near_steps(a.d) > REG_STEPS && c.rows == a.n_rows && c.tiles >= 32 && 5LL * a.n >= 3LL * a.n_rows && !c.in_order &&
           b.batch_bytes >= (size_t)c.tiles * TILE * 8;
}
__global__ void __launch_bounds__(256) near_pair_best_clear_kernel(unsigned long long* __restrict__ best, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) best[i] = 0x7f800000ffffffffull;
}
// (w, position) by position of the copy of all rows -> (distance below which there is no candidate, position) by query
__global__ void __launch_bounds__(256) near_pair_best_kernel(const unsigned long long* __restrict__ best, const int32_t* __restrict__ rows, int n, int n_rows,
                                                             int tiles, const float* __restrict__ negh, const NearScale* __restrict__ sc, float e, float nu,
                                                             int steps, int d, unsigned long long* __restrict__ best_at)
{
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= n) return;
    const int row = rows[q];
    unsigned long long out = ~0ull;
    if ((unsigned int)row < (unsigned int)n_rows) {
        const int pos = near_pos(row, tiles);
        const unsigned long long key = best[pos];
        const float w = __uint_as_float((unsigned int)(key >> 32)), h = -negh[pos];
        if (w < INF && fabsf(h) < INF) {
            // (w = 0: the value itself was cut off)
            const NearBoundArgs a = near_args(sc, steps, d, e, nu);
            const float low = w > 0.f ? near_lower_from(h - w, h, a) / sc->scale / sc->scale : 0.f;
            out = ((unsigned long long)__float_as_uint(low) << 32) | (unsigned int)key;
        }
    }
    best_at[q] = out;
}
static hipError_t near_link_pairs(const NearLink& a, const NearCopy& q, const NearCopy& c, const NearBuffers& b, hipStream_t s)
{
    NearPairs r{};
    r.frag = c.frag; r.negh = c.negh_best; r.colour = c.colour; r.tiles = c.tiles; r.steps = near_steps(a.d); r.filled = (a.d + 15) / 16;
    r.blocks = (c.tiles + 1) / 2; r.spread = near_spread(r.blocks);
    r.best = reinterpret_cast<unsigned long long*>(b.batch);
    const int n = c.tiles * TILE, half = r.blocks / 2 + 1, cus = near_cus();
    hipLaunchKernelGGL(near_pair_best_clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, r.best, n);
    auto shares = [&](int len) { const int seg = (8 * cus + r.blocks - 1) / r.blocks; return seg < 4 ? (len < 4 ? len : 4) : (seg > len ? len : seg); };
    // every row's own block and a few more first: what they leave keeps nearly all updates of the other rows' words away
    const int first = half / 32 > 1 ? half / 32 : 1;
    r.from = 0; r.to = first; r.both = 0; r.nseg = shares(first);
    hipError_t e = pairs_best(r, s);
    if (e != hipSuccess) return e;
    if (half > 1) {
        r.from = 1; r.to = half; r.both = 1; r.nseg = shares(half - 1);
        e = pairs_best(r, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(near_pair_best_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, r.best, a.rows, a.n, a.n_rows, c.tiles, c.negh_best,
                       b.scale, near_e(r.steps), near_nu(r.steps), r.steps, a.d, q.best_at);
    return hipGetLastError();
}

// Connection rounds.  One pass over all candidates leaves per query the distance below which there is none and the 16
// candidates about the nearest.  Bound by that pass: the search that follows is left with a query or two per component (10 of
// 250 000), where every query used to go through it.  250k x 784, ten components: 346 -> 240 ms per call (a pass takes
// 99 ms); 100k x 64: 11.6 -> 9.9 ms.  Without the exact edge of every query (only an interval for its distance), a component
// had no threshold in the next round and queried all its rows again: 324 ms.
hipError_t near_link(const NearLink& a, const NearCopy& q, const NearCopy& c, const NearBuffers& b, hipStream_t s)
{
    if (!q.in_order || !q.colour || !c.colour || !q.best_at || !q.count || !c.negh_best || (a.n + 127) / 128 > b.todo_panels) return hipErrorInvalidValue;
    hipError_t e = near_make(a.X, a.n_rows, a.d, a.rows, a.n, a.colour, b, q, nullptr, nullptr, s, true);
    if (e != hipSuccess) return e;
    NearPlan plan = near_plan(a.n, c.rows, a.d, 1, b.batch_bytes);
    if (plan.batch_tiles < 1) return hipErrorInvalidValue;
    NearSweep p{};
    p.qfrag = q.frag; p.qnegh = q.negh; p.qcolour = q.colour; p.q_tile0 = 0; p.q_tile1 = q.tiles;
    p.cfrag = c.frag; p.cnegh = c.negh_best; p.ccolour = c.colour; p.c_tiles = c.tiles;
    p.sc = b.scale; p.d = a.d; p.steps = near_steps(a.d); p.e = near_e(p.steps); p.nu = near_nu(p.steps);
    p.nseg = plan.nseg; p.stride = 1; p.used = c.tiles; p.kk = 1;
    p.best_at = q.best_at;
    if (near_link_by_pairs(a, c, b)) e = near_link_pairs(a, q, c, b, s);
    else e = near_launch_sweep<NEAR_BLOCK, true>(p, plan.waves, s);
    if (e != hipSuccess) return e;
    NearRange r{};
    r.X = a.X; r.colour = a.colour; r.c_tiles = c.tiles; r.c_in_order = c.in_order; r.d = a.d;
    r.best_at = q.best_at; r.negh = q.negh; r.sc = b.scale;
    r.n = a.n; r.n_rows = a.n_rows; r.rows = a.rows; r.threshold = a.threshold;
    r.out_idx = a.out_idx; r.out_dist = a.out_dist; r.out_low = a.out_low; r.evaluated = a.evaluated;
    r.rows_left = a.rows_left; r.slot_left = a.slot_left; r.reach_left = a.reach_left; r.count_left = b.todo + 1;
    const bool vec4 = a.d % 4 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
    near_edges(r, vec4, s);
    hipLaunchKernelGGL(near_split_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, r);
    // the copy of the queries now holds those that are left
    e = near_make(a.X, a.n_rows, a.d, a.rows_left, a.n, a.colour, b, q, nullptr, nullptr, s, false, r.count_left);
    if (e != hipSuccess) return e;
    p.cnegh = c.negh;
    p.n_dev = r.count_left;
    // few are left: workgroups of two wavefronts (of one kind beyond 128 columns) waste least on a panel that is not full
    const bool wide = p.steps > REG_STEPS;
    const int waves = wide ? plan.waves : (plan.waves > 2 ? plan.waves / 2 : 2);
    p.slots = p.most_seg = (waves == 8 ? 1 : 2) * near_cus();
    p.counts = q.count; p.capl = plan.capl;
    p.reach = a.reach_left;
    NearSelect sel{};
    sel.qnegh = q.negh; sel.sc = b.scale; sel.e = p.e; sel.nu = p.nu; sel.steps = p.steps;
    sel.Xq = sel.Xc = a.X; sel.q_rows = a.rows_left; sel.slot = a.slot_left; sel.n_dev = r.count_left;
    sel.d = a.d; sel.k = sel.kk = 1; sel.nq = a.n; sel.nq_rows = sel.nc = a.n_rows;
    sel.q_tiles = q.tiles; sel.c_tiles = c.tiles; sel.q_in_order = 1; sel.c_in_order = c.in_order;
    sel.out_idx = a.out_idx; sel.out_dist = a.out_dist; sel.evaluated = a.evaluated;
    sel.todo = b.todo; sel.todo_mark = b.todo_mark;
    sel.capl = plan.capl; sel.nsub = 1; sel.by_position = 1; sel.counts = q.count;
    p.entries = reinterpret_cast<uint2*>(b.batch);
    sel.entries = p.entries;
    for (int t0 = 0; t0 < q.tiles; t0 += plan.batch_tiles) {
        p.q_tile0 = t0; p.q_tile1 = t0 + plan.batch_tiles < q.tiles ? t0 + plan.batch_tiles : q.tiles;
        const int nqb = (p.q_tile1 - t0) * TILE;
        p.nq_batch = sel.nq_batch = nqb; sel.q0 = t0 * TILE;
        e = near_launch_sweep<NEAR_NEAREST, true>(p, waves, s);
        if (e != hipSuccess) return e;
        near_select(sel, vec4, dim3((unsigned)((nqb + 3) / 4)), s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

size_t near_linked_batch_bytes(long long rows)
{
    const size_t T = (size_t)near_tiles(rows);
    return 256 * 2 * (T * 2 + 256) + (size_t)128 * 128 * 256 * 8 + 65536;
}

// The same in a row order: the queries (rows, qpos: ascending positions) meet the tiles only whose distance does not exceed their
// component's threshold, which a pass over a few of the nearest tiles of other colours sets first.  Bound by the products of
// the listed pairs (half of the time) and the exact edges.  1M x 128, five rounds of 1.3 million queries: 50 ms with the list kernels
// (128 queries share what they stage, three products), 21 ms; with lists in equal shares per panel instead of equal items 36 ms;
// 16 ms with lists walked by a thousand threads and what is read of a tile held by lanes.
hipError_t near_link_ordered(const NearLink& a, const NearOrder& o, const NearBuffers& b, hipStream_t s)
{
    const int T = o.tiles;
    if (!near_order_ok(o, a.d) || !a.qpos || T > b.todo_panels || b.batch_bytes < near_linked_batch_bytes(o.rows) || !o.all.colour || !o.tile_colour)
        return hipErrorInvalidValue;
    // panels of 512 queries share what they stage; smaller ones where there are too few of them
    const int waves = a.n >= 131072 ? 8 : 4, panel_queries = 64 * waves;
    const size_t per_panel = 2 * ((size_t)near_list_stride(T) * 2 + 64);       // two lists, their lengths and items
    long long batch_panels = (long long)((b.batch_bytes - 16384) / per_panel);
    if (batch_panels > 8192) batch_panels = 8192;
    NearSweep p{};
    p.qcolour = p.ccolour = o.all.colour; p.c_tiles = T;
    p.tile_colour = o.tile_colour;
    p.d = a.d; p.steps = near_steps(a.d); p.e = near_e(p.steps); p.nu = near_nu(p.steps);
    p.stride = 1; p.used = T; p.kk = 1;
    p.qpos = a.qpos; p.n_q = a.n; p.best_at = a.best_at;
    NearRange r{};
    r.X = a.X; r.colour = a.colour; r.c_tiles = T; r.c_in_order = 1; r.c_ids = o.perm; r.n_ids = o.rows; r.d = a.d;
    r.best_at = a.best_at; r.negh = o.all.negh; r.negh_local = o.local.negh; r.sc = b.scale; r.sc_local = o.local_scale;
    r.n = a.n; r.n_rows = a.n_rows; r.rows = a.rows; r.qpos = a.qpos; r.threshold = a.threshold;
    r.edge_at = a.edge_at;
    r.out_idx = a.out_idx; r.out_dist = a.out_dist; r.out_low = a.out_low; r.evaluated = a.evaluated;
    r.rows_left = a.rows_left; r.slot_left = a.slot_left; r.pos_left = a.pos_left; r.counts_left = a.counts_left; r.reach_left = a.reach_left;
    r.count_left = b.todo + 1;
    const bool vec4 = a.d % 4 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
    const dim3 per_row((unsigned)((a.n + 255) / 256));
    hipLaunchKernelGGL(near_range_clear_kernel, per_row, dim3(256), 0, s, r);
    hipLaunchKernelGGL(near_todo_clear_kernel, dim3(64), dim3(256), 0, s, b.todo, 2 + 2 * b.todo_panels);
    NearList l{};
    l.gap = o.gap; l.T = T; l.region = o.region; l.colour = o.all.colour; l.threshold = a.threshold; l.n_rows = a.n_rows; l.tile_colour = o.tile_colour;
    l.pos = a.qpos; l.n_pos = o.rows; l.list_stride = near_list_stride(T);
    hipError_t e = hipSuccess;
    for (int pass = 0; pass < 2; ++pass) {
        for (long long q0 = 0; q0 < a.n; q0 += batch_panels * panel_queries) {
            const int nq = (int)(a.n - q0 < batch_panels * panel_queries ? a.n - q0 : batch_panels * panel_queries);
            const int panels = (nq + panel_queries - 1) / panel_queries;
            unsigned char* at = b.batch;
            auto take = [&](size_t bytes) { unsigned char* x = at; at += (bytes + 255) / 256 * 256; return x; };
            unsigned short *list[2];
            int32_t *len[2], *items[2];
            for (int i = 0; i < 2; ++i) list[i] = reinterpret_cast<unsigned short*>(take((size_t)panels * near_list_stride(T) * 2));
            for (int i = 0; i < 2; ++i) len[i] = reinterpret_cast<int32_t*>(take((size_t)panels * 4));
            for (int i = 0; i < 2; ++i) items[i] = reinterpret_cast<int32_t*>(take((size_t)(panels + 1) * 4));
            l.q0 = (int)q0; l.nq = nq; l.panel_queries = panel_queries;
            for (int i = 0; i <= pass; ++i) {
                l.what = i ? LIST_CROSS : LIST_LOCAL; l.list = list[i]; l.list_len = len[i];
                if (pass) hipLaunchKernelGGL(near_list_kernel, dim3((unsigned)panels), dim3(LIST_THREADS), 0, s, l);
                else hipLaunchKernelGGL(near_first_kernel, dim3((unsigned)panels), dim3(LIST_THREADS), 0, s, l);
                hipLaunchKernelGGL(near_items_kernel, dim3(1), dim3(1024), 0, s, len[i], panels, items[i], panel_queries, nq,
                                   pass ? o.tile_steps : nullptr);
            }
            p.q_tile0 = (int)(q0 / TILE); p.q_tile1 = (int)((q0 + nq + TILE - 1) / TILE); p.nq_batch = nq;
            p.panels = panels; p.nseg = 1;
            for (int side = 1; side <= 2; ++side) {
                near_side(p, o, b, side, list[pass ? side - 1 : 0], len[pass ? side - 1 : 0], nullptr, true);
                p.items = items[pass ? side - 1 : 0];
                e = near_launch_sweep<NEAR_BLOCK, true, true>(p, waves, s);
                if (e != hipSuccess) return e;
            }
        }
        near_edges(r, vec4, s);
        if (!pass) {
            // the thresholds that the lists are made by
            e = hipMemcpyAsync(a.threshold0, a.threshold, (size_t)a.n_rows * 4, hipMemcpyDeviceToDevice, s);
            if (e != hipSuccess) return e;
        }
    }
    r.threshold0 = a.threshold0;
    hipLaunchKernelGGL(near_split_kernel, per_row, dim3(256), 0, s, r);
    // the few that are left
    constexpr int capl = 256, left_waves = 4, left_queries = 256, left_slices = 8;
    l.pos = a.pos_left; l.n_dev = r.count_left; l.panel_queries = left_queries;
    p.qpos = a.pos_left; p.n_dev = r.count_left;
    p.counts = a.counts_left; p.capl = capl; p.reach = a.reach_left;
    NearSelect sel{};
    sel.qnegh = o.all.negh; sel.sc = b.scale; sel.e = p.e; sel.nu = p.nu; sel.steps = p.steps;
    sel.region = o.region; sel.negh_local = o.local.negh; sel.sc_local = o.local_scale;
    sel.Xq = sel.Xc = a.X; sel.q_rows = a.rows_left; sel.slot = a.slot_left; sel.n_dev = r.count_left; sel.qpos = a.pos_left;
    sel.c_ids = o.perm; sel.n_ids = o.rows;
    sel.d = a.d; sel.k = sel.kk = 1; sel.nq = a.n; sel.nq_rows = sel.nc = a.n_rows;
    sel.q_tiles = sel.c_tiles = T; sel.q_in_order = sel.c_in_order = 1;
    sel.out_idx = a.out_idx; sel.out_dist = a.out_dist; sel.evaluated = a.evaluated;
    sel.todo = b.todo; sel.todo_mark = b.todo_mark;
    sel.capl = capl; sel.nsub = 1; sel.by_position = 1; sel.counts = a.counts_left;
    const size_t per_left = per_panel + (size_t)left_queries * capl * 8;
    long long left_panels = (long long)((b.batch_bytes - 16384) / per_left);
    if (left_panels > 8192) left_panels = 8192;
    for (long long q0 = 0; q0 < a.n; q0 += left_panels * left_queries) {
        const int nq = (int)(a.n - q0 < left_panels * left_queries ? a.n - q0 : left_panels * left_queries);
        const int panels = (nq + left_queries - 1) / left_queries;
        unsigned char* at = b.batch;
        auto take = [&](size_t bytes) { unsigned char* x = at; at += (bytes + 255) / 256 * 256; return x; };
        unsigned short *list[2];
        int32_t *len[2], *items[2];
        for (int i = 0; i < 2; ++i) list[i] = reinterpret_cast<unsigned short*>(take((size_t)panels * near_list_stride(T) * 2));
        for (int i = 0; i < 2; ++i) len[i] = reinterpret_cast<int32_t*>(take((size_t)panels * 4));
        for (int i = 0; i < 2; ++i) items[i] = reinterpret_cast<int32_t*>(take((size_t)(panels + 1) * 4));
        p.entries = reinterpret_cast<uint2*>(take((size_t)panels * left_queries * capl * 8));
        l.q0 = (int)q0; l.nq = nq;
        hipLaunchKernelGGL(near_todo_clear_kernel, dim3(8), dim3(256), 0, s, len[0], (long long)(reinterpret_cast<unsigned char*>(items[0]) - reinterpret_cast<unsigned char*>(len[0])) / 4);
        for (int i = 0; i < 2; ++i) {
            l.what = i ? LIST_CROSS : LIST_LOCAL; l.list = list[i]; l.list_len = len[i];
            hipLaunchKernelGGL(near_list_kernel, dim3((unsigned)panels, left_slices), dim3(LIST_THREADS), 0, s, l);
            hipLaunchKernelGGL(near_items_kernel, dim3(1), dim3(1024), 0, s, len[i], panels, items[i], left_queries, nq, static_cast<unsigned long long*>(nullptr));
        }
        p.panels = panels;
        p.q_tile0 = (int)(q0 / TILE); p.q_tile1 = p.q_tile0 + panels * (left_queries / TILE); p.nq_batch = nq;
        for (int side = 1; side <= 2; ++side) {
            near_side(p, o, b, side, list[side - 1], len[side - 1], nullptr, false);
            p.items = items[side - 1];
            e = near_launch_sweep<NEAR_NEAREST, true, true>(p, left_waves, s);
            if (e != hipSuccess) return e;
        }
        sel.entries = p.entries;
        sel.nq_batch = panels * left_queries; sel.q0 = (int)q0;
        near_select(sel, vec4, dim3((unsigned)((sel.nq_batch + 3) / 4)), s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------------------------- colours, assignment
__global__ void __launch_bounds__(256) near_colours_kernel(const int32_t* __restrict__ colour, int n, int tiles, int in_order, int32_t* __restrict__ out)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= tiles * TILE) return;
    const long long row = near_row(p, tiles, in_order);
    out[p] = row < n ? colour[row] : -1;
}

hipError_t near_colours(const NearCopy& c, const int32_t* colour, hipStream_t s)
{
    hipLaunchKernelGGL(near_colours_kernel, dim3((unsigned)((c.tiles + 1) / 2)), dim3(256), 0, s, colour, c.rows, c.tiles, c.in_order ? 1 : 0, c.colour);
    return hipGetLastError();
}

// (product value, position) per query position -> candidate row and exact squared distance by query; eight lanes per query
template <bool VEC4>
__global__ void __launch_bounds__(256) near_unpack_kernel(const unsigned long long* __restrict__ best_at, const float* __restrict__ qnegh,
                                                          const float* __restrict__ Xq, const int32_t* __restrict__ q_rows, int nq,
                                                          int q_tiles, const float* __restrict__ Xc, int nc, int c_tiles, int d,
                                                          int32_t* __restrict__ out_idx, float* __restrict__ out_dist)
{
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    const int p = (int)(t >> 3), g = (int)(t & 7);
    if (p >= q_tiles * TILE) return;
    const long long qi = near_row(p, q_tiles, 0);
    if (qi >= nq) return;
    const unsigned long long key = best_at[p];
    const int pos = (int)(unsigned int)key;
    const long long cand = near_row(pos, c_tiles, 0);
    const bool fine = key != 0ull && cand < nc && fabsf(qnegh[p]) < 1e37f;
    float s = 0.f;
    if (fine) {
        const float* a = Xq + (size_t)(q_rows ? q_rows[qi] : qi) * d;
        const float* b = Xc + (size_t)cand * d;
        for (int c = 4 * g; c < d; c += 32) s = near_quad_sqdist(near_quad<VEC4 ? 2 : 0>(a, c, d), near_quad<VEC4 ? 2 : 0>(b, c, d), s);
    }
    s = lanes_add8(s);
    if (g == 0) {
        out_idx[qi] = fine ? (int32_t)cand : 0;
        out_dist[qi] = fine ? s : INF;
    }
}

hipError_t near_assign(const NearCopy& q, const NearCopy& c, const float* Xq, const int32_t* q_rows, const float* Xc, int d,
                       const NearBuffers& b, unsigned long long* best_at, int32_t* out_idx, float* out_dist, hipStream_t s)
{
    if (!c.finite_padding || !c.negh_best) return hipErrorInvalidValue;
    NearPlan plan = near_plan(q.rows, c.rows, d, 1, (size_t)1 << 62);
    NearSweep p{};
    p.qfrag = q.frag; p.qnegh = q.negh; p.q_tile0 = 0; p.q_tile1 = q.tiles;
    // (without values beyond float16: their +inf would hide every other candidate of its lane)
    p.cfrag = c.frag; p.cnegh = c.negh_best; p.c_tiles = c.tiles;
    p.sc = b.scale; p.d = d; p.steps = near_steps(d); p.e = near_e(p.steps); p.nu = near_nu(p.steps);
    p.nseg = plan.nseg; p.stride = 1; p.used = c.tiles; p.kk = 1;
    p.best_at = best_at;
    const long long words = (long long)q.tiles * TILE;
    hipLaunchKernelGGL(near_clear_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, best_at, words);
    hipError_t e = near_launch_sweep<NEAR_ARG, false>(p, plan.waves, s);
    if (e != hipSuccess) return e;
    const bool vec4 = d % 4 == 0 && ((reinterpret_cast<uintptr_t>(Xq) | reinterpret_cast<uintptr_t>(Xc)) & 15) == 0;
    const dim3 grid((unsigned)(q.tiles * (TILE * 8 / 256)));
    if (vec4) hipLaunchKernelGGL((near_unpack_kernel<true>), grid, dim3(256), 0, s, best_at, q.negh, Xq, q_rows, q.rows, q.tiles, Xc, c.rows, c.tiles, d, out_idx, out_dist);
    else hipLaunchKernelGGL((near_unpack_kernel<false>), grid, dim3(256), 0, s, best_at, q.negh, Xq, q_rows, q.rows, q.tiles, Xc, c.rows, c.tiles, d, out_idx, out_dist);
    return hipGetLastError();
}

}  // namespace slhc
