// Small 1-NN searches: every pair is evaluated exactly, by the vector units.
//
// The half-precision engine (near_kernels.hip) takes nine launches of 4 us and more each, which for a million pairs is more than all
// of them cost: a pair is 2 d operations, a wavefront evaluates 64 at a time, one candidate per lane.  The candidates of a
// workgroup pass through LDS, 16 bytes of every row side by side (no bank is met twice); the queries' values are the same for
// all lanes.  Every distance is the float32 sum of the list kernels in their order of additions (group8_sqdist): slabs of 64
// features, sixteen chains of four features each, the chains of either half added in a tree.  Bound by its three launches
// and one round trip to memory per 64 candidates.  439 x 2414 x 16: 42 -> 17 us.  (The same for k-NN graphs, all distances of
// eight rows in LDS, lost: 2048 x 32, k = 8, 65 us against the engine's 47.)
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "direct_kernels.h"
#include "wave_ops.h"

namespace slhc {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_word __attribute__((ext_vector_type(4), aligned(4)));      // global loads of 16 bytes need the alignment of a word only
constexpr float INF = __builtin_inff();
constexpr int WAVES = 4;                   // per workgroup
constexpr int SLAB = 64;                   // features of a row in LDS at a time
constexpr int QUADS = SLAB / 4;

// Four features of row `row` from feature t on; zeros beyond d or without a row.
__device__ inline v4f direct_quad(const float* __restrict__ X, long long row, int t, int d, bool vec4)
{
    v4f v = {0.f, 0.f, 0.f, 0.f};
    if (row < 0 || t >= d) return v;
    const float* x = X + (size_t)row * d + t;
    if (vec4) return *reinterpret_cast<const v4f*>(x);
    if (t + 4 <= d) return *reinterpret_cast<const v4f_word*>(x);
#pragma unroll
    for (int e = 0; e < 3; ++e)
        if (t + e < d) v[e] = x[e];
    return v;
}

// acc[q]: sixteen chains per query; adds the slab that begins at feature c0, candidate per lane from `tile`, queries from `qs`.
template <int QW>
__device__ inline void direct_slab(float (&acc)[QW][QUADS], const v4f* tile, const v4f* qs, int nquads, int lane)
{
#pragma unroll
    for (int j = 0; j < QUADS; ++j) {
        if (j >= nquads) break;
        const v4f b = tile[j * 64 + lane];
#pragma unroll
        for (int q = 0; q < QW; ++q) {
            const v4f a = qs[q * QUADS + j];
#pragma unroll
            for (int e = 0; e < 4; ++e) { const float x = a[e] - b[e]; acc[q][j] = __builtin_fmaf(x, x, acc[q][j]); }
        }
    }
}
template <int QW>
__device__ inline float direct_sum(const float (&acc)[QW][QUADS], int q)
{
    const auto& p = acc[q];
    const float s0 = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    const float s1 = ((p[8] + p[9]) + (p[10] + p[11])) + ((p[12] + p[13]) + (p[14] + p[15]));
    return s0 + s1;
}

// A row whose squared norm is not a finite float32 is nobody's neighbour.  Its distance to a row of moderate norm is not finite or
// close to the largest float32, so only such distances need the look.
__device__ __attribute__((noinline)) bool direct_bad_row(const float* __restrict__ X, long long row, int d)
{
    float s = 0.f;
    for (int t = 0; t < d; ++t) { const float v = X[(size_t)row * d + t]; s = __builtin_fmaf(v, v, s); }
    return !(s < INF);
}

// One wavefront's QW queries against the candidates c_begin .. c_end - 1, 64 at a time: visit(q, candidate, distance), distance
// +inf where the candidate does not count.  All wavefronts of the workgroup go through it together.
struct DirectRows { const float* Xq; const float* Xc; int d; bool vec4; };
template <int QW, typename V>
__device__ inline void direct_pass(const DirectRows& x, const long long (&row)[QW], const float (&norm)[QW], int c_begin, int c_end, v4f* tile, v4f* qs, V&& visit)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slabs = (x.d + SLAB - 1) / SLAB;
    v4f* mine = qs + wave * QW * QUADS;
    auto queries = [&](int c0) {
        for (int i = lane; i < QW * QUADS; i += 64) {
            long long r = -1;
#pragma unroll
            for (int q = 0; q < QW; ++q) r = i / QUADS == q ? row[q] : r;
            mine[i] = direct_quad(x.Xq, r, c0 + 4 * (i % QUADS), x.d, x.vec4);
        }
    };
    if (slabs == 1) queries(0);
    for (int c = c_begin; c < c_end; c += 64) {
        float acc[QW][QUADS];
#pragma unroll
        for (int q = 0; q < QW; ++q)
#pragma unroll
            for (int j = 0; j < QUADS; ++j) acc[q][j] = 0.f;
        for (int slab = 0; slab < slabs; ++slab) {
            const int c0 = slab * SLAB;
            const int nquads = (x.d - c0 + 3) / 4 < QUADS ? (x.d - c0 + 3) / 4 : QUADS;
            __syncthreads();                        // the tile of the step before is used up
            for (int i = tid; i < 64 * nquads; i += 64 * WAVES) {
                // consecutive lanes read consecutive pieces of a row
                const int r = i / nquads, j = i - r * nquads;
                tile[j * 64 + r] = direct_quad(x.Xc, c + r < c_end ? c + r : -1, c0 + 4 * j, x.d, x.vec4);
            }
            if (slabs > 1) queries(c0);
            __syncthreads();
            direct_slab<QW>(acc, tile, mine, nquads, lane);
        }
        const int cand = c + lane;
#pragma unroll
        for (int q = 0; q < QW; ++q) {
            float dist = direct_sum<QW>(acc, q);
            const bool suspect = cand < c_end && row[q] >= 0 && dist < INF && !(dist < 2e38f && norm[q] < 1e36f);
            if (__any(suspect)) {
                if (suspect && direct_bad_row(x.Xc, cand, x.d)) dist = INF;
            }
            visit(q, cand, cand < c_end && dist < INF ? dist : INF);          // (NaN: +inf)
        }
    }
}

// the squared norm of a row, by a wavefront
__device__ inline float direct_norm(const float* __restrict__ X, long long row, int d, int lane)
{
    float s = 0.f;
    if (row >= 0)
        for (int t = lane; t < d; t += 64) { const float v = X[(size_t)row * d + t]; s = __builtin_fmaf(v, v, s); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    return s;
}

struct Direct1nn {
    const float* Xq; const float* Xc; const int32_t* q_rows; const int32_t* colour;
    int m, nq_rows, nc, d, segments, per_segment; bool vec4;
    int32_t* out_idx; float* out_dist; unsigned long long* keys;
};
constexpr int QW1 = 2;                     // queries per wavefront

__global__ void __launch_bounds__(64 * WAVES) direct_1nn_kernel(Direct1nn p)
{
    __shared__ v4f tile[QUADS * 64];
    __shared__ v4f qs[WAVES * QW1 * QUADS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int panel = blockIdx.x / p.segments, seg = blockIdx.x - panel * p.segments;
    long long row[QW1];
    float norm[QW1];
    int colour[QW1];
#pragma unroll
    for (int q = 0; q < QW1; ++q) {
        const int i = (panel * WAVES + wave) * QW1 + q;
        row[q] = i < p.m ? (p.q_rows ? (long long)p.q_rows[i] : i) : -1;
        if (row[q] >= p.nq_rows) row[q] = -1;
        norm[q] = direct_norm(p.Xq, row[q], p.d, lane);
        colour[q] = p.colour && row[q] >= 0 ? p.colour[row[q]] : 0;
    }
    float best[QW1];
    int at[QW1];
#pragma unroll
    for (int q = 0; q < QW1; ++q) { best[q] = INF; at[q] = -1; }
    const int c0 = seg * p.per_segment, c1 = c0 + p.per_segment < p.nc ? c0 + p.per_segment : p.nc;
    const DirectRows x{p.Xq, p.Xc, p.d, p.vec4};
    int cand_colour = 0, cand_of = -1;
    direct_pass<QW1>(x, row, norm, c0, c1, tile, qs, [&](int q, int cand, float v) {
        if (p.colour) {
            if (cand_of != cand) { cand_colour = cand < c1 ? p.colour[cand] : 0; cand_of = cand; }
            if (cand_colour == colour[q]) v = INF;
        }
        if (v < best[q]) { best[q] = v; at[q] = cand; }              // (ascending candidates: the smallest index of equals)
    });
#pragma unroll
    for (int q = 0; q < QW1; ++q) {
        const int i = (panel * WAVES + wave) * QW1 + q;
        unsigned long long key = at[q] >= 0 && row[q] >= 0 && norm[q] < INF ? ((unsigned long long)__float_as_uint(best[q]) << 32) | (unsigned int)at[q] : ~0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long other = __shfl_xor(key, o);
            key = other < key ? other : key;
        }
        if (lane == 0 && i < p.m) {
            if (p.segments > 1) { if (key != ~0ull) atomicMin(p.keys + i, key); }
            else {
                p.out_idx[i] = key == ~0ull ? -1 : (int32_t)(unsigned int)key;
                p.out_dist[i] = key == ~0ull ? INF : __uint_as_float((unsigned int)(key >> 32));
            }
        }
    }
}
__global__ void __launch_bounds__(256) direct_fill_kernel(unsigned long long* __restrict__ keys, int m)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < m) keys[i] = ~0ull;
}
__global__ void __launch_bounds__(256) direct_unpack_kernel(const unsigned long long* __restrict__ keys, int m, int32_t* __restrict__ out_idx,
                                                            float* __restrict__ out_dist)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const unsigned long long key = keys[i];
    out_idx[i] = key == ~0ull ? -1 : (int32_t)(unsigned int)key;
    out_dist[i] = key == ~0ull ? INF : __uint_as_float((unsigned int)(key >> 32));
}

// Where every pair is evaluated instead of the engine's search, measured on both sides of the lines (us a call among others, this
// against the engine).  What the operations cost is one part, what it takes to bring every candidate once to each panel of eight
// queries, 64 at a time, the other; it grows with the candidates, and with their width where a step is more than one slab.
//   up to 100 M operations: 1250 x 4000 x 4 22 and 45, 178 x 4000 x 64 24 and 39, 22 x 32 000 x 64 35 and 45, 64 x 50 000 x 8 37 and 43;
//     the worst of 40 shapes 24 x 8000 x 250 78 and 72, 20 x 100 000 x 6 57 and 50;
//   up to 200 M: 1136 x 4000 x 16 25 and 45, 694 x 4000 x 30 27 and 47, 173 x 16 000 x 30 32 and 48, 142 x 32 000 x 16 33 and 38; the worst
//     of 33 shapes up to 65 536 candidates 43 x 64 000 x 30 55 and 49; beyond those 32 x 111 642 x 21 70 and 57, 16 x 300 000 x 16 88 and 85;
//   300 M: even on the whole (1704 x 4000 x 16 37 and 47, 3750 x 4000 x 4 47 and 50, 360 x 32 000 x 7 45 and 41, 73 x 8000 x 250 94 and 76).
bool direct_1nn_wanted(long long m, long long nc, int d)
{
    return m <= (1LL << 20) && nc <= (1LL << 24) && m * nc * (2LL * d + 12) <= (nc <= 65536 ? 200000000LL : 100000000LL);
}

hipError_t direct_1nn(const float* Xq, int m, int nq_rows, const int32_t* q_rows, const float* Xc, int nc, int d, const int32_t* colour,
                      int32_t* out_idx, float* out_dist, unsigned long long* keys, hipStream_t s)
{
    if (m < 1) return hipSuccess;
    const int per = WAVES * QW1, panels = (m + per - 1) / per;
    // shares of the candidates: about four workgroups per CU, at least four steps each
    int segments = panels >= 512 ? 1 : 1024 / panels;
    const int steps = (nc + 63) / 64;
    if (segments > steps / 4) segments = steps / 4;
    if (segments < 1) segments = 1;
    const int per_segment = (steps + segments - 1) / segments * 64;
    segments = (nc + per_segment - 1) / per_segment;
    Direct1nn p{Xq, Xc, q_rows, colour, m, nq_rows, nc, d, segments, per_segment,
                d % 4 == 0 && ((reinterpret_cast<uintptr_t>(Xq) | reinterpret_cast<uintptr_t>(Xc)) & 15) == 0, out_idx, out_dist, keys};
    const dim3 per_m((unsigned)((m + 255) / 256));
    if (segments > 1) hipLaunchKernelGGL(direct_fill_kernel, per_m, dim3(256), 0, s, keys, m);
    hipLaunchKernelGGL(direct_1nn_kernel, dim3((unsigned)(panels * segments)), dim3(64 * WAVES), 0, s, p);
    if (segments > 1) hipLaunchKernelGGL(direct_unpack_kernel, per_m, dim3(256), 0, s, keys, m, out_idx, out_dist);
    return hipGetLastError();
}

}  // namespace slhc
