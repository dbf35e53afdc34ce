// Small searches: every pair is evaluated exactly, by the vector units.
//
// The half-precision engine (near_kernels.hip) takes eight or nine launches of 4 us and more each, which for some million pairs is more than
// all of them cost: a pair is 2 d operations, a wavefront evaluates 64 at a time, one candidate per lane; the queries' values are the
// same for all lanes.  Every distance is the float32 sum of the list kernels in their order of additions (group8_sqdist): slabs of 64
// features, sixteen chains of four features each, the chains of either half added in a tree.
//
// 1-NN searches of few queries (direct_1nn): the candidates of a workgroup pass through LDS, 16 bytes of every row side by side (no bank is
// met twice).  Bound by its three launches and one round trip to memory per 64 candidates.  439 x 2414 x 16: 42 -> 13 us.
//
// Searches of the rows among themselves (direct_knn): with the candidates in LDS as well a wavefront's reads took longer than its
// sums (2048 x 32, k = 8, 65 us against the engine's 47); with four of them in a lane's registers it is bound by the sums, 8 us of 18, and by the
// way of the rows into the registers.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include "direct_kernels.h"
#include "wave_ops.h"

namespace slhc {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_word __attribute__((ext_vector_type(4), aligned(4)));      // global loads of 16 bytes need the alignment of a word only
constexpr float INF = __builtin_inff();
constexpr float NONE = __builtin_nanf("");
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
    // The segments of a panel end together, and queue for its queries' words: they are met by one instruction for the eight of them, not by one each
    // (us on the GPU, one each after reductions through LDS, one each after vector instructions, by which more end at once, this: 440 x 2678 x 30 18.1, 18.5,
    // 17.7; 1432 x 2103 x 12 18.2, 19.1, 18.5; 1000 x 3000 x 20 20.3, 19.8, 19.4; 100 x 30 000 x 16 30.4, 30.0, 19.9; 20 x 100 000 x 6 -, 54.6, 18.7).
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(tile);
    __syncthreads();                                // the last tile is used up
#pragma unroll
    for (int q = 0; q < QW1; ++q) {
        const unsigned long long key =
            wave_min(at[q] >= 0 && row[q] >= 0 && norm[q] < INF ? ((unsigned long long)__float_as_uint(best[q]) << 32) | (unsigned int)at[q] : ~0ull);
        if (lane == 0) keys[wave * QW1 + q] = key;
    }
    __syncthreads();
    const int i = panel * WAVES * QW1 + threadIdx.x;
    if (threadIdx.x >= WAVES * QW1 || i >= p.m) return;
    const unsigned long long key = keys[threadIdx.x];
    if (p.segments > 1) { if (key != ~0ull) atomicMin(p.keys + i, key); }
    else {
        p.out_idx[i] = key == ~0ull ? -1 : (int32_t)(unsigned int)key;
        p.out_dist[i] = key == ~0ull ? INF : __uint_as_float((unsigned int)(key >> 32));
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

// ---------------------------------------------------------------------------------------------- blocks of pairs in registers
// Searches of the rows among themselves: a lane holds C candidates in registers, and a wavefront passes over the workgroup's queries, whose values
// come from LDS, the same for all lanes.  NQ: four features each, up to 128; what is beyond d is 0 and adds nothing.  The sum is that of
// direct_sum: chain j adds features 4 j .. 4 j + 3 and the same 64 on.
constexpr int BLOCK = 512;                 // threads, and candidates that are brought in at a time
constexpr int SLAB_QUADS = 8;              // quads of a row in LDS at a time
__host__ __device__ constexpr int block_pitch(int NQ) { return (NQ < SLAB_QUADS ? NQ : SLAB_QUADS) | 1; }      // in quads; odd: no bank is met twice
__host__ __device__ constexpr int block_most(int NQ) { return NQ <= 8 ? 4 : NQ <= 16 ? 2 : 1; }                // candidates of a lane

// adds sixteen chains, those from n on being 0
template <int N>
__device__ inline float block_tree(const float (&p)[N])
{
    float s[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        float t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = 8 * half + i < N ? p[8 * half + i < N ? 8 * half + i : 0] : 0.f;
        // (0 is added to sums of squares only, which it leaves as they are)
        auto add = [&](int a, int b, bool there) { return there ? t[a] + t[b] : t[a]; };
        const float u0 = add(0, 1, 8 * half + 1 < N), u1 = add(2, 3, 8 * half + 3 < N), u2 = add(4, 5, 8 * half + 5 < N), u3 = add(6, 7, 8 * half + 7 < N);
        const float v0 = 8 * half + 2 < N ? u0 + u1 : u0, v1 = 8 * half + 6 < N ? u2 + u3 : u2;
        s[half] = 8 * half + 4 < N ? v0 + v1 : v0;
    }
    return N > 8 ? s[0] + s[1] : s[0];
}

// The candidates on their way into registers: 512 rows, a slab of their features, a step; AHEAD steps are under way, so that the loads pass while the
// rows before are evaluated.  All threads go through it together.
struct BlockRows { const float* Xc; int nc, d, queries; };
template <int NQ>
struct BlockStream {
    static constexpr int SLABS = (NQ + SLAB_QUADS - 1) / SLAB_QUADS, PITCH = block_pitch(NQ), WIDTH = NQ < SLAB_QUADS ? NQ : SLAB_QUADS;
    static constexpr int AHEAD = NQ <= 4 ? 4 : NQ == 16 ? 1 : 2;         // (what registers are left)
    BlockRows x;
    v4f* tile;
    v4f next[AHEAD][WIDTH];
    int step;                                                           // of next[0]
    template <int SLAB>
    __device__ inline __attribute__((always_inline)) void fetch(v4f (&to)[WIDTH], int row0)
    {
        constexpr int J0 = SLAB * SLAB_QUADS, W = NQ - J0 < WIDTH ? NQ - J0 : WIDTH;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            // consecutive lanes read consecutive pieces of a row
            const int at = threadIdx.x + i * BLOCK, r = at / W, j = at - r * W;
            to[i] = quad(row0 + r < x.nc ? row0 + r : x.nc - 1, 4 * (J0 + j));
        }
    }
    // Without branches that lanes part at: the row's last four features stand in for what ends beyond them, which `bring` puts right.
    __device__ inline v4f quad(int row, int t) const
    {
        if constexpr (NQ <= 2)                           // (the only ones for rows so narrow)
            if (x.d < 4) return direct_quad(x.Xc, row, t, x.d, false);
        // (an offset of 32 bits: a million rows of 128 columns at most)
        const unsigned int at = ((unsigned int)row * (unsigned int)x.d + (unsigned int)(t + 4 <= x.d ? t : x.d - 4)) * 4u;
        return *reinterpret_cast<const v4f_word*>(reinterpret_cast<const char*>(x.Xc) + at);
    }
    __device__ inline void start(const BlockRows& x_, v4f* tile_)
    {
        x = x_; tile = tile_; step = 0;
        fetch<0>(next[0], 0);
        if constexpr (AHEAD > 1) fetch<1 % SLABS>(next[1], 1 / SLABS * BLOCK);
        if constexpr (AHEAD > 2) { fetch<2 % SLABS>(next[2], 2 / SLABS * BLOCK); fetch<3 % SLABS>(next[3], 3 / SLABS * BLOCK); }
    }
    // the lane's row of the next 512, features of slab SLAB
    template <int SLAB>
    __device__ inline __attribute__((always_inline)) void bring(v4f (&b)[NQ])
    {
        constexpr int J0 = SLAB * SLAB_QUADS, W = NQ - J0 < WIDTH ? NQ - J0 : WIDTH;
        __syncthreads();                            // the rows of the step before are used up
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const int at = threadIdx.x + i * BLOCK, r = at / W, j = at - r * W;
            tile[r * PITCH + j] = next[0][i];
        }
#pragma unroll
        for (int a = 0; a + 1 < AHEAD; ++a)
#pragma unroll
            for (int i = 0; i < WIDTH; ++i) next[a][i] = next[a + 1][i];
        fetch<(SLAB + AHEAD) % SLABS>(next[AHEAD - 1], (step + AHEAD) / SLABS * BLOCK);
        ++step;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < W; ++j) b[J0 + j] = tile[threadIdx.x * PITCH + j];
        if (x.d < 4 * NQ && x.d >= 4) {
#pragma unroll
            for (int j = 0; j < W; ++j) {
                const int over = 4 * (J0 + j) + 4 - x.d;                     // (the same for all lanes)
                v4f& v = b[J0 + j];
                if (over >= 4) v = v4f{0.f, 0.f, 0.f, 0.f};
                else if (over == 3) v = v4f{v[3], 0.f, 0.f, 0.f};
                else if (over == 2) v = v4f{v[2], v[3], 0.f, 0.f};
                else if (over == 1) v = v4f{v[1], v[2], v[3], 0.f};
            }
        }
    }
};
// The queries qs [queries][NQ] against the next 512 C candidates: visit(q, distances), NaN for candidates that are not finite; ready(c): before that,
// for the lane's c-th candidate.  large: a query's norm is not moderate, see direct_bad_row.  Whether the candidates are finite is looked at once,
// as soon as a distance of the wavefront's is so large that one may not be: the row is in registers, and NaN from then on if it is not.  (With a look at
// the row in memory per pair 2048 x 32, k = 8, all rows of such norms, took 484 us, one row NaN 207; 18 both, as without such rows.)
template <int C, int NQ, typename R, typename V>
__device__ inline __attribute__((always_inline)) void block_pass(BlockStream<NQ>& s, const v4f* qs, bool large, R&& ready, V&& visit)
{
    v4f b[C][NQ];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        s.template bring<0>(b[c]);
        if constexpr (NQ > SLAB_QUADS) s.template bring<1>(b[c]);
        if constexpr (NQ > 2 * SLAB_QUADS) s.template bring<2>(b[c]);
        if constexpr (NQ > 3 * SLAB_QUADS) s.template bring<3>(b[c]);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) ready(c);
    // (AHEAD: quads read before they are used.  With one candidate a lane the compiler reads and waits quad by quad: 1300 x 100 45 us, 37 so.)
    constexpr int CHAINS = NQ < 16 ? NQ : 16, AHEAD = C == 1 && NQ >= 24 ? 2 : 0;
    auto look = [&]() {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            float norm = 0.f;
#pragma unroll
            for (int j = 0; j < NQ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) norm = __builtin_fmaf(b[c][j][e], b[c][j][e], norm);
            if (!(norm < INF)) b[c][0][0] = NONE;
        }
    };
    if (large) look();
    bool looked = large;
#pragma unroll 1
    for (int q = 0; q < s.x.queries; ++q) {
        float p[C][CHAINS];
        v4f ahead[AHEAD + 1];
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) ahead[j] = qs[q * NQ + j];
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            if (AHEAD > 0) __builtin_amdgcn_sched_barrier(0);
            if (j + AHEAD < NQ) ahead[(j + AHEAD) % (AHEAD + 1)] = qs[q * NQ + j + AHEAD];
            const v4f a = ahead[j % (AHEAD + 1)];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                float t = j < 16 ? 0.f : p[c][j & 15];
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float z = a[e] - b[c][j][e]; t = j < 16 && e == 0 ? z * z : __builtin_fmaf(z, z, t); }
                p[c][j & 15] = t;
            }
        }
        float v[C];
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = block_tree<CHAINS>(p[c]);
        if (!looked) {
            bool some = false;
#pragma unroll
            for (int c = 0; c < C; ++c) some = some || !(v[c] < 2e38f);
            if (__any(some)) {
                look();
                looked = true;
#pragma unroll
                for (int c = 0; c < C; ++c) v[c] = b[c][0][0] != b[c][0][0] ? NONE : v[c];
            }
        }
        visit(q, v);
    }
}
// all candidates, and no places beyond the last 512: pass(how many times 512, the first of them)
template <int NQ, typename F>
__device__ inline __attribute__((always_inline)) void block_passes(int nc, F&& pass)
{
    int base = 0;
    if constexpr (block_most(NQ) >= 4)
        for (; nc - base > 3 * BLOCK; base += 4 * BLOCK) pass(std::integral_constant<int, 4>{}, base);
    if constexpr (block_most(NQ) >= 2)
        for (; nc - base > BLOCK; base += 2 * BLOCK) pass(std::integral_constant<int, 2>{}, base);
    for (; nc - base > 0; base += BLOCK) pass(std::integral_constant<int, 1>{}, base);
}

// The k nearest rows of every row.  All distances of a workgroup's QB rows are kept in LDS, NaN where there is no row; then a wavefront per row takes what
// is not beyond the k-th smallest of its lanes' minima, of which k at least are, and ranks that.  Rows so far away that the distance is no
// float32 are neighbours all the same, at +inf, behind all others.
// Time (k = 12, us; engine, this): 500 x 4 43, 10; 1000 x 16 46, 10; 2048 x 32 49, 19; 2048 x 32, k = 64, 73, 22; 1500 x 128 56, 33; 3198 x 16 60, 37.
struct DirectKnn {
    const float* X; int n, d, k, rows; bool vec4;         // rows: per workgroup, KNN_ROWS at most
    int32_t* out_idx; float* out_dist; unsigned long long* pairs; unsigned int* nonfinite;
};
constexpr int KNN_ROWS = 8, KNN_KEEP = 512;       // (a wavefront each); pairs that a row keeps to be ranked

// LDS: the candidates' rows, later the pairs to be ranked; the queries' rows and norms; all distances
__host__ __device__ inline size_t direct_knn_head(int NQ, int rows)
{
    const size_t tile = (size_t)BLOCK * block_pitch(NQ) * 16, keep = (size_t)rows * KNN_KEEP * 8;
    return tile > keep ? tile : keep;
}
__host__ __device__ inline size_t direct_knn_bytes(int NQ, int rows, int n)
{
    return direct_knn_head(NQ, rows) + (size_t)rows * NQ * 16 + KNN_ROWS * 4 + (size_t)rows * ((n + BLOCK - 1) / BLOCK * BLOCK) * 4;
}

template <int NQ>
__global__ void __launch_bounds__(BLOCK) direct_knn_kernel(DirectKnn p)
{
    extern __shared__ __align__(16) unsigned char direct_smem[];
    v4f* tile = reinterpret_cast<v4f*>(direct_smem);
    v4f* qs = reinterpret_cast<v4f*>(direct_smem + direct_knn_head(NQ, p.rows));
    float* norms = reinterpret_cast<float*>(qs + p.rows * NQ);
    float* dist = norms + KNN_ROWS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n64 = (p.n + 63) / 64, pitch = (p.n + BLOCK - 1) / BLOCK * BLOCK;
    const int q0 = blockIdx.x * p.rows;
    BlockStream<NQ> stream;
    stream.start(BlockRows{p.X, p.n, p.d, p.rows}, tile);
    if (p.pairs && blockIdx.x == 0 && tid == 0) atomicAdd(p.pairs, (unsigned long long)p.n * (unsigned long long)(p.n - 1));
    for (int i = tid; i < p.rows * NQ; i += BLOCK) qs[i] = direct_quad(p.X, q0 + i / NQ < p.n ? q0 + i / NQ : -1, 4 * (i % NQ), p.d, p.vec4);
    if (wave < p.rows) {
        const float norm = direct_norm(p.X, q0 + wave < p.n ? q0 + wave : -1, p.d, lane);
        if (lane == 0) norms[wave] = norm;
    }
    __syncthreads();
    bool large = false;
    for (int q = 0; q < p.rows; ++q) large = large || !(norms[q] < 1e36f);
    large = __any(large);
    auto pass = [&](auto per, int base) {
        constexpr int C = decltype(per)::value;
        block_pass<C>(stream, qs, large, [](int) {}, [&](int q, float (&v)[C]) {
#pragma unroll
            for (int c = 0; c < C; ++c) dist[q * pitch + base + c * BLOCK + tid] = v[c];
        });
    };
    block_passes<NQ>(p.n, pass);
    __syncthreads();
    const int row = q0 + wave;
    if (wave >= p.rows || row >= p.n) return;
    float* mine = dist + wave * pitch;
    if (lane == 0) mine[row] = NONE;                                          // itself, and no rows
    if (p.n + lane < n64 * 64) mine[p.n + lane] = NONE;
    __builtin_amdgcn_wave_barrier();
    unsigned long long* keep = reinterpret_cast<unsigned long long*>(direct_smem) + wave * KNN_KEEP;      // (the candidates' rows are used up)
    const bool fine = norms[wave] < INF;
    if (p.nonfinite && !fine && lane == 0) atomicOr(p.nonfinite, 1u);
    // the row's distances, 16 of a lane's at a time: what(first of them, values), +inf from n64 on (not NaN, which the compiler
    // would take out of the minima, and read one value after the other)
    auto all = [&](auto&& what) {
        for (int i0 = 0; i0 < n64; i0 += 16) {
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = i0 + i < n64 ? mine[(i0 + i) * 64 + lane] : INF;
            what(i0, v);
        }
    };
    // a value that k of the row's do not exceed, and few others: the k-th smallest minimum of a lane's values or, from sixteen on, of every fourth of them
    float limit;
    if (p.k <= 16) {
        float least = INF;
        all([&](int, const float (&v)[16]) {
#pragma unroll
            for (int i = 0; i < 16; ++i) least = fminf(least, v[i]);
        });
        int rank = 0;
#pragma unroll
        for (int j = 0; j < 64; ++j) rank += __uint_as_float((unsigned int)__builtin_amdgcn_readlane((int)__float_as_uint(least), j)) < least ? 1 : 0;
        limit = rank < p.k ? least : 0.f;                                     // (distances are not negative)
        limit = wave_max(limit);
    } else {
        float least[4] = {INF, INF, INF, INF};
        all([&](int, const float (&v)[16]) {
#pragma unroll
            for (int i = 0; i < 16; ++i) least[i & 3] = fminf(least[i & 3], v[i]);
        });
        float lo = INF, hi = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) { lo = fminf(lo, least[j]); hi = least[j] < INF ? fmaxf(hi, least[j]) : hi; }
        lo = wave_min(lo); hi = wave_max(hi);
        auto reach = [&](float upto) {
            int n = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) n += __popcll(__ballot(least[j] <= upto));
            return n;
        };
        limit = INF;
        if (reach(hi) >= p.k) {
            limit = hi;
            for (int it = 0; it < 14; ++it) {
                const float mid = 0.5f * lo + 0.5f * limit;
                if (reach(mid) >= p.k) limit = mid; else lo = mid;
            }
        }
    }
    // what does not exceed it, in the order of the rows
    auto prefix = [&](unsigned long long m) { return (int)__builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u)); };
    int kept = 0;
    auto take = [&](auto&& passes) {                                          // passes(value), called by all lanes together
        kept = 0;
        all([&](int i0, const float (&v)[16]) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const bool in = passes(v[i]) && v[i] < INF;
                const unsigned long long m = __ballot(in);
                if (m == 0ull) continue;
                const int at = kept + prefix(m);
                if (in && at < KNN_KEEP) keep[at] = ((unsigned long long)__float_as_uint(v[i]) << 32) | (unsigned int)((i0 + i) * 64 + lane);
                kept += __popcll(m);
            }
        });
    };
    auto count = [&](float upto) {
        int n = 0;
        all([&](int, const float (&v)[16]) {
#pragma unroll
            for (int i = 0; i < 16; ++i) n += __popcll(__ballot(v[i] <= upto));
        });
        return n;
    };
    if (!fine) kept = 0;
    else {
        take([&](float v) { return v <= limit; });
        if (kept > 2 * p.k + 64) {
            // copies by the hundred, or k near the number of lanes: the k-th smallest value itself, and of those equal to it the first
            // (bits of floats that are not negative are in their order)
            unsigned int lo = 0u, hi = __float_as_uint(limit < INF ? limit : 3.4028234663852886e38f);
            while (lo < hi) {
                const unsigned int mid = lo + (hi - lo) / 2;
                if (count(__uint_as_float(mid)) >= p.k) hi = mid; else lo = mid + 1;
            }
            const float kth = __uint_as_float(hi);
            int room = p.k - (hi > 0u ? count(__uint_as_float(hi - 1u)) : 0);
            take([&](float v) {
                const unsigned long long ties = __ballot(v == kth);
                const bool in = v < kth || (v == kth && prefix(ties) < room);
                room -= __popcll(ties);
                return in;
            });
        }
        for (int i = 0; kept < p.k && i < n64; ++i) {
            const bool in = mine[i * 64 + lane] == INF;
            const unsigned long long m = __ballot(in);
            const int at = kept + prefix(m);
            if (in && at < p.k) keep[at] = ((unsigned long long)__float_as_uint(INF) << 32) | (unsigned int)(i * 64 + lane);
            kept = kept + __popcll(m) < p.k ? kept + __popcll(m) : p.k;
        }
        __builtin_amdgcn_wave_barrier();
    }
    // ranks by (distance, row)
    for (int i = 0; i < kept; i += 64) {
        const unsigned long long key = i + lane < kept ? keep[i + lane] : ~0ull;
        int at = 0;
        for (int j = 0; j < kept; ++j) at += keep[j] < key ? 1 : 0;
        if (i + lane < kept && at < p.k) {
            p.out_idx[(size_t)row * p.k + at] = (int32_t)(unsigned int)key;
            p.out_dist[(size_t)row * p.k + at] = __uint_as_float((unsigned int)(key >> 32));
        }
    }
    for (int j = kept + lane; j < p.k; j += 64) { p.out_idx[(size_t)row * p.k + j] = -1; p.out_dist[(size_t)row * p.k + j] = INF; }
}

// The nearest row (of another colour): as direct_knn_kernel, with one (distance, row) per query in LDS instead of all distances.  A workgroup has a panel of
// queries and a segment of the candidates; where there are several segments, they meet at a word per query.
// (Without segments, for rounds of 9 to 46 queries: 24 000 x 128 0.69 ms, 100 000 x 128 3.8, 300 000 x 100 9, 1M x 16 10; the engine 0.15, 0.35, 0.4, 1.0; so
// 0.06, 0.13, 0.11, 0.15.)
struct DirectNear {
    const float* Xq; const float* Xc; const int32_t* q_rows; const int32_t* colour;
    int m, nq_rows, nc, d, rows, segments, per_segment;
    int32_t* out_idx; float* out_dist; unsigned long long *keys, *pairs;
};
constexpr int NEAR_ROWS = 32;              // queries of a workgroup at most

template <int NQ>
__global__ void __launch_bounds__(BLOCK) direct_near_kernel(DirectNear p)
{
    extern __shared__ __align__(16) unsigned char direct_smem[];
    __shared__ unsigned long long best[NEAR_ROWS];
    __shared__ float norms[NEAR_ROWS];
    __shared__ int row_of[NEAR_ROWS], colour_of[NEAR_ROWS];
    v4f* tile = reinterpret_cast<v4f*>(direct_smem);
    v4f* qs = tile + BLOCK * block_pitch(NQ);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int panel = blockIdx.x / p.segments, c0 = (blockIdx.x - panel * p.segments) * p.per_segment;
    const int q0 = panel * p.rows, nc = p.nc - c0 < p.per_segment ? p.nc - c0 : p.per_segment;
    const int32_t* c_colour = p.colour ? p.colour + c0 : nullptr;
    BlockStream<NQ> stream;
    stream.start(BlockRows{p.Xc + (size_t)c0 * p.d, nc, p.d, p.rows}, tile);
    if (tid < p.rows) {
        const int i = q0 + tid;
        int row = i < p.m ? (p.q_rows ? p.q_rows[i] : i) : -1;
        if (row >= p.nq_rows) row = -1;
        row_of[tid] = row;
        colour_of[tid] = p.colour && row >= 0 ? p.colour[row] : -1;
        best[tid] = ~0ull;
    }
    if (p.pairs && blockIdx.x == 0 && tid == 0) atomicAdd(p.pairs, (unsigned long long)p.m * (unsigned long long)p.nc);
    __syncthreads();
    const bool vec4 = p.d % 4 == 0 && (reinterpret_cast<uintptr_t>(p.Xq) & 15) == 0;
    for (int i = tid; i < p.rows * NQ; i += BLOCK) qs[i] = direct_quad(p.Xq, row_of[i / NQ], 4 * (i % NQ), p.d, vec4);
    for (int q = wave; q < p.rows; q += BLOCK / 64) {
        const float norm = direct_norm(p.Xq, row_of[q], p.d, lane);
        if (lane == 0) norms[q] = norm;
    }
    __syncthreads();
    bool large = false;
    for (int q = 0; q < p.rows; ++q) large = large || !(norms[q] < 1e36f);
    large = __any(large);
    block_passes<NQ>(nc, [&](auto per, int base) {
        constexpr int C = decltype(per)::value;
        int colour[C];
        block_pass<C>(stream, qs, large,
            [&](int c) {
                // (beyond the last candidate stands the last one again, with a larger index: it is never the smallest key)
                const int cand = base + c * BLOCK + tid;
                colour[c] = c_colour ? c_colour[cand < nc ? cand : nc - 1] : -2;
            },
            [&](int q, float (&v)[C]) {
                const int mine = colour_of[q];
                float least = INF;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    v[c] = colour[c] == mine ? INF : v[c];
                    least = fminf(least, v[c]);
                }
                // (the distance's word alone: another wavefront may be at it)
                const float upto = __uint_as_float(*(volatile unsigned int*)(reinterpret_cast<unsigned int*>(best + q) + 1));
                if (!__any(least < INF && !(least > upto))) return;          // (all ones, nothing yet, are a NaN)
                int at = 0;
#pragma unroll
                for (int c = C - 1; c > 0; --c) at = v[c] == least ? c * BLOCK : at;
                at = v[0] == least ? 0 : at;
                const unsigned long long key = wave_min(least < INF ? ((unsigned long long)__float_as_uint(least) << 32) | (unsigned int)(c0 + base + at + tid) : ~0ull);
                if (lane == 0) atomicMin(best + q, key);
            });
    });
    __syncthreads();
    if (tid < p.rows && q0 + tid < p.m) {
        const bool some = best[tid] != ~0ull && row_of[tid] >= 0 && norms[tid] < INF;
        if (p.segments > 1) {
            if (some) atomicMin(p.keys + q0 + tid, best[tid]);
            return;
        }
        p.out_idx[q0 + tid] = some ? (int32_t)(unsigned int)best[tid] : -1;
        p.out_dist[q0 + tid] = some ? __uint_as_float((unsigned int)(best[tid] >> 32)) : INF;
    }
}

// Where every pair is evaluated instead of the engine's search, measured on both sides of the line (us a call among others, this against the engine).
// What an evaluation costs here is its operations (0.06 to 0.12 us a million) and what it takes to bring every candidate once to each panel of eight queries; the
// engine makes a copy of all candidates first, which costs what a dozen queries' evaluations cost, and has nine launches.  So as many queries beyond
// twelve as are 240 M operations:
//   300 x 10 000 x 20 22 and 35, 100 x 50 000 x 20 32 and 43, 30 x 150 000 x 20 32 and 58, 10 x 500 000 x 20 47 and 103, 30 x 500 000 x 6 59 and 103,
//   100 x 10 000 x 64 23 and 36, 30 x 150 000 x 64 60 and 66, 10 x 500 000 x 128 170 and 212, 30 x 50 000 x 128 51 and 57, 10 x 500 000 x 250 356 and 589;
//   wide rows: 16 x 10 000 x 784 57 and 97, 12 x 10 000 x 2000 137 and 200, 12 x 10 000 x 8000 596 and 1746, 12 x 3000 x 12 000 795 and 2635, 16 x 30 000 x 784 75 and 144;
//   beyond: 1000 x 10 000 x 20 50 and 37, 100 x 150 000 x 20 74 and 58, 100 x 50 000 x 64 62 and 47, 30 x 500 000 x 64 170 and 127, 300 x 10 000 x 128 76 and 50.
bool direct_1nn_wanted(long long m, long long nc, int d)
{
    return m <= (1LL << 20) && nc <= (1LL << 24) && (m - 12) * nc * (2LL * d + 12) <= 240000000LL;
}
// Those of them that ask for no workspace of the engine (the line of an earlier day; sizes that are reported have not changed).
bool direct_1nn_alone(long long m, long long nc, int d)
{
    return m <= (1LL << 20) && nc <= (1LL << 24) && m * nc * (2LL * d + 12) <= (nc <= 65536 ? 200000000LL : 100000000LL);
}

hipError_t direct_1nn(const float* Xq, int m, int nq_rows, const int32_t* q_rows, const float* Xc, int nc, int d, const int32_t* colour,
                      int32_t* out_idx, float* out_dist, unsigned long long* keys, hipStream_t s)
{
    if (m < 1) return hipSuccess;
    const int per = WAVES * QW1, panels = (m + per - 1) / per;
    // Shares of the candidates: about four workgroups per CU, of at least four slabs of 64 candidates each, which are a round trip to memory each, one after
    // the other.  (With four steps of all slabs at least, 16 x 10 000 x 784 took 202 us, 12 x 10 000 x 2000 581, 4 x 10 000 x 8000 2711 and 8 x 1000 x 250 55; the
    // engine 97, 186 and 1158 of the first three; so 57, 137, 598 and 19.  Two slabs a row, 8 x 3000 x 128 37 and 25, 300 x 300 x 100 29 and 22.)
    int segments = panels >= 512 ? 1 : 1024 / panels;
    const int steps = (nc + 63) / 64, slabs = (d + SLAB - 1) / SLAB, least = slabs >= 4 ? 1 : (3 + slabs) / slabs;
    if (segments > steps / least) segments = steps / least;
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

// quads that the kernels are made for
static int direct_quads(int d)
{
    const int q = (d + 3) / 4;
    return q <= 2 ? 2 : q <= 4 ? 4 : q <= 8 ? 8 : q <= 12 ? 12 : q <= 16 ? 16 : q <= 24 ? 24 : 32;
}
template <typename F>
static hipError_t direct_by_quads(int nq, F&& f)
{
    switch (nq) {
        case 2: return f(std::integral_constant<int, 2>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 12: return f(std::integral_constant<int, 12>{});
        case 16: return f(std::integral_constant<int, 16>{});
        case 24: return f(std::integral_constant<int, 24>{});
        default: return f(std::integral_constant<int, 32>{});
    }
}
constexpr size_t DIRECT_LDS = 160 << 10;
static int direct_cus()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1) return 256;
    return v;
}

// Rows per workgroup, 0: none fit.  Workgroups of one row more each where that saves a round of them.
static int direct_knn_rows(long long n, int nq, int cus)
{
    for (int rounds = 1; rounds <= 64; ++rounds) {
        const long long rows = (n + (long long)cus * rounds - 1) / ((long long)cus * rounds);
        if (rows <= KNN_ROWS && direct_knn_bytes(nq, (int)rows, (int)n) <= DIRECT_LDS) return (int)rows;
        if (rows <= 1) return 0;
    }
    return 0;
}
// What a step, 512 candidates for a workgroup's rows, takes: 130 + 26 per quad to bring them, 8 per quad and 24 for a row; about 4 ns each.
static long long direct_step(int nq, int rows) { return 130 + 26 * nq + (long long)rows * (8 * nq + 24); }

// The line.  Where the caller waits for the lists (clusterings): what the workgroups' rounds take against the engine's eight launches, 45 us and 5 more per thousand
// rows.  Us a clustering of one blob, which has nothing to connect, k = 12, engine and this, below the line and above it: 8 columns 4873 rows 314 and 310,
// 5123 318 and 334; 16 columns 4531 305 and 294, 4724 308 and 329; 32 columns 2919 248 and 239, 3107 254 and 270; 48 columns 2958 259 and 257, 3095 255 and
// 284; 64 columns 2500 237 and 240, 2628 281 and 292; 96 columns 1983 222 and 216, 2097 236 and 263; 128 columns 2026 227 and 227, 2112 274 and 308.
// Lists of 40 others and more the engine collects in half as many segments (near_plan), on half the chip: 20 us more.  k = 36 and 48: 5000 x 16 373 and 369,
// 402 and 380; 3800 x 24 286 and 291, 310 and 290; 3500 x 32 297 and 311, 312 and 309; 2700 x 64 268 and 277, 285 and 276; k = 40: 5900 x 8 409 and 387; but
// 2400 x 96 263 and 280, 2100 x 128 266 and 294.  Up to 8 columns, where rows are most, its selection takes the engine as much longer
// from 24 others on (5300 x 8: k = 8 321 and 324, 24 350 and 338, 36 385 and 364).
// Calls among others: instructions of a lane, two per feature and about 24 for the rest of a pair and its share of the selection.  700 M (k = 12, us): 4183 x 8
// 67 and 51, 2820 x 32 56 and 42, 2415 x 40 56 and 50, 2145 x 64 58 and 53, 1581 x 128 54 and 46; 800 M: 3779 x 16 60 and 50, 3015 x 32 55 and 42,
// 2581 x 40 56 and 58, 2294 x 64 57 and 54; 900 M: 4743 x 8 67 and 65, 3198 x 32 60 and 67, 2738 x 40 57 and 59, 2041 x 96 53 and 41.
int direct_knn_wanted(long long n, int d, int k, bool waited_for)
{
    if (d > 128 || k > 64 || n > 16384) return 0;
    const int nq = direct_quads(d), cus = direct_cus(), rows = direct_knn_rows(n, nq, cus);
    if (rows < 1 || (!waited_for && n * n * (8LL * nq + 24) > 800000000LL)) return 0;
    const long long rounds = ((n + rows - 1) / rows + cus - 1) / cus, steps = (n + BLOCK - 1) / BLOCK;
    const long long longer = d <= 64 && k >= (d <= 8 ? 24 : 40) ? 5200 : 0;
    return rounds * steps * direct_step(nq, rows) <= 11000 + n + n / 6 + longer ? rows : 0;
}

hipError_t direct_knn(const float* X, int n, int d, int k, int rows, int32_t* out_idx, float* out_dist, unsigned long long* pairs, unsigned int* nonfinite, hipStream_t s)
{
    if (rows < 1 || rows > KNN_ROWS || d > 128 || direct_knn_bytes(direct_quads(d), rows, n) > DIRECT_LDS) return hipErrorInvalidValue;
    const DirectKnn p{X, n, d, k, rows, d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0, out_idx, out_dist, pairs, nonfinite};
    return direct_by_quads(direct_quads(d), [&](auto quads) -> hipError_t {
        constexpr int NQ = decltype(quads)::value;
        const size_t lds = direct_knn_bytes(NQ, rows, n);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&direct_knn_kernel<NQ>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((direct_knn_kernel<NQ>), dim3((unsigned)((n + rows - 1) / rows)), dim3(BLOCK), lds, s, p);
        return hipGetLastError();
    });
}

// The line, for a round of connecting components, in the instructions of direct_knn_wanted, against near_link's ten launches (us, kernels of all rounds
// of a clustering whose last one asks for as many rows as make 1000 M, near_link and this): 6000 x 64 173 and 77, 6000 x 128 178 and 83, 24 000 x 32 164 and
// 97, 24 000 x 128 191 and 128, 100 000 x 32 262 and 207, 100 000 x 128 391 and 392.  2000 M: 24 000 x 32 175 and 132, 24 000 x 128 197 and 157,
// 100 000 x 32 271 and 231, 100 000 x 128 390 and 426; 4000 M: 356 and 1266 (all rows once), 204 and 215, 282 and 287, 399 and 490.
bool direct_near_wanted(long long m, long long nc, int d)
{
    return d <= 128 && m >= 1 && nc <= (1LL << 20) && m <= (1LL << 20) && m * nc * (8LL * direct_quads(d) + 24) <= 1000000000LL;
}

// Queries of a workgroup, and segments of the candidates: what takes least by direct_step (24 000 candidates for one query of a workgroup: 128 columns 230 us,
// 64 112, 32 66); the two launches that segments need take 3000 (2 us and 4, and what lies between), and a workgroup has a CU to itself.
struct NearSplit { int rows, segments, per_segment; };
static NearSplit direct_near_split(int m, int nc, int d)
{
    const int nq = direct_quads(d), cus = direct_cus(), steps = (nc + BLOCK - 1) / BLOCK;
    NearSplit best{};
    long long least = 0;
    for (int rows = 1; rows <= NEAR_ROWS; ++rows) {
        const int panels = (m + rows - 1) / rows;
        // all candidates, or as many segments as there are CUs for
        for (int most = panels < cus ? cus / panels : 1;; most = 1) {
            const int per = (steps + most - 1) / most, segments = (steps + per - 1) / per;
            const long long time = (long long)((panels + cus - 1) / cus) * per * direct_step(nq, rows) + (segments > 1 ? 3000 : 0);
            if (best.rows == 0 || time < least) { least = time; best = NearSplit{rows, segments, per * BLOCK}; }
            if (most == 1) break;
        }
    }
    return best;
}

hipError_t direct_near(const float* Xq, int m, int nq_rows, const int32_t* q_rows, const float* Xc, int nc, int d, const int32_t* colour,
                       int32_t* out_idx, float* out_dist, unsigned long long* keys, unsigned long long* pairs, hipStream_t s)
{
    if (m < 1) return hipSuccess;
    const NearSplit split = direct_near_split(m, nc, d);
    const DirectNear p{Xq, Xc, q_rows, colour, m, nq_rows, nc, d, split.rows, split.segments, split.per_segment, out_idx, out_dist, keys, pairs};
    const dim3 per_m((unsigned)((m + 255) / 256));
    if (split.segments > 1) hipLaunchKernelGGL(direct_fill_kernel, per_m, dim3(256), 0, s, keys, m);
    const hipError_t e = direct_by_quads(direct_quads(d), [&](auto quads) -> hipError_t {
        constexpr int NQ = decltype(quads)::value;
        const size_t lds = ((size_t)BLOCK * block_pitch(NQ) + (size_t)split.rows * NQ) * 16;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&direct_near_kernel<NQ>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((direct_near_kernel<NQ>), dim3((unsigned)((m + split.rows - 1) / split.rows * split.segments)), dim3(BLOCK), lds, s, p);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    if (split.segments > 1) hipLaunchKernelGGL(direct_unpack_kernel, per_m, dim3(256), 0, s, keys, m, out_idx, out_dist);
    return hipGetLastError();
}

}  // namespace slhc
