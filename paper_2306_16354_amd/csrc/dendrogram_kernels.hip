// Linkage arrays (children and sizes of every merge) from the edges of a spanning tree in merge order (paper Sec. 3.3.1, which does this
// on the host: one union-find step per edge, each of them waiting for two random reads).
//
// On the device by contracting the tree level by level, as in published parallel dendrogram constructions (Sao, Prokopenko and Lebrun-Grandie,
// "PANDORA", 2024): every vertex's first edge (the smallest number at it) is contracted, which leaves a tree of at most half the vertices.
//   * What is contracted into one vertex V of the next level is a chain: its edges are first edges, so walking away from the smallest their
//     numbers rise, and every prefix of them is one cluster.  The chain lasts until V's own first edge merges it with a neighbour.
//   * An edge contracted into V with a number beyond V's first edge therefore belongs to the chain of the first vertex above V whose own
//     first edge comes later than it.
//   * A merge's children: for each end of which it is the first edge, the last merge of that end's chain (on the first level the row itself);
//     if it is that of one end only, the merge before it in its own chain.
// So: the levels (two launches each, the last 4096 vertices in LDS in one), a walk per merge, one stable sort by chain, and per level a
// sum along its chains for the sizes.  All of it reads at random, a few words per merge and level, and below a million rows most of the
// time is that of its 30 to 45 launches.  Union-find on the host (16 threads from 200 000 rows on), with the copies, and this:
// 100 000 rows 1.0 and 0.21 ms, 300 000 1.8 and 0.31, 1M 4.6 to 6.3 and 0.52.  A path of 200 000 rows whose edges rise along it, the deepest chains
// there are: 0.82.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "dendrogram_kernels.h"
#include "wave_ops.h"

namespace slhc {

constexpr int TB = 256, TB_WIDE = 1024;
constexpr uint32_t NO_EDGE = 0xffffffffu;
static inline int blocks_for(long long n, int tb) { return (int)((n + tb - 1) / tb); }

// Up to this many vertices the rest of the levels takes one workgroup: 96 KiB of LDS.
constexpr int TAIL = 4096;
constexpr int SUM_ITEMS = 4, SUM_SPAN = TB * SUM_ITEMS;      // merges of a workgroup of k_chain_sums
// From the level on whose merges, with all that follow, are this many at most, one workgroup sums them all.
constexpr int SUM_TAIL = 8192;

size_t dendrogram_carry_words(int64_t N) { return (size_t)(N / SUM_SPAN) + DENDRO_LEVELS + 1; }

__device__ __forceinline__ void failed(int32_t* counters, int site) { atomicCAS(&counters[DENDRO_ERROR], 0, site); }

__global__ void __launch_bounds__(TB) k_levels_init(DendrogramWork w, int N, int carry_words)
{
    const long long i = (long long)blockIdx.x * TB + threadIdx.x;
    if (i < 2ll * N) w.lightest[i] = NO_EDGE;
    if (i < carry_words) w.carry[i] = 0ull;
    if (i < DENDRO_WORDS) w.counters[i] = i == DENDRO_ROWS ? N : i == DENDRO_EDGES ? N - 1 : 0;
}

// the first edge of every row
__global__ void __launch_bounds__(TB) k_first_edges(const int32_t* __restrict__ lo, const int32_t* __restrict__ hi, DendrogramWork w, int N)
{
    const int e = blockIdx.x * TB + threadIdx.x;
    if (e >= N - 1) return;
    const int a = lo[e], b = hi[e];
    if ((unsigned int)a >= (unsigned int)N || (unsigned int)b >= (unsigned int)N || a == b) { failed(w.counters, 1); return; }
    min_into(&w.lightest[a], (uint32_t)e);
    min_into(&w.lightest[b], (uint32_t)e);
}

// Contract: every edge that is the first one of an end.  That end hooks to the other; of an edge that is first on both sides the smaller end
// is the root and takes a number (as -1 - number).  The other edges go to the next level's list.
__global__ void __launch_bounds__(TB_WIDE) k_contract(const int32_t* __restrict__ lo, const int32_t* __restrict__ hi, DendrogramWork w,
                                                      int level, v2i_word* __restrict__ children)
{
    const int n = w.counters[DENDRO_ROWS + level], m = w.counters[DENDRO_EDGES + level], base = w.counters[DENDRO_BASE + level];
    if (n <= TAIL || w.counters[DENDRO_ERROR] != 0 || (int)(blockIdx.x * TB_WIDE) >= m) return;
    const int i = blockIdx.x * TB_WIDE + threadIdx.x;
    const bool mine = i < m;
    uint32_t e = 0;
    int2 v = make_int2(0, 0);
    if (mine) {
        e = level == 0 ? (uint32_t)i : w.edge[level & 1][i];
        v = level == 0 ? make_int2(lo[i], hi[i]) : w.ends[level & 1][i];
    }
    const bool fa = mine && w.lightest[(size_t)base + v.x] == e, fb = mine && w.lightest[(size_t)base + v.y] == e;
    const int root = block_append<TB_WIDE>(fa && fb, &w.counters[DENDRO_ROWS + level + 1]);
    const int small = v.x < v.y ? v.x : v.y, large = v.x < v.y ? v.y : v.x;
    if (fa && fb) { w.hook[small] = -1 - root; w.hook[large] = small; }
    else if (fa) w.hook[v.x] = v.y;
    else if (fb) w.hook[v.y] = v.x;
    if (fa || fb) children[e] = v2i_word{fa ? base + v.x : -1, fb ? base + v.y : -1};
    __syncthreads();                                        // (block_append's LDS is used again)
    const int at = block_append<TB_WIDE>(mine && !fa && !fb, &w.counters[DENDRO_EDGES + level + 1]);
    if (mine && !fa && !fb) {
        w.edge[(level + 1) & 1][at] = e;
        w.ends[(level + 1) & 1][at] = v;
    }
}

// The number of the root above v.  Hooks lead to vertices with an earlier first edge, so the walk ends; every eighth step the vertex
// itself is moved up, which shortens the walks through it.
template <typename P>
__device__ __forceinline__ int root_above(P hook, int v)
{
    int x = v;
    for (int step = 1;; ++step) {
        const int h = hook[x];
        if (h < 0) return -1 - h;
        x = h;
        if ((step & 7) == 0) hook[v] = x;
    }
}

// Every vertex's vertex on the next level, and the edges left between those, with their first edges.
__global__ void __launch_bounds__(TB) k_next_level(DendrogramWork w, int level, int N)
{
    const int n = w.counters[DENDRO_ROWS + level], base = w.counters[DENDRO_BASE + level];
    if (n <= TAIL || w.counters[DENDRO_ERROR] != 0) return;
    const int m = w.counters[DENDRO_EDGES + level + 1];
    const int base_up = base + n;
    if (blockIdx.x == 0 && threadIdx.x == 0) w.counters[DENDRO_BASE + level + 1] = base_up;
    const int vertex_blocks = (n + TB - 1) / TB;
    if ((int)blockIdx.x < vertex_blocks) {
        const int v = blockIdx.x * TB + threadIdx.x;
        if (v >= n) return;
        if (w.lightest[(size_t)base + v] == NO_EDGE) { failed(w.counters, 2); return; }      // (not a tree)
        w.up[(size_t)base + v] = base_up + root_above(w.hook, v);
    } else {
        const int i = (blockIdx.x - vertex_blocks) * TB + threadIdx.x;
        if (i >= m) return;
        const uint32_t e = w.edge[(level + 1) & 1][i];
        const int2 v = w.ends[(level + 1) & 1][i];
        const int a = root_above(w.hook, v.x), b = root_above(w.hook, v.y);
        if (a == b) { failed(w.counters, 3); return; }
        w.ends[(level + 1) & 1][i] = make_int2(a, b);
        min_into(&w.lightest[(size_t)base_up + a], e);
        min_into(&w.lightest[(size_t)base_up + b], e);
    }
}

// The levels of at most TAIL vertices.
__global__ void __launch_bounds__(TB_WIDE) k_last_levels(DendrogramWork w, v2i_word* __restrict__ children, int N)
{
    __shared__ uint32_t lightest[TAIL], edge[2][TAIL], ends[2][TAIL];       // ends: 16 bits each
    __shared__ int hook[TAIL];
    __shared__ int left, roots, bad;
    const int tid = threadIdx.x;
    if (w.counters[DENDRO_ERROR] != 0) return;
    int level = 0;
    while (level < DENDRO_LEVELS - 1 && w.counters[DENDRO_ROWS + level] > TAIL) ++level;
    int n = w.counters[DENDRO_ROWS + level], m = w.counters[DENDRO_EDGES + level], base = w.counters[DENDRO_BASE + level];
    if (level < 1 || n < 1 || n > TAIL || m != n - 1 || base + n > 2 * N) { if (tid == 0) failed(w.counters, 4); return; }
    for (int v = tid; v < n; v += TB_WIDE) lightest[v] = w.lightest[(size_t)base + v];
    for (int i = tid; i < m; i += TB_WIDE) {
        const int2 v = w.ends[level & 1][i];
        edge[0][i] = w.edge[level & 1][i];
        ends[0][i] = ((uint32_t)v.x << 16) | (uint32_t)v.y;
    }
    if (tid == 0) { left = 0; roots = 0; bad = 0; }
    __syncthreads();
    for (int turn = 0; n > 1; turn ^= 1) {
        for (int i = tid; i < m; i += TB_WIDE) {
            const uint32_t e = edge[turn][i], v = ends[turn][i];
            const int a = v >> 16, b = v & 0xffffu;
            const bool fa = lightest[a] == e, fb = lightest[b] == e;
            if (!fa && !fb) {
                const int at = atomicAdd(&left, 1);
                edge[turn ^ 1][at] = e;
                ends[turn ^ 1][at] = v;
                continue;
            }
            children[e] = v2i_word{fa ? base + a : -1, fb ? base + b : -1};
            if (fa && fb) { hook[a < b ? a : b] = -1 - atomicAdd(&roots, 1); hook[a < b ? b : a] = a < b ? a : b; }
            else if (fa) hook[a] = b;
            else hook[b] = a;
        }
        __syncthreads();
        const int n_up = roots, m_up = left;
        for (int v = tid; v < n; v += TB_WIDE)
            if (lightest[v] == NO_EDGE) bad = 1;
            else w.up[(size_t)base + v] = base + n + root_above((volatile int*)hook, v);
        for (int i = tid; i < m_up; i += TB_WIDE) {
            const uint32_t v = ends[turn ^ 1][i];
            const int a = root_above((volatile int*)hook, (int)(v >> 16)), b = root_above((volatile int*)hook, (int)(v & 0xffffu));
            if (a == b) bad = 1;
            ends[turn ^ 1][i] = ((uint32_t)a << 16) | (uint32_t)b;
        }
        __syncthreads();
        if (bad || n_up < 1 || m_up != n_up - 1 || level + 2 >= DENDRO_LEVELS) { if (tid == 0) failed(w.counters, 5); return; }
        for (int v = tid; v < n_up; v += TB_WIDE) lightest[v] = NO_EDGE;
        if (tid == 0) { left = 0; roots = 0; }
        __syncthreads();
        for (int i = tid; i < m_up; i += TB_WIDE) {
            const uint32_t e = edge[turn ^ 1][i], v = ends[turn ^ 1][i];
            atomicMin(&lightest[v >> 16], e);
            atomicMin(&lightest[v & 0xffffu], e);
        }
        __syncthreads();
        base += n; n = n_up; m = m_up; ++level;
        for (int v = tid; v < n; v += TB_WIDE) w.lightest[(size_t)base + v] = lightest[v];
        if (tid == 0) { w.counters[DENDRO_BASE + level] = base; w.counters[DENDRO_ROWS + level] = n; }
    }
    if (tid == 0) w.counters[DENDRO_DEPTH] = level;
}

// The chain of every merge (see above), and how many merges lie in chains of each level.  Chains are named by their vertex, so by level first.
__global__ void __launch_bounds__(TB) k_chains(DendrogramWork w, const v2i_word* __restrict__ children, int N)
{
    __shared__ int base[DENDRO_LEVELS], count[DENDRO_LEVELS];
    if (w.counters[DENDRO_ERROR] != 0) return;
    const int depth = w.counters[DENDRO_DEPTH];
    if (threadIdx.x < DENDRO_LEVELS) { base[threadIdx.x] = (int)threadIdx.x <= depth ? w.counters[DENDRO_BASE + threadIdx.x] : 2 * N; count[threadIdx.x] = 0; }
    __syncthreads();
    const int e = blockIdx.x * TB + threadIdx.x;
    if (e < N - 1) {
        const v2i_word c = children[e];
        int v = w.up[c.x >= 0 ? c.x : c.y];
        while (w.lightest[v] < (uint32_t)e) v = w.up[v];    // (the last vertex has no edge)
        w.key[e] = (uint32_t)(v - N);
        w.val[e] = (uint32_t)e;
        int level = 1;
        while (level < depth && v >= base[level + 1]) ++level;
        atomicAdd(&count[level], 1);
    }
    __syncthreads();
    if (threadIdx.x < DENDRO_LEVELS && count[threadIdx.x] != 0) atomicAdd(&w.counters[DENDRO_MERGES + threadIdx.x], count[threadIdx.x]);
}

// One merge of the sorted list: its children and what they add to the sizes.
struct Merge {
    uint32_t e;
    bool first, last;            // of its chain
    int chain, rows;             // rows that come in here
    v2i_word nodes;
};
__device__ __forceinline__ Merge merge_at(const DendrogramWork& w, const v2i_word* children, int N, int p, int begin, int end)
{
    Merge g;
    g.chain = (int)w.key_sorted[p];
    g.e = w.listed[p];
    g.first = p == begin || (int)w.key_sorted[p - 1] != g.chain;
    g.last = p + 1 == end || (int)w.key_sorted[p + 1] != g.chain;
    const v2i_word c = children[g.e];
    const int2 x = c.x >= N ? w.chain[c.x - N] : make_int2(c.x - N, 1), y = c.y >= N ? w.chain[c.y - N] : make_int2(c.y - N, 1);
    g.rows = (c.x >= 0 ? x.y : 0) + (c.y >= 0 ? y.y : 0);
    const int before = g.first ? 0 : (int)w.listed[p - 1];
    const int a = N + (c.x >= 0 ? x.x : before), b = N + (c.y >= 0 ? y.x : before);
    g.nodes = v2i_word{a < b ? a : b, a < b ? b : a};
    return g;
}

// (starts a chain, rows since) over the lanes up to this one: the chain's start cuts what comes before.
__device__ __forceinline__ void scan_lanes(bool& starts, int& rows)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int r = __shfl_up(rows, o);
        const int f = __shfl_up((int)starts, o);
        if (lane >= o && !starts) { rows += r; starts = f != 0; }
    }
}

// Merges [begin, end) of one level: children, sizes (sums along the chains), and the chains' last merges and rows.  A workgroup posts what
// its span ends on (1: no chain starts in it, so what is before it has to be added; 2: all of it) and adds what the spans before it post;
// spans are handed out in the order in which workgroups start, so whoever is waited for is running.
__global__ void __launch_bounds__(TB) k_chain_sums(DendrogramWork w, v2i_word* __restrict__ children, int32_t* __restrict__ sizes, int N,
                                                   int begin, int end, int level, unsigned long long* __restrict__ carry)
{
    __shared__ int span_at, wave_rows[TB / 64], wave_starts[TB / 64], before;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) span_at = atomicAdd(&w.counters[DENDRO_TICKET + level], 1);
    __syncthreads();
    const int span = span_at, p0 = begin + span * SUM_SPAN + tid * SUM_ITEMS;
    Merge g[SUM_ITEMS];
    int upto[SUM_ITEMS];
    bool open[SUM_ITEMS];                                   // no chain starts between the thread's first merge and this one
    int rows = 0;
    bool starts = false;
#pragma unroll
    for (int j = 0; j < SUM_ITEMS; ++j) {
        const int p = p0 + j;
        if (p < end) {
            g[j] = merge_at(w, children, N, p, begin, end);
            if (g[j].first) { rows = 0; starts = true; }
            rows += g[j].rows;
        }
        upto[j] = rows;
        open[j] = !starts;
    }
    scan_lanes(starts, rows);
    if (lane == 63) { wave_rows[wave] = rows; wave_starts[wave] = starts; }
    const int lane_rows = __shfl_up(rows, 1);
    const int lane_starts = __shfl_up((int)starts, 1);
    __syncthreads();
    if (wave == 0) {
        int all = 0, any = 0;
        for (int v = 0; v < TB / 64; ++v) { all = wave_starts[v] ? wave_rows[v] : all + wave_rows[v]; any |= wave_starts[v]; }
        if (lane == 0)
            __hip_atomic_store(&carry[span], ((any ? 2ull : 1ull) << 32) | (unsigned int)all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int sum = 0;
        const bool cut = __shfl((int)(p0 < end && g[0].first), 0) != 0;      // the span starts on a chain: nothing to look for
        for (int back = span - 1; !cut && back >= 0; back -= 64) {
            unsigned long long word = 2ull << 32;           // before the first span: nothing
            if (back - lane >= 0)
                while ((word = __hip_atomic_load(&carry[back - lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0ull) __builtin_amdgcn_s_sleep(1);
            const unsigned long long done = __ballot((word >> 32) == 2ull);
            const int stop = done ? __builtin_ctzll(done) : 63;
            int part = lane <= stop ? (int)(unsigned int)word : 0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) part += __shfl_xor(part, o);
            sum += part;
            if (done) break;
        }
        if (lane == 0) {
            before = sum;
            if (!any) __hip_atomic_store(&carry[span], (2ull << 32) | (unsigned int)(sum + all), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    // what the lanes, wavefronts and spans before this thread leave to the chain that is open where it begins
    int in = lane > 0 ? lane_rows : 0;
    bool in_starts = lane > 0 && lane_starts != 0;
    for (int v = wave - 1; v >= 0 && !in_starts; --v) { in += wave_rows[v]; in_starts = wave_starts[v] != 0; }
    if (!in_starts) in += before;
#pragma unroll
    for (int j = 0; j < SUM_ITEMS; ++j) {
        if (p0 + j >= end) break;
        const int size = upto[j] + (open[j] ? in : 0);
        children[g[j].e] = g[j].nodes;
        sizes[g[j].e] = size;
        if (g[j].last) w.chain[g[j].chain] = make_int2((int)g[j].e, size);
    }
}

// The same for the levels from `level` on, one after the other, in one workgroup; begin: the first level's first merge.
__global__ void __launch_bounds__(TB_WIDE) k_chain_sums_tail(DendrogramWork w, v2i_word* __restrict__ children, int32_t* __restrict__ sizes, int N,
                                                             int begin, int level, int depth)
{
    __shared__ int wave_rows[TB_WIDE / 64], wave_starts[TB_WIDE / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (; level <= depth; ++level) {
        const int end = begin + w.counters[DENDRO_MERGES + level];
        int before = 0;                                     // rows of the chain that is open at p0
        for (int p0 = begin; p0 < end; p0 += TB_WIDE) {
            const int p = p0 + tid;
            Merge g{};
            if (p < end) g = merge_at(w, children, N, p, begin, end);
            int rows = p < end ? g.rows : 0;
            bool starts = p < end && g.first;
            scan_lanes(starts, rows);
            if (lane == 63) { wave_rows[wave] = rows; wave_starts[wave] = starts; }
            __syncthreads();
            int in = 0, all = before;
            for (int v = 0; v < TB_WIDE / 64; ++v) {
                if (v == wave) in = all;
                all = wave_starts[v] ? wave_rows[v] : all + wave_rows[v];
            }
            before = all;
            if (p < end) {
                const int size = rows + (starts ? 0 : in);
                children[g.e] = g.nodes;
                sizes[g.e] = size;
                if (g.last) w.chain[g.chain] = make_int2((int)g.e, size);
            }
            __syncthreads();
        }
        begin = end;
    }
}

hipError_t dendrogram_chains(const int32_t* lo, const int32_t* hi, int N, const DendrogramWork& w, int32_t* children, hipStream_t s)
{
    v2i_word* c = reinterpret_cast<v2i_word*>(children);
    hipLaunchKernelGGL(k_levels_init, dim3(blocks_for(2ll * N > DENDRO_WORDS ? 2ll * N : DENDRO_WORDS, TB)), dim3(TB), 0, s, w, N, (int)dendrogram_carry_words(N));
    hipLaunchKernelGGL(k_first_edges, dim3(blocks_for(N, TB)), dim3(TB), 0, s, lo, hi, w, N);
    // a level has at most half the vertices of the one before
    int level = 0;
    for (int n = N; n > TAIL; n /= 2, ++level) {
        hipLaunchKernelGGL(k_contract, dim3(blocks_for(n, TB_WIDE)), dim3(TB_WIDE), 0, s, lo, hi, w, level, c);
        hipLaunchKernelGGL(k_next_level, dim3(blocks_for(n, TB) + blocks_for(n / 2, TB)), dim3(TB), 0, s, w, level, N);
    }
    hipLaunchKernelGGL(k_last_levels, dim3(1), dim3(TB_WIDE), 0, s, w, c, N);
    hipLaunchKernelGGL(k_chains, dim3(blocks_for(N, TB)), dim3(TB), 0, s, w, c, N);
    return hipGetLastError();
}

hipError_t dendrogram_sizes(int N, const int32_t* merges, const DendrogramWork& w, int32_t* children, int32_t* sizes, hipStream_t s)
{
    v2i_word* c = reinterpret_cast<v2i_word*>(children);
    int depth = 0;
    for (int l = 1; l < DENDRO_LEVELS; ++l) if (merges[l] > 0) depth = l;
    int begin = 0;
    size_t spans = 0;
    for (int l = 1; l <= depth; ++l) {
        if (N - 1 - begin <= SUM_TAIL) {
            hipLaunchKernelGGL(k_chain_sums_tail, dim3(1), dim3(TB_WIDE), 0, s, w, c, sizes, N, begin, l, depth);
            break;
        }
        const int end = begin + merges[l], blocks = blocks_for(merges[l], SUM_SPAN);
        if (blocks > 0) hipLaunchKernelGGL(k_chain_sums, dim3(blocks), dim3(TB), 0, s, w, c, sizes, N, begin, end, l, w.carry + spans);
        begin = end;
        spans += (size_t)blocks;
    }
    return hipGetLastError();
}

}  // namespace slhc
