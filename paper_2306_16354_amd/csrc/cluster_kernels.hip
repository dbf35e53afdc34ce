// Flat clusters from a dendrogram: cut after the first N - n_clusters merges, number the surviving
// roots by ascending node id, give every row the number of the root above it (paper Sec. 3.3.2,
// Alg. "extract_flattened_clusters", Alg. "inherit_labels").
//
// The paper's inherit_labels lets every node walk up its parents until it meets a labelled one, and finds the roots by sorting the children of
// the last merges.  Here a node is a root iff it exists at the cut and nothing kept points above it, and its number is the count of roots
// before it.  Single-linkage dendrograms are often chains thousands of levels deep, and a pass in which every merge follows some links costs
// what the card can read at random (460 G words a second, 9 us for a million merges and four links).  So the merges are thinned: one of every
// eight, chosen by a hash (not by its number, whose last bits a chain may share), is one of the next stage, every merge walks towards the next such
// merge above it, of those one in sixteen does the same, and so on until few are left, whose walks are finished in LDS.  1M rows, 1000
// clusters: nine passes in which every merge followed four links took 79 of 129 us; the stages take 42 of 86, and the scattered writes of the
// links and labels most of the rest.  40 000 rows 30.5 -> 25 us.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "cluster_kernels.h"
#include "wave_ops.h"

namespace slhc {

constexpr int TB = 256;
static inline int blocks_for(long long n) { return (int)((n + TB - 1) / TB); }

// Stage r + 1 holds merge i iff its number in stage r is the one that its group of eight (r = 0) or sixteen sends up.
constexpr int group_bits(int r) { return r == 0 ? 3 : 4; }
constexpr int stage_bits(int r) { return r == 0 ? 0 : group_bits(r - 1) + stage_bits(r - 1); }
template <int r> __device__ __forceinline__ unsigned int sent_up(unsigned int group)
{
    unsigned int h = group * 0x9e3779b1u;
    h = (h ^ (h >> 15)) * 0x85ebca6bu;
    return (h ^ (h >> 13)) & ((1u << group_bits(r)) - 1u);
}
// number n of stage r in stage 0, and whether it is in stage r of what is number n of stage `from`
template <int r> __device__ __forceinline__ unsigned int stage_merge(unsigned int n)
{
    if constexpr (r == 0) return n;
    else return stage_merge<r - 1>((n << group_bits(r - 1)) + sent_up<r - 1>(n));
}
template <int r, int from = 0> __device__ __forceinline__ bool in_stage(unsigned int n)
{
    if constexpr (from == r) return true;
    else {
        const unsigned int group = n >> group_bits(from);
        return sent_up<from>(group) == (n & ((1u << group_bits(from)) - 1u)) && in_stage<r, from + 1>(group);
    }
}
// Links that a merge follows per stage.  A wavefront walks as long as its longest, and what is left is walked later, so a few less than
// the walks' mean: 6 and 12; 1M rows 85.8 us, 8 and 12 88, 12 and 20 (with groups of 4 and 8) 95.7; groups of 8, 16, 8 86.9; of 4, 8, 8 91.7; of 16, 16, 4 93.5.
constexpr int most_links(int r) { return r == 0 ? 6 : 12; }
constexpr int TOP_MAX = 16384;       // merges of the last stage in LDS, a word each: the third stage up to 33 million merges

// above[i]: the merge above merge i, itself for a root, -1 - number once it is known.  joined[v]: whether a kept merge has row v as a child.
__global__ void __launch_bounds__(TB) k_cut_init(int32_t* __restrict__ above, int kept, uint32_t* __restrict__ joined, int words,
                                                 int32_t* __restrict__ open)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *open = 0;
    const int v = (blockIdx.x * TB + threadIdx.x) * 4;
    if (v + 3 < kept) *reinterpret_cast<int4*>(above + v) = make_int4(v, v + 1, v + 2, v + 3);
    else
        for (int i = v; i < kept; ++i) above[i] = i;
    if (v / 4 < words) joined[v / 4] = 0u;
}

// A child whose merge is kept has one parent, so each word has one writer.  Rows are marked by a byte: 1 MB of marks takes the scattered
// writes of 1M rows better than 4 MB of links.  A well-formed dendrogram only joins nodes that already exist; anything else is ignored.
__global__ void __launch_bounds__(TB) k_cut_links(const v2i_word* __restrict__ children, int N, int kept, int32_t* __restrict__ above,
                                                  unsigned char* __restrict__ joined)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i >= kept) return;
    const v2i_word c = children[i];
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int v = side ? c.y : c.x;
        if ((unsigned int)v >= (unsigned int)(N + i)) continue;
        if (v < N) joined[v] = 1;
        else above[v - N] = i;
    }
}

// Merge i of stage R walks to the next merge of stage R + 1 above it, or to its root.  Links lead to higher merges, so walks end; reading a
// link that another thread has already advanced only gets there sooner.
template <int R>
__device__ __forceinline__ void walk_up(int32_t* above, int kept, unsigned int j)
{
    const unsigned int i = stage_merge<R>(j);
    if (i >= (unsigned int)kept) return;
    const int first = above[i];
    if (first < 0 || first == (int)i) return;
    int a = first;
    for (int h = 0; h < most_links(R) && !in_stage<R + 1>((unsigned int)a); ++h) {
        const int up = above[a];
        if (up == a) break;
        a = up;
        if (a < 0) break;
    }
    if (a != first) above[i] = a;
}

// Roots are counted span by span, the rows' spans first: `turns` times 16 rows or 4 merges per thread, one wide load each.
struct RootSpans {
    unsigned int N, kept, turns;
    __host__ __device__ unsigned int rows() const { return (N + turns * TB * 16 - 1) / (turns * TB * 16); }
    __host__ __device__ unsigned int all() const { return rows() + (kept + turns * TB * 4 - 1) / (turns * TB * 4); }
};
static RootSpans root_spans(unsigned int N, unsigned int kept) { return RootSpans{N, kept, 1u + (N >> 20)}; }       // 1300 spans at most

// What this thread looks at in turn t of a span: a bit per root; the first node in `at`.
__device__ __forceinline__ unsigned int root_flags(const int32_t* above, const unsigned char* joined, const RootSpans& r, unsigned int span, unsigned int t, unsigned int& at)
{
    unsigned int flags = 0;
    if (span < r.rows()) {
        at = ((span * r.turns + t) * TB + threadIdx.x) * 16;
        if (at >= r.N) return 0;
        const uint4 m = *reinterpret_cast<const uint4*>(joined + at);          // (a mark is 0 or 1)
        const unsigned int w[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) flags |= ((((w[q] ^ 0x01010101u) * 0x01020408u) >> 24) & 15u) << (4 * q);
        if (r.N - at < 16) flags &= (1u << (r.N - at)) - 1u;
    } else {
        at = (((span - r.rows()) * r.turns + t) * TB + threadIdx.x) * 4;
        if (at >= r.kept) return 0;
        const int4 a = *reinterpret_cast<const int4*>(above + at);
        flags = (a.x == (int)at) | (a.y == (int)at + 1) << 1 | (a.z == (int)at + 2) << 2 | (a.w == (int)at + 3) << 3;
        if (r.kept - at < 4) flags &= (1u << (r.kept - at)) - 1u;
    }
    return flags;
}
__device__ __forceinline__ int block_sum(int x, int* wave_part)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) x += __shfl_xor(x, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = x;
    __syncthreads();
    int all = 0;
    for (int w = 0; w < TB / 64; ++w) all += wave_part[w];
    return all;
}

// First stage; the workgroups beyond its merges count roots.
__global__ void __launch_bounds__(TB) k_cut_first(int32_t* __restrict__ above, const unsigned char* __restrict__ joined, RootSpans r,
                                                  int walkers, int32_t* __restrict__ counts)
{
    __shared__ int part[TB / 64];
    if ((int)blockIdx.x < walkers) { walk_up<0>(above, (int)r.kept, blockIdx.x * TB + threadIdx.x); return; }
    const unsigned int span = blockIdx.x - walkers;
    int n = 0;
    for (unsigned int t = 0, at; t < r.turns; ++t) n += __popc(root_flags(above, joined, r, span, t, at));
    n = block_sum(n, part);
    if (threadIdx.x == 0) counts[span] = n;
}

// Second stage; the workgroups beyond its merges number the roots.  (A walk may find a root with or without its number.)
__global__ void __launch_bounds__(TB) k_cut_second(int32_t* __restrict__ above, const unsigned char* __restrict__ joined, RootSpans r,
                                                   int walkers, const int32_t* __restrict__ counts, int32_t* __restrict__ labels)
{
    __shared__ int part[TB / 64];
    if ((int)blockIdx.x < walkers) { walk_up<1>(above, (int)r.kept, blockIdx.x * TB + threadIdx.x); return; }
    const unsigned int span = blockIdx.x - walkers;
    if (counts[span] == 0) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int before = 0;
    for (unsigned int s = threadIdx.x; s < span; s += TB) before += counts[s];
    before = block_sum(before, part);
    for (unsigned int t = 0; t < r.turns; ++t) {
        unsigned int v0 = 0;
        unsigned int flags = root_flags(above, joined, r, span, t, v0);
        int upto = __popc(flags);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(upto, o);
            if (lane >= o) upto += x;
        }
        __syncthreads();
        if (lane == 63) part[wave] = upto;
        __syncthreads();
        int at = before + upto - __popc(flags);
        for (int w = 0; w < TB / 64; ++w) {
            if (w < wave) at += part[w];
            before += part[w];
        }
        for (; flags; flags &= flags - 1, ++at) {
            const unsigned int v = v0 + __builtin_ctz(flags);
            if (span < r.rows()) labels[v] = at;
            else above[v] = -1 - at;
        }
    }
}

template <int R>
__global__ void __launch_bounds__(TB) k_cut_stage(int32_t* __restrict__ above, int kept)
{
    walk_up<R>(above, kept, blockIdx.x * TB + threadIdx.x);
}

// What is left of the last stage, in LDS by its numbers there: walks over links of four until every one has its root's number.  A merge that no
// merge of the stage lies near above, and those that lead to it, are left as they are.
constexpr int NEAR_LINKS = 64, LEFT_OPEN = -2147483647 - 1;
template <int STAGES>
__global__ void __launch_bounds__(1024) k_cut_top(int32_t* __restrict__ above, int kept, int n)
{
    extern __shared__ int link[];
    volatile int* at = link;
    for (int j = threadIdx.x; j < n; j += 1024) {
        const unsigned int i = stage_merge<STAGES>((unsigned int)j);
        int a = LEFT_OPEN;
        if (i < (unsigned int)kept) {
            a = above[i];
            for (int h = 0; a >= 0 && !in_stage<STAGES>((unsigned int)a); ++h) a = h < NEAR_LINKS ? above[a] : LEFT_OPEN;
            if (a >= 0) a >>= stage_bits(STAGES);
        }
        at[j] = a;
    }
    for (;;) {
        __syncthreads();
        int open = 0;
        for (int j = threadIdx.x; j < n; j += 1024) {
            int a = at[j];
            if (a < 0) continue;
            for (int h = 0; h < 4 && a >= 0; ++h) a = at[a];
            at[j] = a;
            open |= a >= 0;
        }
        if (!__syncthreads_or(open)) break;
    }
    for (int j = threadIdx.x; j < n; j += 1024) {
        const unsigned int i = stage_merge<STAGES>((unsigned int)j);
        if (at[j] != LEFT_OPEN) above[i] = at[j];
    }
}

// Every merge's rows take the number at the end of its walk, one link per stage as a rule.  A chain may avoid the merges that the hash sends up,
// whatever the hash is; where a walk is not through after NEAR_LINKS links, *open says so.
__global__ void __launch_bounds__(TB) k_cut_labels(const v2i_word* __restrict__ children, int N, int kept, const int32_t* __restrict__ above,
                                                   int32_t* __restrict__ labels, int32_t* __restrict__ open)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i >= kept) return;
    const v2i_word c = children[i];
    const bool x = (unsigned int)c.x < (unsigned int)N, y = (unsigned int)c.y < (unsigned int)N;
    if (!x && !y) return;
    int a = above[i];
#pragma unroll 1
    for (int h = 0; a >= 0 && h < NEAR_LINKS; ++h) a = above[a];
    if (a >= 0) { *open = 1; return; }
    if (x) labels[c.x] = -1 - a;
    if (y) labels[c.y] = -1 - a;
}

// Then all merges again, OPEN_SPAN at a time from the last down: what lies above a span is done, and in it every merge keeps where it got to after
// each few links, so links grow as many times each time and a span takes a dozen turns at most.  (Past the caches, which may hold older links.)  Chains that
// avoid all of stage 1, with walks of any length in the launches before: 20 000 rows 630 us, 60 000 2014, so 40 000 72 and 300 000 124, where a plain chain
// takes 49.  Where nothing is open the launch costs 1.7 us (1M rows 85.6 and 87.3).
constexpr int OPEN_BLOCKS = 256, OPEN_SPAN = OPEN_BLOCKS * TB, OPEN_LINKS = 4;
__global__ void __launch_bounds__(TB) k_cut_open(const v2i_word* __restrict__ children, int N, int kept, int32_t* above, int32_t* __restrict__ labels,
                                                 const int32_t* __restrict__ open)
{
    if (*open == 0) return;
    for (int i = kept - 1 - (int)(blockIdx.x * TB + threadIdx.x); i >= 0; i -= OPEN_SPAN) {
        int a = above[i];
        // (one loop, not one of OPEN_LINKS steps inside another: from that the compiler, clang 22 of ROCm 7.2, makes a loop whose lanes that ended in an
        // earlier step than others go on)
        for (int h = 1; a >= 0; ++h) {
            a = __hip_atomic_load(above + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (h % OPEN_LINKS == 0) __hip_atomic_store(above + i, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const v2i_word c = children[i];
        if ((unsigned int)c.x < (unsigned int)N) labels[c.x] = -1 - a;
        if ((unsigned int)c.y < (unsigned int)N) labels[c.y] = -1 - a;
    }
}

// All of it for at most FLAT_SMALL rows, in one workgroup with 16-bit links in LDS: the five to ten launches above cost more
// than what they do.  64 rows 18.6 -> 8.6 us, 3000 rows 26 -> 11.4, 8000 rows 28.8 -> 22.5; at 16 000 rows one workgroup
// takes 45 us against 28, so the line is drawn below that.
constexpr int FLAT_SMALL = 8192;
__global__ void __launch_bounds__(1024) k_flat_small(const int32_t* __restrict__ children, int N, int kept, int32_t* __restrict__ labels)
{
    extern __shared__ __align__(16) unsigned char flat_smem[];
    __shared__ int wave_sum[16];
    volatile unsigned short* above = reinterpret_cast<volatile unsigned short*>(flat_smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int limit = N + kept;                             // the nodes that exist at the cut
    for (int v = tid; v < limit; v += 1024) above[v] = (unsigned short)v;
    __syncthreads();
    for (int i = tid; i < kept; i += 1024) {
        const int a = children[2 * i], b = children[2 * i + 1];
        if ((unsigned int)a < (unsigned int)(N + i)) above[a] = (unsigned short)(N + i);
        if ((unsigned int)b < (unsigned int)(N + i)) above[b] = (unsigned short)(N + i);
    }
    // doubling, until nothing moves (links lead upwards, so it ends)
    for (int pass = 0; pass < 17; ++pass) {
        __syncthreads();
        int moved = 0;
        for (int v = N + tid; v < limit; v += 1024) {
            const unsigned int a = above[v], aa = above[a], a4 = above[aa];
            if (a4 != a) { above[v] = (unsigned short)a4; moved = 1; }
        }
        if (!__syncthreads_or(moved)) break;
    }
    // roots numbered by node id: a run of nodes per thread, a prefix sum over the threads
    const int per = (limit + 1023) / 1024;
    const int v0 = tid * per < limit ? tid * per : limit, v1 = v0 + per < limit ? v0 + per : limit;
    int mine = 0;
    for (int v = v0; v < v1; ++v) mine += above[v] == v ? 1 : 0;
    int upto = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(upto, o);
        if (lane >= o) upto += x;
    }
    if (lane == 63) wave_sum[wave] = upto;
    for (int v = tid; v < N; v += 1024) labels[v] = above[above[v]];
    __syncthreads();
    int at = upto - mine;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
    for (int v = v0; v < v1; ++v)                           // (a run has one writer, and nobody reads links any more)
        if (above[v] == v) above[v] = (unsigned short)(at++);
    __syncthreads();
    for (int v = tid; v < N; v += 1024) labels[v] = above[labels[v]];
}

// Stage R of n merges and those after it.
template <int R>
static void cut_stages(int32_t* above, int kept, unsigned int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_cut_stage<R>, dim3(blocks_for(n)), dim3(TB), 0, s, above, kept);
    const unsigned int up = (n + (1u << group_bits(R)) - 1) >> group_bits(R);
    if constexpr (R < 4) {
        if (up > TOP_MAX) { cut_stages<R + 1>(above, kept, up, s); return; }
    }
    hipLaunchKernelGGL(k_cut_top<R + 1>, dim3(1), dim3(1024), (size_t)up * 4, s, above, kept, (int)up);     // (2^30 merges: 2048 of stage 5)
}

size_t flat_clusters_counts(int64_t N) { return (size_t)root_spans((unsigned int)N, (unsigned int)N).all() + 1; }

hipError_t flat_clusters(const int32_t* children, int N, int n_clusters, int32_t* labels, int32_t* above, unsigned char* joined,
                         int32_t* counts, hipStream_t s)
{
    const int kept = N - n_clusters;
    if (N <= FLAT_SMALL) {
        const size_t lds = (size_t)(N + kept) * 2;
        hipLaunchKernelGGL(k_flat_small, dim3(1), dim3(1024), lds, s, children, N, kept, labels);
        return hipGetLastError();
    }
    const v2i_word* c = reinterpret_cast<const v2i_word*>(children);
    int32_t* open = counts + flat_clusters_counts(N) - 1;
    const int words = (N + 3) / 4, quads = (kept + 3) / 4;
    hipLaunchKernelGGL(k_cut_init, dim3(blocks_for(words > quads ? words : quads)), dim3(TB), 0, s, above, kept, reinterpret_cast<uint32_t*>(joined), words, open);
    if (kept > 0) hipLaunchKernelGGL(k_cut_links, dim3(blocks_for(kept)), dim3(TB), 0, s, c, N, kept, above, joined);
    const RootSpans spans = root_spans((unsigned int)N, (unsigned int)kept);
    const unsigned int stage1 = ((unsigned int)kept + (1u << group_bits(0)) - 1) >> group_bits(0);
    hipLaunchKernelGGL(k_cut_first, dim3(blocks_for(kept) + (int)spans.all()), dim3(TB), 0, s, above, joined, spans, blocks_for(kept), counts);
    hipLaunchKernelGGL(k_cut_second, dim3(blocks_for(stage1) + (int)spans.all()), dim3(TB), 0, s, above, joined, spans, blocks_for(stage1), counts, labels);
    if (kept > 0) {
        cut_stages<2>(above, kept, (stage1 + (1u << group_bits(1)) - 1) >> group_bits(1), s);
        hipLaunchKernelGGL(k_cut_labels, dim3(blocks_for(kept)), dim3(TB), 0, s, c, N, kept, above, labels, open);
        hipLaunchKernelGGL(k_cut_open, dim3(OPEN_BLOCKS), dim3(TB), 0, s, c, N, kept, above, labels, open);
    }
    return hipGetLastError();
}

}  // namespace slhc
