// Flat clusters from a dendrogram: cut after the first N - n_clusters merges, number the surviving
// roots by ascending node id, give every row the number of the root above it (paper Sec. 3.3.2,
// Alg. "extract_flattened_clusters", Alg. "inherit_labels").
//
// The paper's inherit_labels lets every node walk up its parents until it meets a labelled one.
// Single-linkage dendrograms are often chains thousands of levels deep, so here the walk is cut into passes: in each,
// every merge follows a few links and keeps where it got to, so a pass divides the remaining depth by that number; rows are
// linked once and look their end up last.  1M rows: 202 us with doubling over all 2N nodes (21 passes), then 160, 138, 133
// and 140 us with 2, 3, 4 and 8 links; 40 000 rows: 58, 45, 38 and 30.5 us.  So eight links, where a pass costs its launch,
// and four at the size where its walks do; the line at a quarter million merges lies between the two sizes timed.
// The paper finds the roots by sorting the children of the last merges; here a node is a root iff
// it exists at the cut and nothing kept points above it, and the numbering is an exclusive prefix
// sum of that flag over the node ids (the same ascending order, no sort).
#include <hip/hip_runtime.h>
#include <cstring>
#include <rocprim/rocprim.hpp>
#include <stdint.h>
#include "cluster_kernels.h"

namespace slhc {

constexpr int TB = 256;
static inline int blocks_for(long long n) { return (int)((n + TB - 1) / TB); }


// above[v] = v, and merge i < kept puts node N+i above its two children.  A child whose merge is kept is below N + kept, so
// each word has one writer: the thread of a node that is nobody's kept child, or that of its merge (`self` first).
__global__ void __launch_bounds__(TB) k_above_self(int32_t* __restrict__ above, int nodes)
{
    const int v = (blockIdx.x * TB + threadIdx.x) * 4;
    if (v + 3 < nodes) *reinterpret_cast<int4*>(above + v) = make_int4(v, v + 1, v + 2, v + 3);
    else
        for (int i = v; i < nodes; ++i) above[i] = i;
}

__global__ void __launch_bounds__(TB) k_above_kept(const int32_t* __restrict__ children, int N, int kept,
                                                   int32_t* __restrict__ above)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i >= kept) return;
    const int a = children[2 * i], b = children[2 * i + 1];
    // a well-formed dendrogram only joins nodes that already exist; anything else is ignored
    if ((unsigned int)a < (unsigned int)(N + i)) above[a] = N + i;
    if ((unsigned int)b < (unsigned int)(N + i)) above[b] = N + i;
}

// a node that exists at the cut (v < limit) and has nothing above it is a root
struct RootFlag {
    const int32_t* above;
    int limit;
    __host__ __device__ int32_t operator()(int v) const { return v < limit && above[v] == v ? 1 : 0; }
};

// Merges only (nodes from N on): a row is linked once and looks its end up in k_labels.  Reading a value another thread
// has already advanced only gets there sooner; links lead to higher nodes, so walks end.
__global__ void __launch_bounds__(TB) k_above_follow(int32_t* __restrict__ above, int N, int limit, int hops)
{
    const int v = N + blockIdx.x * TB + threadIdx.x;
    if (v >= limit) return;
    const int first = above[v];
    int a = first;
    for (int h = 1; h < hops; ++h) {
        const int up = above[(unsigned int)a < (unsigned int)limit ? a : v];
        if (up == a) break;
        a = up;
    }
    if (a != first) above[v] = a;
}

// the last walk, and the label at its end
__global__ void __launch_bounds__(TB) k_labels(const int32_t* __restrict__ above, const int32_t* __restrict__ rank,
                                               int N, int nodes, int hops, int32_t* __restrict__ labels)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v >= N) return;
    int r = above[v];
    for (int h = 0; h < hops && (unsigned int)r < (unsigned int)nodes; ++h) {
        const int up = above[r];
        if (up == r) break;
        r = up;
    }
    labels[v] = (unsigned int)r < (unsigned int)nodes ? rank[r] : -1;
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

static auto root_flags(const int32_t* above, int limit)
{
    return rocprim::make_transform_iterator(rocprim::make_counting_iterator<int>(0), RootFlag{above, limit});
}

size_t flat_clusters_scan_temp_bytes(int N)
{
    size_t bytes = 0;
    int32_t* out = nullptr;
    (void)rocprim::exclusive_scan(nullptr, bytes, root_flags(nullptr, 0), out, 0, (size_t)(2 * (size_t)N), rocprim::plus<int32_t>());
    return bytes;
}

hipError_t flat_clusters(const int32_t* children, int N, int n_clusters, int32_t* labels, int32_t* above,
                         int32_t* rank, void* scan_temp, size_t scan_temp_bytes, hipStream_t s)
{
    const int nodes = 2 * N - 1;
    const int kept = N - n_clusters;
    if (N <= FLAT_SMALL) {
        const size_t lds = (size_t)(N + kept) * 2;
        hipLaunchKernelGGL(k_flat_small, dim3(1), dim3(1024), lds, s, children, N, kept, labels);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_above_self, dim3(blocks_for((nodes + 3) / 4)), dim3(TB), 0, s, above, nodes);
    if (kept > 0)
        hipLaunchKernelGGL(k_above_kept, dim3(blocks_for(kept)), dim3(TB), 0, s, children, N, kept, above);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = rocprim::exclusive_scan(scan_temp, scan_temp_bytes, root_flags(above, N + kept), rank, 0, (size_t)nodes, rocprim::plus<int32_t>(), s);
    if (e != hipSuccess) return e;
    // nodes from N + kept on were never linked; k_labels takes the last links
    const int hops = kept > (1 << 18) ? 4 : 8;
    long long reach = hops;
    for (; reach < (long long)kept + 1; reach *= hops)
        hipLaunchKernelGGL(k_above_follow, dim3(blocks_for(kept)), dim3(TB), 0, s, above, N, N + kept, hops);
    hipLaunchKernelGGL(k_labels, dim3(blocks_for(N)), dim3(TB), 0, s, above, rank, N, nodes, hops, labels);
    return hipGetLastError();
}

}  // namespace slhc
