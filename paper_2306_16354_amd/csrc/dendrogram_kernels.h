// Launch interface of the device dendrogram (dendrogram_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace slhc {

// Words in `counters` of DendrogramWork: an error site, the number of levels, then per level its vertices, edges, first global id, merges and ticket.
constexpr int DENDRO_LEVELS = 32;
constexpr int DENDRO_ERROR = 0, DENDRO_DEPTH = 1, DENDRO_ROWS = 32, DENDRO_EDGES = 64, DENDRO_BASE = 96, DENDRO_MERGES = 160, DENDRO_TICKET = 192, DENDRO_WORDS = 256;

// Scratch, all of it free to be overwritten: words of 32 bits, N vertices.
struct DendrogramWork {
    uint32_t* lightest;          // [2N] per vertex of every level: its first edge
    int32_t* up;                 // [2N] ... and the vertex of the next level that it becomes
    int32_t* hook;               // [N] per vertex of this level: the vertex that its first edge leads to
    uint32_t* edge[2];           // [N/4], [N/2] the edges left, of even and odd levels: number
    int2* ends[2];               // ... and end points
    uint32_t *key, *val;         // [N] per merge: its chain, its number
    uint32_t *key_sorted, *listed;   // [N] the same sorted by chain
    int2* chain;                 // [N] per chain: its last merge, the rows below that (may lie where ends[] does)
    unsigned long long* carry;   // [dendrogram_carry_words(N)]
    int32_t* counters;           // [DENDRO_WORDS]
};
size_t dendrogram_carry_words(int64_t N);

// The levels of the tree lo/hi [N - 1] (ascending by weight, end points in [0, N)): which merges make up which chain, as pairs in key / val.
// counters[DENDRO_MERGES + level] has the merges per level then.  `children` holds what dendrogram_sizes needs.
hipError_t dendrogram_chains(const int32_t* lo, const int32_t* hi, int N, const DendrogramWork& w, int32_t* children, hipStream_t s);
// Children and sizes of all merges, from the pairs sorted by chain; merges[level] (host): as in counters.
hipError_t dendrogram_sizes(int N, const int32_t* merges, const DendrogramWork& w, int32_t* children, int32_t* sizes, hipStream_t s);

}  // namespace slhc
