// Launch interface of the Boruvka forest kernels and the edge sort (forest_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace slhc {

// Device state of the minimum-spanning-forest construction.  Components are named by the index
// of their root vertex ("colour", paper Sec. 3.2.3); per-component arrays are indexed by it.
struct ForestState {
    int N, k;
    const int32_t* nbr_idx;      // [N, k] ascending by (dist, idx)
    const float* nbr_dist;       // [N, k]
    int32_t* colour;             // [N]
    int32_t* ptr;                // [N] entries before ptr[v] are known to share v's colour
    // what the last cross-component query of v left: a row it reaches (-1: none) and its distance.  ext_low +inf: that row
    // is v's nearest foreign one (or, without a row, ext_dist a lower bound); else a lower bound on the nearest
    int32_t* ext_idx;            // [N]
    float* ext_dist;             // [N]
    float* ext_low;              // [N]
    float* cand_w;               // [N] weight of v's lightest outgoing edge, or a lower bound
    int32_t* cand_u;             // [N] its other endpoint, or -1 when only the bound is known
    uint32_t* best_w;            // [N] per component: min weight bits over exact candidates
    unsigned long long* best_e;  // [N] per component: min (lo << 32 | hi) among those of best_w
    int32_t* hook;               // [N] per component: component it attaches to this round
    int32_t* qlist;              // [N] rows sent to the cross-component 1-NN
    int32_t* counters;           // 0 = queries this round, 1 = edges so far, 2 = a hook chain waits for the host,
                                 // 3 = site of the first failed index check (0 = none), 6 = rounds (forest_small)
    int32_t* e_lo;               // [N-1] committed edges
    int32_t* e_hi;
    float* e_w;
};

hipError_t forest_init(const ForestState& f, hipStream_t s);
hipError_t forest_scan_lists(const ForestState& f, hipStream_t s);
hipError_t forest_classify(const ForestState& f, hipStream_t s);
// qrows[q] is the vertex query q was made for (f.qlist, or a reordered copy of it).  `thresholds`
// (or nullptr): the per-component thresholds the sweep ran under (SweepParams::comp_best); answers
// farther than their component's threshold are kept as a lower bound and an edge.  `q_low` (or nullptr): distances
// below which a query has no foreign row.
hipError_t forest_apply_queries(const ForestState& f, const int32_t* qrows, const int32_t* q_idx,
                                const float* q_dist, const float* q_low, int nq, const uint32_t* thresholds, hipStream_t s);
// Two-phase connection sweeps (n > 0): rows of `list` in every `stride`-th 128-row panel of the row
// order (inv[v] = position of row v) go to part_a, the others to part_b; counts[0], counts[1] (zeroed by
// the caller) receive the part sizes.  forest_still_needed keeps the rows of `list` that the test of
// forest_classify would still list after best_w has dropped; *count zeroed by the caller.
hipError_t forest_split_queries(const ForestState& f, const int32_t* list, int n, const int32_t* inv, int stride,
                                int32_t* part_a, int32_t* part_b, int32_t* counts, hipStream_t s);
hipError_t forest_still_needed(const ForestState& f, const int32_t* list, int n, int32_t* out, int32_t* count,
                               hipStream_t s);
hipError_t forest_select_edges(const ForestState& f, hipStream_t s);
// sizes[c] += 1 for every entry c of colour[0..n) inside [0, bins); sizes zeroed by the caller.  One atomic
// per colour and wavefront where neighbouring entries share their colour.
hipError_t forest_component_sizes(const int32_t* colour, int n, int bins, int32_t* sizes, hipStream_t s);
hipError_t forest_commit(const ForestState& f, hipStream_t s);
// Every component root follows the hooks up to `steps` components far and hooks itself there; with
// `flag`, counters[2] is set when some root has not reached the end of its chain.
hipError_t forest_jump(const ForestState& f, int steps, bool flag, hipStream_t s);
// colour[v] = end of the chain of hooks from colour[v]; the per-component minima are cleared for the next round.  A chain
// longer than 64 hooks sets counters[2], and the rounds enqueued behind do nothing: the host finishes the chains
// (forest_jump), clears the word and calls again.
hipError_t forest_follow(const ForestState& f, hipStream_t s);
// counters[0 .. 7] to host memory (host[1 ..]) and then `seq` to host[0].
hipError_t forest_publish(const ForestState& f, int32_t* host, int32_t seq, hipStream_t s);
// Rounds of a small forest in one launch, until it is complete or rows have to be queried (counters[0] of them in qlist).
constexpr int FOREST_SMALL_MAX = 12288;
hipError_t forest_small(const ForestState& f, bool first, hipStream_t s);

// Sort E edges ascending by (w, lo, hi).  keys/vals are scratch of E elements each; `temp` of
// edge_sort_temp_bytes(E).  Result in out_lo/out_hi/out_w.
// Copies of the sorted edges (each nullptr for none): the weights as heights, the end points in host memory.
struct EdgeCopies { float* heights; int32_t* host_lo; int32_t* host_hi; };
size_t edge_sort_temp_bytes(int E);
hipError_t edge_sort(const int32_t* lo, const int32_t* hi, const float* w, int E, int N /* ids are below N */,
                     unsigned long long* keys_a, unsigned long long* keys_b,
                     uint32_t* vals_a, uint32_t* vals_b, void* temp, size_t temp_bytes,
                     int32_t* out_lo, int32_t* out_hi, float* out_w, const EdgeCopies& copies, hipStream_t s);

// Children and sizes of E merges from host memory.
hipError_t linkage_upload(const int32_t* cj, const int32_t* sj, int E, int32_t* children, int32_t* sizes, hipStream_t s);

// Stable sort of n (key, value) pairs of 32-bit words by key (keys below 2^key_bits).
size_t pair_sort_temp_bytes(int n);
hipError_t pair_sort_u32(const uint32_t* keys_in, uint32_t* keys_out, const uint32_t* vals_in,
                         uint32_t* vals_out, int n, int key_bits, void* temp, size_t temp_bytes,
                         hipStream_t s);

}  // namespace slhc
