// Boruvka minimum spanning forest over cached sorted neighbour lists, with colours instead of
// graph contraction (cuSLINK paper Sec. 3.2: Alg. "MST Algorithm", "Minimum incident edges",
// "Label Propagation"), plus the weight sort of Sec. 3.3.1.
//
// Differences from the paper's kernels, all deliberate:
//   * No weight alteration (Sec. 3.2.1).  Ties are broken by the strict order
//     (weight, min endpoint, max endpoint) on undirected edges, which also handles zero weights
//     and exact duplicates, where a random perturbation below the smallest weight gap cannot work.
//     A component's minimum is found in two atomic passes: 32-bit min over weight bits, then
//     64-bit min over (lo, hi) among the edges of that weight.
//   * The lists are the directed k-NN lists, already ascending, so "minimum edge per vertex" is
//     the first entry of another colour: one lane per entry, one ballot, no reduction tree.
//   * A vertex whose whole list shares its colour contributes a lower bound (its k-th distance,
//     or its last cross-component 1-NN distance) instead of an edge; the host commits a
//     component's edge only when it beats every such bound, and queries the rest.  This is what
//     makes the result the minimum spanning tree of the complete graph and not just of the
//     k-NN graph.
//   * Relabelling is pointer doubling over component roots, then one gather per vertex, instead
//     of iterated atomicMin colour exchange (Alg. "min_pair_colors" / "update_colors").
#include <hip/hip_runtime.h>
#include <cstring>
#include <rocprim/rocprim.hpp>
#include <stdint.h>
#include "forest_kernels.h"
#include "wave_ops.h"

namespace slhc {

constexpr uint32_t INF_BITS = 0x7f800000u;
constexpr int TB = 256;
constexpr int FOLLOW_STEPS = 64;       // hooks a vertex follows in one launch of k_follow

static inline int blocks_for(long long n) { return (int)((n + TB - 1) / TB); }

// Every index that comes out of device memory is range-checked before it is used as an address.
// A failed check records its site in counters[3] (the host turns that into SLHC_INTERNAL) and the
// access is skipped, so corrupt state can never become an out-of-bounds access.
__device__ inline bool in_range(int i, int n) { return (unsigned int)i < (unsigned int)n; }
__device__ inline void report(const ForestState& f, int site) { atomicCAS(&f.counters[3], 0, site); }
// The first failed check of a state error also leaves what it saw in counters[16..23], for the host's message.
__device__ inline void report_with(const ForestState& f, int site, int a, int b, int c, int d, int e, int g)
{
    if (atomicCAS(&f.counters[3], 0, site) == 0) {
        f.counters[16] = site; f.counters[17] = a; f.counters[18] = b; f.counters[19] = c;
        f.counters[20] = d; f.counters[21] = e; f.counters[22] = g;
    }
}

// While a hook chain of an earlier round waits for the host, what is enqueued behind does nothing.
__device__ inline bool forest_halted(const ForestState& f) { return f.counters[2] != 0; }

__global__ void __launch_bounds__(TB) k_forest_init(ForestState f)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v < 8) f.counters[v] = 0;          // before the range test: N may be smaller than 4
    if (v >= f.N) return;
    f.colour[v] = v;
    f.ptr[v] = 0;
    f.ext_idx[v] = -1;
    f.ext_dist[v] = 0.f;
    f.ext_low[v] = __builtin_inff();
    f.best_w[v] = INF_BITS;
    f.best_e[v] = ~0ull;
}

// G lanes per vertex walk its list from ptr[v] on, G entries at a time, until an entry of another colour
// turns up: the lists are ascending, so that entry is the vertex's lightest listed outgoing edge.  Most
// vertices find it in their first step (in the first round entry 0 always is foreign), and ptr only moves
// forward over the rounds, so the colour gathers summed over all rounds stay near N * (k + G * rounds)
// instead of N * k * rounds with one lane per entry.
template <int G>
__global__ void __launch_bounds__(TB) k_scan_lists(ForestState f)
{
    // the scan for the next round is enqueued before the host knows that the tree is complete, or that a hook chain is
    // left to it
    if (f.counters[1] >= f.N - 1 || forest_halted(f)) return;
    const int gid = (int)(((long long)blockIdx.x * TB + threadIdx.x) / G);
    const int j = threadIdx.x & (G - 1);
    const int lane = threadIdx.x & 63;
    const bool live = gid < f.N;
    const int v = live ? gid : 0;
    const int c = f.colour[v];
    int found = -1;
    for (int base = f.ptr[v];; base += G) {
        const bool more = live && base < f.k && found < 0;        // the same for the G lanes of a vertex
        if (!__any(more)) break;
        bool foreign = false;
        const int e = base + j;
        if (more && e < f.k) {
            const int u = f.nbr_idx[(size_t)v * f.k + e];
            if (in_range(u, f.N)) foreign = f.colour[u] != c;
            else report(f, 1);
        }
        unsigned long long mask = __ballot(foreign);
        mask = (mask >> (lane & ~(G - 1))) & ((1ull << G) - 1ull);
        if (more && mask) found = base + __builtin_ctzll(mask);
    }
    const bool head = live && j == 0;
    bool exact = false;
    uint32_t wbits = INF_BITS;
    if (head && !in_range(c, f.N)) report(f, 2);
    else if (head) {
        if (found >= 0) {
            const float w = f.nbr_dist[(size_t)v * f.k + found];
            f.ptr[v] = found;
            f.cand_w[v] = w;
            f.cand_u[v] = f.nbr_idx[(size_t)v * f.k + found];
            wbits = __float_as_uint(w);
            exact = true;
        } else {
            f.ptr[v] = f.k;
            const int eu = f.ext_idx[v];
            const float ed = f.ext_dist[v], el = f.ext_low[v];
            const bool edge = eu >= 0 && eu < f.N && f.colour[eu] != c;
            if (eu >= f.N) report(f, 3);
            else if (edge && !(el < __builtin_inff())) {      // cached answer still leads out of the component
                f.cand_w[v] = ed;
                f.cand_u[v] = eu;
                wbits = __float_as_uint(ed);
                exact = true;
            } else {
                // lower bounds on v's nearest foreign point: its k-th list distance, and whatever the last
                // cross-component query left (an exact answer that has since joined v's component, or what a
                // truncated search knows; 0 when never queried)
                float lb = f.nbr_dist[(size_t)v * f.k + f.k - 1];
                lb = fmaxf(lb, fminf(ed, el));
                f.cand_w[v] = lb;
                f.cand_u[v] = -1;
                // an edge out of the component that need not be v's lightest still bounds the component's lightest; a
                // component whose bound it stays will query v, whose own bound is not above it
                if (edge) { wbits = __float_as_uint(ed); exact = true; }
            }
        }
    }
    wave_min_into(f.best_w, c, wbits, exact);
}

// Vertices that only know a lower bound and whose bound does not exceed their component's best
// exact weight must be queried (<=, so that weight ties are resolved by the edge order).
constexpr int TB_WIDE = 1024;
__global__ void __launch_bounds__(TB_WIDE) k_classify(ForestState f)
{
    const int v = blockIdx.x * TB_WIDE + threadIdx.x;
    bool need = false;
    if (f.counters[1] >= f.N - 1 || forest_halted(f)) return;                // (workgroup-uniform)
    if (v < f.N && f.cand_u[v] < 0) {
        const int c = f.colour[v];
        if (in_range(c, f.N)) need = __float_as_uint(f.cand_w[v]) <= f.best_w[c];
        else report(f, 4);
    }
    const int slot = block_append<TB_WIDE>(need, &f.counters[0]);
    if (need) {
        if (in_range(slot, f.N)) f.qlist[slot] = v;
        else report(f, 5);
    }
}

// `thresholds` (optional): the queries ran under their component's shared threshold, which started at the
// lightest outgoing edge the lists already knew and which the sweep lowered whenever one of the
// component's queries found a lighter one; thresholds[colour] is its value after the sweep, F.  A query's
// tiles were filtered under values that were never below F, so every candidate at most F away was
// examined: an answer at distance <= F is the query's exact nearest foreign row.  Any other query only
// learns that no foreign row is nearer than F: it keeps no candidate, and F becomes its lower bound for the
// following rounds (components only grow).  F = min(start value, lightest edge from a queried row of the
// component to a foreign row) does not depend on the order in which the panels ran.
// Such a query's answer, if it has one, is an edge all the same.
__global__ void __launch_bounds__(TB) k_apply_queries(ForestState f, const int32_t* __restrict__ qrows,
                                                      const int32_t* __restrict__ q_idx,
                                                      const float* __restrict__ q_dist, const float* __restrict__ q_low, int nq,
                                                      const uint32_t* __restrict__ thresholds)
{
    const int q = blockIdx.x * TB + threadIdx.x;
    bool found = false;
    int c = 0;
    float w = 0.f;
    if (q < nq) {
        const int v = qrows[q];
        const int u = q_idx[q];
        w = q_dist[q];
        if (!in_range(v, f.N) || u < -1 || u >= f.N || !in_range(f.colour[v], f.N)) report(f, 6);
        else {
            c = f.colour[v];
            // an answer inside the query's own component can only come from a broken sweep
            if (u >= 0 && f.colour[u] == c) report_with(f, 14, q, v, u, c, (int)__float_as_uint(w), nq);
            bool exact = true;
            if (thresholds) {
                const uint32_t fb = thresholds[c];
                if (!(u >= 0 && __float_as_uint(w) <= fb)) {
                    float low = fmaxf(__uint_as_float(fb), fminf(f.ext_dist[v], f.ext_low[v]));
                    if (q_low && q_low[q] < __builtin_inff()) low = fmaxf(low, q_low[q]);
                    const bool edge = u >= 0 && low < __builtin_inff();
                    f.ext_idx[v] = edge ? u : -1;
                    f.ext_dist[v] = edge ? w : low;
                    f.ext_low[v] = edge ? low : __builtin_inff();
                    f.cand_u[v] = -1;
                    f.cand_w[v] = low;
                    exact = false;
                }
            }
            if (exact) {
                f.ext_idx[v] = u;
                f.ext_dist[v] = w;
                f.ext_low[v] = __builtin_inff();
                f.cand_u[v] = u;
                f.cand_w[v] = w;
                found = u >= 0;
            }
        }
    }
    wave_min_into(f.best_w, c, __float_as_uint(w), found);
}

// Two-phase connection sweeps.  k_split_queries sends the listed rows whose 128-row panel in the row
// order is a sampled one (every `stride`-th panel) to part A and the others to part B.  After the
// sweep over part A has lowered best_w, k_still_needed keeps of part B only the rows whose bound still
// does not exceed their component's best exact weight (the test of k_classify again).
__global__ void __launch_bounds__(TB) k_split_queries(ForestState f, const int32_t* __restrict__ list, int n,
                                                      const int32_t* __restrict__ inv, int stride,
                                                      int32_t* __restrict__ part_a, int32_t* __restrict__ part_b,
                                                      int32_t* __restrict__ counts)
{
    const int q = blockIdx.x * TB + threadIdx.x;
    int v = -1;
    if (q < n) {
        v = list[q];
        if (!in_range(v, f.N)) { report(f, 10); v = -1; }
    }
    const bool sampled = v >= 0 && ((inv[v] >> 7) % stride) == 0;
    const bool other = v >= 0 && !sampled;
    const int slot_a = block_append<TB>(sampled, &counts[0]);
    __syncthreads();
    const int slot_b = block_append<TB>(other, &counts[1]);
    if (sampled) { if (in_range(slot_a, f.N)) part_a[slot_a] = v; else report(f, 10); }
    if (other) { if (in_range(slot_b, f.N)) part_b[slot_b] = v; else report(f, 10); }
}

__global__ void __launch_bounds__(TB) k_still_needed(ForestState f, const int32_t* __restrict__ list, int n,
                                                     int32_t* __restrict__ out, int32_t* __restrict__ count)
{
    const int q = blockIdx.x * TB + threadIdx.x;
    bool keep = false;
    int v = -1;
    if (q < n) {
        v = list[q];
        if (!in_range(v, f.N) || !in_range(f.colour[v], f.N)) report(f, 11);
        else keep = __float_as_uint(f.cand_w[v]) <= f.best_w[f.colour[v]];
    }
    const int slot = block_append<TB>(keep, count);
    if (keep) { if (in_range(slot, f.N)) out[slot] = v; else report(f, 11); }
}

__global__ void __launch_bounds__(TB) k_select_edges(ForestState f)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v >= f.N || forest_halted(f)) return;
    const int u = f.cand_u[v];
    if (u < 0) return;
    const int c = f.colour[v];
    if (u >= f.N || !in_range(c, f.N)) { report(f, 7); return; }
    if (__float_as_uint(f.cand_w[v]) != f.best_w[c]) return;
    const unsigned int lo = (unsigned int)(v < u ? v : u), hi = (unsigned int)(v < u ? u : v);
    min_into(&f.best_e[c], ((unsigned long long)lo << 32) | hi);
}

// One thread per component root: append the component's edge (once per undirected edge) and
// record which component it attaches to.  Two components that chose the same edge keep the
// smaller root.
constexpr int COMMIT_ITEMS = 4;        // vertices per thread: one atomic on the edge counter per 4096 vertices (8: half the chip idle at 1M)
__global__ void __launch_bounds__(TB_WIDE) k_commit(ForestState f)
{
    __shared__ int wave_count[TB_WIDE / 64];
    __shared__ int wave_base[TB_WIDE / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (forest_halted(f)) return;
    int lo[COMMIT_ITEMS], hi[COMMIT_ITEMS];
    uint32_t wbits[COMMIT_ITEMS];
    unsigned int adds = 0;             // bit i: vertex i of this thread appends its component's edge
#pragma unroll
    for (int i = 0; i < COMMIT_ITEMS; ++i) {
        const long long vv = ((long long)blockIdx.x * COMMIT_ITEMS + i) * TB_WIDE + threadIdx.x;
        lo[i] = hi[i] = 0;
        wbits[i] = INF_BITS;
        if (vv >= f.N) continue;
        const int v = (int)vv;
        if (f.colour[v] != v) continue;
        const uint32_t wb = f.best_w[v];
        int hook = v;
        if (wb != INF_BITS) {
            const unsigned long long e = f.best_e[v];
            const int elo = (int)(e >> 32), ehi = (int)(e & 0xffffffffull);
            if (!in_range(elo, f.N) || !in_range(ehi, f.N)) report(f, 8);
            else {
                const int clo = f.colour[elo], chi = f.colour[ehi];
                const int other = (clo == v) ? chi : clo;
                if (!in_range(other, f.N) || other == v || (clo != v && chi != v))
                    report_with(f, 9, v, elo, ehi, clo, chi, (int)wb);
                else {
                    const bool mutual = (f.best_w[other] == wb) && (f.best_e[other] == e);
                    if (!mutual || v < other) { adds |= 1u << i; lo[i] = elo; hi[i] = ehi; wbits[i] = wb; }
                    hook = (mutual && v < other) ? v : other;
                }
            }
        }
        f.hook[v] = hook;
    }
    // exclusive prefix of the per-thread counts over the workgroup
    const int mine = __popc(adds);
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    if (lane == 63) wave_count[wave] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
        for (int w = 0; w < TB_WIDE / 64; ++w) { wave_base[w] = total; total += wave_count[w]; }
        const int base = total > 0 ? atomicAdd(&f.counters[1], total) : 0;
        for (int w = 0; w < TB_WIDE / 64; ++w) wave_base[w] += base;
    }
    __syncthreads();
    int slot = wave_base[wave] + incl - mine;
#pragma unroll
    for (int i = 0; i < COMMIT_ITEMS; ++i) {
        if (!(adds & (1u << i))) continue;
        if (slot < f.N - 1) {
            f.e_lo[slot] = lo[i];
            f.e_hi[slot] = hi[i];
            f.e_w[slot] = __uint_as_float(wbits[i]);
        }
        ++slot;
    }
}

// Every root follows the hooks up to `steps` components far and hooks itself to where it got; other
// roots do the same at the same time, which is harmless: whatever a hook is replaced by is an ancestor
// of what it held.  With `flag` a root that has not reached the end of its chain sets counters[2].
// Two launches of 32 steps resolve chains of up to 1024 hooks; the host loops only beyond that.
__global__ void __launch_bounds__(TB) k_jump(ForestState f, int steps, int flag)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v >= f.N || f.colour[v] != v) return;
    int h = f.hook[v];
    if (!in_range(h, f.N)) { report(f, 10); return; }
    bool at_root = false;
    for (int i = 0; i < steps; ++i) {
        const int hh = *reinterpret_cast<volatile int32_t*>(&f.hook[h]);
        if (!in_range(hh, f.N)) { report(f, 11); return; }
        if (hh == h) { at_root = true; break; }
        h = hh;
    }
    f.hook[v] = h;
    if (flag && !at_root) {
        const int hh = *reinterpret_cast<volatile int32_t*>(&f.hook[h]);
        if (hh != h) atomicOr(&f.counters[2], 1);
    }
}

// Every vertex follows the hooks of its component to their end (hooks of one round: a chain of a few components nearly
// always), takes that root as its colour, and clears its slots of the per-component minima for the next round.  A root
// shortens its own hook on the way, which can only help the others.  A chain longer than `steps` leaves its vertices as
// they are and sets counters[2]: the host finishes it with k_jump and launches this kernel again.
__global__ void __launch_bounds__(TB) k_follow(ForestState f, int steps)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v >= f.N) return;
    if (v == 0) f.counters[0] = 0;
    f.best_w[v] = INF_BITS;
    f.best_e[v] = ~0ull;
    const int c = f.colour[v];
    if (!in_range(c, f.N)) { report(f, 12); return; }
    int r = c;
    bool at_root = false;
    for (int i = 0; i < steps; ++i) {
        const int h = *reinterpret_cast<volatile int32_t*>(&f.hook[r]);
        if (!in_range(h, f.N)) { report(f, 13); return; }
        if (h == r) { at_root = true; break; }
        r = h;
    }
    if (!at_root) { atomicOr(&f.counters[2], 1); return; }
    if (v == c) f.hook[v] = r;
    f.colour[v] = r;
}

// The counters, to host memory: words 1 .. n hold counters[0 .. n-1] and word 0 the sequence number, written last.
__global__ void __launch_bounds__(64) k_publish(const int32_t* __restrict__ counters, int n, int32_t* __restrict__ host, int32_t seq)
{
    const int i = threadIdx.x;
    if (i < n) __hip_atomic_store(host + 1 + i, counters[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();
    if (i == 0) __hip_atomic_store(host, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// All rounds of a forest of at most FOREST_SMALL_MAX vertices in one workgroup, until it is complete or a round has
// rows to query: at this size a round's handful of launches and its read-back are a hundred times its work (4096 rows:
// 5 rounds 0.33 ms as separate launches).  Colours, hooks and the per-component minima live in LDS; an edge's end
// points fit one word there.  Same rules, same edges as the separate kernels.
//   stage 0: first launch;  1: after a round's queries were applied (k_apply_queries): continue at the selection.
// One workgroup has one CU's loads in flight, so the walks along the lists are bound by their latency: a thread has I vertices, tid, tid + 1024, ..,
// whose places in their lists and candidates are registers, and takes four entries of four of them at a time.  With an entry of a vertex
// at a time and candidates in memory the three launches of 10 000 rows, k = 20, took 308 us, of 4096 rows, k = 16, 109; 214 and 82 so (keeping candidates that still lead out: no faster).
typedef int v4i_word __attribute__((ext_vector_type(4), aligned(4)));        // (loads of 16 bytes need the alignment of a word only)
template <int I>
__global__ void __launch_bounds__(1024) k_forest_small(ForestState f, int stage)
{
    extern __shared__ __align__(16) unsigned char small_smem[];
    __shared__ int s_edges, s_queries, s_bad;
    const int N = f.N;
    int tid = threadIdx.x;
    unsigned int* bw = reinterpret_cast<unsigned int*>(small_smem);
    unsigned int* be = bw + N;
    unsigned short* col = reinterpret_cast<unsigned short*>(be + N);
    unsigned short* hk = col + N;
    if (tid == 0) {
        if (stage == 0) for (int i = 0; i < 8; ++i) f.counters[i] = 0;
        s_edges = stage == 0 ? 0 : f.counters[1];
        s_bad = 0;
    }
    int ptr[I], cand_u[I];
    float cand_w[I];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int v = tid + i * 1024;
        ptr[i] = 0; cand_u[i] = -1; cand_w[i] = 0.f;
        if (v >= N) continue;
        if (stage == 0) {
            col[v] = (unsigned short)v;
            f.ext_idx[v] = -1; f.ext_dist[v] = 0.f; f.ext_low[v] = __builtin_inff();
        } else {
            const int c = f.colour[v];
            col[v] = (unsigned short)(in_range(c, N) ? c : 0);
            bw[v] = f.best_w[v];
            ptr[i] = f.ptr[v]; cand_u[i] = f.cand_u[v]; cand_w[i] = f.cand_w[v];
        }
    }
    __syncthreads();
    int rounds = stage == 0 ? 0 : f.counters[6];
    bool selected = stage == 1;               // the candidates of this round are complete
    for (int guard = 0; guard < 64; ++guard) {
        asm volatile("" : "+v"(tid));             // (every round works its addresses out: kept, they push the candidates out of the registers)
        if (!selected) {
            if (tid == 0) s_queries = 0;
#pragma unroll
            for (int i = 0; i < I; ++i)
                if (tid + i * 1024 < N) bw[tid + i * 1024] = INF_BITS;
            __syncthreads();
            ++rounds;
#pragma unroll
            for (int i0 = 0; i0 < I; i0 += 4) {
                // every vertex's first foreign entry from ptr on (f.k: there is none)
                unsigned int c[4];
                bool more[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int v = tid + (i0 + j) * 1024;
                    c[j] = v < N ? col[v] : 0u;
                    more[j] = v < N && ptr[i0 + j] < f.k;
                    if (v < N) cand_u[i0 + j] = -1;
                }
                while (more[0] || more[1] || more[2] || more[3]) {
                    int u[4][4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (!more[j]) continue;
                        // (the last quad of a list starts where it ends with the list)
                        const int p = ptr[i0 + j], e = p + 4 <= f.k ? p : f.k - 4;
                        const unsigned int list = (unsigned int)((tid + (i0 + j) * 1024) * f.k);
                        if (f.k >= 4) {
                            const v4i_word q = *reinterpret_cast<const v4i_word*>(f.nbr_idx + (list + (unsigned int)e));
#pragma unroll
                            for (int t = 0; t < 4; ++t) u[j][t] = q[t];
                        } else {
#pragma unroll
                            for (int t = 0; t < 4; ++t) u[j][t] = e + t >= 0 ? f.nbr_idx[list + (unsigned int)(e + t)] : -1;
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (!more[j]) continue;
                        const int p = ptr[i0 + j], e = p + 4 <= f.k ? p : f.k - 4;
                        int at = f.k;
#pragma unroll
                        for (int t = 3; t >= 0; --t) {
                            if (e + t < p) continue;
                            if (!in_range(u[j][t], N)) { report(f, 1); continue; }
                            if (col[u[j][t]] != c[j]) { at = e + t; cand_u[i0 + j] = u[j][t]; }
                        }
                        more[j] = at == f.k && e + 4 < f.k;
                        ptr[i0 + j] = more[j] ? e + 4 : at;
                    }
                }
                float w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int v = tid + (i0 + j) * 1024;
                    w[j] = 0.f;
                    if (v < N) w[j] = f.nbr_dist[(unsigned int)(v * f.k) + (unsigned int)(ptr[i0 + j] < f.k ? ptr[i0 + j] : f.k - 1)];
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int v = tid + (i0 + j) * 1024;
                    if (v >= N) continue;
                    float reach = INFINITY;              // an edge that need not be v's lightest (see k_scan_lists)
                    if (cand_u[i0 + j] >= 0) reach = w[j];
                    else if (stage == 1) {               // (nothing has been asked for before)
                        const int eu = f.ext_idx[v];
                        const float ed = f.ext_dist[v], el = f.ext_low[v];
                        const bool edge = eu >= 0 && eu < N && col[eu] != c[j];
                        if (edge) reach = ed;
                        if (edge && !(el < INFINITY)) { w[j] = ed; cand_u[i0 + j] = eu; }
                        else w[j] = fmaxf(w[j], fminf(ed, el));
                    } else w[j] = fmaxf(w[j], 0.f);
                    cand_w[i0 + j] = w[j];
                    if (reach < INFINITY) atomicMin(&bw[c[j]], __float_as_uint(reach));
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < I; ++i) {
                const int v = tid + i * 1024;
                if (v < N && cand_u[i] < 0 && __float_as_uint(cand_w[i]) <= bw[col[v]]) f.qlist[atomicAdd(&s_queries, 1)] = v;
            }
            __syncthreads();
            if (s_queries > 0) {
#pragma unroll
                for (int i = 0; i < I; ++i) {
                    const int v = tid + i * 1024;
                    if (v >= N) continue;
                    f.colour[v] = col[v]; f.best_w[v] = bw[v];
                    f.ptr[v] = ptr[i]; f.cand_u[v] = cand_u[i]; f.cand_w[v] = cand_w[i];
                }
                if (tid == 0) { f.counters[0] = s_queries; f.counters[1] = s_edges; f.counters[6] = rounds; }
                return;
            }
        }
        selected = false;
        // the component's edge among those of its lightest weight
        for (int v = tid; v < N; v += 1024) be[v] = ~0u;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int v = tid + i * 1024, u = cand_u[i];
            if (v >= N || u < 0) continue;
            const unsigned int c = col[v];
            if (u >= N) { report(f, 7); continue; }
            if (__float_as_uint(cand_w[i]) != bw[c]) continue;
            const unsigned int lo = v < u ? v : u, hi = v < u ? u : v;
            atomicMin(&be[c], (lo << 16) | hi);
        }
        __syncthreads();
        const int before = s_edges;
        __syncthreads();
        for (int v = tid; v < N; v += 1024) {
            if (col[v] != v) continue;
            unsigned int hook = v;
            const unsigned int wb = bw[v], e = be[v];
            if (wb != INF_BITS) {
                const int elo = (int)(e >> 16), ehi = (int)(e & 0xffffu);
                if (elo >= N || ehi >= N) { report(f, 8); s_bad = 1; }
                else {
                    const int clo = col[elo], chi = col[ehi];
                    const int other = clo == v ? chi : clo;
                    if (other == v || (clo != v && chi != v)) { report_with(f, 9, v, elo, ehi, clo, chi, (int)wb); s_bad = 1; }
                    else {
                        const bool mutual = bw[other] == wb && be[other] == e;
                        if (!mutual || v < other) {
                            const int slot = atomicAdd(&s_edges, 1);
                            if (slot < N - 1) { f.e_lo[slot] = elo; f.e_hi[slot] = ehi; f.e_w[slot] = __uint_as_float(wb); }
                        }
                        hook = mutual && v < other ? v : other;
                    }
                }
            }
            hk[v] = (unsigned short)hook;
        }
        __syncthreads();
        for (int v = tid; v < N; v += 1024) {
            if (col[v] != v) continue;
            unsigned int r = v;
            for (int i = 0; i < N; ++i) {                 // (a chain visits a component once)
                const unsigned int h = *reinterpret_cast<volatile unsigned short*>(&hk[r]);
                if (h == r) break;
                r = h;
            }
            *reinterpret_cast<volatile unsigned short*>(&hk[v]) = (unsigned short)r;
        }
        __syncthreads();
        for (int v = tid; v < N; v += 1024) col[v] = hk[col[v]];
        __syncthreads();
        if (s_edges >= N - 1 || s_edges == before || s_bad) break;
    }
    for (int v = tid; v < N; v += 1024) f.colour[v] = col[v];
    if (tid == 0) { f.counters[0] = 0; f.counters[1] = s_edges; f.counters[6] = rounds; }
}

// Rows per component: sizes[c] += 1 for every row of colour c (entries outside [0, bins) are skipped;
// sizes zeroed by the caller).  Meant for colours in a spatially coherent row order, where the lanes of a
// wavefront share one or two colours: those are counted with one atomic each.
__global__ void __launch_bounds__(TB) k_component_sizes(const int32_t* __restrict__ colour, int n, int bins,
                                                        int32_t* __restrict__ sizes)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int c = i < n ? colour[i] : -1;
    bool active = (unsigned int)c < (unsigned int)bins;
    unsigned long long todo = __ballot(active);
#pragma unroll 1
    for (int pass = 0; pass < 4 && todo; ++pass) {
        const int leader = __builtin_ctzll(todo);
        const int c0 = __shfl(c, leader);
        const bool mine = active && c == c0;
        const unsigned long long served = __ballot(mine);
        if (lane == leader) atomicAdd(&sizes[c0], __popcll(served));
        todo &= ~served;
        active = active && !mine;
    }
    if (active) atomicAdd(&sizes[c], 1);
}

#define LAUNCH1(kern, n, s, ...)                                                       \
    do {                                                                               \
        hipLaunchKernelGGL(kern, dim3(blocks_for(n)), dim3(TB), 0, s, __VA_ARGS__);    \
        return hipGetLastError();                                                      \
    } while (0)

hipError_t forest_init(const ForestState& f, hipStream_t s) { LAUNCH1(k_forest_init, f.N, s, f); }

hipError_t forest_scan_lists(const ForestState& f, hipStream_t s)
{
    if (f.k <= 2) LAUNCH1(k_scan_lists<2>, (long long)f.N * 2, s, f);
    LAUNCH1(k_scan_lists<4>, (long long)f.N * 4, s, f);
}

hipError_t forest_classify(const ForestState& f, hipStream_t s)
{
    hipLaunchKernelGGL(k_classify, dim3((f.N + TB_WIDE - 1) / TB_WIDE), dim3(TB_WIDE), 0, s, f);
    return hipGetLastError();
}

hipError_t forest_apply_queries(const ForestState& f, const int32_t* qrows, const int32_t* q_idx, const float* q_dist,
                                const float* q_low, int nq, const uint32_t* thresholds, hipStream_t s)
{
    LAUNCH1(k_apply_queries, nq, s, f, qrows, q_idx, q_dist, q_low, nq, thresholds);
}

hipError_t forest_split_queries(const ForestState& f, const int32_t* list, int n, const int32_t* inv, int stride,
                                int32_t* part_a, int32_t* part_b, int32_t* counts, hipStream_t s)
{
    LAUNCH1(k_split_queries, n, s, f, list, n, inv, stride, part_a, part_b, counts);
}

hipError_t forest_still_needed(const ForestState& f, const int32_t* list, int n, int32_t* out, int32_t* count,
                               hipStream_t s)
{
    LAUNCH1(k_still_needed, n, s, f, list, n, out, count);
}

hipError_t forest_select_edges(const ForestState& f, hipStream_t s) { LAUNCH1(k_select_edges, f.N, s, f); }
hipError_t forest_component_sizes(const int32_t* colour, int n, int bins, int32_t* sizes, hipStream_t s)
{
    LAUNCH1(k_component_sizes, n, s, colour, n, bins, sizes);
}
hipError_t forest_commit(const ForestState& f, hipStream_t s)
{
    const int per_block = TB_WIDE * COMMIT_ITEMS;
    hipLaunchKernelGGL(k_commit, dim3((f.N + per_block - 1) / per_block), dim3(TB_WIDE), 0, s, f);
    return hipGetLastError();
}
hipError_t forest_jump(const ForestState& f, int steps, bool flag, hipStream_t s) { LAUNCH1(k_jump, f.N, s, f, steps, flag ? 1 : 0); }
hipError_t forest_follow(const ForestState& f, hipStream_t s) { LAUNCH1(k_follow, f.N, s, f, FOLLOW_STEPS); }
hipError_t forest_publish(const ForestState& f, int32_t* host, int32_t seq, hipStream_t s)
{
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, f.counters, 8, host, seq);
    return hipGetLastError();
}
hipError_t forest_small(const ForestState& f, bool first, hipStream_t s)
{
    const size_t lds = (size_t)f.N * 12;
    auto run = [&](auto kernel) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), lds, s, f, first ? 0 : 1);
        return hipGetLastError();
    };
    if (f.N <= 4 * 1024) return run(&k_forest_small<4>);
    if (f.N <= 8 * 1024) return run(&k_forest_small<8>);
    static_assert(FOREST_SMALL_MAX <= 12 * 1024, "");
    return run(&k_forest_small<12>);
}

// ------------------------------------------------------------------------------- edge sort
__global__ void __launch_bounds__(TB) k_pack_edges(const int32_t* __restrict__ lo,
                                                   const int32_t* __restrict__ hi,
                                                   const float* __restrict__ w, int bits, int E,
                                                   unsigned long long* __restrict__ keys,
                                                   uint32_t* __restrict__ vals)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i >= E) return;
    keys[i] = ((unsigned long long)(unsigned int)lo[i] << bits) | (unsigned int)hi[i];
    vals[i] = __float_as_uint(w[i]);
}

// children / sizes of all merges from host memory
__global__ void __launch_bounds__(256) k_linkage_upload(const int32_t* __restrict__ cj, const int32_t* __restrict__ sj, int E,
                                                        int32_t* __restrict__ children, int32_t* __restrict__ sizes)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= E) return;
    children[2 * j] = cj[2 * j];
    children[2 * j + 1] = cj[2 * j + 1];
    sizes[j] = sj[j];
}

hipError_t linkage_upload(const int32_t* cj, const int32_t* sj, int E, int32_t* children, int32_t* sizes, hipStream_t s)
{
    hipLaunchKernelGGL(k_linkage_upload, dim3((E + 255) / 256), dim3(256), 0, s, cj, sj, E, children, sizes);
    return hipGetLastError();
}

// Radix passes from 32 768 pairs on: the library's default sorts up to a million of them by merging, ten and more
// launches over the whole data (1M edges: 390 us for both sorts, 130 us by radix passes).
using radix_passes = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config, rocprim::default_config, 32768>;

// Trees of at most 2^16 vertices: weight and both end points fit one 64-bit key, so one sort of keys does.
constexpr int SMALL_IDS = 1 << 16;
__global__ void __launch_bounds__(TB) k_pack_small(const int32_t* __restrict__ lo, const int32_t* __restrict__ hi,
                                                   const float* __restrict__ w, int E, unsigned long long* __restrict__ keys)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i < E) keys[i] = ((unsigned long long)__float_as_uint(w[i]) << 32) | ((unsigned int)lo[i] << 16) | (unsigned int)hi[i];
}
// ends: (lo << shift | hi), wbits apart (nullptr: the small form).  heights, host_lo, host_hi: optional copies, the latter
// two in host memory.
__global__ void __launch_bounds__(TB) k_unpack_edges(const unsigned long long* __restrict__ ends, const uint32_t* __restrict__ wbits,
                                                     int shift, int E, int32_t* __restrict__ lo, int32_t* __restrict__ hi,
                                                     float* __restrict__ w, EdgeCopies c)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i >= E) return;
    const unsigned long long e = ends[i];
    const int a = wbits ? (int)(e >> shift) : (int)((e >> 16) & 0xffffu);
    const int b = wbits ? (int)(e & ((1ull << shift) - 1ull)) : (int)(e & 0xffffu);
    const float x = __uint_as_float(wbits ? wbits[i] : (uint32_t)(e >> 32));
    lo[i] = a; hi[i] = b; w[i] = x;
    if (c.heights) c.heights[i] = x;
    if (c.host_lo) { c.host_lo[i] = a; c.host_hi[i] = b; }
}

size_t edge_sort_temp_bytes(int E)
{
    size_t a = 0, b = 0, d = 0;
    unsigned long long* k64 = nullptr;
    uint32_t* k32 = nullptr;
    (void)rocprim::radix_sort_pairs<radix_passes>(nullptr, a, k64, k64, k32, k32, (size_t)E, 0, 64, (hipStream_t)0);
    (void)rocprim::radix_sort_pairs<radix_passes>(nullptr, b, k32, k32, k64, k64, (size_t)E, 0, 32, (hipStream_t)0);
    (void)rocprim::radix_sort_keys<radix_passes>(nullptr, d, k64, k64, (size_t)E, 0, 64, (hipStream_t)0);
    a = a > b ? a : b;
    return ((a > d ? a : d) + 255) & ~(size_t)255;
}

// Up to 2^16 vertices one sort of 64-bit keys; beyond, two stable passes: by (lo, hi), packed into as many bits as N
// needs, then by the weight bits (non-negative floats order like their bit patterns).
hipError_t edge_sort(const int32_t* lo, const int32_t* hi, const float* w, int E, int N,
                     unsigned long long* keys_a, unsigned long long* keys_b,
                     uint32_t* vals_a, uint32_t* vals_b, void* temp, size_t temp_bytes,
                     int32_t* out_lo, int32_t* out_hi, float* out_w, const EdgeCopies& copies, hipStream_t s)
{
    size_t tb = temp_bytes;
    hipError_t e;
    if (N <= SMALL_IDS) {
        hipLaunchKernelGGL(k_pack_small, dim3(blocks_for(E)), dim3(TB), 0, s, lo, hi, w, E, keys_a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = rocprim::radix_sort_keys<radix_passes>(temp, tb, keys_a, keys_b, (size_t)E, 0, 64, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_unpack_edges, dim3(blocks_for(E)), dim3(TB), 0, s, keys_b, (const uint32_t*)nullptr, 16, E, out_lo, out_hi, out_w, copies);
        return hipGetLastError();
    }
    int bits = 17;
    while (bits < 31 && (1LL << bits) < (long long)N) ++bits;
    hipLaunchKernelGGL(k_pack_edges, dim3(blocks_for(E)), dim3(TB), 0, s, lo, hi, w, bits, E, keys_a, vals_a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = rocprim::radix_sort_pairs<radix_passes>(temp, tb, keys_a, keys_b, vals_a, vals_b, (size_t)E, 0, (unsigned int)(2 * bits), s);
    if (e != hipSuccess) return e;
    tb = temp_bytes;
    e = rocprim::radix_sort_pairs<radix_passes>(temp, tb, vals_b, vals_a, keys_b, keys_a, (size_t)E, 0, 32, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_unpack_edges, dim3(blocks_for(E)), dim3(TB), 0, s, keys_a, vals_a, bits, E, out_lo, out_hi, out_w, copies);
    return hipGetLastError();
}

size_t pair_sort_temp_bytes(int n)
{
    size_t a = 0;
    uint32_t* k32 = nullptr;
    (void)rocprim::radix_sort_pairs<radix_passes>(nullptr, a, k32, k32, k32, k32, (size_t)n, 0, 32, (hipStream_t)0);
    return (a + 255) & ~(size_t)255;
}

hipError_t pair_sort_u32(const uint32_t* keys_in, uint32_t* keys_out, const uint32_t* vals_in,
                         uint32_t* vals_out, int n, int key_bits, void* temp, size_t temp_bytes,
                         hipStream_t s)
{
    size_t tb = temp_bytes;
    if (key_bits < 1) key_bits = 1;
    if (key_bits > 32) key_bits = 32;
    return rocprim::radix_sort_pairs<radix_passes>(temp, tb, keys_in, keys_out, vals_in, vals_out, (size_t)n, 0,
                                     (unsigned int)key_bits, s);
}

}  // namespace slhc
