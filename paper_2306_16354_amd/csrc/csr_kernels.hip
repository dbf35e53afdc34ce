// Spanning forest of a CSR graph (cuSLINK paper Sec. 3.2, Alg. "MST Algorithm"): the rounds of forest_kernels.hip, same rules and
// same edges, for a graph whose rows are its neighbour lists.
//
// A round only looks at what is left of the graph: the vertices that had an edge out of their component in the round before
// and the roots of components that had one, both kept as lists.  Components only grow, so a vertex without such an edge never
// has one again; its colour is complemented, which tells its neighbours, all in its own component, without being kept up to date.
// (Walking up from stale colours instead: two random reads per entry where one does, 610 us of scans.)
// What bounds it: random 4-byte reads in the first four rounds (330 us), then the chain of dependent reads and the end of every launch
// (30 us a round, whatever is left of the graph).  Road-like graph of 1 048 576 vertices and 2.6 million entries: rounds over all
// vertices 750 us, over the lists 580, over all vertices and an edge to a word in the first two 530.
#include <hip/hip_runtime.h>
#include <cstring>
#include <rocprim/rocprim.hpp>
#include <stdint.h>
#include "csr_kernels.h"
#include "wave_ops.h"

namespace slhc {

constexpr uint32_t INF_BITS = 0x7f800000u;
constexpr int TB = 256, WIDE = 1024;      // (WIDE: kernels that append to a list, one atomic per workgroup)
constexpr int FOLLOW_STEPS = 64;       // hooks followed in one launch
static inline int blocks_for(long long n, int threads = TB) { return (int)((n + threads - 1) / threads); }
// Up to FEW vertices rows are read by workgroups of TB threads: the fewer CUs read, the longer they take, and there are few additions to a list
// then.  Calls with 1024 threads and 256, in us, 2.5 entries a vertex: 20 000 vertices 305 and 270, 130 000 470 and 431, 200 000 493
// and 466; 20 entries: 395 and 303, 627 and 547, 804 and 821.
constexpr int FEW = 131072;
static inline int append_blocks(long long n) { const int b = blocks_for(n < 1 ? 1 : n, WIDE); return b > 512 ? 512 : b; }

__device__ inline bool in_range(int i, int n) { return (unsigned int)i < (unsigned int)n; }
__device__ inline void report(const CsrForest& f, int site) { atomicCAS(f.words + CSR_ERROR, 0, site); }
// a failed check, or hooks that are not followed to their end yet, leave all rounds enqueued to the host
__device__ inline bool halted(const CsrForest& f) { return (f.words[CSR_ERROR] | f.words[CSR_CHAINS]) != 0; }
// The same for a whole workgroup, where barriers follow: another workgroup of the launch may report while this one starts, and wavefronts that each
// read the word could part then, the counts of those that left never written.
__device__ inline bool all_halted(const CsrForest& f)
{
    __shared__ int state;
    if (threadIdx.x == 0) state = halted(f);
    __syncthreads();
    return state != 0;
}

// A row of up to LONG_ROW entries is read by its vertex's thread (road-like graphs have two or three edges per vertex), which takes 0.2 us per
// entry; one of up to HUGE_ROW by 16 lanes, four such rows at once; a longer one by the whole wavefront.  Calls with long rows by
// threads and so: a star of 70 000 vertices 27 and 0.5 ms (one scan less, too: see k_csr_scan), 300 000 vertices with 300
// hubs 4.6 and 0.7; with 80 entries on average 20 000 vertices 1.46 and 0.56, 500 000 6.2 and 2.4.  (One row at a time by the whole wavefront:
// 20 000 vertices with 80 entries 0.87; the line at 32, 48 and 64, 200 000 vertices with 24 and 48 entries: 956, 888, 889 and
// 1420, 1486, 1757 us.)
constexpr unsigned int LONG_ROW = 48, HUGE_ROW = 1024;

// Entries of v's row: from `at` on, four side by side (their loads wait for memory together), then `step` further.  Returns the first in
// the order (weight, smaller end, larger end) that leads out of component c, as its weight's bits and the other end; among the edges of
// one vertex that is the order of the ends.  (Unsigned, because the step behind the last ones may lie beyond 2^31.)
constexpr unsigned long long NO_EDGE = ((unsigned long long)INF_BITS << 32) | 0xffffffffull;
template <bool FIRST>
__device__ inline unsigned long long row_part(const CsrForest& f, int v, int c, unsigned int at, unsigned int end, unsigned int step)
{
    unsigned long long best = NO_EDGE;
    for (unsigned int e0 = at; e0 < end; e0 += step) {
        int u[4], cu[4];
        float w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u[j] = e0 + j < end ? f.indices[e0 + j] : -1;
            w[j] = e0 + j < end ? f.weights[e0 + j] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (FIRST) {
                if (e0 + j < end && !in_range(u[j], f.V)) report(f, 23);
                if (!(w[j] >= 0.f) || w[j] == __builtin_inff()) report(f, 24);
                cu[j] = u[j];
            } else cu[j] = in_range(u[j], f.V) ? *reinterpret_cast<volatile int32_t*>(f.colour + u[j]) : -1;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!in_range(u[j], f.V) || cu[j] < 0 || cu[j] == c) continue;
            const unsigned long long key = ((unsigned long long)(__float_as_uint(w[j]) & 0x7fffffffu) << 32) | (unsigned int)u[j];       // (-0 is 0)
            best = key < best ? key : best;
        }
    }
    return best;
}

// The edge of v's row out of component c (v < 0: none), as row_part has it.  Every lane of the wavefront must call it.
template <bool FIRST>
__device__ inline unsigned long long row_edge(const CsrForest& f, int v, int c)
{
    unsigned int at = 0, end = 0;
    if (v >= 0) {
        const int o0 = f.offsets[v], o1 = f.offsets[v + 1];
        if (FIRST) {
            if (o0 < 0 || o1 < o0 || o1 > f.E) report(f, 20);
            if (v == 0 && o0 != 0) report(f, 21);
            if (v == f.V - 1 && o1 != f.E) report(f, 22);
        }
        at = o0 < 0 ? 0u : (unsigned int)o0;
        end = o1 < 0 ? 0u : o1 > f.E ? (unsigned int)f.E : (unsigned int)o1;
    }
    const unsigned int length = at < end ? end - at : 0u;
    unsigned long long best = length > LONG_ROW ? NO_EDGE : row_part<FIRST>(f, v, c, at, end, 4);
    const int lane = threadIdx.x & 63, group = lane >> 4;
    // four rows at once: group g takes the g-th of those that are left
    unsigned long long todo = __ballot(length > LONG_ROW && length <= HUGE_ROW);
    while (todo != 0) {
        unsigned long long m = todo;
        for (int i = 0; i < group; ++i) m &= m - 1;
        const int owner = m != 0 ? __builtin_ctzll(m) : 0;
        const unsigned int o_at = (unsigned int)__shfl((int)at, owner), o_end = (unsigned int)__shfl((int)end, owner);
        const int o_v = __shfl(v, owner), o_c = __shfl(c, owner);
        unsigned long long key = m != 0 ? row_part<FIRST>(f, o_v, o_c, o_at + 4 * (lane & 15), o_end, 64) : NO_EDGE;
        key = lanes_min<8>(lanes_min<4>(lanes_min<2>(lanes_min<1>(key))));
        const int mine = __builtin_amdgcn_mbcnt_hi((unsigned int)(todo >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)todo, 0u));       // (this lane's, if it has one)
        const unsigned long long result = __shfl(key, (mine & 3) * 16);
        if ((todo >> lane & 1) != 0 && mine < 4) best = result;
        for (int i = 0; i < 4; ++i) todo &= todo - 1;              // (0 & ~0 is 0)
    }
    for (todo = __ballot(length > HUGE_ROW); todo != 0; todo &= todo - 1) {
        const int owner = __builtin_ctzll(todo);
        unsigned long long key = row_part<FIRST>(f, __shfl(v, owner), __shfl(c, owner), (unsigned int)__shfl((int)at, owner) + 4 * lane, (unsigned int)__shfl((int)end, owner), 256);
        key = wave_min(key);
        if (lane == owner) best = key;
    }
    return best;
}
__device__ inline uint32_t edge_weight(unsigned long long e) { return (uint32_t)(e >> 32); }
__device__ inline int edge_end(unsigned long long e) { return e == NO_EDGE ? -1 : (int)(e & 0xffffffffull); }
// the ends of v's edge to u in their order
__device__ inline unsigned long long edge_ends(int v, int u)
{
    return ((unsigned long long)(unsigned int)(v < u ? v : u) << 32) | (unsigned int)(v < u ? u : v);
}

// Beyond FEW vertices the lists of the first rounds would hold nearly all of them: rounds 0 to LAST_ALL make none, and what would read them goes over
// all vertices, of which those without an edge have a complemented colour.  The words that count a list's entries say V.  (Road-like graph of 1M
// vertices: round 0's lists 20 us with the vertices' edges, 10 without; with LAST_ALL of 1 to 4 the calls take the same, within 0.5 %.)
constexpr int LAST_ALL = 1;
__host__ __device__ inline bool list_is_all(const CsrForest& f, int round) { return f.V > FEW && round <= LAST_ALL; }

// Round 0: every vertex is a component, and its edge the component's.
template <int THREADS, bool ALL>
__global__ void __launch_bounds__(THREADS) k_csr_first(CsrForest f)
{
    const int v = blockIdx.x * THREADS + threadIdx.x;
    const unsigned long long e = row_edge<true>(f, v < f.V ? v : -1, v);
    if (v < f.V) {
        f.colour[v] = v;
        f.hook[v] = v;
        f.cand[v] = e;
    }
    if (ALL) return;
    const int at = block_append<THREADS>(v < f.V && edge_end(e) >= 0, f.words + CSR_ACTIVE + 1);
    if (at >= 0) f.active[1][at] = v;
}

// Round r: the active vertices' edges, and the weight of every component's lightest.  Also tells the host how the round before
// ended, in words that carry `seq` each (so no fence has to stand between them and one number for all).
template <int THREADS, bool ALL_IN, bool ALL_OUT>
__global__ void __launch_bounds__(THREADS) k_csr_scan(CsrForest f, int round, unsigned long long* __restrict__ host, uint32_t seq)
{
    if (blockIdx.x == 0 && threadIdx.x < CSR_TOLD) {
        const int at[CSR_TOLD] = {CSR_ACTIVE + round % 3, CSR_EDGES, CSR_CHAINS, CSR_ERROR};
        const unsigned int word = (unsigned int)f.words[at[threadIdx.x]] | (threadIdx.x == 0 ? (unsigned int)f.words[CSR_TIES] : 0u);
        __hip_atomic_store(host + threadIdx.x, ((unsigned long long)seq << 32) | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if ((ALL_OUT ? halted(f) : all_halted(f)) || f.words[CSR_EDGES] >= f.V - 1) return;       // (one tree: nothing is left to find)
    const int n = ALL_IN ? f.V : f.words[CSR_ACTIVE + round % 3];
    const int32_t* from = f.active[round & 1];
    int32_t* to = f.active[(round + 1) & 1];
    uint32_t* best_w = f.best_w[round & 1];
    for (long long base = (long long)blockIdx.x * THREADS; base < n; base += (long long)gridDim.x * THREADS) {
        const long long i = base + threadIdx.x;
        int v = -1, c = 0;
        if (i < n) {
            v = ALL_IN ? (int)i : from[i];
            c = f.colour[v];
            if (ALL_IN && c < 0 && in_range(~c, f.V)) v = -1;     // (without an edge since an earlier round)
            else if (!in_range(c, f.V)) { report(f, 11); v = -1; }
        }
        const unsigned long long e = row_edge<false>(f, v, c);
        const bool some = edge_end(e) >= 0;
        if (some) f.cand[v] = e;
        else if (v >= 0) f.colour[v] = ~c;
        wave_min_into(best_w, c, edge_weight(e), some);
        if (ALL_OUT) continue;
        const int at = block_append<THREADS>(some, f.words + CSR_ACTIVE + (round + 1) % 3);
        if (some) to[at] = v;
        __syncthreads();
    }
}

// ... and which of the edges of that weight it is
__global__ void __launch_bounds__(TB) k_csr_select(CsrForest f, int round)
{
    if (halted(f)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        f.words[CSR_ACTIVE + (round + 2) % 3] = list_is_all(f, round + 1) ? f.V : 0;
        f.words[CSR_ROOTS + (round + 2) % 3] = 0;
    }
    const int n = f.words[CSR_ACTIVE + (round + 1) % 3];
    const int32_t* list = f.active[(round + 1) & 1];
    const bool all = list_is_all(f, round);
    for (long long i = (long long)blockIdx.x * TB + threadIdx.x; i < n; i += (long long)gridDim.x * TB) {
        const int v = all ? (int)i : list[i], c = f.colour[v];
        if (all && c < 0) continue;
        const unsigned long long e = f.cand[v];
        if (edge_weight(e) == f.best_w[round & 1][c]) min_into(&f.best_e[round & 1][c], edge_ends(v, edge_end(e)));
    }
}

// Whether component `other` has no edge that is e or comes before it, though e leads to it: then e is not in both rows.  Hooks that
// pass this never form a cycle.
__device__ inline bool one_sided(uint32_t other_w, unsigned long long other_e, uint32_t w, unsigned long long e)
{
    return other_w > w || (other_w == w && other_e > e);
}

// Additions to two lists at once: `a` and `b` become the places of those of a thread's items that are on.  Every thread of the workgroup of
// WIDE must call it.
template <int ITEMS>
__device__ inline void append_two(int (&a)[ITEMS], int (&b)[ITEMS], int32_t* count_a, int32_t* count_b)
{
    constexpr int WAVES = WIDE / 64;
    __shared__ int count[2][WAVES], first[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int na = 0, nb = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const unsigned long long ma = __ballot(a[k] != 0), mb = __ballot(b[k] != 0);
        a[k] = a[k] ? na + __popcll(ma & ((1ull << lane) - 1)) : -1;
        b[k] = b[k] ? nb + __popcll(mb & ((1ull << lane) - 1)) : -1;
        na += __popcll(ma);
        nb += __popcll(mb);
    }
    if (lane == 0) { count[0][wave] = na; count[1][wave] = nb; }
    __syncthreads();
    int before_a = 0, before_b = 0, total[2] = {0, 0};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        before_a += w < wave ? count[0][w] : 0;
        before_b += w < wave ? count[1][w] : 0;
        total[0] += count[0][w];
        total[1] += count[1][w];
    }
    if (lane == 0 && wave < 2) first[wave] = total[wave] > 0 ? atomicAdd(wave == 0 ? count_a : count_b, total[wave]) : 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        a[k] += a[k] >= 0 ? first[0] + before_a : 0;
        b[k] += b[k] >= 0 ? first[1] + before_b : 0;
    }
    __syncthreads();
}

// One thread per root: append the component's edge (once per undirected edge) and hook it to the component at the other end.  Two
// that chose the same edge keep the smaller root; roots that stay get cleared minima for the next round.
__global__ void __launch_bounds__(WIDE) k_csr_commit(CsrForest f, int round)
{
    if (all_halted(f)) return;
    const int n = f.words[CSR_ROOTS + round % 3];
    const int32_t* from = f.roots[round & 1];
    int32_t* to = f.roots[(round + 1) & 1];
    const uint32_t* best_w = f.best_w[round & 1];
    const unsigned long long* best_e = f.best_e[round & 1];
    for (long long base = (long long)blockIdx.x * WIDE; base < n; base += (long long)gridDim.x * WIDE) {
        const long long i = base + threadIdx.x;
        int adds[1] = {0}, stays[1] = {0};
        int c = 0, lo = 0, hi = 0;
        uint32_t w = INF_BITS;
        if (i < n) {
            c = from[i];
            w = best_w[c];
            if (w != INF_BITS) {                                   // (else: a finished tree)
                const unsigned long long e = best_e[c];
                lo = (int)(e >> 32); hi = (int)(e & 0xffffffffull);
                int other = -1;
                if (!in_range(lo, f.V) || !in_range(hi, f.V)) report(f, 8);
                else {
                    const int cl = f.colour[lo], ch = f.colour[hi];        // (both are active)
                    other = cl == c ? ch : (ch == c ? cl : -1);
                    if (!in_range(other, f.V) || other == c) { report(f, 9); other = -1; }
                }
                if (other >= 0) {
                    const uint32_t other_w = best_w[other];
                    const unsigned long long other_e = other_w == w ? best_e[other] : 0ull;
                    const bool mutual = other_w == w && other_e == e;
                    if (one_sided(other_w, other_e, w, e)) report(f, 15);
                    else {
                        adds[0] = !mutual || c < other;
                        stays[0] = mutual && c < other;
                        if (!stays[0]) f.hook[c] = other;
                    }
                }
            }
        }
        append_two(adds, stays, f.words + CSR_EDGES, f.words + CSR_ROOTS + (round + 1) % 3);
        if (adds[0] >= 0 && adds[0] < f.V - 1) { f.e_lo[adds[0]] = lo; f.e_hi[adds[0]] = hi; f.e_w[adds[0]] = __uint_as_float(w); }
        if (stays[0] >= 0) { to[stays[0]] = c; f.best_w[(round + 1) & 1][c] = INF_BITS; f.best_e[(round + 1) & 1][c] = ~0ull; }
    }
}

// ... in round 0, where every vertex is a root and what it needs of the other one is in one word.  ITEMS vertices a thread, because additions
// to one word come one after another, about 10 ns each.  1M vertices: 47 us with weights, ends and colours in words of their own and two additions
// per 1024 vertices, 32 with the one word, 21 with two per 4096.
template <int ITEMS>
__global__ void __launch_bounds__(WIDE) k_csr_commit_first(CsrForest f)
{
    if (all_halted(f)) return;
    const long long base = (long long)blockIdx.x * (WIDE * ITEMS) + threadIdx.x;
    unsigned long long mine[ITEMS], theirs[ITEMS];
    int adds[ITEMS], stays[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) mine[k] = base + k * WIDE < f.V ? f.cand[base + k * WIDE] : NO_EDGE;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) theirs[k] = edge_end(mine[k]) >= 0 ? f.cand[edge_end(mine[k])] : NO_EDGE;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int c = (int)(base + k * WIDE), other = edge_end(mine[k]);
        const bool mutual = edge_weight(theirs[k]) == edge_weight(mine[k]) && edge_end(theirs[k]) == c;
        adds[k] = stays[k] = 0;
        if (other < 0) continue;
        if (one_sided(edge_weight(theirs[k]), edge_ends(other, edge_end(theirs[k])), edge_weight(mine[k]), edge_ends(c, other))) report(f, 15);
        else {
            adds[k] = !mutual || c < other;
            stays[k] = mutual && c < other;
            if (!stays[k]) f.hook[c] = other;
        }
    }
    append_two(adds, stays, f.words + CSR_EDGES, f.words + CSR_ROOTS + 1);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int c = (int)(base + k * WIDE);
        if (adds[k] >= 0 && adds[k] < f.V - 1) {
            const unsigned long long e = edge_ends(c, edge_end(mine[k]));
            f.e_lo[adds[k]] = (int)(e >> 32); f.e_hi[adds[k]] = (int)(e & 0xffffffffull); f.e_w[adds[k]] = __uint_as_float(edge_weight(mine[k]));
        }
        if (stays[k] >= 0) { f.roots[1][stays[k]] = c; f.best_w[1][c] = INF_BITS; f.best_e[1][c] = ~0ull; }
    }
}

// Active vertex v takes the root at the end of its component's hooks as its colour and shortens the way for the others; false where
// that is more than FOLLOW_STEPS away: the colour it has then is one to go on from.
__device__ inline bool follow(const CsrForest& f, int v, bool again)
{
    const int c = f.colour[v];
    int r = c;
    bool end = false;
    for (int s = 0; s < FOLLOW_STEPS && !end; ++s) {
        if (!in_range(r, f.V)) { report(f, 13); return true; }
        const int h = *reinterpret_cast<volatile int32_t*>(f.hook + r);
        end = h == r;
        r = h;
    }
    if (r != c) {
        f.colour[v] = r;
        if (end || again) f.hook[c] = r;
    }
    return end;
}
__global__ void __launch_bounds__(TB) k_csr_follow(CsrForest f, int round, int again)
{
    if (f.words[CSR_ERROR] != 0 || (!again && f.words[CSR_CHAINS] != 0)) return;
    const int n = f.words[CSR_ACTIVE + (round + 1) % 3];
    const int32_t* list = f.active[(round + 1) & 1];
    const bool all = list_is_all(f, round);
    for (long long i = (long long)blockIdx.x * TB + threadIdx.x; i < n; i += (long long)gridDim.x * TB) {
        const int v = all ? (int)i : list[i];
        if (all && f.colour[v] < 0) continue;
        if (!follow(f, v, again != 0)) atomicMax(f.words + CSR_CHAINS, round + 1);
    }
}

// All rounds from `round` on in one workgroup, once few vertices are active: a round's four launches take 30 us whatever they do.
// A call with 1600 vertices: 202 us with rounds over all vertices, 199 over lists, 150 so; 4096 to 4900 vertices: 223 so and 201 by
// launches; 14 400: 480 and 250.  So up to 2048; and fewer where they have more than 12 entries each, which one CU reads: 1500 vertices with 40
// entries 402 so and 280 by launches, 300 with 80 260 and 297.
__global__ void __launch_bounds__(WIDE) k_csr_tail(CsrForest f, int round, unsigned long long* __restrict__ host, uint32_t seq)
{
    __shared__ int s_active, s_roots, s_edges, s_chain;
    const int tid = threadIdx.x;
    int n = f.words[CSR_ACTIVE + round % 3], nr = f.words[CSR_ROOTS + round % 3], rounds = round;
    bool done = halted(f) || f.words[CSR_EDGES] >= f.V - 1;
    if (tid == 0) s_edges = f.words[CSR_EDGES];
    __syncthreads();
    for (int r = round; !done; ++r) {
        const int32_t* from = f.active[r & 1];
        int32_t* to = f.active[(r + 1) & 1];
        uint32_t *best_w = f.best_w[r & 1], *next_w = f.best_w[(r + 1) & 1];
        unsigned long long *best_e = f.best_e[r & 1], *next_e = f.best_e[(r + 1) & 1];
        const int before = s_edges;
        if (tid == 0) { s_active = s_roots = 0; }
        __syncthreads();
        for (int i0 = 0; i0 < n; i0 += WIDE) {
            const int i = i0 + tid;
            int v = -1, c = 0;
            if (i < n) {
                v = from[i];
                c = f.colour[v];
                if (!in_range(c, f.V)) { report(f, 11); v = -1; }
            }
            const unsigned long long e = row_edge<false>(f, v, c);
            const bool some = edge_end(e) >= 0;
            if (some) {
                f.cand[v] = e;
                to[atomicAdd(&s_active, 1)] = v;
            } else if (v >= 0) f.colour[v] = ~c;
            wave_min_into(best_w, c, edge_weight(e), some);
        }
        __syncthreads();
        n = s_active;
        for (int i = tid; i < n; i += WIDE) {
            const int v = to[i], c = f.colour[v];
            const unsigned long long e = f.cand[v];
            if (edge_weight(e) == __hip_atomic_load(best_w + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) min_into(&best_e[c], edge_ends(v, edge_end(e)));
        }
        __syncthreads();
        for (int i = tid; i < nr; i += WIDE) {
            const int c = f.roots[r & 1][i];
            const uint32_t w = __hip_atomic_load(best_w + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (w == INF_BITS) continue;
            const unsigned long long e = __hip_atomic_load(best_e + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int lo = (int)(e >> 32), hi = (int)(e & 0xffffffffull);
            if (!in_range(lo, f.V) || !in_range(hi, f.V)) { report(f, 8); continue; }
            const int cl = f.colour[lo], ch = f.colour[hi];
            const int other = cl == c ? ch : (ch == c ? cl : -1);
            if (!in_range(other, f.V) || other == c) { report(f, 9); continue; }
            const uint32_t other_w = __hip_atomic_load(best_w + other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long other_e = __hip_atomic_load(best_e + other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (one_sided(other_w, other_e, w, e)) { report(f, 15); continue; }
            const bool mutual = other_w == w && other_e == e;
            if (!mutual || c < other) {
                const int slot = atomicAdd(&s_edges, 1);
                if (slot < f.V - 1) { f.e_lo[slot] = lo; f.e_hi[slot] = hi; f.e_w[slot] = __uint_as_float(w); }
            }
            if (mutual && c < other) {
                f.roots[(r + 1) & 1][atomicAdd(&s_roots, 1)] = c;
                __hip_atomic_store(next_w + c, INF_BITS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(next_e + c, ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else f.hook[c] = other;
        }
        __syncthreads();
        nr = s_roots;
        for (int turn = 0;; ++turn) {
            if (tid == 0) s_chain = 0;
            __syncthreads();
            for (int i = tid; i < n; i += WIDE)
                if (!follow(f, to[i], true)) s_chain = 1;
            __syncthreads();
            if (s_chain == 0 || turn > 64) break;
            __syncthreads();
        }
        if (tid == 0 && s_chain != 0) report(f, 10);
        ++rounds;
        __syncthreads();
        done = s_edges == before || s_edges >= f.V - 1 || rounds > 64 + round || f.words[CSR_ERROR] != 0;
        __syncthreads();
    }
    if (tid == 0) {
        f.words[CSR_EDGES] = s_edges;
        const int said[CSR_TOLD] = {rounds | f.words[CSR_TIES], s_edges, f.words[CSR_CHAINS], f.words[CSR_ERROR]};
        for (int i = 0; i < CSR_TOLD; ++i)
            __hip_atomic_store(host + i, ((unsigned long long)seq << 32) | (unsigned int)said[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// (a colour was up to date when its vertex stopped being active)
__global__ void __launch_bounds__(TB) k_csr_colours(CsrForest f, int32_t* __restrict__ out)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v >= f.V || halted(f)) return;
    int r = f.colour[v];
    r = r < 0 ? ~r : r;
    for (int s = 0; s < f.V; ++s) {
        if (!in_range(r, f.V)) { report(f, 14); r = -1; break; }
        const int h = f.hook[r];
        if (h == r) break;
        r = h;
    }
    out[v] = r;
}

// Every entry leads to the same tree as its row belongs to.  (The rounds take an entry to a vertex that is no longer active for one
// inside the component, which it is only where the other row has it too.)
__device__ inline bool closed_part(const CsrForest& f, const int32_t* __restrict__ colours, int c, unsigned int at, unsigned int end, unsigned int step)
{
    bool closed = true;
    for (unsigned int e0 = at; e0 < end; e0 += step) {
        int u[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = e0 + j < end ? f.indices[e0 + j] : -1;
#pragma unroll
        for (int j = 0; j < 4; ++j) closed = closed && (u[j] < 0 || colours[u[j]] == c);
    }
    return closed;
}
__global__ void __launch_bounds__(TB) k_csr_closed(CsrForest f, const int32_t* __restrict__ colours)
{
    const int v = blockIdx.x * TB + threadIdx.x, lane = threadIdx.x & 63;
    // (a failed check or unfollowed hooks: no colours, and perhaps no rows that may be read)
    if (halted(f)) return;
    const bool mine = v < f.V;
    const int c = mine ? colours[v] : 0;
    const unsigned int at = mine ? (unsigned int)f.offsets[v] : 0u, end = mine ? (unsigned int)f.offsets[v + 1] : 0u;
    const bool is_long = end - at > LONG_ROW;
    bool closed = is_long || closed_part(f, colours, c, at, end, 4);
    for (unsigned long long todo = __ballot(is_long); todo != 0; todo &= todo - 1) {
        const int owner = __builtin_ctzll(todo);
        closed &= closed_part(f, colours, __shfl(c, owner), (unsigned int)__shfl((int)at, owner) + 4 * lane, (unsigned int)__shfl((int)end, owner), 256);
    }
    if (!closed) report(f, 16);
}

// Lowest bits of the weights that the sort of that many edges leaves to runs: three passes of 8 bits for the other 24, of which there are 65 536
// values between powers of two.  Beyond 2^20 edges the runs grow longer, the sample finds too many of the same, and the fourth pass is made.  Forests of road-like
// graphs with weights U[1, 100), three passes and four, in us: 90 000 vertices 371 and 400, 490 000 528 and 550, 1 048 576 746 and 765, 1.2M 818 and 836, 1.5M 987 (too
// many of the same) and 937, 2M 1135 and 1150, 3M 1613 and 1615, 4M 2604 (too many) and 2087.
static inline int low_bits(int E) { return E <= (1 << 20) ? 7 : 0; }
// The words of a call; and whether many edges have the same weight in the bits that are sorted by, by a sample of the entries: each looks for its
// weight in a table of those before it.  Many: more pairs than runs of 16 edges would give, or one weight that as many have as LONG_RUN edges would, beyond which
// k_csr_long_runs takes longer than the other sort (a hundredth of 160 000 vertices' edges 463 us and 440 by the other, 3 % of 90 000's 417 and 386, a hundredth of
// 2.25M's 1614 and 1374).  1024 entries, 4.2 us; beyond 2^21 vertices, where so few entries have hardly a pair in runs of 16, 4096 (15 us; whole weights up to 100 000 of 4M
// vertices, in runs of 40, passed for few of the same by 1024: 3530 us, and 2280 so).
constexpr long long LONG_RUN = 1200;
template <int SAMPLE>
__global__ void __launch_bounds__(WIDE) k_csr_words(CsrForest f, int low)
{
    constexpr int TABLE = 4 * (SAMPLE < 2048 ? SAMPLE : 2048), EACH = SAMPLE / WIDE;
    static_assert(TABLE == 4096 || TABLE == 8192, "the hash has 12 bits or 13");
    __shared__ uint32_t table[TABLE], times[TABLE / 2];       // (times: 16 bits each)
    const int tid = threadIdx.x;
    for (int i = tid; i < TABLE; i += WIDE) table[i] = 0xffffffffu;
    for (int i = tid; i < TABLE / 2; i += WIDE) times[i] = 0u;
    __syncthreads();
    int found = 0;
    bool common = false;
    const long long often = SAMPLE * LONG_RUN / f.V;
    if (f.E >= SAMPLE) {
        uint32_t w[EACH];
#pragma unroll
        for (int k = 0; k < EACH; ++k) w[k] = (__float_as_uint(f.weights[(long long)f.E * (k * WIDE + tid) / SAMPLE]) & 0x7fffffffu) >> low;
#pragma unroll
        for (int k = 0; k < EACH; ++k) {
            uint32_t at = (w[k] * 0x9e3779b1u) >> (TABLE == 4096 ? 20 : 19), was = 0u;
#pragma unroll 1
            for (int i = 0; i < TABLE; ++i, at = (at + 1) & (TABLE - 1)) {
                was = atomicCAS(&table[at], 0xffffffffu, w[k]);
                if (was == w[k] || was == 0xffffffffu) break;
            }
            if (was != w[k]) continue;
            ++found;
            const uint32_t before = atomicAdd(&times[at >> 1], at & 1 ? 1u << 16 : 1u);
            common = common || (int)(at & 1 ? before >> 16 : before & 0xffffu) >= (often < 3 ? 3 : (int)often);
        }
    }
    int ties = 0;
    for (int k = 1; k <= EACH; ++k) ties += __syncthreads_count(found >= k);
    const bool many = __syncthreads_or(common) != 0 || ties > 4 + (int)((16ll * SAMPLE * SAMPLE / 2) / f.V);
    const bool all = (tid == CSR_ACTIVE + 1 && list_is_all(f, 0)) || (tid == CSR_ACTIVE + 2 && list_is_all(f, 1));
    if (tid < 64) f.words[tid] = all ? f.V : tid == CSR_TIES && many ? (int)CSR_MANY_TIES : 0;
}

hipError_t csr_start(const CsrForest& f, hipStream_t s)
{
    if (f.V > 1 << 21) hipLaunchKernelGGL(k_csr_words<4096>, dim3(1), dim3(WIDE), 0, s, f, low_bits(f.V));
    else hipLaunchKernelGGL(k_csr_words<1024>, dim3(1), dim3(WIDE), 0, s, f, low_bits(f.V));
    if (list_is_all(f, 0)) hipLaunchKernelGGL((k_csr_first<TB, true>), dim3(blocks_for(f.V)), dim3(TB), 0, s, f);
    else hipLaunchKernelGGL((k_csr_first<TB, false>), dim3(blocks_for(f.V)), dim3(TB), 0, s, f);
    if (f.V > FEW) hipLaunchKernelGGL(k_csr_commit_first<4>, dim3(blocks_for(f.V, 4 * WIDE)), dim3(WIDE), 0, s, f);
    else hipLaunchKernelGGL(k_csr_commit_first<1>, dim3(blocks_for(f.V, WIDE)), dim3(WIDE), 0, s, f);
    hipLaunchKernelGGL(k_csr_follow, dim3(blocks_for(f.V)), dim3(TB), 0, s, f, 0, 0);
    return hipGetLastError();
}

hipError_t csr_round(const CsrForest& f, int round, int vertices, int roots, unsigned long long* host, uint32_t seq, hipStream_t s)
{
    const dim3 per_vertex(blocks_for(vertices < 1 ? 1 : vertices));
    if (list_is_all(f, round)) hipLaunchKernelGGL((k_csr_scan<TB, true, true>), per_vertex, dim3(TB), 0, s, f, round, host, seq);
    else if (list_is_all(f, round - 1)) hipLaunchKernelGGL((k_csr_scan<WIDE, true, false>), dim3(append_blocks(vertices)), dim3(WIDE), 0, s, f, round, host, seq);
    else if (vertices > FEW) hipLaunchKernelGGL((k_csr_scan<WIDE, false, false>), dim3(append_blocks(vertices)), dim3(WIDE), 0, s, f, round, host, seq);
    else hipLaunchKernelGGL((k_csr_scan<TB, false, false>), per_vertex, dim3(TB), 0, s, f, round, host, seq);
    hipLaunchKernelGGL(k_csr_select, per_vertex, dim3(TB), 0, s, f, round);
    hipLaunchKernelGGL(k_csr_commit, dim3(append_blocks(roots)), dim3(WIDE), 0, s, f, round);
    hipLaunchKernelGGL(k_csr_follow, per_vertex, dim3(TB), 0, s, f, round, 0);
    return hipGetLastError();
}

hipError_t csr_follow_again(const CsrForest& f, int round, int vertices, hipStream_t s)
{
    hipLaunchKernelGGL(k_csr_follow, dim3(blocks_for(vertices < 1 ? 1 : vertices)), dim3(TB), 0, s, f, round, 1);
    return hipGetLastError();
}

hipError_t csr_tail(const CsrForest& f, int round, unsigned long long* host, uint32_t seq, hipStream_t s)
{
    hipLaunchKernelGGL(k_csr_tail, dim3(1), dim3(WIDE), 0, s, f, round, host, seq);
    return hipGetLastError();
}

hipError_t csr_colours(const CsrForest& f, int32_t* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_csr_colours, dim3(blocks_for(f.V)), dim3(TB), 0, s, f, out);
    return hipGetLastError();
}

hipError_t csr_closed(const CsrForest& f, const int32_t* colours, hipStream_t s)
{
    hipLaunchKernelGGL(k_csr_closed, dim3(blocks_for(f.V)), dim3(TB), 0, s, f, colours);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------- sort
// By (weight, smaller end, larger end).  Where few edges have nearly the same weight: one sort of weights with the edges' numbers, by all but the
// lowest bits while the runs that leaves are short, and every edge counts those of its run that come before it.  The edges of runs of more than RUN_MOST
// are listed, and the caller has them placed in a launch of their own, or, where they are many, takes another way.  1M edges: 220 us by the smaller ends first
// (below), 165 by all bits, 140 so, of which the three passes take 83 and the runs 30 (random words of the edges' ends; 41 with the neighbours' weights read from memory).
constexpr int RUN_MOST = 64;
__global__ void __launch_bounds__(TB) k_csr_in_runs(const uint32_t* __restrict__ wbits, const uint32_t* __restrict__ number, const int32_t* __restrict__ lo,
                                                   const int32_t* __restrict__ hi, int E, int low, int32_t* __restrict__ out_lo, int32_t* __restrict__ out_hi,
                                                   float* __restrict__ out_w, int32_t* __restrict__ listed, unsigned long long* __restrict__ ends, int32_t* __restrict__ count)
{
    __shared__ uint32_t near[RUN_MOST + TB + RUN_MOST];        // the workgroup's weights and those a run can reach
    const int first = blockIdx.x * TB, i = first + threadIdx.x;
    for (int j = threadIdx.x; j < RUN_MOST + TB + RUN_MOST; j += TB) {
        const int at = first - RUN_MOST + j;
        near[j] = at >= 0 && at < E ? wbits[at] : 0u;
    }
    const uint32_t e = i < E ? number[i] : 0u;
    const int a = lo[e], b = hi[e];
    __syncthreads();
    if (i >= E) return;
    const uint32_t* mine = near + RUN_MOST + threadIdx.x;
    const uint32_t w = *mine;
    auto before = [&](int j, uint32_t o) -> int {
        if (o != w) return o < w ? 1 : 0;
        const uint32_t n = number[j];
        const int oa = lo[n];
        return oa < a || (oa == a && hi[n] < b) ? 1 : 0;
    };
    int from = i, to = i + 1;
    for (; from > 0 && i - from < RUN_MOST && ((mine[from - 1 - i] ^ w) >> low) == 0u; --from) {}
    for (; to < E && to - i <= RUN_MOST && ((mine[to - i] ^ w) >> low) == 0u; ++to) {}
    const bool is_long = to - from > RUN_MOST;
    const unsigned long long all = __ballot(is_long);
    if (all != 0) {
        const int first = __builtin_ctzll(all);
        int base = 0;
        if ((int)(threadIdx.x & 63) == first) base = atomicAdd(count, __popcll(all));
        base = __shfl(base, first);
        if (is_long) {
            listed[base + __builtin_amdgcn_mbcnt_hi((unsigned int)(all >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)all, 0u))] = i;
            ends[i] = ((unsigned long long)(unsigned int)a << 32) | (unsigned int)b;
            return;
        }
    }
    int at = from;
    for (int j = from; j < to; ++j)
        if (j != i) at += before(j, mine[j - i]);
    out_lo[at] = a; out_hi[at] = b; out_w[at] = __uint_as_float(w);
}
// The first of [lo, hi] from which on beyond(j) holds, as it does from hi on, looked for by a wavefront at 64 places at a time (lo, hi the same for all lanes).
template <typename F>
__device__ inline int wave_first(int lo, int hi, F&& beyond)
{
    const int lane = threadIdx.x & 63;
    while (lo < hi) {
        const int step = (hi - lo + 63) / 64;
        const long long at = lo + (long long)lane * step;
        const unsigned long long yes = __ballot(at >= hi || beyond((int)at));
        const int k = yes != 0 ? __builtin_ctzll(yes) : 64;
        if (k < 64 && lo + (long long)k * step < hi) hi = lo + k * step;
        if (k > 0) lo += (k - 1) * step + 1;
    }
    return lo;
}
// 64 listed edges a workgroup, whose wavefronts share out their run: what it is compared with is the same for all lanes, and comes by scalar loads (by vector loads of one
// address, 16 cycles each, a run of 1600 edges took 30 us).  Edges of several runs look for their own.
// Road-like graphs, a share of the weights the same, us of the whole call (a run of 65 made the whole sort vain before; this kernel takes 9 to 13):
//   90 000 vertices, .001: 562 and 399; 160 000, .003: 613 and 443; 490 000, .003: 743 and 570; 1M, .001: 1014 and 795; 4M, .0002: 2619 and 2125
__global__ void __launch_bounds__(WIDE) k_csr_long_runs(const uint32_t* __restrict__ wbits, const unsigned long long* __restrict__ ends, const int32_t* __restrict__ listed,
                                                        int n, int E, int low, int32_t* __restrict__ out_lo, int32_t* __restrict__ out_hi, float* __restrict__ out_w)
{
    constexpr int WAVES = WIDE / 64, AT_ONCE = 8;
    __shared__ int before[WAVES][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), at = blockIdx.x * 64 + lane;
    const int i = at < n ? listed[at] : -1;
    const uint32_t w = i >= 0 ? wbits[i] : 0u;
    const unsigned long long mine = i >= 0 ? ends[i] : 0ull;
    int less = 0;
    auto count = [&](uint32_t o, unsigned long long other) { less += (int)(o < w) | ((int)(o == w) & (int)(other < mine)); };
    // (sorted by the bits above `low`; the first lane has an edge)
    const int i0 = __builtin_amdgcn_readfirstlane(i);
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)w);
    int from = wave_first(0, i0, [&](int j) { return ((wbits[j] ^ w0) >> low) == 0u; });
    const int to0 = wave_first(i0 + 1, E, [&](int j) { return ((wbits[j] ^ w0) >> low) != 0u; });
    if (__all(i < 0 || (i >= from && i < to0))) {
        const int from0 = __builtin_amdgcn_readfirstlane(from), len = __builtin_amdgcn_readfirstlane(to0) - from0;
        const int j1 = from0 + (int)((long long)len * (wave + 1) / WAVES);
        int j = from0 + (int)((long long)len * wave / WAVES);
        for (; j + AT_ONCE <= j1; j += AT_ONCE) {
            uint32_t o[AT_ONCE];
            unsigned long long other[AT_ONCE];
#pragma unroll
            for (int k = 0; k < AT_ONCE; ++k) { o[k] = wbits[j + k]; other[k] = ends[j + k]; }
#pragma unroll
            for (int k = 0; k < AT_ONCE; ++k) count(o[k], other[k]);
        }
        for (; j < j1; ++j) count(wbits[j], ends[j]);
    } else {
        int to = 0;
        from = 0;
        if (i >= 0) {
            for (int end = i; from < end;) {
                const int mid = from + (end - from) / 2;
                if ((wbits[mid] ^ w) >> low) from = mid + 1; else end = mid;
            }
            to = i + 1;
            for (int end = E; to < end;) {
                const int mid = to + (end - to) / 2;
                if ((wbits[mid] ^ w) >> low) end = mid; else to = mid + 1;
            }
        }
        const int j1 = from + (int)((long long)(to - from) * (wave + 1) / WAVES);
        for (int j = from + (int)((long long)(to - from) * wave / WAVES); j < j1; ++j) count(wbits[j], ends[j]);
    }
    before[wave][lane] = less;
    __syncthreads();
    if (wave != 0 || i < 0) return;
    int place = from;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) place += before[v][lane];
    out_lo[place] = (int)(mine >> 32); out_hi[place] = (int)(mine & 0xffffffffull); out_w[place] = __uint_as_float(w);
}

// Where many do: the smaller ends are counted and the edges placed by them, which takes a few passes of
// random words where a radix sort by both ends takes five over all of them; each vertex then orders its few edges by the other
// end, and one stable sort by weight follows.  A vertex with more than LO_MOST edges to larger ones raises a flag while they are
// counted; nothing is placed then, and the caller, whom the placing tells, takes edge_sort instead.  1M edges: 240 us with two radix
// sorts, 205 so.
constexpr int LO_MOST = 32;
__global__ void __launch_bounds__(TB) k_lo_clear(int32_t* __restrict__ count, int V, int32_t* __restrict__ flag)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v <= V) count[v] = 0;
    if (v == 0) *flag = 0;
}
// Additions to one word come one after another: a star of 1M vertices, 12 ms with one for every edge.  So a wavefront adds once for all
// edges of its first one's vertex, and looks for the flag first; LO_COUNT_BLOCKS bounds how many can add before they see it.
constexpr int LO_COUNT_BLOCKS = 1024;
__global__ void __launch_bounds__(TB) k_lo_count(const int32_t* __restrict__ lo, int E, int32_t* __restrict__ count, int32_t* __restrict__ rank, int32_t* __restrict__ flag)
{
    for (long long base = (long long)blockIdx.x * TB; base < E; base += (long long)gridDim.x * TB) {
        if (*reinterpret_cast<volatile int32_t*>(flag) != 0) return;
        const long long e = base + threadIdx.x;
        const int v = e < E ? lo[e] : -1;
        const unsigned long long same = __ballot(v >= 0 && v == __builtin_amdgcn_readfirstlane(v));
        int r = 0;
        if (same >> (threadIdx.x & 63) & 1) {
            const int first = __builtin_ctzll(same);
            if ((threadIdx.x & 63) == first) r = atomicAdd(count + v, __popcll(same));
            r = __shfl(r, first) + __builtin_amdgcn_mbcnt_hi((unsigned int)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)same, 0u));
        } else if (v >= 0) r = atomicAdd(count + v, 1);
        if (e < E) rank[e] = r;
        if (r >= LO_MOST) *flag = 1;
    }
}
__global__ void __launch_bounds__(TB) k_lo_place(const int32_t* __restrict__ lo, const int32_t* __restrict__ hi, const float* __restrict__ w, int E,
                                                 const int32_t* __restrict__ offset, const int32_t* __restrict__ rank, uint32_t* __restrict__ wbits,
                                                 unsigned long long* __restrict__ ends, const int32_t* __restrict__ flag, unsigned long long* __restrict__ host, uint32_t seq)
{
    const int e = blockIdx.x * TB + threadIdx.x;
    if (e == 0) __hip_atomic_store(host, ((unsigned long long)seq << 32) | (unsigned int)*flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (e >= E || *flag != 0) return;
    const int at = offset[lo[e]] + rank[e];
    wbits[at] = __float_as_uint(w[e]);
    ends[at] = ((unsigned long long)(unsigned int)lo[e] << 32) | (unsigned int)hi[e];
}
__global__ void __launch_bounds__(TB) k_lo_order(const int32_t* __restrict__ offset, int V, uint32_t* __restrict__ wbits, unsigned long long* __restrict__ ends,
                                                 const int32_t* __restrict__ flag)
{
    const int v = blockIdx.x * TB + threadIdx.x;
    if (v >= V || *flag != 0) return;
    const int a = offset[v], b = offset[v + 1];
    for (int i = a + 1; i < b; ++i) {
        const unsigned long long e = ends[i];
        const uint32_t w = wbits[i];
        int j = i - 1;
        for (; j >= a && ends[j] > e; --j) { ends[j + 1] = ends[j]; wbits[j + 1] = wbits[j]; }
        ends[j + 1] = e; wbits[j + 1] = w;
    }
}
__global__ void __launch_bounds__(TB) k_lo_unpack(const unsigned long long* __restrict__ ends, const uint32_t* __restrict__ wbits, int E, int32_t* __restrict__ lo,
                                                  int32_t* __restrict__ hi, float* __restrict__ w)
{
    const int i = blockIdx.x * TB + threadIdx.x;
    if (i >= E) return;
    lo[i] = (int)(ends[i] >> 32); hi[i] = (int)(ends[i] & 0xffffffffull); w[i] = __uint_as_float(wbits[i]);
}

// (radix passes from 32 768 pairs on, as in edge_sort)
using radix_passes = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config, rocprim::default_config, 32768>;
bool csr_sort_fits(int V, int E, size_t temp_bytes)
{
    size_t a = 0, b = 0;
    int32_t* i = nullptr; uint32_t* k32 = nullptr; unsigned long long* k64 = nullptr;
    (void)rocprim::exclusive_scan(nullptr, a, i, i, 0, (size_t)V + 1, rocprim::plus<int32_t>(), (hipStream_t)0);
    (void)rocprim::radix_sort_pairs<radix_passes>(nullptr, b, k32, k32, k64, k64, (size_t)E, 0, 32, (hipStream_t)0);
    return a <= temp_bytes && b <= temp_bytes;
}
// (bits of weights that are not negative)
static hipError_t sort_weights_numbers(void* temp, size_t& bytes, const uint32_t* w, uint32_t* w_out, uint32_t* number, int E, hipStream_t s)
{
    return rocprim::radix_sort_pairs<radix_passes>(temp, bytes, w, w_out, rocprim::make_counting_iterator<uint32_t>(0u), number, (size_t)E, low_bits(E), 31, s);
}
bool csr_sort_in_runs_fits(int E, size_t temp_bytes)
{
    size_t a = 0;
    (void)sort_weights_numbers(nullptr, a, nullptr, nullptr, nullptr, E, (hipStream_t)0);
    return a <= temp_bytes;
}
hipError_t csr_sort_in_runs(const int32_t* lo, const int32_t* hi, const float* w, int E, const CsrSortScratch& t, int32_t* out_lo, int32_t* out_hi,
                            float* out_w, int32_t* count, hipStream_t s)
{
    size_t tb = t.temp_bytes;
    const hipError_t e = sort_weights_numbers(t.temp, tb, reinterpret_cast<const uint32_t*>(w), t.wbits_b, t.number, E, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_csr_in_runs, dim3(blocks_for(E)), dim3(TB), 0, s, t.wbits_b, t.number, lo, hi, E, low_bits(E), out_lo, out_hi, out_w, t.rank, t.ends_a, count);
    return hipGetLastError();
}
hipError_t csr_sort_long_runs(int n, int E, const CsrSortScratch& t, int32_t* out_lo, int32_t* out_hi, float* out_w, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_csr_long_runs, dim3(blocks_for(n, 64)), dim3(WIDE), 0, s, t.wbits_b, t.ends_a, t.rank, n, E, low_bits(E), out_lo, out_hi, out_w);
    return hipGetLastError();
}
hipError_t csr_sort_ends(const int32_t* lo, const int32_t* hi, const float* w, int E, int V, const CsrSortScratch& t, int32_t* flag, unsigned long long* host, uint32_t seq,
                         hipStream_t s)
{
    hipLaunchKernelGGL(k_lo_clear, dim3(blocks_for((long long)V + 1)), dim3(TB), 0, s, t.count, V, flag);
    const int blocks = blocks_for(E);
    hipLaunchKernelGGL(k_lo_count, dim3(blocks < LO_COUNT_BLOCKS ? blocks : LO_COUNT_BLOCKS), dim3(TB), 0, s, lo, E, t.count, t.rank, flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    size_t tb = t.temp_bytes;
    e = rocprim::exclusive_scan(t.temp, tb, t.count, t.offset, 0, (size_t)V + 1, rocprim::plus<int32_t>(), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lo_place, dim3(blocks_for(E)), dim3(TB), 0, s, lo, hi, w, E, t.offset, t.rank, t.wbits_a, t.ends_a, flag, host, seq);
    hipLaunchKernelGGL(k_lo_order, dim3(blocks_for(V)), dim3(TB), 0, s, t.offset, V, t.wbits_a, t.ends_a, flag);
    return hipGetLastError();
}
hipError_t csr_sort_weights(int E, const CsrSortScratch& t, int32_t* out_lo, int32_t* out_hi, float* out_w, hipStream_t s)
{
    size_t tb = t.temp_bytes;
    const hipError_t e = rocprim::radix_sort_pairs<radix_passes>(t.temp, tb, t.wbits_a, t.wbits_b, t.ends_a, t.ends_b, (size_t)E, 0, 32, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lo_unpack, dim3(blocks_for(E)), dim3(TB), 0, s, t.ends_b, t.wbits_b, E, out_lo, out_hi, out_w);
    return hipGetLastError();
}

}  // namespace slhc
