// Launch interface of the spanning forest of a CSR graph (csr_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace slhc {

// words: active vertices and roots of a round, three in turn; the number, from 1 on, of a round whose hooks are not followed to
// their end; edges (added to along with the roots, so not in their line); the first failed check; what the sort says; CSR_MANY_TIES where
// many weights are the same
enum { CSR_ACTIVE = 0, CSR_ROOTS = 32, CSR_CHAINS = 6, CSR_EDGES = 7, CSR_ERROR = 8, CSR_FLAG = 9, CSR_TIES = 10 };
constexpr unsigned int CSR_MANY_TIES = 0x80000000u;
struct CsrForest {
    const int32_t *offsets, *indices; const float* weights; int V, E;
    int32_t *colour, *hook;                    // [V]
    unsigned long long* cand;                  // [V] an active vertex's first edge out of its component: its weight's bits, the other end
    uint32_t* best_w[2]; unsigned long long* best_e[2];      // [V] by root, of even and odd rounds
    int32_t *active[2], *roots[2];             // [V] lists, likewise
    int32_t *e_lo, *e_hi; float* e_w;          // [V - 1]
    int32_t* words;                            // [64]
};
// Round 0: the input check and every vertex's lightest edge.
hipError_t csr_start(const CsrForest& f, hipStream_t s);
// Round 1, 2, ... for at most so many active vertices and roots.  On the way host[0 .. 3] get what round - 1 left: active vertices (and
// CSR_MANY_TIES), edges so far, the word of hooks not followed to their end (nothing is done then), the first failed check, each in the low half
// of a word with `seq` above it.
constexpr int CSR_TOLD = 4;
hipError_t csr_round(const CsrForest& f, int round, int vertices, int roots, unsigned long long* host, uint32_t seq, hipStream_t s);
// All rounds from `round` on; host[0] gets the rounds there were in all (and CSR_MANY_TIES).  For at most csr_tail_most active vertices (see k_csr_tail).
inline long long csr_tail_most(long long V, long long E)
{
    constexpr long long most = 2048, entries = 12;
    return E <= entries * V ? most : most * entries * V / E + 128;
}
hipError_t csr_tail(const CsrForest& f, int round, unsigned long long* host, uint32_t seq, hipStream_t s);
hipError_t csr_follow_again(const CsrForest& f, int round, int vertices, hipStream_t s);
// Colours of all vertices.  And the check that no entry leads from one tree to another (words[CSR_ERROR]), for which they have to be
// there and more than one.  Nothing after a failed check or with hooks not followed to their end.
hipError_t csr_colours(const CsrForest& f, int32_t* out, hipStream_t s);
hipError_t csr_closed(const CsrForest& f, const int32_t* colours, hipStream_t s);

// Edges by (weight, smaller end, larger end).
struct CsrSortScratch {
    int32_t *count, *offset;                   // [V + 1]
    int32_t* rank;                             // [E]
    uint32_t *number, *wbits_a, *wbits_b; unsigned long long *ends_a, *ends_b;        // [E]
    void* temp; size_t temp_bytes;
};
// Where few have the same weight.  *count (0 before) is the number of edges of long runs, whose places in the outputs are left open: up to CSR_LONG_MOST of them
// csr_sort_long_runs fills these, of more the outputs have to be made another way.
constexpr int CSR_LONG_MOST = 1 << 15;
bool csr_sort_in_runs_fits(int E, size_t temp_bytes);
hipError_t csr_sort_in_runs(const int32_t* lo, const int32_t* hi, const float* w, int E, const CsrSortScratch& t, int32_t* out_lo, int32_t* out_hi,
                            float* out_w, int32_t* count, hipStream_t s);
hipError_t csr_sort_long_runs(int n, int E, const CsrSortScratch& t, int32_t* out_lo, int32_t* out_hi, float* out_w, hipStream_t s);
// Else, in two steps: the first sets *flag where edge_sort has to do it instead, and tells host[0], with `seq` above the flag.
bool csr_sort_fits(int V, int E, size_t temp_bytes);
hipError_t csr_sort_ends(const int32_t* lo, const int32_t* hi, const float* w, int E, int V, const CsrSortScratch& t, int32_t* flag, unsigned long long* host, uint32_t seq,
                         hipStream_t s);
hipError_t csr_sort_weights(int E, const CsrSortScratch& t, int32_t* out_lo, int32_t* out_hi, float* out_w, hipStream_t s);

}  // namespace slhc
