// Launch interface of the passes that multiply every pair of rows once (pairs_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include "near_kernels.h"

namespace slhc {

constexpr int PAIRS_MOST = 1024;           // entries of a row's list at most

struct NearPairs {
    const unsigned char* frag; const float* negh; const int32_t* colour;      // the copy (colour: pairs_best)
    int tiles, steps, filled;              // steps of 16 columns a row's place has, and how many of them hold columns
    int blocks, from, to, nseg;            // block i meets the blocks i + from .. i + to - 1, in nseg shares
    // Pairs in either order may be searched for some blocks' rows at a time, `rows` from position `row0` on, which are the first ones of block `first`:
    // limit, counts, entries, lost and what follows are theirs.  (Else all rows: 0, 0, 128 tiles.)
    int first, row0, rows;
    int once;                              // every pair once, for both of its rows (to: half way round), or in either order for its first row
    int spread;                            // near_spread(blocks): place i of the circle has block i * spread % blocks of the copy
    float* limit;                          // pairs_emit: by position, the u from which on a pair matters to the row (NaN: none does)
    uint2* entries; int32_t* counts; int cap;      // pairs_emit: lists [rows][cap] of (u, position), appended to; counts beyond cap: some were lost
    // pairs_emit: rows whose lists overflowed, as far as pairs_tighten has counted them; beyond lost_most of them pairs_emit does nothing
    int32_t* lost; int lost_most;
    int cap_again;                         // pairs_left: entries of the lists of the search for the rows left over
    // (as NearBuffers) panels some of whose rows are not searched for again
    int32_t *todo, *todo_mark; int full_gone;      // full_gone: pairs in either order, those of rows whose lists are full
    // pairs_best: by position (w, position of the first of the 16 rows about it), w = max(0, -u) of the nearest row of another
    // colour so far; not 0x7f.. / all ones in the beginning.  both = 0: the block's own rows only are served
    unsigned long long* best; int both;
};
// waves: wavefronts per workgroup up to 128 columns (a block is half as many tiles; beyond, two)
hipError_t pairs_emit(const NearPairs& p, int waves, hipStream_t s);
hipError_t pairs_best(const NearPairs& p, hipStream_t s);
// Rows whose lists overflowed, or all of them after more than lost_most: their number in the matrix, position, an upper end of the squared
// distance of their kk-th nearest row, a counter set to 0; the list's counter becomes 0.
struct PairsLeft { int32_t *row, *pos, *counts, *count; float* reach; };
hipError_t pairs_left(const NearPairs& p, int kk, const NearScale* sc, float e, float nu, int d, int n_rows, const PairsLeft& out, hipStream_t s);
// The n rows left from `first` on, with lists [n][cap] of (product value, position): those that overflowed get the distance that follows
// and an empty list, the others a distance that nothing is within, and so does one to whom the distance is no news: its list would overflow again.
hipError_t pairs_again(const NearPairs& p, int kk, const NearScale* sc, float e, float nu, int d, int first, int n, const PairsLeft& left, hipStream_t s);
// last: by position, entries after the last call, 0 at first
hipError_t pairs_tighten(const NearPairs& p, int kk, const NearScale* sc, float e, float nu, int d, int32_t* last, hipStream_t s);

}  // namespace slhc
