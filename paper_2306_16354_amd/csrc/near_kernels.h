// Launch interface of the half-precision nearest-row engine (near_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace slhc {

// What the copies of one problem share (device): the power of two the rows are multiplied by, and the largest
// relative distance of a row from its rounded copy.
struct NearScale {
    float scale;
    unsigned int eps_bits;
    unsigned int huge;         // not 0: some row has values beyond float16
};

// The rows of a matrix rounded to float16, in tiles of 128 in the order the matrix instruction reads them.
// Every tile is an even sample of the rows, whatever order they are in (near_row); with `in_order` position p holds row p.
struct NearCopy {
    unsigned char* frag;       // [tiles][steps of 16 columns][4 blocks of 32 rows][64 lanes][16 bytes]
    float* negh;               // [tiles * 128] minus the half norm; -inf: no such row, +inf: values beyond float16
    float* negh_best;          // [tiles * 128] or nullptr: the same with -inf for the latter (candidates of 1-NN searches and near_assign)
    int32_t* colour;           // [tiles * 128] or nullptr
    // scratch of 1-NN searches for these rows as queries, or nullptr
    int32_t* left;             // [4 * tiles * 128]
    int32_t* count;            // [tiles * 128], cleared by near_make
    unsigned long long* best_at;    // [tiles * 128], set to ~0 by near_make (near_link)
    bool finite_padding;       // -1e38 instead of -inf (near_assign)
    bool in_order;
    int rows, tiles;
};

inline int near_tiles(long long n) { return (int)((n + 127) / 128); }
// steps of 16 columns: beyond 128 columns whole chunks of 64
inline int near_steps(int d) { return d <= 128 ? (d + 15) / 16 : (d + 63) / 64 * 4; }
inline size_t near_frag_bytes(long long n, int d) { return (size_t)near_tiles(n) * (size_t)near_steps(d) * 4096; }

struct NearBuffers {           // scratch of one call
    NearScale* scale;
    float* shift;              // [d]
    float* partial;            // near_stats_scratch_floats(d)
    unsigned char* batch; size_t batch_bytes;     // bounds, group maxima, entries and counts of one batch of queries
    unsigned char* pairs; size_t pairs_bytes;     // limits and lists of all rows (near_pairs_bytes), possibly the same memory; 0: none
    int32_t* todo;             // [2 + panels of 128 queries]: count, queries left by near_link, panels left to the list kernels
    int32_t* todo_mark;        // [panels]
    long long todo_panels;
};

struct NearProblem {
    const float* Xq; const float* Xc;      // the rows themselves (exact evaluation)
    int d, k;
    const int32_t* q_rows;                 // row of Xq behind query i (nullptr: i); entries outside [0, nq_rows) answer "nothing"
    int nq, nq_rows, nc;
    int exclude_self;                      // queries are the candidates; a row is not its own neighbour
    int coloured;                          // only candidates of another colour count
    int32_t* out_idx; float* out_dist;     // [nq, k]
    int32_t* evaluated;                    // optional [nq]: exactly evaluated pairs are added per query
};

size_t near_stats_scratch_floats(int d);
// (kk: k, plus one where a query meets itself)
size_t near_batch_bytes(long long nq, long long nc, int d, int kk);       // what NearBuffers::batch wants (less also works, down to one panel)
size_t near_least_batch_bytes(long long nq, long long nc, int d, int kk);
// what NearBuffers::pairs wants for a search of the rows among themselves; 0: such a search does not use it
size_t near_pairs_bytes(long long n, int d, int kk, bool* once = nullptr);

// (clears `clear` [clear_words], optional, on the way)
hipError_t near_stats(const float* X, int n, int d, const NearBuffers& b, uint32_t* clear, int clear_words, hipStream_t s);
// fills `out` from rows (clear_todo: and clears the panels left to the list kernels, as near_stats does)
// `rows` (nullptr: 0 .. n-1 of a matrix with n_src rows; n_dev: only the first *n_dev of them); hn / nonfinite (optional): the float32
// half norms by row and the flag of launch_half_norms; colour (optional): by row
hipError_t near_make(const float* X, int n_src, int d, const int32_t* rows, int n, const int32_t* colour, const NearBuffers& b,
                     const NearCopy& out, float* hn, unsigned int* nonfinite, hipStream_t s, bool clear_todo = false,
                     const int32_t* n_dev = nullptr, const int32_t* shift_row = nullptr);
// the colours of the rows of `c` into c.colour
hipError_t near_colours(const NearCopy& c, const int32_t* colour, hipStream_t s);
// For every row of q the row of c with the (nearly) largest product value, i.e. a nearest row up to the rounding of the
// copies, and the distance to that row: one pass.  best_at: [q.tiles * 128] words of scratch; c has finite padding.
hipError_t near_assign(const NearCopy& q, const NearCopy& c, const float* Xq, const int32_t* q_rows, const float* Xc, int d,
                       const NearBuffers& b, unsigned long long* best_at, int32_t* out_idx, float* out_dist, hipStream_t s);
// The queries of a connection round (1-NN among the rows of other colours, all of one matrix).  A component needs its
// lightest outgoing edge only, so after one pass that leaves every query an interval for its distance, the component's
// threshold falls to the smallest upper end of its queries, and only the queries whose lower end does not exceed it are
// searched for and evaluated.  The others answer the row that their upper end belongs to.
struct NearLink {
    const float* X; int d, n_rows;
    const int32_t* rows; int n;            // the queries
    const int32_t* colour;                 // [n_rows]
    uint32_t* threshold;                   // [n_rows] by colour, float bits: known outgoing edges, lowered here
    int32_t* out_idx; float *out_dist, *out_low; int32_t* evaluated;     // [n]; out_low: the lower ends
    int32_t *rows_left, *slot_left; float* reach_left;         // [n] scratch
    // near_link_ordered: the queries' ascending positions in the order, and more scratch
    const int32_t* qpos;
    int32_t *pos_left, *counts_left, *edge_at; unsigned long long* best_at; uint32_t* threshold0;
};
hipError_t near_link(const NearLink& p, const NearCopy& q, const NearCopy& c, const NearBuffers& b, hipStream_t s);
// Searches in a row order whose tiles have bounding balls: a tile meets the tiles only that may hold what it looks for.
// Two float16 copies in that order: `local` relative to the centre of every tile's region (a run of tiles close together), for the
// pairs of one region, and `all` for the other pairs.
struct NearOrder {
    const float* gap; int tiles;           // lower bounds of the squared distances between the rows of two tiles
    const int32_t* perm; int rows;         // row of X behind a position (-1: none), positions in use
    const int32_t* region;                 // [tiles], -1: too short for its pairs to matter
    NearCopy all, local; NearScale* local_scale;
    float* ratios;                         // near_make_ordered: scale of `local` over that of `all`; squared norms of the rows as they
                                           // are over those relative to the common shift
    const int32_t* tile_colour;            // near_link_ordered: the colour all rows of a tile share, -1 where they differ
    unsigned long long* tile_steps;        // pairs of tiles multiplied are added here
};
// (tile_first: the tile whose centre a tile of the local copy is relative to, -1 where region is)
hipError_t near_make_ordered(const float* X, int n_src, int d, const NearOrder& o, const float* tile_c, const float* tile_r,
                             const int32_t* tile_first, const float* hn, const NearBuffers& b, hipStream_t s);
size_t near_ordered_batch_bytes(long long rows, int kk);
size_t near_least_ordered_batch_bytes(long long rows, int kk);
size_t near_linked_batch_bytes(long long rows);
hipError_t near_search_ordered(const NearProblem& p, const NearOrder& o, const NearBuffers& b, hipStream_t s);
hipError_t near_link_ordered(const NearLink& p, const NearOrder& o, const NearBuffers& b, hipStream_t s);
hipError_t near_search(const NearProblem& p, const NearCopy& q, const NearCopy& c, const NearBuffers& b, hipStream_t s);

}  // namespace slhc
