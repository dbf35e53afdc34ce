// Launch interface of the searches that evaluate every pair (direct_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace slhc {

// Nearest row of Xc (nc rows) for m queries: rows of Xq (q_rows: which, nullptr: 0 .. m-1; entries outside [0, nq_rows) answer
// "nothing"); colours (optional, by row; Xq and Xc are one matrix then): only candidates of another colour.
// keys: m words of scratch.
bool direct_1nn_wanted(long long m, long long nc, int d);
bool direct_1nn_alone(long long m, long long nc, int d);
hipError_t direct_1nn(const float* Xq, int m, int nq_rows, const int32_t* q_rows, const float* Xc, int nc, int d, const int32_t* colour,
                      int32_t* out_idx, float* out_dist, unsigned long long* keys, hipStream_t s);

// The k nearest other rows of every row, in one launch.  pairs (optional): what is evaluated is added; nonfinite (optional): set where a row is not finite.
// direct_knn_wanted: rows per workgroup where it is what searches, else 0 (waited_for: the caller waits for the lists).
int direct_knn_wanted(long long n, int d, int k, bool waited_for);
hipError_t direct_knn(const float* X, int n, int d, int k, int rows, int32_t* out_idx, float* out_dist, unsigned long long* pairs, unsigned int* nonfinite, hipStream_t s);

// As direct_1nn, by blocks of pairs in registers: in one launch where the queries alone occupy the chip; pairs (optional): what is evaluated is added.
bool direct_near_wanted(long long m, long long nc, int d);
hipError_t direct_near(const float* Xq, int m, int nq_rows, const int32_t* q_rows, const float* Xc, int nc, int d, const int32_t* colour,
                       int32_t* out_idx, float* out_dist, unsigned long long* keys, unsigned long long* pairs, hipStream_t s);

}  // namespace slhc
