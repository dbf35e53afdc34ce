// Launch interface of the searches that evaluate every pair (direct_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace slhc {

// Nearest row of Xc (nc rows) for m queries: rows of Xq (q_rows: which, nullptr: 0 .. m-1; entries outside [0, nq_rows) answer
// "nothing"); colours (optional, by row; Xq and Xc are one matrix then): only candidates of another colour.
// keys: m words of scratch.
bool direct_1nn_wanted(long long m, long long nc, int d);
hipError_t direct_1nn(const float* Xq, int m, int nq_rows, const int32_t* q_rows, const float* Xc, int nc, int d, const int32_t* colour,
                      int32_t* out_idx, float* out_dist, unsigned long long* keys, hipStream_t s);

}  // namespace slhc
